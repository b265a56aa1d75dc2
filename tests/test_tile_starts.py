"""The binning's tile starts past 2^32 instances, on the CPU: the header's
arithmetic compiled for the host and run as a workgroup's threads run it (a
slice of tiles each), against Python's integers."""
import os
import subprocess

import numpy as np
import pytest

from paper_2505_19175_amd import build

PROBE = r"""
#include "tile_starts.h"
#include <stdio.h>
#include <vector>
// stdin: T capacity, then per tile its count and the instances before a group's
int main(void) {
  unsigned T, cap;
  if (scanf("%u %u", &T, &cap) != 2) return 1;
  std::vector<uint32_t> s(T), before(T);
  for (unsigned t = 0; t < T; ++t)
    if (scanf("%u %u", &s[t], &before[t]) != 2) return 1;
  const int per = (T + 1023) / 1024;
  uint32_t M = 0;
  for (int tid = 0; tid < 1024; ++tid) {
    const int t0 = tid * per < (int)T ? tid * per : T, t1 = t0 + per < (int)T ? t0 + per : T;
    const uint32_t sum = ts::slice_sum(s.data(), t0, t1);
    ts::slice_starts(s.data(), t0, t1, M);
    M = ts::add_sat(M, sum);
  }
  printf("%u\n", M);
  for (unsigned t = 0; t < T; ++t) {
    const uint2 r = ts::clamp_run(s[t], t + 1 < T ? s[t + 1] : M, cap);
    printf("%u %u %u\n", r.x, r.y, ts::first_slot(s[t], before[t], cap));
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    d = tmp_path_factory.mktemp("tile_starts")
    src, exe = str(d / "probe.hip"), str(d / "probe")
    open(src, "w").write(PROBE)
    subprocess.check_call([build.HIPCC, "-x", "hip", "--offload-host-only", "-O1", "-std=c++17",
                           "-I", build.CSRC, "-I", build.INCLUDE, src, "-o", exe])
    return exe


# 3M triangles of 1500 tiles each; one of whole tiles 2048 of which are 2^32
# instances (the 2049th start is 0 in 32 bits); the last start just below, at and
# past 2^32; few instances; capacities from one slot to the most a list has
@pytest.mark.parametrize("counts", [
    np.full(3600, 1_250_000), np.full(3600, 1 << 21), np.full(12288, 0xffffffff),
    np.array([0xfffffffe, 5]), np.array([0xffffffff, 5, 7]), np.array([0xffffffff, 1, 0, 3]),
    np.array([3, 0, 0, 7, 1]), np.zeros(40)], ids=lambda c: f"{len(c)}x{int(c[0])}")
@pytest.mark.parametrize("cap", [1, 9, 12_000_000, 0xffffffff - 1024])
def test_runs_and_cursors(probe, counts, cap):
    counts = [int(c) for c in counts]
    rng = np.random.default_rng(cap % 1000)
    before = [int(x * c) for x, c in zip(rng.random(len(counts)), counts)]
    text = f"{len(counts)} {cap}\n" + "\n".join(f"{c} {b}" for c, b in zip(counts, before))
    out = subprocess.run([probe], input=text, capture_output=True, text=True, check=True).stdout
    got = np.array(out.split(), np.uint64)
    start, want = 0, [min(sum(counts), 0xffffffff)]
    for c, b in zip(counts, before):
        x, y = min(start, cap), min(start + c, cap)
        want += [x, y, min(start + b, cap)] if x != y else [0, 0, min(start + b, cap)]
        start += c
    assert got.tolist() == want
