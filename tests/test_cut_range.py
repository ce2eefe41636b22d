"""The counting rounds that find the cut of a selection (csrc/cut_range.h) replayed on the host: the integer ranges the kernels
narrow must hold exactly the keys of the bin that was counted, up to the largest key there is (NaN scores sit there)."""
import os
import subprocess

import numpy as np
import pytest

from paper_2604_10235_amd import build

# Reads keys (0: no candidate, 0xFFFFFFFF: admitted whatever the cut) and a rank; prints the rank-th largest competing key and its
# rank among equals; exits with 1 where the narrowed range and the counted bin hold different numbers of keys.
REPLAY = r"""
#include <cstdio>
#include <vector>
#include "cut_range.h"
using namespace codecomp;
int main(int, char** argv) {
  std::FILE* f = std::fopen(argv[1], "rb");
  std::vector<uint32_t> keys(1 << 20);
  keys.resize(std::fread(keys.data(), 4, keys.size(), f));
  uint32_t rank = keys.back(), lo = 0xFFFFFFFFu, hi = 0;
  keys.pop_back();
  for (uint32_t k : keys) if (k != 0 && k != 0xFFFFFFFFu) { if (k < lo) lo = k; if (k > hi) hi = k; }
  for (;;) {
    const uint32_t width = hi - lo;
    const int shift = cut_shift(width);
    std::vector<uint32_t> bins(kCutBins);
    for (uint32_t k : keys) if (k - lo <= width) ++bins.at((k - lo) >> shift);
    int bin = kCutBins - 1;
    while (bin > 0 && rank > bins[bin]) rank -= bins[bin--];
    cut_narrow(lo, hi, (uint32_t)bin, shift);
    uint32_t in = 0;
    for (uint32_t k : keys) in += k - lo <= hi - lo;
    if (in != bins[bin]) return 1;
    if (shift == 0) { std::printf("%u %u\n", lo, rank); return 0; }
  }
}
"""


@pytest.fixture(scope="module")
def replay(tmp_path_factory):
    d = tmp_path_factory.mktemp("cut")
    src, exe = d / "replay.cpp", d / "replay"
    src.write_text(REPLAY)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(build.ROCM, "include"), "-I", build.CSRC,
                    str(src), "-o", str(exe)], check=True)

    def run(keys, rank):
        np.append(keys, np.uint32(rank)).astype(np.uint32).tofile(d / "keys")
        return tuple(int(x) for x in subprocess.run([str(exe), str(d / "keys")], check=True, capture_output=True, text=True).stdout.split())
    return run


def order_keys(x):
    u = np.asarray(x, np.float32).view(np.uint32)
    return np.clip(np.where(u >> 31 == 1, ~u, u | 0x80000000), 1, 0xFFFFFFFE).astype(np.uint32)


def patterns():
    g = np.random.default_rng(5)
    scores = g.uniform(0.2, 1.2, 5000).astype(np.float32)
    nans = scores.copy(); nans.view(np.uint32)[[10, 400, 4999]] = 0x7FFFFFFF
    yield "three of the largest NaN above ordinary scores", order_keys(nans), (1, 2, 3, 4, 2500, 5000)
    nans = g.standard_normal(3000).astype(np.float32); nans.view(np.uint32)[:700] = g.integers(0x7F800001, 0x80000000, 700)
    nans.view(np.uint32)[700:900] = g.integers(0xFF800001, 0x100000000, 200)
    yield "NaN of both signs and all payloads", order_keys(nans), (1, 3, 699, 700, 701, 2800, 3000)
    for top in (0xFFFFFFFE, 0xFFFFFFFD, 0xFFF00000):
        for low in (1, 2, 0x7FFFFFFF, 0xBF000000, top - 2047, top - 2048, top - 4096):
            keys = np.concatenate([[top, low], g.integers(low, top + 1, 500)])
            yield f"from {low:#x} to {top:#x}", keys, (1, 2, 250, 502)
    yield "one key only", np.full(300, 0xFFFFFFFE), (1, 300)
    yield "scores and a zero", order_keys(np.append(scores, 0.0)), (1, 500, 5001)


@pytest.mark.parametrize("keys,ranks", [pytest.param(k, r, id=name) for name, k, r in patterns()])
def test_narrowed_ranges_hold_the_keys_that_were_counted(replay, keys, ranks):
    keys = np.asarray(keys, np.uint32)
    order = np.sort(keys)[::-1]
    for unused in (np.zeros(100, np.uint32), np.full(7, 0xFFFFFFFF, np.uint32)):       # slots past the row, protected tokens
        for rank in ranks:
            tau, ties = replay(np.concatenate([keys, unused]), rank)
            assert tau == order[rank - 1] and ties == rank - int((keys > tau).sum())
