"""The threshold search of the drop (csrc/threshold.h) compiled for the host, as a block of one thread, against a sort."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="g++ is needed")

HARNESS = r"""
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <vector>
#define __device__
#define __forceinline__ inline
#define __clz __builtin_clz
static struct { int x; } threadIdx;
static std::vector<int> counters;
static void __syncthreads() {}
static void atomicAdd(int* at, int v) {
    if (at < counters.data() || at >= counters.data() + counters.size()) { puts("outside the counters"); exit(3); }
    *at += v;
}
#include "threshold.h"
namespace capmoe {
template <int NT>
inline int block_exclusive_scan(int v, int*, int* total) { *total = v; return 0; }
}
template <int BINS>
static void run(std::vector<uint32_t>& keys, int rem) {
    uint32_t lo = 0xffffffffu, hi = 0u;
    for (uint32_t k : keys)
        if (k) { lo = k < lo ? k : lo; hi = k > hi ? k : hi; }
    counters.assign(BINS, 0);
    int sh[3] = {BINS - 1, 1, 2};  // what LDS held before
    uint32_t tau = capmoe::select_threshold<1, BINS>(lo, hi, rem, counters.data(), nullptr, sh, [&](auto&& f) { for (uint32_t k : keys) f(k); });
    printf("%u %d\n", tau, rem);
}
int main() {
    int bins, rem, n;
    while (scanf("%d %d %d", &bins, &rem, &n) == 3) {
        std::vector<uint32_t> keys(n);
        for (auto& k : keys)
            if (scanf("%u", &k) != 1) return 2;
        if (bins == 1024) run<1024>(keys, rem); else run<2048>(keys, rem);
    }
}
"""


@pytest.fixture(scope="module")
def search(tmp_path_factory):
    folder = tmp_path_factory.mktemp("threshold")
    (folder / "main.cpp").write_text(HARNESS)
    subprocess.run(["g++", "-O1", "-std=c++17", "-w", "-I", os.path.join(ROOT, "paper_2503_05066_amd", "csrc"), "-o",
                    str(folder / "main"), str(folder / "main.cpp")], check=True)

    def call(keys, cap, bins):
        text = f"{bins} {cap} {len(keys)} " + " ".join(str(int(k)) for k in keys)
        r = subprocess.run([str(folder / "main")], input=text, capture_output=True, text=True, timeout=20)
        assert r.returncode == 0, r.stdout
        return [int(v) for v in r.stdout.split()]

    return call


def _kept(keys, tau, rem):
    """What the compaction keeps: keys above the threshold, and the first `rem` of those equal to it."""
    equal = keys == tau
    return (keys != 0) & ((keys > tau) | (equal & (np.cumsum(equal) <= rem)))


def _check(search, keys, cap):
    keys = np.asarray(keys, np.uint32)
    want = np.zeros(len(keys), bool)
    want[np.lexsort((np.arange(len(keys)), -keys.astype(np.int64)))[:cap]] = True
    want &= keys != 0
    for bins in (1024, 2048):
        np.testing.assert_array_equal(_kept(keys, *search(keys, cap, bins)), want, err_msg=f"{bins} bins, capacity {cap}")


@pytest.mark.parametrize("low,high", [(1, 1), (1, 2), (5, 1028), (5, 1029), (0x3d000001, 0x3d000801), (1, 0x3f800001), (1, 0xff800001),
                                      (0x80000001, 0xff800001), (1, 0xffffffff), (0xfffffc00, 0xffffffff), (0xff000000, 0xffffffff)])
def test_threshold_of_ranges(search, low, high):
    rng = np.random.default_rng(low ^ high)
    keys = rng.integers(low, high, 300, endpoint=True, dtype=np.uint32)
    keys[:2] = low, high
    keys[rng.random(300) < 0.3] = 0                       # pairs that are no candidates
    keys[rng.random(300) < 0.2] = keys[keys > 0][0]       # and equal ones
    for cap in (1, 2, 8, 50, int((keys > 0).sum()) - 1):
        _check(search, keys, cap)


@pytest.mark.parametrize("top", [0xff800001, 0xffc00001, 0xffe00001, 0xffffffff])
def test_threshold_in_the_last_bin_of_the_word(search, top):
    """The wanted key in a bin whose end lies past the largest word (scores that are not a number, in a high class)."""
    rng = np.random.default_rng(top)
    keys = np.concatenate([np.full(20, top), np.ones(5), rng.integers(1, 0x3f800002, 30), np.zeros(200)]).astype(np.uint32)
    rng.shuffle(keys)
    for cap in (1, 8, 19, 20, 21, 52):
        _check(search, keys, cap)


@pytest.mark.parametrize("keys", [[0, 0, 0], [5], [7, 0, 7, 7], [1, 0, 0x3f800001], [0xffffffff, 3, 0, 9, 9],
                                  list(range(0x3d000001, 0x3d000001 + 50 * 4096, 4096))])
def test_fewer_keys_than_the_capacity(search, keys):
    """Lists that name an expert twice count more candidates than there are keys: the search ends, and keeps them all."""
    keys = np.asarray(keys, np.uint32)
    for more in (1, 2, 1000):
        _check(search, keys, int((keys > 0).sum()) + more)
