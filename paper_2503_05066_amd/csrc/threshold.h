// The threshold of a block's keys: a header of its own, because tests also compile it for the host, as a block of one thread.
#pragma once

#include <stdint.h>

namespace capmoe {

template <int NT>
__device__ inline int block_exclusive_scan(int v, int* red, int* total);  // of the block's NT threads (drop.hip)

// The rem-th largest of the non-zero keys, which lie in [lo, hi]: kept are the keys above the threshold that is returned, and the
// first `rem` (as it is left) of those equal to it.  Each step spreads what is left of the range over BINS bins, finds the bin
// with that key and goes on inside it; it ends when the bin is one key wide or all of it is kept (no key equal to the threshold is, then).
// It ends after four steps at most whatever the keys are: with fewer than `rem` of them (a list that names an expert twice) all are kept.
// The bins divide the range in which the keys lie: gating scores share a few exponents, and counted by fixed digits, most lanes of
// a wave meet in one counter (us against four passes of eight bits: 64 segments of 65536 drawn ranks 34 -> 25, the whole drop by score
// 90 -> 65; 1024 segments of 2048 keys 12.3 -> 9.3; the whole drop of 4096 tokens, 64 experts, all scores equal 30 -> 15).
// walk(f) calls f(key) for every key of the calling thread; hist: BINS words of LDS, zero; sh: three.  Called by the whole block after a barrier.
template <int NT>
constexpr int kSelectBins = NT >= 1024 ? 2048 : 1024;
template <int NT, int BINS = kSelectBins<NT>, class Walk>
__device__ __forceinline__ uint32_t select_threshold(uint32_t lo, uint32_t hi, int& rem, int* hist, int* red, int* sh, Walk&& walk) {
    constexpr int kPer = BINS / NT;
    const int tid = threadIdx.x;
    for (;;) {
        if (lo >= hi) return lo;  // one key is left (or there is none at all)
        const uint32_t range = hi - lo;
        const int width = 32 - __clz(range), shift = width > __builtin_ctz(BINS) ? width - __builtin_ctz(BINS) : 0;
        walk([&](uint32_t key) __attribute__((always_inline)) {
            if (key - lo <= range) atomicAdd(&hist[(key - lo) >> shift], 1);  // (below lo wraps around; key 0 is below)
        });
        __syncthreads();
        if (tid == 0) sh[0] = sh[1] = sh[2] = 0;  // what holds if there are fewer keys than that: no bin is cut (the scan's barriers order it)
        // thread i owns the bins from BINS - 1 - kPer * i downwards: a scan over the threads counts the keys of higher bins
        int h[kPer], sum = 0, total;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            h[j] = hist[BINS - 1 - (tid * kPer + j)];
            sum += h[j];
        }
        int above = block_exclusive_scan<NT>(sum, red, &total);
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            if (above < rem && above + h[j] >= rem) {  // exactly one bin of one thread
                sh[0] = BINS - 1 - (tid * kPer + j);
                sh[1] = rem - above;
                sh[2] = h[j];
            }
            above += h[j];
            hist[BINS - 1 - (tid * kPer + j)] = 0;
        }
        __syncthreads();
        lo += (uint32_t)sh[0] << shift;
        rem = sh[1];
        if (sh[2] == rem) {  // all of the bin is kept, or all that there is
            rem = 0;
            return lo - 1u;
        }
        if (shift == 0) return lo;
        const uint32_t rest = (1u << shift) - 1u;
        if (hi - lo > rest) hi = lo + rest;  // (lo + rest itself may lie past the largest word)
    }
}

}  // namespace capmoe
