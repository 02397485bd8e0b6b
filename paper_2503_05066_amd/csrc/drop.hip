// Capacity enforcement: Token Drop (Eqs. 8-10, Alg. 1) and Expanded Drop (Alg. 2).
//
// Three kernels, all integer work on score bit patterns (scores are >= +0, so the unsigned
// order of the bits is the order of the values):
//   1. drop_prepare   per token: candidate set (top-k, plus the experts of the token's own device
//                     for Expanded Drop) -> key = rank + 1 for candidates, 0 otherwise, written
//                     expert-major so that a capacity segment is one contiguous run.  The rank is
//                     the score's bit pattern (Score metric), the token's position (Order, Reverse
//                     Order) or a hashed draw (Random), below an optional 2-bit token class.
//   2. drop_select    per segment: the cap-th largest key by histograms in LDS of the range
//                     the keys lie in (the threshold tau of Eq. 8) and how many keys equal to it survive
//                     (drop_big_*: the same for segments that many blocks share; which form: select_form).
//   3. drop_emit      per segment (a block per 4096 tokens of it): ordered compaction of the survivors,
//                     which yields rows in ascending token order and gives ties at the threshold to
//                     the lower token index.
// Every kernel first pulls what it needs from global memory in one batch of independent loads
// (these kernels are latency-bound: a dependent load per loop iteration costs a microsecond each).
// Small problems with per-expert capacities run all three steps in one launch (drop_fused, below),
// the optional per-token limit adds a fourth kernel and a second emit.
#include <type_traits>

#include "common.h"
#include "schedule.h"
#include "threshold.h"

namespace capmoe {

constexpr int kPrepTokens = 16;  // tokens per block: small, the kernel is latency-bound and wants every CU

// The draw of MOE_METRIC_RANDOM: a 32-bit integer hash (two multiply-xorshift rounds) of the pair's
// counter, offset by the seed; the header states the same formula.
__device__ inline uint32_t pair_hash(uint32_t seed, uint32_t counter) {
    uint32_t x = counter + seed * 0x9E3779B9u;
    x ^= x >> 16;
    x *= 0x7FEB352Du;
    x ^= x >> 15;
    x *= 0x846CA68Bu;
    x ^= x >> 16;
    return x;
}

// A pair's rank within its class, below 2^30: score bits (scores are in [0,1]), position in the segment, or a draw.
template <class ScoreBits>
__device__ __forceinline__ uint32_t pair_rank(int metric, int local, int seg_tokens, uint32_t seed, uint32_t pair, ScoreBits&& score_bits) {
    if (metric == MOE_METRIC_ORDER) return (uint32_t)(seg_tokens - 1 - local);
    if (metric == MOE_METRIC_REVERSE_ORDER) return (uint32_t)local;
    if (metric == MOE_METRIC_RANDOM) return pair_hash(seed, pair) >> 3;
    return score_bits();
}

// Expanded Drop, in the one-launch kernels: the tokens of capacity block `block` that sit on the device of expert `e` (all of them have it as
// a candidate), and the experts of a token's device (from g0 on) with a lower id than e (candidates below it, listed or not).
__device__ __forceinline__ int tokens_on_device(int e, int block, int group_experts, int group_tokens, int seg_tokens) {
    const int lo = e / group_experts * group_tokens, hi = lo + group_tokens;
    const int s0 = block * seg_tokens, s1 = s0 + seg_tokens;
    const int a = lo > s0 ? lo : s0, z = hi < s1 ? hi : s1;
    return z > a ? z - a : 0;
}
__device__ __forceinline__ int device_experts_below(int e, int g0, int group_experts) {
    const int lower = e - g0;
    return lower < 0 ? 0 : (lower > group_experts ? group_experts : lower);
}

// ---------------------------------------------------------------------------------------------
// 1. candidate keys, transposed
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void drop_prepare_kernel(const float* __restrict__ scores,
                                                           const int32_t* __restrict__ topk_idx,
                                                           uint32_t* __restrict__ key_t, uint8_t* __restrict__ slot_t,
                                                           int32_t* __restrict__ pair_row, int N, int E, int k, int S,
                                                           int expanded, int group_tokens, int group_experts,
                                                           int metric, int seg_tokens,
                                                           const uint8_t* __restrict__ token_class, uint32_t seed,
                                                           uint32_t* __restrict__ clear, long long clear_words,
                                                           int32_t* __restrict__ clear_count,
                                                           int32_t* __restrict__ clear_need, int segs) {
    // what the launches that share segments among blocks add to (clear_count == nullptr: there are none)
    if (clear_count) {
        for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < clear_words; i += (long long)gridDim.x * 256)
            clear[i] = 0u;
        for (int i = blockIdx.x * 256 + threadIdx.x; i < segs; i += gridDim.x * 256) clear_count[i] = clear_need[i] = 0;
    }
    extern __shared__ uint32_t lds[];
    const int ld = E | 1;                                  // odd row pitch: conflict-free transposed reads
    uint32_t* key_s = lds;                                 // [kPrepTokens][ld] score bits, then keys
    uint8_t* slot_s = (uint8_t*)(lds + kPrepTokens * ld);  // [kPrepTokens][ld] candidate flags, then slots
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int t0 = blockIdx.x * kPrepTokens;
    const int nt = N - t0 < kPrepTokens ? N - t0 : kPrepTokens;  // tokens of this block

    for (int i = tid; i < kPrepTokens * ld; i += 256) slot_s[i] = 0;
    // the block's scores are one contiguous run of nt*E floats
    for (int i = tid; i < nt * E; i += 256) {
        const int tl = i / E, e = i - tl * E;
        key_s[tl * ld + e] = __float_as_uint(scores[(size_t)t0 * E + i]);
    }
    __syncthreads();
    for (int i = tid; i < nt * k; i += 256) slot_s[(i / k) * ld + topk_idx[(size_t)t0 * k + i]] = 1;
    if (expanded) {
        for (int i = tid; i < nt * group_experts; i += 256) {
            const int tl = i / group_experts, j = i - tl * group_experts;
            slot_s[tl * ld + ((t0 + tl) / group_tokens) * group_experts + j] = 1;
        }
    }
    __syncthreads();
    // flags -> keys and slots (slot = number of candidate experts with a lower id); a wave walks its tokens
    constexpr int kWalk = kPrepTokens / 4;
    for (int i = 0; i < kWalk; ++i) {
        const int tl = wv * kWalk + i, t = t0 + tl;
        if (tl >= nt) break;
        int base = 0;
        const uint32_t cls = token_class ? (uint32_t)(token_class[t] & 3) << 30 : 0u;
        const int local = t % seg_tokens;  // position inside the capacity segment
        for (int e0 = 0; e0 < E; e0 += kWave) {
            const int e = e0 + lane;
            const bool c = e < E && slot_s[tl * ld + e] != 0;
            const uint64_t mask = __ballot(c);
            if (e < E) {
                const uint32_t rank = pair_rank(metric, local, seg_tokens, seed, (uint32_t)t * (uint32_t)E + (uint32_t)e,
                                                [&] { return key_s[tl * ld + e]; });
                key_s[tl * ld + e] = c ? cls + rank + 1u : 0u;
                slot_s[tl * ld + e] = (uint8_t)(base + __popcll(mask & ((1ull << lane) - 1ull)));
            }
            base += __popcll(mask);
        }
        // slots beyond the token's candidate count stay unused
        for (int s = base + lane; s < S; s += kWave) pair_row[(size_t)t * S + s] = -1;
    }
    __syncthreads();
    // transposed write: a wave writes the block's consecutive tokens of 64 / kPrepTokens experts at a time
    constexpr int kRows = kWave / kPrepTokens;
    const int tl = lane % kPrepTokens;
    for (int e = wv * kRows + lane / kPrepTokens; e < E; e += 4 * kRows) {
        if (tl < nt) {
            key_t[(size_t)e * N + t0 + tl] = key_s[tl * ld + e];
            slot_t[(size_t)e * N + t0 + tl] = slot_s[tl * ld + e];
        }
    }
}

// ---------------------------------------------------------------------------------------------
// block-wide helpers (NT threads, a multiple of the wave width)
// ---------------------------------------------------------------------------------------------
template <int NT>
__device__ inline int block_sum(int v, int* red) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int w = 0; w < NT / kWave; ++w) total += red[w];
    return total;
}
__device__ inline int block_sum_256(int v, int* red) { return block_sum<256>(v, red); }

// exclusive prefix sum of v over the block's threads; *total gets the block sum
template <int NT>
__device__ inline int block_exclusive_scan(int v, int* red, int* total) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int incl = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const int o = __shfl_up(incl, off, kWave);
        if (lane >= off) incl += o;
    }
    __syncthreads();
    if (lane == 63) red[wv] = incl;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < NT / kWave; ++w) {
        if (w < wv) before += red[w];
        all += red[w];
    }
    *total = all;
    return before + incl - v;
}
__device__ inline int block_exclusive_scan_256(int v, int* red, int* total) {
    return block_exclusive_scan<256>(v, red, total);
}

// f(0), f(1), .. f(N - 1) with compile-time arguments
template <int N, class F, int I = 0>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, F, I + 1>(static_cast<F&&>(f));
    }
}

// minimum and maximum of the block's candidate keys and their number, for all threads (lo > hi without any)
template <int NT>
__device__ __forceinline__ void key_extent(uint32_t& lo, uint32_t& hi, int& count, uint32_t (*red)[3]) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const uint32_t a = __shfl_xor(lo, off, kWave), b = __shfl_xor(hi, off, kWave);
        lo = a < lo ? a : lo;
        hi = b > hi ? b : hi;
        count += __shfl_xor(count, off, kWave);
    }
    if ((threadIdx.x & 63) == 0) {
        red[threadIdx.x >> 6][0] = lo;
        red[threadIdx.x >> 6][1] = hi;
        red[threadIdx.x >> 6][2] = (uint32_t)count;
    }
    __syncthreads();
    count = 0;
#pragma unroll
    for (int w = 0; w < NT / kWave; ++w) {
        lo = red[w][0] < lo ? red[w][0] : lo;
        hi = red[w][1] > hi ? red[w][1] : hi;
        count += (int)red[w][2];
    }
}

// ---------------------------------------------------------------------------------------------
// 2. threshold per segment
// ---------------------------------------------------------------------------------------------
// One block per capacity segment: `span` experts (1, or the E/G experts of a device when the
// capacity is a device budget) over seg_tokens tokens.  The keys of expert e0+r form run r.
// Outputs, per (block, expert): the threshold, how many keys equal to it survive, the kept count.
// Several experts under one budget share the threshold; the keys equal to it are granted to the
// lower tokens first and, inside a token, to the lower expert ids.
// NT threads: 256 for short segments, 1024 for long ones (a segment is one block's work, and its
// passes over the keys are chains of load latencies that only more loads in flight shorten).
// VEC keys per load: 4 when every run starts on a 16-byte boundary (N and seg_tokens multiples of 4).
// The threads keep the segment's keys in registers, VEC * BATCH each, and only the first pass loads
// them (from L2 or LDS in every pass: 65536 keys of 8192 tokens x 8 experts 43 -> 34 us, 3000 tokens 9.5 -> 6.9).
// Longer segments: see select_form.
// HELD == false: longer segments, read from L2 in every pass, BATCH loads at a time.
template <int NT, int VEC, int BATCH, bool HELD>
__global__ __launch_bounds__(NT) void drop_select_kernel(const uint32_t* __restrict__ key_t,
                                                          uint32_t* __restrict__ seg_tau,
                                                          int32_t* __restrict__ seg_need,
                                                          int32_t* __restrict__ seg_count, int N, int E, int seg_tokens,
                                                          int span, int cap) {
    __shared__ int hist[kSelectBins<NT>];
    __shared__ int gt_s[kMaxExperts], eq_s[kMaxExperts];
    __shared__ int red[NT / kWave], sh_bin[3];
    __shared__ uint32_t extent[NT / kWave][3];
    const int groups = E / span;
    const int b = blockIdx.x / groups, e0 = (blockIdx.x - b * groups) * span;
    const uint32_t* keys = key_t + (size_t)e0 * N + (size_t)b * seg_tokens;  // run r starts at keys + r*N
    const int tid = threadIdx.x;
    const int n_keys = span * seg_tokens;
    if (cap == 0) {  // nothing passes
        for (int r = tid; r < span; r += NT) {
            seg_tau[b * E + e0 + r] = 0xffffffffu;
            seg_need[b * E + e0 + r] = seg_count[b * E + e0 + r] = 0;
        }
        return;
    }

    // Every pass walks all keys of the segment, key i = run i / seg_tokens, token i % seg_tokens, and calls
    // f(run, token, key) key by key, in ascending i per thread.
    struct alignas(4 * VEC) KeyVec {
        uint32_t c[VEC];
    };
    // VEC divides seg_tokens: the keys of a load share a run
    auto run_of = [&](int i) __attribute__((always_inline)) { return span == 1 ? 0 : i / seg_tokens; };
    // no branch, so that all loads are under way together; past the end: key 0, not used
    auto load = [&](int i) __attribute__((always_inline)) {
        const int run = run_of(i);
        return *(const KeyVec*)(keys + (i < n_keys ? (size_t)run * N + (i - run * seg_tokens) : 0));
    };
    KeyVec held[BATCH];
    auto load_batch = [&](int i0) __attribute__((always_inline)) {
        static_for<BATCH>([&](auto uc) __attribute__((always_inline)) {
            held[decltype(uc)::value] = load(i0 + NT * VEC * decltype(uc)::value);
        });
    };
    auto walk_batch = [&](int i0, auto&& f) __attribute__((always_inline)) {
        static_for<BATCH>([&](auto uc) __attribute__((always_inline)) {
            constexpr int u = decltype(uc)::value;
            const int i = i0 + NT * VEC * u, run = run_of(i);
            if (i < n_keys)
                static_for<VEC>([&](auto cc) __attribute__((always_inline)) {
                    constexpr int c = decltype(cc)::value;
                    f(run, i - run * seg_tokens + c, held[u].c[c]);
                });
        });
    };
    if (HELD) load_batch(tid * VEC);
    auto for_each_key = [&](auto&& f) __attribute__((always_inline)) {
        if (HELD) {
            walk_batch(tid * VEC, f);
        } else {
            for (int i0 = tid * VEC; i0 < n_keys; i0 += NT * VEC * BATCH) {
                load_batch(i0);
                walk_batch(i0, f);
            }
        }
    };

    for (int i = tid; i < kSelectBins<NT>; i += NT) hist[i] = 0;
    for (int r = tid; r < span; r += NT) gt_s[r] = eq_s[r] = 0;
    uint32_t lo = 0xffffffffu, hi = 0u;
    int n_cand = 0;
    for_each_key([&](int, int, uint32_t key) {
        if (key != 0u) {  // non-candidates (key 0) never matter
            ++n_cand;
            lo = key < lo ? key : lo;
            hi = key > hi ? key : hi;
        }
    });
    key_extent<NT>(lo, hi, n_cand, extent);  // its barrier also orders the LDS writes before the reads

    // threshold: keys above tau are kept, `rem` of the keys equal to tau are kept
    uint32_t tau = 0;  // every candidate (key >= 1) passes
    int rem = 0;
    if (n_cand > cap) {
        rem = cap;
        tau = select_threshold<NT>(lo, hi, rem, hist, red, sh_bin,
                                   [&](auto&& f) __attribute__((always_inline)) { for_each_key([&](int, int, uint32_t key) { f(key); }); });
    }
    if (span == 1) {  // one expert: the counts follow from the selection itself
        if (tid == 0) {
            const int seg = b * E + e0;
            seg_tau[seg] = tau;
            seg_need[seg] = rem;
            seg_count[seg] = n_cand > cap ? cap : n_cand;
        }
        return;
    }
    // per expert: keys above the threshold and keys equal to it (a thread's keys change run rarely)
    auto count_runs = [&](int tie_token, int tie_run) __attribute__((always_inline)) {
        int run = -1, gt = 0, eq = 0;
        for_each_key([&](int r, int tl, uint32_t key) {
            if (r != run) {
                if (gt) atomicAdd(&gt_s[run], gt);
                if (eq) atomicAdd(&eq_s[run], eq);
                run = r;
                gt = eq = 0;
            }
            gt += key > tau;
            eq += key == tau && key != 0u && (tl < tie_token || (tl == tie_token && r <= tie_run));
        });
        if (gt) atomicAdd(&gt_s[run], gt);
        if (eq) atomicAdd(&eq_s[run], eq);
    };
    count_runs(seg_tokens, span);  // every key equal to the threshold
    __syncthreads();
    int eq_total = 0;
    for (int r = 0; r < span; ++r) eq_total += eq_s[r];
    if (rem > 0 && eq_total > rem) {
        // More keys equal the threshold than the budget has room for: they are granted in
        // (token, expert) order.  A thread owns a run of consecutive tokens; the thread in whose
        // run the budget ends finds the last granted pair (token tie_token, expert run tie_run).
        __shared__ int sh_tie_token, sh_tie_run;
        const int per = (seg_tokens + NT - 1) / NT;
        const int tb = tid * per < seg_tokens ? tid * per : seg_tokens;
        const int te = tb + per < seg_tokens ? tb + per : seg_tokens;
        auto key_at = [&](int r, int tl) { return keys[(size_t)r * N + tl]; };
        int c = 0;
        for (int tl = tb; tl < te; ++tl)
            for (int r = 0; r < span; ++r) c += key_at(r, tl) == tau;
        int total;
        const int before = block_exclusive_scan<NT>(c, red, &total);
        if (before < rem && rem <= before + c) {  // exactly one thread: 1 <= rem < eq_total = total
            int left = rem - before;
            for (int tl = tb; tl < te && left > 0; ++tl)
                for (int r = 0; r < span && left > 0; ++r)
                    if (key_at(r, tl) == tau && --left == 0) {
                        sh_tie_token = tl;
                        sh_tie_run = r;
                    }
        }
        __syncthreads();
        const int tie_token = sh_tie_token, tie_run = sh_tie_run;
        for (int r = tid; r < span; r += NT) gt_s[r] = eq_s[r] = 0;
        __syncthreads();
        count_runs(tie_token, tie_run);
        __syncthreads();
    }
    if (tid < span) {
        const int seg = b * E + e0 + tid;
        seg_tau[seg] = tau;
        const int granted = rem > 0 ? eq_s[tid] : 0;
        seg_need[seg] = granted;  // inside an expert the granted keys are its first ones in token order
        seg_count[seg] = gt_s[tid] + granted;
    }
}

// ---------------------------------------------------------------------------------------------
// 2b. threshold of segments that one block would walk for long
// ---------------------------------------------------------------------------------------------
// A device budget makes one segment of all keys of a device's experts, a million and more with a single device.  One block
// needs several passes over them, at one compute unit's bandwidth.  Here many
// blocks share a segment: three launches build the histograms of an 11, 11 and 10 bit digit (every block first picks the
// digit before it from the histogram of the launch before), one counts per expert, one small one settles ties.  Integer
// atomics throughout: the same numbers run to run.  Which segments come here: select_form.
constexpr int kBigChunk = 8192;   // keys (or tokens of a run) of a block
constexpr int kBigBins = 2048;    // of a level
struct BigState {                 // of a segment; cleared by drop_prepare_kernel
    uint32_t hist[3][kBigBins];
    uint32_t prefix[2];           // digits picked after the first and the second level
    int32_t rem[3];               // keys of the prefix still to keep; after the last level: of the threshold
    int32_t eq_total;             // keys equal to the threshold
    int32_t pad[2];
};
constexpr int kBigPiece = 1024;   // tokens of an entry in the table of equal keys, see drop_big_count_kernel
static int big_pieces(int seg_tokens) { return (seg_tokens + kBigPiece - 1) / kBigPiece; }
static_assert(sizeof(BigState) % 16 == 0, "whole words");

// The digit of `hist` in which the rem-th key from above lies, for the whole block of 256 threads: *digit, and in *left how
// many of that digit's keys are kept.  All counts together are *total; with fewer than rem keys *digit stays -1.
__device__ inline void pick_digit(const uint32_t* hist, int rem, int* digit, int* left, int* total, int* red) {
    __shared__ int sh_digit, sh_left;
    constexpr int kPer = kBigBins / 256;
    if (threadIdx.x == 0) sh_digit = -1;
    int h[kPer], sum = 0;
#pragma unroll
    for (int j = 0; j < kPer; ++j) {  // thread i owns the digits from kBigBins - 1 - kPer * i downwards
        h[j] = (int)hist[kBigBins - 1 - (threadIdx.x * kPer + j)];
        sum += h[j];
    }
    int above = block_exclusive_scan_256(sum, red, total);  // its barriers order the reset before the writes
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        if (above < rem && above + h[j] >= rem) {  // one digit of one thread at most
            sh_digit = kBigBins - 1 - (threadIdx.x * kPer + j);
            sh_left = rem - above;
        }
        above += h[j];
    }
    __syncthreads();
    *digit = sh_digit;
    *left = sh_left;
    __syncthreads();
}

template <int VEC>
struct alignas(4 * VEC) BigVec {
    uint32_t c[VEC];
};

// LEVEL: digit counted here, 0 (bits 31-21), 1 (20-10) or 2 (9-0)
template <int LEVEL, int VEC>
__global__ __launch_bounds__(256) void drop_big_hist_kernel(const uint32_t* __restrict__ key_t, BigState* __restrict__ state,
                                                            int N, int E, int seg_tokens, int span, int cap, int chunks) {
    __shared__ int hist[kBigBins];
    __shared__ int red[4];
    const int ds = blockIdx.x / chunks, chunk = blockIdx.x - ds * chunks, groups = E / span;
    const int b = ds / groups, e0 = (ds - b * groups) * span, tid = threadIdx.x;
    const uint32_t* keys = key_t + (size_t)e0 * N + (size_t)b * seg_tokens;
    const long long n_keys = (long long)span * seg_tokens;
    BigState* st = state + ds;
    constexpr int kLoads = kBigChunk / 256 / VEC;
    BigVec<VEC> v[kLoads];
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {  // requested before the pick waits
        const long long i = (long long)chunk * kBigChunk + (tid + 256 * u) * VEC;
        const int run = (int)(i / seg_tokens);  // VEC divides seg_tokens: the keys of a load share a run
        if (i < n_keys) {
            v[u] = *(const BigVec<VEC>*)(keys + (size_t)run * N + (i - (long long)run * seg_tokens));
        } else {
#pragma unroll
            for (int c = 0; c < VEC; ++c) v[u].c[c] = 0u;
        }
    }
    for (int i = tid; i < kBigBins; i += 256) hist[i] = 0;
    uint32_t prefix = 0;
    if (LEVEL > 0) {
        int digit, left, total;
        const int rem = LEVEL == 1 ? cap : st->rem[0];
        if (LEVEL == 2 && rem == 0) return;  // every candidate passes: nothing to pick
        pick_digit(st->hist[LEVEL - 1], rem, &digit, &left, &total, red);
        if (LEVEL == 1 && total <= cap) return;  // rem stays 0
        prefix = LEVEL == 1 ? (uint32_t)digit << 21 : st->prefix[0] | ((uint32_t)digit << 10);
        if (chunk == 0 && tid == 0) {
            st->prefix[LEVEL - 1] = prefix;
            st->rem[LEVEL - 1] = left;
        }
    }
    __syncthreads();
    constexpr uint32_t kMask = LEVEL == 0 ? 0u : (LEVEL == 1 ? 0xffe00000u : 0xfffffc00u);
    constexpr int kShift = LEVEL == 0 ? 21 : (LEVEL == 1 ? 10 : 0);
#pragma unroll
    for (int u = 0; u < kLoads; ++u)
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
            const uint32_t key = v[u].c[c];  // non-candidates (key 0) never matter
            if (key != 0u && (key & kMask) == prefix) atomicAdd(&hist[(key >> kShift) & (LEVEL == 2 ? 1023u : 2047u)], 1);
        }
    __syncthreads();
    for (int i = tid; i < kBigBins; i += 256)
        if (hist[i]) atomicAdd(&st->hist[LEVEL][i], (uint32_t)hist[i]);
}

// Keys above and equal to the threshold, per expert: sums in seg_count and seg_need (cleared before), and for budgets over
// several experts the number of equal keys of every kBigPiece tokens in eq_table [expert segment][piece].  A wave takes a
// piece at a time.  state == nullptr: there is room for every key, the counts are all there is to find.
__global__ __launch_bounds__(256) void drop_big_count_kernel(const uint32_t* __restrict__ key_t, BigState* __restrict__ state,
                                                             int32_t* __restrict__ eq_table, uint32_t* __restrict__ seg_tau,
                                                             int32_t* __restrict__ seg_need, int32_t* __restrict__ seg_count,
                                                             int N, int E, int seg_tokens, int span, int parts, int pieces) {
    __shared__ int red[4];
    const int seg = blockIdx.x / parts, part = blockIdx.x - seg * parts;
    const int b = seg / E, e = seg - b * E, ds = b * (E / span) + e / span, tid = threadIdx.x, lane = tid & 63;
    const uint32_t* keys = key_t + (size_t)e * N + (size_t)b * seg_tokens;
    BigState* st = state + ds;
    uint32_t tau = 0;  // every candidate (key >= 1) passes
    const bool threshold = state && st->rem[0] > 0;
    if (threshold) {
        int digit, left, total;
        pick_digit(st->hist[2], st->rem[1], &digit, &left, &total, red);
        tau = st->prefix[1] | (uint32_t)digit;
        if (part == 0 && e % span == 0 && tid == 0) {
            st->rem[2] = left;
            st->eq_total = (int)st->hist[2][digit];
        }
    }
    int gt = 0, eq = 0;  // of this wave
    for (int q = tid >> 6; q < kBigChunk / kBigPiece; q += 4) {
        const int piece = part * (kBigChunk / kBigPiece) + q, t0 = piece * kBigPiece + lane;
        if (piece >= pieces) break;
        constexpr int kLoads = kBigPiece / kWave;
        uint32_t key[kLoads];
#pragma unroll
        for (int j = 0; j < kLoads; ++j) key[j] = t0 + kWave * j < seg_tokens ? keys[t0 + kWave * j] : 0u;
        int here = 0;
#pragma unroll
        for (int j = 0; j < kLoads; ++j) {
            gt += __popcll(__ballot(key[j] > tau));
            here += __popcll(__ballot(key[j] == tau && key[j] != 0u));
        }
        if (threshold && span > 1 && lane == 0) eq_table[(size_t)seg * pieces + piece] = here;
        eq += here;
    }
    const int gt_total = block_sum_256(lane == 0 ? gt : 0, red), eq_total = block_sum_256(lane == 0 ? eq : 0, red);
    if (tid == 0) {
        if (part == 0) seg_tau[seg] = tau;
        if (gt_total) atomicAdd(&seg_count[seg], gt_total);
        if (eq_total) atomicAdd(&seg_need[seg], eq_total);
    }
}

// One block per segment.  seg_need: how many of the keys equal to the threshold an expert keeps.  Where a budget over several
// experts has room for a part of them they are granted in (token, expert) order, as in drop_select_kernel: the table tells
// the piece of tokens in which the budget ends, a thread per token of that piece the pair.
constexpr int kFinishThreads = kBigPiece;
__global__ __launch_bounds__(kFinishThreads) void drop_big_finish_kernel(const uint32_t* __restrict__ key_t,
                                                                         const BigState* __restrict__ state,
                                                                         const int32_t* __restrict__ eq_table,
                                                                         const uint32_t* __restrict__ seg_tau,
                                                                         int32_t* __restrict__ seg_need,
                                                                         int32_t* __restrict__ seg_count, int N, int E,
                                                                         int seg_tokens, int span, int pieces) {
    __shared__ int red[kFinishThreads / kWave];
    __shared__ int need_s[kMaxExperts];
    __shared__ int sh_piece, sh_left, sh_tie_token, sh_tie_run;
    const int groups = E / span, b = blockIdx.x / groups, e0 = (blockIdx.x - b * groups) * span, tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    const uint32_t* keys = key_t + (size_t)e0 * N + (size_t)b * seg_tokens;
    const BigState* st = state + blockIdx.x;
    const int seg0 = b * E + e0, rem = st->rem[2];
    for (int r = tid; r < span; r += kFinishThreads) need_s[r] = span == 1 && seg_need[seg0] > rem ? rem : seg_need[seg0 + r];
    __syncthreads();
    if (span > 1 && st->eq_total > rem) {
        const uint32_t tau = seg_tau[seg0];
        const int32_t* table = eq_table + (size_t)seg0 * pieces;
        // the piece: a thread adds up a run of consecutive ones
        const int per = (pieces + kFinishThreads - 1) / kFinishThreads;
        const int pb = tid * per < pieces ? tid * per : pieces, pe = pb + per < pieces ? pb + per : pieces;
        int c = 0, total;
        for (int p = pb; p < pe; ++p)
#pragma unroll 8
            for (int r = 0; r < span; ++r) c += table[(size_t)r * pieces + p];
        int before = block_exclusive_scan<kFinishThreads>(c, red, &total);
        if (before < rem && rem <= before + c) {  // exactly one thread: 1 <= rem < eq_total = total
            for (int p = pb; p < pe; ++p) {
                int here = 0;
                for (int r = 0; r < span; ++r) here += table[(size_t)r * pieces + p];
                if (before < rem && rem <= before + here) {
                    sh_piece = p;
                    sh_left = rem - before;
                }
                before += here;
            }
        }
        for (int r = tid; r < span; r += kFinishThreads) need_s[r] = 0;
        __syncthreads();
        // the pair
        const int piece = sh_piece, left = sh_left, t = piece * kBigPiece + tid;
        c = 0;
        if (t < seg_tokens)
#pragma unroll 8
            for (int r = 0; r < span; ++r) c += keys[(size_t)r * N + t] == tau;
        before = block_exclusive_scan<kFinishThreads>(c, red, &total);
        if (before < left && left <= before + c) {
            int open = left - before;
            for (int r = 0; r < span; ++r)
                if (keys[(size_t)r * N + t] == tau && --open == 0) {
                    sh_tie_token = t;
                    sh_tie_run = r;
                }
        }
        __syncthreads();
        // what each expert keeps: its pieces before that one, its tokens before the pair
        const int tie_token = sh_tie_token, tie_run = sh_tie_run;
        for (int r0 = 0; r0 < span; r0 += 8) {
            uint32_t key[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) key[u] = r0 + u < span && t <= tie_token ? keys[(size_t)(r0 + u) * N + t] : 0u;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int n = __popcll(__ballot(key[u] == tau && (t < tie_token || r0 + u <= tie_run)));
                if (lane == 0 && n) atomicAdd(&need_s[r0 + u], n);
            }
        }
        for (int r = wv; r < span; r += kFinishThreads / kWave) {
            int n = 0;
            for (int p = lane; p < piece; p += kWave) n += table[(size_t)r * pieces + p];
            if (n) atomicAdd(&need_s[r], n);
        }
        __syncthreads();
    }
    for (int r = tid; r < span; r += kFinishThreads) {
        seg_need[seg0 + r] = need_s[r];
        seg_count[seg0 + r] += need_s[r];
    }
}

// ---------------------------------------------------------------------------------------------
// The tile schedule of the expert GEMMs, built by the drop itself
// ---------------------------------------------------------------------------------------------
// One block of the kernel that finishes the plan adds up every segment's kept count anyway (it needs its own
// first row).  When the whole layer is enqueued by one call, that block also turns the per-expert totals into
// row offsets (in LDS) and builds the tile lists of the expert GEMMs from them, so that no kernel has to be
// launched between the plan and the first GEMM just to read expert_offset back.
// tot[e]: rows of expert e (complete, block-visible); off: kMaxExperts + 1 words of LDS.  Called by the whole
// block after a barrier; its first wave does the work.
__device__ inline void build_schedule_from_totals(const int* tot, int* off, const FfnScheduleArgs& a) {
    if (threadIdx.x >= kWave) return;
    const int lane = threadIdx.x;
    int base = 0;
#pragma unroll
    for (int c = 0; c < kMaxExperts / kWave; ++c) {
        const int e = c * kWave + lane;
        const int v = e < a.E ? tot[e] : 0;
        int incl = v;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
            const int up = __shfl_up(incl, o, kWave);
            if (lane >= o) incl += up;
        }
        if (e < a.E) off[e] = base + incl - v;
        base += __shfl(incl, kWave - 1, kWave);
    }
    if (lane == 0) off[a.E] = base;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();  // LDS operations of one wave complete in order: the offsets are there
    build_ffn_schedule(off, a);
}

// ---------------------------------------------------------------------------------------------
// 3. ordered compaction
// ---------------------------------------------------------------------------------------------
constexpr int kEmitRun = 16;                // consecutive tokens per thread
constexpr int kEmitChunk = 256 * kEmitRun;  // tokens per pass of the block

// A thread owns a run of 16 consecutive tokens and holds their keys and slots in registers.  The kernel is a chain of latencies:
// everything it reads is requested in one batch, the gating scores of the kept pairs in a second.  Against keys and slots staged
// through LDS a word and a byte at a time: 65536 tokens, 64 experts 36 -> 29 us, ranked by score 35 -> 25; 16384, 128 experts
// (2048 tokens a segment) 24.9 -> 21.7.
// A run may start at any word of the keys and any byte of the slots and is fetched in pieces of 16 bytes all the same (24001 tokens, 250
// experts without a capacity: the whole drop 75 us by words and bytes, 57 now; 250 experts on 25 devices, 4 tokens a segment, 73 and 63).
// ALIGNED: runs start on 16-byte boundaries of keys and slots (N and seg_tokens are multiples of 16).
template <bool ALIGNED>
__global__ __launch_bounds__(256) void drop_emit_kernel(const float* __restrict__ scores,
                                                        const uint32_t* __restrict__ key_t,
                                                        const uint8_t* __restrict__ slot_t,
                                                        const uint32_t* __restrict__ seg_tau,
                                                        const int32_t* __restrict__ seg_need,
                                                        const int32_t* __restrict__ seg_count,
                                                        int32_t* __restrict__ expert_count,
                                                        int32_t* __restrict__ expert_offset,
                                                        int32_t* __restrict__ row_token, float* __restrict__ row_weight,
                                                        int32_t* __restrict__ pair_row, int N, int E, int n_blocks,
                                                        int seg_tokens, int S, int weight_from_key,
                                                        FfnScheduleArgs sched) {
    __shared__ int red[4];
    __shared__ int red4[4][4];
    __shared__ int sched_tot[kMaxExperts], sched_off[kMaxExperts + 1];
    // With a schedule to build the grid has one block more, the first, which builds the GEMMs' tile schedule beside the others (as
    // one of theirs, its chain of scans followed the block's own: 128 experts on 8 devices 21.7 -> 14.0 us)
    if (sched.enabled && blockIdx.x == 0) {
        for (int i = threadIdx.x; i < kMaxExperts; i += 256) sched_tot[i] = 0;
        __syncthreads();
        for (int i = threadIdx.x; i < n_blocks * E; i += 256) atomicAdd(&sched_tot[i % E], seg_count[i]);
        __syncthreads();
        build_schedule_from_totals(sched_tot, sched_off, sched);
        return;
    }
    const int id = blockIdx.x - (sched.enabled ? 1 : 0);
    // a block owns one chunk of kEmitChunk tokens of one segment; what the chunks before it keep it counts itself
    const int parts = seg_tokens > kEmitChunk ? (seg_tokens + kEmitChunk - 1) / kEmitChunk : 1;
    // The blocks of one chunk (an expert each) write 4-byte entries of the same rows of pair_row and read entries of the
    // same rows of scores: where the chunks divide among the XCDs (block id mod 8) they share one, so that its L2 merges
    // the lines (65536 tokens, 64 experts on 8 devices: 53 -> 35 us).  The chunks of a long segment all read the keys
    // before them: they stay neighbours, so that those come from L2 (8 parts equal, 16: 118 -> 103 us, 64: 340 -> 209).
    const int chunks = n_blocks * parts;
    int chunk, e;
    if (chunks % 8 == 0 && parts <= 8) {
        const int slot = id >> 3;
        chunk = slot / E * 8 + (id & 7);
        e = slot % E;
    } else {
        e = id / parts % E;
        chunk = id / (parts * E) * parts + id % parts;
    }
    const int b = chunk / parts, c0 = (chunk - b * parts) * kEmitChunk, seg = b * E + e;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;

    const uint32_t* keys = key_t + (size_t)e * N + (size_t)b * seg_tokens;
    const uint8_t* slots = slot_t + (size_t)e * N + (size_t)b * seg_tokens;
    const int n = seg_tokens - c0 < kEmitChunk ? seg_tokens - c0 : kEmitChunk;
    const int i0 = tid * kEmitRun;  // this thread's first token of the chunk
    // ---- requested together: this run's keys and slots, threshold, the counts before it ----
    const uint32_t tau = seg_tau[seg];
    const int need = seg_need[seg];
    // (a thread without a run fetches the first one; a run that is cut short by the segment's end is fetched whole: what follows either
    // array in the workspace is longer than a run)
    const int at = c0 + (i0 < n ? i0 : 0);
    uint32_t kx[kEmitRun];
    uint8_t sx[kEmitRun];
    if (ALIGNED) {
#pragma unroll
        for (int j = 0; j < kEmitRun / 4; ++j) *(uint4*)&kx[4 * j] = *(const uint4*)(keys + at + 4 * j);
        *(uint4*)sx = *(const uint4*)(slots + at);
    } else {
        struct alignas(4) Words {
            uint32_t w[4];
        };
#pragma unroll
        for (int j = 0; j < kEmitRun / 4; ++j) *(Words*)&kx[4 * j] = *(const Words*)(keys + at + 4 * j);
        const uint32_t odd = (uint32_t)(uintptr_t)(slots + at) & 3u;  // bytes past a word
        const uint32_t* words = (const uint32_t*)(slots + at - odd);
        uint32_t raw[kEmitRun / 4 + 1];
        *(Words*)raw = *(const Words*)words;
        raw[kEmitRun / 4] = words[kEmitRun / 4];
#pragma unroll
        for (int j = 0; j < kEmitRun / 4; ++j) *(uint32_t*)&sx[4 * j] = __builtin_amdgcn_alignbyte(raw[j + 1], raw[j], odd);
    }
    // first row of this segment: all segments of lower experts, then lower blocks of this expert
    int before = 0, own = 0;
    constexpr int kAhead = 4;
    for (int k0 = tid; k0 < n_blocks * E; k0 += 256 * kAhead) {
        int c[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) c[u] = k0 + 256 * u < n_blocks * E ? seg_count[k0 + 256 * u] : 0;
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int i = k0 + 256 * u, bb = i / E, ee = i - bb * E;
            if (ee < e || (ee == e && bb < b)) before += c[u];
            if (ee == e) own += c[u];
        }
    }
    // the segment's tokens before this chunk: keys above the threshold, and keys equal to it (the first
    // `need` of those, in token order, are kept)
    int gt = 0, eq = 0;
    if (c0 > 0) {
        if (((N | seg_tokens) & 3) == 0) {  // every run starts on a 16-byte boundary
            const uint4* k4 = (const uint4*)keys;
            for (int i1 = tid; i1 < c0 / 4; i1 += 256 * 8) {
                uint4 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = i1 + 256 * u < c0 / 4 ? k4[i1 + 256 * u] : make_uint4(0, 0, 0, 0);
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    gt += (v[u].x > tau) + (v[u].y > tau) + (v[u].z > tau) + (v[u].w > tau);
                    eq += (v[u].x == tau) + (v[u].y == tau) + (v[u].z == tau) + (v[u].w == tau);
                }
            }
        } else {
            for (int i1 = tid; i1 < c0; i1 += 256 * 8) {
                uint32_t v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = i1 + 256 * u < c0 ? keys[i1 + 256 * u] : 0u;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    gt += v[u] > tau;
                    eq += v[u] == tau;
                }
            }
        }
        if (tau == 0u) eq = 0;  // key 0 is "not a candidate", never an equal key
    }
    int eq_cnt = 0;
#pragma unroll
    for (int j = 0; j < kEmitRun; ++j) {
        if (i0 + j >= n) kx[j] = 0u;
        eq_cnt += kx[j] != 0u && kx[j] == tau;
    }
    // block sums of the four (one barrier)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        before += __shfl_xor(before, off, kWave);
        own += __shfl_xor(own, off, kWave);
        gt += __shfl_xor(gt, off, kWave);
        eq += __shfl_xor(eq, off, kWave);
    }
    if (lane == 0) {
        red4[wv][0] = before;
        red4[wv][1] = own;
        red4[wv][2] = gt;
        red4[wv][3] = eq;
    }
    int total;
    int eq_rank = block_exclusive_scan_256(eq_cnt, red, &total);  // its barriers order the sums before their use
    int row0 = 0, own_total = 0, gt_base = 0, eq_base = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        row0 += red4[w][0];
        own_total += red4[w][1];
        gt_base += red4[w][2];
        eq_base += red4[w][3];
    }
    eq_rank += eq_base;
    const int kept_base = gt_base + (eq_base < need ? eq_base : need);
    if (b == 0 && c0 == 0 && tid == 0) {
        expert_count[e] = own_total;
        expert_offset[e] = row0;
        if (e == E - 1) expert_offset[E] = row0 + own_total;
    }
    uint32_t keep_bits = 0;
    int keep_cnt = 0;
#pragma unroll
    for (int j = 0; j < kEmitRun; ++j) {
        const bool cand = kx[j] != 0u;
        const bool is_eq = cand && kx[j] == tau;
        const bool keep = cand && (kx[j] > tau || (is_eq && eq_rank < need));
        eq_rank += is_eq;
        keep_cnt += keep;
        keep_bits |= (uint32_t)keep << j;
    }
    const int t0 = b * seg_tokens + c0 + i0;
    // the gating score, whatever ranked the pair (under the Score metric it is the key itself); pairs that are dropped, and runs
    // past the end, read the first token's
    uint32_t weight[kEmitRun];
#pragma unroll
    for (int j = 0; j < kEmitRun; ++j)
        weight[j] = weight_from_key ? kx[j] - 1u : __float_as_uint(scores[((keep_bits >> j) & 1u ? (size_t)(t0 + j) * E : (size_t)0) + e]);
    int pos = row0 + kept_base + block_exclusive_scan_256(keep_cnt, red, &total);
#pragma unroll
    for (int j = 0; j < kEmitRun; ++j) {
        if (kx[j] == 0u) continue;
        const bool keep = (keep_bits >> j) & 1u;
        if (keep) {
            row_token[pos] = t0 + j;
            row_weight[pos] = __uint_as_float(weight[j]);
        }
        pair_row[(size_t)(t0 + j) * S + sx[j]] = keep ? pos : -1;
        pos += keep;
    }
}

// ---------------------------------------------------------------------------------------------
// 4. at most k experts per token (optional; appendix "Maximum Number of Selected Experts")
// ---------------------------------------------------------------------------------------------
// Runs after a first emit.  For every token: its surviving pairs are listed, ranked by gating score
// (equal scores: lower expert id first), and those ranked k-th or worse are removed.  Keys of every pair
// that does not survive (dropped by capacity, or removed here) become 0, the per-segment counts are
// lowered, and thresholds are reset so that a second emit keeps exactly the non-zero keys.
// A block moves the keys of TOKENS tokens and all experts through LDS (the key matrix is expert-major: rows of
// consecutive tokens go in and out as whole sectors); then a wave takes a token at a time, lanes
// over experts: the c-th candidate in ascending expert id owns slot c of the token (ballot prefix counts).
// EPL = experts per lane (E <= 64 * EPL).  Nothing in the per-token loop waits for global memory: the
// tokens' slot rows are staged in LDS beside the keys and their score rows are requested up front.  A survivor is
// ranked where it lies: the scores of the others come out of their lanes one after another (uniform).
// Bound by latencies, a wave's tokens one after another, until its launch fills the chip: 3000 tokens x 64 experts 24.3 -> 9.7 us
// against blocks of 64 tokens that fetched key by key, score row by token and ranked through a list in LDS (300 tokens 20.7 -> 6.7,
// 32 768 25.5 -> 18.8, 16 384 x 256 48.4 -> 22.3).
template <int EPL, int TOKENS>
__global__ __launch_bounds__(256) void drop_limit_kernel(const float* __restrict__ scores, uint32_t* __restrict__ key_t,
                                                         int32_t* __restrict__ pair_row,
                                                         uint32_t* __restrict__ seg_tau, int32_t* __restrict__ seg_need,
                                                         int32_t* __restrict__ seg_count, int N, int E, int S, int k,
                                                         int seg_tokens, int segs) {
    constexpr int kPitch = TOKENS + 1;            // words per expert row of the block's key tile
    extern __shared__ uint32_t tile[];            // [E][kPitch] keys, then [TOKENS][S] rows of pair_row
    __shared__ int removed[kMaxExperts];          // pairs this block removes per expert (one global atomic each at the end)
    int32_t* rows = (int32_t*)(tile + (size_t)E * kPitch);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    constexpr int kPerWave = TOKENS / 4;    // tokens of a wave: wv, wv + 4, ...
    const int t_first = blockIdx.x * TOKENS;
    const int t_last = t_first + TOKENS - 1 < N ? t_first + TOKENS - 1 : N - 1;
    float sc[kPerWave][EPL];
#pragma unroll
    for (int q = 0; q < kPerWave; ++q)
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
            const int t = t_first + wv + 4 * q, e = lane + kWave * i;
            sc[q][i] = scores[(size_t)(t < N ? t : N - 1) * E + (e < E ? e : E - 1)];  // (lanes past E keep nothing)
        }
    for (int i = blockIdx.x * 256 + tid; i < segs; i += gridDim.x * 256) {
        seg_tau[i] = 0u;
        seg_need[i] = 0;
    }
    for (int e = tid; e < E; e += 256) removed[e] = 0;
    // the block's tokens lie in one capacity block when its first and last do
    const bool one_block = t_first / seg_tokens == t_last / seg_tokens;
    // both stagings request a batch before the first answer is stored (clamped addresses: a branch would serialise them)
    constexpr int kBatch = 8;
    const int n_rows = (t_last - t_first + 1) * S;  // the block's rows of pair_row are consecutive in memory
    for (int base = tid; base < E * TOKENS; base += 256 * kBatch) {
        uint32_t v[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const int i = base + 256 * j, e = i / TOKENS < E ? i / TOKENS : E - 1, t = t_first + i % TOKENS;
            v[j] = key_t[(size_t)e * N + (t < N ? t : N - 1)];
        }
#pragma unroll
        for (int j = 0; j < kBatch; ++j) asm volatile("" : "+v"(v[j]));
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const int i = base + 256 * j;
            if (i < E * TOKENS) tile[i / TOKENS * kPitch + i % TOKENS] = v[j];  // (tokens from N up are not looked at)
        }
    }
    for (int base = tid; base < n_rows; base += 256 * kBatch) {
        int32_t v[kBatch];
#pragma unroll
        for (int j = 0; j < kBatch; ++j) {
            const int i = base + 256 * j;
            v[j] = pair_row[(size_t)t_first * S + (i < n_rows ? i : n_rows - 1)];
        }
#pragma unroll
        for (int j = 0; j < kBatch; ++j) asm volatile("" : "+v"(v[j]));
#pragma unroll
        for (int j = 0; j < kBatch; ++j)
            if (base + 256 * j < n_rows) rows[base + 256 * j] = v[j];
    }
#pragma unroll
    for (int q = 0; q < kPerWave; ++q)
#pragma unroll
        for (int i = 0; i < EPL; ++i) asm volatile("" : "+v"(sc[q][i]));  // in flight since the start, not fetched per token
    __syncthreads();
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int q = 0; q < kPerWave; ++q) {
        const int tl = wv + 4 * q, t = t_first + tl;
        if (t >= N) break;  // wave-uniform
        int slot_base = 0, n = 0;
        int slot[EPL];
        uint64_t kept_mask[EPL];
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
            const int e = lane + kWave * i;
            const uint32_t key = e < E ? tile[e * kPitch + tl] : 0u;
            const bool cand = key != 0u;
            const uint64_t cand_mask = __ballot(cand);
            slot[i] = slot_base + __popcll(cand_mask & below);
            slot_base += __popcll(cand_mask);
            const bool kept = cand && rows[tl * S + slot[i]] >= 0;  // survived the capacity
            if (cand && !kept) tile[e * kPitch + tl] = 0u;
            kept_mask[i] = __ballot(kept);
            n += __popcll(kept_mask[i]);
        }
        if (n > k) {  // wave-uniform
            int better[EPL] = {};  // survivors ahead of mine: higher score, or equal score and lower expert id
#pragma unroll
            for (int i = 0; i < EPL; ++i)
                for (uint64_t left = kept_mask[i]; left; left &= left - 1) {
                    const int from = __builtin_ctzll(left);
                    const uint32_t other = (uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(sc[q][i]), from);
#pragma unroll
                    for (int j = 0; j < EPL; ++j) {
                        const uint32_t mine = __float_as_uint(sc[q][j]);
                        better[j] += other > mine || (other == mine && from + kWave * i < lane + kWave * j);
                    }
                }
            const int b = t / seg_tokens;
#pragma unroll
            for (int i = 0; i < EPL; ++i) {
                const int e = lane + kWave * i;
                if ((kept_mask[i] >> lane & 1) && better[i] >= k) {
                    tile[e * kPitch + tl] = 0u;
                    pair_row[(size_t)t * S + slot[i]] = -1;
                    if (one_block)
                        atomicAdd(&removed[e], 1);
                    else
                        atomicSub(&seg_count[b * E + e], 1);
                }
            }
        }
    }
    __syncthreads();
    for (int i = tid; i < E * TOKENS; i += 256) {
        const int e = i / TOKENS, tl = i - e * TOKENS;
        if (t_first + tl < N) key_t[(size_t)e * N + t_first + tl] = tile[e * kPitch + tl];
    }
    if (one_block)
        for (int e = tid; e < E; e += 256)
            if (removed[e]) atomicSub(&seg_count[(t_first / seg_tokens) * E + e], removed[e]);
}

// ---------------------------------------------------------------------------------------------
// 5. all of it in one launch, for small problems
// ---------------------------------------------------------------------------------------------
// With a few thousand tokens the three kernels above are a chain of short launches, each of which
// waits for the previous one to drain.  When every expert has its own capacity (no device budget, no
// per-token limit) a block can do the whole job for its segment alone: it needs the other segments
// only for its first output row, and their kept counts are min(candidates, capacity), which the
// block gets by counting the candidates of every segment itself from the top-k lists (read from L2
// by every block: small next to a launch as long as the lists are short).
constexpr int kFusedThreads = 1024;
constexpr int kFusedMaxTokens = 8 * kFusedThreads;  // tokens of a segment: its keys and slots live in LDS
constexpr int kFusedMaxSegs = 2048;    // capacity segments (one candidate counter each)
constexpr int kFusedCounters = 4096;   // counters in LDS: as many private copies of the segment counters as fit
constexpr long long kFusedMaxWork = 8ll << 20;  // segments x top-k list entries: above it, three launches are cheaper
constexpr int kFusedBins = 1024;       // counters of the threshold search
static_assert(kFusedBins <= kFusedCounters && kFusedBins % kFusedThreads == 0, "they may lie in the candidate counters' place");

// EXPANDED: Expanded Drop; ONE_BLOCK: a single capacity block (every token belongs to the block's segment
// list); VW: entries of a top-k list fetched per load (divides k).  The pass over the lists is the bulk of
// the kernel's instructions, so it is specialised.  NT: threads of the block, a segment holds at most 8 * NT
// tokens (short segments of short batches take small blocks: several per CU).
template <bool EXPANDED, bool ONE_BLOCK, int VW, int NT>
__global__ __launch_bounds__(NT) void drop_fused_kernel(
    const float* __restrict__ scores, const int32_t* __restrict__ topk_idx, const uint8_t* __restrict__ token_class,
    uint32_t seed, int32_t* __restrict__ expert_count, int32_t* __restrict__ seg_count,
    int32_t* __restrict__ expert_offset, int32_t* __restrict__ row_token, float* __restrict__ row_weight,
    int32_t* __restrict__ pair_row, int N, int E, int k, int S, int group_tokens, int group_experts, int metric,
    int seg_tokens, int n_blocks, int cap, int weight_from_key, FfnScheduleArgs sched) {
    constexpr int kWaves = NT / kWave, kMaxTok = NT * 8;
    __shared__ int sched_tot[kMaxExperts], sched_off[kMaxExperts + 1];
    // With a schedule to build the grid has one block more, which counts like the others but then, instead of finishing
    // a segment, builds the GEMMs' tile schedule: its chain of scans runs beside the segments' work
    // (1 token, 64 experts: 10.5 -> 7.1 us, with fewer copies of the counters; 8192 tokens, 8 experts on 4 devices 27 -> 21).
    const bool scheduler = blockIdx.x == (unsigned)(n_blocks * E);
    // a thread owns a run of consecutive tokens of the segment; one padding word per 16 keeps the runs of
    // neighbouring threads on different LDS banks
    __shared__ uint32_t key_s[kMaxTok + kMaxTok / 16];
    __shared__ uint8_t slot_s[kMaxTok];
    __shared__ int cand[kFusedCounters];
    // The counters of the threshold search.  A small block, of which a compute unit holds several, has them in the place of the candidate
    // counters, which are done with by then (its LDS decides how many: with 33 KB four fit, with 29 five; 500 tokens, 240 experts
    // on 5 devices 18.1 and 14.0 us); a large one in a place of their own, that is cleared ahead of time.
    constexpr bool kOwnBins = NT >= kFusedBins;
    __shared__ int bins[kOwnBins ? kFusedBins : 1];
    int* hist = kOwnBins ? bins : cand;
    __shared__ int red[kWaves], sh_bin[3];
    __shared__ uint32_t red5[kWaves][5];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int seg = blockIdx.x, b = seg / E, e = seg - b * E;
    const int segs = n_blocks * E;
    // Candidate counters: one private copy per lane of a wave where they fit (lanes that meet the same hot
    // expert in one instruction would otherwise serialise on its counter), an odd-ish pitch so that the
    // copies of one expert sit in different banks.
    const int pitch = segs + 1;
    // (short batches need few copies, and every copy is cleared and added up)
    const int wanted = N >= 16 * kWave ? kWave : (N + 15) / 16;
    const int copies = kFusedCounters / pitch < wanted ? kFusedCounters / pitch : wanted;  // >= 1
    auto pad = [](int i) { return i + (i >> 4); };

    for (int i = tid; i < copies * pitch; i += NT) cand[i] = 0;
    if (kOwnBins)
        for (int i = tid; i < kFusedBins; i += NT) hist[i] = 0;
    if (scheduler)
        for (int i = tid; i < kMaxExperts; i += NT) sched_tot[i] = 0;
    __syncthreads();

    // ---- one pass over the top-k lists, a thread per token: candidates of every segment (the experts of a
    // token's own device are counted later), and for the tokens of this block's segment what their list says
    // about expert e: listed experts with a lower id (bits 0-9), listed experts in all (bits 10-19), e itself
    // listed (bit 20); under Expanded Drop the experts of the token's own device do not count as listed, they
    // are candidates anyway
    {
        typedef int32_t vec_t __attribute__((ext_vector_type(VW)));
        int* mine = cand + (lane % copies) * pitch;
        constexpr int kTok = 4;        // tokens per thread and round
        constexpr int kVec = 8 / VW;   // loads per token and chunk of eight entries
        const int t_end = N;
        for (int t0 = tid; t0 < t_end; t0 += NT * kTok) {
            uint32_t info[kTok] = {0u, 0u, 0u, 0u};
            int tq[kTok];
#pragma unroll
            for (int q = 0; q < kTok; ++q) {
                const int t = t0 + NT * q;
                tq[q] = t < t_end ? t : t_end - 1;  // a token past the end re-reads the last one and is ignored below
            }
            for (int j0 = 0; j0 < k; j0 += 8) {
                vec_t x[kTok][kVec];  // independent loads, all issued before anything waits
#pragma unroll
                for (int q = 0; q < kTok; ++q)
#pragma unroll
                    for (int c = 0; c < kVec; ++c) {
                        const int j = j0 + c * VW < k ? j0 + c * VW : k - VW;  // past the list: a valid re-read
                        x[q][c] = *(const vec_t*)(topk_idx + (size_t)tq[q] * k + j);
                    }
#pragma unroll
                for (int q = 0; q < kTok; ++q) {
                    if (t0 + NT * q >= t_end) continue;
                    const int t = tq[q];
                    const int bb = ONE_BLOCK ? 0 : t / seg_tokens;
                    const int g0 = EXPANDED ? (t / group_tokens) * group_experts : 0;
                    int* row = mine + bb * E;
#pragma unroll
                    for (int c = 0; c < kVec; ++c) {
                        if (j0 + c * VW >= k) continue;  // the same for every thread
#pragma unroll
                        for (int u = 0; u < VW; ++u) {
                            const int xe = x[q][c][u];
                            const bool outside = !EXPANDED || xe < g0 || xe >= g0 + group_experts;
                            if (outside) atomicAdd(&row[xe], 1);
                            info[q] += (outside && xe < e ? 1u : 0u) + (outside ? 1u << 10 : 0u) + (xe == e ? 1u << 20 : 0u);
                        }
                    }
                }
            }
#pragma unroll
            for (int q = 0; q < kTok; ++q) {
                const int t = t0 + NT * q;
                if (t < t_end && !scheduler && (ONE_BLOCK || t / seg_tokens == b)) key_s[pad(t - b * seg_tokens)] = info[q];
            }
        }
    }
    __syncthreads();

    // ---- keys and slots of this block's segment ----
    uint32_t key_lo = 0xffffffffu, key_hi = 0u;
    if (!scheduler) {
        constexpr int kPer = 8;
        const int g_e = e / group_experts;  // device of this expert
        uint32_t info[kPer], rank[kPer];
        bool c[kPer];
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int tl = tid + NT * j;
            const int t = b * seg_tokens + tl;
            info[j] = tl < seg_tokens ? key_s[pad(tl)] : 0u;
            c[j] = tl < seg_tokens && ((info[j] >> 20) != 0u || (EXPANDED && t / group_tokens == g_e));
            rank[j] = 0u;
            if (c[j]) {
                rank[j] = pair_rank(metric, tl, seg_tokens, seed, (uint32_t)t * (uint32_t)E + (uint32_t)e,
                                    [&] { return __float_as_uint(scores[(size_t)t * E + e]); });
                if (token_class) rank[j] += (uint32_t)(token_class[t] & 3) << 30;
            }
        }
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int tl = tid + NT * j;
            if (tl >= seg_tokens) continue;
            const int t = b * seg_tokens + tl;
            int below = (int)(info[j] & 1023u);
            const int listed = (int)((info[j] >> 10) & 1023u);
            if (EXPANDED) below += device_experts_below(e, t / group_tokens * group_experts, group_experts);
            const uint32_t key = c[j] ? rank[j] + 1u : 0u;
            if (c[j]) {
                key_lo = key < key_lo ? key : key_lo;
                key_hi = key > key_hi ? key : key_hi;
            }
            key_s[pad(tl)] = key;
            slot_s[tl] = (uint8_t)below;
            if (e == 0) {  // slots beyond the token's candidate count stay unused
                const int n_c = listed + (EXPANDED ? group_experts : 0);
                for (int sl = n_c; sl < S; ++sl) pair_row[(size_t)t * S + sl] = -1;
            }
        }
    }
    __syncthreads();

    // ---- kept rows of every segment: this block's first row, its expert's total ----
    int before = 0, own_total = 0, n_cand = 0;
    for (int i = tid; i < segs; i += NT) {
        int c = 0;
        for (int r = 0; r < copies; ++r) c += cand[r * pitch + i];
        const int bb = i / E, ee = i - bb * E;
        if (EXPANDED) c += tokens_on_device(ee, bb, group_experts, group_tokens, seg_tokens);
        const int kept = c < cap ? c : cap;
        if (scheduler) atomicAdd(&sched_tot[ee], kept);
        if (ee < e || (ee == e && bb < b)) before += kept;
        if (ee == e) own_total += kept;
        if (i == seg) n_cand = c;
    }
    if (scheduler) {
        __syncthreads();
        build_schedule_from_totals(sched_tot, sched_off, sched);
        return;
    }
    // block sums of the three and the extent of the keys (one barrier)
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        before += __shfl_xor(before, off, kWave);
        own_total += __shfl_xor(own_total, off, kWave);
        n_cand += __shfl_xor(n_cand, off, kWave);
        const uint32_t a = __shfl_xor(key_lo, off, kWave), z = __shfl_xor(key_hi, off, kWave);
        key_lo = a < key_lo ? a : key_lo;
        key_hi = z > key_hi ? z : key_hi;
    }
    if (lane == 0) {
        red5[wv][0] = (uint32_t)before;
        red5[wv][1] = (uint32_t)own_total;
        red5[wv][2] = (uint32_t)n_cand;
        red5[wv][3] = key_lo;
        red5[wv][4] = key_hi;
    }
    __syncthreads();
    int row0 = 0, total;
    own_total = n_cand = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        row0 += (int)red5[w][0];
        own_total += (int)red5[w][1];
        n_cand += (int)red5[w][2];
        key_lo = red5[w][3] < key_lo ? red5[w][3] : key_lo;
        key_hi = red5[w][4] > key_hi ? red5[w][4] : key_hi;
    }
    if (tid == 0) {
        seg_count[seg] = n_cand < cap ? n_cand : cap;
        if (b == 0) {
            expert_count[e] = own_total;
            expert_offset[e] = row0;
            if (e == E - 1) expert_offset[E] = row0 + own_total;
        }
    }

    // ---- threshold: keys above tau are kept, `need` of the keys equal to tau are kept (Eq. 8) ----
    uint32_t tau = 0;  // every candidate (key >= 1) passes
    int need = 0;
    if (cap == 0) {
        tau = 0xffffffffu;  // nothing passes
    } else if (n_cand > cap) {
        need = cap;
        if (!kOwnBins) {
            for (int i = tid; i < kFusedBins; i += NT) hist[i] = 0;
            __syncthreads();
        }
        tau = select_threshold<NT, kFusedBins>(key_lo, key_hi, need, hist, red, sh_bin, [&](auto&& f) __attribute__((always_inline)) {
            for (int tl = tid; tl < seg_tokens; tl += NT) f(key_s[pad(tl)]);
        });
    }

    // ---- ordered compaction: rows in ascending token order, ties at the threshold to the lower tokens ----
    const int run = (seg_tokens + NT - 1) / NT;  // at most 8
    const int tb = tid * run;
    uint32_t kx[8];
    int eq_cnt = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        kx[j] = j < run && tb + j < seg_tokens ? key_s[pad(tb + j)] : 0u;
        eq_cnt += kx[j] != 0u && kx[j] == tau;
    }
    int eq_rank = block_exclusive_scan<NT>(eq_cnt, red, &total);
    uint32_t keep_bits = 0;
    int keep_cnt = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const bool c = kx[j] != 0u;
        const bool eq = c && kx[j] == tau;
        const bool keep = c && (kx[j] > tau || (eq && eq_rank < need));
        eq_rank += eq;
        keep_cnt += keep;
        keep_bits |= (uint32_t)keep << j;
    }
    int pos = row0 + block_exclusive_scan<NT>(keep_cnt, red, &total);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (kx[j] == 0u) continue;
        const int t = b * seg_tokens + tb + j;
        const bool keep = (keep_bits >> j) & 1u;
        if (keep) {
            row_token[pos] = t;
            // the gating score, whatever ranked the pair (under the Score metric it is the key itself)
            row_weight[pos] = weight_from_key ? __uint_as_float(kx[j] - 1u) : scores[(size_t)t * E + e];
        }
        pair_row[(size_t)t * S + slot_s[tb + j]] = keep ? pos : -1;
        pos += keep;
    }
}

// ---------------------------------------------------------------------------------------------
// 6. the same for a few tokens: a wave per segment
// ---------------------------------------------------------------------------------------------
// Decoding steps: segments of at most 64 tokens.  What bounds them is the chain of steps, each a barrier or a latency of the
// kernel above; here a wave holds its segment (a token per lane), ranks its keys against each other
// instead of looking for a threshold, and the only thing the waves of a block share is the number of candidates of every segment.
// us, alone: 1 token, 64 experts 6.8 -> 4.4; 16 tokens, 8 experts 8.8 -> 3.7; 37, 64 experts 9.1 -> 5.6; 256 on 8 devices, Expanded
// Drop 12.3 -> 7.7.
constexpr int kSmallSegTokens = kWave;
constexpr int kSmallSegs = 1024;
// What it costs is reading lists: its own tokens', each lane a list, and all of them, four entries a thread at a time; the kernel above
// reads vectors, a thread per token and round, but has a larger block per segment.  The times meet where k * (2 * seg_tokens + N) is
// about 5000 + 8 * segments (against the kernel above, 64 experts: 64 tokens with lists of 16 0.82, of 32 1.02, of 64 1.26; 256 on 4
// devices of 8 0.81, of 16 0.98, of 32 1.26; 512 on 8 of 8 0.88, of 16 1.10; 128 experts 256 on 8 of 32 0.77): 16 of 1354 sizes,
// up to 2048 tokens in 1024 segments, are more than 5 % off the better of the two.  Two tokens per lane, for up to 128 in a segment, took 0.9 to 2.6 of its time.
static bool small_lists(int k, int seg_tokens, int N, int segs) { return (long long)k * (2 * seg_tokens + N) <= 5000 + 8 * segs; }

template <bool EXPANDED>
__global__ __launch_bounds__(256) void drop_small_kernel(
    const float* __restrict__ scores, const int32_t* __restrict__ topk_idx, const uint8_t* __restrict__ token_class,
    uint32_t seed, int32_t* __restrict__ expert_count, int32_t* __restrict__ seg_count,
    int32_t* __restrict__ expert_offset, int32_t* __restrict__ row_token, float* __restrict__ row_weight,
    int32_t* __restrict__ pair_row, int N, int E, int k, int S, int group_tokens, int group_experts, int metric,
    int seg_tokens, int n_blocks, int cap, FfnScheduleArgs sched) {
    __shared__ int cand[kSmallSegs];
    __shared__ int sched_tot[kMaxExperts], sched_off[kMaxExperts + 1];
    const int tid = threadIdx.x, lane = tid & 63;
    const int segs = n_blocks * E;
    const bool scheduler = sched.enabled && blockIdx.x == gridDim.x - 1;  // the last block builds the GEMMs' tile schedule
    const int seg = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool mine = !scheduler && seg < segs;
    const int b = mine ? seg / E : 0, e = mine ? seg - b * E : 0;
    for (int i = tid; i < segs; i += 256) cand[i] = 0;
    if (scheduler)
        for (int i = tid; i < kMaxExperts; i += 256) sched_tot[i] = 0;

    // ---- this segment's scores and lists: listed experts below e and in all, e itself (under Expanded Drop without the experts of the
    // token's own device, which are candidates anyway) ----
    const int t = b * seg_tokens + lane;
    const bool live = mine && lane < seg_tokens;
    const size_t row = live ? t : 0;  // past the segment: the first token's, not used
    const uint32_t bits = __float_as_uint(scores[row * E + e]);
    uint32_t key;
    int below = 0, listed = 0;
    {
        const uint32_t cls = token_class ? (uint32_t)(token_class[row] & 3) << 30 : 0u;
        const int dev = EXPANDED ? t / group_tokens : 0, g0 = dev * group_experts;
        bool cnd = EXPANDED && e >= g0 && e < g0 + group_experts;
        const int32_t* list = topk_idx + row * k;
        for (int j0 = 0; j0 < k; j0 += 8) {
            int x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = list[j0 + u < k ? j0 + u : k - 1];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const bool counts = j0 + u < k && (!EXPANDED || x[u] < g0 || x[u] >= g0 + group_experts);
                listed += counts;
                below += counts && x[u] < e;
                cnd = cnd || (counts && x[u] == e);
            }
        }
        if (EXPANDED) below += device_experts_below(e, g0, group_experts);
        const uint32_t rank = pair_rank(metric, lane, seg_tokens, seed, (uint32_t)t * (uint32_t)E + (uint32_t)e, [&] { return bits; });
        key = live && cnd ? rank + cls + 1u : 0u;
        if (live && e == 0) {  // slots beyond the token's candidate count stay unused
            const int n_c = listed + (EXPANDED ? group_experts : 0);
            for (int sl = n_c; sl < S; ++sl) pair_row[(size_t)t * S + sl] = -1;
        }
    }
    __syncthreads();  // the counters are clear

    // ---- candidates of every segment, from all lists (the experts of a token's own device are counted below) ----
    const int entries = N * k;
    for (int i0 = tid; i0 < entries; i0 += 256 * 4) {
        int x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = i0 + 256 * u < entries ? topk_idx[i0 + 256 * u] : -1;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (x[u] < 0) continue;
            int at = x[u];
            if (EXPANDED || n_blocks > 1) {
                const int t = (i0 + 256 * u) / k;
                if (EXPANDED) {
                    const int g0 = t / group_tokens * group_experts;
                    if (x[u] >= g0 && x[u] < g0 + group_experts) continue;
                }
                at += t / seg_tokens * E;
            }
            atomicAdd(&cand[at], 1);
        }
    }
    __syncthreads();

    // ---- kept rows of every segment: this one's first row, its expert's total ----
    auto kept_of = [&](int i, int ee, int bb) {
        int c = cand[i];
        if (EXPANDED) c += tokens_on_device(ee, bb, group_experts, group_tokens, seg_tokens);
        return c < cap ? c : cap;
    };
    if (scheduler) {
        for (int i = tid; i < segs; i += 256) {
            const int bb = i / E, ee = i - bb * E;
            atomicAdd(&sched_tot[ee], kept_of(i, ee, bb));
        }
        __syncthreads();
        build_schedule_from_totals(sched_tot, sched_off, sched);
        return;
    }
    if (!mine) return;
    int before = 0, own_total = 0;
    for (int i = lane; i < segs; i += kWave) {
        const int bb = i / E, ee = i - bb * E, kept = kept_of(i, ee, bb);
        if (ee < e || (ee == e && bb < b)) before += kept;
        if (ee == e) own_total += kept;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        before += __shfl_xor(before, off, kWave);
        own_total += __shfl_xor(own_total, off, kWave);
    }
    const int n_cand = __popcll(__ballot(key != 0u));
    if (lane == 0) {
        seg_count[seg] = n_cand < cap ? n_cand : cap;
        if (b == 0) {
            expert_count[e] = own_total;
            expert_offset[e] = before;
            if (e == E - 1) expert_offset[E] = before + own_total;
        }
    }

    // ---- a pair stays if fewer than cap pairs are ahead of it: larger keys, and equal keys of lower tokens ----
    int ahead = 0;
    if (n_cand > cap) {
        for (int j0 = 0; j0 < seg_tokens; j0 += 8) {  // (past the segment keys are 0: ahead of no candidate)
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint32_t other = __builtin_amdgcn_readlane(key, j0 + u);
                ahead += other > key - (j0 + u < lane ? 1u : 0u);  // (a candidate's key is at least 1)
            }
        }
    }
    const bool keep = key != 0u && (n_cand <= cap || ahead < cap);
    const uint64_t mask = __ballot(keep);
    const int pos = before + __popcll(mask & ((1ull << lane) - 1ull));
    if (keep) {
        row_token[pos] = t;
        row_weight[pos] = __uint_as_float(bits);  // the gating score, whatever ranked the pair
    }
    if (key != 0u) pair_row[(size_t)t * S + below] = keep ? pos : -1;
}

// The plan of a batch without tokens: every count is zero.
__global__ __launch_bounds__(256) void drop_empty_kernel(int32_t* __restrict__ expert_count, int32_t* __restrict__ seg_count,
                                                         int32_t* __restrict__ expert_offset, int E, int segs) {
    for (int i = threadIdx.x; i < segs; i += 256) seg_count[i] = 0;
    for (int i = threadIdx.x; i <= E; i += 256) {
        expert_offset[i] = 0;
        if (i < E) expert_count[i] = 0;
    }
}

// keys are fetched four at a time: every run starts on a 16-byte boundary
static bool select_by_four(const Sizes& s, int n_tokens) { return n_tokens % 4 == 0 && s.seg_tokens % 4 == 0; }

// How the segments' thresholds are found.
enum class Select { kHeld, kLoop, kShared, kCount };
static Select select_form(const moe_desc_t& d, const Sizes& s) {
    const long long n_keys = (long long)s.seg_tokens * s.span;
    // A block holds the keys in its registers (at an odd pitch one load each, 32 a thread); no capacity: nothing to walk.
    if (n_keys <= (select_by_four(s, d.n_tokens) ? 65536 : 32768) || s.cap == 0) return Select::kHeld;
    // Room for every key: there is no threshold to find.
    if (s.cap >= n_keys) return Select::kCount;
    // One block reads its segment from L2 once for the extent of its keys and once or twice more, however many others do; shared segments
    // cost five launches and four passes over all keys at the chip's bandwidth.  A block each as a share of many blocks' time (the whole
    // drop): 8 segments of 50001 keys 0.96, of 65540 0.90, of 80000 0.99, of 98304 1.03, of 131072 1.07, of 262144 1.25; 32 of them
    // 0.91, 0.89, 0.97, 1.00, 1.02, 1.08; 48 of 131072 0.99, 64 of any 0.81 to 0.99; all scores equal 0.5 to 0.95.  Budgets over several
    // experts (the walk divides by the run length, and ties need a search): 16384 tokens x 64 269 us and 38; 256 segments of
    // 66560 keys 135 and 162, but up to a millisecond for ties.
    const int segs = s.n_blocks * (d.n_experts / s.span);
    return s.span > 1 || (n_keys > 98304 && segs < 48) ? Select::kShared : Select::kLoop;
}

size_t drop_big_state_bytes(const moe_desc_t& d, const Sizes& s) {
    if (select_form(d, s) != Select::kShared) return 0;
    const size_t segs = (size_t)s.n_blocks * d.n_experts;
    return segs / s.span * sizeof(BigState) + (s.span > 1 ? segs * big_pieces(s.seg_tokens) * sizeof(int32_t) : 0);
}

hipError_t launch_capacity_drop(const moe_desc_t& d, const Sizes& s, const DropWorkspace& ws, const float* scores,
                                const int32_t* topk_idx, const uint8_t* token_class, uint32_t seed,
                                int32_t* expert_count, int32_t* seg_count,
                                int32_t* expert_offset, int32_t* row_token, float* row_weight, int32_t* pair_row,
                                const FfnScheduleArgs* schedule, hipStream_t st) {
    const int N = d.n_tokens, E = d.n_experts;
    FfnScheduleArgs no_schedule = {};  // enabled = 0
    const FfnScheduleArgs& sched = schedule ? *schedule : no_schedule;
    if (N == 0) {  // scores, lists and pair_row may be null: no kernel that fetches from them is launched (and no row needs a schedule)
        ProfileScope prof(MOE_KERNEL_DROP_EMIT, st);
        hipLaunchKernelGGL(drop_empty_kernel, dim3(1), dim3(256), 0, st, expert_count, seg_count, expert_offset, E, s.n_blocks * E);
        return hipGetLastError();
    }
    {
        const int segs_all = s.n_blocks * E;
        constexpr int kSmallBlock = 256;  // threads of a block for short segments of short batches
        const bool fused = s.span == 1 && !(d.max_experts && s.slots > d.top_k) &&
                           s.seg_tokens <= kFusedMaxTokens && segs_all + 1 <= kFusedCounters &&
                           segs_all <= kFusedMaxSegs && (long long)segs_all * N * s.list_k <= kFusedMaxWork;
        if (fused && s.seg_tokens <= kSmallSegTokens && segs_all <= kSmallSegs && small_lists(s.list_k, s.seg_tokens, N, segs_all)) {
            ProfileScope prof(MOE_KERNEL_DROP_SELECT, st);
            auto kern = d.mode == MOE_MODE_EXPANDED_DROP ? drop_small_kernel<true> : drop_small_kernel<false>;
            hipLaunchKernelGGL(kern, dim3((segs_all + 3) / 4 + (sched.enabled ? 1 : 0)), dim3(256), 0, st, scores, topk_idx,
                               token_class, seed, expert_count, seg_count, expert_offset, row_token, row_weight, pair_row, N, E,
                               s.list_k, s.slots, s.group_tokens, s.group_experts, d.metric, s.seg_tokens, s.n_blocks, s.cap, sched);
            return hipGetLastError();
        }
        if (fused) {
            // every block reads all N lists: small blocks only where that is a single round for them too
            const bool small = s.seg_tokens <= 8 * kSmallBlock && N <= 8 * kSmallBlock;
            const bool ex = d.mode == MOE_MODE_EXPANDED_DROP, one = s.n_blocks == 1;
            auto launch = [&](auto kern, int threads) {
                ProfileScope prof(MOE_KERNEL_DROP_SELECT, st);
                hipLaunchKernelGGL(kern, dim3(segs_all + (sched.enabled ? 1 : 0)), dim3(threads), 0, st, scores, topk_idx, token_class, seed,
                                   expert_count, seg_count, expert_offset, row_token, row_weight, pair_row, N, E, s.list_k,
                                   s.slots, s.group_tokens, s.group_experts, d.metric, s.seg_tokens, s.n_blocks, s.cap,
                                   d.metric == MOE_METRIC_SCORE && !token_class ? 1 : 0, sched);
            };
            auto by_size = [&](auto ex_c, auto one_c, auto vw_c) {
                constexpr bool EX = decltype(ex_c)::value, ONE = decltype(one_c)::value;
                constexpr int VW = decltype(vw_c)::value;
                if (small)
                    launch(drop_fused_kernel<EX, ONE, VW, kSmallBlock>, kSmallBlock);
                else
                    launch(drop_fused_kernel<EX, ONE, VW, kFusedThreads>, kFusedThreads);
            };
            auto by_width = [&](auto ex_c, auto one_c) {
                if (s.list_k % 4 == 0)
                    by_size(ex_c, one_c, std::integral_constant<int, 4>{});
                else if (s.list_k % 2 == 0)
                    by_size(ex_c, one_c, std::integral_constant<int, 2>{});
                else
                    by_size(ex_c, one_c, std::integral_constant<int, 1>{});
            };
            if (ex && one)
                by_width(std::true_type{}, std::true_type{});
            else if (ex)
                by_width(std::true_type{}, std::false_type{});
            else if (one)
                by_width(std::false_type{}, std::true_type{});
            else
                by_width(std::false_type{}, std::false_type{});
            return hipGetLastError();
        }
    }
    const Select form = select_form(d, s);
    const bool many = form == Select::kShared || form == Select::kCount;  // blocks per segment
    const int segs = s.n_blocks * E, dsegs = segs / s.span;
    BigState* state = form == Select::kShared ? (BigState*)ws.big_state : nullptr;
    {
        const int grid = (N + kPrepTokens - 1) / kPrepTokens;
        const size_t lds = (size_t)kPrepTokens * (E | 1) * 5;
        if (lds > 64 * 1024)
            (void)hipFuncSetAttribute((const void*)drop_prepare_kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                      (int)lds);
        ProfileScope prof(MOE_KERNEL_DROP_PREPARE, st);
        hipLaunchKernelGGL(drop_prepare_kernel, dim3(grid), dim3(256), lds, st, scores, topk_idx, ws.key_t, ws.slot_t,
                           pair_row, N, E, s.list_k, s.slots, d.mode == MOE_MODE_EXPANDED_DROP ? 1 : 0, s.group_tokens,
                           s.group_experts, d.metric, s.seg_tokens, token_class, seed,
                           (uint32_t*)state, state ? (long long)dsegs * (long long)(sizeof(BigState) / 4) : 0ll,
                           many ? seg_count : nullptr, ws.seg_need, segs);
    }
    if (many) {
        ProfileScope prof(MOE_KERNEL_DROP_SELECT, st);
        const int chunks = (int)(((long long)s.seg_tokens * s.span + kBigChunk - 1) / kBigChunk);
        const int parts = (s.seg_tokens + kBigChunk - 1) / kBigChunk;
        auto hist = [&](auto kern) {
            hipLaunchKernelGGL(kern, dim3(dsegs * chunks), dim3(256), 0, st, ws.key_t, state, N, E, s.seg_tokens, s.span, s.cap,
                               chunks);
        };
        if (state && select_by_four(s, N)) {
            hist(drop_big_hist_kernel<0, 4>);
            hist(drop_big_hist_kernel<1, 4>);
            hist(drop_big_hist_kernel<2, 4>);
        } else if (state) {
            hist(drop_big_hist_kernel<0, 1>);
            hist(drop_big_hist_kernel<1, 1>);
            hist(drop_big_hist_kernel<2, 1>);
        }
        const int pieces = big_pieces(s.seg_tokens);
        int32_t* eq_table = state ? (int32_t*)(state + dsegs) : nullptr;  // (several experts under a budget)
        hipLaunchKernelGGL(drop_big_count_kernel, dim3(segs * parts), dim3(256), 0, st, ws.key_t, state, eq_table, ws.seg_tau,
                           ws.seg_need, seg_count, N, E, s.seg_tokens, s.span, parts, pieces);
        if (state)
            hipLaunchKernelGGL(drop_big_finish_kernel, dim3(dsegs), dim3(kFinishThreads), 0, st, ws.key_t, state, eq_table,
                               ws.seg_tau, ws.seg_need, seg_count, N, E, s.seg_tokens, s.span, pieces);
    } else {
        ProfileScope prof(MOE_KERNEL_DROP_SELECT, st);
        const size_t n_keys = (size_t)s.seg_tokens * s.span;
        const bool vec = select_by_four(s, N);
        // Threads per block: short segments are often many (1024 of 3190 keys at an odd pitch: 36 us with 1024 threads,
        // 11 with 256).
        const bool wide = n_keys > 4096;
        auto kern = !wide ? (vec ? drop_select_kernel<256, 4, 8, true>
                                 : (n_keys <= 2048 ? drop_select_kernel<256, 1, 8, true> : drop_select_kernel<256, 1, 16, true>))
                    : form == Select::kLoop
                        ? (vec ? drop_select_kernel<1024, 4, 16, false> : drop_select_kernel<1024, 1, 16, false>)
                    : vec ? drop_select_kernel<1024, 4, 16, true>
                          : (n_keys <= 16384 ? drop_select_kernel<1024, 1, 16, true> : drop_select_kernel<1024, 1, 32, true>);
        hipLaunchKernelGGL(kern, dim3(dsegs), dim3(wide ? 1024 : 256), 0, st, ws.key_t, ws.seg_tau,
                           ws.seg_need, seg_count, N, E, s.seg_tokens, s.span, s.cap);
    }
    auto emit = [&](bool last) {
        ProfileScope prof(MOE_KERNEL_DROP_EMIT, st);
        const int parts = s.seg_tokens > kEmitChunk ? (s.seg_tokens + kEmitChunk - 1) / kEmitChunk : 1;
        auto kern = N % 16 == 0 && s.seg_tokens % 16 == 0 ? drop_emit_kernel<true> : drop_emit_kernel<false>;
        const int extra = last && sched.enabled ? 1 : 0;
        hipLaunchKernelGGL(kern, dim3(segs * parts + extra), dim3(256), 0, st, scores, ws.key_t, ws.slot_t, ws.seg_tau,
                           ws.seg_need, seg_count, expert_count, expert_offset, row_token, row_weight, pair_row, N, E,
                           s.n_blocks, s.seg_tokens, s.slots, d.metric == MOE_METRIC_SCORE && !token_class ? 1 : 0,
                           last ? sched : no_schedule);
    };
    const bool limit = d.max_experts && s.slots > d.top_k;
    emit(!limit);
    if (limit) {
        // the first plan tells which pairs survive the capacity; trim every token to k of them, emit again
        // 16 tokens a block up to 16384 (32: 12.3 us against 9.7 at 3000, 23.9 against 22.3 at 16384 x 256); above, the blocks of
        // 16 run in many rounds and move half lines of the key matrix (32 768 x 64: 21.8 against 18.8, 65 536: 47.4 against 28.1)
        const int tokens = N <= 16384 ? 16 : 32;
        // the key tile and the tokens' rows of pair_row: at most 256 * 33 + 32 * 255 words
        const size_t lds = ((size_t)E * (tokens + 1) + (size_t)tokens * s.slots) * 4;
        auto kern = tokens == 16
                        ? (E <= 64 ? drop_limit_kernel<1, 16> : (E <= 128 ? drop_limit_kernel<2, 16> : drop_limit_kernel<4, 16>))
                        : (E <= 64 ? drop_limit_kernel<1, 32> : (E <= 128 ? drop_limit_kernel<2, 32> : drop_limit_kernel<4, 32>));
        if (lds > 48 * 1024)
            (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        {
            ProfileScope prof(MOE_KERNEL_DROP_LIMIT, st);
            hipLaunchKernelGGL(kern, dim3((N + tokens - 1) / tokens), dim3(256), lds, st, scores, ws.key_t,
                               pair_row, ws.seg_tau, ws.seg_need, seg_count, N, E, s.slots, d.top_k, s.seg_tokens, segs);
        }
        emit(true);
    }
    return hipGetLastError();
}

}  // namespace capmoe
