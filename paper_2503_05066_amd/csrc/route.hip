// Router: logits = x W_r^T + b, softmax over experts and top-k (Eq. 1).
//
// This translation unit is compiled with -ffp-contract=off: the softmax is a fixed sequence of
// individually rounded fp32 operations, so equal logits give bit-equal scores on any conforming
// implementation of the same sequence.
#include <hip/hip_bf16.h>

#include <type_traits>

#include "common.h"

namespace capmoe {

// ---------------------------------------------------------------------------------------------
// Router logits of bf16 activations whose width the matrix-core kernel does not take (router_mfma.hip: multiples of
// 32): a skinny GEMM [N,d] x [d,E], fp32 accumulation.
// One block computes 64 tokens x all experts; K is walked in slabs of 32 staged in LDS.
// Thread (ty,tx) of a 16x16 block owns tokens ty*4..+3 and experts tx + 16*i.
// ---------------------------------------------------------------------------------------------
__device__ inline float load_as_float(const __hip_bfloat16* p) {
    return __uint_as_float((uint32_t)(*(const uint16_t*)p) << 16);
}

constexpr int kRtTokens = 64;
constexpr int kRtSlab = 32;

template <int EPT>
__global__ __launch_bounds__(256) void router_logits_kernel(const __hip_bfloat16* __restrict__ x, const float* __restrict__ w,
                                                            const float* __restrict__ bias,
                                                            float* __restrict__ logits, int N, int d, int E) {
    extern __shared__ float smem[];
    float* xs = smem;                               // [64][33]
    float* wsm = smem + kRtTokens * (kRtSlab + 1);  // [16*EPT][33]
    const int tid = threadIdx.x;
    const int tx = tid & 15, ty = tid >> 4;
    const int t0 = blockIdx.x * kRtTokens;
    const int e_rows = 16 * EPT;

    float acc[4][EPT];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < EPT; ++j) acc[i][j] = 0.f;

    for (int k0 = 0; k0 < d; k0 += kRtSlab) {
        for (int idx = tid; idx < kRtTokens * kRtSlab; idx += 256) {
            const int r = idx >> 5, c = idx & 31;
            const int t = t0 + r, kk = k0 + c;
            xs[r * (kRtSlab + 1) + c] = (t < N && kk < d) ? load_as_float(x + (size_t)t * d + kk) : 0.f;
        }
        for (int idx = tid; idx < e_rows * kRtSlab; idx += 256) {
            const int r = idx >> 5, c = idx & 31;
            const int kk = k0 + c;
            wsm[r * (kRtSlab + 1) + c] = (r < E && kk < d) ? w[(size_t)r * d + kk] : 0.f;
        }
        __syncthreads();
#pragma unroll 8
        for (int c = 0; c < kRtSlab; ++c) {
            float xv[4], wv[EPT];
#pragma unroll
            for (int i = 0; i < 4; ++i) xv[i] = xs[(ty * 4 + i) * (kRtSlab + 1) + c];
#pragma unroll
            for (int j = 0; j < EPT; ++j) wv[j] = wsm[(tx + 16 * j) * (kRtSlab + 1) + c];
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < EPT; ++j) acc[i][j] = __builtin_fmaf(xv[i], wv[j], acc[i][j]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int t = t0 + ty * 4 + i;
        if (t >= N) continue;
#pragma unroll
        for (int j = 0; j < EPT; ++j) {
            const int e = tx + 16 * j;
            if (e < E) logits[(size_t)t * E + e] = acc[i][j] + (bias ? bias[e] : 0.f);
        }
    }
}

template <int EPT>
static void launch_rl(const __hip_bfloat16* x, const float* w, const float* bias, float* logits, int N, int d, int E,
                      hipStream_t st) {
    const int grid = (N + kRtTokens - 1) / kRtTokens;
    const size_t lds = sizeof(float) * (kRtSlab + 1) * (kRtTokens + 16 * EPT);
    hipLaunchKernelGGL((router_logits_kernel<EPT>), dim3(grid), dim3(256), lds, st, x, w, bias, logits, N, d, E);
}

static void dispatch_rl(const __hip_bfloat16* x, const float* w, const float* bias, float* logits, int N, int d, int E,
                        hipStream_t st) {
    const int ept = (E + 15) / 16;
    if (ept <= 1)
        launch_rl<1>(x, w, bias, logits, N, d, E, st);
    else if (ept <= 2)
        launch_rl<2>(x, w, bias, logits, N, d, E, st);
    else if (ept <= 4)
        launch_rl<4>(x, w, bias, logits, N, d, E, st);
    else if (ept <= 8)
        launch_rl<8>(x, w, bias, logits, N, d, E, st);
    else if (ept <= 16)
        launch_rl<16>(x, w, bias, logits, N, d, E, st);
    else
        launch_rl<32>(x, w, bias, logits, N, d, E, st);
}

// ---------------------------------------------------------------------------------------------
// fp32 activations on the matrix cores.  v_mfma_f32_16x16x4_f32 adds its four products as a chain of fused
// multiply-adds in ascending k (measured bit for bit, subnormal products included), so a logit is the same chain over
// the whole of K, in order, as one thread adding product after product: K is not split, whatever the size of the batch.
//
// The chain is what bounds it (32 cycles per four k; 1024 k 3.4 us) as long as the slabs arrive in time: WT x WE waves take
// 16 tokens x 16 experts each, slabs of 64 k are fetched as whole cache lines, wait R deep in registers and pass through
// one of two LDS buffers (rows of 68 words: the reads of an instruction, 16 rows x 4 words, then fall into 64 banks).
// 1024 tokens x 1024, 16 experts: 138 -> 10 us against 64 x 16 outputs per block on vector instructions.
// ---------------------------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4u;  // x may start at any float

constexpr int kRfSlab = 64;   // k per LDS buffer
constexpr int kRfPitch = 68;  // words of a row in LDS

template <int WT, int WE>
__global__ __launch_bounds__(64 * WT * WE) void router_logits_f32_kernel(const float* __restrict__ x,
                                                                         const float* __restrict__ w,
                                                                         const float* __restrict__ bias,
                                                                         float* __restrict__ logits, int N, int d, int E) {
    constexpr int kThreads = 64 * WT * WE, kRows = 16 * (WT + WE);  // token rows, then expert rows
    constexpr int kLoads = kRows * (kRfSlab / 4) / kThreads;        // 16-byte pieces a thread fetches per slab
    constexpr int R = 4;
    static_assert(kRows * (kRfSlab / 4) % kThreads == 0, "whole rounds of loads");
    __shared__ __attribute__((aligned(16))) float buf[2][kRows * kRfPitch];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int lr = lane & 15, p = lane >> 4;
    const int t0 = blockIdx.x * 16 * WT, e0 = blockIdx.y * 16 * WE;
    const float* src[kLoads];
    int dst[kLoads], kc[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
        const int idx = tid + kThreads * i, r = idx / (kRfSlab / 4);
        kc[i] = idx % (kRfSlab / 4) * 4;
        dst[i] = r * kRfPitch + kc[i];
        // rows past the last token or expert repeat it and are not stored
        const int t = t0 + r < N ? t0 + r : N - 1, e = e0 + r - 16 * WT < E ? e0 + r - 16 * WT : E - 1;
        src[i] = (r < 16 * WT ? x + (size_t)t * d : w + (size_t)e * d) + kc[i];
    }
    const int full = d / kRfSlab, rest = d - full * kRfSlab;  // rest: a multiple of four
    f32x4 ring[R][kLoads];
    auto request = [&](int u, int s) {  // past the last whole slab: that one again
        const int at = (s < full ? s : full - 1) * kRfSlab;
#pragma unroll
        for (int i = 0; i < kLoads; ++i) ring[u][i] = *(const f32x4u*)(src[i] + at);
    };
    const float* a_row = &buf[0][(16 * WT + (wv % WE) * 16 + lr) * kRfPitch + p];  // experts: the first operand
    const float* b_row = &buf[0][(wv / WE * 16 + lr) * kRfPitch + p];
    constexpr int kBuf = kRows * kRfPitch;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    f32x4 last[kLoads];  // what d leaves after its whole slabs (a piece lies inside a row or past its end)
    if (rest > 0) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i)
            last[i] = *(const f32x4u*)(src[i] + (kc[i] < rest ? full * kRfSlab : full * kRfSlab - kc[i] + rest - 4));
    }
    if (full > 0) {
#pragma unroll
        for (int u = 0; u < R; ++u) {
            __builtin_amdgcn_sched_barrier(0);
            request(u, u);
        }
        __builtin_amdgcn_sched_barrier(0);
        // buffer s & 1 was last read two slabs ago, and every wave has passed a barrier since
        auto slab = [&](auto u_c, auto refill_c, int s) {
            constexpr int u = decltype(u_c)::value;
            float* here = &buf[0][(u & 1) * kBuf];
#pragma unroll
            for (int i = 0; i < kLoads; ++i) *(f32x4*)(here + dst[i]) = ring[u][i];
            __builtin_amdgcn_sched_barrier(0);
            if (decltype(refill_c)::value) request(u, s + R);
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
            const float *a = a_row + (u & 1) * kBuf, *b = b_row + (u & 1) * kBuf;
            float av[kRfSlab / 4], bv[kRfSlab / 4];
#pragma unroll
            for (int q = 0; q < kRfSlab / 4; ++q) {
                av[q] = a[4 * q];
                bv[q] = b[4 * q];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < kRfSlab / 4; ++q) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[q], bv[q], acc, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        const std::integral_constant<int, 0> c0{};
        const std::integral_constant<int, 1> c1{};
        const std::integral_constant<int, 2> c2{};
        const std::integral_constant<int, 3> c3{};
        int s = 0;
        for (; s + R <= full; s += R) {  // no branch inside: the compiler's wait counts stay exact
            slab(c0, std::true_type{}, s);
            slab(c1, std::true_type{}, s + 1);
            slab(c2, std::true_type{}, s + 2);
            slab(c3, std::true_type{}, s + 3);
        }
        if (s < full) slab(c0, std::false_type{}, s);
        if (s + 1 < full) slab(c1, std::false_type{}, s + 1);
        if (s + 2 < full) slab(c2, std::false_type{}, s + 2);
    }
    if (rest > 0) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) *(f32x4*)(&buf[0][(full & 1) * kBuf + dst[i]]) = last[i];
        __syncthreads();
        for (int q = 0; q < rest / 4; ++q)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a_row[(full & 1) * kBuf + 4 * q], b_row[(full & 1) * kBuf + 4 * q], acc,
                                                       0, 0, 0);
    }
    // lane: four consecutive experts of token lr
    const int t = t0 + wv / WE * 16 + lr, e = e0 + wv % WE * 16 + 4 * p;
    if (t < N) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (e + v < E) logits[(size_t)t * E + e + v] = acc[v] + (bias ? bias[e + v] : 0.f);
    }
}

static void launch_router_f32(const float* x, const float* w, const float* bias, float* logits, int N, int d, int E,
                              hipStream_t st) {
    if (E <= 16)
        hipLaunchKernelGGL((router_logits_f32_kernel<1, 1>), dim3((N + 15) / 16), dim3(64), 0, st, x, w, bias, logits, N, d,
                           E);
    else
        hipLaunchKernelGGL((router_logits_f32_kernel<2, 2>), dim3((N + 31) / 32, (E + 31) / 32), dim3(256), 0, st, x, w, bias,
                           logits, N, d, E);
}

hipError_t launch_router_logits(const moe_desc_t& d, const void* x, const float* w, const float* bias, float* logits,
                                hipStream_t st) {
    ProfileScope prof(MOE_KERNEL_ROUTER_LOGITS, st);
    if (d.dtype == MOE_DTYPE_BF16)
        dispatch_rl((const __hip_bfloat16*)x, w, bias, logits, d.n_tokens, d.d_model, d.n_experts, st);
    else
        launch_router_f32((const float*)x, w, bias, logits, d.n_tokens, d.d_model, d.n_experts, st);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Softmax + top-k, one wavefront per token; lane l owns experts l, l+64, ...
//
// exp(z), z <= 0, by a fixed fp32 sequence: cut to zero below -80 (keeps every later value a
// normal number), n = rint(z*log2 e), r = z - n*ln2 in two fused steps, degree-7 Taylor polynomial
// by Horner with fused multiply-adds, scaling by 2^n.  The denominator is the sum of the
// numerators in ascending expert order; the quotient is an IEEE division.
// ---------------------------------------------------------------------------------------------
__device__ inline float exp_nonpositive(float z) {
    if (z < -80.0f) return 0.0f;
    const float n = __builtin_rintf(__fmul_rn(z, 0x1.715476p+0f));
    float r = __builtin_fmaf(n, -0x1.62e400p-1f, z);
    r = __builtin_fmaf(n, -0x1.7f7d1cp-20f, r);
    float q = 0x1.a01a02p-13f;
    q = __builtin_fmaf(q, r, 0x1.6c16c2p-10f);
    q = __builtin_fmaf(q, r, 0x1.111112p-7f);
    q = __builtin_fmaf(q, r, 0x1.555556p-5f);
    q = __builtin_fmaf(q, r, 0x1.555556p-3f);
    q = __builtin_fmaf(q, r, 0.5f);
    q = __builtin_fmaf(q, r, 1.0f);
    q = __builtin_fmaf(q, r, 1.0f);
    return __builtin_ldexpf(q, (int)n);
}

__device__ inline float wave_max(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, kWave));
    return v;
}

constexpr uint32_t kNoNumber = 0x3fffffffu;  // above every score

template <int EPL>
__global__ __launch_bounds__(256) void softmax_topk_kernel(float* __restrict__ logits,
                                                           const float* __restrict__ partial, int ksplit,
                                                           const float* __restrict__ bias, float* __restrict__ scores,
                                                           int32_t* __restrict__ topk_idx,
                                                           float* __restrict__ topk_score, int N, int E, int k) {
    __shared__ __attribute__((aligned(16))) float numer[4][EPL * kWave];
    __shared__ uint2 winners[4][kMaxTopK];  // (score bits, expert) of a token's k winners, ascending expert
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    // a wave works alone: its LDS row is private, and LDS operations of one wave complete in order
    for (int base = blockIdx.x * 4; base < N; base += gridDim.x * 4) {
        const int t = base + wv;
        const bool live = t < N;
        if (!live) break;
        float* l = logits + (size_t)(live ? t : 0) * E;
        float v[EPL];
        float m = -INFINITY;
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
            const int e = lane + kWave * i;
            if (e < E && partial) {
                // the router GEMM left one partial sum per K slice: add them in slice order
                // (eight loads in flight at a time: one dependent load per addition costs a microsecond each)
                float sum = bias ? bias[e] : 0.0f;
                for (int s0 = 0; s0 < ksplit; s0 += 8) {
                    float p[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        p[u] = s0 + u < ksplit ? partial[((size_t)(s0 + u) * N + t) * E + e] : 0.0f;
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (s0 + u < ksplit) sum = __fadd_rn(sum, p[u]);
                }
                v[i] = sum;
                if (live) l[e] = sum;
            } else {
                v[i] = e < E ? l[e] : -INFINITY;
            }
            m = fmaxf(m, v[i]);
        }
        m = wave_max(m);
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
            const int e = lane + kWave * i;
            v[i] = e < E ? exp_nonpositive(__fsub_rn(v[i], m)) : 0.0f;
            numer[wv][e] = v[i];
        }
        __builtin_amdgcn_wave_barrier();
        // every lane adds the numerators in ascending expert order (same address for all lanes, four per
        // read; the entries past E are +0 and leave the sum as it is)
        float sum = 0.0f;
        for (int e = 0; e < E; e += 4) {
            const float4 n4 = *(const float4*)&numer[wv][e];
            sum = __fadd_rn(__fadd_rn(__fadd_rn(__fadd_rn(sum, n4.x), n4.y), n4.z), n4.w);
        }
        __builtin_amdgcn_wave_barrier();  // the row is rewritten for the wave's next token only after these reads
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
            const int e = lane + kWave * i;
            v[i] = __fdiv_rn(v[i], sum);
            if (e < E)
                scores[(size_t)t * E + e] = v[i];
            else
                v[i] = -1.0f;
        }
        // top-k by selection: scores are >= +0, so their bit patterns order like the values.
        // (1) the k-th largest pattern by a 30-step binary search on ballots (1.0f has bit 29 as its highest), which ends
        //     as soon as a step has exactly k patterns above it (65536 tokens, 64 experts: 46 -> 38 us),
        // (2) winners = patterns above it, plus the lowest expert ids among those equal to it,
        // (3) every winner finds its place (larger score first, then lower expert id) by counting the
        //     winners ahead of it in a list the wave keeps in LDS.
        // Repeated wave-wide arg-max costs k rounds of cross-lane steps; this is a few ballots per bit.
        uint32_t bits[EPL];
#pragma unroll
        for (int i = 0; i < EPL; ++i) bits[i] = __float_as_uint(v[i] >= 0.0f ? v[i] : 0.0f);  // (a token without numbers: all the same)
        uint32_t tau = 0;
        for (int bit = 29; bit >= 0; --bit) {
            const uint32_t cand = tau | (1u << bit);
            int cnt = 0;
#pragma unroll
            for (int i = 0; i < EPL; ++i) cnt += __popcll(__ballot(lane + kWave * i < E && bits[i] >= cand));
            if (cnt >= k) tau = cand;
            if (cnt == k) {  // exactly the winners: any threshold between them and the rest will do
                tau = cand - 1u;
                break;
            }
        }
        int n_gt = 0;
#pragma unroll
        for (int i = 0; i < EPL; ++i) n_gt += __popcll(__ballot(lane + kWave * i < E && bits[i] > tau));
        const int need = k - n_gt;  // how many of the patterns equal to tau win (none if the search ended early)
        const uint64_t below = (1ull << lane) - 1ull;
        int eq_before = 0, win_before = 0;
        uint2* list = &winners[wv][0];
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
            const int e = lane + kWave * i;
            const bool valid = e < E;
            const bool eq = valid && bits[i] == tau;
            const uint64_t eq_mask = __ballot(eq);
            const bool win = valid && (bits[i] > tau || (eq && eq_before + __popcll(eq_mask & below) < need));
            const uint64_t win_mask = __ballot(win);
            if (win) list[win_before + __popcll(win_mask & below)] = make_uint2(bits[i], (uint32_t)e);
            eq_before += __popcll(eq_mask);
            win_before += __popcll(win_mask);
            if (!win) bits[i] = 0xffffffffu;  // marks "no output"
        }
        __builtin_amdgcn_wave_barrier();
        int place[EPL];
#pragma unroll
        for (int i = 0; i < EPL; ++i) place[i] = 0;
        for (int j = 0; j < k; ++j) {
            const uint2 w = list[j];  // same address in every lane
#pragma unroll
            for (int i = 0; i < EPL; ++i)
                place[i] += (w.x > bits[i] || (w.x == bits[i] && (int)w.y < lane + kWave * i)) ? 1 : 0;
        }
#pragma unroll
        for (int i = 0; i < EPL; ++i)
            if (bits[i] != 0xffffffffu) {
                topk_idx[(size_t)t * k + place[i]] = lane + kWave * i;
                topk_score[(size_t)t * k + place[i]] = v[i];
            }
        __builtin_amdgcn_wave_barrier();  // the list is rewritten for the wave's next token only after these reads
    }
}

// ---------------------------------------------------------------------------------------------
// The same for batches that fill the chip with four lanes per token: lane q of a token's four owns experts 16 i + 4 q .. + 3.
// Vector instructions are what bounds softmax and top-k (the bytes take 8 us where they took 38), and with a wave per token
// the sum's chain, the search and the ranking of the winners serve one token each; here they serve sixteen.
// 65536 tokens, 64 experts, top-8 38 -> 15.5 us (2.4 TB/s), 16384, 128 experts 18 -> 12.6.  The same bits as above.
// ---------------------------------------------------------------------------------------------
template <int CTRL>
__device__ inline int quad_perm(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
__device__ inline int quad_xor1(int v) { return quad_perm<0xB1>(v); }
__device__ inline int quad_xor2(int v) { return quad_perm<0x4E>(v); }
__device__ inline int quad_sum(int v) {
    v += quad_xor1(v);
    return v + quad_xor2(v);
}
template <int LANE>
__device__ inline float quad_from(float v) {  // the value of the quad's lane LANE
    return __int_as_float(quad_perm<LANE * 0x55>(__float_as_int(v)));
}

constexpr int kQuadTokens = 64;  // tokens of a block

// C: 16 * C experts at most; VEC: four experts per load (E % 4 == 0); FULL: exactly 16 * C experts
template <int C, bool VEC, bool FULL>
__global__ __launch_bounds__(256) void softmax_topk_quad_kernel(float* __restrict__ logits, const float* __restrict__ partial,
                                                                int ksplit, const float* __restrict__ bias,
                                                                float* __restrict__ scores, int32_t* __restrict__ topk_idx,
                                                                float* __restrict__ topk_score, int N, int experts, int k) {
    extern __shared__ unsigned long long quad_lists[];  // [64 tokens][k + 1]: keys of the winners
    constexpr int V = 4 * C;
    const int E = FULL ? 16 * C : experts;
    const int lane = threadIdx.x & 63, q = lane & 3;
    unsigned long long* list = quad_lists + (size_t)(threadIdx.x >> 2) * (k + 1);
    const int t = blockIdx.x * kQuadTokens + (threadIdx.x >> 2);
    const bool live = t < N;
    const size_t row = (size_t)(live ? t : N - 1) * E;  // past the last token: that one again, not stored
    if (blockIdx.x * kQuadTokens + (threadIdx.x & ~63) / 4 >= N) return;  // nothing for this wave
    auto expert = [&](int i) { return 16 * (i / 4) + 4 * q + i % 4; };
    auto valid = [&](int i) -> int { return FULL || expert(i) < E; };
    // four values of a row of E floats
    auto fetch = [&](const float* p, int c, float* out, float none) {
        const int e = 16 * c + 4 * q;
        float x[4];
        if (VEC) {
            *(f32x4*)x = *(const f32x4u*)(p + (FULL || e < E ? e : E - 4));
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] = p[e + j < E ? e + j : E - 1];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) out[j] = FULL || e + j < E ? x[j] : none;
    };
    auto store = [&](float* p, int c, const float* in) {
        const int e = 16 * c + 4 * q;
        if (VEC) {
            if (FULL || e < E) *(f32x4u*)(p + e) = f32x4{in[0], in[1], in[2], in[3]};
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (e + j < E) p[e + j] = in[j];
        }
    };
    float v[V];
    if (partial) {
        // the router GEMM left one partial sum per K slice: they are added in slice order, a few slices in flight
        constexpr int kAhead = C >= 8 ? 2 : 4;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            if (bias)
                fetch(bias, c, v + 4 * c, 0.0f);
            else
                v[4 * c] = v[4 * c + 1] = v[4 * c + 2] = v[4 * c + 3] = 0.0f;
        }
        for (int s0 = 0; s0 < ksplit; s0 += kAhead) {
            float p[kAhead][V];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int s = s0 + u < ksplit ? s0 + u : ksplit - 1;
#pragma unroll
                for (int c = 0; c < C; ++c) fetch(partial + (size_t)s * N * E + row, c, p[u] + 4 * c, 0.0f);
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
                if (s0 + u < ksplit)
#pragma unroll
                    for (int i = 0; i < V; ++i) v[i] = __fadd_rn(v[i], p[u][i]);
        }
        if (live)
#pragma unroll
            for (int c = 0; c < C; ++c) store(logits + row, c, v + 4 * c);
#pragma unroll
        for (int i = 0; i < V; ++i) v[i] = valid(i) ? v[i] : -INFINITY;
    } else {
#pragma unroll
        for (int c = 0; c < C; ++c) fetch(logits + row, c, v + 4 * c, -INFINITY);
    }
    float m = v[0];
#pragma unroll
    for (int i = 1; i < V; ++i) m = fmaxf(m, v[i]);
    m = fmaxf(m, __int_as_float(quad_xor1(__float_as_int(m))));
    m = fmaxf(m, __int_as_float(quad_xor2(__float_as_int(m))));
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] = valid(i) ? exp_nonpositive(__fsub_rn(v[i], m)) : 0.0f;
    // ascending expert order: the sum goes round the four lanes, four experts at each (the entries past E are +0)
    float sum = 0.0f;
    auto add4 = [&](float s, int c) {
        return __fadd_rn(__fadd_rn(__fadd_rn(__fadd_rn(s, v[4 * c]), v[4 * c + 1]), v[4 * c + 2]), v[4 * c + 3]);
    };
#pragma unroll
    for (int c = 0; c < C; ++c) {
        sum = add4(c == 0 ? 0.0f : quad_from<3>(sum), c);
        sum = add4(quad_from<0>(sum), c);
        sum = add4(quad_from<1>(sum), c);
        sum = add4(quad_from<2>(sum), c);
    }
    sum = quad_from<3>(sum);
    uint32_t bits[V];
    // IEEE quotients by one divisor: with y = 1 / sum rounded, two steps of q + (a - sum q) y from q = a y give a / sum rounded
    // (Markstein) as long as no remainder falls below the smallest number; others take the general division.
    uint32_t least = 0xffffffffu;
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const uint32_t b = __float_as_uint(v[i]) - 1u;  // zero is above all
        least = b < least ? b : least;
    }
    if (__any((least < __float_as_uint(0x1p-99f)) | (sum != sum))) {
#pragma unroll
        for (int i = 0; i < V; ++i) v[i] = __fdiv_rn(v[i], sum);
    } else {
        const float y = __fdiv_rn(1.0f, sum);
#pragma unroll
        for (int i = 0; i < V; ++i) {
            float r = __fmul_rn(v[i], y);
            r = __builtin_fmaf(__builtin_fmaf(-sum, r, v[i]), y, r);
            v[i] = __builtin_fmaf(__builtin_fmaf(-sum, r, v[i]), y, r);
        }
    }
    if (live)
#pragma unroll
        for (int c = 0; c < C; ++c) store(scores + row, c, v + 4 * c);
#pragma unroll
    for (int i = 0; i < V; ++i) bits[i] = sum != sum ? kNoNumber : __float_as_uint(v[i]);
#pragma unroll
    for (int i = 0; i < V; ++i) bits[i] = valid(i) ? bits[i] : 0u;  // never above a threshold
    // the k-th largest pattern, as in the kernel above; a token whose search has ended keeps its threshold
    uint32_t tau = 0;
    bool found = false;
    for (int bit = 29; bit >= 0; --bit) {
        const uint32_t cand = tau | (1u << bit);
        int cnt = 0;  // minus the number: all patterns are below 2^30
#pragma unroll
        for (int i = 0; i < V; ++i) cnt += (int)(cand - 1u - bits[i]) >> 31;
        cnt = -quad_sum(cnt);
        if (!found) {
            if (cnt >= k) tau = cand;
            if (cnt == k) {
                tau = cand - 1u;
                found = true;
            }
        }
        if (__all(found)) break;
    }
    int n_gt = 0, n_eq = 0;
#pragma unroll
    for (int i = 0; i < V; ++i) {
        n_gt += bits[i] > tau ? 1 : 0;
        n_eq += (int)(valid(i) & (bits[i] == tau));
    }
    const int own_gt = n_gt;
    n_gt = quad_sum(n_gt);
    const int need = k - n_gt, eq_all = quad_sum(n_eq);  // of the patterns equal to tau, the `need` lowest experts win
    int limit = need > 0 ? E : 0, own = own_gt + (need > 0 ? n_eq : 0);
    if (__any(need > 0 && need < eq_all)) {  // equal scores at the threshold: below which expert do `need` of them lie
        int low = 0;
        for (int b = kMaxExperts / 2; b > 0; b >>= 1) {
            int c = 0;
#pragma unroll
            for (int i = 0; i < V; ++i) c += (int)(valid(i) & (bits[i] == tau) & (expert(i) < low + b));
            if (quad_sum(c) <= need) low += b;
        }
        if (need > 0 && need < eq_all) {
            limit = low;
            own = own_gt;
#pragma unroll
            for (int i = 0; i < V; ++i) own += (int)(valid(i) & (bits[i] == tau) & (expert(i) < limit));
        }
    }
    int at = own;  // inclusive prefix over the four lanes, then exclusive
    const int from1 = quad_perm<0x90>(at);  // lanes 0 0 1 2
    at += q >= 1 ? from1 : 0;
    const int from2 = quad_perm<0x40>(at);  // lanes 0 0 0 1
    at += q >= 2 ? from2 : 0;
    at -= own;
    // winners by a key that orders them: larger score first, then lower expert id
    typedef unsigned long long u64;
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const bool win = (bits[i] > tau) | ((bits[i] == tau) & (expert(i) < limit));
        if (win) list[at] = (u64)bits[i] << 32 | (uint32_t)(kMaxExperts - 1 - expert(i));
        at += win ? 1 : 0;
    }
    if (q == 0) list[k] = 0;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();  // LDS operations of one wave complete in order
    // every winner's place is the number of larger keys; two winners at a time, eight of the list per round
    for (int j = q; j < k; j += 8) {
        const int j1 = j + 4 < k ? j + 4 : j;
        const u64 mine[2] = {list[j], list[j1]};
        int place[2] = {0, 0};
        for (int i0 = 0; i0 < k; i0 += 8) {
            u64 w[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) w[i] = list[i0 + i < k ? i0 + i : k];  // entry k: below every winner
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int u = 0; u < 2; ++u) place[u] += w[i] > mine[u] ? 1 : 0;
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (live & (j + 4 * u < k)) {
                topk_idx[(size_t)t * k + place[u]] = kMaxExperts - 1 - (int32_t)(uint32_t)mine[u];
                topk_score[(size_t)t * k + place[u]] = sum != sum ? sum : __uint_as_float((uint32_t)(mine[u] >> 32));
            }
    }
}

template <int C>
static void launch_quad(float* logits, const float* partial, int ksplit, const float* bias, float* scores, int32_t* topk_idx,
                        float* topk_score, int N, int E, int k, hipStream_t st) {
    const size_t lds = (size_t)kQuadTokens * (k + 1) * sizeof(unsigned long long);
    auto kern = E == 16 * C ? softmax_topk_quad_kernel<C, true, true>
                            : (E % 4 == 0 ? softmax_topk_quad_kernel<C, true, false> : softmax_topk_quad_kernel<C, false, false>);
    hipLaunchKernelGGL(kern, dim3((N + kQuadTokens - 1) / kQuadTokens), dim3(256), lds, st, logits, partial, ksplit, bias, scores,
                       topk_idx, topk_score, N, E, k);
}

// The tokens from which four lanes per token beat a wave per token, which is many rounds of waves by then; below, its shorter chain
// wins.  us, wave -> four lanes: 64 experts top-8 12288 tokens 8.8 -> 7.5, 16384 11.7 -> 8.4, 65536 37.5 -> 15.5; 128 top-8 12288 13.9 -> 11.9;
// 8 top-2 8192 1.2 times as fast, 12288 6.8 -> 4.4.  Quads that are not full walk the entries past E too (36 experts 1.0 to 1.08 of the
// wave's time at 12288, 0.95 to 1.05 at 14336, 0.8 to 0.9 at 16384; 160 1.05 to 1.25, 0.9 to 1.1, 0.65 to 1.0: the more the shorter
// the list).  Rows of experts that four does not divide are loaded by elements: 61 experts 1.06 to 1.15 at 12288, 0.85 to 0.95 at 16384;
// 127 top-8 1.25, 1.00, 0.88 at 24576; above 128 the registers hold one wave per SIMD: 255 top-8 1.28 at 24576, 1.23 at 65536, only long
// lists gain (top-33 1.02 at 40000, 0.90).  Every entry of a long list is ranked against all of it by the quad alone: 64 top-64 1.05 at
// 16384, 1.10 at 20480, 0.93 at 24576.
static int quad_tokens(int E, int k) {
    if (E % 4 != 0) {
        if (E <= 32) return 12288;
        if (E <= 64) return k <= 32 ? 16384 : 24576;
        if (E <= 128) return k < 16 ? 24576 : 16384;
        return k <= 16 ? INT_MAX : 32768;
    }
    if (E <= 64 && k > 32) return k > 48 ? 24576 : 16384;
    if (E <= 32 || E == 64 || E == 128) return 12288;
    return k <= 2 ? 16384 : (E > 64 && k >= 16 ? 12288 : 14336);
}

hipError_t launch_softmax_topk(const moe_desc_t& d, float* logits, const float* partial, int ksplit, const float* bias,
                               float* scores, int32_t* topk_idx, float* topk_score, hipStream_t st) {
    ProfileScope prof(MOE_KERNEL_SOFTMAX_TOPK, st);
    const int N = d.n_tokens, E = d.n_experts, k = d.top_k + d.overselect;
    if (N >= quad_tokens(E, k)) {
        if (E <= 16)
            launch_quad<1>(logits, partial, ksplit, bias, scores, topk_idx, topk_score, N, E, k, st);
        else if (E <= 32)
            launch_quad<2>(logits, partial, ksplit, bias, scores, topk_idx, topk_score, N, E, k, st);
        else if (E <= 64)
            launch_quad<4>(logits, partial, ksplit, bias, scores, topk_idx, topk_score, N, E, k, st);
        else if (E <= 128)
            launch_quad<8>(logits, partial, ksplit, bias, scores, topk_idx, topk_score, N, E, k, st);
        else
            launch_quad<16>(logits, partial, ksplit, bias, scores, topk_idx, topk_score, N, E, k, st);
        return hipGetLastError();
    }
    int grid = (N + 3) / 4;
    if (grid > 2048) grid = 2048;
    const int epl = (E + kWave - 1) / kWave;
    if (epl <= 1)
        hipLaunchKernelGGL((softmax_topk_kernel<1>), dim3(grid), dim3(256), 0, st, logits, partial, ksplit, bias, scores,
                           topk_idx, topk_score, N, E, k);
    else if (epl <= 2)
        hipLaunchKernelGGL((softmax_topk_kernel<2>), dim3(grid), dim3(256), 0, st, logits, partial, ksplit, bias, scores,
                           topk_idx, topk_score, N, E, k);
    else if (epl <= 4)
        hipLaunchKernelGGL((softmax_topk_kernel<4>), dim3(grid), dim3(256), 0, st, logits, partial, ksplit, bias, scores,
                           topk_idx, topk_score, N, E, k);
    else
        hipLaunchKernelGGL((softmax_topk_kernel<8>), dim3(grid), dim3(256), 0, st, logits, partial, ksplit, bias, scores,
                           topk_idx, topk_score, N, E, k);
    return hipGetLastError();
}

}  // namespace capmoe
