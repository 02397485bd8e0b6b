// Permutation into expert-major order and the weighted sum of Eq. (2).  Both are pure
// memory movement: every lane moves 16-byte pieces, consecutive lanes touch consecutive
// pieces of a row.
#include <algorithm>

#include "common.h"

namespace capmoe {

// xp[r,:] = x[row_token[r],:] for r < P.  `pieces` = 16-byte pieces per row.
__global__ __launch_bounds__(256) void dispatch_kernel(const uint4* __restrict__ x,
                                                       const int32_t* __restrict__ expert_offset,
                                                       const int32_t* __restrict__ row_token, uint4* __restrict__ xp,
                                                       int E, int pieces, long long max_items) {
    const long long P = expert_offset[E];
    const long long items = P * pieces < max_items ? P * pieces : max_items;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < items; i += (long long)gridDim.x * 256) {
        const long long r = i / pieces;
        const int c = (int)(i - r * pieces);
        xp[i] = x[(long long)row_token[r] * pieces + c];
    }
}

__device__ inline void accumulate_bf16x8(float* acc, const uint4& v, float w) {
    const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        acc[2 * i] = fmaf(w, __uint_as_float(u[i] << 16), acc[2 * i]);
        acc[2 * i + 1] = fmaf(w, __uint_as_float(u[i] & 0xffff0000u), acc[2 * i + 1]);
    }
}

// two floats -> two bf16 (round to nearest even) in one word: the hardware conversion
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
__device__ inline uint32_t combine_pack(float lo, float hi) {
    const f32x2 v = {lo, hi};
    const bf16x2 b = __builtin_convertvector(v, bf16x2);
    return *(const uint32_t*)&b;
}

// y[t,:] = sum over the token's slots (ascending) of row_weight[r] * yp[r,:], fp32 accumulation.
//
// A wave takes U pieces per lane (64 * U consecutive ones) of one token: lane s fetches slot s and its weight, a ballot
// tells which slots hold a row, and ROWS rows at a time are then fetched from wave-uniform addresses.
// The bytes bound it; what kept a thread per piece from them was three dependent loads per eight slots, taken or not, and
// every slot's index in every lane.  16384 tokens of 24 slots, 46 k rows x 2048 62 -> 41 us (6.2 TB/s), 8192 x 4096 29 -> 23,
// 4096 x 2048 15.1 -> 12.7, 3000 tokens of 32 slots 21 -> 17, 1 token 2.8 -> 2.2.
template <bool BF16, int U, int ROWS>
__global__ __launch_bounds__(256) void combine_kernel(const uint4* __restrict__ yp,
                                                      const float* __restrict__ row_weight,
                                                      const int32_t* __restrict__ pair_row, uint4* __restrict__ y,
                                                      long long units, int parts, int pieces, int S) {
    constexpr int kVals = BF16 ? 8 : 4;
    const int lane = threadIdx.x & 63;
    for (long long unit = (long long)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); unit < units;
         unit += (long long)gridDim.x * 4) {
        const long long t = unit / parts;
        const int c0 = (int)(unit - t * parts) * (64 * U) + lane;
        int col[U];  // a piece past the row's end: its last one, fetched but not stored
#pragma unroll
        for (int u = 0; u < U; ++u) col[u] = c0 + 64 * u < pieces ? c0 + 64 * u : pieces - 1;
        float acc[U][kVals];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < kVals; ++i) acc[u][i] = 0.f;
        for (int s0 = 0; s0 < S; s0 += 64) {
            const int r = s0 + lane < S ? pair_row[t * S + s0 + lane] : -1;
            const int w = r >= 0 ? __float_as_int(row_weight[r]) : 0;
            uint64_t left = __ballot(r >= 0);
            while (left) {
                uint4 v[ROWS][U];
                float wj[ROWS];
                int n = 0, slot = 0;
#pragma unroll
                for (int j = 0; j < ROWS; ++j) {
                    if (left) {  // past the last row: that one again
                        slot = __builtin_ctzll(left);
                        left &= left - 1;
                        ++n;
                    }
                    const uint4* row = yp + (long long)__builtin_amdgcn_readlane(r, slot) * pieces;
                    wj[j] = __int_as_float(__builtin_amdgcn_readlane(w, slot));
#pragma unroll
                    for (int u = 0; u < U; ++u) v[j][u] = row[col[u]];
                }
                // all of them are requested before any is used (the compiler otherwise moves each load behind the branch below)
#pragma unroll
                for (int j = 0; j < ROWS; ++j)
#pragma unroll
                    for (int u = 0; u < U; ++u) asm volatile("" : "+v"(v[j][u].x), "+v"(v[j][u].y), "+v"(v[j][u].z), "+v"(v[j][u].w));
#pragma unroll
                for (int j = 0; j < ROWS; ++j) {
                    if (j >= n) break;
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        if (BF16) {
                            accumulate_bf16x8(acc[u], v[j][u], wj[j]);
                        } else {
                            acc[u][0] = fmaf(wj[j], __uint_as_float(v[j][u].x), acc[u][0]);
                            acc[u][1] = fmaf(wj[j], __uint_as_float(v[j][u].y), acc[u][1]);
                            acc[u][2] = fmaf(wj[j], __uint_as_float(v[j][u].z), acc[u][2]);
                            acc[u][3] = fmaf(wj[j], __uint_as_float(v[j][u].w), acc[u][3]);
                        }
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (c0 + 64 * u >= pieces) continue;
            uint4 o;
            if (BF16)
                o = make_uint4(combine_pack(acc[u][0], acc[u][1]), combine_pack(acc[u][2], acc[u][3]),
                               combine_pack(acc[u][4 % kVals], acc[u][5 % kVals]), combine_pack(acc[u][6 % kVals], acc[u][7 % kVals]));
            else
                o = make_uint4(__float_as_uint(acc[u][0]), __float_as_uint(acc[u][1]), __float_as_uint(acc[u][2]),
                               __float_as_uint(acc[u][3]));
            y[t * pieces + c0 + 64 * u] = o;
        }
    }
}

// The same for rows shorter than a wave: a thread takes one piece, so that a wave serves several tokens (see choose_combine).
template <bool BF16>
__global__ __launch_bounds__(256) void combine_narrow_kernel(const uint4* __restrict__ yp,
                                                      const float* __restrict__ row_weight,
                                                      const int32_t* __restrict__ pair_row, uint4* __restrict__ y,
                                                      long long items, int pieces, int S) {
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < items; i += (long long)gridDim.x * 256) {
        const long long t = i / pieces;
        const int c = (int)(i - t * pieces);
        float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        // eight slots at a time: all row indices, then all weights, then all rows are requested before
        // any is used (three dependent memory levels per batch instead of three per slot); the sum
        // still runs in ascending slot order
        for (int s0 = 0; s0 < S; s0 += 8) {
            int r[8];
            float w[8];
            uint4 v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) r[j] = s0 + j < S ? pair_row[t * S + s0 + j] : -1;
#pragma unroll
            for (int j = 0; j < 8; ++j) w[j] = r[j] >= 0 ? row_weight[r[j]] : 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = r[j] >= 0 ? yp[(long long)r[j] * pieces + c] : make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                if (r[j] < 0) continue;
                if (BF16) {
                    accumulate_bf16x8(acc, v[j], w[j]);
                } else {
                    acc[0] = fmaf(w[j], __uint_as_float(v[j].x), acc[0]);
                    acc[1] = fmaf(w[j], __uint_as_float(v[j].y), acc[1]);
                    acc[2] = fmaf(w[j], __uint_as_float(v[j].z), acc[2]);
                    acc[3] = fmaf(w[j], __uint_as_float(v[j].w), acc[3]);
                }
            }
        }
        uint4 o;
        if (BF16) {
            o = make_uint4(combine_pack(acc[0], acc[1]), combine_pack(acc[2], acc[3]), combine_pack(acc[4], acc[5]),
                           combine_pack(acc[6], acc[7]));
        } else {
            o.x = __float_as_uint(acc[0]);
            o.y = __float_as_uint(acc[1]);
            o.z = __float_as_uint(acc[2]);
            o.w = __float_as_uint(acc[3]);
        }
        y[i] = o;
    }
}

static int grid_for(long long items) {
    long long g = (items + 255) / 256;
    const long long cap = 256 * 32;  // a few waves per SIMD; the kernels stride over the rest
    if (g > cap) g = cap;
    if (g < 1) g = 1;
    return (int)g;
}

hipError_t launch_dispatch(const moe_desc_t& d, const Sizes& s, const void* x, const int32_t* expert_offset,
                           const int32_t* row_token, void* xp, hipStream_t st) {
    const int pieces = (int)((size_t)d.d_model * s.elem / 16);
    const long long max_items = (long long)s.max_rows * pieces;
    ProfileScope prof(MOE_KERNEL_DISPATCH, st);
    hipLaunchKernelGGL(dispatch_kernel, dim3(grid_for(max_items)), dim3(256), 0, st, (const uint4*)x, expert_offset,
                       row_token, (uint4*)xp, d.n_experts, pieces, max_items);
    return hipGetLastError();
}

constexpr long long kMaxBlocks = 1 << 22;  // a launch has fewer than 2^32 threads; the kernel strides over the rest

template <bool BF16, int U, int ROWS>
static void launch_combine_units(const void* yp, const float* row_weight, const int32_t* pair_row, void* y, int tokens,
                                 int pieces, int slots, hipStream_t st) {
    const int parts = (pieces + 64 * U - 1) / (64 * U);
    const long long units = (long long)tokens * parts;
    hipLaunchKernelGGL((combine_kernel<BF16, U, ROWS>), dim3((unsigned)std::min<long long>((units + 3) / 4, kMaxBlocks)), dim3(256), 0,
                       st, (const uint4*)yp, row_weight, pair_row, (uint4*)y, units, parts, pieces, slots);
}

template <bool BF16>
static void choose_combine(const moe_desc_t& d, const Sizes& s, const void* yp, const float* row_weight, const int32_t* pair_row,
                           void* y, hipStream_t st) {
    const int pieces = (int)((size_t)d.d_model * s.elem / 16);
    const int n = d.n_tokens, slots = s.slots;
    // Short rows of many tokens: a wave for each token is many rounds of waves with idle lanes, against which its list, fetched at once,
    // weighs more the longer it is.  A wave per token against a thread per piece: rows of 8 pieces, 8 slots 1.04 times its time at 3000
    // tokens, 1.44 at 8192, 3.1 at 65536; of 32 1.06, 1.27, 1.18; of 48 0.98, 1.07, 1.00; of 64 1.02, 1.00, 0.97; 16 slots, 16
    // pieces 0.96 at 4096, 1.2 at 8192; of 40 0.94 and 0.99; 24 slots, 16 pieces 0.98 at 8192, 1.14 at 12000.
    const int widest = slots <= 8 ? 48 : (slots <= 16 ? 32 : 16);
    const int fewest = slots <= 8 ? 2048 : (slots <= 16 ? 256 : 400) * slots;
    if (pieces <= widest && n > fewest) {
        const long long items = (long long)n * pieces;
        hipLaunchKernelGGL((combine_narrow_kernel<BF16>), dim3(grid_for(items)), dim3(256), 0, st, (const uint4*)yp, row_weight,
                           pair_row, (uint4*)y, items, pieces, slots);
        return;
    }
    // Two pieces per lane from four rounds of waves on (8192 fit the chip), and where the rows' last waves would be half idle: the lists
    // are fetched half as often.  One piece -> two, in a layer: 65536 units of 24 slots 44 -> 41 us, of 2 26 -> 24, of 6 42 -> 34, of 8
    // 48.4 -> 47.6; 32768 of 8 24.3 -> 24.0; but 16384 of 8 12.7 -> 12.9, 12000 of 32 16.7 -> 17.4.  By itself, 96 pieces: 4096
    // tokens 5.4 -> 5.0, 300 2.7 -> 3.0.  Four pieces: never better.
    const long long units = (long long)n * ((pieces + 63) / 64);
    const bool two = pieces > 64 && (units >= 32768 || (pieces < 128 && units >= 4000));
    // As many rows in flight as short lists have: eight requests for one or two rows took 1.08 to 1.24 of the old kernel's time, four in
    // two pieces 25.2 us for 22.5 (8192 tokens of 512 pieces); and more of them where two pieces are fetched are no use (43 for 34).
    if (two && slots <= 2)
        launch_combine_units<BF16, 2, 2>(yp, row_weight, pair_row, y, n, pieces, slots, st);
    else if (two)
        launch_combine_units<BF16, 2, 4>(yp, row_weight, pair_row, y, n, pieces, slots, st);
    else if (slots <= 2)
        launch_combine_units<BF16, 1, 2>(yp, row_weight, pair_row, y, n, pieces, slots, st);
    else if (slots <= 4)
        launch_combine_units<BF16, 1, 4>(yp, row_weight, pair_row, y, n, pieces, slots, st);
    else
        launch_combine_units<BF16, 1, 8>(yp, row_weight, pair_row, y, n, pieces, slots, st);
}

hipError_t launch_combine(const moe_desc_t& d, const Sizes& s, const void* yp, const float* row_weight,
                          const int32_t* pair_row, void* y, hipStream_t st) {
    ProfileScope prof(MOE_KERNEL_COMBINE, st);
    if (d.dtype == MOE_DTYPE_BF16)
        choose_combine<true>(d, s, yp, row_weight, pair_row, y, st);
    else
        choose_combine<false>(d, s, yp, row_weight, pair_row, y, st);
    return hipGetLastError();
}

}  // namespace capmoe
