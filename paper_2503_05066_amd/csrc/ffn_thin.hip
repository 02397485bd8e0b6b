// The bf16 expert products of batches whose experts have few rows (see ffn.hip for the tile schedule and
// the other kernels): decoding steps, and any batch with a small capacity.
//
// The work is streaming weights.  The blocks of ffn.hip take 256 weight rows each: with few experts or narrow ones
// these are fewer than the chip has compute units, and with one block per compute unit its start is a gap in the stream.
// Here a block has 32 weight rows, and two blocks of four independent waves share a compute unit: 8 x 2048 x 1024, one
// row each, gate/up 24.4 -> 11.1 us, down 14.9 -> 7.2 us; 64 x 4096 x 1408, 16 tokens, 205 -> 179 and 107 -> 88 us
// (7.0 TB/s; without the non-temporal policy on the weights 201 and 101).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "schedule.h"

namespace capmoe {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((address_space(3))) void* lptr_t;

constexpr int kThinPiece = 32;                   // activation rows of a block, in sub-tiles of 16
constexpr int kThinWeightRows = 32;              // weight rows of a block
constexpr int kThinWaves = 4;                    // waves of a block; each multiplies a quarter of K
constexpr int kThinRingBytes = 18 * 1024;        // LDS of a wave: two blocks fit a compute unit

__device__ inline uint32_t thin_pack(float lo, float hi) {
    const f32x2 v = {lo, hi};
    const bf16x2 b = __builtin_convertvector(v, bf16x2);
    return *(const uint32_t*)&b;
}

// s_waitcnt immediate: at most n vector-memory operations outstanding, LDS/scalar counter at zero (gfx9 encoding)
__host__ __device__ constexpr int thin_waitcnt(int n) { return (n & 15) | (7 << 4) | ((n >> 4) << 14); }

// f(N), f(N - 1), .. f(0) with compile-time arguments
template <int N, class F>
__device__ __forceinline__ void count_down(F&& f) {
    f(std::integral_constant<int, N>{});
    if constexpr (N > 0) count_down<N - 1>(f);
}

// One block: up to 16 * TM rows of an expert times 32 weight rows: 32 output columns, or the gate and up rows of 16
// hidden columns.  The waves split K and share nothing until the end: each keeps a ring of its own in LDS, filled by
// direct loads (the layout and the piece swizzle of ffn.hip), waits for its own slabs only and needs no barrier.
// ONCE: the weights' lines need not be kept.
template <int TM, bool SWIGLU, bool ONCE>
struct ThinTile {
    static constexpr int kRows = 16 * TM;
    static constexpr int kCols = SWIGLU ? kThinWeightRows / 2 : kThinWeightRows;
    static constexpr int kLoads = (kRows + kThinWeightRows) / 8;  // wave-wide loads per slab, eight 128-byte rows each
    static constexpr int kSlot = kLoads * 1024;                   // bytes of a slab: activation rows, then weight rows
    static constexpr int kRing = kThinRingBytes / kSlot;          // slabs of 64 k in flight

    static __device__ __forceinline__ void run(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B0,
                                               const uint16_t* __restrict__ B1, uint16_t* __restrict__ C,
                                               const int32_t* __restrict__ gather, int e, int row0, int rows, int n0, int K,
                                               int Nout, uint8_t* smem) {
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));  // what follows from it is computed here, not for all three shapes at the block's start
        const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int lr = lane & 15, p = lane >> 4;

        constexpr int kRsrcFlags = 0x00020000;  // raw buffer of 32-bit words, no swizzle
        const __amdgpu_buffer_rsrc_t ra =
            __builtin_amdgcn_make_buffer_rsrc((void*)(gather ? A : A + (size_t)row0 * K), 0, -1, kRsrcFlags);
        const __amdgpu_buffer_rsrc_t r0 =
            __builtin_amdgcn_make_buffer_rsrc((void*)(B0 + ((size_t)e * Nout + n0) * K), 0, -1, kRsrcFlags);
        const __amdgpu_buffer_rsrc_t r1 =
            SWIGLU ? __builtin_amdgcn_make_buffer_rsrc((void*)(B1 + ((size_t)e * Nout + n0) * K), 0, -1, kRsrcFlags) : r0;
        uint32_t voff[kLoads];
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            const int r = i * 8 + lane / 8, kc = (lane % 8) ^ ((r >> 1) & 7);
            uint32_t row;
            if (r < kRows) {
                const int rr = r < rows ? r : rows - 1;  // rows past the expert's end repeat its last row
                row = gather ? (uint32_t)gather[row0 + rr] : (uint32_t)rr;
            } else {
                row = (uint32_t)(r - kRows);
                if (SWIGLU && row >= kCols) row -= kCols;
            }
            voff[i] = (row * (uint32_t)K + kc * 8) * 2u;
        }
        const int slabs_all = K / 64;
        const int first = wv * slabs_all / kThinWaves, n = (wv + 1) * slabs_all / kThinWaves - first;
        // column blocks start their walks at different slabs (see ffn.hip)
        const int turn = (int)((long long)n0 * n / Nout);
        uint8_t* ring = smem + wv * kThinRingBytes;
        auto request = [&](int s) {
            int at = s + turn;
            at = first + (at < n ? at : at - n);
            uint8_t* dst = ring + s % kRing * kSlot;
            const uint32_t k_bytes = (uint32_t)at * 128u;
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                const bool act = i < kRows / 8;
                const __amdgpu_buffer_rsrc_t r = act ? ra : (SWIGLU && i >= (kRows + kCols) / 8 ? r1 : r0);
                if (act)
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lptr_t)(dst + i * 1024), 16, voff[i], k_bytes, 0, 0);
                else
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lptr_t)(dst + i * 1024), 16, voff[i], k_bytes, 0, ONCE ? 2 : 0);
            }
        };
        const int piece = lr * 128 + ((p ^ ((lr >> 1) & 7)) << 4);  // this lane's operand piece of a sub-tile, first half slab
        f32x4 acc[2][TM];
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int m = 0; m < TM; ++m) acc[q][m] = f32x4{0.f, 0.f, 0.f, 0.f};
        auto multiply = [&](int s) {
            const uint8_t* slot = ring + s % kRing * kSlot;
            bf16x8 x[2][TM], w[2][2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int m = 0; m < TM; ++m) x[i][m] = *(const bf16x8*)(slot + 16 * m * 128 + (piece ^ (64 * i)));
#pragma unroll
                for (int q = 0; q < 2; ++q) w[i][q] = *(const bf16x8*)(slot + (kRows + 16 * q) * 128 + (piece ^ (64 * i)));
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int m = 0; m < TM; ++m)
#pragma unroll
                    for (int q = 0; q < 2; ++q)
                        acc[q][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[i][q], x[i][m], acc[q][m], 0, 0, 0);
        };
#pragma unroll
        for (int u = 0; u < kRing; ++u)
            if (u < n) request(u);
        // a slab has landed when only the younger requests are still out; its slot is refilled once its reads have returned
        int s = 0;
        for (; s + kRing < n; ++s) {
            __builtin_amdgcn_s_waitcnt(thin_waitcnt((kRing - 1) * kLoads));
            __builtin_amdgcn_sched_barrier(0);
            multiply(s);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(thin_waitcnt((kRing - 1) * kLoads));
            request(s + kRing);
            __builtin_amdgcn_sched_barrier(0);
        }
        const int left = n - s;  // at most a ring
        count_down<kRing - 1>([&](auto t) {
            constexpr int younger = decltype(t)::value;
            if (younger < left) {
                __builtin_amdgcn_s_waitcnt(thin_waitcnt(younger * kLoads));
                __builtin_amdgcn_sched_barrier(0);
                multiply(n - 1 - younger);
                __builtin_amdgcn_sched_barrier(0);
            }
        });
        // ---- the four partial tiles meet in LDS (every wave in its own ring) and are added in wave order ----
        f32x4* mine = (f32x4*)ring;
        if (wv > 0) {
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int m = 0; m < TM; ++m) mine[(q * TM + m) * 64 + lane] = acc[q][m];
        }
        __syncthreads();
        if (wv > 0) return;
#pragma unroll
        for (int u = 1; u < kThinWaves; ++u) {
            const f32x4* part = (const f32x4*)(smem + u * kThinRingBytes);
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int m = 0; m < TM; ++m) {
                    const f32x4 o = part[(q * TM + m) * 64 + lane];
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[q][m][v] += o[v];
                }
        }
#pragma unroll
        for (int m = 0; m < TM; ++m) {
            const int r = m * 16 + lr;
            if (r >= rows) continue;
            uint16_t* out = C + (size_t)(row0 + r) * Nout + n0 + 4 * p;
            if (SWIGLU) {
                float o[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float g = acc[0][m][v];
                    o[v] = g * acc[1][m][v] * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(g * -1.4426950408889634f));
                }
                *(uint2*)out = make_uint2(thin_pack(o[0], o[1]), thin_pack(o[2], o[3]));
            } else {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const f32x4 o = acc[q][m];
                    *(uint2*)(out + 16 * q) = make_uint2(thin_pack(o[0], o[1]), thin_pack(o[2], o[3]));
                }
            }
        }
    }
};

// An expert may have more than 64 rows (see ffn_is_thin; and expert_offset is the caller's: in a plan from elsewhere also more
// than the capacity leaves it), and then has big tiles too.  So the blocks walk the joint list, as often around as it takes.
// A tile of more than 32 rows is done in passes of its blocks over the same weights, which are fetched to be kept: the passes
// after the first find them in the L2 or, where the blocks that run together have more of them than its 4 MB, in the
// memory-side cache (64 tokens top-6, 64 x 4096 x 1408, 56 rows on one expert 210 -> 187 us, 64 top-2, 8 x 4096 x 1024, 53 rows
// 53 -> 47).
template <bool SWIGLU, bool STREAM>
__global__ __launch_bounds__(64 * kThinWaves, 2) void ffn_thin_kernel(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ B0, const uint16_t* __restrict__ B1,
    uint16_t* __restrict__ C, const int32_t* __restrict__ gather, const int32_t* __restrict__ tile_expert,
    const int32_t* __restrict__ tile_row0, const int32_t* __restrict__ tile_rows, const int32_t* __restrict__ n_tiles, int K,
    int Nout, int col_blocks) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    const int first = blockIdx.x / col_blocks, n0 = (blockIdx.x - first * col_blocks) * ThinTile<1, SWIGLU, STREAM>::kCols;
    const int step = gridDim.x / col_blocks, nt = *n_tiles;
    for (int tile = first; tile < nt; tile += step) {
        const int e = tile_expert[tile], row0 = tile_row0[tile], rows = tile_rows[tile] & kTileRowsMask;
        for (int at = 0; at < rows; at += kThinPiece) {
            if (tile > first || at > 0) __syncthreads();  // the first wave reads the others' sums out of their rings
            const int left = rows - at;
            if (rows > kThinPiece)
                ThinTile<2, SWIGLU, false>::run(A, B0, B1, C, gather, e, row0 + at, left < kThinPiece ? left : kThinPiece, n0, K,
                                                Nout, smem);
            else if (rows > 16)
                ThinTile<2, SWIGLU, STREAM>::run(A, B0, B1, C, gather, e, row0, rows, n0, K, Nout, smem);
            else
                ThinTile<1, SWIGLU, STREAM>::run(A, B0, B1, C, gather, e, row0, rows, n0, K, Nout, smem);
        }
    }
}

// most rows the capacity leaves an expert
static long long rows_bound(const moe_desc_t& d, const Sizes& s) {
    const long long kept = (long long)s.n_blocks * s.cap;
    return kept < d.n_tokens ? kept : d.n_tokens;
}

// Where the line lies (whole layers, ffn.hip -> this file).  Experts with at most 16 rows on average stream their weights
// faster here: 1 token, 64 experts x 2048 x 1024, top-8 62 -> 43 us; 2 of 96 experts x 3328 x 896 75 -> 40; 16 tokens,
// 64 x 4096 x 1408 331 -> 286, 8 x 4096 x 14336 458 -> 449; 37 and 64 tokens, 64 x 4096 x 1408 351 -> 340, 365 -> 362.
// With more rows a block fetches as many activations as weights and loses (256 tokens, 24 rows per expert 382 -> 393),
// except where the wide blocks are too few to fill half the chip: 64 tokens, 16 x 4096 x 512, 24 rows 90 -> 77 us, but
// 8 x 4096 x 1024, 64 rows 97 -> 101 and x 2048 126 -> 176.
// Where the capacity lets an expert have more than 64 rows, what it gets is not known here, and a tile of 256 rows is eight
// passes over the expert's weights.  With at most 256 rows in all, 8 on average, this is faster however they lie, as long as the
// weights that all tokens may share stay below 48 MB (the passes after the first then come from the caches) and the wide blocks
// do not split K either: tokens dealt evenly, half of them on one expert, all on one: 72 top-1, 16 x 4096 x 2048, 173, 155, 82 ->
// 125, 128, 37 us for both products; 256 top-1, 32 x 4096 x 2048, 276, 275, 119 -> 248, 270, 88, 128 x 4096 x 2048, 901, 633, 120 ->
// 840, 630, 88, 256 x 2048 x 768, 258, 162, 66 -> 252, 146, 46; 128 top-2, 64 x 2048 x 2048, 248, 233, 65 -> 237, 226, 41.
// Above each bound some plan loses: 256 top-1, 32 x 4096 x 4096, half on one 524 -> 557, 32 x 4096 x 14336, all on one
// 149 -> 474; 256 top-2, 96 x 2048 x 1024, 181 -> 192, 160 top-3, 64 x 2048 x 1024, over twelve experts 53 -> 57;
// 256 top-1, 32 x 8192 x 1024, all on one 82 -> 118, 32 x 1024 x 8192 72 -> 99.
bool ffn_is_thin(const moe_desc_t& d, const Sizes& s) {
    if (d.dtype != MOE_DTYPE_BF16) return false;
    if (rows_bound(d, s) > kFfnTileSmall) {
        const long long n = d.n_tokens, rows = std::max<long long>(s.max_rows, n);
        return rows <= 256 && s.max_rows <= 8ll * d.n_experts && d.d_model / 64 < kFfnSplitMinK && d.d_hidden / 64 < kFfnSplitMinK &&
               rows * d.d_model * d.d_hidden <= n << 23;
    }
    if (s.max_rows <= 16ll * d.n_experts) return true;
    return s.max_rows <= 24ll * d.n_experts && (long long)d.n_experts * (d.d_hidden / 128) <= 128;
}

template <bool SWIGLU, bool STREAM>
static void launch_thin(const Sizes& s, int experts, const void* A, const void* B0, const void* B1, void* C,
                        const int32_t* gather, const FfnWorkspace& ws, int K, int Nout, hipStream_t st) {
    constexpr int lds = kThinWaves * kThinRingBytes;
    auto kern = ffn_thin_kernel<SWIGLU, STREAM>;
    static std::atomic<uint64_t> configured{0};
    once_per_device(configured, [&] {
        (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    });
    const int col_blocks = Nout / ThinTile<1, SWIGLU, STREAM>::kCols;
    const long long tiles = s.max_rows < experts ? s.max_rows : experts;
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles * col_blocks)), dim3(64 * kThinWaves), lds, st, (const uint16_t*)A, (const uint16_t*)B0,
                       (const uint16_t*)B1, (uint16_t*)C, gather, ws.all.expert, ws.all.row0, ws.all.rows,
                       ws.all.count, K, Nout, col_blocks);
}

template <bool STREAM>
static void launch_both(const moe_desc_t& d, const Sizes& s, const FfnWorkspace& ws, const void* xp, const int32_t* row_token,
                        const void* w_gate, const void* w_up, const void* w_down, void* yp, hipStream_t st) {
    {
        ProfileScope prof(MOE_KERNEL_FFN_GATE_UP, st);
        launch_thin<true, STREAM>(s, d.n_experts, xp, w_gate, w_up, ws.hidden, row_token, ws, d.d_model, d.d_hidden, st);
    }
    ProfileScope prof(MOE_KERNEL_FFN_DOWN, st);
    launch_thin<false, STREAM>(s, d.n_experts, ws.hidden, w_down, nullptr, yp, nullptr, ws, d.d_hidden, d.d_model, st);
}

void launch_ffn_thin(const moe_desc_t& d, const Sizes& s, const FfnWorkspace& ws, const void* xp, const int32_t* row_token,
                     const void* w_gate, const void* w_up, const void* w_down, void* yp, hipStream_t st) {
    if (ffn_weights_stream(d, s))
        launch_both<true>(d, s, ws, xp, row_token, w_gate, w_up, w_down, yp, st);
    else
        launch_both<false>(d, s, ws, xp, row_token, w_gate, w_up, w_down, yp, st);
}

}  // namespace capmoe
