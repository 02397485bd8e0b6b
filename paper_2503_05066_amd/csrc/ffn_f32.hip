// The grouped SwiGLU FFN in fp32 (see ffn.hip for the bf16 kernels and the tile schedule).
//
// Both products run on v_mfma_f32_16x16x4_f32, whose result is the chain of fused multiply-adds over its four k
// (256 flops per cycle and compute unit, twice the unpacked vector rate).
#include <type_traits>

#include "common.h"
#include "schedule.h"

namespace capmoe {

typedef __attribute__((ext_vector_type(4))) float f32x4;
// four consecutive floats of a row whose pitch is any number of floats: dword alignment is all the loads need
typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4u;

constexpr int kF32Slab = 32;  // k of one slab: 128 bytes of every row, one cache line where the pitch allows it

// A block of NW waves computes up to 64 activation rows times 16 * TN * NW weight rows; a wave takes all rows of 16 * TN
// weight rows.  For the gate/up product TN = 2: 16 gate rows and the 16 up rows of the same hidden columns.
//
// What bounds it: the matrix cores where experts have rows (one row tile is 2048 cycles of matrix work per slab), the
// weight stream where they have few.  1024 tokens, 16 experts, 1024 x 2048: gate/up 659 -> 153 us, down 486 -> 74 us
// against one block per 16 x 16 outputs on vector instructions; 2048 tokens, top-4: 124 of the 154 TFLOP/s that the
// matrix instruction alone reaches.
//
// Slabs are fetched in 16-byte pieces, eight lanes to a row (whole cache lines: fetching the MFMA operands themselves,
// 16 rows x 64 bytes per load, thrashes the 32 KB first-level cache: 180 to 261 us for the same gate/up product), wait in
// registers, R slabs deep, and pass through one of two LDS buffers; piece kc of row r lies at position kc ^ ((r >> 1) & 7), which keeps the operand reads free of bank conflicts.  Lane l feeds row
// (l & 15) of a sub-tile; with p = l >> 4 its operands of a slab are pieces p and 4 + p, and element j of piece 4i + p goes
// into matrix instruction 4i + j.  Weight rows are the first operand (they become the four consecutive output columns of
// a lane), activation rows the second.
template <int NW, int TM, int TN, bool SWIGLU>
struct TileF32 {
    static_assert(!SWIGLU || TN == 2, "gate and up");
    static constexpr int kThreads = 64 * NW;
    static constexpr int BM = 16 * TM, BN = 16 * TN * NW;
    static constexpr int NB = BN * 8 / kThreads;                          // weight pieces a thread fetches per slab
    static constexpr int NA = (BM * 8 + kThreads - 1) / kThreads;         // activation pieces
    static constexpr int R = TM <= 2 ? 4 : 2;                             // slabs in registers
    static constexpr int kBuf = (64 + BN) * 128;                          // bytes of an LDS buffer

    static __device__ __forceinline__ int position(int idx) {
        const int r = idx >> 3, kc = idx & 7;
        return r * 128 + ((kc ^ ((r >> 1) & 7)) << 4);
    }

    static __device__ __forceinline__ void run(const float* __restrict__ A, const float* __restrict__ B0,
                                               const float* __restrict__ B1, float* __restrict__ C,
                                               const int32_t* __restrict__ gather, int e, int row0, int rows, int n0,
                                               int K, int Nout, uint8_t* smem) {
        const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
        const int lr = lane & 15, p = lane >> 4;
        // ---- sources: thread tid fetches pieces tid, tid + kThreads, .. of each operand ----
        const float *xs[NA], *ws[NB];
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int idx = tid + kThreads * i, r = (idx >> 3) < rows ? idx >> 3 : rows - 1;  // past the end: the last row
            xs[i] = A + (size_t)(gather ? gather[row0 + r] : row0 + r) * K + 4 * (idx & 7);
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int idx = tid + kThreads * i, rb = idx >> 3;
            const int c = SWIGLU ? n0 + (rb >> 5) * 16 + (rb & 15) : n0 + rb;
            const float* b = SWIGLU && (rb & 16) ? B1 : B0;
            ws[i] = b + ((size_t)e * Nout + (c < Nout ? c : Nout - 1)) * K + 4 * (idx & 7);
        }
        f32x4 xr[R][NA], wr[R][NB];
        const int slabs = K / kF32Slab, tail = K - slabs * kF32Slab;
        // Column blocks start their walks over K at different slabs: in step, they all read at the same offset of the row
        // pitch, from few memory channels when that is a power of two.  The start depends on the columns alone, the same for the
        // 64 columns of a wide block and of the narrow blocks in its place: a row's bits do not depend on its batch.
        const int turn = (int)((long long)(n0 & ~63) * slabs / Nout);
        // element offset of slab s; past the last slab: that one again
        auto slab_at = [&](int s) {
            s = (s < slabs ? s : slabs - 1) + turn;
            return (s < slabs ? s : s - slabs) * kF32Slab;
        };
        // fetch i: weight pieces first, then activation pieces
        auto request_one = [&](int u, int i, int at) {
            if (i < NB)
                wr[u][i] = *(const f32x4u*)(ws[i < NB ? i : 0] + at);
            else
                xr[u][i - NB] = *(const f32x4u*)(xs[i < NB ? 0 : i - NB] + at);
        };
        auto request = [&](int u, int s) {
            const int at = slab_at(s);
#pragma unroll
            for (int i = 0; i < NB + NA; ++i) request_one(u, i, at);
        };
        auto store_one = [&](int i, const f32x4(&x)[NA], const f32x4(&w)[NB], uint8_t* buf) {
            if (i < NB) {
                *(f32x4*)(buf + 64 * 128 + position(tid + kThreads * i)) = w[i < NB ? i : 0];
            } else {
                const int idx = tid + kThreads * (i - NB);
                if (BM * 8 % kThreads == 0 || idx < BM * 8) *(f32x4*)(buf + position(idx)) = x[i < NB ? 0 : i - NB];
            }
        };
        auto store = [&](const f32x4(&x)[NA], const f32x4(&w)[NB], uint8_t* buf) {
#pragma unroll
            for (int i = 0; i < NB + NA; ++i) store_one(i, x, w, buf);
        };
        f32x4 acc[TN][TM];
#pragma unroll
        for (int n = 0; n < TN; ++n)
#pragma unroll
            for (int m = 0; m < TM; ++m) acc[n][m] = f32x4{0.f, 0.f, 0.f, 0.f};
        // sub-tiles start at multiples of 16 rows: the swizzle depends on the lane alone
        const int piece0 = (p ^ ((lr >> 1) & 7)) << 4;
        const int a_at = lr * 128 + piece0, b_at = (64 + wv * 16 * TN + lr) * 128 + piece0;
        f32x4 xa[2][TM], wb[2][TN];  // operands of the two halves of a slab
        constexpr int NM = 4 * TM * TN, NR = TN + TM;
        auto read_one = [&](int half, int i, const uint8_t* buf) {
            if (i < TN)
                wb[half][i] = *(const f32x4*)(buf + i * 16 * 128 + (b_at ^ (64 * half)));
            else
                xa[half][i - TN] = *(const f32x4*)(buf + (i - TN) * 16 * 128 + (a_at ^ (64 * half)));
        };
        // the products of one half slab, with `extra` other operations spread between them (the scheduling barriers keep
        // them there: the compiler otherwise moves them to their use)
        auto multiply = [&](int half, auto n_extra, auto&& extra) {
            constexpr int NE = decltype(n_extra)::value;
#pragma unroll
            for (int q = 0; q < NM; ++q) {
                const int j = q / (TM * TN), m = q / TN % TM, n = q % TN;
                acc[n][m] = __builtin_amdgcn_mfma_f32_16x16x4f32(wb[half][n][j], xa[half][m][j], acc[n][m], 0, 0, 0);
#pragma unroll
                for (int i = 0; i < NE; ++i)
                    if (i * NM / NE == q) extra(i);
                if (NE > 0) __builtin_amdgcn_sched_barrier(0);
            }
        };
        const std::integral_constant<int, 0> nothing{};
        const std::integral_constant<int, NR + NB + NA> reads_and_pieces{};

        // ---- what K leaves after its last whole slab goes first: its loads and the first slabs' are under way together ----
        if (tail > 0) {
            const int at = slabs * kF32Slab;
            f32x4 xt[NA], wt[NB];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    const int k = 4 * ((tid + kThreads * i) & 7) + j;
                    wt[i][j] = ws[i][at + j + (k < tail ? 0 : tail - 1 - k)];
                }
#pragma unroll
                for (int i = 0; i < NA; ++i) {
                    const int k = 4 * ((tid + kThreads * i) & 7) + j;
                    xt[i][j] = xs[i][at + j + (k < tail ? 0 : tail - 1 - k)];
                }
            }
            if (slabs > 0) {
#pragma unroll
                for (int u = 0; u < R; ++u) {
                    __builtin_amdgcn_sched_barrier(0);
                    request(u, u);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 4; ++j) {  // both operands are zero past the row's end
#pragma unroll
                for (int i = 0; i < NB; ++i) wt[i][j] = 4 * ((tid + kThreads * i) & 7) + j < tail ? wt[i][j] : 0.f;
#pragma unroll
                for (int i = 0; i < NA; ++i) xt[i][j] = 4 * ((tid + kThreads * i) & 7) + j < tail ? xt[i][j] : 0.f;
            }
            store(xt, wt, smem + kBuf);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < 2 * NR; ++i) read_one(i / NR, i % NR, smem + kBuf);
            multiply(0, nothing, [](int) {});
            multiply(1, nothing, [](int) {});
        } else {
#pragma unroll
            for (int u = 0; u < R; ++u) {
                request(u, u);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // ---- whole slabs.  Operand reads run half a slab ahead of the matrix instructions:
        //     reads of slab s, second half | slab s + 1 goes to the other buffer | products of the first half
        //     barrier (slab s + 1 is there, slab s has been read)
        //     reads of slab s + 1, first half | request for slab s + 1 + R | products of the second half
        if (slabs > 0) {
            store(xr[0], wr[0], smem);
            request(0, R);
            __syncthreads();
#pragma unroll
            for (int i = 0; i < NR; ++i) read_one(0, i, smem);
            __builtin_amdgcn_sched_barrier(0);
            for (int s0 = 0;; s0 += R) {
#pragma unroll
                for (int u = 0; u < R; ++u) {
                    if (s0 + u >= slabs) goto walked;
                    constexpr int kR = R;
                    const int un = (u + 1) % kR;
                    const uint8_t* here = smem + (u & 1) * kBuf;
                    uint8_t* next = smem + ((u + 1) & 1) * kBuf;
                    const int at = slab_at(s0 + u + 1 + R);
                    multiply(0, reads_and_pieces, [&](int i) {
                        if (i < NR)
                            read_one(1, i, here);
                        else
                            store_one(i - NR, xr[un], wr[un], next);
                    });
                    __syncthreads();
                    multiply(1, reads_and_pieces, [&](int i) {
                        if (i < NR)
                            read_one(0, i, next);
                        else
                            request_one(un, i - NR, at);
                    });
                }
            }
        }
    walked:
        // ---- lane: four consecutive columns of row lr of every sub-tile ----
#pragma unroll
        for (int m = 0; m < TM; ++m) {
            const int r = m * 16 + lr;
            if (r >= rows) continue;
#pragma unroll
            for (int n = 0; n < (SWIGLU ? 1 : TN); ++n) {
                f32x4 o = acc[n][m];
                if (SWIGLU) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) o[v] = o[v] / (1.0f + expf(-o[v])) * acc[TN - 1][m][v];
                }
                const int c = n0 + wv * (SWIGLU ? 16 : 16 * TN) + n * 16 + 4 * p;
                float* out = C + (size_t)(row0 + r) * Nout + c;
                if (c + 3 < Nout) {
                    *(f32x4u*)out = o;
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        if (c + v < Nout) out[v] = o[v];
                }
            }
        }
    }
};

// Work items: row tiles (fastest) x column blocks; every XCD (block id mod 8) takes a contiguous eighth, so that the tiles of
// an expert that read the same weight rows run side by side on one L2.  Of a 64-row tile's four sub-tiles only those that
// hold rows are multiplied: one after the other (PIECES == 1), or each by a block of its own (4).
template <int NW, int TN, bool SWIGLU, int PIECES>
__global__ __launch_bounds__(64 * NW, NW < 4 ? 2 : 3) void ffn_gemm_f32_kernel(
    const float* __restrict__ A, const float* __restrict__ B0, const float* __restrict__ B1, float* __restrict__ C,
    const int32_t* __restrict__ tile_expert, const int32_t* __restrict__ tile_row0, const int32_t* __restrict__ tile_rows,
    const int32_t* __restrict__ n_tiles, const int32_t* __restrict__ gather, int K, int Nout, int col_blocks) {
    static_assert(kFfnTileMF32 == 64 && (PIECES == 1 || PIECES == 4), "four sub-tiles");
    __shared__ __attribute__((aligned(16))) uint8_t smem[2 * TileF32<NW, 4 / PIECES, TN, SWIGLU>::kBuf];
    const int nt = *n_tiles * PIECES;
    const long long total = (long long)nt * col_blocks, chunk = (total + 7) >> 3;
    const long long slot = blockIdx.x >> 3, logical = (blockIdx.x & 7) * chunk + slot;
    if (slot >= chunk || logical >= total) return;
    const int nb = (int)(logical / nt), item = (int)(logical - (long long)nb * nt), tile = item / PIECES;
    const int first = 16 * (item % PIECES);  // of the tile's rows
    const int e = tile_expert[tile], row0 = tile_row0[tile] + first, rows = (tile_rows[tile] & kTileRowsMask) - first;
    const int n0 = nb * (SWIGLU ? 16 : 16 * TN) * NW;
    if (PIECES > 1) {
        if (rows > 0)
            TileF32<NW, 1, TN, SWIGLU>::run(A, B0, B1, C, gather, e, row0, rows < 16 ? rows : 16, n0, K, Nout, smem);
    } else if (rows <= 16) {
        TileF32<NW, 1, TN, SWIGLU>::run(A, B0, B1, C, gather, e, row0, rows, n0, K, Nout, smem);
    } else if (rows <= 32) {
        TileF32<NW, 2, TN, SWIGLU>::run(A, B0, B1, C, gather, e, row0, rows, n0, K, Nout, smem);
    } else if (rows <= 48) {
        TileF32<NW, 3, TN, SWIGLU>::run(A, B0, B1, C, gather, e, row0, rows, n0, K, Nout, smem);
    } else {
        TileF32<NW, 4, TN, SWIGLU>::run(A, B0, B1, C, gather, e, row0, rows, n0, K, Nout, smem);
    }
}

template <int NW, int PIECES, bool SWIGLU>
static void launch_gemm_f32(const void* A, const void* B0, const void* B1, void* C, const int32_t* gather,
                            const FfnWorkspace& ws, int K, int Nout, hipStream_t st) {
    constexpr int TN = SWIGLU ? 2 : 1, kCols = 16 * NW;
    const int col_blocks = (Nout + kCols - 1) / kCols;
    const long long grid = ((long long)col_blocks * ws.big.max_tiles * PIECES + 7) / 8 * 8;
    hipLaunchKernelGGL((ffn_gemm_f32_kernel<NW, TN, SWIGLU, PIECES>), dim3((unsigned)grid), dim3(64 * NW), 0, st, (const float*)A,
                       (const float*)B0, (const float*)B1, (float*)C, ws.big.expert, ws.big.row0, ws.big.rows, ws.big.count,
                       gather, K, Nout, col_blocks);
}

template <bool SWIGLU>
static void choose_gemm_f32(const moe_desc_t& d, const Sizes& s, const void* A, const void* B0, const void* B1, void* C,
                            const int32_t* gather, const FfnWorkspace& ws, int K, int Nout, hipStream_t st) {
    // Four waves share the activation rows; one wave per block gives four times the blocks, which a weight stream without
    // much matrix work needs as long as the wide blocks are few.  Wide -> narrow, gate/up + down: 64 tokens top-2,
    // 8 experts x 1024 x 1024 37 -> 34 us, 16 x 1024 x 2048 66 -> 57, 64 x 600 x 300 23 -> 20; but 400 tokens,
    // 8 x 512 x 1000 (100 rows per expert) 43 -> 46, 1000 tokens 63 -> 92.
    const long long tiles = (s.max_rows < d.n_experts ? s.max_rows : d.n_experts) + s.max_rows / kFfnTileMF32;
    const long long wide_blocks = tiles * ((Nout + 63) / 64);
    // Few blocks are few chains of matrix instructions: a wave per sub-tile of 16 rows shortens them.  Products of up to half
    // the chip's wide blocks, whole tiles -> sub-tiles, gate/up + down: 429 tokens, 8 x 84 x 7 16.6 -> 14.4 us; 1000 top-2,
    // 8 x 64 x 128 (39 and 78 blocks) 16.2 -> 14.6; but 2000, 8 x 128 x 100 (140) 20 -> 24, 1024, 8 x 256 x 256 (160) 25 -> 29,
    // and with a handful of rows per expert most pieces are empty (131 tokens, 32 x 312 x 6 14.9 -> 15.3).
    if (wide_blocks <= 128 && s.max_rows > 8ll * d.n_experts)
        launch_gemm_f32<1, 4, SWIGLU>(A, B0, B1, C, gather, ws, K, Nout, st);
    else if (s.max_rows <= 32ll * d.n_experts && wide_blocks < 1024)
        launch_gemm_f32<1, 1, SWIGLU>(A, B0, B1, C, gather, ws, K, Nout, st);
    else
        launch_gemm_f32<4, 1, SWIGLU>(A, B0, B1, C, gather, ws, K, Nout, st);
}

void launch_ffn_gate_up_f32(const moe_desc_t& d, const Sizes& s, const FfnWorkspace& ws, const void* xp,
                            const int32_t* row_token, const void* w_gate, const void* w_up, hipStream_t st) {
    ProfileScope prof(MOE_KERNEL_FFN_GATE_UP, st);
    choose_gemm_f32<true>(d, s, xp, w_gate, w_up, ws.hidden, row_token, ws, d.d_model, d.d_hidden, st);
}

void launch_ffn_down_f32(const moe_desc_t& d, const Sizes& s, const FfnWorkspace& ws, const void* w_down, void* yp,
                         hipStream_t st) {
    ProfileScope prof(MOE_KERNEL_FFN_DOWN, st);
    choose_gemm_f32<false>(d, s, ws.hidden, w_down, nullptr, yp, nullptr, ws, d.d_hidden, d.d_model, st);
}

}  // namespace capmoe
