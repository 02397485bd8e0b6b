// Expert computation E_i(x) of Eq. (2): a grouped SwiGLU FFN over the expert-major rows.
//
//   hidden[r,:] = silu(W_gate[e] xp[r,:]) * (W_up[e] xp[r,:])        (GEMM 1, fused epilogue)
//   yp[r,:]     = W_down[e] hidden[r,:]                               (GEMM 2)
//
// Rows per expert are only known on the device, so one wave (a kernel of its own, or the tail of the
// capacity drop's last launch) first turns expert_offset into lists of row tiles (expert, first row,
// valid rows); the GEMM kernels run one block per compute unit, which takes items off these lists until none is left.
//
// bf16: both operands are K-contiguous ("NT" GEMM), staged through LDS in 16-byte pieces with an
// XOR swizzle and multiplied on the matrix cores with fp32 accumulation (v_mfma_f32_16x16x32_bf16):
// 256 x 256 blocks of 2 x 2 waves with 128 x 128 wave tiles, of which a block with fewer rows fetches and
// multiplies what is filled.  The weight rows feed the MFMA's first operand and the activation
// rows the second, so a lane ends up with 4 consecutive output columns of one row.
// The fp32 kernels are in ffn_f32.hip, those of the smallest bf16 batches in ffn_thin.hip.
#include <type_traits>
#include <utility>

#include "common.h"
#include "schedule.h"

namespace capmoe {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

// ---------------------------------------------------------------------------------------------
// tile schedule (schedule.h) as a kernel of its own: one wave
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(64) void ffn_schedule_kernel(const int32_t* __restrict__ expert_offset, FfnScheduleArgs args) {
    build_ffn_schedule(expert_offset, args);
}

// ---------------------------------------------------------------------------------------------
// bf16 MFMA path
// ---------------------------------------------------------------------------------------------
// two floats -> two bf16 (round to nearest even) in one word, lo in the low half: the hardware conversion
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
__device__ inline uint32_t pack_bf16x2(float lo, float hi) {
    const f32x2_t v = {lo, hi};
    const bf16x2_t b = __builtin_convertvector(v, bf16x2_t);
    return *(const uint32_t*)&b;
}

typedef __attribute__((address_space(3))) void* lptr_t;

// s_waitcnt immediate for "at most n vector-memory operations outstanding, LDS/scalar counter
// at zero" (gfx9 encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4 left at 7, lgkmcnt 11:8).
__host__ __device__ constexpr int waitcnt_vm(int n) { return (n & 15) | (7 << 4) | ((n >> 4) << 14); }

// ---------------------------------------------------------------------------------------------
// tiles on 16x16x32 matrix instructions, four waves
// ---------------------------------------------------------------------------------------------
// Under sustained load the chip is power-limited, so what a kernel reaches is set by the energy it spends
// per flop.  Measured on this part with random operands: the 16x16x32 instruction sustains about 10 % more
// flops than 32x32x16 (half the accumulator traffic per flop), and a wave tile of 128 x 128 needs a third
// fewer LDS operand reads per flop than 128 x 64.  With one wave per SIMD nothing hides a stalled
// instruction, so the requests for the next slabs are spread over the whole slab (a burst of fills from
// every wave right after the barrier backs up the address unit and stalls the matrix pipe behind it).
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

constexpr int kRsrcFlags = 0x00020000;  // raw buffer of 32-bit words, no swizzle (gfx9 descriptor word 3)
constexpr int kDeviceScope = 16;        // cache policy bit sc1 of the buffer instructions

// f(0), f(1), .. f(N - 1) with compile-time arguments
template <class F, int... Is>
__device__ __forceinline__ void each_of(std::integer_sequence<int, Is...>, F&& f) {
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void each(F&& f) {
    each_of(std::make_integer_sequence<int, N>{}, f);
}

// The accumulators: a wave of the 256-wide tiles holds 256 values, exactly the accumulation half of its register budget, and must
// never move them.  As variables they leave that to the compiler, whose allocator, with no register to spare, moved hundreds of
// them between the loops for the different tile heights (and knows neither the instruction inside an asm statement nor the
// wait states it asks for).  So they have fixed places, named in the statements: fragment F in a[4F .. 4F+3].  The compiler
// itself uses none of these registers (it has 256 others, and the kernels need no more; the kernel's first statement
// makes it count them; the build ends if its output shows otherwise, see accumulators.py).  The code that reads them after
// the last matrix instruction waits out its latency itself.
template <int F>
__device__ __forceinline__ void acc_mfma(const bf16x8& a, const bf16x8& b) {
    asm volatile("v_mfma_f32_16x16x32_bf16 a[%0:%1], %2, %3, a[%0:%1]" ::"n"(4 * F), "n"(4 * F + 3), "v"(a), "v"(b));
}
template <int F>
__device__ __forceinline__ void acc_zero() {
    asm volatile(
        "v_accvgpr_write_b32 a[%0], 0\n\tv_accvgpr_write_b32 a[%1], 0\n\t"
        "v_accvgpr_write_b32 a[%2], 0\n\tv_accvgpr_write_b32 a[%3], 0" ::"n"(4 * F), "n"(4 * F + 1), "n"(4 * F + 2), "n"(4 * F + 3));
}
template <int F>
__device__ __forceinline__ f32x4 acc_read() {
    f32x4 c;
    asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(c[0]) : "n"(4 * F));
    asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(c[1]) : "n"(4 * F + 1));
    asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(c[2]) : "n"(4 * F + 2));
    asm volatile("v_accvgpr_read_b32 %0, a[%1]" : "=v"(c[3]) : "n"(4 * F + 3));
    return c;
}

// The block tile: 256 activation rows x BN weight rows over 64-wide K slabs, 2 x 2 waves.
//
// LDS rows are 128 bytes (64 bf16).  They are filled by direct global->LDS loads: one wave-wide load writes
// 1 KB of consecutive LDS (64 lanes x 16 bytes = 8 rows), and each lane chooses WHICH 16-byte piece of its
// row it fetches, so that piece kc of row r lands at position kc ^ ((r >> 1) & 7): with the 64 LDS banks of
// this chip, the 16 lanes that a 16-byte read serves per cycle then fall into 16 different bank groups, for
// the fill as well as for the operand reads.  Lane l reads row (l & 15), piece (l >> 4) of a k-step and ends
// with output columns 4*(l >> 4) .. +3 of activation row (l & 15) of each 16 x 16 sub-tile.
//
// The waves of a column take the 16-row activation sub-tiles in turn, so that a partly filled tile keeps all four waves
// multiplying: its time follows its rows in steps of 32.  (With halves of a tile instead, 128 x 2048 x 768 with 129 to 200
// rows on most experts 638 -> 618 us a layer, 60 x 2048 x 1408 with at most 127 227 -> 224.)
//
// SWIGLU: weight rows [0,BN/2) of the tile come from W_gate, [BN/2,BN) from W_up, for the same BN/2 hidden
// columns; a wave holds matching gate and up columns and applies silu(g)*u itself.
template <int BN_, bool SWIGLU_>
struct Shape {
    static constexpr int BM = kFfnTileM, BN = BN_, NW = 4, BK = 64;
    static constexpr bool SWIGLU = SWIGLU_;
    static constexpr int kThreads = 64 * NW;
    static constexpr int kNCols = SWIGLU ? BN / 2 : BN;  // output columns of a block
    static constexpr int TM = BM / 2 / 16, TN = BN / 2 / 16;
    static constexpr int A_LOADS = BM / 8 / NW, B_LOADS = BN / 8 / NW;  // wave-wide loads of eight 128-byte rows per slab
    static constexpr int A_SLOT = BM * 128, B_SLOT = BN * 128, B_BASE = 2 * A_SLOT;
    static constexpr int kLdsBytes = 2 * A_SLOT + 3 * B_SLOT;
    // Slabs in LDS for a tile of `live` x 32 rows: up to five of these, activations and weights of a slab lie side by side in a
    // ring of three slots, up to two in a ring of four; above, two slots of activations and three of weights.
    static constexpr int kRingLive = 5;
    static __host__ __device__ constexpr int ring(int live) { return live <= 2 ? 4 : (live <= kRingLive ? 3 : 2); }
    static __host__ __device__ constexpr int a_stride(int live) { return live <= kRingLive ? live * 4096 + B_SLOT : A_SLOT; }
    static __host__ __device__ constexpr int b_stride(int live) { return live <= kRingLive ? live * 4096 + B_SLOT : B_SLOT; }
    static __host__ __device__ constexpr int b_base(int live) { return live <= kRingLive ? live * 4096 : B_BASE; }
    static_assert(4 * (2 * 4096 + B_SLOT) <= kLdsBytes && 3 * (kRingLive * 4096 + B_SLOT) <= kLdsBytes, "rings");
    static constexpr int TNO = SWIGLU ? TN / 2 : TN;  // 16-column output sub-tiles of a wave
    static constexpr int fragment(int i, int j) { return i * TM + j; }  // of weight sub-tile i, activation sub-tile j
    static_assert(TNO % 2 == 0 && B_LOADS % 2 == 0, "sub-tiles leave in pairs; a load must not straddle two tensors");
};

// Which part of the product a block does next (uniform over the block).
struct WorkItem {
    int valid;
    int e, row0, rows, n0;  // output rows [row0, row0 + rows) of expert e, output columns from n0
    int first, slabs;       // its K slabs (all of them unless the item is cut along K)
    int turn;               // the slab of these that the walk begins with (it wraps around)
    int once;               // the weights are fetched with the non-temporal policy
    int slices, slice;      // units of an item that is cut along K (1: not cut)
    int unit, stride;       // where this unit's partial tile lies: unit of slice 0, units between slices
    int ticket;             // index of the item's ticket
    int short_unit;         // its partial tiles are in the region of the short items
};

// What a wave needs to request its pieces of a K slab: one buffer descriptor per operand tensor (the
// block's activation rows, its weight rows, and for SwiGLU tiles the up-projection rows) and one 32-bit
// byte offset per wave-wide load.  The loads are MUBUF loads with an LDS destination: unlike the global
// (FLAT-encoded) form, the compiler does not count them against the LDS counter, so the operand reads of the
// matrix loop keep fine-grained waits; the K advance goes into the scalar offset.
// Each descriptor opens the block's own window of a tensor (its activation rows, its weight rows), so
// 32-bit byte offsets suffice whatever the tensor size; with a gather list the window is the whole
// unpermuted input, whose size the host checks.
template <class S>
struct Fills {
    __amdgpu_buffer_rsrc_t a, b0, b1;
    uint32_t va[S::A_LOADS], vb[S::B_LOADS];
    int first, slabs, turn;
    uint8_t* smem;
    int wv;

    __device__ __forceinline__ void weights_of_lane(int lane, int K) {  // the same for every item
#pragma unroll
        for (int i = 0; i < S::B_LOADS; ++i) {
            const int r = (wv + S::NW * i) * 8 + lane / 8, kc = (lane % 8) ^ ((r >> 1) & 7);
            const int rb = S::SWIGLU && r >= S::BN / 2 ? r - S::BN / 2 : r;  // the up-projection rows of the same hidden columns
            vb[i] = ((uint32_t)rb * (uint32_t)K + kc * 8) * 2u;
        }
    }
    __device__ __forceinline__ void aim(const WorkItem& w, const uint16_t* A, const uint16_t* B0, const uint16_t* B1,
                                        const int32_t* gather, int lane, int K, int Nout) {
        a = __builtin_amdgcn_make_buffer_rsrc((void*)(gather ? A : A + (size_t)w.row0 * K), 0, -1, kRsrcFlags);
        b0 = __builtin_amdgcn_make_buffer_rsrc((void*)(B0 + ((size_t)w.e * Nout + w.n0) * K), 0, -1, kRsrcFlags);
        b1 = S::SWIGLU ? __builtin_amdgcn_make_buffer_rsrc((void*)(B1 + ((size_t)w.e * Nout + w.n0) * K), 0, -1, kRsrcFlags) : b0;
        first = w.first;
        slabs = w.slabs;
        turn = w.turn;
        uint32_t row[S::A_LOADS];
#pragma unroll
        for (int i = 0; i < S::A_LOADS; ++i) {
            const int r = (wv + S::NW * i) * 8 + lane / 8;
            const int rr = r < w.rows ? r : w.rows - 1;  // rows past the expert's end repeat its last row
            row[i] = gather ? (uint32_t)gather[w.row0 + rr] : (uint32_t)rr;
        }
#pragma unroll
        for (int i = 0; i < S::A_LOADS; ++i) {
            const int r = (wv + S::NW * i) * 8 + lane / 8, kc = (lane % 8) ^ ((r >> 1) & 7);
            va[i] = (row[i] * (uint32_t)K + kc * 8) * 2u;
        }
    }
    __device__ __forceinline__ uint32_t k_bytes(int kt) const {
        kt += turn;
        kt = kt < slabs ? kt : kt - slabs;
        return (uint32_t)(kt + first) * (S::BK * 2);
    }
    // load i of slab kt's activations / weights into the slot that begins at byte `slot` of LDS
    __device__ __forceinline__ void one_a(int i, int kt, int slot) const {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(a, (lptr_t)(smem + slot + (wv + S::NW * i) * 1024), 16, va[i], k_bytes(kt), 0, 0);
    }
    __device__ __forceinline__ void one_b(int i, int kt, int slot, bool once) const {
        // i and once are compile-time constants after unrolling
        uint8_t* dst = smem + slot + (wv + S::NW * i) * 1024;
        const __amdgpu_buffer_rsrc_t r = S::SWIGLU && i >= S::B_LOADS / 2 ? b1 : b0;
        if (once)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lptr_t)dst, 16, vb[i], k_bytes(kt), 0, 2);  // bit 1: non-temporal
        else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lptr_t)dst, 16, vb[i], k_bytes(kt), 0, 0);
    }
    // The first slabs of an item, as many as its loop keeps in LDS.  Returns how many requests are younger than those of the
    // first slab.
    __device__ __forceinline__ int start(int live, bool once) const {
        const int n = min(S::ring(live), slabs);
        for (int kt = 0; kt < n; ++kt) {
            const int sa = kt * S::a_stride(live), sb = S::b_base(live) + kt * S::b_stride(live);
            if (once) {
#pragma unroll
                for (int i = 0; i < S::B_LOADS; ++i) one_b(i, kt, sb, true);
            } else {
#pragma unroll
                for (int i = 0; i < S::B_LOADS; ++i) one_b(i, kt, sb, false);
            }
#pragma unroll
            for (int i = 0; i < S::A_LOADS; ++i)
                if (i < live) one_a(i, kt, sa);
            __builtin_amdgcn_sched_barrier(0);  // their order is what the waits count
        }
        return (n - 1) * (S::B_LOADS + live);
    }
};

// K loop of a wave.  A slab is two 32-wide k-steps; matrix instructions lag the operand reads by one k-step.  LIVE = number of
// 16-row activation sub-tiles per wave that are fetched and multiplied (the rest lie past the expert's last row).
//
// High tiles (LIVE above kRingLive).  LDS: two slots of activation rows, then a ring of three slots of weight rows (the
// operand that streams from HBM gets a window of up to two slabs to land):
//     k-step 0 of slab kt:  MFMAs  |  operand reads of k-step 1  |  requests for the weights of slab kt+2
//     barrier kt (slab kt+1 landed, slab kt no longer read)
//     k-step 1 of slab kt:  MFMAs  |  operand reads of slab kt+1 |  requests for the activations of slab kt+2
// Loads complete in order, so "all but the last B_LOADS" at barrier kt means the activations and weights of
// slab kt+1 have landed while the weights of slab kt+2 may still be in flight.
//
// Low tiles.  A slab takes 0.2 to 0.9 us of matrix instructions, less than a fetch takes, so what bounds them is how much a
// compute unit has in flight.  LDS: a ring of R slots (three; four up to two live sub-tiles) that hold activations and weights
// of a slab:
//     k-step 0 of slab kt:  MFMAs  |  operand reads of k-step 1
//     barrier kt (slab kt+1 landed, slabs kt+2 .. kt+R-1 may fly, slab kt no longer read)
//     k-step 1 of slab kt:  MFMAs  |  operand reads of slab kt+1 |  requests for slab kt+R
// (with the slots of the high tiles 32 rows took 33.8 us over 32 slabs, with four 29.8: 1531 tokens of 60 x 2048 x 1408)
//
// The caller has requested the first slabs (Fills::start) and waited for the first one.
//
// ONCE (layers whose weights the memory-side cache does not keep, see ffn_weights_stream): an expert's only row tile, short
// or partly filled, whose weight rows no other block reads, and the short tiles, row pieces and cut short items that run
// after the big ones.  Two things bound such a stream, measured
// on a read-only kernel with the same fills (256 rows of 128 bytes per slab, 3 GiB):
//   - blocks that walk K in step all read at the same offset of a power-of-two row pitch, i.e. from a few memory
//     channels: 4.9 TB/s at K = 4096, 5.0 at 2048; with the walk of the blocks starting at different slabs 6.3, 6.0;
//   - keeping lines that nobody reads again: with the non-temporal policy on top 7.0, 6.9 (K = 1408, whose pitch
//     spreads over the channels by itself: 6.3 -> 7.1).
// Whole layers, before -> after: 64 experts x 4096 x 1408 with 37 tokens 392 -> 346 us, with 256 tokens 431 -> 380;
// 8 experts x 4096 x 14336 with 16 tokens 503 -> 445; 60 x 2048 x 1408 with 1531 tokens 253 -> 228.
// Other tiles share their weight rows with the blocks that run beside them at the same K: neither applies (the
// policy on the short tiles of the joint list, whose experts' big tiles run beside them: 1 % slower).
template <class S, bool ONCE>
struct MatrixLoop {
    const Fills<S>& fills;
    int a_lane, b_lane;  // byte offset, inside a slot, of this lane's piece of the wave's first row (k-step 0)

    // byte offset of weight sub-tile i relative to the wave's first weight row: with SwiGLU the second half
    // of the sub-tiles are the up-projection rows of the same hidden columns
    static __device__ __forceinline__ constexpr int b_tile(int i) {
        return S::SWIGLU ? ((i / (S::TN / 2)) * (S::BN / 2) + (i % (S::TN / 2)) * 16) * 128 : i * 16 * 128;
    }

    // PHASE (0..3): where in a k-step this wave places its fill requests.  The four waves leave every barrier
    // together and run the same instruction stream; with the same placement they would hand their requests to
    // the address unit in the same few cycles, its queue fills, and the waves that wait cannot issue their
    // next matrix instruction.  Each wave therefore shifts its requests by a different number of matrix
    // instructions.
    // draw(): called with two to four slabs left.  before_last(at): called between the last two slabs; what it writes to this
    // wave's LDS from byte `at` (of a slot that is read no more) is seen by the whole block when run() returns.
    template <int LIVE, int PHASE, class D, class F>
    __device__ __forceinline__ void run(D&& draw, F&& before_last) const {
        constexpr int TN = S::TN, B_LOADS = S::B_LOADS;
        constexpr int NMFMA = TN * LIVE, NREAD = LIVE + TN;
        constexpr int R = S::ring(LIVE);
        constexpr bool RING = LIVE <= S::kRingLive;
        constexpr int A_USED = LIVE * 2 * 16 / (S::NW * 8);  // loads of eight rows a wave that hold live rows
        static_assert(A_USED == LIVE && LIVE <= S::A_LOADS, "live rows");
        constexpr int PER = B_LOADS + A_USED;  // requests per slab
        constexpr int A_STRIDE = S::a_stride(LIVE), B_STRIDE = S::b_stride(LIVE), B_BASE = S::b_base(LIVE);
        // reads go out in the first half of a k-step, so that they have returned long before the barrier
        constexpr int READ_PER = NMFMA >= 2 * NREAD ? 1 : (2 * NREAD + NMFMA - 1) / NMFMA;  // reads per MFMA that has some
        constexpr int READ_EVERY = READ_PER > 1 ? 1 : NMFMA / 2 / NREAD;
        constexpr int B_EVERY = NMFMA / B_LOADS;
        constexpr int A_EVERY = NMFMA / A_USED;
        constexpr int B_OFF = PHASE * B_EVERY / 4 + (B_EVERY >= 8 ? B_EVERY / 8 : 0);
        constexpr int A_OFF = PHASE * A_EVERY / 4 + (A_EVERY >= 8 ? A_EVERY / 8 : 0);
        static_assert(B_EVERY > 0 && A_EVERY > 0 && B_OFF < B_EVERY && A_OFF < A_EVERY, "request placement");
        constexpr int F_EVERY = NMFMA >= PER ? NMFMA / PER : 1, F_PER = (PER + NMFMA - 1) / NMFMA;  // low tiles
        static_assert(NMFMA * READ_PER >= NREAD * READ_EVERY, "k-step too short");
        bf16x8 xa[2][LIVE], wb[2][TN];
        uint8_t* const smem = fills.smem;
        const int KT = fills.slabs;
        int a_lane = this->a_lane, b_lane = this->b_lane;
        asm volatile("" : "+v"(a_lane), "+v"(b_lane));  // the first operand reads stay here, not ahead of all instances

        // r-th operand read of a k-step, in the order the MFMAs (activation sub-tile major) need them:
        // weight 0, activation 0, weights 1.., activations 1..  pa / pb: this lane's piece of the wave's first
        // activation / weight row in the slot and k-step being read.
        auto read_item = [&](int r, int set, const uint8_t* pa, const uint8_t* pb) {
            if (r == 0)
                wb[set][0] = *(const bf16x8*)(pb + b_tile(0));
            else if (r == 1)
                xa[set][0] = *(const bf16x8*)(pa);
            else if (r <= TN)
                wb[set][r - 1] = *(const bf16x8*)(pb + b_tile(r - 1));
            else
                xa[set][r - TN] = *(const bf16x8*)(pa + (r - TN) * 2 * 16 * 128);
        };
        auto reads_at = [&](int q, int set, const uint8_t* pa, const uint8_t* pb) {
            if (q % READ_EVERY != 0) return;
#pragma unroll
            for (int r = q / READ_EVERY * READ_PER; r < q / READ_EVERY * READ_PER + READ_PER; ++r)
                if (r < NREAD) read_item(r, set, pa, pb);
        };
#pragma unroll
        for (int r = 0; r < NREAD; ++r) read_item(r, 0, smem + a_lane, smem + B_BASE + b_lane);

        // One slab.  MORE: there is a next slab to read operands of; REFILL: slab kt+2 (low tiles: kt+R) exists and is
        // requested.  Compile-time, so that the steady state carries no branches between its matrix instructions; the last
        // slabs run the other instances.  sa, sb: slots of the slab's activations and weights.
        auto slab = [&](int kt, int sa, int sb, auto more_c, auto refill_c) {
            constexpr bool MORE = decltype(more_c)::value, REFILL = decltype(refill_c)::value;
            constexpr int SA = RING ? R : 2, SB = RING ? R : 3;  // slots
            const int sa1 = sa == SA - 1 ? 0 : sa + 1, sb1 = sb == SB - 1 ? 0 : sb + 1;
            const int sb2 = sb1 == SB - 1 ? 0 : sb1 + 1;
            {
                // the second k-step's pieces sit four pieces further: bit 6 of the byte offset
                const uint8_t* pa = smem + sa * A_STRIDE + (a_lane ^ 64);
                const uint8_t* pb = smem + B_BASE + sb * B_STRIDE + (b_lane ^ 64);
                each<NMFMA>([&](auto q_c) {
                    constexpr int q = decltype(q_c)::value, j = q / TN, i = q % TN;
                    acc_mfma<S::fragment(i, j)>(wb[0][i], xa[0][j]);
                    reads_at(q, 1, pa, pb);
                    if (!RING && REFILL && q % B_EVERY == B_OFF && q / B_EVERY < B_LOADS)
                        fills.one_b(q / B_EVERY, kt + 2, B_BASE + sb2 * B_STRIDE, ONCE);
                    __builtin_amdgcn_sched_barrier(0);
                });
            }
            // slab kt+1 has landed for this wave (younger requests may still fly), this wave's
            // operand reads of slab kt have returned (the LDS counter is part of the wait)
            if (REFILL)
                __builtin_amdgcn_s_waitcnt(waitcnt_vm(RING ? (R - 2) * PER : B_LOADS));
            else if (R > 3 && kt + 3 < KT)  // slabs kt+2 and kt+3 are the last
                __builtin_amdgcn_s_waitcnt(waitcnt_vm(2 * PER));
            else if (R > 2 && kt + 2 < KT)
                __builtin_amdgcn_s_waitcnt(waitcnt_vm(PER));
            else
                __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            {
                const uint8_t* pa = smem + sa1 * A_STRIDE + a_lane;
                const uint8_t* pb = smem + B_BASE + sb1 * B_STRIDE + b_lane;
                each<NMFMA>([&](auto q_c) {
                    constexpr int q = decltype(q_c)::value, j = q / TN, i = q % TN;
                    acc_mfma<S::fragment(i, j)>(wb[1][i], xa[1][j]);
                    if (MORE) reads_at(q, 0, pa, pb);
                    if (!RING && REFILL && q % A_EVERY == A_OFF && q / A_EVERY < A_USED) fills.one_a(q / A_EVERY, kt + 2, sa * A_STRIDE);
                    if (RING && REFILL && q % F_EVERY == 0)
#pragma unroll
                        for (int f = q / F_EVERY * F_PER; f < q / F_EVERY * F_PER + F_PER; ++f) {
                            if (f < B_LOADS)
                                fills.one_b(f, kt + R, B_BASE + sb * B_STRIDE, ONCE);
                            else if (f < PER)
                                fills.one_a(f - B_LOADS, kt + R, sa * A_STRIDE);
                        }
                    __builtin_amdgcn_sched_barrier(0);
                });
            }
        };
        int kt = 0, sa = 0, sb = 0;
        const std::true_type yes{};
        const std::false_type no{};
        auto advance = [&]() {
            ++kt;
            if (RING) {
                sa = sb = sb == R - 1 ? 0 : sb + 1;
            } else {
                sa ^= 1;
                sb = sb == 2 ? 0 : sb + 1;
            }
        };
        while (kt + R < KT) {
            slab(kt, sa, sb, yes, yes);
            advance();
        }
        draw();
        int at = 0;
        do {  // (an item has two slabs at least)
            slab(kt, sa, sb, yes, no);
            at = sa * A_STRIDE;
            advance();
        } while (R > 2 && kt + 1 < KT);
        before_last(at);
        __builtin_amdgcn_sched_barrier(0);
        slab(kt, sa, sb, no, no);
        // the last matrix instructions retire before anything else reads the accumulators
        asm volatile("s_nop 15\n\ts_nop 15");
    }
};

// a read-only word that is the same for the whole wave, through the scalar cache (written by earlier kernels only)
__device__ __forceinline__ int scalar_word(const int32_t* p, int i) {
    return ((const __attribute__((address_space(4))) int32_t*)(uintptr_t)p)[i];
}

// A word of LDS for another wave or from one.  (Through a generic pointer it would be a FLAT access, which waits for the
// vector-memory counter as well: the whole round trip and all younger requests, with nothing else on the SIMD to run.)
typedef __attribute__((address_space(3))) volatile int* lds_int_t;
__device__ __forceinline__ lds_int_t lds_word(uint8_t* smem, int at) { return (lds_int_t)(smem + at); }

// Decode a block's position in a list of `total` = tiles x column blocks work items, ordered
// [column group][row tile][column in group].
__device__ inline void decode_item(int logical, int nt, int col_group, int& tile, int& nb) {
    const int per_group = nt * col_group;
    const int cg = logical / per_group, rem = logical - cg * per_group;
    tile = rem / col_group;
    nb = cg * col_group + (rem - tile * col_group);
}

// The order of the work.  Every XCD (block id mod 8) gets a contiguous eighth of it, so that blocks that run together on an
// XCD share row and weight tiles in its L2, and its blocks take the next position of that eighth as they get free.
//
// split_hdr[4] set (see the tile schedule: a long launch that is never cut along K): the blocks walk the list
// that holds both kinds expert by expert, so the short tiles of an expert run next to its big tiles and their
// weight streaming overlaps matrix work.
//
// Otherwise the two lists one after the other: the XCD's eighth of the big items, then its eighth of the short
// ones (longest first; ordered by height instead, with an eighth of every height for each XCD, the items that stream weights
// no longer ran beside those that multiply: 279 -> 297 and 419 -> 456 us).  The last split_hdr[0] big items of an XCD's
// share run as split_hdr[1] units each; the units follow the XCD's whole items, slice by slice, so that the units that run
// together read the same K range of the tiles they share.  A GEMM too short in K to be cut there runs the few big items left
// over after the XCD's last full round (split_hdr[6]) as kFfnRowPieces quarters of their rows each: twice the compute-unit
// time, on compute units that would have idled, in half the item's time.
//
// The last split_hdr[5] items of the order (of the joint list, or of the short items) are not dealt out in eighths: whichever
// XCD has a compute unit free takes the next one, so that an XCD that runs a few per cent slower than the others
// (they differ) does not end the launch alone.
template <class S>
struct WorkOrder {
    const TileListArgs& L;
    int slabs, Nout, group_big, group_short, xcd;
    bool stream;
    bool joint;
    int nt_big, nt_short;        // row tiles (joint: all of them in nt_big)
    int base_big, base_short;    // first item of this XCD's eighth
    int whole, pieces, whole_s, units, units_s;  // positions of each kind, in this order
    int cut, cut_here, slices, cut_s, cut_s_here, slices_s;
    int fixed, pool;             // joint, short items: those dealt out in eighths, those shared at the end
    int few_big;                 // less than a round of big items

    __device__ __forceinline__ WorkOrder(const TileListArgs& lists, const int32_t* hdr, int K, int Nout_, int gb, int gs, bool stream_)
        : L(lists), slabs(K / S::BK), Nout(Nout_), group_big(gb), group_short(gs), xcd(blockIdx.x & 7), stream(stream_) {
        const int ncol = Nout / S::kNCols;
        // everything at once: a block that starts waits for one fetch, not for one after the other
        int h[7];
#pragma unroll
        for (int i = 0; i < 7; ++i) h[i] = scalar_word(hdr, i);
        const int n_all = scalar_word(L.u_count, 0), n_big = scalar_word(L.b_count, 0), n_short = scalar_word(L.s_count, 0);
        joint = h[4];
        pool = h[5];
        pieces = whole_s = units = units_s = 0;
        cut = cut_here = cut_s = cut_s_here = 0;
        slices = slices_s = 1;
        nt_short = base_short = fixed = few_big = 0;
        if (joint) {
            nt_big = n_all;
            fixed = nt_big * ncol - pool;
            const int chunk = (fixed + 7) >> 3;
            base_big = xcd * chunk;
            whole = max(0, min(chunk, fixed - base_big));
        } else {
            nt_big = n_big, nt_short = n_short;
            cut = h[0], slices = h[1];
            cut_s = h[2], slices_s = h[3];
            const int in_rows = h[6];
            const int total_b = nt_big * ncol, total_s = nt_short * ncol;
            fixed = total_s - pool;
            const int chunk_b = (total_b + 7) >> 3, chunk_s = (fixed + 7) >> 3;
            few_big = chunk_b <= kFfnSplitUnits / 8;
            base_big = xcd * chunk_b, base_short = xcd * chunk_s;
            const int mine = max(0, min(chunk_b, total_b - base_big)), mine_s = max(0, min(chunk_s, fixed - base_short));
            whole = min(mine, chunk_b - cut - in_rows);
            whole_s = min(mine_s, chunk_s - cut_s);
            pieces = in_rows > 0 ? (mine - whole) * kFfnRowPieces : 0;
            cut_here = cut > 0 ? mine - whole : 0, cut_s_here = mine_s - whole_s;
            units = cut_here * slices, units_s = cut_s_here * slices_s;
        }
    }
    __device__ __forceinline__ int positions() const { return whole + pieces + whole_s + units + units_s; }

    // position p of this XCD's share, or item p - kPoolItem of the shared end of the order
    static constexpr int kPoolItem = 1 << 30;
    __device__ __forceinline__ WorkItem at(int p) const {
        WorkItem w;
        w.valid = 0;
        int logical, rows_word, tile, nb, quarter = -1, alone;
        w.slices = 1, w.slice = w.unit = w.stride = w.ticket = w.short_unit = 0;
        bool is_short = false;  // of the list of short tiles
        if (p >= kPoolItem) {
            if (p - kPoolItem >= pool) return w;
            logical = fixed + p - kPoolItem;
            is_short = !joint;
        } else if (p < whole) {
            logical = base_big + p;
        } else if ((p -= whole) < pieces) {
            logical = base_big + whole + p / kFfnRowPieces;
            quarter = p % kFfnRowPieces;
        } else if ((p -= pieces) < whole_s) {
            logical = base_short + p;
            is_short = true;
        } else if ((p -= whole_s) < units) {
            w.slices = slices, w.stride = cut;
            w.slice = p / cut_here;
            const int idx = p - w.slice * cut_here;
            logical = base_big + whole + idx;
            w.unit = w.ticket = xcd * (kFfnSplitUnits / 8) + idx;
        } else if ((p -= units) < units_s) {
            w.slices = slices_s, w.stride = cut_s;
            w.slice = p / cut_s_here;
            const int idx = p - w.slice * cut_s_here;
            logical = base_short + whole_s + idx;
            w.unit = xcd * (kFfnSplitUnits / 8) + idx;
            w.ticket = kFfnSplitUnits + w.unit;
            is_short = true, w.short_unit = 1;
        } else {
            return w;
        }
        if (is_short)
            decode_item(logical, nt_short, group_short, tile, nb);
        else
            decode_item(logical, nt_big, group_big, tile, nb);
        // uniform, also where the divisions ran on the vector unit
        tile = __builtin_amdgcn_readfirstlane(tile), nb = __builtin_amdgcn_readfirstlane(nb);
        w.valid = 1;
        w.n0 = nb * S::kNCols;
        w.e = scalar_word(is_short ? L.s_expert : (joint ? L.u_expert : L.b_expert), tile);
        w.row0 = scalar_word(is_short ? L.s_row0 : (joint ? L.u_row0 : L.b_row0), tile);
        rows_word = scalar_word(is_short ? L.s_rows : (joint ? L.u_rows : L.b_rows), tile);
        w.rows = rows_word & kTileRowsMask;
        alone = stream && (rows_word & kAloneTileFlag);
        if (is_short)
            // with less than a round of big items those of the same expert run beside it and read the same weights (314 tokens,
            // all at 8 experts x 3840 x 640: 169 -> 155 us)
            w.once = stream && (alone || !few_big || w.slices > 1);
        else
            w.once = w.slices > 1 ? 0 : (quarter >= 0 ? stream : alone);
        if (quarter >= 0) {  // a big tile has more than 64 rows: no quarter is empty
            const int from = quarter * w.rows / kFfnRowPieces, to = (quarter + 1) * w.rows / kFfnRowPieces;
            w.row0 += from;
            w.rows = to - from;
        }
        w.first = 0;
        w.slabs = slabs;
        if (w.slices > 1) {  // (a division is forty instructions, and nothing runs beside a launch's first look-up)
            w.first = w.slice * slabs / w.slices;
            w.slabs = (w.slice + 1) * slabs / w.slices - w.first;
        }
        // The start of the walk depends on the output columns alone and only moves where the expert has a single tile: in a
        // GEMM that is not cut along K a row's sums run in the same order whatever other experts share the launch.  (Which
        // items are cut follows from the tiles of all experts.)
        w.turn = alone && w.once ? (int)((long long)w.n0 * w.slabs / Nout) : 0;
        return w;
    }
};

// Writes sub-tile row j (16 rows of this wave) of a block's output tile: a lane holds 4 consecutive columns of a row in each
// sub-tile; the lanes exchange halves between two sub-tiles (v_permlane16_swap), hold 16 bytes each, and a wave's store writes
// 64 consecutive bytes of 16 rows.  Nothing passes through LDS, which by then receives the next item's first slabs.  Rows past
// the tile's end lie past the end of the descriptor's window and are not written: the number of stores is the same for all.
template <class S>
struct TileWriter {
    __amdgpu_buffer_rsrc_t c;
    uint32_t at;      // byte offset of this lane's first column in row 0
    uint32_t pitch;   // bytes of a row
    __device__ __forceinline__ TileWriter(uint16_t* C, const WorkItem& w, int Nout, int wm, int wn, int lane) {
        c = __builtin_amdgcn_make_buffer_rsrc((void*)(C + (size_t)w.row0 * Nout + w.n0), 0,
                                              ((w.rows - 1) * Nout + S::kNCols) * 2, kRsrcFlags);
        const int lr = lane & 15, lk = lane >> 4;
        pitch = (uint32_t)Nout * 2u;
        at = (uint32_t)(wm * 16 + lr) * pitch + (uint32_t)(wn * (S::kNCols / 2) + (lk & 1) * 16 + (lk >> 1) * 8) * 2u;
    }
    template <class Frag>
    __device__ __forceinline__ void rows(int j, Frag&& frag) const {  // frag(i): sub-tile i's values, i a compile-time argument
        each<S::TNO / 2>([&](auto pair_c) {
            constexpr int i = 2 * decltype(pair_c)::value;
            uint32_t half[2][2];
            each<2>([&](auto s_c) {
                constexpr int s = decltype(s_c)::value;
                const f32x4 g = frag(std::integral_constant<int, i + s>{});
                float o[4];
                if constexpr (S::SWIGLU) {
                    const f32x4 u = frag(std::integral_constant<int, i + s + S::TNO>{});
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        o[v] = g[v] * u[v] * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(g[v] * -1.4426950408889634f));
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v) o[v] = g[v];
                }
                half[s][0] = pack_bf16x2(o[0], o[1]);
                half[s][1] = pack_bf16x2(o[2], o[3]);
            });
            const auto lo = __builtin_amdgcn_permlane16_swap(half[0][0], half[1][0], false, false);
            const auto hi = __builtin_amdgcn_permlane16_swap(half[0][1], half[1][1], false, false);
            const u32x4 out = {lo[0], hi[0], lo[1], hi[1]};
            __builtin_amdgcn_raw_buffer_store_b128(out, c, at + (uint32_t)(j * 32) * pitch + i * 32, 0, 0);
        });
    }
};

// An item cut along K: partial tiles through the workspace; of the waves that hold the same part of the item's units, the last
// one to finish adds them and writes the output.
// The units of an item may run on different XCDs, whose L2 caches do not see each other's lines.  A fence
// that writes back and invalidates a whole L2 per unit costs more than the cut saves, so the partial tiles
// are stored and loaded with device-scope cache policy instead (written through to memory, read around
// caches that may be stale), each store is acknowledged before the ticket is taken, and the ticket is a
// device-scope atomic (a byte of it for each of the four waves).
template <class S>
__device__ __forceinline__ void finish_unit(const WorkItem& w, const TileWriter<S>& out,
                                            float* split_partial, int32_t* split_counter, int wv, int lane, int live) {
    constexpr int TN = S::TN, TM = S::TM;
    // a unit's partial tile is stored in register order (fragment, lane): whole 1 KB lines per wave store
    const size_t unit_floats = (size_t)(w.short_unit ? kFfnTileSmall : S::BM) * S::BN;
    float* item = split_partial + (w.short_unit ? (size_t)kFfnSplitUnits * kFfnTileM * 256 : 0) + (size_t)w.unit * unit_floats;
    // (a short item has two live sub-tiles at most: its fragments are packed)
    const int height = w.short_unit ? kFfnTileSmall / 32 : TM;
    const uint32_t at = (uint32_t)((wv * TN * height * 64 + lane) * 16);  // + fragment * 1024 bytes
    {
        const __amdgpu_buffer_rsrc_t mine = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(item + (size_t)(w.slice * w.stride) * unit_floats), 0, -1, kRsrcFlags);
        each<TM>([&](auto j_c) {
            constexpr int j = decltype(j_c)::value;
            if (j < live)
                each<TN>([&](auto i_c) {
                    constexpr int i = decltype(i_c)::value;
                    const f32x4 v = acc_read<S::fragment(i, j)>();
                    __builtin_amdgcn_raw_buffer_store_b128(*(const u32x4*)&v, mine, at + (j * TN + i) * 1024, 0, kDeviceScope);
                });
        });
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));  // every store of this lane has been acknowledged
    int order = 0;
    if (lane == 0) order = __hip_atomic_fetch_add(split_counter + w.ticket, 1 << (8 * wv), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    order = (__builtin_amdgcn_readfirstlane(order) >> (8 * wv)) & 255;
    if (order != w.slices - 1) return;  // another unit of this item finishes later and does the sum
    const __amdgpu_buffer_rsrc_t all = __builtin_amdgcn_make_buffer_rsrc((void*)item, 0, -1, kRsrcFlags);
    const uint32_t unit_bytes = (uint32_t)(w.stride * unit_floats * 4);
#pragma unroll 1
    for (int j = 0; j < live; ++j) {
        f32x4 sum[TN];
#pragma unroll
        for (int i = 0; i < TN; ++i) sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int s0 = 0; s0 < w.slices; s0 += 4) {  // slice order, whichever unit does it: the same sum every run
            // four slices in flight at a time: a load that goes around the caches takes microseconds
            u32x4 q[4][TN];
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < TN; ++i)
                    q[t][i] = __builtin_amdgcn_raw_buffer_load_b128(
                        all, at + (j * TN + i) * 1024, (uint32_t)(s0 + t < w.slices ? s0 + t : s0) * unit_bytes, kDeviceScope);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (s0 + t < w.slices) {
#pragma unroll
                    for (int i = 0; i < TN; ++i) sum[i] += *(const f32x4*)&q[t][i];
                }
        }
        out.rows(j, [&](auto i_c) { return sum[decltype(i_c)::value]; });
    }
}

// Waits until at most n memory operations of this wave are outstanding (the instruction takes a constant).
__device__ __forceinline__ void wait_for_all_but(int n) {
    switch (n) {
#define CAPMOE_WAIT(k) \
    case k: __builtin_amdgcn_s_waitcnt(waitcnt_vm(k)); break;
#define CAPMOE_WAIT8(k) \
    CAPMOE_WAIT(k) CAPMOE_WAIT(k + 1) CAPMOE_WAIT(k + 2) CAPMOE_WAIT(k + 3) CAPMOE_WAIT(k + 4) CAPMOE_WAIT(k + 5) \
    CAPMOE_WAIT(k + 6) CAPMOE_WAIT(k + 7)
        CAPMOE_WAIT8(0) CAPMOE_WAIT8(8) CAPMOE_WAIT8(16) CAPMOE_WAIT8(24) CAPMOE_WAIT8(32) CAPMOE_WAIT8(40) CAPMOE_WAIT8(48)
        CAPMOE_WAIT8(56)
#undef CAPMOE_WAIT8
#undef CAPMOE_WAIT
        default: __builtin_amdgcn_s_waitcnt(waitcnt_vm(0)); break;
    }
}

// Tickets of the blocks of an XCD lie in the last of its split units' tickets, that of the shared end in the last ticket of
// the short items: at most kFfnSplitUnits / 8 - 1 items of an XCD are cut (what is left after full rounds).
constexpr int kXcdTicket = kFfnSplitUnits / 8 - 1, kPoolTicket = kFfnSplitUnits + kFfnSplitUnits / 8 - 1;

// One block per compute unit, for the whole launch: it requests the first slabs of its next item before it writes the
// output of the last, so that an item's start (its tile's description, then the first slabs: two to four microseconds in which
// a block of its own would only wait) hides behind the output of the one before, and no blocks without work have to be
// started and ended on every compute unit.  With a block per item and the output through LDS an item of 256 rows and 32 slabs
// took 46 us of loop, 5 of output and 4 between it and the next; now 45, 3.5 and 3.  Layers of 60 x 2048 x 1408 with 1531
// tokens 222 -> 219 us, 64 x 2048 x 1024 with 4096 285 -> 283 and with 3000 in separate calls 430 -> 419, 128 x 2048 x 768 with
// 16384 596 -> 580.
template <class S>
__global__ __launch_bounds__(S::kThreads) void ffn_gemm_bf16_kernel(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ B0, const uint16_t* __restrict__ B1,
    uint16_t* __restrict__ C, const int32_t* __restrict__ gather, const TileListArgs L, int K, int Nout,
    int col_group_big, int col_group_small, const int32_t* __restrict__ split_hdr, float* split_partial,
    int32_t* split_counter, int stream) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    if constexpr (S::TN * S::TM == 64)
        asm volatile("" ::: "a255");  // the kernel has all accumulation registers
    else
        asm volatile("" ::: "a127");
    static_assert(S::TN * S::TM == 64 || S::TN * S::TM == 32, "accumulators");
    const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wv >> 1, wn = wv & 1;
    int per_xcd = gridDim.x >> 3;
    asm volatile("" : "+s"(per_xcd));  // kept, not fetched again with every ticket
    const WorkOrder<S> order(L, split_hdr, K, Nout, col_group_big, col_group_small, stream);
    int place = blockIdx.x >> 3;
    if (order.pool > 0 && place >= order.positions()) {
        // No position of the XCD's share is left for this block (big items that do not divide by eight): it starts in the
        // shared end.  258 big and 120 short items, 768 x 384: 95.5 -> 94.8 us for both products.
        if (wv == 0) {
            int n = 0;
            if (lane == 0)
                n = WorkOrder<S>::kPoolItem +
                    __hip_atomic_fetch_add(split_counter + kPoolTicket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            n = __builtin_amdgcn_readfirstlane(n);
            if (lane < S::NW) *lds_word(smem, lane * 1024) = n;  // a copy per wave, in the quarter that only it overwrites
        }
        __syncthreads();
        place = __builtin_amdgcn_readfirstlane(*lds_word(smem, wv * 1024));
    }
    WorkItem cur = order.at(place);
    if (!cur.valid) return;
    // Whether a block may find another item.  In a launch of no more items than compute units it does not, and draws and hands
    // over nothing (512 tokens on 4 experts of 2048 x 1024, even and skewed, 66.3 -> 65.4 and 80.0 -> 79.1 us for both products).
    const bool more = order.pool > 0 || order.positions() > per_xcd;

    // ---- this lane's operand pieces: row (lane & 15) of a sub-tile, piece (lane >> 4) of a k-step ----
    // every sub-tile starts at a multiple of 16 rows, so the piece swizzle (row >> 1) & 7 depends on the
    // lane only and the sub-tiles differ by constant offsets
    const int lr = lane & 15, lk = lane >> 4;
    const int piece0 = (lk ^ ((lr >> 1) & 7)) << 4;
    const int a_lane = (wm * 16 + lr) * 128 + piece0;
    const int b_lane = ((S::SWIGLU ? wn * (S::BN / 4) : wn * (S::BN / 2)) + lr) * 128 + piece0;

    Fills<S> fills;
    fills.smem = smem;
    fills.wv = wv;
    fills.weights_of_lane(lane, K);
    fills.aim(cur, A, B0, B1, gather, lane, K, Nout);
    // memory operations of this wave that are younger than the requests for the item's first slab: those for the slabs after it,
    // and the stores of the item before; they complete in order
    int younger = fills.start((cur.rows + 31) >> 5, cur.once);
    for (;;) {
        const int live = (cur.rows + 31) >> 5;
        each<S::TM>([&](auto j_c) {
            if (decltype(j_c)::value < live)
                each<S::TN>([](auto i_c) { acc_zero<S::fragment(decltype(i_c)::value, decltype(j_c)::value)>(); });
        });
        __builtin_amdgcn_sched_barrier(0);
        wait_for_all_but(younger);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        // The block's next position.  (The offset of zero is one that the compiler takes for a value per lane: with an address
        // that is the same in all lanes it would wait for the ticket at once, to hand it to the whole wave.)
        int next = __builtin_nondeterministic_value(0), none = 0, handed = 0;
        asm volatile("" : "+v"(none));
        auto draw = [&]() {
            if (more && tid == 0)
                next = __hip_atomic_fetch_add(split_counter + (blockIdx.x & 7) * (kFfnSplitUnits / 8) + kXcdTicket + none, 1,
                                              __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        // Every wave gets a copy of it.  Slots begin at multiples of 4 KB, of which wave w's own requests fill the w-th quarter:
        // no other wave's requests for the next item overwrite what this one has not read yet.
        auto hand_over = [&](int at) {
            handed = at + wv * 1024;
            if (more && wv == 0) {
                int n = 0;
                if (lane == 0) {
                    n = next + per_xcd;
                    if (order.pool > 0 && n >= order.positions())
                        n = WorkOrder<S>::kPoolItem + __hip_atomic_fetch_add(split_counter + kPoolTicket, 1, __ATOMIC_RELAXED,
                                                                             __HIP_MEMORY_SCOPE_AGENT);
                }
                n = __builtin_amdgcn_readfirstlane(n);
                if (lane < S::NW) *lds_word(smem, at + lane * 1024) = n;
            }
        };
        auto loop = [&](auto once_c) {
            const MatrixLoop<S, decltype(once_c)::value> m{fills, a_lane, b_lane};
            switch (live) {
                case 8:
                    switch (wv) {
                        case 0: m.template run<8, 0>(draw, hand_over); break;
                        case 1: m.template run<8, 1>(draw, hand_over); break;
                        case 2: m.template run<8, 2>(draw, hand_over); break;
                        default: m.template run<8, 3>(draw, hand_over); break;
                    }
                    break;
                case 7: m.template run<7, 0>(draw, hand_over); break;
                case 6: m.template run<6, 0>(draw, hand_over); break;
                case 5: m.template run<5, 0>(draw, hand_over); break;
                case 4: m.template run<4, 0>(draw, hand_over); break;
                case 3: m.template run<3, 0>(draw, hand_over); break;
                case 2: m.template run<2, 0>(draw, hand_over); break;
                default: m.template run<1, 0>(draw, hand_over); break;
            }
        };
        if (cur.once)
            loop(std::true_type{});
        else
            loop(std::false_type{});
        WorkItem nxt;
        nxt.valid = 0;
        if (more) nxt = order.at(__builtin_amdgcn_readfirstlane(*lds_word(smem, handed)));
        younger = 0;
        if (nxt.valid) {
            fills.aim(nxt, A, B0, B1, gather, lane, K, Nout);
            younger = fills.start((nxt.rows + 31) >> 5, nxt.once);
        }
        const TileWriter<S> out(C, cur, Nout, wm, wn, lane);
        if (cur.slices > 1) {
            finish_unit<S>(cur, out, split_partial, split_counter, wv, lane, live);  // (its stores, if any, are not counted)
        } else {
            each<S::TM>([&](auto j_c) {
                constexpr int j = decltype(j_c)::value;
                if (j < live)
                    out.rows(j, [&](auto i_c) { return acc_read<S::fragment(decltype(i_c)::value, j)>(); });
            });
            younger += live * (S::TNO / 2);
        }
        if (!nxt.valid) return;
        cur = nxt;
    }
}

// The three tile lists of a workspace as the kernels take them; joint == false leaves the joint list unwritten
// (the fp32 kernels walk the list of big tiles only).
static TileListArgs tile_list_args(const FfnWorkspace& ws, bool joint) {
    return TileListArgs{ws.big.expert, ws.big.row0,  ws.big.rows,      ws.big.count,       ws.small.expert,
                        ws.small.row0, ws.small.rows, ws.small.count,   ws.big.max_tiles,   ws.small.max_tiles,
                        ws.all.expert, ws.all.row0,  ws.all.rows,      ws.all.count,       joint ? ws.all.max_tiles : 0};
}

static int column_group(int nb_total) {
    for (int g = 4; g > 1; --g)
        if (nb_total % g == 0) return g;
    return 1;
}

template <int BN, bool SWIGLU>
static void launch_bf16(bool stream, const void* A, const void* B0, const void* B1, void* C, const int32_t* gather,
                        const FfnWorkspace& ws, int K, int Nout, const int32_t* split_hdr, int32_t* split_counter,
                        hipStream_t st) {
    using S = Shape<BN, SWIGLU>;
    auto kern = ffn_gemm_bf16_kernel<S>;
    static std::atomic<uint64_t> configured{0};
    once_per_device(configured, [&] {
        (void)hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, S::kLdsBytes);
    });
    const int nb = Nout / S::kNCols;
    // a block per compute unit, the same number on every XCD; fewer where the plan cannot hold as many items (an item cut
    // along K or into row pieces is eight at most)
    const int per_xcd = std::max(1, compute_units() / 8);
    const long long items = (long long)kFfnSplitMaxSlices * nb * ((long long)ws.big.max_tiles + ws.small.max_tiles);
    const int grid = 8 * (int)std::min<long long>(per_xcd, (items + 7) / 8);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(S::kThreads), S::kLdsBytes, st, (const uint16_t*)A,
                       (const uint16_t*)B0, (const uint16_t*)B1, (uint16_t*)C, gather, tile_list_args(ws, true), K, Nout,
                       // short items that stream: all column blocks of a tile in a row, so that those that run together
                       // start their walks over K at different slabs (they share activation rows only)
                       column_group(nb), stream ? nb : column_group(nb), split_hdr, ws.split_partial, split_counter, (int)stream);
}

// The arguments of the tile schedule for a descriptor and its workspace layout (host side).
FfnScheduleArgs ffn_schedule_args(const moe_desc_t& d, const FfnWorkspace& ws, int cus) {
    const bool bf16 = d.dtype == MOE_DTYPE_BF16;
    const int K1 = d.d_model, N1 = d.d_hidden, K2 = d.d_hidden, N2 = d.d_model;
    const int bn_down = N2 % 256 == 0 ? 256 : 128;
    auto log2i = [](int v) {
        int sh = 0;
        while ((1 << sh) < v) ++sh;
        return sh;
    };
    FfnScheduleArgs a;
    a.enabled = 1;
    a.E = d.n_experts;
    a.big_sh = log2i(ws.big.tile_m);
    a.small_sh = log2i(ws.small.tile_m);
    a.small_max = ws.small_max;
    a.cus = cus;
    a.L = tile_list_args(ws, bf16);
    // gate/up: a big item covers 128 hidden columns (gate and up rows of them)
    const bool split = bf16;
    a.first = SplitArgs{split ? ws.split_hdr : nullptr, split ? ws.split_counter : nullptr, N1 / 128, N1 / 128, K1 / 64};
    a.second = SplitArgs{split ? ws.split_hdr + kFfnSplitHdr : nullptr, split ? ws.split_counter + 2 * kFfnSplitUnits : nullptr,
                         N2 / bn_down, N2 / bn_down, K2 / 64};
    return a;
}

// What the schedule decides for given per-expert row counts, on the host (moe_ffn_schedule_query).
void ffn_schedule_on_host(const moe_desc_t& d, const FfnWorkspace& ws, const int32_t* expert_count, int cus,
                          int32_t* tiles, int32_t* header) {
    FfnWorkspace layout = ws;
    int32_t hdr_gate_up[kFfnSplitHdr] = {}, hdr_down[kFfnSplitHdr] = {};
    layout.split_hdr = nullptr;  // the headers are written below, not through the workspace
    const FfnScheduleArgs a = ffn_schedule_args(d, layout, cus);
    int nb = 0, ns = 0;
    for (int e = 0; e < d.n_experts; ++e) {
        const ExpertTiles t = expert_tiles(0, expert_count[e], a.big_sh, a.small_sh, a.small_max);
        nb += t.nb;
        ns += t.ns;
    }
    if (d.dtype == MOE_DTYPE_BF16) {
        ffn_schedule_header(nb, ns, a.first.ncol_big, a.first.ncol_small, a.first.slabs, cus, true, true, hdr_gate_up);
        ffn_schedule_header(nb, ns, a.second.ncol_big, a.second.ncol_small, a.second.slabs, cus, true, true, hdr_down);
    }
    tiles[0] = nb;
    tiles[1] = ns;
    for (int i = 0; i < kFfnSplitHdr; ++i) {
        header[i] = hdr_gate_up[i];
        header[kFfnSplitHdr + i] = hdr_down[i];
    }
}

// Whether the expert weights are fetched with the streaming policy.  Weights that fit the memory-side cache (256 MB) are read
// from there by the layer's next pass unless they were: 37 tokens, 2 x 3584 x 1408 (61 MB) 50 us a pass, streaming 69; 412,
// 16 x 2944 x 768 (217 MB) 84 and 95; few rows: 16, 1 x 1024 x 14336 (88 MB) 34 and 46, 60 top-8, 32 x 1024 x 1024 (201 MB)
// 42 and 46 (from HBM 47 and 46, 48 and 46).  While they do not exceed it by much, most of what a pass uses still is there:
// 91 tokens top-1, 96 x 2048 x 256 (302 MB) 37 and 46 (50 and 47 from HBM).  256 tokens, 16 x 4096 x 1024 (403 MB) 125 and 120,
// 1000, 16 x 2048 x 2048 (403 MB) 134 and 119; 37, 64 x 4096 x 1408 (2.2 GB) 306 and 273.
bool ffn_weights_stream(const moe_desc_t& d, const Sizes& s) {
    constexpr uint64_t kKeptWeights = 320ull << 20;
    return 3ull * d.n_experts * d.d_model * d.d_hidden * s.elem > kKeptWeights;
}

// row_token == nullptr: xp holds the permuted rows.  Otherwise xp is the unpermuted x and row r of the
// plan is fetched from x[row_token[r]] (dispatch fused into the first GEMM's operand fetch).
// schedule_ready: the tile schedule is in the workspace already (built by the drop), no schedule kernel is launched.
hipError_t launch_grouped_ffn(const moe_desc_t& d, const Sizes& s, const FfnWorkspace& ws, const void* xp,
                              const int32_t* row_token, const int32_t* expert_offset, const void* w_gate,
                              const void* w_up, const void* w_down, void* yp, bool schedule_ready, hipStream_t st) {
    const int K1 = d.d_model, N1 = d.d_hidden, K2 = d.d_hidden, N2 = d.d_model;
    const bool bf16 = d.dtype == MOE_DTYPE_BF16;
    const int bn_down = N2 % 256 == 0 ? 256 : 128;  // d is a multiple of 128 at least: output columns per block
    if (!schedule_ready) {
        ProfileScope prof(MOE_KERNEL_FFN_SCHEDULE, st);
        hipLaunchKernelGGL(ffn_schedule_kernel, dim3(1), dim3(64), 0, st, expert_offset, ffn_schedule_args(d, ws, compute_units()));
    }
    if (ffn_is_thin(d, s)) {
        launch_ffn_thin(d, s, ws, xp, row_token, w_gate, w_up, w_down, yp, st);
    } else if (bf16) {
        const int32_t* split_gu = ws.split_hdr;
        const int32_t* split_dn = ws.split_hdr + kFfnSplitHdr;
        int32_t* tickets_dn = ws.split_counter + 2 * kFfnSplitUnits;
        const bool stream = ffn_weights_stream(d, s);
        {
            ProfileScope prof(MOE_KERNEL_FFN_GATE_UP, st);
            launch_bf16<256, true>(stream, xp, w_gate, w_up, ws.hidden, row_token, ws, K1, N1, split_gu, ws.split_counter, st);
        }
        ProfileScope prof(MOE_KERNEL_FFN_DOWN, st);
        if (bn_down == 256)
            launch_bf16<256, false>(stream, ws.hidden, w_down, nullptr, yp, nullptr, ws, K2, N2, split_dn, tickets_dn, st);
        else
            launch_bf16<128, false>(stream, ws.hidden, w_down, nullptr, yp, nullptr, ws, K2, N2, split_dn, tickets_dn, st);
    } else {
        launch_ffn_gate_up_f32(d, s, ws, xp, row_token, w_gate, w_up, st);
        launch_ffn_down_f32(d, s, ws, w_down, yp, st);
    }
    return hipGetLastError();
}

}  // namespace capmoe
