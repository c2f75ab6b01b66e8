// bf16 matrix-core GEMM for the Newton-Schulz iteration of Muon (the optimizer the paper pairs AdaGC with in
// "Optimizer Compatibility: Muon and Lion", Sec. 5.4), for gfx950.
//
//   C[i][j] = bf16( alpha * sum_k P[i][k] * Q[j][k]  +  beta * D[i][j] )            ("NT": both operands K-contiguous)
//
// P is M x K, Q is N x K, both row-major bf16 with K contiguous, which is the layout the matrix-core
// instruction wants for both operands: every lane's fragment is 16 contiguous bytes.  The result is written row-major (C),
// transposed (Ct, N x M), or both; D is read through its transpose Dt (N x M).  The three products of a Newton-Schulz step are
//   A  = X X^T                P = Q = X                       (alpha 1, beta 0)
//   B  = b A + c A A          P = Q = A (A is symmetric)      (alpha c, beta b, D = A)
//   X' = a X + B X            as X'^T = a X^T + X^T B with P = X^T, given by its transpose X, and Q = B; X is Dt, X' is Ct
// so that X is kept and written in one orientation only.  (With X and its transpose, written by each step, 12 products of
// 4096 x 14336 x 4096 took 4973 us and 24 of 768 x 3072 x 768 167 us; with X alone 4369 and 114.)
//
// A = X X^T and A A are symmetric: for those only the tiles on and below the diagonal are computed and each is
// written twice, to its place and to its mirror image, which saves about a quarter of a step's multiplications.
//
// M and N are multiples of the 128 x 128 block tile and K of 128 (two 64-deep tiles): the caller (muon.hip) keeps every matrix
// in zero-padded workspace buffers, and zero rows and columns stay zero through the iteration.
//
// Tiling: 128 x 128 block tile with 4 waves, or, where the launch has enough of them to fill the compute units,
// 256 x 256 with 8; every wave has 4 quadrants of the block tile's rows and columns, in accumulators of
// v_mfma_f32_16x16x32_bf16.  One launch can cover a batch of equal-shaped products.  Operand tiles, 64 deep, are loaded
// from global memory straight into LDS (global_load_lds_dwordx4, no staging registers), swizzled against bank conflicts, by
// halves into a ring of five places (see "Main loop").  A compute unit's workgroups stay and take tile after tile: the next
// tile's first loads are on their way while this one's results are stored (see "Between tiles").  The 256-tile kernels are at the
// register limit of 256.  The loop spills none, but those with D spill 8 registers (the one that reads P transposed 12) in the last
// operand tile of an output tile, and each of the two (three) places where they are read back waits for all of the wave's loads.

#include <algorithm>
#include <type_traits>
#include <utility>

#include "muon_internal.h"

namespace adagc {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

#define ADAGC_LDS __attribute__((address_space(3)))
#define ADAGC_CONST __attribute__((address_space(4)))

// A batch of products of one shape; matrix z of every array at its base + z times its stride (elements).
struct GemmGroup {
    const uint16_t *p, *q, *dt;
    uint16_t *c, *ct;
    int64_t stride_p, stride_q, stride_dt, stride_c, stride_ct;
    int32_t ldp, ldq, lddt, ldc, ldct;
    int32_t k;
    int32_t tiles_m, tiles_n;       // block tiles of one matrix
    int32_t tiles;                  // the ones of them that are computed (SYM: on and below the diagonal)
    int32_t all;                    // ... of the whole batch
};

// A launch: the tiles of several groups as planned (muon_plan.h), or, without a plan, of one group in their order.  The argument of a
// launch without a plan is no larger than it has to be: 1 KB of it takes 0.3 us longer to launch (a product of 128 x 128 x 128 7.0 us,
// with room for one group 6.6).
template <bool PLANNED>
struct GemmWork {
    const GemmItem* items;
    const int32_t*  first;
    float           alpha, beta;
    GemmGroup       g[PLANNED ? kMaxGroups : 1];
};

constexpr int kBK = 64;

// Two floats to bf16, round to nearest even, NaNs quieted: one instruction, with the bits of float_to_bf16_bits for every float.
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    const f32x2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// An output tile: its place in matrix z of a group.  z < 0: none.
struct TilePlace {
    int group, z, tile_m, tile_n;
};

// The tile of this workgroup in a round.  Without a plan a round is as many consecutive tiles of the batch as there are
// workgroups, dealt to the 8 XCDs (workgroup b runs on XCD b mod 8, one L2 each) in contiguous eighths: the whole chip is on one
// or two matrices at a time, and what the XCDs' patches have in common comes out of the memory-side cache.  With a contiguous
// eighth of the whole batch per XCD, 8 matrices at a time, 12 products X X^T of 4096 x 14336 took 2321 us, now 2223.
// (Both kinds of launch ask for a plan: with the answer known at compile time two 256-tile kernels spill registers.)
template <bool SYM, bool PLANNED>
__device__ __forceinline__ TilePlace tile_of_workgroup(const ADAGC_CONST GemmWork<PLANNED>& w, int round)
{
    const int wg = (int)blockIdx.x;
    if (w.items) {
        const ADAGC_CONST int32_t* first = (const ADAGC_CONST int32_t*)w.first;
        const int i = first[wg] + round;
        if (i >= first[wg + 1]) return {0, -1, 0, 0};
        const u32x2v item = *(const ADAGC_CONST u32x2v*)(w.items + i);
        return {(int)(item.x & 0xFFFFu), (int)(item.x >> 16), (int)(item.y & 0xFFFFu), (int)(item.y >> 16)};
    }
    const int xcd = wg % 8, slot = wg / 8, wgs = (int)gridDim.x;                                // a multiple of 8
    const int64_t before = (int64_t)round * wgs, left = w.g[0].all - before;
    const int now = (int)(left < wgs ? left : wgs);
    const int lo = now * xcd / 8, hi = now * (xcd + 1) / 8;
    if (slot >= hi - lo) return {0, -1, 0, 0};
    const int i = (int)before + lo + slot;
    TilePlace t;
    t.group = 0;
    t.z = __builtin_amdgcn_readfirstlane(i / w.g[0].tiles);
    tile_of_matrix<SYM>(i - t.z * w.g[0].tiles, w.g[0].tiles_m, w.g[0].tiles_n, &t.tile_m, &t.tile_n);
    t.tile_m = __builtin_amdgcn_readfirstlane(t.tile_m);
    t.tile_n = __builtin_amdgcn_readfirstlane(t.tile_n);
    return t;
}
static_assert(sizeof(GemmItem) == 8, "tile_of_workgroup takes the item apart by hand");

// s_waitcnt for "at most n vector-memory operations of this wave still outstanding", nothing else waited for
#define ADAGC_WAIT_VMEM(n) __builtin_amdgcn_s_waitcnt(((n) & 0xF) | (((n) >> 4) << 14) | (7 << 4) | (0xF << 8))
// nothing is moved across this point by the compiler's instruction scheduler
#define ADAGC_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

// Wait for this wave's LDS reads, then meet the workgroup's other waves.  Unlike __syncthreads this leaves the loads
// into LDS that are still on their way alone.
__device__ __forceinline__ void barrier_keeping_loads()
{
    __builtin_amdgcn_s_waitcnt(0xF | (3 << 14) | (7 << 4) | (0 << 8));
    __builtin_amdgcn_s_barrier();
    ADAGC_SCHED_FENCE();
}

// f(integral_constant 0), ..., f(integral_constant N-1)
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// 16 bytes per lane from global memory straight into LDS: lane i's data, at base + off_i bytes (base: the same in all
// lanes), lands at lds_dst + 16 i (lds_dst: the same in all lanes).  The instruction takes the LDS byte address from
// M0, and wants one wait state after M0 is written; M0 is put back afterwards, so the compiler's own uses of it are not
// disturbed.
// Written as inline assembly rather than through the compiler's builtin so that the compiler does not track these
// loads: it would count each as outstanding in both of its memory counters ("flat" access) and, while one is, turn
// every wait for an LDS read into a wait for all LDS reads, which serialises the fragment reads with the
// multiplications.  The waits for these loads are explicit (ADAGC_WAIT_VMEM) wherever their data is needed.
__device__ __forceinline__ void load_to_lds_16(const void* base, uint32_t off, const uint16_t* lds_dst)
{
    const uint32_t lds_addr = (uint32_t)reinterpret_cast<uintptr_t>(lds_dst);      // low half of the flat address = LDS offset
    uint32_t saved_m0;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, %3\n\ts_mov_b32 m0, %0"
                 : "=&s"(saved_m0)
                 : "s"(lds_addr), "v"(off), "s"(base)
                 : "memory");
}

// The same at base + off_i with offsets that 32 bits do not hold.
__device__ __forceinline__ void load_to_lds_16(const void* base, uint64_t off, const uint16_t* lds_dst)
{
    const uint32_t lds_addr = (uint32_t)reinterpret_cast<uintptr_t>(lds_dst);
    const uint64_t at = reinterpret_cast<uintptr_t>(base) + off;
    uint32_t saved_m0;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, off\n\ts_mov_b32 m0, %0"
                 : "=&s"(saved_m0)
                 : "s"(lds_addr), "v"(at)
                 : "memory");
}

// Main loop.  What bounds it: on ordinary data the power the chip may draw (its clock falls to 1.65 - 1.75 GHz under this
// loop; 4096 x 4096 x 16384 takes 376 us on normal random operands and 294 on zeros, a library kernel 345 - 391 and 247 - 265
// on the cards tried), otherwise the time an operand load takes.
//
// The block tile's rows and columns are cut in halves: P0, P1 of P and Q0, Q1 of Q, and a wave's accumulators in the four
// quadrants P0 Q0, P0 Q1, P1 Q1, P1 Q0, in this order.  Group g of the loads is half g mod 2 of both operands of the 64-deep
// tile g / 2, and LDS is a ring of five places of a group each (32 KB with 256-tiles, 160 KB in all).  In half step h
//   h even:  P0 Q0, then P0 Q1 are multiplied while Q1 and P1 are read from group h + 1,
//   h odd:   P1 Q1, then P1 Q0, while P0 and Q0 of the next 64-deep tile are read from group h + 1,
// and group h + 5 is loaded into the place of group h, whose last reader is behind the barrier.  Every load so has three and
// a half half steps to arrive.  (With P and Q tiles whole in the ring, half of the loads had less than two half steps: on zeros
// 339 us against 295, on random operands 395 against 387, 12 products X X^T of 4096 x 14336 2520 against 2425 us.)
// One access is issued after every few multiplications: a load into LDS occupies the issue for about 16 clocks per wave.
// Q0 is read where Q1 was, so the two swap their registers from tile to tile.
//
// 16 x 16 x 32 multiplications instead of 32 x 32 x 16: half the accumulator traffic per multiplication, and so a
// higher clock (1313 -> 1343 TFLOP/s when it was introduced), and successive multiplications share an operand all the way
// through.  The results are the same bit for bit: every sum runs over k in order.
//
// Between tiles.  The last half steps have no operands left to load: the ring takes the four quadrants of D then, or, without D, the
// next tile's first four groups.  Accumulator register r of lane l is element (row (l / 16) * 4 + r, column l % 16) of its 16 x 16
// block: 8 bytes along a row of Ct.  Exchanging half of the lanes' values between two neighbouring blocks (v_permlane16_swap) makes
// 16 bytes of it, stored without a detour through LDS; C, whose rows run the other way, is transposed through the wave's own part
// of a place of the ring (ds_read_b64_tr_b16).  Where a quadrant of D has been used, the next tile's groups are loaded.  The stores
// complete during the next tile's first half steps.  (On 256-tiles the waits for spilled registers, above, come while D's last quadrants
// are on their way: those have less than three and a half half steps.)
// Measured: one workgroup per tile and all of LDS as the staging tile, 12 products of 4096 x 14336 x 4096 with D, C and Ct 4866 us,
// with workgroups that stay 4706; X X^T as above 2373, 2296.  D loaded to registers after the sums, with the waits that takes, against
// the ring: b A + c A A of 48 matrices of 768 rows on 256-tiles 61, 52 us, of 6 of 2048 rows 59, 54, a X + B X of 32 of 1024 rows
// 235, 225, of Llama-3-8B shapes 5315, 5220.
//
// PTR: P is given by its transpose, K rows of M consecutive elements (X itself in B X), and its fragments are read transposed
// (ds_read_b64_tr_b16, two for the 16 bytes of a lane).  Only Ct then.
//
// WIDE: a lane's offset from the wave's address, up to 15 rows and a few vectors, is kept in 64 bits, for rows of more than
// kNarrowRow elements (the others have no registers to spare for that).
template <int BT, bool PLANNED, bool SYM, bool PTR, bool HAS_D, bool WIDE, int kGemmThreads>
__global__ __launch_bounds__(kGemmThreads, 2) void gemm_nt_bf16_kernel(const GemmWork<PLANNED>)
{
    typedef std::conditional_t<WIDE, uint64_t, uint32_t> Offset;           // bytes
    constexpr int kWaves = kGemmThreads / 64;
    // waves in a kWM x kWN grid; with PTR the reads of P are the more expensive ones, so a wave has fewer of its rows
    constexpr int kWM = PTR ? kWaves / 2 : 2, kWN = kWaves / kWM;
    constexpr int kTM = BT / kWM, kTN = BT / kWN;          // wave tile
    constexpr int kHM = kTM / 32, kHN = kTN / 32;          // 16 x 16 accumulators per quadrant
    constexpr int kUnitElems = BT / 2 * kBK;               // half of an operand tile
    constexpr int kPlaceElems = 2 * kUnitElems;            // Q's half, then P's
    constexpr int kGL = 2 * kUnitElems / 512 / kWaves;     // loads per wave and group
    constexpr int kStores = BT * BT / 512 / kWaves;        // stores per wave of one output array
    constexpr int kQuadRow = kTM / 2;                      // a quadrant's results: kTN / 2 rows (of Ct) of kQuadRow elements
    constexpr int kDL = kStores / 4;                       // loads per wave of its part of D, per quadrant
    static_assert(kWaves % 2 == 0, "the swizzle of a load is taken from the wave's parity");
    __shared__ __attribute__((aligned(16))) uint16_t lds[5 * kPlaceElems];

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);     // the same in all lanes: kept in a scalar register
    const int wm = wave / kWN, wn = wave % kWN;
    const uint32_t lds0 = (uint32_t)reinterpret_cast<uintptr_t>(&lds[0]);
    // The arguments, read anew where a tile begins and ends: kept through the main loop they would not fit the scalar registers.
    auto arguments = []() __attribute__((always_inline)) -> const ADAGC_CONST GemmWork<PLANNED>& {
        const ADAGC_CONST GemmWork<PLANNED>* a = (const ADAGC_CONST GemmWork<PLANNED>*)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(a));
        return *a;
    };
    auto place = [&](int p) { return lds + p * kPlaceElems; };
    auto at_place = [&](int p) { return lds0 + (uint32_t)(p * kPlaceElems * 2); };
    auto next_place = [](int p) { return p == 4 ? 0 : p + 1; };
    auto previous_place = [](int p) { return p == 0 ? 4 : p - 1; };

    // Loads.  One global_load_lds_dwordx4 of a wave writes 1024 contiguous LDS bytes, lane i the i-th 16: that is 8 rows of a
    // 64-deep half tile stored without padding.  Bank conflicts of the fragment reads (16 lanes = 16 consecutive rows per
    // clock over 64 banks) are avoided by a swizzle instead: the 16-byte vector v of row r sits at position v ^ ((r / 2) mod 8)
    // of its LDS row, which the loading lane applies on the global side.  The rows of a load start at a multiple of 8, and
    // (r / 2) mod 8 = (4 (wave mod 2) + lane / 16) mod 8 because kWaves is even.
    // PTR: P's half is 64 rows (k) of BT / 2 elements, 4 (8) rows per load.  A fragment read takes 32 bytes, a block's 16 columns, of
    // 4 rows each for 16 lanes: of rows 0 .. 3 and 8 .. 11 (and 16 more) at a time.  The 32-byte unit u of row r is at position
    // u ^ swizzle_p(r), so that these lie in different banks.
    // The address is split into a part common to the wave (scalar registers) and one offset per lane.
    auto swizzle_p = [](int r) { return BT == 256 ? ((r & 3) | ((r >> 3) & 1) << 2) : (((r >> 1) & 1) | ((r >> 3) & 1) << 1); };
    constexpr int kPtrRows = 1024 / BT;                    // rows per load
    struct Source {
        const uint16_t *p, *q;
        int ldp, ldq, groups;                              // groups: of loads, a multiple of 4, at least 4
        Offset off_p, off_q;
    };
    auto source = [&](const TilePlace& t) {
        const ADAGC_CONST GemmGroup& w = arguments().g[t.group];
        int l = lane;
        asm volatile("" : "+v"(l));                        // the offsets are made here, not kept through the main loop
        const int row = l >> 3, vec = (l & 7) ^ ((((wave & 1) << 2) + (l >> 4)) & 7);
        Source s;
        s.ldp = w.ldp;
        s.ldq = w.ldq;
        s.groups = 2 * (w.k / kBK);
        s.p = w.p + (size_t)t.z * w.stride_p + (PTR ? (size_t)t.tile_m * BT : (size_t)t.tile_m * BT * w.ldp);
        s.q = w.q + (size_t)t.z * w.stride_q + (size_t)t.tile_n * BT * w.ldq;
        if constexpr (PTR) {
            constexpr int kRowLanes = BT / 16;
            const int r = l / kRowLanes;
            s.off_p = ((Offset)r * (Offset)w.ldp + (Offset)(((l % kRowLanes) ^ (2 * swizzle_p(wave * kPtrRows + r))) * 8)) * 2u;
        } else {
            s.off_p = ((Offset)row * (Offset)w.ldp + (Offset)(vec * 8)) * 2u;
        }
        s.off_q = ((Offset)row * (Offset)w.ldq + (Offset)(vec * 8)) * 2u;
        return s;
    };
    auto load = [&](const Source& s, int n, int g, uint16_t* dst) {
        const int first = ((n >> 1) * kWaves + wave) * 8, k0 = (g >> 1) * kBK;
        const size_t row = (size_t)((g & 1) * (BT / 2) + first);
        if (n & 1) {
            load_to_lds_16(s.q + row * s.ldq + k0, s.off_q, dst + first * kBK);
        } else if constexpr (PTR) {
            // kWaves kPtrRows is a multiple of 16: the swizzle does not depend on n
            const int r = ((n >> 1) * kWaves + wave) * kPtrRows;
            load_to_lds_16(s.p + (size_t)(k0 + r) * s.ldp + (g & 1) * (BT / 2), s.off_p, dst + kUnitElems + r * (BT / 2));
        } else {
            load_to_lds_16(s.p + row * s.ldp + k0, s.off_p, dst + kUnitElems + first * kBK);
        }
    };

    // A wave's quadrant in LDS, where D is loaded and results are staged: in the same 1024-byte pieces of a place that the wave loads
    // operands into, so that nobody else ever touches them.  16-byte vector c of row r is at position c ^ quad_swizzle(r): the 8
    // rows that one half of the lanes reads 32 bytes of, 0 .. 3 and 8 .. 11 of 16, lie in different banks, and so do 16 rows' vectors c.
    constexpr int kRowVecs = kQuadRow / 8, kPieceRows = 64 / kRowVecs;
    auto quad_swizzle = [](int r) {
        return kQuadRow == 64 ? (((r >> 1) & 1) * 2 | ((r >> 3) & 1) * 4 | ((r >> 2) & 1)) : (((r >> 3) & 1) * 2 | ((r >> 2) & 1));
    };
    auto quad_at = [&](uint32_t at, int r, int c) {
        const int n = r / kPieceRows;
        return at + (uint32_t)(((n & 1) ? 0 : kUnitElems * 2) + ((n >> 1) * kWaves + wave) * 1024 + (r % kPieceRows) * kQuadRow * 2 + (c ^ quad_swizzle(r)) * 16);
    };
    struct SourceD {
        const uint16_t* p;
        int ld;
    };
    auto source_d = [&](const TilePlace& t) {
        const ADAGC_CONST GemmGroup& w = arguments().g[t.group];
        SourceD s;
        s.ld = w.lddt;
        s.p = w.dt + (size_t)t.z * w.stride_dt + ((size_t)t.tile_n * BT + wn * (kTN / 2)) * w.lddt + (size_t)t.tile_m * BT + wm * (kTM / 2);
        return s;
    };
    auto load_d = [&](const SourceD& s, int n, int q, uint16_t* dst) {
        const uint16_t* from = s.p + (size_t)((q & 1) * (BT / 2) + n * kPieceRows) * s.ld + (q >> 1) * (BT / 2);
        int l = lane;
        asm volatile("" : "+v"(l));                        // made for each load: there are no registers to keep it in
        const int r = l / kRowVecs;
        const Offset off = ((Offset)r * (Offset)s.ld + (Offset)(((l % kRowVecs) ^ quad_swizzle(n * kPieceRows + r)) * 8)) * 2u;
        load_to_lds_16(from, off, dst + ((n & 1) ? 0 : kUnitElems) + ((n >> 1) * kWaves + wave) * 512);
    };

    // Fragments.  Lane l holds row l mod 16 of its 16-row block and the 16-byte vector 4 kk + l / 16 of that row; a block's first
    // row is a multiple of 16, so (row / 2) mod 8 = (l / 2) mod 8, and slice kk = 1 is 64 bytes from slice 0 by exclusive or.
    // PTR: lane l gets column l mod 16 of a block in slice kk, 8 rows from 8 (l / 16) on, and supplies the address of 4 columns in
    // one of them; block i is 32 i bytes away by exclusive or, slices and rows by addition.
    // The addresses in the place that is read are made once per half step (opaque, so that what is left of them is immediate).
    const uint32_t frag = (uint32_t)((lane & 15) * kBK * 2 + (((lane >> 4) ^ ((lane >> 1) & 7)) * 16));
    const uint32_t frag_q = frag + (uint32_t)(wn * (kTN / 2) * kBK * 2);
    const int ptr_row = 8 * (lane >> 4) + ((lane >> 2) & 3);
    const uint32_t frag_p = PTR ? (uint32_t)(kUnitElems * 2 + ptr_row * BT + ((wm * kHM) ^ swizzle_p(ptr_row)) * 32 + (lane & 3) * 8)
                                : frag + (uint32_t)((kUnitElems + wm * (kTM / 2) * kBK) * 2);
    constexpr int kPA = PTR ? kHM : 2;
    auto addresses_p = [](uint32_t offset, uint32_t at, uint32_t (&a)[kPA]) {
#pragma unroll
        for (int i = 0; i < kPA; ++i) {
            a[i] = (offset ^ (uint32_t)(i * (PTR ? 32 : 64))) + at;
            asm("" : "+v"(a[i]));
        }
    };
    auto addresses_q = [](uint32_t offset, uint32_t at, uint32_t (&a)[2]) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            a[kk] = (offset ^ (uint32_t)(kk * 64)) + at;
            asm("" : "+v"(a[kk]));
        }
    };
    auto read = [](const uint32_t (&a)[2], int block, int kk) {
        return *reinterpret_cast<const ADAGC_LDS bf16x8*>(a[kk] + (uint32_t)(block * 16 * kBK * 2));
    };
    auto read_p = [&](const uint32_t (&a)[kPA], int block, int kk) {
        if constexpr (PTR) {
            const uint32_t at = a[block] + (uint32_t)(kk * 32 * BT);
            const s16x4 x = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<ADAGC_LDS s16x4*>(at));
            const s16x4 y = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<ADAGC_LDS s16x4*>(at + 4u * BT));
            return __builtin_bit_cast(bf16x8, __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7));
        } else {
            return read(a, block, kk);
        }
    };

    f32x4 acc[2 * kHM][2 * kHN];
    bf16x8 p0[kHM][2], p1[kHM][2], qa[kHN][2], qb[kHN][2];
    constexpr int S = 2 * kHM * kHN;                       // multiplications per quadrant and 64-deep tile
    constexpr std::integral_constant<int, 0> no{};
    constexpr std::integral_constant<int, 1> yes{};
    // A half step: PART 0 multiplies P0 Q0 (qx), P0 Q1 (qy), PART 1 P1 Q1 (qy), P1 Q0 (qx).  READ: what the next one needs is
    // read from the place at rd.  side(t) is called after multiplication t.
    auto half = [&](auto PART, auto READ, bf16x8 (&qx)[kHN][2], bf16x8 (&qy)[kHN][2], uint32_t rd, auto&& side) __attribute__((always_inline)) {
        constexpr int part = decltype(PART)::value;
        uint32_t pa[kPA], qd[2];
        if constexpr (decltype(READ)::value) {
            addresses_p(frag_p, rd, pa);
            addresses_q(frag_q, rd, qd);
        }
        static_for<2 * S>([&](auto T) __attribute__((always_inline)) {
            constexpr int t = decltype(T)::value;
            constexpr int u = t % S, kk = u / (kHM * kHN), v = u % (kHM * kHN);
            constexpr int j = v / kHM, i = (j + kk) % 2 ? kHM - 1 - v % kHM : v % kHM;      // rows up and down in turn
            constexpr bool use_y = part ^ (t / S);
            constexpr int ai = part * kHM + i, aj = (use_y ? kHN : 0) + j;
            acc[ai][aj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(part ? p1[i][kk] : p0[i][kk], use_y ? qy[j][kk] : qx[j][kk], acc[ai][aj], 0, 0, 0);
            ADAGC_SCHED_FENCE();
            if constexpr (decltype(READ)::value) {
                constexpr int NQ = 2 * kHN, NP = 2 * kHM;
                static_for<NQ + NP>([&](auto R) __attribute__((always_inline)) {
                    constexpr int n = decltype(R)::value;
                    if constexpr (part == 0) {             // all of it may be overwritten from the start: in one row, Q1 first
                        if constexpr (n * (3 * S / 2) / (NQ + NP) == t) {
                            if constexpr (n < NQ) qy[n % kHN][n / kHN] = read(qd, n % kHN, n / kHN);
                            else p1[(n - NQ) % kHM][(n - NQ) / kHM] = read_p(pa, (n - NQ) % kHM, (n - NQ) / kHM);
                        }
                    } else if constexpr (n < NP) {         // P0 during the first quadrant, Q0 when the second no longer needs qy
                        if constexpr (n * S / NP == t) p0[n % kHM][n / kHM] = read_p(pa, n % kHM, n / kHM);
                    } else {
                        if constexpr (S + (n - NP) * (S / 2) / NQ == t)
                            qy[(n - NP) % kHN][(n - NP) / kHN] = read(qd, (n - NP) % kHN, (n - NP) / kHN);
                    }
                });
            }
            side(T);
            ADAGC_SCHED_FENCE();
        });
    };

    TilePlace tp = tile_of_workgroup<SYM, PLANNED>(arguments(), 0);
    if (tp.z < 0) return;
    Source src = source(tp);
    SourceD src_d;
#pragma unroll
    for (int n = 0; n < 4 * kGL; ++n) load(src, n % kGL, n / kGL, place(n / kGL));
    ADAGC_WAIT_VMEM(2 * kGL);                              // groups 0 and 1
    int rp = 0;                                            // the place of group h
    for (int round = 0;; ++round) {
        const int groups = src.groups;
#pragma unroll
        for (int i = 0; i < 2 * kHM; ++i)
#pragma unroll
            for (int j = 0; j < 2 * kHN; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
        // Waits count the wave's accesses that may be outstanding.  After group 1 of a tile that is not the first come, without D,
        // groups 2, 3 and the last tile's stores, kStores or more (more only makes a wait stricter); with D the stores of its last
        // three quadrants and groups 2, 3, in turn.
        if (round) ADAGC_WAIT_VMEM(2 * kGL + (HAS_D ? kStores * 3 / 4 : kStores));
        barrier_keeping_loads();
        {
            uint32_t pa[kPA], qd[2];
            addresses_p(frag_p, at_place(rp), pa);
            addresses_q(frag_q, at_place(rp), qd);
            static_for<2 * kHN>([&](auto N) { constexpr int n = decltype(N)::value; qa[n % kHN][n / kHN] = read(qd, n % kHN, n / kHN); });
            static_for<2 * kHM>([&](auto N) { constexpr int n = decltype(N)::value; p0[n % kHM][n / kHM] = read_p(pa, n % kHM, n / kHM); });
        }
        ADAGC_SCHED_FENCE();
        if (groups > 4 && (!HAS_D || round == 0)) {
#pragma unroll
            for (int n = 0; n < kGL; ++n) load(src, n, 4, place(previous_place(rp)));
        }
        barrier_keeping_loads();
        const TilePlace tp_next = tile_of_workgroup<SYM, PLANNED>(arguments(), round + 1);
        const bool more = tp_next.z >= 0;
        // What follows the last group of the tile's operands in the ring: the four quadrants of D, or the next tile's first groups.
        auto begin_extras = [&]() {
            if constexpr (HAS_D) src_d = source_d(tp);
            else if (more) src = source(tp_next);
        };
        auto load_extra = [&](int n, int e, uint16_t* dst) __attribute__((always_inline)) {
            if constexpr (HAS_D) {
                if (n < kDL) load_d(src_d, n, e, dst);
            } else if (more) {
                load(src, n, e, dst);
            }
        };
        // at most `own` loads of the tile's groups and `extras` of those outstanding
        auto wait_with_extras = [&](auto OWN, auto EXTRAS) __attribute__((always_inline)) {
            constexpr int own = decltype(OWN)::value, extras = decltype(EXTRAS)::value;
            if constexpr (HAS_D) ADAGC_WAIT_VMEM(own + extras * kDL);
            else if (more) ADAGC_WAIT_VMEM(own + extras * kGL);
            else ADAGC_WAIT_VMEM(own);
        };
        if (groups == 4) {
            begin_extras();
#pragma unroll
            for (int n = 0; n < kGL; ++n) load_extra(n, 0, place(previous_place(rp)));
        }
        int h = 0;
        auto spread = [&](auto&& f) __attribute__((always_inline)) {         // f(0) .. f(kGL - 1) over a half step
            return [&](auto T) __attribute__((always_inline)) {
                static_for<kGL>([&](auto N) __attribute__((always_inline)) {
                    constexpr int n = decltype(N)::value;
                    if constexpr (n * 2 * S / kGL + 1 == decltype(T)::value) f(n);
                });
            };
        };
        constexpr std::integral_constant<int, kGL> w1{};
        constexpr std::integral_constant<int, 2 * kGL> w2{};
        constexpr std::integral_constant<int, 2> two{};
        constexpr std::integral_constant<int, 3> three{};
        // The first half step of a 64-deep tile, and both: each reads group h + 1 and loads group h + 5 into the place of group h.
        auto loads = [&](int g, uint16_t* dst) __attribute__((always_inline)) {
            return [&, g, dst](auto T) __attribute__((always_inline)) {
                static_for<kGL>([&](auto N) __attribute__((always_inline)) {
                    constexpr int n = decltype(N)::value;
                    if constexpr (n * 2 * S / kGL + 1 == decltype(T)::value) load(src, n, g, dst);
                });
            };
        };
        auto first_half = [&](bf16x8 (&x)[kHN][2], bf16x8 (&y)[kHN][2]) __attribute__((always_inline)) {
            const int pl1 = next_place(rp);
            half(no, yes, x, y, at_place(pl1), loads(h + 5, place(rp)));
            ADAGC_WAIT_VMEM(3 * kGL);
            barrier_keeping_loads();
            rp = pl1;
            ++h;
        };
        auto tile = [&](bf16x8 (&x)[kHN][2], bf16x8 (&y)[kHN][2]) __attribute__((always_inline)) {
            const int pl1 = next_place(rp), pl2 = next_place(pl1);
            half(no, yes, x, y, at_place(pl1), loads(h + 5, place(rp)));
            ADAGC_WAIT_VMEM(3 * kGL);
            barrier_keeping_loads();
            half(yes, yes, x, y, at_place(pl2), loads(h + 6, place(pl1)));
            ADAGC_WAIT_VMEM(3 * kGL);
            barrier_keeping_loads();
            rp = pl2;
            h += 2;
        };
        // the same near the end, where group h + 5 is extra number E
        auto extra = [&](auto PART, auto E, bf16x8 (&x)[kHN][2], bf16x8 (&y)[kHN][2]) __attribute__((always_inline)) {
            uint16_t* dst = place(rp);
            half(PART, yes, x, y, at_place(next_place(rp)), spread([&](int n) __attribute__((always_inline)) { load_extra(n, decltype(E)::value, dst); }));
            if constexpr (decltype(E)::value == 0) wait_with_extras(w2, yes);
            if constexpr (decltype(E)::value == 1) wait_with_extras(w1, two);
            if constexpr (decltype(E)::value == 2) wait_with_extras(no, three);
            barrier_keeping_loads();
            rp = next_place(rp);
            ++h;
        };
        while (h + 12 <= groups) {
            tile(qa, qb);
            tile(qb, qa);
        }
        if (groups > 4) {
            tile(qa, qb);
            first_half(qb, qa);                            // loads the last group
            begin_extras();
            extra(yes, no, qb, qa);
        }
        extra(no, yes, qa, qb);
        extra(yes, two, qa, qb);
        extra(no, three, qb, qa);
        // All operands are in registers; rp is the place of the last group, free.  With D the next tile's first group goes there, without,
        // results are staged there.
        half(yes, no, qb, qa, 0u, [](auto) __attribute__((always_inline)) {});
        if (HAS_D && more) {
            src = source(tp_next);
#pragma unroll
            for (int n = 0; n < kGL; ++n) load(src, n, 0, place(rp));
        }

        // epilogue
        const ADAGC_CONST GemmGroup& w = arguments().g[tp.group];
        const float alpha = arguments().alpha, beta = arguments().beta;
        const size_t v0 = (size_t)tp.tile_m * BT + wm * (kTM / 2), w0 = (size_t)tp.tile_n * BT + wn * (kTN / 2);
        uint16_t* Ct = w.ct ? w.ct + (size_t)tp.z * w.stride_ct + w0 * w.ldct + v0 : nullptr;
        uint16_t* C = !PTR && (SYM ? tp.tile_m != tp.tile_n : w.c != nullptr) ? w.c + (size_t)tp.z * w.stride_c + v0 * w.ldc + w0 : nullptr;
        int le = lane;
        asm volatile("" : "+v"(le));                       // the addresses below are made here, not kept through the main loop
        const int er = le & 15, eg = le >> 4;
        // after the exchange, lane l has 8 elements of row l mod 16: of the first block (even l / 16) or the second, from 0 or from 8
        const uint32_t lane_v = (uint32_t)((eg & 1) * 16 + (eg >> 1) * 8);
        const Offset off_ct = ((Offset)er * (Offset)w.ldct + lane_v) * 2u;
        const Offset off_c = ((Offset)er * (Offset)w.ldc + (Offset)eg * 8u) * 2u;
        constexpr int kPer = kHM / 2 * kHN;                // 16-byte vectors per lane and quadrant
        auto swap16 = [](uint32_t& x, uint32_t& y) {
            const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
            x = r[0];
            y = r[1];
        };
        int quad_place = HAS_D ? next_place(rp) : rp;
        if constexpr (HAS_D) {
            if (more) ADAGC_WAIT_VMEM(kGL);                // all of D; only this wave reads what it loaded
            else ADAGC_WAIT_VMEM(0);
        }
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const uint32_t quad = at_place(quad_place);
                u32x4 dv[kPer];
                if constexpr (HAS_D) {
#pragma unroll
                    for (int n = 0; n < kPer; ++n) {
                        const int i = (n % (kHM / 2)) * 2, j = n / (kHM / 2);
                        dv[n] = *reinterpret_cast<const ADAGC_LDS u32x4*>(quad_at(quad, j * 16 + er, (i + (eg & 1)) * 2 + (eg >> 1)));
                    }
                }
#pragma unroll
                for (int n = 0; n < kPer; ++n) {
                    const int i = (n % (kHM / 2)) * 2, j = n / (kHM / 2);
                    const f32x4 s0 = acc[a * kHM + i][b * kHN + j], s1 = acc[a * kHM + i + 1][b * kHN + j];
                    float x[4] = {alpha * s0[0], alpha * s0[1], alpha * s0[2], alpha * s0[3]};
                    float y[4] = {alpha * s1[0], alpha * s1[1], alpha * s1[2], alpha * s1[3]};
                    if constexpr (HAS_D) {
                        uint32_t d0 = dv[n].x, d1 = dv[n].y, e0 = dv[n].z, e1 = dv[n].w;
                        swap16(d0, e0);
                        swap16(d1, e1);
                        x[0] = fmaf(beta, bf16_lo(d0), x[0]);
                        x[1] = fmaf(beta, bf16_hi(d0), x[1]);
                        x[2] = fmaf(beta, bf16_lo(d1), x[2]);
                        x[3] = fmaf(beta, bf16_hi(d1), x[3]);
                        y[0] = fmaf(beta, bf16_lo(e0), y[0]);
                        y[1] = fmaf(beta, bf16_hi(e0), y[1]);
                        y[2] = fmaf(beta, bf16_lo(e1), y[2]);
                        y[3] = fmaf(beta, bf16_hi(e1), y[3]);
                    }
                    uint32_t x0 = pack_bf16(x[0], x[1]), x1 = pack_bf16(x[2], x[3]), y0 = pack_bf16(y[0], y[1]), y1 = pack_bf16(y[2], y[3]);
                    swap16(x0, y0);
                    swap16(x1, y1);
                    const u32x4 o = {x0, x1, y0, y1};
                    if (Ct)
                        *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(Ct + (size_t)(b * (BT / 2) + j * 16) * w.ldct + a * (BT / 2) + i * 16) + off_ct) = o;
                    if (C) {
                        *reinterpret_cast<ADAGC_LDS u32x4*>(quad_at(quad, j * 16 + er, (i + (eg & 1)) * 2 + (eg >> 1))) = o;
                    }
                }
                if (C) {
                    asm volatile("" ::: "memory");
#pragma unroll
                    for (int vb = 0; vb < kQuadRow / 16; ++vb) {
                        // 16 lanes read 4 rows x 16 elements and get a column each: 4 consecutive elements of a row of C
                        u32x2v t[2];
#pragma unroll
                        for (int e = 0; e < 2; ++e) {
                            const int r = 8 * eg + 4 * e + (er >> 2), c = vb * 2 + ((er & 3) >> 1);
                            const uint32_t at = quad_at(quad, r, c) + (uint32_t)((er & 1) * 8);
                            t[e] = __builtin_bit_cast(u32x2v, __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<ADAGC_LDS s16x4*>(at)));
                        }
                        const u32x4 o = {t[0].x, t[0].y, t[1].x, t[1].y};
                        *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(C + (size_t)(a * (BT / 2) + vb * 16) * w.ldc + b * (BT / 2)) + off_c) = o;
                    }
                    asm volatile("" ::: "memory");
                }
                if constexpr (HAS_D) {
                    // the quadrant's place takes the next group of the next tile
                    const int g = 2 * a + b + 1;
                    if (more && (g < 4 || src.groups > 4)) {
#pragma unroll
                        for (int n = 0; n < kGL; ++n) load(src, n, g, place(quad_place));
                    }
                    quad_place = next_place(quad_place);
                }
            }
        if (!more) return;
        tp = tp_next;
        if (!HAS_D) rp = next_place(rp);                   // where the next tile's first group was loaded
    }
}


// The block tile of a launch, and how many there are of one matrix and in all.
struct Tiles {
    int     side;
    int64_t one, all;
};

// A compute unit holds one 256 x 256 workgroup or two 128 x 128 ones, and multiplies about a quarter faster on the large tile
// (fewer LDS reads per matrix-core instruction); a launch costs whole rounds of workgroups.  Compare the two in units of "one
// 128-tile on a shared compute unit": a round of large tiles is 4 / 1.25 of them.
Tiles choose_tiles(int M, int N, bool symmetric, int64_t batch, bool wide)
{
    auto tiles = [&](int64_t side) { return symmetric ? M / side * (M / side + 1) / 2 : (M / side) * (N / side); };
    const int64_t n128 = tiles(128) * batch, n256 = tiles(256) * batch;
    const double cost128 = 2.0 * (double)((n128 + 511) / 512);
    const double cost256 = 3.2 * (double)((n256 + 255) / 256);
    if (!wide && M % 256 == 0 && N % 256 == 0 && cost256 < cost128) return {256, tiles(256), n256};
    return {128, tiles(128), n128};
}

// Rows of up to this many elements: 15 of them and a few vectors are less than 4 GiB.
constexpr int kNarrowRow = 1 << 27;

template <bool PLANNED, bool SYM, bool PTR, bool D, bool WIDE = false>
void launch_kernel(int side, int grid, const GemmWork<PLANNED>& w, hipStream_t stream)
{
    if constexpr (!WIDE) {
        if (side == 256) {
            gemm_nt_bf16_kernel<256, PLANNED, SYM, PTR, D, false, 512><<<dim3((uint32_t)grid), dim3(512), 0, stream>>>(w);
            return;
        }
    }
    gemm_nt_bf16_kernel<128, PLANNED, SYM, PTR, D, WIDE, 256><<<dim3((uint32_t)grid), dim3(256), 0, stream>>>(w);
}

template <bool WIDE>
void launch_unplanned(bool symmetric, bool d, int side, int grid, const GemmWork<false>& w, hipStream_t stream)
{
    if (symmetric && d) launch_kernel<false, true, false, true, WIDE>(side, grid, w, stream);
    else if (symmetric) launch_kernel<false, true, false, false, WIDE>(side, grid, w, stream);
    else if (d) launch_kernel<false, false, false, true, WIDE>(side, grid, w, stream);
    else launch_kernel<false, false, false, false, WIDE>(side, grid, w, stream);
}

}  // namespace

// M, N, K must be multiples of 128 and every leading dimension a multiple of 8 elements (16-byte rows).
// symmetric: P = Q (and D symmetric), so the result is symmetric: C and Ct are then the same array (pass it as Ct)
// and only the lower triangle of tiles is computed.
// batch > 1: that many products of the same shape in one launch, matrix z of every array at its base + z * stride
// (elements).  One launch over many matrices keeps all compute units busy where one matrix has too few tiles, and
// spreads the partly filled last round of workgroups over the whole batch instead of paying it per matrix.
hipError_t launch_gemm_nt_bf16(const void* P, int ldp, const void* Q, int ldq, int M, int N, int K, float alpha,
                               float beta, const void* Dt, int lddt, void* C, int ldc, void* Ct, int ldct,
                               hipStream_t stream, bool symmetric, int batch, int64_t stride_p, int64_t stride_q,
                               int64_t stride_dt, int64_t stride_c, int64_t stride_ct)
{
    if (M <= 0 || N <= 0 || K <= 0 || M % 128 || N % 128 || K % 128 || ldp % 8 || ldq % 8 || (Dt && lddt % 8) ||
        (Ct && ldct % 8) || (!C && !Ct) || batch < 1)
        return hipErrorInvalidValue;
    if ((stride_p | stride_q | stride_dt | stride_c | stride_ct) % 8 || stride_p < 0 || stride_q < 0 || stride_dt < 0 ||
        stride_c < 0 || stride_ct < 0)
        return hipErrorInvalidValue;
    auto misaligned = [](const void* a) { return (reinterpret_cast<uintptr_t>(a) & 15u) != 0; };      // 16-byte vector accesses
    if (misaligned(P) || misaligned(Q) || misaligned(Dt) || misaligned(C) || misaligned(Ct)) return hipErrorInvalidValue;
    if (symmetric && (M != N || P != Q || stride_p != stride_q || !Ct || (C && (C != Ct || stride_c != stride_ct))))
        return hipErrorInvalidValue;
    const bool wide = ldp > kNarrowRow || ldq > kNarrowRow || (Dt && lddt > kNarrowRow) || (C && ldc > kNarrowRow) || (Ct && ldct > kNarrowRow);
    const Tiles t = choose_tiles(M, N, symmetric, batch, wide);
    if (t.all > INT32_MAX) return hipErrorInvalidValue;
    GemmWork<false> work{};
    work.alpha = alpha;
    work.beta = beta;
    GemmGroup& w = work.g[0];
    w.p = static_cast<const uint16_t*>(P);
    w.q = static_cast<const uint16_t*>(Q);
    w.dt = static_cast<const uint16_t*>(Dt);
    w.ct = static_cast<uint16_t*>(Ct);
    w.c = symmetric ? w.ct : static_cast<uint16_t*>(C);
    w.stride_p = stride_p;
    w.stride_q = stride_q;
    w.stride_dt = stride_dt;
    w.stride_c = symmetric ? stride_ct : stride_c;
    w.stride_ct = stride_ct;
    w.ldp = ldp;
    w.ldq = ldq;
    w.lddt = lddt;
    w.ldc = symmetric ? ldct : ldc;
    w.ldct = ldct;
    w.k = K;
    w.tiles_m = M / t.side;
    w.tiles_n = N / t.side;
    w.tiles = (int32_t)t.one;
    w.all = (int32_t)t.all;
    // as many workgroups as the chip holds at a time, if there are tiles for them: 32 (128-tiles: 64) on each of 8 XCDs
    const int grid = 8 * (int)std::min<int64_t>((t.all + 7) / 8, t.side == 256 ? 32 : 64);
    if (wide) launch_unplanned<true>(symmetric, Dt != nullptr, t.side, grid, work, stream);
    else launch_unplanned<false>(symmetric, Dt != nullptr, t.side, grid, work, stream);
    return hipGetLastError();
}

hipError_t launch_muon_product(MuonProduct product, const MuonLaunch& l, const MuonGroup* groups, hipStream_t stream)
{
    constexpr float kA = 3.4445f, kB = -4.7750f, kC = 2.0315f;
    GemmWork<true> work{};
    work.items = l.items;
    work.first = l.first;
    for (size_t i = 0; i < l.groups.size(); ++i) {
        const MuonGroup& g = groups[l.groups[i]];
        const int64_t mn = (int64_t)g.mp * g.np, mm = (int64_t)g.mp * g.mp;
        GemmGroup& w = work.g[i];
        if (product == MuonProduct::gram) {
            w.p = w.q = g.x;
            w.c = w.ct = g.a;
            w.stride_p = w.stride_q = mn;
            w.stride_c = w.stride_ct = mm;
            w.ldp = w.ldq = w.k = g.np;
            w.ldc = w.ldct = g.mp;
        } else if (product == MuonProduct::poly) {
            w.p = w.q = w.dt = g.a;
            w.c = w.ct = g.b;
            w.stride_p = w.stride_q = w.stride_dt = w.stride_c = w.stride_ct = mm;
            w.ldp = w.ldq = w.lddt = w.ldc = w.ldct = w.k = g.mp;
        } else {
            w.p = w.dt = g.x;
            w.q = g.b;
            w.ct = g.x2;
            w.stride_p = w.stride_dt = w.stride_ct = mn;
            w.stride_q = mm;
            w.ldp = w.lddt = w.ldct = g.np;
            w.ldq = w.k = g.mp;
        }
    }
    work.alpha = product == MuonProduct::poly ? kC : 1.0f;
    work.beta = product == MuonProduct::poly ? kB : kA;
    if (product == MuonProduct::gram) launch_kernel<true, true, false, false>(l.side, l.workgroups, work, stream);
    else if (product == MuonProduct::poly) launch_kernel<true, true, false, true>(l.side, l.workgroups, work, stream);
    else launch_kernel<true, false, true, true>(l.side, l.workgroups, work, stream);
    return hipGetLastError();
}

}  // namespace adagc

// The matrix-core GEMM through the C ABI, single and batched (see include/adagc.h).
extern "C" int adagc_muon_gemm_nt_batched(const void* P, int64_t ldp, const void* Q, int64_t ldq, int64_t M, int64_t N, int64_t K,
                                          float alpha, float beta, const void* Dt, int64_t lddt, void* C, int64_t ldc, void* Ct,
                                          int64_t ldct, int32_t symmetric, int64_t batch, const int64_t* strides, void* stream)
{
    if (!P || !Q || batch < 1 || (batch > 1 && !strides)) return ADAGC_ERR_INVALID_ARG;
    if (M > INT32_MAX || N > INT32_MAX || K > INT32_MAX || ldp > INT32_MAX || ldq > INT32_MAX || lddt > INT32_MAX ||
        ldc > INT32_MAX || ldct > INT32_MAX || batch > INT32_MAX)
        return ADAGC_ERR_TOO_LARGE;
    if (ldp < K || ldq < K || (Dt && lddt < M) || (C && ldc < N) || (Ct && ldct < M)) return ADAGC_ERR_INVALID_ARG;
    int64_t st[5] = {0, 0, 0, 0, 0};
    if (strides) {
        st[0] = strides[0];
        st[1] = strides[1];
        st[2] = Dt ? strides[2] : 0;
        st[3] = C ? strides[3] : 0;
        st[4] = Ct ? strides[4] : 0;
        if (symmetric && C == nullptr) st[3] = st[4];
    }
    const hipError_t e = adagc::launch_gemm_nt_bf16(P, (int)ldp, Q, (int)ldq, (int)M, (int)N, (int)K, alpha, beta, Dt, (int)lddt,
                                                    C, (int)ldc, Ct, (int)ldct, static_cast<hipStream_t>(stream), symmetric != 0,
                                                    (int)batch, st[0], st[1], st[2], st[3], st[4]);
    if (e == hipErrorInvalidValue) return ADAGC_ERR_INVALID_ARG;
    return e == hipSuccess ? ADAGC_OK : ADAGC_ERR_HIP;
}

extern "C" int adagc_muon_gemm_nt(const void* P, int64_t ldp, const void* Q, int64_t ldq, int64_t M, int64_t N, int64_t K,
                                  float alpha, float beta, const void* Dt, int64_t lddt, void* C, int64_t ldc, void* Ct,
                                  int64_t ldct, int32_t symmetric, void* stream)
{
    return adagc_muon_gemm_nt_batched(P, ldp, Q, ldq, M, N, K, alpha, beta, Dt, lddt, C, ldc, Ct, ldct, symmetric, 1, nullptr, stream);
}
