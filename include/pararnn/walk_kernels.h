// Forward solves in which a WAVE owns a group of channels of one sequence and walks it from the first step to the last:
// no tickets, no carry records, and no barrier inside a Newton iteration.
//
// Decomposition: a lane owns one channel and C consecutive steps, the LL segments of a wave hold consecutive chunks of
// CW = 64 / LL channels, so a wave's tile is T = C LL steps.  The W waves of a workgroup hold neighbouring channel
// groups and walk the same tiles; what they share is the way to memory: a tile's rows of u are copied straight into LDS,
// W CW channels wide, while the tile before is being solved, and h leaves through LDS as whole pieces of rows.
//
// Iteration k of a tile needs delta^k at the end of the tile before, which the same wave left in LDS: the same Newton
// iterates as in one tile.  When a tile is done: newton_short_kernel's rule (short_kernels.h), here for every wave on its
// own.  That is where a third of the gain comes from: 4 channels x 192 steps of the benchmark's GRU meet 1e-5 after 4.1
// iterations on the mean, 64 channels x 96 steps (a tile of the fused blocks) after 4.6, the whole solve after 5.  The rest
// comes from the workgroup level that is gone, two barriers and a look at memory in every iteration.
//
// Bound by vector arithmetic.  Solve to the tolerance, us, with carry records / one workgroup per group -> here: GRU fp32
// 16 x 4096 x 1024 437 -> 357, bf16 4 x 65536 x 4096 6570 -> 5170, LSTM fp32 8 x 2048 x 2048 476 -> 400, bf16 369, rot_tanh bf16
// 8 x 1000 x 1536 135 -> 91.  Of the first one (12 steps, 8 waves, 4 channels) two thirds of a wave's cycles are iterations, a
// sixth the wait for the slowest wave of the workgroup, a tenth its share of the copies and stores (each holds the memory
// pipeline 16 cycles and more), 4 % reading u from LDS.  The copies are there when their tile starts.
#pragma once
#include "short_kernels.h"

namespace pararnn {

// Waves per SIMD the register allocation must leave room for: 128 registers for scalar cells, 256 or 168 for 2x2 blocks.
constexpr int walk_min_waves(int S, int C) { return S == 1 ? 4 : C <= 8 ? 3 : 2; }

// Bytes per element in LDS: copies of 16 bytes leave u as it is; copies of one element per lane, for rows or tensors that
// are not aligned to 16 bytes, write a dword each.
template <typename UT, bool WIDE> constexpr int walk_esize() { return WIDE ? (int)sizeof(UT) : 4; }

template <class Cell, int C, int W, int CWL, typename UT, bool WIDE> constexpr size_t walk_lds_bytes()
{
    return (size_t)C * Cell::G * kWave * W * walk_esize<UT, WIDE>() + ((size_t)W * kShortCarries * Cell::S << CWL) * 4;
}
// Shapes that are compiled (the choice: walk_forward_shape in driver.h): scalar cells with eight steps per thread and four
// waves or twelve and eight, 2x2 blocks with eight or sixteen and four; 1 to 16 channels per wave.  Fewer steps spend more on
// the scan between the lanes, more steps leave fewer waves on a SIMD.
template <class Cell, int C, int W, int CWL, typename UT, bool WIDE> constexpr bool walk_offered()
{
    return Cell::S <= 2 && Cell::G >= Cell::S && (Cell::S == 1 ? (C == 8 && W == 4) || (C == 12 && W == 8) : (C == 8 || C == 16) && W == 4) &&
           CWL <= 4 && (W << CWL) * walk_esize<UT, WIDE>() >= 16 && walk_lds_bytes<Cell, C, W, CWL, UT, WIDE>() <= 160 * 1024 - 256;
}

// One level of the scan inside a row of 16 lanes: lane i composes the map of lane i - DIST (applied first) into its own;
// lanes without such a neighbour keep theirs.  The cross-lane operand is part of the multiply-add, and the two wait states
// that a vector write needs before it are in front.
template <int S, int DIST> __device__ __forceinline__ void walk_scan_level(float *A, float *B)
{
#define PARARNN_LEVEL(CTRL)                                                                                             \
    if constexpr (S == 1) {                                                                                             \
        asm("s_nop 1\n\t"                                                                                               \
            "v_fmac_f32_dpp %1, %1, %0 " CTRL "\n\t"                                                                    \
            "v_mul_f32_dpp %0, %0, %0 " CTRL                                                                            \
            : "+v"(A[0]), "+v"(B[0]));                                                                                  \
    } else {                                                                                                            \
        float n0 = A[0], n1 = A[1], n2 = A[2], n3 = A[3], m0 = B[0], m1 = B[1];                                         \
        asm("s_nop 1\n\t"                                                                                               \
            "v_fmac_f32_dpp %4, %10, %6 " CTRL "\n\t"                                                                   \
            "v_fmac_f32_dpp %5, %10, %8 " CTRL "\n\t"                                                                   \
            "v_mul_f32_dpp %0, %6, %6 " CTRL "\n\t"                                                                     \
            "v_mul_f32_dpp %1, %7, %6 " CTRL "\n\t"                                                                     \
            "v_mul_f32_dpp %2, %6, %8 " CTRL "\n\t"                                                                     \
            "v_mul_f32_dpp %3, %7, %8 " CTRL "\n\t"                                                                     \
            "v_fmac_f32_dpp %4, %11, %7 " CTRL "\n\t"                                                                   \
            "v_fmac_f32_dpp %5, %11, %9 " CTRL "\n\t"                                                                   \
            "v_fmac_f32_dpp %0, %8, %7 " CTRL "\n\t"                                                                    \
            "v_fmac_f32_dpp %1, %9, %7 " CTRL "\n\t"                                                                    \
            "v_fmac_f32_dpp %2, %8, %9 " CTRL "\n\t"                                                                    \
            "v_fmac_f32_dpp %3, %9, %9 " CTRL                                                                           \
            : "+&v"(n0), "+&v"(n1), "+&v"(n2), "+&v"(n3), "+&v"(m0), "+&v"(m1)                                          \
            : "v"(A[0]), "v"(A[1]), "v"(A[2]), "v"(A[3]), "v"(B[0]), "v"(B[1]));                                        \
        A[0] = n0; A[1] = n1; A[2] = n2; A[3] = n3; B[0] = m0; B[1] = m1;                                               \
    }
    if constexpr (DIST == 1) { PARARNN_LEVEL("row_shr:1 row_mask:0xf bank_mask:0xf") }
    else if constexpr (DIST == 2) { PARARNN_LEVEL("row_shr:2 row_mask:0xf bank_mask:0xf") }
    else if constexpr (DIST == 4) { PARARNN_LEVEL("row_shr:4 row_mask:0xf bank_mask:0xf") }
    else if constexpr (DIST == 8) { PARARNN_LEVEL("row_shr:8 row_mask:0xf bank_mask:0xf") }
    else if constexpr (DIST == 16) { PARARNN_LEVEL("row_bcast:15 row_mask:0xa bank_mask:0xf") }   // last lane of rows 0, 2 to rows 1, 3
    else { PARARNN_LEVEL("row_bcast:31 row_mask:0xc bank_mask:0xf") }                            // lane 31 to the upper half
#undef PARARNN_LEVEL
}

// Where a lane's channel and segment lie: up to 4 channels one or more rows of 16 lanes each, segments in lane order;
// more channels share a row, CWR = CW / 4 of them, neighbouring segments CWR lanes apart.
struct WalkLane { int seg, col; };
__device__ __forceinline__ WalkLane walk_lane(int lane, int cw_log2)
{
    if (cw_log2 <= 2) return {lane & ((64 >> cw_log2) - 1), lane >> (6 - cw_log2)};
    const int r = cw_log2 - 2;
    return {(lane & 15) >> r, ((lane >> 4) << r) | (lane & ((1 << r) - 1))};
}

// (A, B): in, the map of the lane's own chunk; out, the composition of all chunks of the wave up to and with its own.
template <int S> __device__ __forceinline__ void walk_scan(int cw_log2, float *A, float *B)
{
    if (cw_log2 <= 2) walk_scan_level<S, 1>(A, B);
    if (cw_log2 <= 3) walk_scan_level<S, 2>(A, B);
    if (cw_log2 <= 4) walk_scan_level<S, 4>(A, B);
    if (cw_log2 <= 5) walk_scan_level<S, 8>(A, B);
    if (cw_log2 <= 1) walk_scan_level<S, 16>(A, B);
    if (cw_log2 <= 0) walk_scan_level<S, 32>(A, B);
}

// x of the segment before the own one; `first` where there is none
__device__ __forceinline__ float walk_shift(int cw_log2, int seg, float x, float first)
{
    const int f = __float_as_int(first), v = __float_as_int(x);
    if (cw_log2 <= 1) {
        const int y = __builtin_amdgcn_update_dpp(f, v, 0x138, 0xf, 0xf, false);                       // wave_shr:1
        return seg == 0 ? first : __int_as_float(y);
    }
    if (cw_log2 == 2) return __int_as_float(__builtin_amdgcn_update_dpp(f, v, 0x111, 0xf, 0xf, false));   // row_shr:1
    if (cw_log2 == 3) return __int_as_float(__builtin_amdgcn_update_dpp(f, v, 0x112, 0xf, 0xf, false));
    if (cw_log2 == 4) return __int_as_float(__builtin_amdgcn_update_dpp(f, v, 0x114, 0xf, 0xf, false));
    if (cw_log2 == 5) return __int_as_float(__builtin_amdgcn_update_dpp(f, v, 0x118, 0xf, 0xf, false));
    return first;
}

typedef unsigned int walk_u4 __attribute__((ext_vector_type(4)));

// A wave's copy from memory into LDS, BYTES per lane, lanes in order from `lds` on (dwords where BYTES is less than four).
// Asm statements: the compiled code then has no wait for it of its own, which would come with the first LDS read of the
// tile that is solved meanwhile.  walk_arrived() is the wait.
template <int BYTES> __device__ __forceinline__ void walk_copy(walk_u4 rsrc, unsigned int lds, unsigned int voff, unsigned int soff)
{
    if constexpr (BYTES == 16)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
    else if constexpr (BYTES == 4)
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dword %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
    else
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_ushort %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc), "s"(soff) : "memory", "m0");
}
// x + step, computed where it stands: sums that are known early are kept in scalar registers, which run out.
__device__ __forceinline__ unsigned int walk_next(unsigned int x, unsigned int step)
{
    x += step;
    asm volatile("" : "+s"(x));
    return x;
}
// The copies of every wave of the workgroup have arrived.
__device__ __forceinline__ void walk_arrived() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <class Cell, int C, int W, int CWL, typename UT, bool WIDE>
__global__ __launch_bounds__(kWave * W) __attribute__((amdgpu_waves_per_eu(walk_min_waves(Cell::S, C)))) void newton_walk_kernel(const ShortArgs a)
{
    constexpr int S = Cell::S, G = Cell::G, SS = S * S, PR = Cell::PR;
    using RawU = typename RawVec<UT, 1>::type;
    constexpr unsigned int E = sizeof(UT), ES = walk_esize<UT, WIDE>();
    constexpr unsigned int kBlock = kWave * W * ES;    // bytes in LDS of one (step of a chunk, gate): [segment][channel]
    static_assert(G >= S && (C * G * W * ES) % 16 == 0 && (C * S * W * ES) % 16 == 0, "copies of whole waves");
    // u of a tile [C][G][LL][W CW]; the waves' carries [W][kShortCarries][S][CW]
    __shared__ __align__(16) char s_walk[walk_lds_bytes<Cell, C, W, CWL, UT, WIDE>()];
    __shared__ unsigned int s_max[16];
    const int item = short_item(a.n_items);
    if (item < 0) return;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    constexpr int cwl = CWL, CW = 1 << cwl, LL = kWave >> cwl, NCH = W << cwl;
    const WalkLane me = walk_lane(lane, cwl);
    const int b = item / a.n_cg, cg = item - b * a.n_cg;
    const int ch0 = cg * NCH, ch = ch0 + w * CW + me.col;
    const bool ch_ok = ch < a.H;
    constexpr int T = C * LL;
    const int lt0 = me.seg * C;            // this lane's first step within a tile
    const unsigned int Hn = (unsigned int)a.H;
    const unsigned int lds0 = (unsigned int)(unsigned long long)(__attribute__((address_space(3))) const void *)s_walk;
    float *s_carry = reinterpret_cast<float *>(s_walk + (size_t)C * G * kBlock) + ((size_t)w * kShortCarries * S << cwl) + me.col;

    // A row of a segment is rb bytes wide; its pieces of 16 bytes lie at their position XOR a number that goes up with the
    // segment, so that the segments of a wave, which read the same column, do not all meet in the same banks.
    constexpr unsigned int rb = (unsigned int)NCH * ES;
    constexpr unsigned int pieces = rb >> 4 < 8 ? rb >> 4 : 8;      // pieces that change places (16 bytes at least: W ES >= 16)
    auto turn = [&](unsigned int seg) { return (seg * rb >> 7) & (pieces - 1u); };
    const unsigned int my_col = (unsigned int)(w * CW + me.col) * ES;
    const unsigned int my_lds = (unsigned int)me.seg * rb + (((my_col >> 4) ^ turn((unsigned int)me.seg)) << 4) + (my_col & 15u);

    // The copies of a tile: copy n takes 64 pieces of 16 bytes in the order of LDS (WIDE), or 64 elements of every block.
    constexpr int kPieces = kBlock / 16;               // of a block
    constexpr int kCopies = WIDE ? C * G * kPieces / kWave : C * G * W;
    constexpr int kStores = WIDE ? C * S * kPieces / kWave : C * S * W;
    constexpr int kParts = kPieces > kWave ? kPieces / kWave : 1;          // copies that a block takes
    constexpr int kBlocksPer = kPieces < kWave ? kWave / kPieces : 1;     // blocks that a copy takes
    // A wave's copies are n = w, w + W, ...: always the same part of a block, so that one offset per lane serves them all.
    static_assert(W % kParts == 0, "parts of a block");
    unsigned int piece_seg, piece_col, piece_blk = 0;  // this lane's piece: segment, byte in the row, block
    if constexpr (WIDE) {
        unsigned int q = (unsigned int)lane + (unsigned int)(w % kParts) * kWave;
        piece_blk = q / kPieces;
        q = q % kPieces * 16u;
        piece_seg = q / rb;
        const unsigned int at = q % rb >> 4;
        piece_col = (at ^ turn(piece_seg)) << 4;
    } else {
        const unsigned int q = (unsigned int)(w * kWave + lane) * 4u;
        piece_seg = q / rb;
        const unsigned int at = q % rb;
        piece_col = (((at >> 4) ^ turn(piece_seg)) << 4) | (at & 15u);
    }
    const unsigned int piece_ch = piece_col / ES;
    const unsigned int copy_off = (piece_seg * C * G + piece_blk) * Hn * E + ((unsigned int)ch0 + piece_ch) * E;
    const bool piece_ok = ch0 + (int)piece_ch < a.H;

    const unsigned int first_row = WIDE ? (unsigned int)(w / kParts * kBlocksPer) * Hn * E : 0u;
    const unsigned int row_step = (WIDE ? (unsigned int)(W / kParts * kBlocksPer) : 1u) * Hn * E;

    auto bytes = [&](int tile, unsigned int per_row) {
        const unsigned long long n = (unsigned long long)(a.L - tile * T) * per_row;
        return n < 0x7fffffffull ? (unsigned int)n : 0x7fffffffu;
    };
    // A wave's share of the copies of a tile, one by one: they go out between other work, because each takes the memory
    // pipeline 16 cycles and more, and a wave that has several to issue waits for it.
    constexpr int kShare = (kCopies + W - 1) / W;
    struct Copies { walk_u4 rsrc; unsigned int lds, soff; };
    auto copies_of = [&](int tile) {
        const unsigned long long p = (unsigned long long)(static_cast<const UT *>(a.u) + ((size_t)b * a.L + (size_t)tile * T) * G * Hn);
        Copies c;
        c.rsrc = walk_u4{(unsigned int)__builtin_amdgcn_readfirstlane((unsigned int)p),
                         (unsigned int)__builtin_amdgcn_readfirstlane((unsigned int)(p >> 32)) & 0xffffu, bytes(tile, G * Hn * E), 0x27000u};
        c.lds = lds0 + (unsigned int)w * (WIDE ? 1024u : 256u);
        c.soff = first_row;
        return c;
    };
    auto copy_one = [&](Copies &c, int m) {
        if (m * W + W <= kCopies || m * W + w < kCopies) walk_copy<WIDE ? 16 : (int)E>(c.rsrc, c.lds, copy_off, c.soff);
        c.soff = walk_next(c.soff, row_step);
        c.lds = walk_next(c.lds, WIDE ? W * 1024u : kBlock);
    };
    // What the waves left of h in LDS, where u of gates 0 .. S - 1 had been, goes out as pieces of rows.
    constexpr int kMine = (kStores + W - 1) / W;
    using Piece = std::conditional_t<WIDE, walk_u4, RawU>;
    auto fetch_h = [&](Piece (&x)[kMine]) {
#pragma unroll
        for (int m = 0; m < kMine; ++m) {
            const int n = m * W + w;
            if (n < kStores) {
                if constexpr (WIDE) {
                    const unsigned int blk = (unsigned int)(n / kParts * kBlocksPer) + piece_blk;        // step * S + state
                    const unsigned int q = ((unsigned int)lane + (unsigned int)(w % kParts) * kWave) % kPieces * 16u;
                    x[m] = *reinterpret_cast<const walk_u4 *>(s_walk + (blk / S * G + blk % S) * kBlock + q);
                } else {
                    const unsigned int blk = (unsigned int)m;
                    x[m] = *reinterpret_cast<const RawU *>(s_walk + (blk / S * G + blk % S) * kBlock + (unsigned int)(w * kWave + lane) * 4u);
                }
            }
        }
    };
    struct Stores { buf_rsrc rsrc; unsigned int soff; };
    auto stores_of = [&](int tile) {
        return Stores{bounded_rsrc(static_cast<UT *>(a.h) + ((size_t)b * a.L + (size_t)tile * T) * S * Hn, bytes(tile, S * Hn * E)), first_row};
    };
    const unsigned int store_off = (piece_seg * C * S + piece_blk) * Hn * E + ((unsigned int)ch0 + piece_ch) * E;
    auto store_one = [&](Stores &t, const Piece (&x)[kMine], int m) {
        if ((m * W + W <= kStores || m * W + w < kStores) && piece_ok) {
            if constexpr (WIDE) __builtin_amdgcn_raw_buffer_store_b128(x[m], t.rsrc, store_off, t.soff, 0);
            else if constexpr (E == 4) __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, x[m]), t.rsrc, store_off, t.soff, 0);
            else __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(unsigned short, x[m]), t.rsrc, store_off, t.soff, 0);
        }
        t.soff = walk_next(t.soff, row_step);
    };
    auto leave_h = [&](const float (&ho)[C][S]) {
#pragma unroll
        for (int i = 0; i < C; ++i)
#pragma unroll
            for (int s = 0; s < S; ++s) {
                char *at = s_walk + (unsigned int)(i * G + s) * kBlock + my_lds;
                if constexpr (E == 4) *reinterpret_cast<float *>(at) = ho[i][s];
                else *reinterpret_cast<unsigned short *>(at) = f32_to_bf16(ho[i][s]);
            }
    };

    {
        Copies c = copies_of(0);
#pragma unroll
        for (int m = 0; m < kShare; ++m) copy_one(c, m);
    }
    float p[PR], pq[Cell::PQ > 0 ? Cell::PQ : 1], h0v[S];
#pragma unroll
    for (int r = 0; r < PR; ++r) p[r] = ch_ok ? a.params[(size_t)r * Hn + ch] : 0.0f;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        float t[1] = {0.0f};
        if (ch_ok && a.h0) load_vec<1>(static_cast<const UT *>(a.h0) + ((size_t)b * S + s) * Hn + ch, t);
        h0v[s] = t[0];
    }
    Cell::fold_params(p, pq);

    const unsigned int tol_bits = __float_as_uint(fabsf(a.tol)), eighth_bits = __float_as_uint(0.125f * fabsf(a.tol));
    unsigned int v = 0u;                               // this wave's verdict
    int k_before = 0, k_final = 0;                     // iterations of the tile before; the first with a final boundary
    float ho[C][S], guess_end[S];                      // guess_end: the initial guess of the last step of the tile before
#pragma unroll
    for (int s = 0; s < S; ++s) guess_end[s] = h0v[s];
    for (int tile = 0; tile < a.n_tiles; ++tile) {
        __builtin_amdgcn_s_setprio(3);
        walk_arrived();
        float uu[C][G];
        RawU uur[C][G];
#pragma unroll
        for (int i = 0; i < C; ++i)
#pragma unroll
            for (int q = 0; q < G; ++q) uur[i][q] = *reinterpret_cast<const RawU *>(s_walk + (unsigned int)(i * G + q) * kBlock + my_lds);
        Piece x[kMine];
        if (tile > 0) {
            leave_h(ho);
            lds_barrier_keep_vmem();
            fetch_h(x);
        }
        lds_barrier_keep_vmem();
        const bool more = tile + 1 < a.n_tiles;
        Copies c = copies_of(more ? tile + 1 : tile);
        Stores t = stores_of(tile > 0 ? tile - 1 : tile);

        // initial guess h^0_l = f(h0, u_l) (App. A); the step in front of the chunk belongs to the segment before
        const int l0 = tile * T + lt0;
        float hprev[S];
#pragma unroll
        for (int i = 0; i < C; ++i) {
#pragma unroll
            for (int q = 0; q < G; ++q) {
                float t[1];
                raw_to_float<UT, 1>(uur[i][q], t);
                uu[i][q] = t[0];
            }
            Cell::fold_u(p, uu[i]);
            Cell::template step<true>(p, h0v, uu[i], ho[i], pq);
            gates_done<S>(ho[i]);
            if (tile > 0) {
#pragma unroll
                for (int m = i * kMine / C; m < (i + 1) * kMine / C; ++m) store_one(t, x, m);
            }
            if (more) {
#pragma unroll
                for (int m = i * kShare / C; m < (i + 1) * kShare / C; ++m) copy_one(c, m);
            }
        }
#pragma unroll
        for (int s = 0; s < S; ++s) hprev[s] = walk_shift(cwl, me.seg, ho[C - 1][s], guess_end[s]);
        if (more) {
            const int src = cwl <= 2 ? lane | (LL - 1) : lane | (15 & ~((1 << (cwl - 2)) - 1));   // the last segment's lane
#pragma unroll
            for (int s = 0; s < S; ++s) guess_end[s] = __shfl(ho[C - 1][s], src, 64);
        }

        __builtin_amdgcn_s_setprio(0);
        const int n_valid = ch_ok ? min(max(a.L - l0, 0), C) : 0;      // steps of this lane inside the tensor
        const bool all_valid = __all(n_valid == C);
        int k = 0, k_met = 1;                          // k_met: the first iteration after which every update met the tolerance
        // The largest update only takes part in comparisons, which every lane makes for itself: the bits of a value that is not
        // negative are in its order, those of a NaN above them all.
        bool finite = true, over = false;
        unsigned int wmax_bits = 0u;
        while (k < a.max_iter) {
            ++k;
            float dt[S];                               // what enters the tile
#pragma unroll
            for (int s = 0; s < S; ++s) dt[s] = 0.0f;
            if (k <= k_final) {
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    dt[s] = s_carry[((k - 1) * S + s) << cwl];
                    if (k == k_final && k_before > k_final) dt[s] += s_carry[(k * S + s) << cwl];
                }
            }
            // ---- thread level
            float PA[C][SS], qb[C][S], accA[SS], accB[S];
#pragma unroll
            for (int i = 0; i < C; ++i) {
                float J[SS], r[S], hp[S], F[S];
#pragma unroll
                for (int s = 0; s < S; ++s) hp[s] = i == 0 ? hprev[s] : ho[i > 0 ? i - 1 : 0][s];
                eval_step<Cell>(p, pq, hp, uu[i], F, J);
#pragma unroll
                for (int s = 0; s < S; ++s) r[s] = F[s] - ho[i][s];
                if (i == 0) {
#pragma unroll
                    for (int e = 0; e < SS; ++e) accA[e] = J[e];
#pragma unroll
                    for (int s = 0; s < S; ++s) accB[s] = r[s];
                } else {
                    push_step<S>(J, r, accA, accB);
                }
                gates_done<SS>(accA);
                gates_done<S>(accB);
#pragma unroll
                for (int e = 0; e < SS; ++e) PA[i][e] = accA[e];
#pragma unroll
                for (int s = 0; s < S; ++s) qb[i][s] = accB[s];
            }
            // ---- wave level: the update at the end of every chunk, which enters the next one
            walk_scan<S>(cwl, accA, accB);
            float x[S], din[S];
            affine<S>(accA, dt, accB, x);
#pragma unroll
            for (int s = 0; s < S; ++s) din[s] = walk_shift(cwl, me.seg, x[s], dt[s]);
            // ---- back-substitution
            wmax_bits = 0u;
            float d[S];
            auto substitute = [&](auto guard) {
                float m = 0.0f, last = 0.0f;
#pragma unroll
                for (int i = 0; i < C; ++i) {
                    affine<S>(PA[i], din, qb[i], d);
#pragma unroll
                    for (int s = 0; s < S; ++s) {
                        ho[i][s] += d[s];
                        if constexpr (decltype(guard)::value) {
                            if (i < n_valid) wmax_bits = max(wmax_bits, __float_as_uint(d[s]) & 0x7fffffffu);
                        } else {
                            if ((i * S + s) & 1) abs_max(m, last, d[s]);
                            last = d[s];
                        }
                    }
                }
                if constexpr (!decltype(guard)::value) wmax_bits = __float_as_uint(m) & 0x7fffffffu;
            };
            if (all_valid) substitute(std::false_type{});
            else substitute(std::true_type{});
            // the state in front of the chunk: what the segment before holds, or what the tile before left
#pragma unroll
            for (int s = 0; s < S; ++s) hprev[s] = walk_shift(cwl, me.seg, ho[C - 1][s], hprev[s] + dt[s]);
            if (more && me.seg == LL - 1) {
                float *c = s_carry + (((min(k, kShortCarries) - 1) * S) << cwl);
#pragma unroll
                for (int s = 0; s < S; ++s) c[s << cwl] = k > kShortCarries ? c[s << cwl] + d[s] : d[s];
            }
            // ---- the stopping test of this group of channels
            finite = !__any(wmax_bits >= 0x7f800000u);
            if (!finite) break;
            if (a.tol >= 0.0f) {
                over = __any(wmax_bits > tol_bits);
                if (over) k_met = k + 1;
                else if (k >= k_final) break;
            }
        }
        if (!finite) v = max(v, short_verdict(kStNonFinite, k));
        else if (over) v = max(v, short_verdict(kStNotConverged, k));
        else v = max(v, short_verdict(kStOk, a.tol >= 0.0f ? k_met : k));
        k_before = k_final = min(k, kShortCarries);
        if (k_before == k && k > 1 && finite && a.tol >= 0.0f && !__any(wmax_bits > eighth_bits)) k_final = k - 1;
    }
    {
        leave_h(ho);                                   // nobody reads u any more since the tile's barriers
        if (lane == 0) s_max[w] = v;
        lds_barrier_keep_vmem();
        Piece x[kMine];
        fetch_h(x);
        Stores t = stores_of(a.n_tiles - 1);
#pragma unroll
        for (int m = 0; m < kMine; ++m) store_one(t, x, m);
        v = wave_max_u32(s_max[lane < W ? lane : 0]);
    }
    short_collect(a, item, v, W, s_max);
}

}  // namespace pararnn
