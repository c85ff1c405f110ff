// Definitions of Kernels<Cell, UT>; included only by the inst_*.hip files.
#pragma once
#include "launch.h"

namespace pararnn {

// workgroups of a persistent launch: what fits on the device at once
template <typename K> static int persistent_grid(K kernel, int threads, int n_tiles)
{
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess || per_cu < 1)
        per_cu = 1;
    const long long cap = (long long)per_cu * device_cu_count();
    return (int)(n_tiles < cap ? n_tiles : cap);
}

// Tile shapes instantiated for a cell.  Blocks of 3x3 and larger keep S*S + S prefix values per
// step in registers: beyond eight (3x3) or four (4x4) steps per thread and one channel per lane the
// kernels spill by the hundred, so those shapes are not built (the launch reports UNSUPPORTED).
template <class Cell, int VEC, int C> constexpr bool shape_offered()
{
    return Cell::S <= 2 || (VEC == 1 && C <= (Cell::S == 3 ? 8 : 4));
}

// static LDS of the forward kernels must stay within 64 KiB
template <class Cell, int VEC, int LL, int W> constexpr bool forward_fits_lds()
{
    constexpr int S = Cell::S, SS = S * S;
    return (size_t)(W * (SS + S) + 4 * S) * (kWave / LL) * VEC * sizeof(float) + 4 * W + 64 <= 65536;
}

// static LDS of the backward kernel must stay within 64 KiB (backward_tile_fits in driver.h is the same on the host)
template <class Cell, int VEC, int LL, int W> constexpr bool backward_fits_lds()
{
    constexpr int S = Cell::S, SS = S * S, PRX = Cell::PR > 0 ? Cell::PR : 1;
    constexpr int rows = (SS + S) > PRX ? (SS + S) : PRX;
    return (size_t)(W * rows + S) * (kWave / LL) * VEC * sizeof(float) + 16 <= 65536;
}

template <class Cell, typename UT>
hipError_t Kernels<Cell, UT>::init_guess(int vec, const FwdArgs &a, hipStream_t st)
{
    if constexpr (IsRaw<Cell>::value) {
        return hipErrorInvalidValue;
    } else {
        const size_t n = (size_t)a.g.B * a.g.L * (a.g.H / vec);
        size_t blocks = (n + 255) / 256;
        const size_t cap = (size_t)device_cu_count() * 32;
        if (blocks > cap) blocks = cap;
#define PARARNN_CASE(V)                                                                       \
    if (vec == V) {                                                                           \
        hipLaunchKernelGGL((init_guess_kernel<Cell, V, UT>), dim3((unsigned)blocks), dim3(256), 0, st, a); \
        return hipGetLastError();                                                             \
    }
        PARARNN_VECS(PARARNN_CASE)
#undef PARARNN_CASE
        return hipErrorInvalidValue;
    }
}

template <class Cell, typename UT>
hipError_t Kernels<Cell, UT>::residual_norm(int vec, const ResArgs &a, hipStream_t st)
{
    if constexpr (IsRaw<Cell>::value) {
        return hipErrorInvalidValue;
    } else {
        const size_t n = (size_t)a.B * ((a.L + kResRun - 1) / kResRun) * (a.H / vec);
        size_t blocks = (n + 255) / 256;
        const size_t cap = (size_t)device_cu_count() * 8;
        if (blocks > cap) blocks = cap;
#define PARARNN_CASE(V)                                                                       \
    if (vec == V) {                                                                           \
        hipLaunchKernelGGL((residual_norm_kernel<Cell, V, UT>), dim3((unsigned)blocks), dim3(256), 0, st, a); \
        return hipGetLastError();                                                             \
    }
        PARARNN_VECS(PARARNN_CASE)
#undef PARARNN_CASE
        return hipErrorInvalidValue;
    }
}

template <class Cell, typename UT>
hipError_t Kernels<Cell, UT>::newton_iter(const TileCfg &cfg, const FwdArgs &a, bool fold_guess, hipStream_t st)
{
#define PARARNN_CASE(V, LLv, C, W)                                                             \
    if (cfg.vec == V && cfg.ll == LLv && cfg.c == C && cfg.w == W) {                           \
        if constexpr (shape_offered<Cell, V, C>() && forward_fits_lds<Cell, V, LLv, W>()) {    \
            static int grid_cap[2] = {0, 0}; /* per instantiation */                           \
            constexpr bool kFoldGuess = !IsRaw<Cell>::value;                                   \
            const int first = (kFoldGuess && fold_guess) ? 1 : 0;                              \
            auto kern = newton_iter_kernel<Cell, V, LLv, C, W, UT, false>;                     \
            if constexpr (kFoldGuess) {                                                        \
                if (first) kern = newton_iter_kernel<Cell, V, LLv, C, W, UT, true>;            \
            }                                                                                  \
            if (grid_cap[first] == 0) grid_cap[first] = persistent_grid(kern, kWave * W, 1 << 30); \
            const int grid = a.g.n_tiles < grid_cap[first] ? a.g.n_tiles : grid_cap[first];    \
            hipLaunchKernelGGL(kern, dim3(grid), dim3(kWave * W), 0, st, a);                   \
            return hipGetLastError();                                                          \
        } else {                                                                               \
            return hipErrorInvalidValue;                                                       \
        }                                                                                      \
    }
    PARARNN_SHAPES(PARARNN_CASE)
#undef PARARNN_CASE
    return hipErrorInvalidValue;
}

template <class Cell, typename UT>
hipError_t Kernels<Cell, UT>::newton_fused(const TileCfg &cfg, const FusedArgs &a, hipStream_t st)
{
    if constexpr (IsRaw<Cell>::value) {
        return hipErrorInvalidValue;
    } else {
#define PARARNN_CASE(V, LLv, C, W)                                                             \
    if (cfg.vec == V && cfg.ll == LLv && cfg.c == C && cfg.w == W) {                           \
        if constexpr (shape_offered<Cell, V, C>()) {                                           \
            static int grid_cap[2] = {0, 0};                                                   \
            const int tl = a.tail ? 1 : 0;                                                     \
            auto kern = a.tail ? newton_fused_kernel<Cell, V, LLv, C, W, UT, true>             \
                               : newton_fused_kernel<Cell, V, LLv, C, W, UT, false>;           \
            if (grid_cap[tl] == 0) grid_cap[tl] = persistent_grid(kern, kWave * W, 1 << 30);   \
            const int grid = a.g.n_tiles < grid_cap[tl] ? a.g.n_tiles : grid_cap[tl];          \
            hipLaunchKernelGGL(kern, dim3(grid), dim3(kWave * W), 0, st, a);                   \
            return hipGetLastError();                                                          \
        } else {                                                                               \
            return hipErrorInvalidValue;                                                       \
        }                                                                                      \
    }
        PARARNN_SHAPES(PARARNN_CASE)
#undef PARARNN_CASE
        return hipErrorInvalidValue;
    }
}

template <class Cell, typename UT>
hipError_t Kernels<Cell, UT>::newton_short(int c, int w, const ShortArgs &a, hipStream_t st)
{
    if constexpr (IsRaw<Cell>::value) {
        return hipErrorInvalidValue;
    } else {
        const unsigned int grid = 8u * (unsigned int)((a.n_items + 7) / 8);
        // the last tile starts inside the sequence (its descriptor ends with it), the tiles cover it, and the carries
        // of several tiles cross the workgroup's barriers
        const long long steps = (long long)c * (kWave >> a.lps_log2) * w;
        if (a.n_tiles < 1 || (a.n_tiles - 1) * steps >= a.L || a.n_tiles * steps < a.L || (a.n_tiles > 1 && w < 2))
            return hipErrorInvalidValue;
        const size_t lds = w > 1 ? ((size_t)(w * (Cell::S * Cell::S + Cell::S) + (a.n_tiles > 1 ? 2 * kShortCarries * Cell::S : 0))
                                    << a.lps_log2) * sizeof(float) : 0;
#define PARARNN_CASE(C, MANY)                                                                                         \
    if constexpr (short_offered<Cell, C>(MANY)) {                                                                     \
        if (c == C && (a.n_tiles > 1 || (C > 8 && Cell::S > 1)) == MANY && w <= (MANY ? 8 : short_max_waves<Cell, C>())) { \
            hipLaunchKernelGGL((newton_short_kernel<Cell, C, UT, MANY>), dim3(grid), dim3(kWave * w), lds, st, a);    \
            return hipGetLastError();                                                                                 \
        }                                                                                                             \
    }
        PARARNN_CASE(4, false) PARARNN_CASE(8, false) PARARNN_CASE(16, false) PARARNN_CASE(8, true) PARARNN_CASE(16, true)
#undef PARARNN_CASE
        return hipErrorInvalidValue;
    }
}

template <class Cell, typename UT>
hipError_t Kernels<Cell, UT>::newton_walk(int c, int w, bool wide, const ShortArgs &a, hipStream_t st)
{
    if constexpr (IsRaw<Cell>::value) {
        return hipErrorInvalidValue;
    } else {
        const unsigned int grid = 8u * (unsigned int)((a.n_items + 7) / 8);
        // the last tile starts inside the sequence, the tiles cover it
        const long long steps = (long long)c * (kWave >> a.lps_log2);
        if (a.n_tiles < 1 || (a.n_tiles - 1) * steps >= a.L || a.n_tiles * steps < a.L) return hipErrorInvalidValue;
#define PARARNN_CASE(C, W, CWL, WIDE)                                                                                 \
    if constexpr (walk_offered<Cell, C, W, CWL, UT, WIDE>()) {                                                        \
        if (c == C && w == W && a.lps_log2 == CWL && wide == WIDE) {                                                  \
            hipLaunchKernelGGL((newton_walk_kernel<Cell, C, W, CWL, UT, WIDE>), dim3(grid), dim3(kWave * W), 0, st, a); \
            return hipGetLastError();                                                                                 \
        }                                                                                                             \
    }
#define PARARNN_WIDTHS(C, W)                                                                                          \
    PARARNN_CASE(C, W, 0, true) PARARNN_CASE(C, W, 1, true) PARARNN_CASE(C, W, 2, true) PARARNN_CASE(C, W, 3, true)   \
    PARARNN_CASE(C, W, 4, true) PARARNN_CASE(C, W, 0, false) PARARNN_CASE(C, W, 1, false) PARARNN_CASE(C, W, 2, false) \
    PARARNN_CASE(C, W, 3, false) PARARNN_CASE(C, W, 4, false)
        PARARNN_WIDTHS(8, 4) PARARNN_WIDTHS(12, 8) PARARNN_WIDTHS(16, 4)
#undef PARARNN_WIDTHS
#undef PARARNN_CASE
        return hipErrorInvalidValue;
    }
}

template <class Cell, typename UT>
hipError_t Kernels<Cell, UT>::backward_short(int c, int w, const ShortArgs &a, hipStream_t st)
{
    if constexpr (IsRaw<Cell>::value) {
        return hipErrorInvalidValue;
    } else {
        constexpr int SA = Cell::S * Cell::S + Cell::S, rows = SA > Cell::PR ? SA : Cell::PR;
        if ((long long)c * (kWave >> a.lps_log2) * w < a.L) return hipErrorInvalidValue;
        const unsigned int grid = 8u * (unsigned int)((a.n_items + 7) / 8);
        const size_t lds = w > 1 ? ((size_t)w * rows << a.lps_log2) * sizeof(float) : 0;
#define PARARNN_CASE(C)                                                                                           \
    if constexpr (short_offered<Cell, C>(false)) {                                                                  \
        if (c == C && w <= short_max_waves<Cell, C>()) {                                                          \
            hipLaunchKernelGGL((backward_short_kernel<Cell, C, UT>), dim3(grid), dim3(kWave * w), lds, st, a);          \
            return hipGetLastError();                                                                             \
        }                                                                                                         \
    }
        PARARNN_CASE(4) PARARNN_CASE(8)
#undef PARARNN_CASE
        return hipErrorInvalidValue;
    }
}

// The LDS-staged variant of the backward kernel exists for bf16 storage, one channel per lane, one
// segment per wave and steps per thread in multiples of 8 (one copy instruction moves 8 rows).
template <class Cell, int VEC, int LL, int C, typename UT> constexpr bool backward_stage_offered()
{
    return !IsRaw<Cell>::value && sizeof(UT) == 2 && VEC == 1 && LL == 1 && C % 8 == 0;
}

// The plain kernel with streamed rows: of the shapes that choose_tile and backward_tile take for rows of whole cache lines, but the
// one that it does not pay for (backward_stream in driver.h).
template <class Cell, int VEC, int LL, int C, int W> constexpr bool backward_stream_offered()
{
    return !IsRaw<Cell>::value && VEC == 1 && C != 12 && (LL == 1 || (LL == 2 && C == 8 && W == 8));
}

// ... and the one with a queue for each XCD.
template <class Cell, int VEC, int LL, int C, int W> constexpr bool backward_queues_offered()
{
    return !IsRaw<Cell>::value && backward_queues_shape(Cell::S, Cell::G, VEC, LL, C, W);
}

// static LDS of the staged backward kernel: its staging rows on top of the plain kernel's.  All of a compute unit's may be
// taken: one workgroup of LSTM's 64 x 128 tile has 128 KB of rows on their way (8 x 2048 x 2048 bf16 260 -> 206 us).
template <class Cell, int C, int W> constexpr bool backward_stage_fits_lds()
{
    constexpr int S = Cell::S, SS = S * S, PRX = Cell::PR > 0 ? Cell::PR : 1;
    constexpr int rows = (SS + S) > PRX ? (SS + S) : PRX;
    return (size_t)(W * rows + S) * kWave * sizeof(float) + (size_t)W * C * (Cell::G + 2 * S) * 128 + 64 <= 163840 - 256;
}

template <class Cell, typename UT>
hipError_t Kernels<Cell, UT>::backward(const TileCfg &cfg, const BwdArgs &a, hipStream_t st)
{
#define PARARNN_CASE(V, LLv, C, W)                                                             \
    if (cfg.vec == V && cfg.ll == LLv && cfg.c == C && cfg.w == W) {                           \
        if constexpr (shape_offered<Cell, V, C>() && backward_fits_lds<Cell, V, LLv, W>()) {   \
            static int grid_cap[4] = {0, 0, 0, 0};                                             \
            auto kern = backward_kernel<Cell, V, LLv, C, W, UT, false>;                        \
            int form = 0;                                                                      \
            if constexpr (backward_stream_offered<Cell, V, LLv, C, W>()) {                     \
                if (a.stream == 1) {                                                           \
                    kern = backward_kernel<Cell, V, LLv, C, W, UT, false, true>;               \
                    form = 2;                                                                  \
                }                                                                              \
            }                                                                                  \
            if constexpr (backward_queues_offered<Cell, V, LLv, C, W>()) {                     \
                if (a.stream == 2) {                                                           \
                    kern = backward_kernel<Cell, V, LLv, C, W, UT, false, false, true>;        \
                    form = 3;                                                                  \
                }                                                                              \
            }                                                                                  \
            if constexpr (backward_stage_offered<Cell, V, LLv, C, UT>()) {                     \
                if constexpr (backward_stage_fits_lds<Cell, C, W>()) {                         \
                    if (a.stage) {                                                             \
                        kern = backward_kernel<Cell, V, LLv, C, W, UT, true>;                  \
                        form = 1;                                                              \
                    }                                                                          \
                }                                                                              \
            }                                                                                  \
            if (grid_cap[form] == 0) grid_cap[form] = persistent_grid(kern, kWave * W, 1 << 30); \
            const int grid = a.g.n_tiles < grid_cap[form] ? a.g.n_tiles : grid_cap[form];      \
            hipLaunchKernelGGL(kern, dim3(grid), dim3(kWave * W), 0, st, a);                   \
            return hipGetLastError();                                                          \
        } else {                                                                               \
            return hipErrorInvalidValue;                                                       \
        }                                                                                      \
    }
    PARARNN_SHAPES(PARARNN_CASE)
#undef PARARNN_CASE
    return hipErrorInvalidValue;
}

}  // namespace pararnn
