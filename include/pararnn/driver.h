// Host-side driver of the diagonal / small-block paths, generic in the cell:
// argument checks, workspace layout, tile-shape choice and the enqueue
// sequence of a forward solve (Sec. 2, Alg. 1a) and of a backward pass (Eq. (6)).
// Used by the C ABI of the built-in cells and by libraries that add a cell of
// their own (pararnn_cell.h).  No kernel code here.
#pragma once
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <initializer_list>

#include "../pararnn.h"
#include "launch.h"

namespace pararnn {

// G gate pre-activations per step, S state values per channel, PR parameter rows of H floats;
// kind is the PARARNN_* constant of a built-in cell, -1 for any other cell
struct CellInfo { int G, S, PR, kind; };

// Process-wide settings of the library (pararnn_set_fused, pararnn_set_fused_head,
// pararnn_set_tile); one instance, owned by libpararnn.so.
struct Settings {
    int fused_enabled;     // launches that run several Newton iterations are allowed
    int fused_head;        // iterations in the first launch of a solve to a tolerance (0 = none)
    int tile[4];           // tile-shape override {vec, ll, c, w}; vec = 0 none
    unsigned int spin_limit;   // polls of one predecessor before a tile gives up (pararnn_set_spin_limit)
    int stage_enabled;         // kernels that copy their inputs straight into LDS are allowed (pararnn_set_staging)
    int fused_tail;            // the blocks after a solve's first launch share one persistent launch (pararnn_set_fused_tail)
    int ws_reuse;              // the caller promises that nothing else writes to a workspace between calls (pararnn_set_workspace_reuse)
    int streaming;             // streamed accesses of the HBM-bound kernels: 0 chosen by size, 1 never, 2 always (pararnn_set_streaming)
};
Settings &settings();

// Choices of one forward solve.  The C ABI's plain entry points take them from the process-wide
// settings; pararnn_forward_ex takes them from its options argument, so that two threads with
// different wishes do not meet in the settings.
struct SolveOpts {
    int fused_enabled;     // launches that run several Newton iterations are allowed
    int fused_head;        // iterations in the first launch of a solve to a tolerance (0 = none)
    bool blocks;           // the caller has chosen fused_head: a solve to a tolerance runs the blocks that follow from it
};
constexpr int kFusedHead = 5;      // the library's own choice
inline SolveOpts default_opts()
{
    const Settings &s = settings();
    return {s.fused_enabled, s.fused_head, s.fused_head != kFusedHead};
}

inline size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }

// The memory-side cache of the device (256 MiB) keeps what a launch wrote or read for the next one when
// it is left room.  A per-iteration launch reads u and reads and rewrites the fp32 iterate: u is
// streamed as soon as the two together exceed that cache (the iterate then has it to itself: measured
// 8 % on 0.8 GB of u with a 0.27 GB iterate), the iterate too once it is larger than twice the cache,
// where nothing of it survives until the next launch and streamed accesses are the faster ones (3 %).
constexpr size_t kMemCacheBytes = (size_t)256 << 20;
inline int forward_stream_level(size_t u_bytes, size_t iterate_bytes)
{
    const int mode = settings().streaming;
    if (mode == 1) return 0;
    if (mode == 2) return 2;
    if (iterate_bytes > 2 * kMemCacheBytes) return 2;
    return u_bytes + iterate_bytes > kMemCacheBytes ? 1 : 0;
}
// The backward kernel reads and writes every byte once.  Marked as streams its tensors stay out of each other's way, and out
// of the way of what the pass before left in the cache (u and h of the last steps, where this one begins).  Pays from one
// and a half times the cache on; below that the next reader of dL/du finds it in the cache.  Only rows of whole cache
// lines: a line that two channel groups share leaves the L2 before the second one asks.  Not in tiles of twelve steps a
// thread, whatever the cell (backward_tile_by_size: fp32 LSTM but for many channels of short sequences, ParaLSTM in fp32 and, of few
// channels, in bf16), which lose up to 5 % or stay level.  us of the pass, plain / streamed:
//   twelve steps  fp32 LSTM 16 x 4096 x 1024 612 / 643, 16 x 2049 x 1024 325 / 329, 8 x 4096 x 2048 604 / 607, 4 x 2048 x 2048 157 / 164;
//                 ParaLSTM 16 x 4096 x 1024 526 / 549, 7 x 3000 x 1536 262 / 271, bf16 4 x 8192 x 1024 212 / 214
//   others        fp32 16 x 2048 x 1024 GRU 212 / 192, LSTM 294 / 270, rot_tanh 223 / 200; bf16 16 x 2048 x 1024 LSTM 223 / 212, rot_tanh 146 /
//                 135, ParaLSTM 205 / 198
//   sizes         384 MB GRU fp32 87 / 79, LSTM bf16 126 / 119; 256 MB rot_tanh bf16 78 / 81; 192 MB GRU bf16 57 / 61
//   lines         rows of 1500 channels (16 x 2000) GRU fp32 371 / 412, bf16 232 / 298
inline int backward_stream(size_t bytes, bool pays)
{
    const int mode = settings().streaming;
    if (mode == 1) return 0;
    if (mode == 2) return 1;
    return pays && 2 * bytes >= 3 * kMemCacheBytes ? 1 : 0;
}

// Queues of a backward pass's tiles, one for each XCD.  Rows that are no multiple of 64 bytes: what two channel groups share of a
// cache line is read and written by both, and where they are on different XCDs comes into two L2s and leaves them in two pieces.
// With the queues neighbouring groups are on one XCD (GRU 16 x 4096 x 1025: read 1.86 -> 1.34 GB, written 0.88 -> 0.82; bf16 1.25 ->
// 0.67, 0.52 -> 0.46).  What a launch pays: who finds its queue empty looks at the others and goes on with one that is not, a few us;
// and a queue has whole groups, so there have to be enough of them.  us, one queue / eight:
//   from 512 MB on    GRU fp32 16 x 4096 x 1021 551 / 464, 64 x 4096 x 300 666 / 555, 1 x 8192 x 4091 264 / 245, bf16 16 x 4096 x 1021 354 / 317; LSTM
//                     fp32 8 x 1000 x 1531 160 / 157, 32 x 512 x 763 174 / 163, bf16 2 x 30000 x 1001 506 / 483; ParaLSTM 33 x 1999 x 500 342 / 328,
//                     bf16 16 x 4096 x 1021 521 / 464; rot_tanh fp32 9 x 700 x 3333 175 / 176, bf16 1 x 8192 x 4091 190 / 191
//   less              GRU fp32 32 x 512 x 763 114 / 109, 3 x 1531 x 1001 44 / 48, bf16 9 x 700 x 3333 117 / 123; rot_tanh 8 x 1000 x 1531 108 / 117
//   few groups        GRU fp32 11 (1 x 65536 x 700) 368 / 429, 18 560 / 611, 24 742 / 723, 33 1034 / 1010, 40 1135 / 1058; bf16 28 202 / 214
//   rows of 64 bytes  GRU fp32 1 x 60000 x 2800 1016 / 1129, LSTM 1625 / 1720
//   one group in a row (nothing is shared)  GRU fp32 64 x 16000 x 40 368 / 439, x 63 510 / 517, bf16 64 x 40000 x 50 887 / 943; LSTM fp32 64 x 12000 x 24
//                     270 / 278, bf16 64 x 20000 x 41 681 / 693; ParaLSTM 64 x 16000 x 50 545 / 561; rot_tanh bf16 64 x 40000 x 60 980 / 1029
inline bool backward_queues_pay(size_t bytes, size_t row_bytes, int n_cg, int groups)
{
    return n_cg > 1 && row_bytes % 64 != 0 && bytes >= 2 * kMemCacheBytes && groups >= 32 && 32 * ((groups + 7) / 8) <= 5 * groups;
}
// Two groups in a row of which the second has few channels: its lines are few, and scalar cells and two gates in bf16 gain less
// from them than a launch pays.  One queue / eight, of 0.7 and 2 GB: GRU fp32 x 66 234 / 248, 667 / 685, x 70 235 / 237, 651 / 654, x 74 228 / 230,
// 644 / 631, x 78 229 / 223, 643 / 599; bf16 x 70 385 / 393, 1091 / 1099, x 86 324 / 327, 925 / 904, x 90 316 / 314, 895 / 871; rot_tanh bf16 x 70 415 / 429,
// 1167 / 1194, x 86 350 / 354, x 90 341 / 341, fp32 x 66 277 / 267.  The others: LSTM fp32 x 66 241 / 241, 704 / 670, bf16 430 / 424; ParaLSTM 265 / 265.
inline bool backward_queues(const CellInfo &ci, int dtype, size_t bytes, const ScanGeom &g, const TileCfg &cfg)
{
    const bool bf = dtype == PARARNN_BF16;
    if (!backward_queues_shape(ci.S, ci.G, cfg.vec, cfg.ll, cfg.c, cfg.w)) return false;
    const int last = g.H - (g.n_cg - 1) * (kWave / cfg.ll) * cfg.vec;
    if (g.n_cg == 2 && (ci.S == 1 || (ci.G <= 2 && bf)) && last < (bf ? 24 : 10)) return false;
    return settings().streaming == 0 && backward_queues_pay(bytes, (size_t)g.H * (bf ? 2 : 4), g.n_cg, g.n_groups);
}

// Tile shape for a problem.  The table is the result of sweeps on MI355X over
// the compiled shapes (fp32 and bf16 storage, forward and backward, GRU and
// LSTM at 2^25..2^30 timestep-channels): one channel per lane
// with 128..256-byte row segments and 64..128 steps per tile.
// PARARNN_TILE="vec,ll,c,w" or pararnn_set_tile() overrides it (tuning aid; the
// combination must be one that is compiled in and allowed by H and alignment).
inline TileCfg choose_tile(const CellInfo &ci, int dtype, bool backward, int H, int align_elems, bool fused = false)
{
    int vmax = 1;
    if (H % 4 == 0 && align_elems >= 4) vmax = 4;
    else if (H % 2 == 0 && align_elems >= 2) vmax = 2;
    TileCfg cfg = {1, 2, 8, 8};                          // 32 channels x 128 steps
    const bool lstm = ci.S >= 2, bf = dtype == PARARNN_BF16;
    if (H <= 8) {
        cfg = {1, 8, 4, 2};                              // 8 channels x 64 steps
    } else if (ci.S >= 4) {
        // 4x4 blocks: 20 prefix values per step; four steps per thread (a few registers spill in the
        // fused and backward kernels, the next larger shape spills a hundred)
        cfg = {1, 1, 4, 8};                              // 64 channels x 32 steps
    } else if (ci.S == 3) {
        // 3x3 blocks: a step keeps S*S + S prefix values in registers; eight steps per thread is the
        // most that fits without spilling (190-230 registers, two waves per SIMD) and measured
        // fastest forward, fused and backward alike
        cfg = {1, 1, 8, 8};                              // 64 channels x 64 steps
    } else if (H <= 32) {
        cfg = {1, 2, 8, 8};
    } else if (fused) {
        // the fused blocks are bound by vector arithmetic, not by HBM: long per-thread chunks spread the
        // per-thread cost of the wave / workgroup / look-back levels over more cell evaluations
        if (lstm) cfg = {1, 1, 16, 4};                   // 64 channels x 64 steps
        else cfg = {1, 1, 12, 8};                        // 64 channels x 96 steps
    } else if (!backward) {
        if (lstm) cfg = {1, 1, 8, 16};                   // 64 channels x 128 steps
        else if (bf) cfg = {1, 1, 16, 8};                // 64 channels x 128 steps (3 % faster than two channels per lane on config 5)
        else cfg = {1, 1, 8, 16};                        // 64 channels x 128 steps
    } else {                                             // (backward_tile below goes by B and L as well)
        if (ci.kind == PARARNN_PARALSTM_DIAG) cfg = {1, 1, 12, 8};   // 64 channels x 96 steps
        else if (lstm && !bf) cfg = {1, 2, 8, 8};        // 32 channels x 128 steps (3 % faster than 64 x 128 on config 3)
        else if (lstm) cfg = {1, 1, 16, 8};              // 64 channels x 128 steps
        else if (bf) cfg = {1, 1, 8, 8};                 // 64 channels x 64 steps
        else cfg = {1, 1, 8, 16};                        // 64 channels x 128 steps (3-4 % faster than 32 x 256 on config 2)
    }
    // 32-bit byte offsets from a wave's first row, of u or the states or, where there are no gates, of the Jacobians
    const int *ov = settings().tile, rows = ci.PR == 0 ? ci.S * ci.S : ci.G > ci.S ? ci.G : ci.S;
    if (ov[0] > 0 && ov[0] <= vmax && (double)ov[1] * ov[2] * rows * H * 4.0 <= 4294967296.0) {
        cfg.vec = ov[0]; cfg.ll = ov[1]; cfg.c = ov[2]; cfg.w = ov[3];
    }
    return cfg;
}

// Channels that groups of `width` work on for H of them.
inline int padded_channels(int H, int width) { return (H + width - 1) / width * width; }

// The tile of the fused blocks of a scalar or 2x2 cell.  A group wider than H works for channels that are not there, and a short
// tile makes a long chain of carries: so of 8 channels x 512 steps, 16 x 256, 32 and 64 the one whose channels, times what one
// costs in it, are the fewest.  A channel costs 1.25 in groups of 8 and 1.15 in groups of 16 of what it does in 64 (scans between
// the segments of a wave).  us, before / now: GRU fp32 12 x 48925 x 8 230 / 80, 42 x 3207 x 8 113 / 38, 31 x 35271 x 16 333 / 179, 18 x
// 12000 x 24 94 / 81, 8 x 11690 x 40 83 / 68, 1 x 8609 x 72 44 / 35, 30 x 20768 x 96 509 / 442 (records asked for; else it is walked, 481); LSTM bf16 12 x 48925 x 8 460 / 200, 31 x 35271 x
// 16 700 / 543, 3 x 20000 x 48 173 / 153; ParaLSTM fp32 12 x 48925 x 8 439 / 182, 18 x 12000 x 24 164 / 127, 2 x 20000 x 288 227 / 199.
// Cells of four gates and two states have their 64 channels in fewer instructions, the others of two states their 32 (64 / 32): LSTM fp32 3 x 27718 x 256
// 499 / 522, bf16 192 438 / 480, 256 542 / 610; ParaLSTM fp32 192 269 / 258, 256 337 / 328; rot_tanh bf16 192 236 / 217.
// Scratch memory: LSTM in 32 x 128 56 to 72 bytes a lane, in 64 x 64 8 to 28, ParaLSTM in 32 x 128 28 to 52; GRU in 64 x 96 16 to 40.
// Beyond 320 channels what the padding still costs is little (64 / 32 channels): GRU fp32 2 x 30000 x 336 206 / 210, 352 204 / 202, bf16 217 / 205, 480
// 298 / 300; LSTM fp32 352 889 / 880, bf16 336 603 / 642; ParaLSTM and rot_tanh, whose 32 channels cost less, could gain: fp32 352 361 / 329, 301 / 257.
// Two-state cells have lines beside the costs (12000 problems of 5 to 340 channels with records, against the tiles before: 0.76 of the time on the mean; by costs
// alone 364 were slower by more than 3 %, worst 1.31; with the lines 13, worst 1.04):
//   25 to 32 channels   16 x 256 for few timesteps, for short tiles make long chains of carries (LSTM bf16 4 x 4721 x 32 32 x 128 in four waves 59.4, in eight 49.6,
//                       16 x 256 46.8; rot_tanh 4 x 2324 41 / 38 / 36), four waves for many (ParaLSTM 0.78-0.83 of eight from 256000 on); LSTM with whole rows in between
//                       eight (bf16 42 x 7228 x 32 524 / 428 / 433)
//   large LSTM          32 and 64 only, and 32 at 1.15 (1.5e7 elements and more: fp32 10 x 39350 x 47 610 in 64 channels, in 16 689; 12 x 47928 x 35 834, in 8 922; bf16
//                       4 x 36024 x 280 1137, in 32 1228; 6 x 39406 x 71 in 32 702, in 8 820)
//   three gates         32 at 1.08 where there are many groups (ParaLSTM fp32 53 x 7016 x 117 950 in 64 channels, in 32 1014; 53 x 2458 x 240 399 / 436)
//   up to 8 channels    more gates below 3000 timesteps the table's tile (ParaLSTM 1 x 1285 x 8 31.4, of 512 steps 33.0; LSTM 1 x 1567 34.3 / 36.5)
// lines: false for the costs alone (a workspace that does not hold the records of the short tiles: fused_layout).
struct FusedWidth { int channels; float costs; TileCfg tile; };
inline FusedWidth fused_width(const CellInfo &ci, int B, int L, int H, bool lines = true)
{
    const bool two = ci.S == 2, more = two && ci.G >= 4;
    const double steps = (double)B * L;
    const bool large = lines && more && steps * H >= 1.5e7;
    const float c32 = !two ? 1.08f : more ? (large ? 1.15f : 1.06f) : lines && ci.G == 3 && (double)B * ((H + 63) / 64) >= 100.0 ? 1.08f : 0.98f;
    const FusedWidth x64 = {64, 1.0f, two ? TileCfg{1, 1, 16, 4} : TileCfg{1, 1, 12, 8}}, x32 = {32, c32, two ? TileCfg{1, 2, 16, 4} : TileCfg{1, 2, 8, 8}},
                     x16 = {16, 1.15f, {1, 4, 8, 8}}, x8 = {8, 1.25f, {1, 8, 8, 8}};
    if (lines && two && ci.G > 2 && H <= 8 && steps < 3000.0) return {8, 1.25f, {1, 8, 4, 2}};
    if (lines && two && H > 24 && H <= 32) {
        if (steps >= (more ? 6e5 : 5e4)) return x32;
        return more && H == 32 && steps >= 2.5e5 ? FusedWidth{32, c32, {1, 2, 8, 8}} : x16;
    }
    FusedWidth best = x64;
    for (const FusedWidth &x : {x32, x16, x8}) {
        if (large && H > 32 && x.channels < 32) break;
        if (x.costs * (float)padded_channels(H, x.channels) < best.costs * (float)padded_channels(H, best.channels)) best = x;
    }
    return best;
}
inline bool fused_by_width(const CellInfo &ci, int L, int H) { return ci.S <= 2 && L > 256 && H <= 320; }
inline TileCfg fused_tile(const CellInfo &ci, int B, int L, int H, const TileCfg &table)
{
    return settings().tile[0] <= 0 && fused_by_width(ci, L, H) ? fused_width(ci, B, L, H).tile : table;
}

// The tile of a backward pass of a scalar or 2x2 cell with carry records, by sweeps over 300 to 60000 steps of 2048 to 65792
// channels in all (times / times of choose_tile's shape with its rows staged whenever they can be).  Rows of whole lines
// (64 channels, bf16) are worth staging once the tensors are far larger than the last-level cache; before that, and for
// other rows, plain loads are faster (GRU 8 x 1000 x 1536 0.85, 32 x 700 x 2056 0.71).
//   scalar   bf16: 64 channels x 64 steps; of few channels, or of up to 8192 with long sequences, x 128 (2 x 1536 x 1024 0.67, 2 x 32768 x
//            2048 staged 0.88)
//   2x2      two gates: 64 x 64 in four waves (bf16 8 x 700 x 1536 0.87, fp32 8 x 4096 x 1536 0.87); of few channels eight waves
//            in bf16 (2 x 1001 x 1024 0.64), 32 x 128 in fp32
//   more     bf16 LSTM: x 128 staged from 1.8e7 elements on (8 x 2048 x 2048 260 -> 206 us), before that x 96 and, with 8192
//   gates    channels or more, x 32 (16 x 300 x 2048 0.86); rows of other lengths 0.8-0.9 with the same.  ParaLSTM: x 96, or x 64
//            staged (16 x 2048 x 2048 0.91).  fp32: x 96 instead of 32 x 128 (0.81-0.98), x 32 for many channels up to 2048
//            steps (8 x 2048 x 1536 0.90)
inline TileCfg backward_tile_by_size(const CellInfo &ci, int dtype, int B, int L, int H, const TileCfg &table)
{
    const bool bf = dtype == PARARNN_BF16, whole = H % 64 == 0;
    const double channels = (double)B * H, n = channels * L;
    const TileCfg x32 = {1, 1, 4, 8}, x64 = {1, 1, 8, 8}, x96 = {1, 1, 12, 8}, x128 = {1, 1, 16, 8}, x128w = {1, 1, 8, 16}, x64n = {1, 1, 16, 4};
    if (ci.S == 1) return !bf ? table : channels < 4096 || (channels <= 8192 && L >= 4096) ? x128w : x64;
    if (ci.G <= 2) return channels >= 6000 ? x64n : bf ? x128 : table;
    if (ci.kind == PARARNN_PARALSTM_DIAG) {
        if (!bf || channels < 8192) return x96;
        return whole ? (n >= 1.6e7 ? x64 : x96) : channels >= 32768 ? x32 : x96;
    }
    if (!bf) return channels < 1024 ? table : channels >= 12288 && L <= 2048 ? x32 : x96;
    if (whole && n >= 1.8e7) return x128;
    return channels >= (whole ? 8192 : 32768) ? x32 : x96;
}
// ... as far as a workgroup's sums for the parameter rows leave room for it: shapes beyond 64 KB of LDS are not built
// (backward_fits_lds in launch_impl.h).
inline bool backward_tile_fits(const CellInfo &ci, const TileCfg &t)
{
    const size_t rows = (size_t)(ci.S * ci.S + ci.S > ci.PR ? ci.S * ci.S + ci.S : ci.PR);
    return (t.w * rows + ci.S) * (size_t)(64 / t.ll) * t.vec * sizeof(float) + 16 <= 65536;
}
// Narrow rows, as the fused blocks' tile above (a pass is bound by memory sooner, so that narrow groups cost more).  us, before / now: GRU fp32 12 x 48925 x 8
// 190 / 48, 42 x 3207 x 8 67 / 19, 31 x 35271 x 16 352 / 163, 18 x 12000 x 24 70 / 54, 30 x 20768 x 96 434 / 401; LSTM bf16 12 x 48925 x 8 179 / 62, 31 x 35271 x 16
// 345 / 171, 18 x 12000 x 24 82 / 68, 3 x 20000 x 48 52 / 42; ParaLSTM fp32 60 x 16549 x 8 289 / 101, 31 x 35271 x 16 432 / 196; rot_tanh bf16 30 x 20768 x 96
// 494 / 351.  12000 passes of 5 to 340 channels, against the tiles before: 0.86 of the time on the mean, 73 slower by more than 3 % (worst 1.10).
// A group of 32 channels is a line of 128 bytes in fp32 and half of one in bf16: where rows are no multiple of it, neighbouring groups share lines, which costs more than the
// padding of 64 channels.  And where the tiles are one round of the device (256, a workgroup on each unit) and the narrower ones are too, those are faster; where only they
// or only the wider ones are, these (ParaLSTM fp32 16 x 749 x 94 256 wide tiles 21.2, 288 narrow 25.7; bf16 13 x 862 x 81 234, 22.6, and 312, 25.4; GRU bf16 4 x 4895 x 92
// 312, 26.6, and 240, 23.3).  Lines of the rule (narrow / wide):
//   scalar, 17 to 32  256 steps from 28000 timesteps on (fp32; 8000 to 16000 1.03-1.10, 32000 0.92, 45000 0.82), in bf16 from 40000 (2 x 15789 x 24 25.2 / 23.1,
//                     12 x 3000 x 17 22.4 / 21.8, x 24 22.6 / 22.9, 4 x 12000 24.0 / 27.7, 1 x 60000 29.5 / 37.3), rows of 32 from 34000 (2 x 15789 22.2 / 21.7, 12 x 3000
//                     17.8 / 18.8, 6 x 6000 18.4 / 20.0)
//   scalar, 65 to 96  fp32 96 0.94-0.99, others up to 28000 timesteps 0.86-1.01, beyond 1.00-1.17 (not of one sequence, 0.93-1.0); bf16 96 0.80-0.97, others of 10000 steps
//                     and more 0.84-1.06, of less 1.0-1.12; 160, in place of 64 x 128, 0.87-1.03.  Other rows: bf16 129 to 160 0.97-1.27, 193 to 224 0.94-1.31, 257 to 288
//                     0.96-1.30
//   two gates, bf16   17 to 32: four waves of 16 steps from 40000 timesteps on (8000 to 32000 1.02-1.11, 128000 0.85-0.95); 65 to 96 0.76-1.0, 129 to 160 0.82-1.09, 224 and
//                     288 0.87-0.95, other rows of these widths 0.96-1.13.  fp32: the shapes by size (76 x 2683 x 81 178, 32 x 128 191)
//   more gates, fp32  65 to 96: whole rows 0.83-1.06; others LSTM up to 3.5e6 elements 0.90-1.06, beyond 0.92-1.10 (1.03 on the mean), ParaLSTM of more than a round 1.0-1.22
//   more gates, bf16  groups of 16 where they save channels and both are a round; else five eighths of the channels up to 8e6 elements 0.79-1.05 (beyond 1.05-1.14), three
//                     quarters, of one group of 64 the same, of several up to 2.5e6 (beyond 1.05-1.3); groups of 32 for 65 to 96 channels 0.84-1.10, for 129 to 160 1.0-1.14
// Groups of 16 for 17 to 32 channels (16 / 32): more gates in bf16 (LSTM 3 x 2000 x 24 16.5 / 18.5, 12 x 12000 x 24 51 / 60, 18 x 12000 x 32 68 / 79; ParaLSTM 64 x 12000 x 24
// 241 / 293); in fp32 they lose more than they gain (LSTM 3 x 2000 x 24 16.3 / 18.1, 64 x 12000 x 24 340 / 279, 18 x 12000 x 32 109 / 94; ParaLSTM 58 / 64 of 12 x 12000 x 24,
// 99 / 84 of 18 x 12000 x 32).  Beyond 320 channels the shapes by size are the faster ones or within 5 % but for ParaLSTM fp32 4 x 4000 x 352 (56 / 52) and rot_tanh bf16
// (3 x 6000 x 416 51 / 47, 2 x 9000 x 544 61 / 57).  Not at sizes and rows for which there are queues, for which these shapes are not built (GRU fp32 64 x 16000 x 90 in queues
// 796, these shapes 947; x 72 from one queue 734, 765; rot_tanh bf16 40 x 20000 x 72 would gain, 528 / 449).  Registers (of 128 for four waves a SIMD): scalar cells take 129 in
// tiles of 512 steps and of 16 channels, 131 in 32 x 128, so that a unit holds one workgroup of eight waves; 32 x 256 is one of sixteen within 128, with 20 bytes of
// scratch a lane (35 x 14020 x 24 123, 32 x 128 168).
inline TileCfg backward_tile_narrow(const CellInfo &ci, int dtype, int B, int L, int H, const TileCfg &wide)
{
    const bool bf = dtype == PARARNN_BF16, two_gates = ci.S == 2 && ci.G <= 2;
    const TileCfg x8 = {1, 8, 8, 8}, x16 = {1, 4, 8, 8}, x32 = {1, 2, 8, 8}, x32l = ci.S == 1 ? TileCfg{1, 2, 8, 16} : TileCfg{1, 2, 16, 4};
    const double steps = (double)B * L, n = steps * H;
    if (L <= 256 || H > 320) return wide;
    // (less than a workgroup of the short tile for each unit: LSTM bf16 7 x 1404 x 8 16.8, of 512 steps 19.2; 8 x 1800 18.4 / 17.8)
    if (H <= 8) return ci.S == 2 && steps < 12800.0 ? wide : x8;
    if (H <= 16) return x16;
    if (H <= 32) {
        if (ci.S == 1) return steps < (!bf ? 2.8e4 : H == 32 ? 3.4e4 : 4e4) ? x32 : x32l;
        if (two_gates) return bf && steps >= 4e4 ? x32l : x32;
        return bf && n < 8e6 ? x16 : x32;
    }
    const size_t row = (size_t)H * (bf ? 2 : 4);
    if (backward_queues_pay((size_t)B * L * row * (2 * ci.G + 2 * ci.S), row, (H + 63) / 64, B * ((H + 63) / 64))) return wide;
    // of the channels that groups of 64 work on, and whether tiles are one round
    const float part32 = (float)padded_channels(H, 32) / (float)padded_channels(H, 64), part16 = (float)padded_channels(H, 16) / (float)padded_channels(H, 64);
    auto one_round = [&](int width, int T) { return (double)B * ((H + width - 1) / width) * ((L + T - 1) / T) <= 256.0; };
    const bool whole = H % 32 == 0, save32 = part32 < 0.76f;
    if (ci.S == 1) {
        if (whole && (save32 || (bf && part32 < 0.84f && wide.w == 16))) return x32l;
        if (!save32) return wide;
        if (!bf) return steps < 2.8e4 || B == 1 ? x32l : wide;
        return (L >= 10000 && steps >= 1.8e4) || (one_round(32, 256) && !one_round(64, 128)) ? x32l : wide;
    }
    if (two_gates) return bf && (part32 < (whole ? 0.91f : 0.84f) || (part32 < 0.95f && one_round(32, 128))) ? x32l : wide;
    const bool one = one_round(64, 96);
    if (!bf) return save32 && (whole || (ci.G >= 4 ? n < 3.5e6 : one && one_round(32, 128))) ? x32 : wide;
    if (one && part16 < 0.89f) return one_round(16, 256) ? x16 : save32 && one_round(32, 128) ? x32 : wide;
    if (part16 < 0.76f && n < (part16 < 0.63f || H <= 64 ? 8e6 : 2.5e6)) return x16;
    return save32 ? x32 : wide;
}
inline TileCfg backward_tile(const CellInfo &ci, int dtype, int B, int L, int H, const TileCfg &table)
{
    if (ci.S > 2 || settings().tile[0] > 0) return table;
    const TileCfg wide = H <= 32 ? table : backward_tile_by_size(ci, dtype, B, L, H, table), t = backward_tile_narrow(ci, dtype, B, L, H, wide);
    return backward_tile_fits(ci, t) ? t : backward_tile_fits(ci, wide) ? wide : table;
}
// ... and whether its rows are staged.  3x3 blocks: one workgroup of 64 x 64 steps on a compute unit then, for its rows take 99 KB of
// LDS; tri_tanh staged / plain: 2e6 to 4e6 elements 1.05-1.27, 8e6 0.98-1.06, 1.2e7 0.95-1.0, 6e7 0.85-0.89.
inline bool backward_staged(const CellInfo &ci, int B, int L, int H)
{
    const double n = (double)B * L * H;
    if (ci.S > 2) return H % 64 == 0 && n >= 1.2e7;
    return H % 64 == 0 && n >= (ci.S == 1 ? 4e7 : ci.G <= 2 ? 3e7 : 0.0);
}

struct Layout {
    ScanGeom g;
    TileCfg cfg;
    size_t off_rec, n_rec, off_bnd, off_iter, off_part, total;
};

// What decides where a call's carry records lie and how they are read: two calls with the same
// signature on the same workspace use every record word for the same thing.  Never 0.
inline unsigned long long layout_signature(int pass, const CellInfo &ci, int dtype, const Layout &lo, int rec_slots)
{
    unsigned long long h = 1469598103934665603ull;
    const long long v[] = {pass, ci.kind, ci.S, ci.G, ci.PR, dtype, lo.g.B, lo.g.L, lo.g.H, lo.g.T, lo.g.n_lt, lo.g.n_cg,
                           lo.cfg.vec, lo.cfg.ll, lo.cfg.c, lo.cfg.w, rec_slots, (long long)lo.n_rec,
                           (long long)lo.off_rec, (long long)lo.total};
    for (long long x : v) {
        for (int i = 0; i < 8; ++i) {
            h ^= (unsigned long long)(x >> (8 * i)) & 0xffull;
            h *= 1099511628211ull;
        }
    }
    return h ? h : 1ull;
}

// largest max_iter whose epochs fit below the per-call number in a record tag (tag = epoch * 4 + state,
// epoch = number * 1024 + iteration)
constexpr int kMaxIterWithReuse = 1000;

// Workspace: [Ctrl | carry records (rec_slots sets) | boundary rows | fp32 iterate (bf16 forward) |
// parameter-gradient partials (backward)]
inline Layout make_layout(const CellInfo &ci, int dtype, int B, int L, int H, bool backward, int align_elems,
                          bool fused = false, int rec_slots = 1, const TileCfg *force = nullptr)
{
    Layout lo;
    lo.cfg = force ? *force : choose_tile(ci, dtype, backward, H, align_elems, fused);
    if (backward && !force) lo.cfg = backward_tile(ci, dtype, B, L, H, lo.cfg);
    if (fused && !force) lo.cfg = fused_tile(ci, B, L, H, lo.cfg);
    const int CW = (kWave / lo.cfg.ll) * lo.cfg.vec, T = lo.cfg.c * lo.cfg.ll * lo.cfg.w;
    ScanGeom &g = lo.g;
    g.B = B; g.L = L; g.H = H; g.T = T;
    g.n_lt = (L + T - 1) / T;
    g.n_cg = (H + CW - 1) / CW;
    g.n_groups = B * g.n_cg;
    g.n_tiles = g.n_groups * g.n_lt;
    g.spin_limit = settings().spin_limit;
    g.epoch_base = 0;
    const size_t NW = (size_t)ci.S * ci.S + 2 * ci.S;
    size_t off = round256(sizeof(Ctrl));
    lo.n_rec = (size_t)g.n_tiles * NW * CW;
    lo.off_rec = off;   off += round256(lo.n_rec * (size_t)rec_slots * sizeof(unsigned long long));
    lo.off_bnd = off;
    if (!backward) off += round256((size_t)2 * g.n_lt * B * ci.S * H * sizeof(float));
    lo.off_iter = off;
    if (!backward && dtype == PARARNN_BF16) off += round256((size_t)B * L * ci.S * H * sizeof(float));
    lo.off_part = off;
    if (backward) off += round256((size_t)g.n_lt * B * ci.PR * H * sizeof(float));
    lo.total = off;
    return lo;
}

// The layout of a solve's blocks that `fits` takes, given the layout and its bytes; false where there is none.  Short tiles need more records, 64 x 64
// four times those of 16 x 256: a workspace that holds only the latter still has its iterations in one launch (LSTM fp32 10 x 39350 x 47 on 32 MiB 687 us, with
// a launch for each iteration 1130).
template <class F>
inline bool fused_layout(const CellInfo &ci, int dtype, int B, int L, int H, int align_elems, int n_fused, bool to_tol, F fits, Layout *lf)
{
    *lf = make_layout(ci, dtype, B, L, H, false, align_elems, true, n_fused);
    if (fits(*lf, to_tol ? lf->total : lf->off_bnd)) return true;
    if (settings().tile[0] > 0 || !fused_by_width(ci, L, H)) return false;
    const TileCfg other = fused_width(ci, B, L, H, false).tile;
    *lf = make_layout(ci, dtype, B, L, H, false, align_elems, true, n_fused, &other);
    return fits(*lf, to_tol ? lf->total : lf->off_bnd);
}

// Shape of the kernels of short_kernels.h for a problem: c steps per thread, 64 >> lps_log2 segments per wave, w waves;
// n_items workgroups that walk their sequence in n_tiles tiles.
// `walk`: of those of walk_kernels.h, where the group of a workgroup is w times as wide.
struct ShortShape { int c, lps_log2, w, n_cg, n_items, n_tiles; bool walk = false; };

// What a forward solve takes with the kernels that have carry records and with these, in us.  With records the time follows
// the number of timestep-channels, and tiles of one channel group wait for each other: few groups cost more per
// timestep-channel.  Without, the workgroups of a solve go through the device in rounds, as many at a time as the kernel's
// registers allow; a round is the whole sequence, tile by tile, and the time of a tile depends on how many waves share a
// SIMD.  So just above a full round the solve takes up to twice as long (two-state cell, bf16, 16000 steps, best shapes:
// 1024 channels 0.83 of the time with records, 1100 channels 1.16, 2048 0.82, 2100 1.10), and a shape is chosen that fills
// its last one.
// The constants are a least-squares fit to 1100 problems on MI355X, each with every shape and with records (scalar and 2x2
// cells, fp32 and bf16, to a tolerance and with three fixed iterations, 200 to 50000 steps of 300 to 131072 channels): 5-6 %
// root mean square of either side.  Of 1560 problems 4 take more than 3 % longer this way than with records (worst 7 %), of
// 920 random ones the fit has not seen 9 (worst 1.3 times: a fixed count of eight); lines drawn by size had left 247 and 127
// (worst 2.3 times).  On 520 of the random ones, timed with every shape, the time is 2.9 % above the fastest on the mean, where
// those lines were 9.5 % above; 24 of them are more than 3 % slower than by the lines (worst 1.54: a single fixed iteration).
// A fit to those 520 themselves does no better on the half it has not seen.
struct ShortCost {
    float step, step_gate;            // per million timestep-channels and iteration: a part, and one for each gate
    float rec_more, rec_tol, rec_fixed;   // with records: iterations' worth of loads and stores; launches, to a tolerance and fixed
    float rec_tile, rec_narrow;       // a tile of the sequence and iteration; log2 of how far the groups are from 512
    float more, start;                // without: the same two
    struct { float one, wave; } tile[2][2];   // [8, 16 steps][one tile, several]: of a tile, and for each wave on its SIMD
    float piece[4];                   // rows in pieces of 4, 8, 16, 32 channels
    float wide;                       // workgroups of more than four waves, for pieces of four channels (wider ones: less)
    float uneven;                     // five to seven waves take the places of eight and less of the arithmetic
    float last, drift[2], bf16, few;  // a last round after two; doubling of the tiles (fp32, bf16); bf16; few workgroups
    float overlap[2];                 // each of up to four rounds, one tile and several: workgroups do not end at once
};
constexpr ShortCost kCostScalar = {0.0f, 0.263f, 3.14f, 27.7f, 20.7f, 0.0171f, 0.0637f, 3.56f, 5.59f,
                                   {{{0.411f, 0.557f}, {0.595f, 0.504f}}, {{0.664f, 1.077f}, {0.716f, 1.184f}}},
                                   {1.0f, 0.917f, 0.887f, 0.878f}, 0.272f, 0.705f, 0.799f, {0.0161f, 0.0066f}, 0.968f, 0.166f,
                                   {0.0333f, 0.0215f}};
constexpr ShortCost kCostBlock2 = {0.512f, 0.456f, 0.847f, 33.4f, 24.0f, 0.0196f, 0.0728f, 2.36f, 5.97f,
                                   {{{0.299f, 0.448f}, {0.519f, 0.363f}}, {{0.623f, 0.764f}, {0.623f, 0.764f}}},
                                   {1.0f, 0.918f, 0.879f, 0.846f}, 0.283f, 0.561f, 0.906f, {0.0144f, 0.0097f}, 0.981f, 0.140f,
                                   {0.0333f, 0.0f}};
constexpr int kShortUnits = 256;      // compute units
constexpr int kShortIters = 5;        // iterations of a solve to a tolerance: what the cells take nearly everywhere

// n_iters: of a solve of a fixed count, 0 = to a tolerance
inline float records_us(const ShortCost &k, const CellInfo &ci, int dtype, int B, int L, int H, int n_iters)
{
    // the tiles that the constants are of: choose_tile's of the fused blocks
    const int width = H <= 8 ? 8 : H <= 32 ? 32 : 64, T = H <= 8 ? 64 : H <= 32 ? 128 : ci.S == 1 ? 96 : 64;
    const float groups = (float)B * (float)((H + width - 1) / width), n_lt = (float)((L + T - 1) / T);
    const float n = groups * (float)width * n_lt * (float)T * 1e-6f;
    // a fixed count beyond the fused blocks is one launch per iteration, at the rate of the memory
    if (n_iters > kMaxFused)
        return (float)n_iters * (6.0f + n * ((float)ci.G * (dtype == PARARNN_BF16 ? 2.0f : 4.0f) + 8.0f * (float)ci.S) / 5.4f);
    const float its = (float)(n_iters ? n_iters : kShortIters);
    float step = (k.step + k.step_gate * (float)ci.G) * (its + k.rec_more), fixed = n_iters ? k.rec_fixed : k.rec_tol;
    // The LSTM's sixth iteration is a launch of its own, which reads and writes the iterate, and there are channels that
    // take a seventh: 1.45 of the time of five, or twice it, where a walk takes 1.05.  Six or seven is what the
    // benchmark's weights (up to 0.9, forget bias 1) take; they are not known here.  With weights up to 0.5 or without the
    // bias it is five, and where the two are close records would be faster, by up to 1.46 (1024 channels x 50000 fp32: 882 us
    // against 1284; with six iterations 1233 against 1302; 4200 x 50000 3237 against 4407, with seven 6916 against 4982).
    if (ci.kind == PARARNN_LSTM_DIAG && !n_iters) { step *= 1.45f; fixed += 8.7f; }
    const float narrow = groups < 512.0f ? log2f(512.0f / groups) : 0.0f;
    const float us = fixed + step * n * (1.0f + k.rec_narrow * narrow) + k.rec_tile * its * n_lt;
    // Narrow rows take narrower tiles (fused_width), and the time is that of the channels that these work on; of 9 to 16 channels about
    // half.  1.3 times that where it is less: against 13000 problems of 5 to 320 channels, timed with records, in one workgroup
    // and walked, this changes 49 choices, 46 to kernels that take 0.58 to 0.97 of the time (GRU fp32 68 x 48892 x 16 walked 738,
    // with records 424; LSTM fp32 47 x 14802 x 16, three iterations, one workgroup 254, 159; ParaLSTM 52 x 52160 x 16 1023 / 749), the worst 1.02.
    // Without the factor it is a hundred slower by more than 3 % (worst 1.6), for the estimates of the others are up to a third
    // above their times there; nor up to 2048 steps (GRU bf16 85 x 1664 x 16, eight iterations, 49 us, in one workgroup 44) and
    // for two gates and two states (rot_tanh bf16 43 x 15499 x 16 186 / 159).
    if (fused_by_width(ci, L, H) && L > 2048 && !(ci.S == 2 && ci.G <= 2)) {
        const FusedWidth w = fused_width(ci, B, L, H);
        const float part = w.costs * (float)padded_channels(H, w.channels) / (float)padded_channels(H, width);
        const float by_width = 1.3f * (fixed + step * n * part * (1.0f + k.rec_narrow * narrow) + k.rec_tile * its * n_lt);
        if (by_width < us) return by_width;
    }
    return us;
}
inline float short_us(const ShortCost &k, const CellInfo &ci, int dtype, const ShortShape &sh, int n_iters)
{
    const bool many = sh.n_tiles > 1, bf = dtype == PARARNN_BF16;
    // waves of a workgroup on one SIMD; a workgroup of five takes two on each, as one of eight does
    const float waves = sh.w <= 4 ? 0.25f * (float)sh.w : (float)((sh.w + 3) / 4);
    int per_unit = (int)((float)short_min_waves(ci.S, sh.c, many || (sh.c > 8 && ci.S > 1)) / waves);
    if (per_unit < 1) per_unit = 1;
    const int full = sh.n_items / (kShortUnits * per_unit), left = sh.n_items - full * kShortUnits * per_unit;
    const auto &t = k.tile[sh.c > 8][many];
    auto round = [&](int per) {
        float on = waves * (float)per;
        if (sh.w > 4 && sh.w < 8) on *= 1.0f - k.uneven * (1.0f - 0.125f * (float)sh.w);
        return t.one + t.wave * on;
    };
    float rounds = (float)full * round(per_unit);
    if (left) rounds += round((left + kShortUnits - 1) / kShortUnits) * (full > 1 ? k.last : 1.0f);
    rounds *= 1.0f - k.overlap[many] * (float)(full < 4 ? full : 4);
    if (sh.w > 4) rounds *= 1.0f + k.wide / (float)(sh.lps_log2 - 1);
    rounds *= k.piece[sh.lps_log2 < 5 ? sh.lps_log2 - 2 : 3] * (bf ? k.bf16 : 1.0f);
    rounds *= 1.0f + k.drift[bf] * log2f((float)sh.n_tiles);
    if (sh.n_items < kShortUnits) rounds *= 1.0f - k.few * (1.0f - (float)sh.n_items / (float)kShortUnits);
    const float its = (float)(n_iters ? n_iters : kShortIters);
    return k.start + (k.step + k.step_gate * (float)ci.G) * (its + k.more) * (float)sh.n_tiles * rounds;
}

// Completes a shape (c, lps_log2, w); false where it is outside the kernels' bounds.
inline bool short_complete(const CellInfo &ci, int dtype, int B, int L, int H, ShortShape *sh)
{
    const int T = sh->c * (64 >> sh->lps_log2) * sh->w;
    // 32-bit offsets within a tile, of u and of the states, whichever rows are wider
    const double esz = dtype == PARARNN_BF16 ? 2.0 : 4.0;
    if ((double)(ci.G > ci.S ? ci.G : ci.S) * H * esz * (T + 1.0) >= 2147483647.0) return false;
    sh->n_cg = (H + (1 << sh->lps_log2) - 1) >> sh->lps_log2;
    if ((double)B * sh->n_cg > 131072.0) return false;       // verdicts that workgroup 0 collects
    sh->n_items = B * sh->n_cg;
    sh->n_tiles = (L + T - 1) / T;
    return true;
}

// One tile: the fewest segments per wave with which `want` waves hold the sequence, as few waves as that takes.
inline bool short_one_tile(int L, int c, int want, int most, ShortShape *sh)
{
    int ll = 1;
    while (ll < 16 && c * ll * want < L) ll *= 2;
    sh->c = c;
    sh->w = (L + c * ll - 1) / (c * ll);
    sh->lps_log2 = 6;
    while ((64 >> sh->lps_log2) < ll) --sh->lps_log2;
    return sh->w <= most;
}

// Channels that the kernels with records work on for each one there is, in groups of choose_tile's width: the time of a
// narrow H is that of a full group (3x3 cells fp32, 478 steps x 52 x 19, 260 workgroups, three iterations: 0.66 of it).  Backward passes of
// scalar and 2x2 cells have narrower tiles there (backward_tile_narrow), but at the 257 to 2048 steps that ask for it, full groups are the better
// estimate: of 5400 passes of 5 to 320 channels what they choose is 1.1 % above the faster kernel on the mean, the tiles' own widths 1.2 %.
inline double records_padding(const CellInfo &ci, int dtype, int H, bool backward)
{
    const TileCfg cfg = choose_tile(ci, dtype, backward, H, 1, !backward);
    const int width = cfg.vec * (64 / cfg.ll);
    return (double)((H + width - 1) / width) * width / (double)H;
}

// The shape of a forward solve, or false where the kernels with carry records do better.  n_iters: 0 = to a tolerance.
inline bool short_forward_shape(const CellInfo &ci, int dtype, int B, int L, int H, int n_iters, ShortShape *out)
{
    const bool tiny = (double)B * L * H < 512.0 * 512.0 && L <= 1024;
    const ShortCost &k = ci.S == 1 ? kCostScalar : kCostBlock2;
    // the fit has counts of three; two or twelve are estimated from it
    const float better = n_iters == 0 || (n_iters >= 3 && n_iters <= 5) ? 0.97f : 0.85f;
    ShortShape sh;
    if (tiny || L <= 512 || ci.S > 2) {
        // One tile.  Steps per thread: below half a wave per SIMD at eight of them the chunk's own latency counts (GRU
        // 4 x 250 x 100: eight steps 10.9 us, four 9.8), blocks of 3x3 and larger spill beyond four.  Four waves iterate
        // fastest: two barriers in every iteration, and workgroups of eight leave fewer of them on a compute unit.
        const int c = ci.S > 2 || tiny ? 4 : 8;
        if (!short_one_tile(L, c, 4, ci.S * c <= 8 ? 16 : 8, &sh) || !short_complete(ci, dtype, B, L, H, &sh)) return false;
        *out = sh;
        if (ci.S > 2) {
            // 3x3 / 4x4 cells, times / times with records.  To a tolerance up to 256 steps 0.3-0.98.  Three fixed iterations: 40-64
            // steps 0.47-0.96, 3x3 72-128 steps of 2000 workgroups 0.84-0.94, of 4000 0.9-1.02, 192-256 of 1000 0.72-0.81, of 2000
            // 0.97-1.03; 4x4 72-256 of 1000 0.85-1.02, of 2000 0.96-1.3.  Eight: 72-256 of 500 0.6-0.78, of 1000 0.84-1.24.  More than
            // eight are a launch each with records: up to 256 steps 0.18-0.82, 320-500 of 2000 0.83-1.03, of 4000 0.91-1.22.
            // Beyond 256 steps, with five to eight waves, of which a unit holds one workgroup: 256 of them 0.4-0.8, 500 to a
            // tolerance 0.8-1.0 and fixed 1.2-1.5, 1000 1.0-1.2 and 1.4-2.0.
            const double units = kShortUnits * records_padding(ci, dtype, H, false);
            if (n_iters > kMaxFused) return L <= 256 || sh.n_items <= 8 * units;
            if (L > 256) return sh.n_items <= units * (n_iters ? 1 : 2);
            return L <= 64 || n_iters == 0 || sh.n_items <= units * (n_iters > 5 ? 3 : ci.S > 3 ? 4 : L <= 128 ? 12 : 6);
        }
        // below 160 steps the kernels with records are nowhere faster (131072 channels: 0.87-0.93 of their time)
        return tiny || L < 160 || short_us(k, ci, dtype, sh, n_iters) < better * records_us(k, ci, dtype, B, L, H, n_iters);
    }
    // what long sequences of scalar cells lose by their groups drifting apart in time (they no longer share the cache lines
    // of a row) is fitted up to 16384 steps: 65536 x 4 x 4096 in bf16 took 8453 us against 7602 with records
    if (ci.S == 1 && L > 16384) return false;
    float best = better * records_us(k, ci, dtype, B, L, H, n_iters);
    bool found = false;
    for (int c = 8; c <= 16; c += 8)
        for (int lps = 2; lps <= 5; ++lps)
            for (int w = 4; w <= 8; w += 4) {
                const int row = c * (64 >> lps), most = (L + row - 1) / row;
                sh.c = c; sh.lps_log2 = lps; sh.w = w < most ? w : most;
                if (!short_complete(ci, dtype, B, L, H, &sh)) continue;
                const float us = short_us(k, ci, dtype, sh, n_iters);
                if (us < best) { best = us; *out = sh; found = true; }
            }
    return found;
}

// The shape of a backward pass: one pass over one tile.  It takes all the waves there may be, for longer pieces of rows; two-state
// cells of 65 to 192 steps take four where a round of the device does not hold all groups, because a unit holds three
// such workgroups and one of five to eight waves (LSTM bf16 192 x 16 x 2048: 0.72 of the time with records, with six waves
// 0.95; 192 x 4 x 1024: 0.56 and 0.53).  Long sequences mean short pieces (four channels per group in the end), for which the
// memory pipeline needs as many cycles as for whole lines: fine where latency bounds the other kernels too, not on large
// tensors.  Bounds on the bytes of a pass, where the two are level: times / times with records,
//   scalar   128 steps fp32 131072 channels 1.13-1.27, 65536 0.98; 256: fp32 32768 0.97-1.03, bf16 65536 1.0, 131072 1.2; 512:
//            fp32 16384 0.93, bf16 32768 1.1; 1024: fp32 1332 1.0, bf16 8000 0.94; 1500: bf16 1024 0.73, 1332 1.33; 1537-2048: up
//            to 64 workgroups 0.66-0.96, 128 0.82-1.22, 250 0.72-1.32
//   2x2      96 steps fp32 65536 0.7-0.9, 131072 0.9-1.1; 160: fp32 32768 0.65-0.8, 65536 0.85-1.2; 192: fp32 16384 0.75-0.87,
//            32768 0.77-1.07; 256: fp32 16384 0.82-0.99, 32768 0.84 (two gates) to 1.32, bf16 32768 0.8-1.0, 65536 0.92 (two
//            gates) to 1.31; 320-384: one round of the device, 2048 channels, 0.6-0.9; two 0.98-1.18; 448-512: two 0.9-1.0,
//            four 0.92-1.07; two gates: two rounds 0.8-0.95, four 0.8-1.1
//   3x3, 4x4 up to 64 steps 1000 workgroups 0.84-0.96, 4000 1.05; 72-128 500 0.68-0.88, 1000 0.89-1.16, 2000 0.97-1.3; 192-256
//            500 0.86-0.95, 1000 1.1-1.3; 320-512 one round (a workgroup on each unit) 0.6-0.85, two 0.99-1.4
inline bool short_backward_shape(const CellInfo &ci, int dtype, int B, int L, int H, ShortShape *out)
{
    const double n = (double)B * L * H, bytes = n * (dtype == PARARNN_BF16 ? 2.0 : 4.0) * (2 * ci.G + 2 * ci.S);
    const int c = ci.S > 2 || (n < 512.0 * 512.0 && L <= 1024) ? 4 : 8, most = ci.S * c <= 8 ? 16 : 8;
    if (!short_one_tile(L, c, most, most, out) || !short_complete(ci, dtype, B, L, H, out)) return false;
    const int per_gate = ci.G <= 2 ? 2 : 1;
    const double units = kShortUnits * records_padding(ci, dtype, H, true);
    if (ci.S == 2 && c == 8 && L > 64 && L <= 192 && out->n_items > kShortUnits * per_gate &&
        (!short_one_tile(L, c, 4, most, out) || !short_complete(ci, dtype, B, L, H, out)))
        return false;
    if (ci.S == 1)
        return L <= 64 || (bytes <= (L <= 256 ? 400e6 : L <= 512 ? 192e6 : L <= 1024 ? 96e6 : 32e6) &&
                           (L <= 1024 || out->n_items <= units * (L <= 1536 ? 1.0 : 0.25)));
    if (L > 512) return false;
    if (ci.S > 2) return L <= 32 || out->n_items <= units * (L <= 64 ? 8 : L <= 128 ? 3 : L <= 256 ? 2 : 1);
    if (L <= 256) return L <= 64 || bytes <= (L <= 96 ? 420e6 : L <= 160 ? 340e6 : L <= 192 ? 250e6 : 280e6);
    return bytes <= 192e6 && (c == 4 || out->n_items <= units * per_gate * (L > 384 || per_gate > 1 ? 2 : 1));
}

inline bool short_shape(const CellInfo &ci, int dtype, int B, int L, int H, bool backward, int n_iters, ShortShape *out)
{
    return backward ? short_backward_shape(ci, dtype, B, L, H, out) : short_forward_shape(ci, dtype, B, L, H, n_iters, out);
}
// What a forward solve takes where waves walk sequences on their own (walk_kernels.h), in us: rounds of the device as above,
// with the copies and stores of the tiles beside them.  Rows shorter than a cache line (128 bytes) cost a request each, and what
// neighbouring workgroups share of a line comes in again once these have drifted apart, the more the longer the sequence.  The
// constants are a fit to 3400 measurements (scalar and 2x2 cells, fp32 and bf16, to a tolerance and with three fixed
// iterations, 200 to 65536 steps of 1024 to 131072 channels, every shape): 5-7 % root mean square.  On those 600 problems the
// shape it takes is 3.0 % (scalar) and 1.8 % (2x2) above the fastest one on the mean (worst 1.3 times); against the kernels
// with records and the one-workgroup ones the walk takes 0.65 to 0.95 of the time from 3000 channels on.
struct WalkCost {
    int c, w, waves;                  // steps per thread, waves, workgroups on a unit by registers
    float start, one, more_each;      // launch; a tile's iteration: a part, and one for each workgroup on the unit
    float tol_iters, more;            // iterations of a solve to a tolerance; loads, guess and stores as iterations
    float last, bf16, level, few;     // a last round after others; bf16; doubling of the channels; few workgroups
    float bytes, shared, apart;       // TB/s; what the other bytes of a line cost, at once and for each doubling of 1000 steps
};
constexpr WalkCost kWalkScalar[2] = {
    {8, 4, 5, 6.55f, 0.766f, 0.3614f, 4.25f, 0.744f, 0.981f, 1.014f, 0.0533f, 0.0f, 4.89f, 0.088f, 0.0417f},
    {12, 8, 2, 7.12f, 0.877f, 1.2527f, 4.17f, 1.106f, 0.974f, 0.963f, 0.0574f, 0.044f, 5.24f, 0.169f, 0.0246f}};
constexpr WalkCost kWalkBlock2[2] = {
    {8, 4, 3, 7.16f, 1.204f, 0.7797f, 4.73f, 0.751f, 0.947f, 0.990f, 0.0584f, 0.066f, 4.62f, 0.110f, 0.0291f},
    {16, 4, 2, 7.06f, 2.236f, 1.3244f, 4.99f, 1.025f, 1.003f, 0.900f, 0.0549f, 0.103f, 2.86f, 0.077f, 0.0026f}};

// wide: copies of 16 bytes
inline float walk_us(const WalkCost &k, const CellInfo &ci, int dtype, bool wide, int L, const ShortShape &sh, double n, int n_iters)
{
    const int esz = dtype == PARARNN_BF16 ? 2 : 4, lds_esz = wide ? esz : 4;
    const size_t lds = (size_t)k.c * ci.G * 64 * k.w * lds_esz + ((size_t)k.w * kShortCarries * ci.S << sh.lps_log2) * 4 + 64;
    // tensors off 16 bytes are copied a dword per element: the kernel for them has to fit too (walk_offered)
    if ((size_t)k.c * ci.G * 64 * k.w * 4 + ((size_t)k.w * kShortCarries * ci.S << sh.lps_log2) * 4 > 163840 - 256) return 1e30f;
    int per_unit = (int)(163840 / lds);
    if (per_unit > k.waves) per_unit = k.waves;
    const int full = sh.n_items / (kShortUnits * per_unit), left = sh.n_items - full * kShortUnits * per_unit;
    auto round = [&](int on) { return k.one + k.more_each * (float)on; };
    float rounds = (float)full * round(per_unit);
    if (left) rounds += round((left + kShortUnits - 1) / kShortUnits) * (full > 0 ? k.last : 1.0f);
    // the fit is of cells with three gates and one state value, and four and two
    const ShortCost &c = ci.S == 1 ? kCostScalar : kCostBlock2;
    const float work = (c.step + c.step_gate * (float)ci.G) / (c.step + c.step_gate * (ci.S == 1 ? 3.0f : 4.0f));
    const float its = n_iters ? (float)n_iters : k.tol_iters;
    float t = work * (its + k.more) * (float)sh.n_tiles * rounds * (1.0f - k.level * (float)sh.lps_log2);
    if (esz == 2) t *= k.bf16;
    if (sh.n_items < kShortUnits) t *= 1.0f - k.few * (1.0f - (float)sh.n_items / (float)kShortUnits);
    const int row = (k.w << sh.lps_log2) * esz;
    const float shared = row < 128 ? 128.0f / (float)row - 1.0f : 0.0f;
    const float m = (float)(n * esz * (ci.G + ci.S)) / (k.bytes * 1e6f) *
                    (1.0f + shared * (k.shared + (L > 1000 ? k.apart * log2f(0.001f * (float)L) : 0.0f)));
    return k.start + cbrtf(t * t * t + m * m * m);
}

// The shape of a forward solve by walk_kernels.h, or false where the other kernels do better: the one-workgroup ones in the
// shape `other`, with records where that is NULL.  n_iters: 0 = to a tolerance.
inline bool walk_forward_shape(const CellInfo &ci, int dtype, int B, int L, int H, int n_iters, const ShortShape *other, ShortShape *out)
{
    // Fewer waves than there are SIMDs, or a solve of a few launches' time: the others are faster everywhere, and the estimates
    // below take a microsecond that such a solve does not have.
    if (ci.S > 2 || ci.G < ci.S || (double)B * H < 1024.0 || (double)B * L * H < 524288.0) return false;
    const ShortCost &c = ci.S == 1 ? kCostScalar : kCostBlock2;
    const int esz = dtype == PARARNN_BF16 ? 2 : 4;
    const bool wide = (size_t)H * esz % 16 == 0;
    // the estimates of the others are of earlier kernels: the present ones take 0.94 and 0.9 of them
    const float better = n_iters == 0 || (n_iters >= 3 && n_iters <= 5) ? 0.97f : 0.85f;
    float best = better * (other ? 0.94f * short_us(c, ci, dtype, *other, n_iters) : 0.9f * records_us(c, ci, dtype, B, L, H, n_iters));
    bool found = false;
    for (const WalkCost &k : ci.S == 1 ? kWalkScalar : kWalkBlock2)
        for (int cwl = 0; cwl <= 4; ++cwl) {
            ShortShape sh;
            const int width = k.w << cwl, T = k.c * (64 >> cwl);
            if (wide && width * esz < 16) continue;
            if ((double)ci.G * H * esz * (T + 1.0) >= 2147483647.0) continue;      // 32-bit offsets within a tile
            sh.c = k.c; sh.lps_log2 = cwl; sh.w = k.w; sh.walk = true;
            sh.n_cg = (H + width - 1) / width;
            if ((double)B * sh.n_cg > 131072.0) continue;
            sh.n_items = B * sh.n_cg;
            sh.n_tiles = (L + T - 1) / T;
            const float us = walk_us(k, ci, dtype, wide, L, sh, (double)B * L * H, n_iters);
            if (us < best) { best = us; *out = sh; found = true; }
        }
    return found;
}

// workspace of such a solve: the control block (not used) and the workgroups' verdicts
inline size_t short_workspace_bytes(size_t n_items)
{
    return round256(sizeof(Ctrl)) + round256(n_items * 2 * sizeof(rec_t));
}
// ... of whatever shape and number of iterations: four channels are the smallest group
inline size_t short_workspace_most(int B, int H)
{
    const size_t n = (size_t)B * (((size_t)H + 3) / 4);
    return short_workspace_bytes(n < 131072 ? n : 131072);
}

// Polls (half a microsecond at least) after which workgroup 0 gives up waiting for the verdicts.  It waits for all
// workgroups of the solve, so beside the limit of one wait the work there is counts: the iterations of all tiles, as often as
// the 256 compute units take workgroups in turn (one at a time is the least they hold), 10 us each at most.  A limit of
// 2^21 polls, the default, covers 2^15 of them three times.
inline unsigned int short_wait_limit(unsigned int limit, const ShortShape &sh, int max_iter)
{
    const double steps = (double)sh.n_tiles * max_iter * ((sh.n_items + 255) / 256);
    const double polls = (double)limit * ceil(steps < 1.0 ? 1.0 : steps / 32768.0);
    return polls < 4294967295.0 ? (unsigned int)polls : 0xffffffffu;
}

inline bool dims_ok(int B, int L, int H)
{
    if (B < 1 || L < 1 || H < 1) return false;
    // keep every element count inside size_t/int ranges the kernels assume.  The bound on H keeps the
    // 32-bit byte offsets of the buffer instructions in range: at any H the tiles that are chosen have a wave address
    // up to 16 steps, of four gates 64 rows of H elements of 4 bytes from its base; one that is forced (64 steps in
    // eight segments of eight) keeps to the range by choose_tile
    const double n = (double)B * (double)L * (double)H;
    return n < 3.0e10 && (double)B * H < 2.0e9 && L < (1 << 30) && H <= (1 << 22);
}

inline bool aligned(const void *p, size_t a) { return ((uintptr_t)p % a) == 0; }

// widest vector (in elements of size esz: 4, 2 or 1) every pointer in the list allows; NULL allows any
inline int align_elems(size_t esz, std::initializer_list<const void *> ptrs)
{
    int a = 4;
    for (const void *p : ptrs) {
        if (!p) continue;
        const int here = aligned(p, 4 * esz) ? 4 : aligned(p, 2 * esz) ? 2 : 1;
        if (here < a) a = here;
    }
    return a;
}

// Carry-record slots a solve would like to have: the whole solve when the count is fixed
// (tol < 0) and short enough, else its first fused_head iterations; 0 = no fused launches.
inline int fused_slots_wanted(float tol, int max_iter, const SolveOpts &s = default_opts())
{
    if (!s.fused_enabled || max_iter < 1) return 0;
    if (tol < 0.0f) return max_iter <= kMaxFused ? max_iter : 0;
    return max_iter < s.fused_head ? max_iter : s.fused_head;
}

// Workspace size of a forward solve to a tolerance (or of a backward pass); does not depend on
// pointer alignment: the larger footprint is taken when the layouts differ.
inline size_t diag_workspace_bytes(const CellInfo &ci, int dtype, int B, int L, int H, bool backward,
                                   const SolveOpts &s = default_opts())
{
    size_t need = 0;
    for (int al = 1; al <= 4; al *= 2) {
        const Layout lo = make_layout(ci, dtype, B, L, H, backward, al);
        if (lo.total > need) need = lo.total;
        if (!backward && s.fused_enabled && s.fused_head > 0) {
            const Layout lf = make_layout(ci, dtype, B, L, H, false, al, true, s.fused_head);
            if (lf.total > need) need = lf.total;
        }
    }
    if (!backward && short_workspace_most(B, H) > need) need = short_workspace_most(B, H);
    return need;
}

// The front of such a workspace that a call with the same layout can make use of again (control block, carry records);
// n_iters > 0: of a fixed-count solve.  *rest: what the call needs behind it, which nothing reads afterwards.
inline size_t diag_workspace_parts(const CellInfo &ci, int dtype, int B, int L, int H, bool backward, int n_iters, size_t *rest)
{
    const SolveOpts s = default_opts();
    const int slots = backward || !s.fused_enabled ? 0 : n_iters > 0 ? (n_iters <= kMaxFused ? n_iters : 0) : s.fused_head;
    size_t front = 0;
    *rest = 0;
    for (int al = 1; al <= 4; al *= 2) {
        for (int fused = 0; fused <= (slots > 0 ? 1 : 0); ++fused) {
            const Layout lo = make_layout(ci, dtype, B, L, H, backward, al, fused != 0, fused ? slots : 1);
            if (lo.off_bnd > front) front = lo.off_bnd;
            if (lo.total - lo.off_bnd > *rest) *rest = lo.total - lo.off_bnd;
        }
    }
    if (!backward && short_workspace_most(B, H) > front) front = short_workspace_most(B, H);
    return front;
}

// Workspace size of a fixed-count solve of n_iters iterations in one launch.
inline size_t diag_workspace_bytes_fused(const CellInfo &ci, int dtype, int B, int L, int H, int n_iters)
{
    size_t need = diag_workspace_bytes(ci, dtype, B, L, H, false);
    if (n_iters < 1 || n_iters > kMaxFused) return need;
    for (int al = 1; al <= 4; al *= 2) {
        const Layout lf = make_layout(ci, dtype, B, L, H, false, al, true, n_iters);
        if (lf.off_bnd > need) need = lf.off_bnd;
    }
    return need;
}

// n_fused = number of carry-record slots the workspace holds (0: none; fused launches are not used).
// tol < 0: the whole fixed-count solve is one fused launch of n_fused = max_iter iterations.
// tol >= 0: the solve is a sequence of launches, each checked by the stopping test on the
// device: a fused block of n_fused iterations from the initial guess, then blocks of 1, 2,
// 4, ... (at most n_fused) iterations from the iterate; a block of one iteration that is a
// launch of its own is the per-iteration kernel.  With `tail` the blocks after the second (scalar
// cells: the first) share ONE launch of the fused kernel, which returns at once when the tolerance was met before;
// without it every block is a launch of its own.  Launches after the one that met the
// tolerance return at once.
template <class Cell>
int forward_diag(const CellInfo &ci, int dtype, const Layout &lo, FwdArgs &a, hipStream_t st, void *h,
                 int status0, int max_iter, int n_fused)
{
    char *ws = reinterpret_cast<char *>(a.ctrl);
    const bool bf = dtype == PARARNN_BF16;
    const bool to_tol = a.tol >= 0.0f;
    hipError_t e;
    // the fp32 iterate lies behind the boundary rows
    a.hit = bf ? reinterpret_cast<float *>(reinterpret_cast<char *>(a.bnd) + (lo.off_iter - lo.off_bnd)) : static_cast<float *>(h);
    const int slots = n_fused > 0 ? n_fused : 1;
    bool fill = true;
    if (max_iter <= kMaxIterWithReuse) a.g.epoch_base = workspace_epoch(ws, layout_signature(0, ci, dtype, lo, slots), st, &fill);
    else workspace_forget(ws);
    e = launch_reset(a.ctrl, a.rec, fill ? lo.n_rec * (size_t)slots : 0, a.iters_out, status0, st);
    if (e != hipSuccess) return PARARNN_HIP_ERROR;
    if (max_iter == 0) {
        // only the initial guess is asked for; otherwise the first iteration computes it on the fly
        e = bf ? Kernels<Cell, unsigned short>::init_guess(lo.cfg.vec, a, st) : Kernels<Cell, float>::init_guess(lo.cfg.vec, a, st);
        if (e != hipSuccess) return PARARNN_HIP_ERROR;
    }
    FusedArgs f;
    memset(&f, 0, sizeof(f));
    f.g = a.g; f.params = a.params; f.u = a.u; f.h0 = a.h0; f.h = h;
    f.rec = a.rec; f.rec_stride = lo.n_rec;
    f.gmaxk = reinterpret_cast<unsigned int *>(ws + 64);
    f.ctrl = a.ctrl; f.iters_out = a.iters_out; f.trace = a.trace;
    f.head = to_tol ? 1 : 0; f.max_iter = max_iter; f.tol = a.tol;
    f.hit = to_tol ? a.hit : nullptr;
    f.bnd = a.bnd;
    f.n_slots = n_fused; f.spin_limit = settings().spin_limit;
    const bool tail = settings().fused_tail != 0;
    // Scalar cells need a second block so rarely that it is not worth a launch of its own, which finds nothing to do
    // (5 us each); two-state cells do need it, and one iteration is what the per-iteration kernel does fastest.
    const int tail_from = ci.S == 1 ? 1 : 2;
    bool whole_h = n_fused > 0;            // every launch writes the output itself
    int done = 0, cur = 0;
    for (int launches = 0; done < max_iter; ++launches) {
        const int K = next_block_size(done, launches, max_iter, n_fused);
        if (to_tol && n_fused > 0 && launches == tail_from && tail) {
            // everything that is left in one launch that goes through the plan on the device
            f.n_iters = K; f.k0 = done; f.epoch0 = f.g.epoch_base + (unsigned int)done; f.bnd_cur = cur; f.tail = 1; f.launch_no = launches;
            e = bf ? Kernels<Cell, unsigned short>::newton_fused(lo.cfg, f, st) : Kernels<Cell, float>::newton_fused(lo.cfg, f, st);
            if (e != hipSuccess) return e == hipErrorInvalidValue ? PARARNN_UNSUPPORTED : PARARNN_HIP_ERROR;
            break;
        }
        if (n_fused > 0 && (K > 1 || done == 0)) {
            f.n_iters = K; f.k0 = done; f.epoch0 = f.g.epoch_base + (unsigned int)done; f.bnd_cur = cur; f.tail = 0; f.launch_no = launches;
            e = bf ? Kernels<Cell, unsigned short>::newton_fused(lo.cfg, f, st) : Kernels<Cell, float>::newton_fused(lo.cfg, f, st);
        } else {
            a.k = done + 1; a.bnd_cur = cur;
            whole_h = false;
            e = bf ? Kernels<Cell, unsigned short>::newton_iter(lo.cfg, a, done == 0, st)
                   : Kernels<Cell, float>::newton_iter(lo.cfg, a, done == 0, st);
        }
        if (e != hipSuccess) return e == hipErrorInvalidValue ? PARARNN_UNSUPPORTED : PARARNN_HIP_ERROR;
        done += K;
        cur ^= 1;
    }
    if (bf && !whole_h) {
        // rounds the fp32 iterate into the output; skipped on the device when a fused block
        // already wrote the final iterate
        e = launch_store_bf16(a.hit, h, (size_t)lo.g.B * lo.g.L * ci.S * lo.g.H, a.ctrl, st);
        if (e != hipSuccess) return PARARNN_HIP_ERROR;
    }
    return PARARNN_OK;
}

template <class Cell>
int backward_diag(const CellInfo &ci, int dtype, const Layout &lo, BwdArgs &a, hipStream_t st, float *dparams)
{
    bool fill = true;
    a.g.epoch_base = workspace_epoch(a.ctrl, layout_signature(1, ci, dtype, lo, 1), st, &fill);
    // Nothing to clear, no launch for it: the reduction at the end of the call before left the control block cleared.
    hipError_t e = fill ? launch_reset(a.ctrl, a.rec, lo.n_rec, nullptr, 0, st) : hipSuccess;
    if (e != hipSuccess) return PARARNN_HIP_ERROR;
    e = dtype == PARARNN_BF16 ? Kernels<Cell, unsigned short>::backward(lo.cfg, a, st)
                              : Kernels<Cell, float>::backward(lo.cfg, a, st);
    if (e != hipSuccess) return e == hipErrorInvalidValue ? PARARNN_UNSUPPORTED : PARARNN_HIP_ERROR;
    e = launch_param_reduce(a.part, dparams, lo.g.n_lt * lo.g.B, ci.PR * lo.g.H, st,
                            a.g.epoch_base ? a.ctrl : nullptr);
    return e == hipSuccess ? PARARNN_OK : PARARNN_HIP_ERROR;
}

// Argument checks shared by every forward entry point; PARARNN_OK or the status to return.
inline int check_forward_args(int dtype, const float *params, const void *u, const void *h0, int B, int L, int H,
                              float tol, int max_iter, void *h, int *iters, void *workspace)
{
    if (dtype != PARARNN_F32 && dtype != PARARNN_BF16) return PARARNN_INVALID_ARG;
    if (!dims_ok(B, L, H) || max_iter < 0 || !params || !u || !h || !iters || !workspace) return PARARNN_INVALID_ARG;
    if (tol != tol) return PARARNN_INVALID_ARG;
    if (!aligned(workspace, 256) || !aligned(params, 4) || !aligned(iters, 4)) return PARARNN_INVALID_ARG;
    const size_t esz = dtype == PARARNN_BF16 ? 2 : 4;
    if (!aligned(u, esz) || !aligned(h, esz) || (h0 && !aligned(h0, esz))) return PARARNN_INVALID_ARG;
    return PARARNN_OK;
}

inline int check_backward_args(int dtype, const float *params, const void *u, const void *h0, const void *h,
                               const void *dL_dh, int B, int L, int H, void *dL_du, float *dL_dparams, void *dL_dh0,
                               void *workspace)
{
    if (dtype != PARARNN_F32 && dtype != PARARNN_BF16) return PARARNN_INVALID_ARG;
    if (!dims_ok(B, L, H) || !params || !u || !h || !dL_dh || !dL_du || !dL_dparams || !workspace)
        return PARARNN_INVALID_ARG;
    const size_t esz = dtype == PARARNN_BF16 ? 2 : 4;
    if (!aligned(workspace, 256) || !aligned(params, 4) || !aligned(dL_dparams, 4) || !aligned(u, esz) ||
        !aligned(h, esz) || !aligned(dL_dh, esz) || !aligned(dL_du, esz) || (h0 && !aligned(h0, esz)) ||
        (dL_dh0 && !aligned(dL_dh0, esz)))
        return PARARNN_INVALID_ARG;
    return PARARNN_OK;
}

// The whole solve in one launch, sequences inside workgroups.
template <class Cell>
int forward_short(int dtype, const ShortShape &sh, const float *params, const void *u, const void *h0, int B, int L,
                  int H, float tol, int max_iter, void *h, int *iters, void *workspace, hipStream_t st)
{
    char *ws = static_cast<char *>(workspace);
    ShortArgs a;
    memset(&a, 0, sizeof(a));
    a.B = B; a.L = L; a.H = H; a.n_cg = sh.n_cg; a.lps_log2 = sh.lps_log2; a.n_items = sh.n_items; a.n_tiles = sh.n_tiles;
    a.params = params; a.u = u; a.h0 = h0; a.h = h; a.tol = tol; a.max_iter = max_iter; a.iters_out = iters;
    a.spin_limit = short_wait_limit(settings().spin_limit, sh, max_iter);
    a.slots = reinterpret_cast<rec_t *>(ws + round256(sizeof(Ctrl)));
    a.nonce = call_nonce();
    if (sh.walk) {
        // Nothing here needs what an earlier call left or leaves what a later one could use, but the large problems that are
        // walked keep their workspaces as those with records do: the block that the caller allocates is as large.
        unsigned long long sig = 1469598103934665603ull;
        for (long long x : {2LL, (long long)dtype, (long long)B, (long long)L, (long long)H, (long long)sh.c, (long long)sh.lps_log2, (long long)sh.w})
            sig = (sig ^ (unsigned long long)x) * 1099511628211ull;
        bool fill;
        workspace_epoch(workspace, sig, st, &fill);
    } else {
        workspace_forget(workspace);
    }
    // a captured launch replays its nonce: the verdicts are cleared in front of it
    if (sh.n_items > 1 && stream_is_capturing(st) &&
        launch_reset(reinterpret_cast<Ctrl *>(ws), a.slots, (size_t)sh.n_items * 2, nullptr, 0, st) != hipSuccess)
        return PARARNN_HIP_ERROR;
    const size_t esz = dtype == PARARNN_BF16 ? 2 : 4;
    const bool wide = (size_t)H * esz % 16 == 0 && aligned(u, 16) && aligned(h, 16);
    hipError_t e;
    if (sh.walk)
        e = dtype == PARARNN_BF16 ? Kernels<Cell, unsigned short>::newton_walk(sh.c, sh.w, wide, a, st)
                                  : Kernels<Cell, float>::newton_walk(sh.c, sh.w, wide, a, st);
    else
        e = dtype == PARARNN_BF16 ? Kernels<Cell, unsigned short>::newton_short(sh.c, sh.w, a, st)
                                  : Kernels<Cell, float>::newton_short(sh.c, sh.w, a, st);
    if (e == hipSuccess) return PARARNN_OK;
    workspace_forget(workspace);
    return PARARNN_HIP_ERROR;
}

// Whether a solve without a trace is one launch without blocks, given the workspace for it.
inline bool without_blocks(const CellInfo &ci, int dtype, int B, int L, int H, float tol, int max_iter, const SolveOpts &opts,
                           ShortShape *sh)
{
    if (!opts.fused_enabled || opts.fused_head <= 0 || (opts.blocks && tol >= 0.0f) || max_iter < 1 || settings().tile[0] > 0) return false;
    const int n_iters = tol < 0.0f ? max_iter : 0;
    ShortShape other;
    const bool one_workgroup = short_shape(ci, dtype, B, L, H, false, n_iters, &other);
    if (walk_forward_shape(ci, dtype, B, L, H, n_iters, one_workgroup ? &other : nullptr, sh)) return true;
    if (one_workgroup) *sh = other;
    return one_workgroup;
}

// A forward solve with checked arguments: layout, then the launches.
template <class Cell>
int forward_solve(const CellInfo &ci, int dtype, const float *params, const void *u, const void *h0, int B, int L,
                  int H, float tol, int max_iter, void *h, int *iters, float *delta_trace, void *workspace,
                  size_t workspace_bytes, hipStream_t st, const SolveOpts &opts = default_opts())
{
    const size_t esz = dtype == PARARNN_BF16 ? 2 : 4;
    const int status0 = tol < 0.0f ? PARARNN_OK : PARARNN_NOT_CONVERGED;
    int al = align_elems(esz, {u, h, h0});
    const int alp = align_elems(4, {params});
    if (alp < al) al = alp;
    // Fused launches need one carry-record slot per iteration they run; they are used when the
    // workspace holds those.
    Layout lo = make_layout(ci, dtype, B, L, H, false, al), lf;
    int n_fused = fused_slots_wanted(tol, max_iter, opts);
    WorkspaceRest rest = {nullptr, 0};
    bool asked = false;                    // for memory for the rest: only where the workspace is too small, and where there is some it is taken
    auto fits = [&](const Layout &l, size_t whole) {
        if (!rest.ptr && workspace_bytes >= whole) return true;
        if (!asked) { rest = workspace_rest(workspace); asked = true; }
        return rest.ptr && workspace_bytes >= l.off_bnd && rest.bytes >= whole - l.off_bnd;
    };
    if (n_fused > 0 && !fused_layout(ci, dtype, B, L, H, al, n_fused, tol >= 0.0f, fits, &lf)) n_fused = 0;
    if (n_fused == 0 && !fits(lo, lo.total)) return PARARNN_WORKSPACE_TOO_SMALL;
    if (n_fused > 0) lo = lf;
    ShortShape sh;
    if (!delta_trace && without_blocks(ci, dtype, B, L, H, tol, max_iter, opts, &sh) &&
        workspace_bytes >= short_workspace_bytes((size_t)sh.n_items))
        return forward_short<Cell>(dtype, sh, params, u, h0, B, L, H, tol, max_iter, h, iters, workspace, st);
    char *ws = static_cast<char *>(workspace);
    FwdArgs a;
    memset(&a, 0, sizeof(a));
    a.g = lo.g;
    a.params = params; a.u = u; a.h0 = h0; a.jac = nullptr;
    a.bnd = reinterpret_cast<float *>(rest.ptr ? rest.ptr : ws + lo.off_bnd);
    a.rec = reinterpret_cast<unsigned long long *>(ws + lo.off_rec);
    a.ctrl = reinterpret_cast<Ctrl *>(ws);
    a.iters_out = iters; a.trace = delta_trace;
    a.k = 0; a.max_iter = max_iter; a.tol = tol;
    {
        const size_t n = (size_t)B * L * H, esz = dtype == PARARNN_BF16 ? 2 : 4;
        a.stream = forward_stream_level(n * ci.G * esz, n * ci.S * sizeof(float));
    }
    const int rc = forward_diag<Cell>(ci, dtype, lo, a, st, h, status0, max_iter, n_fused);
    if (rc != PARARNN_OK) workspace_forget(workspace);
    return rc;
}

// Residual max-norm of given states (App. A); out is a device float.
inline int check_residual_args(int dtype, const float *params, const void *u, const void *h0, const void *h, int B,
                               int L, int H, float *out)
{
    if (dtype != PARARNN_F32 && dtype != PARARNN_BF16) return PARARNN_INVALID_ARG;
    if (!dims_ok(B, L, H) || !params || !u || !h || !out) return PARARNN_INVALID_ARG;
    const size_t esz = dtype == PARARNN_BF16 ? 2 : 4;
    if (!aligned(params, 4) || !aligned(out, 4) || !aligned(u, esz) || !aligned(h, esz) || (h0 && !aligned(h0, esz)))
        return PARARNN_INVALID_ARG;
    return PARARNN_OK;
}

template <class Cell>
int residual_norm_diag(int dtype, const float *params, const void *u, const void *h0, const void *h, int B, int L,
                       int H, float *out, hipStream_t st)
{
    const size_t esz = dtype == PARARNN_BF16 ? 2 : 4;
    int al = align_elems(esz, {u, h, h0});
    const int alp = align_elems(4, {params});
    if (alp < al) al = alp;
    const int vec = (H % 4 == 0 && al >= 4) ? 4 : (H % 2 == 0 && al >= 2) ? 2 : 1;
    ResArgs a;
    memset(&a, 0, sizeof(a));
    a.B = B; a.L = L; a.H = H;
    a.params = params; a.u = u; a.h0 = h0; a.h = h;
    a.out = reinterpret_cast<unsigned int *>(out);
    if (launch_zero_words(a.out, 1, st) != hipSuccess) return PARARNN_HIP_ERROR;
    const hipError_t e = dtype == PARARNN_BF16 ? Kernels<Cell, unsigned short>::residual_norm(vec, a, st)
                                               : Kernels<Cell, float>::residual_norm(vec, a, st);
    return e == hipSuccess ? PARARNN_OK : PARARNN_HIP_ERROR;
}

// A backward pass with checked arguments.
template <class Cell>
int backward_pass(const CellInfo &ci, int dtype, const float *params, const void *u, const void *h0, const void *h,
                  const void *dL_dh, int B, int L, int H, void *dL_du, float *dL_dparams, void *dL_dh0,
                  void *workspace, size_t workspace_bytes, hipStream_t st)
{
    const size_t esz = dtype == PARARNN_BF16 ? 2 : 4;
    int al = align_elems(esz, {u, h, h0, dL_dh, dL_du, dL_dh0});
    const int alp = align_elems(4, {params, dL_dparams});
    if (alp < al) al = alp;
    const Layout lo = make_layout(ci, dtype, B, L, H, true, al);
    const WorkspaceRest rest = workspace_bytes < lo.total ? workspace_rest(workspace) : WorkspaceRest{nullptr, 0};
    if (workspace_bytes < lo.total && !(rest.ptr && workspace_bytes >= lo.off_bnd && rest.bytes >= lo.total - lo.off_bnd))
        return PARARNN_WORKSPACE_TOO_SMALL;
    char *part = rest.ptr ? rest.ptr + (lo.off_part - lo.off_bnd) : static_cast<char *>(workspace) + lo.off_part;
    ShortShape sh;
    if (settings().tile[0] <= 0 && short_shape(ci, dtype, B, L, H, true, 0, &sh)) {
        ShortArgs a;
        memset(&a, 0, sizeof(a));
        a.B = B; a.L = L; a.H = H; a.n_cg = sh.n_cg; a.lps_log2 = sh.lps_log2; a.n_items = sh.n_items;
        a.params = params; a.u = u; a.h0 = h0; a.hs = h; a.gl = dL_dh; a.du = dL_du; a.dh0 = dL_dh0;
        a.part = B > 1 ? reinterpret_cast<float *>(part) : dL_dparams;   // a single sequence's sums are the gradient
        workspace_forget(workspace);
        hipError_t e = dtype == PARARNN_BF16 ? Kernels<Cell, unsigned short>::backward_short(sh.c, sh.w, a, st)
                                             : Kernels<Cell, float>::backward_short(sh.c, sh.w, a, st);
        if (e == hipSuccess && B > 1) e = launch_param_reduce(a.part, dL_dparams, B, ci.PR * H, st);
        return e == hipSuccess ? PARARNN_OK : PARARNN_HIP_ERROR;
    }
    char *ws = static_cast<char *>(workspace);
    BwdArgs a;
    memset(&a, 0, sizeof(a));
    a.g = lo.g;
    a.params = params; a.u = u; a.h0 = h0; a.h = h; a.gl = dL_dh; a.jac = nullptr;
    a.du = dL_du; a.dh0 = dL_dh0;
    a.part = reinterpret_cast<float *>(part);
    a.rec = reinterpret_cast<unsigned long long *>(ws + lo.off_rec);
    a.ctrl = reinterpret_cast<Ctrl *>(ws);
    // rows that the kernel may copy straight into LDS, 16 bytes per lane: bf16 rows that start on 16-byte
    // boundaries, and row offsets that stay inside the 32-bit range of a buffer instruction
    a.stage = settings().stage_enabled && dtype == PARARNN_BF16 && H % 8 == 0 && aligned(u, 16) && aligned(h, 16) &&
              aligned(dL_dh, 16) && (double)H * 2.0 * (16.0 * ci.G) < 4.0e9 &&
              (settings().tile[0] > 0 || backward_staged(ci, B, L, H));
    a.stream = backward_stream((size_t)B * L * H * esz * (2 * ci.G + 2 * ci.S),
                               lo.cfg.c != 12 && H * esz % 128 == 0 && aligned(u, 128) && aligned(h, 128) && aligned(dL_dh, 128) && aligned(dL_du, 128));
    if (!a.stage && !a.stream && backward_queues(ci, dtype, (size_t)B * L * H * esz * (2 * ci.G + 2 * ci.S), lo.g, lo.cfg)) a.stream = 2;
    const int rc = backward_diag<Cell>(ci, dtype, lo, a, st, dL_dparams);
    if (rc != PARARNN_OK) workspace_forget(workspace);
    return rc;
}

}  // namespace pararnn
