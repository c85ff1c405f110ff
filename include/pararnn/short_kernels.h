// Solves and backward passes in which nothing passes between workgroups: workgroup (b, cg) owns a group of channels
// of one sequence, all its timesteps.  No tickets, no carry records and no clearing of them, and the stopping test
// is the workgroup's own: a group of channels iterates until its own updates meet the tolerance, in one launch,
// however many iterations that takes (the channels are independent recurrences; the count reported is the largest).
//
// Decomposition as in scan_kernels.h: a lane owns one channel and C consecutive steps, the LL = 64 / lps segments of
// a wave hold consecutive chunks, the waves of the workgroup consecutive stretches; the workgroup covers T = C LL W steps.
// C is a template argument, LL and the number of waves are chosen per call (short_shape in driver.h).
//
// Sequences of up to T steps are one tile.  A small problem is then bound by the latency of its chain (per iteration: the
// chunk's instructions at four cycles each for a wave that has its SIMD to itself, two exchanges through LDS, two
// barriers), a large one by vector arithmetic like the fused blocks, with fewer iterations.
//
// Longer sequences (forward only) are walked tile by tile.  Iteration k of a tile needs delta^k at the end of the
// tile before, which has been solved by then and left one value per iteration and channel in LDS: the same Newton
// iterates as in one tile.  A tile is done when its own updates meet the tolerance and the state in front of it
// has its final value.  The latter holds from the iteration on after which nothing but negligible updates (the
// predecessor's maximum at most an eighth of the tolerance) would still arrive: they are added to that one's.
//
// Rows past the end of the sequence read as zero through the bounds of the buffer descriptor and are not stored;
// they come after every valid step, so what they compute reaches no valid one.
#pragma once
#include "scan_kernels.h"

namespace pararnn {

struct ShortArgs {
    int B, L, H;
    int n_cg;              // channel groups of a sequence
    int lps_log2;          // log2 of the channels per group = lanes per segment
    int n_items;           // B * n_cg
    int n_tiles;           // tiles a sequence is walked in
    const float *params;
    const void *u, *h0;
    void *h;
    float tol;
    int max_iter;
    int *iters_out;
    // the workgroups' verdicts, collected by workgroup 0: [n_items][2] words that carry the call's nonce, so that
    // whatever the workspace holds needs no clearing (two atomics per workgroup to one address cost 25 ns each, more
    // than the solve for 16384 of them)
    rec_t *slots;
    unsigned long long nonce;
    unsigned int spin_limit;
    // backward
    const void *hs, *gl;   // states, dL/dh
    void *du, *dh0;
    float *part;           // [B][PR][H]
};

// Iterations whose carry into the next tile is kept one by one; those of later ones are added to the last.
constexpr int kShortCarries = 16;

// Waves a workgroup may have, by the registers of a thread: 128 with sixteen waves, 256 with eight.
template <class Cell, int C> constexpr int short_max_waves() { return Cell::S * C <= 8 ? 16 : 8; }
// Waves per SIMD the register allocation must leave room for.  Sixteen steps of a scalar cell come out one register above
// the four-wave limit by themselves, and a workgroup of eight waves then has its compute unit to itself (2 x).
constexpr int short_min_waves(int S, int C, bool many)
{
    return S == 1 ? (C <= 8 ? (many ? 5 : 6) : 4) : S == 2 ? (C <= 4 ? 4 : C == 8 ? 3 : 2) : 2;
}
// Shapes that are compiled (the choice: short_shape in driver.h): a single tile with four and eight steps per thread
// and, for scalar cells, sixteen; several tiles with eight and sixteen; blocks of 3x3 and larger spill beyond four.
template <class Cell, int C> constexpr bool short_offered(bool many)
{
    return many ? Cell::S <= 2 && C >= 8 : C == 4 || (C == 8 && Cell::S <= 2) || (C == 16 && Cell::S == 1);
}

// Block index -> item, consecutive items on one XCD: neighbouring channel groups share the cache lines of their rows.
__device__ __forceinline__ int short_item(int n_items)
{
    const int per = (n_items + 7) / 8;
    const int item = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    return (int)(blockIdx.x >> 3) < per && item < n_items ? item : -1;
}

// The values of x in the lower and in the upper half of the lane pair-of-groups this lane belongs to, groups of DIST
// lanes: same position within the group.  Vector instructions only (lane-row swaps for 32 and 16 lanes, rotations
// inside a row of 16 for 8 and 4); a cross-lane read through LDS is a trip of about 100 cycles each.
template <int DIST> __device__ __forceinline__ void halves(int lane, float x, float &lo, float &up)
{
    const unsigned int u = __float_as_uint(x);
    if constexpr (DIST == 32 || DIST == 16) {
        const auto r = DIST == 32 ? __builtin_amdgcn_permlane32_swap(u, u, false, false) : __builtin_amdgcn_permlane16_swap(u, u, false, false);
        lo = __uint_as_float(r[0]);
        up = __uint_as_float(r[1]);
    } else {
        constexpr int kRor = 0x120;                    // row_ror:n, lane i takes lane i - n of its row
        const float below = __uint_as_float(__builtin_amdgcn_update_dpp(0u, u, kRor + DIST, 0xf, 0xf, true));
        const float above = DIST == 8 ? below : __uint_as_float(__builtin_amdgcn_update_dpp(0u, u, kRor + 16 - DIST, 0xf, 0xf, true));
        lo = lane & DIST ? below : x;
        up = lane & DIST ? x : above;
    }
}

// One level of wave_scan: pairs of groups of DIST lanes.  REV: the segments run from the upper lanes down.
template <int S, int DIST, bool REV>
__device__ __forceinline__ void scan_level(int lane, float *accA, float *accB, float *exA, float *exB)
{
    constexpr int SS = S * S;
    float fA[SS], fB[S], lA[SS], lB[S];                // the map applied first, the one applied last
#pragma unroll
    for (int e = 0; e < SS; ++e) halves<DIST>(lane, accA[e], REV ? lA[e] : fA[e], REV ? fA[e] : lA[e]);
#pragma unroll
    for (int s = 0; s < S; ++s) halves<DIST>(lane, accB[s], REV ? lB[s] : fB[s], REV ? fB[s] : lB[s]);
#pragma unroll
    for (int e = 0; e < SS; ++e) accA[e] = lA[e];
#pragma unroll
    for (int s = 0; s < S; ++s) accB[s] = lB[s];
    compose_after<S>(fA, fB, accA, accB);
    if (((lane & DIST) != 0) != REV) compose_after<S>(fA, fB, exA, exB);
}

// (accA, accB): in, the map of the lane's own segment; out, the composition of all segments of the wave.
// (exA, exB): out, the composition of the segments before the own one.  Segments of 1 << lps_log2 lanes, at least 4.
template <int S, bool REV = false>
__device__ __forceinline__ void wave_scan(int lane, int lps_log2, float *accA, float *accB, float *exA, float *exB)
{
    set_identity<S>(exA);
#pragma unroll
    for (int s = 0; s < S; ++s) exB[s] = 0.0f;
    if (lps_log2 <= 2) scan_level<S, 4, REV>(lane, accA, accB, exA, exB);
    if (lps_log2 <= 3) scan_level<S, 8, REV>(lane, accA, accB, exA, exB);
    if (lps_log2 <= 4) scan_level<S, 16, REV>(lane, accA, accB, exA, exB);
    if (lps_log2 <= 5) scan_level<S, 32, REV>(lane, accA, accB, exA, exB);
}

__device__ __forceinline__ buf_rsrc bounded_rsrc(const void *base, unsigned int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, bytes, 0x27000);
}

// How a workgroup's solve ended, ordered so that the maximum over workgroups is the verdict of the whole
// solve: converged after k, not converged, a NaN or infinity in iteration k (the earliest one counts).
__device__ __forceinline__ unsigned int short_verdict(int status, int k)
{
    if (status == kStNonFinite) return 0xc0000000u - (unsigned int)k;
    if (status == kStNotConverged) return 0x40000000u;
    return (unsigned int)k;
}
__device__ __forceinline__ void short_report(unsigned int v, int max_iter, int *iters_out)
{
    int k = (int)v, status = kStOk;
    if (v == 0xffffffffu) { k = max_iter; status = kStInternal; }
    else if (v > 0x40000000u) { k = (int)(0xc0000000u - v); status = kStNonFinite; }
    else if (v == 0x40000000u) { k = max_iter; status = kStNotConverged; }
    iters_out[0] = k;
    iters_out[1] = status;
}

// The verdict of the whole solve from those of its workgroups: v of workgroup `item`, of W waves; s_max is scratch for them.
__device__ __forceinline__ void short_collect(const ShortArgs &a, int item, unsigned int v, int W, unsigned int *s_max)
{
    const int lane = threadIdx.x & 63, w = (int)(threadIdx.x >> 6);
    if (a.n_items == 1) {
        if (threadIdx.x == 0) short_report(v, a.max_iter, a.iters_out);
    } else {
        const unsigned int hi = (unsigned int)(a.nonce >> 32), lo = (unsigned int)a.nonce;
        if (item > 0) {
            if (threadIdx.x == 0) {
                __hip_atomic_store(a.slots + 2 * (size_t)item, ((rec_t)hi << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(a.slots + 2 * (size_t)item + 1, ((rec_t)lo << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            return;
        }
        // workgroup 0 waits for the others, which wait for nothing; eight verdicts per trip to memory
        constexpr int kBatch = 8;
        for (int i0 = 1 + (int)threadIdx.x; i0 < a.n_items; i0 += kBatch * (int)blockDim.x) {
            unsigned int polls = 0;
            for (;;) {
                rec_t w0[kBatch], w1[kBatch];
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    const int i = min(i0 + j * (int)blockDim.x, a.n_items - 1);
                    w0[j] = rec_load(a.slots + 2 * (size_t)i);
                    w1[j] = rec_load(a.slots + 2 * (size_t)i + 1);
                }
                bool all = true;
                unsigned int vb = 0u;
#pragma unroll
                for (int j = 0; j < kBatch; ++j) {
                    all = all && (unsigned int)(w0[j] >> 32) == hi && (unsigned int)(w1[j] >> 32) == lo &&
                          (unsigned int)w0[j] == (unsigned int)w1[j];
                    vb = max(vb, (unsigned int)w0[j]);
                }
                if (all) { v = max(v, vb); break; }
                if (++polls >= a.spin_limit) { v = 0xffffffffu; break; }
                // A workgroup that polls without a pause takes its compute unit from the one beside it, which is what it
                // waits for: it ended at 547 us where the others had by 428 (GRU fp32 4096 x 16 x 1024, five iterations).
                // Pauses of up to a fortieth of the time waited.
                if (polls < 16) __builtin_amdgcn_s_sleep(1);
                else if (polls < 64) __builtin_amdgcn_s_sleep(4);
                else if (polls < 128) __builtin_amdgcn_s_sleep(16);
                else __builtin_amdgcn_s_sleep(64);
            }
        }
        __syncthreads();                               // s_max is free again
        v = wave_max_u32(v);
        if (lane == 0) s_max[w] = v;
        __syncthreads();
        if (w == 0) {
            v = wave_max_u32(s_max[lane < W ? lane : 0]);
            if (lane == 0) short_report(v, a.max_iter, a.iters_out);
        }
    }
}

// MANY: more than one tile (at most eight waves)
template <class Cell, int C, typename UT, bool MANY>
__global__ __launch_bounds__((kWave * (MANY ? 8 : short_max_waves<Cell, C>()))) __attribute__((amdgpu_waves_per_eu(short_min_waves(Cell::S, C, MANY)))) void newton_short_kernel(const ShortArgs a)
{
    constexpr int S = Cell::S, G = Cell::G, SS = S * S, PR = Cell::PR;
    constexpr bool kMark = C > 4 || S > 2;             // scalar and 2x2 cells: four steps are for problems of a few waves
    extern __shared__ float s_agg[];                   // [W][SS + S][CW] wave aggregates; several tiles: [2][kShortCarries][S][CW] carries
    __shared__ unsigned int s_max[16];
    const int item = short_item(a.n_items);
    if (item < 0) return;
    const int lane = threadIdx.x & 63, W = (int)(blockDim.x >> 6);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int LPS = 1 << a.lps_log2, LL = kWave >> a.lps_log2;
    const int seg = lane >> a.lps_log2, col = lane & (LPS - 1);
    const int b = item / a.n_cg, cg = item - b * a.n_cg;
    const int ch = cg * LPS + col;
    const bool ch_ok = ch < a.H;
    const int lt0 = (w * LL + seg) * C;                // this lane's first step within a tile
    const unsigned int Hn = (unsigned int)a.H;
    const int T = C * LL * W;
    constexpr unsigned int E = sizeof(UT);
    float *s_carry = s_agg + ((size_t)W * (SS + S) << a.lps_log2) + col;
    const int carry_set = (kShortCarries * S) << a.lps_log2;

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

    unsigned int v = 0u;                               // this workgroup's verdict
    int k_before = 0, k_final = 0;                     // iterations of the tile before; the first with a final boundary
    const int n_tiles = MANY ? a.n_tiles : 1;
    for (int tile = 0; tile < n_tiles; ++tile) {
        const int l0 = tile * T + lt0;
        const unsigned int rows = (unsigned int)(a.L - tile * T);      // from the tile's first row to the end
        const unsigned int lead = tile > 0 ? 1u : 0u;                  // the descriptor starts a row early where there is one
        auto bytes = [&](unsigned int per_row) {
            const unsigned long long n = (unsigned long long)rows * per_row;
            return n < 0x7fffffffull ? (unsigned int)n : 0x7fffffffu;
        };
        const buf_rsrc ru = bounded_rsrc(static_cast<const UT *>(a.u) + ((size_t)b * a.L + (size_t)tile * T - lead) * G * Hn,
                                         bytes(G * Hn * E) + lead * G * Hn * E);
        const buf_rsrc rh = bounded_rsrc(static_cast<UT *>(a.h) + ((size_t)b * a.L + (size_t)tile * T) * S * Hn, bytes(S * Hn * E));
        const unsigned int vu = (((unsigned int)lt0 + lead) * G * Hn + (unsigned int)ch) * E;
        const unsigned int vh = ch_ok ? ((unsigned int)lt0 * S * Hn + (unsigned int)ch) * E : 0xffffffffu;

        using RawU = typename RawVec<UT, 1>::type;
        RawU uur[C][G], uhalo[G];
#pragma unroll
        for (int i = 0; i < C; ++i)
#pragma unroll
            for (int q = 0; q < G; ++q) uur[i][q] = buf_load<UT, 1>(ru, vu, (unsigned int)(i * G + q) * Hn * E);
#pragma unroll
        for (int q = 0; q < G; ++q) uhalo[q] = buf_load<UT, 1>(ru, vu + ((unsigned int)q - G) * Hn * E, 0);   // l0 = 0: not used

        // initial guess h^0_l = f(h0, u_l) (App. A), also of the step in front of the chunk
        float uu[C][G], ho[C][S], hprev[S];
#pragma unroll
        for (int i = -1; i < C; ++i) {
            float ug[G], F0[S];
#pragma unroll
            for (int q = 0; q < G; ++q) {
                float t[1];
                raw_to_float<UT, 1>(i < 0 ? uhalo[q] : uur[i < 0 ? 0 : i][q], t);
                ug[q] = t[0];
            }
            Cell::fold_u(p, ug);
            Cell::template step<true>(p, h0v, ug, F0, pq);
            if (i < 0) {
#pragma unroll
                for (int s = 0; s < S; ++s) hprev[s] = l0 > 0 ? F0[s] : h0v[s];
            } else {
#pragma unroll
                for (int q = 0; q < G; ++q) uu[i][q] = ug[q];
#pragma unroll
                for (int s = 0; s < S; ++s) ho[i][s] = F0[s];
            }
        }

        const int n_valid = ch_ok ? min(max(a.L - l0, 0), C) : 0;      // steps of this lane inside the tensor
        const bool all_valid = __all(n_valid == C);
        const float *carry_in = s_carry + (tile & 1 ? carry_set : 0);
        float *carry_out = s_carry + (tile & 1 ? 0 : carry_set);
        int k = 0, k_met = 1;                          // k_met: the first iteration after which every update met the tolerance
        float mk = 0.0f;
        while (k < a.max_iter) {
            ++k;
            // ---- thread level
            float PA[C][SS], qb[C][S], accA[SS], accB[S];
            set_identity<S>(accA);
#pragma unroll
            for (int s = 0; s < S; ++s) accB[s] = 0.0f;
#pragma unroll
            for (int i = 0; i < C; ++i) {
                float J[SS], r[S], hp[S], F[S];
#pragma unroll
                for (int s = 0; s < S; ++s) hp[s] = i == 0 ? hprev[s] : ho[i > 0 ? i - 1 : 0][s];
                eval_step<Cell, kMark>(p, pq, hp, uu[i], F, J);
#pragma unroll
                for (int s = 0; s < S; ++s) r[s] = F[s] - ho[i][s];
                push_step<S>(J, r, accA, accB);
                if constexpr (kMark) {
                    gates_done<SS>(accA);
                    gates_done<S>(accB);
                }
#pragma unroll
                for (int e = 0; e < SS; ++e) PA[i][e] = accA[e];
#pragma unroll
                for (int s = 0; s < S; ++s) qb[i][s] = accB[s];
            }
            // ---- wave level: the wave's aggregate in every lane, the map of the segments before the own one in lex
            float lexA[SS], lexB[S];
            wave_scan<S>(lane, a.lps_log2, accA, accB, lexA, lexB);
            // ---- workgroup level: what enters the tile is a vector (zero in front of the first one), so what enters a
            //      wave is one too
            float din[S];
#pragma unroll
            for (int s = 0; s < S; ++s) din[s] = 0.0f;
            if (MANY && k <= k_final) {
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    din[s] = carry_in[((k - 1) * S + s) << a.lps_log2];
                    if (k == k_final && k_before > k_final) din[s] += carry_in[(k * S + s) << a.lps_log2];
                }
            }
            if (W > 1) {
                float *mine = s_agg + ((size_t)w * (SS + S) << a.lps_log2) + col;
                if (seg == LL - 1) {
#pragma unroll
                    for (int e = 0; e < SS; ++e) mine[e << a.lps_log2] = accA[e];
#pragma unroll
                    for (int s = 0; s < S; ++s) mine[(SS + s) << a.lps_log2] = accB[s];
                }
                __syncthreads();
                for (int j0 = 0; j0 < w; j0 += 4) {    // four aggregates per trip to LDS
                    float A4[4][SS], b4[4][S];
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float *t = s_agg + ((size_t)min(j0 + j, w) * (SS + S) << a.lps_log2) + col;
#pragma unroll
                        for (int e = 0; e < SS; ++e) A4[j][e] = t[e << a.lps_log2];
#pragma unroll
                        for (int s = 0; s < S; ++s) b4[j][s] = t[(SS + s) << a.lps_log2];
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (j0 + j < w) affine<S>(A4[j], din, b4[j], din);
                }
            }
            affine<S>(lexA, din, lexB, din);
            // ---- back-substitution
            unsigned int wmax_bits = 0u;
            float d[S];
#pragma unroll
            for (int s = 0; s < S; ++s) hprev[s] += din[s];
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
            if (MANY && tile + 1 < n_tiles && w == W - 1 && seg == LL - 1) {
                float *c = carry_out + (((min(k, kShortCarries) - 1) * S) << a.lps_log2);
#pragma unroll
                for (int s = 0; s < S; ++s) c[s << a.lps_log2] = k > kShortCarries ? c[s << a.lps_log2] + d[s] : d[s];
            }
            // ---- the stopping test of this group of channels
            unsigned int m = wave_max_u32(wmax_bits);
            if (W > 1) {
                if (lane == 0) s_max[w] = m;
                __syncthreads();
                m = wave_max_u32(s_max[lane < W ? lane : 0]);
            }
            mk = __uint_as_float(m);
            if (!(mk - mk == 0.0f)) break;
            if (a.tol >= 0.0f) {
                if (mk > a.tol) k_met = k + 1;
                else if (k >= k_final) break;
            }
        }

#pragma unroll
        for (int i = 0; i < C; ++i)
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const float t[1] = {ho[i][s]};
                buf_store<UT, 1>(rh, vh, (unsigned int)(i * S + s) * Hn * E, t);
            }
        if (!(mk - mk == 0.0f)) v = max(v, short_verdict(kStNonFinite, k));
        else if (a.tol >= 0.0f && mk > a.tol) v = max(v, short_verdict(kStNotConverged, k));
        else v = max(v, short_verdict(kStOk, a.tol >= 0.0f ? k_met : k));
        k_before = k_final = min(k, kShortCarries);
        if (k_before == k && k > 1 && mk <= 0.125f * a.tol) k_final = k - 1;
    }

    short_collect(a, item, v, W, s_max);
}

// The adjoint scan and the gradients (Eq. (6)), formulas and variables as in backward_kernel.
template <class Cell, int C, typename UT>
__global__ __launch_bounds__((kWave * short_max_waves<Cell, C>())) __attribute__((amdgpu_waves_per_eu(short_min_waves(Cell::S, C, false)))) void backward_short_kernel(const ShortArgs a)
{
    constexpr int S = Cell::S, G = Cell::G, SS = S * S, PR = Cell::PR, NC = Cell::NC;
    extern __shared__ float s_agg[];                   // [W][max(SS + S, PR)][CW]
    const int item = short_item(a.n_items);
    if (item < 0) return;
    const int lane = threadIdx.x & 63, W = (int)(blockDim.x >> 6);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int LPS = 1 << a.lps_log2, LL = kWave >> a.lps_log2;
    const int seg = lane >> a.lps_log2, col = lane & (LPS - 1);
    const int b = item / a.n_cg, cg = item - b * a.n_cg;
    const int ch = cg * LPS + col;
    const bool ch_ok = ch < a.H;
    const int l0 = (w * LL + seg) * C;
    const unsigned int Hn = (unsigned int)a.H, L = (unsigned int)a.L;
    constexpr unsigned int E = sizeof(UT);
    const buf_rsrc ru = bounded_rsrc(static_cast<const UT *>(a.u) + (size_t)b * L * G * Hn, L * G * Hn * E);
    const buf_rsrc rh = bounded_rsrc(static_cast<const UT *>(a.hs) + (size_t)b * L * S * Hn, L * S * Hn * E);
    const buf_rsrc rg = bounded_rsrc(static_cast<const UT *>(a.gl) + (size_t)b * L * S * Hn, L * S * Hn * E);
    const buf_rsrc rdu = bounded_rsrc(static_cast<UT *>(a.du) + (size_t)b * L * G * Hn, L * G * Hn * E);
    const unsigned int vu = ((unsigned int)l0 * G * Hn + (unsigned int)ch) * E;
    const unsigned int vh = ((unsigned int)l0 * S * Hn + (unsigned int)ch) * E;

    using RawU = typename RawVec<UT, 1>::type;
    RawU uur[C][G], hpr[C][S], ggr[C][S];
#pragma unroll
    for (int i = 0; i < C; ++i) {
#pragma unroll
        for (int q = 0; q < G; ++q) uur[i][q] = buf_load<UT, 1>(ru, vu, (unsigned int)(i * G + q) * Hn * E);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            ggr[i][s] = buf_load<UT, 1>(rg, vh, (unsigned int)(i * S + s) * Hn * E);
            // h one step earlier; in front of the sequence (l0 = 0): out of bounds, replaced by h0 below
            if (i == 0) hpr[i][s] = buf_load<UT, 1>(rh, vh + ((unsigned int)s - S) * Hn * E, 0);
            else hpr[i][s] = buf_load<UT, 1>(rh, vh, (unsigned int)((i - 1) * S + s) * Hn * E);
        }
    }
    float p[PR], h0v[S];
#pragma unroll
    for (int r = 0; r < PR; ++r) p[r] = ch_ok ? a.params[(size_t)r * Hn + ch] : 0.0f;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        float t[1] = {0.0f};
        if (ch_ok && a.h0) load_vec<1>(static_cast<const UT *>(a.h0) + ((size_t)b * S + s) * Hn + ch, t);
        h0v[s] = t[0];
    }

    // ---- thread level, right to left: lam_i = PX_i nu_in + qx_i
    float PX[C][SS], qx[C][S], kk[C][NC], accA[SS], accB[S], zero[S];
    set_identity<S>(accA);
#pragma unroll
    for (int s = 0; s < S; ++s) { accB[s] = 0.0f; zero[s] = 0.0f; }
    const int n_valid = min(max((int)L - l0, 0), C);
#pragma unroll
    for (int i = C - 1; i >= 0; --i) {
        float ug[G], hp[S], J[SS];
#pragma unroll
        for (int q = 0; q < G; ++q) { float t[1]; raw_to_float<UT, 1>(uur[i][q], t); ug[q] = t[0]; }
#pragma unroll
        for (int s = 0; s < S; ++s) {
            float t[1];
            raw_to_float<UT, 1>(hpr[i][s], t);
            hp[s] = i == 0 && l0 == 0 ? h0v[s] : t[0];
            raw_to_float<UT, 1>(ggr[i][s], t);
            qx[i][s] = accB[s] + t[0];
        }
#pragma unroll
        for (int e = 0; e < SS; ++e) PX[i][e] = accA[e];
        Cell::bwd_prep(p, hp, ug, J, kk[i]);
        transpose_inplace<S>(J);
        if (i < n_valid) {                             // steps past the end pass zero on
            affine<S>(J, qx[i], zero, accB);
            mat_mul<S>(J, accA, accA);
        }
    }
    float cA[SS], cB[S];                               // nu at the chunk's first step
#pragma unroll
    for (int e = 0; e < SS; ++e) cA[e] = accA[e];
#pragma unroll
    for (int s = 0; s < S; ++s) cB[s] = accB[s];

    // ---- wave level: the segments to the right come first
    float lexA[SS], lexB[S];
    wave_scan<S, true>(lane, a.lps_log2, accA, accB, lexA, lexB);
    // ---- workgroup level
    float nin[S];
#pragma unroll
    for (int s = 0; s < S; ++s) nin[s] = 0.0f;
    if (W > 1) {
        float *mine = s_agg + ((size_t)w * (SS + S) << a.lps_log2) + col;
        if (seg == 0) {
#pragma unroll
            for (int e = 0; e < SS; ++e) mine[e << a.lps_log2] = accA[e];
#pragma unroll
            for (int s = 0; s < S; ++s) mine[(SS + s) << a.lps_log2] = accB[s];
        }
        __syncthreads();
        for (int j = W - 1; j > w; --j) {
            const float *t = s_agg + ((size_t)j * (SS + S) << a.lps_log2) + col;
            float Aj[SS], bj[S];
#pragma unroll
            for (int e = 0; e < SS; ++e) Aj[e] = t[e << a.lps_log2];
#pragma unroll
            for (int s = 0; s < S; ++s) bj[s] = t[(SS + s) << a.lps_log2];
            affine<S>(Aj, nin, bj, nin);
        }
        __syncthreads();                               // s_agg takes the gradient sums below
    }
    affine<S>(lexA, nin, lexB, nin);

    // ---- lam for every step, then du and the parameter gradients
    float acc[PR];
#pragma unroll
    for (int r = 0; r < PR; ++r) acc[r] = 0.0f;
    const unsigned int vo = ch_ok ? vu : 0xffffffffu;
#pragma unroll
    for (int i = 0; i < C; ++i) {
        float lam[S], d1[G];
        affine<S>(PX[i], nin, qx[i], lam);
#pragma unroll
        for (int q = 0; q < G; ++q) d1[q] = 0.0f;
        if (i < n_valid) Cell::bwd_emit(kk[i], lam, d1, acc);
#pragma unroll
        for (int q = 0; q < G; ++q) {
            const float t[1] = {d1[q]};
            buf_store<UT, 1>(rdu, vo, (unsigned int)(i * G + q) * Hn * E, t);
        }
    }
    if (a.dh0 && ch_ok && l0 == 0) {
        float n0[S];
        affine<S>(cA, nin, cB, n0);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const float t[1] = {n0[s]};
            store_vec<1>(static_cast<UT *>(a.dh0) + ((size_t)b * S + s) * Hn + ch, t);
        }
    }
    for (int d = LL / 2; d >= 1; d >>= 1)
#pragma unroll
        for (int r = 0; r < PR; ++r) acc[r] += __shfl_down(acc[r], (unsigned int)(d << a.lps_log2), 64);
    float *out = a.part + (size_t)b * PR * Hn + ch;
    if (W == 1) {
        if (seg == 0 && ch_ok)
#pragma unroll
            for (int r = 0; r < PR; ++r) out[(size_t)r * Hn] = acc[r];
        return;
    }
    if (seg == 0) {
#pragma unroll
        for (int r = 0; r < PR; ++r) s_agg[((size_t)(w * PR + r) << a.lps_log2) + col] = acc[r];
    }
    __syncthreads();
    for (int idx = (int)threadIdx.x; idx < PR << a.lps_log2; idx += (int)blockDim.x) {
        const int r = idx >> a.lps_log2, c = idx & (LPS - 1);
        float s = 0.0f;
        for (int j = 0; j < W; ++j) s += s_agg[((size_t)(j * PR + r) << a.lps_log2) + c];
        const int chn = cg * LPS + c;
        if (chn < a.H) a.part[((size_t)b * PR + r) * Hn + chn] = s;
    }
}

}  // namespace pararnn
