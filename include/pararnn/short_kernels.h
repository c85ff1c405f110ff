// Solves and backward passes whose sequence fits one workgroup: workgroup (b, cg) holds all timesteps of one
// sequence for a group of channels, so nothing passes between workgroups.  No tickets, no carry records and no
// clearing of them, and the stopping test is the workgroup's own: a group of channels iterates until its own
// updates meet the tolerance, in one launch, however many iterations that takes (the channels are independent
// recurrences; the count reported is the largest).
//
// Decomposition as in scan_kernels.h: a lane owns one channel and C consecutive steps, the LL = 64 / lps segments of
// a wave hold consecutive chunks, the waves of the workgroup consecutive stretches.  C is a template argument,
// LL and the number of waves are chosen per call (short_shape in driver.h): the shortest chunk that still
// fills the device, because a small problem is bound by the latency of its chain (per iteration: the chunk's
// instructions at four cycles each for a wave that has its SIMD to itself, two exchanges through LDS, two barriers).
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

// Waves a workgroup may have, by the registers of a thread: 128 with sixteen waves, 256 with eight.
template <class Cell, int C> constexpr int short_max_waves() { return Cell::S * C <= 8 ? 16 : 8; }
// Waves per SIMD the register allocation must leave room for.  Sixteen steps of a scalar cell come out one register above
// the four-wave limit by themselves, and a workgroup of eight waves then has its compute unit to itself (2 x).
template <class Cell, int C> constexpr int short_min_waves()
{
    return Cell::S == 1 ? (C <= 8 ? 6 : 4) : Cell::S == 2 ? (C <= 4 ? 4 : C == 8 ? 3 : 2) : 2;
}
// Steps per thread that are compiled (the choice: short_shape in driver.h); blocks of 3x3 and larger spill beyond four.
template <class Cell, int C> constexpr bool short_offered(bool backward)
{
    return C == 4 || (C == 8 && Cell::S <= 2) || (C == 16 && Cell::S <= 2 && !backward);
}

// Block index -> item, consecutive items on one XCD: neighbouring channel groups share the cache lines of their rows.
__device__ __forceinline__ int short_item(int n_items)
{
    const int per = (n_items + 7) / 8;
    const int item = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    return (int)(blockIdx.x >> 3) < per && item < n_items ? item : -1;
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

template <class Cell, int C, typename UT>
__global__ __launch_bounds__((kWave * short_max_waves<Cell, C>())) __attribute__((amdgpu_waves_per_eu(short_min_waves<Cell, C>()))) void newton_short_kernel(const ShortArgs a)
{
    constexpr int S = Cell::S, G = Cell::G, SS = S * S, PR = Cell::PR;
    extern __shared__ float s_agg[];                   // [W][SS + S][CW] wave aggregates
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
    const int l0 = (w * LL + seg) * C;
    const unsigned int Hn = (unsigned int)a.H, L = (unsigned int)a.L;
    constexpr unsigned int E = sizeof(UT);
    const buf_rsrc ru = bounded_rsrc(static_cast<const UT *>(a.u) + (size_t)b * L * G * Hn, L * G * Hn * E);
    const buf_rsrc rh = bounded_rsrc(static_cast<UT *>(a.h) + (size_t)b * L * S * Hn, L * S * Hn * E);
    const unsigned int vu = ((unsigned int)l0 * G * Hn + (unsigned int)ch) * E;
    const unsigned int vh = ch_ok ? ((unsigned int)l0 * S * Hn + (unsigned int)ch) * E : 0xffffffffu;

    using RawU = typename RawVec<UT, 1>::type;
    RawU uur[C][G], uhalo[G];
#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
        for (int q = 0; q < G; ++q) uur[i][q] = buf_load<UT, 1>(ru, vu, (unsigned int)(i * G + q) * Hn * E);
#pragma unroll
    for (int q = 0; q < G; ++q) uhalo[q] = buf_load<UT, 1>(ru, vu + ((unsigned int)q - G) * Hn * E, 0);   // l0 = 0: not used
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

    const int n_valid = ch_ok ? min(max((int)L - l0, 0), C) : 0;     // steps of this lane inside the tensor
    const bool all_valid = __all(n_valid == C);
    int k = 0, status = a.tol < 0.0f ? kStOk : kStNotConverged;
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
            Cell::template fwd<true>(p, hp, uu[i], F, J, pq);
#pragma unroll
            for (int s = 0; s < S; ++s) r[s] = F[s] - ho[i][s];
            push_step<S>(J, r, accA, accB);
#pragma unroll
            for (int e = 0; e < SS; ++e) PA[i][e] = accA[e];
#pragma unroll
            for (int s = 0; s < S; ++s) qb[i][s] = accB[s];
        }
        // ---- wave level
        float lexA[SS], lexB[S];
        set_identity<S>(lexA);
#pragma unroll
        for (int s = 0; s < S; ++s) lexB[s] = 0.0f;
        if (LL > 1) {
            for (int d = 1; d < LL; d <<= 1) {
                float pA[SS], pB[S];
#pragma unroll
                for (int e = 0; e < SS; ++e) pA[e] = __shfl_up(accA[e], (unsigned int)(d << a.lps_log2), 64);
#pragma unroll
                for (int s = 0; s < S; ++s) pB[s] = __shfl_up(accB[s], (unsigned int)(d << a.lps_log2), 64);
                if (seg >= d) compose_after<S>(pA, pB, accA, accB);
            }
#pragma unroll
            for (int e = 0; e < SS; ++e) {
                const float t = __shfl_up(accA[e], (unsigned int)LPS, 64);
                if (seg > 0) lexA[e] = t;
            }
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const float t = __shfl_up(accB[s], (unsigned int)LPS, 64);
                if (seg > 0) lexB[s] = t;
            }
        }
        // ---- workgroup level: delta is zero in front of the first wave, so what enters a wave is a vector
        float din[S];
#pragma unroll
        for (int s = 0; s < S; ++s) din[s] = 0.0f;
        if (W > 1) {
            float *mine = s_agg + ((size_t)w * (SS + S) << a.lps_log2) + col;
            if (seg == LL - 1) {
#pragma unroll
                for (int e = 0; e < SS; ++e) mine[e << a.lps_log2] = accA[e];
#pragma unroll
                for (int s = 0; s < S; ++s) mine[(SS + s) << a.lps_log2] = accB[s];
            }
            __syncthreads();
            for (int j0 = 0; j0 < w; j0 += 4) {        // four aggregates per trip to LDS
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
#pragma unroll
        for (int s = 0; s < S; ++s) hprev[s] += din[s];
        auto substitute = [&](auto guard) {
#pragma unroll
            for (int i = 0; i < C; ++i) {
                float d[S];
                affine<S>(PA[i], din, qb[i], d);
#pragma unroll
                for (int s = 0; s < S; ++s) {
                    ho[i][s] += d[s];
                    if (!decltype(guard)::value || i < n_valid) wmax_bits = max(wmax_bits, __float_as_uint(d[s]) & 0x7fffffffu);
                }
            }
        };
        if (all_valid) substitute(std::false_type{});
        else substitute(std::true_type{});
        // ---- the stopping test of this group of channels
        unsigned int m = wave_max_u32(wmax_bits);
        if (W > 1) {
            if (lane == 0) s_max[w] = m;
            __syncthreads();
            m = wave_max_u32(s_max[lane < W ? lane : 0]);
        }
        const float mk = __uint_as_float(m);
        if (!(mk - mk == 0.0f)) { status = kStNonFinite; break; }
        if (a.tol >= 0.0f && mk <= a.tol) { status = kStOk; break; }
    }

#pragma unroll
    for (int i = 0; i < C; ++i)
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const float t[1] = {ho[i][s]};
            buf_store<UT, 1>(rh, vh, (unsigned int)(i * S + s) * Hn * E, t);
        }

    // ---- the verdict of the whole solve
    unsigned int v = short_verdict(status, k);
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
                __builtin_amdgcn_s_sleep(1);
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

// The adjoint scan and the gradients (Eq. (6)), formulas and variables as in backward_kernel.
template <class Cell, int C, typename UT>
__global__ __launch_bounds__((kWave * short_max_waves<Cell, C>())) __attribute__((amdgpu_waves_per_eu(short_min_waves<Cell, C>()))) void backward_short_kernel(const ShortArgs a)
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

    // ---- wave level: suffix scan over the segments to the right
    float lexA[SS], lexB[S];
    set_identity<S>(lexA);
#pragma unroll
    for (int s = 0; s < S; ++s) lexB[s] = 0.0f;
    if (LL > 1) {
        for (int d = 1; d < LL; d <<= 1) {
            float pA[SS], pB[S];
#pragma unroll
            for (int e = 0; e < SS; ++e) pA[e] = __shfl_down(accA[e], (unsigned int)(d << a.lps_log2), 64);
#pragma unroll
            for (int s = 0; s < S; ++s) pB[s] = __shfl_down(accB[s], (unsigned int)(d << a.lps_log2), 64);
            if (seg + d < LL) compose_after<S>(pA, pB, accA, accB);
        }
#pragma unroll
        for (int e = 0; e < SS; ++e) {
            const float t = __shfl_down(accA[e], (unsigned int)LPS, 64);
            if (seg < LL - 1) lexA[e] = t;
        }
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const float t = __shfl_down(accB[s], (unsigned int)LPS, 64);
            if (seg < LL - 1) lexB[s] = t;
        }
    }
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
