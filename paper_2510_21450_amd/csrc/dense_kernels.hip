// Dense-Jacobian path: h' = tanh(W h + u), J_l = diag(1 - F_l^2) W (the generic
// dense case of Sec. 2.1), H = 64, fp32.
//
// The linear solve of a Newton iteration is block bi-diagonal.  Two ways through it (wavefront_plan chooses):
// forward substitution, all iterations of a block at once as a wavefront (dense_wavefront_kernel,
// dense_adjoint_kernel: latency-bound, one workgroup per sequence, whole solves in two launches; sequences fewer than the
// compute units are cut into stretches that run side by side, in one launch, DenseStretch), and the chunked scan:
//
// One Newton iteration (Alg. 1a) is four launches (chunk_products and the local sweep share one):
//   residual  F_l = tanh(W h_{l-1} + u_l), d_l = 1 - F_l^2, r_l = F_l - h_l   (Eq. (3))
//   chunk_products   A_c = J_e ... J_s for every chunk of CD timesteps: the
//             64x64x64 Jacobian compositions of the scan, on the matrix cores
//             (v_mfma_f32_32x32x2_f32), one wave per (sequence, chunk)
//   sweep (local)    b_c = solution at the chunk's end for a zero input
//   carry            x_c = A_c x_{c-1} + b_c, sequential over the chunks of a sequence
//   sweep (final)    delta_l = J_l delta_{l-1} + r_l from x_{c-1}; h += delta; max|delta|
// The sweeps batch 16 (sequence, chunk) columns per workgroup so that the
// mat-vecs W delta of different columns become one MFMA product W [delta];
// the per-column factor d_l is applied to the product afterwards.
//
// Backward (Eq. (6)): with mu_l = d_l * lam_l (which is dL/du_l) the adjoint
// recurrence lam_l = g_l + W^T (d_{l+1} * lam_{l+1}) becomes
//   mu_l = diag(d_l) W^T mu_{l+1} + d_l * g_l,
// the same affine recurrence as the forward solve with W^T in place of W, the
// time axis reversed and r_l = d_l * g_l: the same kernels run it (rev = 1,
// W = the transposed matrix), followed by dL/dh0 = W^T mu_1 and
// dL/dW = sum_{b,l} mu_l h_{l-1}^T (one more MFMA reduction).
//
// MFMA operand trick: the 32x32 accumulator layout (lane = column, register v
// of lane half h = row 8*(v/4) + 4*h + v%4) is used unchanged as the B operand
// of the next product; the k-pair an instruction consumes is then (row(v,0),
// row(v,1)), and W is held in registers permuted to supply exactly those
// columns as the A operand.  No layout change is ever needed between products.
#include "pararnn.h"
#include "pararnn/common.h"
#include "dense.h"
#include "dense_plan.h"
#include "pararnn/driver.h"
#include "pararnn/launch.h"

#include <string.h>

#include <type_traits>

namespace pararnn {

namespace {

constexpr int DH = 64;          // hidden size this path is built for
constexpr int CD = 16;          // timesteps per chunk
typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef __bf16 bf2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef unsigned int u4v __attribute__((ext_vector_type(4)));

struct DenseArgs {
    const float *W;      // [64][64] row-major
    const float *u;      // [B][L][64]
    const float *h0;     // [B][64] or NULL
    float *h;            // [B][L][64] iterate, in place
    float *d;            // [B][L][64]
    float *r;            // [B][L][64]
    float *Ac;           // [B][n_c][64][64] row-major chunk products
    float *bc;           // [B][n_c][64] chunk-local end values
    float *xc;           // [B][n_c][64] delta at each chunk's end
    float *hend;         // [B][n_c][64] the iterate at each chunk's last step, as it was before this iteration's update (or NULL)
    Ctrl *ctrl;
    int *iters_out;
    float *trace;
    int B, L, n_c;
    int k, max_iter;
    float tol;
    // backward
    const float *g;      // dL/dh [B][L][64]
    float *du;           // out [B][L][64]: mu
    int rev;             // 1: scan step t of the recurrence is timestep L-1-t
    unsigned int *norm;  // residual max-norm only: bits of the result, zero on entry
    unsigned int *gmax;  // one-launch solve only: where the final sweep leaves max|delta| of this iteration
    unsigned int spin_limit;   // one-launch solve only: polls of a grid-wide barrier before a workgroup gives up
};

// row of the [B][L][64] arrays that scan step t of sequence b touches
__device__ __forceinline__ size_t scan_row(const DenseArgs &a, size_t b, int t)
{
    return b * a.L + (a.rev ? a.L - 1 - t : t);
}

__device__ __forceinline__ int mfma_row(int v, int half) { return 8 * (v >> 2) + 4 * half + (v & 3); }

// W in A-operand form: wr[mt][kt][v] = W[32 mt + lane%32][32 kt + row(v, lane/32)]
__device__ __forceinline__ void load_w_operand(const float *W, int lane, float (&wr)[2][2][16])
{
    const int n = lane & 31, half = lane >> 5;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                // rows(4g .. 4g+3, half) are four consecutive columns of W
                const float4 t = *reinterpret_cast<const float4 *>(W + (32 * mt + n) * DH + 32 * kt + 8 * g + 4 * half);
                wr[mt][kt][4 * g] = t.x; wr[mt][kt][4 * g + 1] = t.y; wr[mt][kt][4 * g + 2] = t.z; wr[mt][kt][4 * g + 3] = t.w;
            }
}

// W in A-operand form for the 16x16x4 products of wave w:
// wa[ww][v] = W[16w + n][16ww + 4g + v], lane = (n = lane % 16, g = lane / 16)
__device__ __forceinline__ void load_w_operand16(const float *W, int w, int n, int g, float (&wa)[4][4])
{
#pragma unroll
    for (int ww = 0; ww < 4; ++ww) {
        const f4v t = *reinterpret_cast<const f4v *>(W + (16 * w + n) * DH + 16 * ww + 4 * g);
#pragma unroll
        for (int v = 0; v < 4; ++v) wa[ww][v] = t[v];
    }
}

// ---------------------------------------------------------------- residual
// F = tanh(W h_{l-1} + u_l) for 16 consecutive rows (b, l) per workgroup as one
// 64 x 64 x 16 product W [h_{l-1} rows] on v_mfma_f32_16x16x4_f32: wave w owns
// channels 16w .. 16w+15, lane (n = lane % 16, g = lane / 16) ends up with
// channels 16w + 4g .. +3 of row n, so u, h, d and r move as float4.  The B
// operand of k-step (ww, v) is component v of the float4 at channels
// 16ww + 4g of the previous state, read straight from memory.
// mode 0: write d = 1 - F^2 and r = F - h for the current iterate;
// mode 1: write the initial guess h = tanh(W h0 + u) (App. A);
// mode 2: write nothing but max |F - h| over all rows to a.norm (no control block is read);
// mode 3: as mode 0, but d is the diagonal of the Jacobian, (1 - F^2) * W_ii (quasi-Newton);
// mode 4: modes 1 and 0 in one pass: the initial guess is written, and the residual and row factors of the
//         first iteration are formed from it.  The guess of the row before, which the residual needs, is
//         recomputed rather than read (it is tanh(W h0 + u_{l-1}), and W h0 is one product per row's sequence,
//         shared with the row's own guess): same bits as the two launches, one pass over u instead of two and
//         none over h;
// mode 5: d alone (no control block is read).
__device__ __forceinline__ void residual_body(const DenseArgs &a, int mode)
{
    float nmax = 0.0f;
    f4v wdiag = {1.0f, 1.0f, 1.0f, 1.0f};
    if (mode == 3) {
        const int c0 = 16 * __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) + 4 * (int)((threadIdx.x & 63) >> 4);
#pragma unroll
        for (int v = 0; v < 4; ++v) wdiag[v] = a.W[(c0 + v) * DH + c0 + v];
    }
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n = lane & 15, g = lane >> 4;
    const int chn = 16 * w + 4 * g;
    const size_t rows = (size_t)a.B * a.L;
    const size_t n_items = (rows + 15) / 16;
    float wa[4][4];
    load_w_operand16(a.W, w, n, g, wa);
    const f4v zero = {0.0f, 0.0f, 0.0f, 0.0f};
    __shared__ f4v s_c[4][64];
    for (size_t item = blockIdx.x; item < n_items; item += gridDim.x) {
        const size_t row = item * 16 + n;
        const bool ok = row < rows;
        const int l = ok ? (int)(row % a.L) : 0;
        const size_t b = ok ? row / a.L : 0;
        if (mode == 4) {
            // W h0 of this row's sequence: own part (channels chn ..) and, through LDS, every wave's part
            f4v cbo = zero, cbk[4] = {zero, zero, zero, zero};
            f4v h0k[4] = {zero, zero, zero, zero};
            if (a.h0) {
#pragma unroll
                for (int ww = 0; ww < 4; ++ww)
                    if (ok) h0k[ww] = *reinterpret_cast<const f4v *>(a.h0 + b * DH + 16 * ww + 4 * g);
                f4v c0 = zero, c1 = zero;
#pragma unroll
                for (int ww = 0; ww < 4; ww += 2)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[ww][v], h0k[ww][v], c0, 0, 0, 0);
                        c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[ww + 1][v], h0k[ww + 1][v], c1, 0, 0, 0);
                    }
                cbo = c0 + c1;
                __syncthreads();                      // the previous item's reads of s_c
                s_c[w][lane] = cbo;
                __syncthreads();
#pragma unroll
                for (int ww = 0; ww < 4; ++ww) cbk[ww] = s_c[ww][lane];
            }
            f4v uv = zero;
            f4v xb[4] = {zero, zero, zero, zero};
            if (ok) {
                uv = *reinterpret_cast<const f4v *>(a.u + row * DH + chn);
                if (l == 0) {
#pragma unroll
                    for (int ww = 0; ww < 4; ++ww) xb[ww] = h0k[ww];
                } else {
#pragma unroll
                    for (int ww = 0; ww < 4; ++ww) {
                        const f4v y = cbk[ww] + *reinterpret_cast<const f4v *>(a.u + (row - 1) * DH + 16 * ww + 4 * g);
#pragma unroll
                        for (int v = 0; v < 4; ++v) xb[ww][v] = fast_tanh(y[v]);
                    }
                }
            }
            f4v acc0 = zero, acc1 = zero;
#pragma unroll
            for (int ww = 0; ww < 4; ww += 2)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[ww][v], xb[ww][v], acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[ww + 1][v], xb[ww + 1][v], acc1, 0, 0, 0);
                }
            if (ok) {
                const f4v y0 = cbo + uv, y = acc0 + acc1 + uv;
                f4v hv, F;
#pragma unroll
                for (int v = 0; v < 4; ++v) { hv[v] = fast_tanh(y0[v]); F[v] = fast_tanh(y[v]); }
                *reinterpret_cast<f4v *>(a.h + row * DH + chn) = hv;
                *reinterpret_cast<f4v *>(a.d + row * DH + chn) = (1.0f - F * F) * wdiag;
                *reinterpret_cast<f4v *>(a.r + row * DH + chn) = F - hv;
            }
            continue;
        }
        // previous state of this row: h0 (or zero) at l = 0 and for the guess, else the row before
        const float *hp = nullptr;
        if (ok) {
            if (mode == 1 || l == 0) hp = a.h0 ? a.h0 + b * DH : nullptr;
            else hp = a.h + (row - 1) * DH;
        }
        f4v xb[4];
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) xb[ww] = hp ? *reinterpret_cast<const f4v *>(hp + 16 * ww + 4 * g) : zero;
        f4v uv = zero, hv = zero;
        if (ok) {
            uv = *reinterpret_cast<const f4v *>(a.u + row * DH + chn);
            if (mode != 1 && mode != 5) hv = *reinterpret_cast<const f4v *>(a.h + row * DH + chn);
        }
        f4v acc0 = zero, acc1 = zero;
#pragma unroll
        for (int ww = 0; ww < 4; ww += 2)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[ww][v], xb[ww][v], acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[ww + 1][v], xb[ww + 1][v], acc1, 0, 0, 0);
            }
        if (ok) {
            const f4v y = acc0 + acc1 + uv;
            f4v F;
#pragma unroll
            for (int v = 0; v < 4; ++v) F[v] = fast_tanh(y[v]);
            if (mode == 1) {
                *reinterpret_cast<f4v *>(a.h + row * DH + chn) = F;
            } else if (mode == 2) {
#pragma unroll
                for (int v = 0; v < 4; ++v) nmax = nanmax(nmax, fabsf(hv[v] - F[v]));
            } else {
                *reinterpret_cast<f4v *>(a.d + row * DH + chn) = (1.0f - F * F) * wdiag;
                if (mode != 5) *reinterpret_cast<f4v *>(a.r + row * DH + chn) = F - hv;
            }
        }
    }
    if (mode == 2) {
        // one atomic per workgroup: they all go to one address
        __shared__ float s_nmax[4];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) nmax = nanmax(nmax, __shfl_xor(nmax, off, 64));
        if (lane == 0) s_nmax[w] = nmax;
        __syncthreads();
        if (threadIdx.x == 0) {
            nmax = nanmax(nanmax(s_nmax[0], s_nmax[1]), nanmax(s_nmax[2], s_nmax[3]));
            atomicMax(a.norm, nmax != nmax ? 0x7fc00000u : __float_as_uint(nmax));
        }
    }
}

__global__ __launch_bounds__(256) void dense_residual_kernel(const DenseArgs a, int mode)
{
    if (mode != 2 && mode != 5 && a.ctrl->stop) return;
    residual_body(a, mode);
}

// ------------------------------------------------------------ chunk products
// A_c = J_e ... J_{s+1} J_s with J_l = diag(d_l) W, one wave per (b, chunk).
// Chunk 0 and the last chunk are skipped: nothing enters chunk 0 (delta_0 = 0)
// and nothing follows the last one.
__device__ __forceinline__ void chunk_products_body(const DenseArgs &a, int block)
{
    const int lane = threadIdx.x & 63, n = lane & 31, half = lane >> 5;
    const int item = block * 4 + (threadIdx.x >> 6);
    const int per_seq = a.n_c - 2;
    if (per_seq <= 0 || item >= a.B * per_seq) return;
    const int b = item / per_seq, c = 1 + item % per_seq;
    const int ls = c * CD, n_steps = min(a.L, ls + CD) - ls;

    float wr[2][2][16];
    load_w_operand(a.W, lane, wr);

    // P = J_ls in accumulator layout: P[mt][nt][v] = d[row] W[row][32 nt + n]
    f16v P[2][2], Q[2][2];
    const float *dl0 = a.d + scan_row(a, b, ls) * DH;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int row = 32 * mt + mfma_row(v, half);
            const float dv = dl0[row];
            P[mt][0][v] = dv * a.W[row * DH + n];
            P[mt][1][v] = dv * a.W[row * DH + 32 + n];
        }
    // dst = diag(d) W src.  The two products alternate between P and Q, so no
    // accumulator is ever copied: the result of one step is the B operand of the next.
    auto compose = [&](const f16v(&src)[2][2], f16v(&dst)[2][2], float d0, float d1) {
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int v = 0; v < 16; ++v) dst[mt][nt][v] = 0.0f;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float a0 = wr[0][kt][v] * d0, a1 = wr[1][kt][v] * d1;
                const float b0 = src[kt][0][v], b1 = src[kt][1][v];
                dst[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b0, dst[0][0], 0, 0, 0);
                dst[0][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b1, dst[0][1], 0, 0, 0);
                dst[1][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b0, dst[1][0], 0, 0, 0);
                dst[1][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b1, dst[1][1], 0, 0, 0);
            }
    };
    // row factors of the next two steps are fetched while the current two run
    // (indices clamped to the chunk: the extra values are never used)
    auto dload = [&](int i, int hi) { return a.d[scan_row(a, b, ls + min(i, n_steps - 1)) * DH + 32 * hi + n]; };
    float da0 = dload(1, 0), da1 = dload(1, 1), db0 = dload(2, 0), db1 = dload(2, 1);
    int i = 1;
#pragma unroll 1
    for (; i + 1 < n_steps; i += 2) {
        const float na0 = dload(i + 2, 0), na1 = dload(i + 2, 1), nb0 = dload(i + 3, 0), nb1 = dload(i + 3, 1);
        compose(P, Q, da0, da1);
        compose(Q, P, db0, db1);
        da0 = na0; da1 = na1; db0 = nb0; db1 = nb1;
    }
    const bool odd = i < n_steps;                 // one step left: the result ends up in Q
    if (odd) compose(P, Q, da0, da1);
    float *out = a.Ac + ((size_t)b * a.n_c + c) * DH * DH;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                out[(32 * mt + mfma_row(v, half)) * DH + 32 * nt + n] = odd ? Q[mt][nt][v] : P[mt][nt][v];
}

// ------------------------------------------- chunk products, bf16 matrix cores
// The same compositions with the operands split into bf16 terms (an inexact
// Jacobian for the Newton step: the residual stays fp32, so the solve converges to
// the same states; only the carries x_c are computed from approximate A_c).
// TERMS = 3: x = hi + lo with hi = bf16(x), lo = bf16(x - hi), and
//   W B ~ W_hi B_hi + W_hi B_lo + W_lo B_hi   (relative error ~2^-16 per product);
// TERMS = 1: W_hi B_hi only (~2^-8).
// v_mfma_f32_32x32x16_bf16 takes eight consecutive k per lane half.  As in the
// fp32 kernel the accumulator is fed back as the B operand without a layout
// change: k-slot j of lane half g of k-block kb stands for row
// 16 kb + 8 (j / 4) + 4 g + j % 4 of the 32-row block, which is accumulator
// register 8 kb + j, and W is held in registers with its columns in that order.
// The row factor d_l is applied to the fp32 result, so W's split is done once.
__device__ __forceinline__ unsigned int pack_bf16(float x0, float x1)
{
    const bf2v p = {(__bf16)x0, (__bf16)x1};
    return __builtin_bit_cast(unsigned int, p);
}

// registers 8 kb .. 8 kb + 7 of an accumulator as bf16 operand(s)
template <int TERMS>
__device__ __forceinline__ void split_operand(const f16v &x, int kb, bf8v &hi, bf8v &lo)
{
    u4v ph, pl = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float x0 = x[8 * kb + 2 * j], x1 = x[8 * kb + 2 * j + 1];
        const unsigned int pk = pack_bf16(x0, x1);
        ph[j] = pk;
        if (TERMS > 1) {
            const float h0 = __builtin_bit_cast(float, pk << 16), h1 = __builtin_bit_cast(float, pk & 0xffff0000u);
            pl[j] = pack_bf16(x0 - h0, x1 - h1);
        }
    }
    hi = __builtin_bit_cast(bf8v, ph);
    lo = __builtin_bit_cast(bf8v, pl);
}

template <int TERMS>
__device__ __forceinline__ void chunk_products_bf16_body(const DenseArgs &a, int block)
{
    const int lane = threadIdx.x & 63, n = lane & 31, half = lane >> 5;
    const int item = block * 4 + (threadIdx.x >> 6);
    const int per_seq = a.n_c - 2;
    if (per_seq <= 0 || item >= a.B * per_seq) return;
    const int b = item / per_seq, c = 1 + item % per_seq;
    const int ls = c * CD, n_steps = min(a.L, ls + CD) - ls;

    // W as A operands: whi[mt][kt][kb] slot j = W[32 mt + n][32 kt + 16 kb + 8 (j/4) + 4 half + j%4]
    bf8v whi[2][2][2], wlo[2][2][2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int kb = 0; kb < 2; ++kb) {
                f16v t;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const f4v w4 = *reinterpret_cast<const f4v *>(a.W + (32 * mt + n) * DH + 32 * kt + 16 * kb + 8 * q + 4 * half);
#pragma unroll
                    for (int e = 0; e < 4; ++e) t[4 * q + e] = w4[e];
                }
                split_operand<TERMS>(t, 0, whi[mt][kt][kb], wlo[mt][kt][kb]);
            }

    // The row factors of the chunk go through LDS (one region per wave): rows of d arrive as
    // coalesced float4 loads and are read back in accumulator order, dq[mt][q] =
    // d[32 mt + 8 q + 4 half .. +3], the same 16 bytes for all lanes of a half.  Only this
    // wave touches its region, and a wave's LDS operations complete in order.
    __shared__ __attribute__((aligned(16))) float s_d[4][CD][DH];
    float(*sd)[DH] = s_d[threadIdx.x >> 6];
#pragma unroll
    for (int j = 0; j < CD / 4; ++j) {
        const int i = 4 * j + (lane >> 4);
        const f4v t = *reinterpret_cast<const f4v *>(a.d + scan_row(a, b, ls + min(i, n_steps - 1)) * DH + 4 * (lane & 15));
        *reinterpret_cast<f4v *>(&sd[i][4 * (lane & 15)]) = t;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    auto dload = [&](int i, f4v(&dq)[2][4]) {
        const int ii = min(i, CD - 1);                // the value past the last step is never used
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int q = 0; q < 4; ++q) dq[mt][q] = *reinterpret_cast<const f4v *>(&sd[ii][32 * mt + 8 * q + 4 * half]);
    };
    // acc = J_ls in accumulator layout: acc[mt][nt][v] = d[row] W[row][32 nt + n]
    f16v acc[2][2];
    {
        f4v d0[2][4];
        dload(0, d0);
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = 32 * mt + mfma_row(v, half);
                const float dv = d0[mt][v >> 2][v & 3];
                acc[mt][0][v] = dv * a.W[row * DH + n];
                acc[mt][1][v] = dv * a.W[row * DH + 32 + n];
            }
    }
    f4v dcur[2][4], dnext[2][4];
    dload(1, dcur);
#pragma unroll 1
    for (int i = 1; i < n_steps; ++i) {
        dload(i + 1, dnext);
        bf8v bhi[2][2][2], blo[2][2][2];              // [kt][nt][kb]
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) split_operand<TERMS>(acc[kt][nt], kb, bhi[kt][nt][kb], blo[kt][nt][kb]);
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int nt = 0; nt < 2; ++nt) {
                f16v s;
#pragma unroll
                for (int v = 0; v < 16; ++v) s[v] = 0.0f;
                if (TERMS > 1) {
                    // the small terms first
#pragma unroll
                    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb) {
                            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(whi[mt][kt][kb], blo[kt][nt][kb], s, 0, 0, 0);
                            s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wlo[mt][kt][kb], bhi[kt][nt][kb], s, 0, 0, 0);
                        }
                }
#pragma unroll
                for (int kt = 0; kt < 2; ++kt)
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb)
                        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(whi[mt][kt][kb], bhi[kt][nt][kb], s, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[mt][nt][v] = s[v] * dcur[mt][v >> 2][v & 3];
            }
#pragma unroll
        for (int mt = 0; mt < 2; ++mt)
#pragma unroll
            for (int q = 0; q < 4; ++q) dcur[mt][q] = dnext[mt][q];
    }
    float *out = a.Ac + ((size_t)b * a.n_c + c) * DH * DH;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int v = 0; v < 16; ++v) out[(32 * mt + mfma_row(v, half)) * DH + 32 * nt + n] = acc[mt][nt][v];
}

// The last workgroup of the final sweep closes the iteration: stopping test,
// results, reset of the counters (same protocol as the scan kernels).
__device__ __forceinline__ void finish_iteration(const DenseArgs &a, float block_max)
{
    Ctrl *ctrl = a.ctrl;
    atomicMax(&ctrl->gmax_bits, __float_as_uint(block_max));
    __threadfence();
    const unsigned int prev = atomicAdd(&ctrl->done, 1u);
    if (prev == gridDim.x - 1) {
        __threadfence();
        const float mk = __uint_as_float(atomicMax(&ctrl->gmax_bits, 0u));
        int status, stop = 0;
        if (a.trace) a.trace[a.k - 1] = mk;
        if (!(mk - mk == 0.0f)) { status = kStNonFinite; stop = 1; }
        else if (a.tol >= 0.0f && mk <= a.tol) { status = kStOk; stop = 1; }
        else status = a.tol < 0.0f ? kStOk : kStNotConverged;
        a.iters_out[0] = a.k;
        a.iters_out[1] = status;
        ctrl->iters = a.k;
        ctrl->status = status;
        ctrl->stop = stop;
        ctrl->done = 0u;
        ctrl->gmax_bits = 0u;
        __threadfence();
    }
}

// -------------------------------------------------------------------- sweeps
// x <- diag(d_l) (W x) + r_l over the CD steps of a chunk.  The chain is
// sequential, so what counts is the latency of one step; every (sequence,
// chunk) pair is an independent column, and one workgroup advances 16 columns
// with the 64 x 64 x 16 product of a step split over its four waves: wave w
// owns rows 16w .. 16w+15 and issues 16 v_mfma_f32_16x16x4_f32.
//
// Operand layout: the 16x16 accumulator gives lane (n = lane % 16, g = lane / 16)
// the rows 16w + 4g + v, v = 0..3, of column n.  Each wave drops its float4 into
// LDS at [w][lane]; for the next step every wave reads the four float4 at
// [ww][lane], ww = 0..3, and uses component v of wave ww's value as the B
// operand of k-step (ww, v), whose four k-slots (one per lane group g) are then
// the rows 16ww + 4g + v.  W is held in registers in the matching A-operand
// order, so the exchange is one float4 write and four conflict-free float4
// reads per step, with no index arithmetic.
//
// d and r (and h) of all CD steps are loaded before the chain starts; the barrier
// between steps orders LDS only.
// final = 0: x starts at 0, only the end value is kept (b_c).
// final = 1: x starts at x_{c-1}; afterwards h += delta and max|delta|.
// BWD: the backward recurrence (r_l = d_l * g_l; the final sweep writes mu = dL/du and nothing else).
// LATE_H: the iterate's rows are read after the chain instead of before it (48 fewer registers held
// through the chain; the one-launch solve shares its register budget with the chunk products).
//
// Forward solves: the delta of a chunk's last step exists twice, as the end of this chain and as the carried
// value x_c that every later chunk started from; the update takes x_c, so that the iterate at a chunk's last
// step is (old value + x_c), which the next chunk's column can form by itself.  The chunk-local sweep leaves the
// old values of those steps in a.hend for that purpose (the final sweeps of neighbouring chunks run side by side
// and update h in place).
// NEXT (final forward sweep): the residual and row factors of the NEXT iteration are formed here, from the
// new rows this column holds, instead of by a launch of their own that would read the iterate again:
// row l needs the new h_{l-1} (for l = ls: hend + x_{c-1}, or h0) and the new h_l.  Same products in the same
// order as dense_residual_kernel, so both give the same bits.
template <int FINAL, bool BWD, bool LATE_H = false, bool NEXT = false>
__device__ __forceinline__ void sweep_body(const DenseArgs &a, int block)
{
    static_assert(!NEXT || (FINAL && !BWD && !LATE_H), "the next residual belongs to the forward final sweep");
    __shared__ f4v s_x[2][4][64];
    __shared__ float s_max[4];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n = lane & 15, g = lane >> 4;
    const int n_cols = a.B * a.n_c;
    const int col = block * 16 + n;
    const bool ok = col < n_cols;
    const int cc = ok ? col : n_cols - 1;         // a column past the end reads valid memory and stores nothing
    const int b = cc / a.n_c, c = cc - b * a.n_c;
    const int ls = c * CD;
    const int chn = 16 * w + 4 * g;               // first of this lane's four channels

    float wa[4][4];
    load_w_operand16(a.W, w, n, g, wa);
    const f4v zero = {0.0f, 0.0f, 0.0f, 0.0f};
    f4v dv[CD], rv[CD], hv[(FINAL && !BWD && !LATE_H) ? CD : 1];
#pragma unroll
    for (int i = 0; i < CD; ++i) {
        const int l = ls + i;
        const size_t off = scan_row(a, b, min(l, a.L - 1)) * DH + chn;
        dv[i] = *reinterpret_cast<const f4v *>(a.d + off);
        if (BWD) rv[i] = dv[i] * *reinterpret_cast<const f4v *>(a.g + off);
        else rv[i] = *reinterpret_cast<const f4v *>(a.r + off);
        if (FINAL && !BWD && !LATE_H) hv[i] = *reinterpret_cast<const f4v *>(a.h + off);
        if (!(ok && l < a.L)) { dv[i] = zero; rv[i] = zero; }     // steps past the end leave x = 0
    }
    f4v x = zero;
    if (FINAL && ok && c > 0) x = *reinterpret_cast<const f4v *>(a.xc + ((size_t)b * a.n_c + (c - 1)) * DH + chn);
    // forward: the carried delta of this chunk's last step, and (chunk-local sweep) the iterate there
    const bool carried_end = !BWD && a.hend && ok && c < a.n_c - 1;
    f4v xend = zero;
    if (FINAL && carried_end) xend = *reinterpret_cast<const f4v *>(a.xc + ((size_t)b * a.n_c + c) * DH + chn);
    if (!FINAL && carried_end)
        *reinterpret_cast<f4v *>(a.hend + ((size_t)b * a.n_c + c) * DH + chn) =
            *reinterpret_cast<const f4v *>(a.h + ((size_t)b * a.L + ls + CD - 1) * DH + chn);
    const f4v xstart = x;
    s_x[0][w][lane] = x;
    lds_barrier();
#pragma unroll
    for (int i = 0; i < CD; ++i) {
        f4v acc0 = zero, acc1 = zero;
#pragma unroll
        for (int ww = 0; ww < 4; ww += 2) {
            const f4v xa = s_x[i & 1][ww][lane], xb = s_x[i & 1][ww + 1][lane];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[ww][v], xa[v], acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[ww + 1][v], xb[v], acc1, 0, 0, 0);
            }
        }
        x = dv[i] * (acc0 + acc1) + rv[i];
        if (FINAL) rv[i] = x;                     // delta_l, applied to h after the chain
        if (i + 1 < CD) {
            s_x[(i + 1) & 1][w][lane] = x;
            lds_barrier();
        }
    }
    if (!FINAL) {
        if (ok) *reinterpret_cast<f4v *>(a.bc + ((size_t)b * a.n_c + c) * DH + chn) = x;
        return;
    }
    if (BWD) {
#pragma unroll
        for (int i = 0; i < CD; ++i) {
            const int l = ls + i;
            if (ok && l < a.L) *reinterpret_cast<f4v *>(a.du + scan_row(a, b, l) * DH + chn) = rv[i];
        }
        return;
    }
    if (carried_end) rv[CD - 1] = xend;
    float wmax = 0.0f;
    if constexpr (NEXT) {
        // u of this column's rows (the registers of the row factors are free now)
        f4v uv[CD];
#pragma unroll
        for (int i = 0; i < CD; ++i)
            uv[i] = *reinterpret_cast<const f4v *>(a.u + ((size_t)b * a.L + min(ls + i, a.L - 1)) * DH + chn);
        // the state in front of the column's first row
        f4v hprev = zero;
        if (ok) {
            if (c == 0) {
                if (a.h0) hprev = *reinterpret_cast<const f4v *>(a.h0 + (size_t)b * DH + chn);
            } else {
                hprev = *reinterpret_cast<const f4v *>(a.hend + ((size_t)b * a.n_c + (c - 1)) * DH + chn) + xstart;
            }
        }
        // every wave needs all 64 values of each state: slot i holds the state in front of row i
        __shared__ f4v s_h[CD][4][64];
        s_h[0][w][lane] = hprev;
#pragma unroll
        for (int i = 0; i < CD; ++i) {
            const int l = ls + i;
#pragma unroll
            for (int v = 0; v < 4; ++v) wmax = nanmax(wmax, __builtin_fabsf(rv[i][v]));
            rv[i] = hv[i] + rv[i];                                  // the new row
            if (ok && l < a.L) *reinterpret_cast<f4v *>(a.h + ((size_t)b * a.L + l) * DH + chn) = rv[i];
            if (i + 1 < CD) s_h[i + 1][w][lane] = rv[i];
        }
        lds_barrier();
#pragma unroll
        for (int i = 0; i < CD; ++i) {
            const int l = ls + i;
            f4v acc0 = zero, acc1 = zero;
#pragma unroll
            for (int ww = 0; ww < 4; ww += 2) {
                const f4v xa = s_h[i][ww][lane], xb = s_h[i][ww + 1][lane];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[ww][v], xa[v], acc0, 0, 0, 0);
                    acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[ww + 1][v], xb[v], acc1, 0, 0, 0);
                }
            }
            if (ok && l < a.L) {
                const f4v y = acc0 + acc1 + uv[i];
                f4v F;
#pragma unroll
                for (int v = 0; v < 4; ++v) F[v] = fast_tanh(y[v]);
                const size_t off = ((size_t)b * a.L + l) * DH + chn;
                *reinterpret_cast<f4v *>(a.d + off) = (1.0f - F * F);
                *reinterpret_cast<f4v *>(a.r + off) = F - rv[i];
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < CD; ++i) {
            const int l = ls + i;
            if (ok && l < a.L) {
                f4v *hp = reinterpret_cast<f4v *>(a.h + ((size_t)b * a.L + l) * DH + chn);
                if (LATE_H) *hp = *hp + rv[i];
                else *hp = hv[i] + rv[i];
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) wmax = nanmax(wmax, __builtin_fabsf(rv[i][v]));
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) wmax = nanmax(wmax, __shfl_xor(wmax, off, 64));
    if (lane == 0) s_max[w] = wmax;
    __syncthreads();
    if (threadIdx.x == 0) {
        const float bm = nanmax(nanmax(s_max[0], s_max[1]), nanmax(s_max[2], s_max[3]));
        if (a.gmax) atomicMax(a.gmax, __float_as_uint(bm));       // the one-launch solve decides after its barrier
        else finish_iteration(a, bm);
    }
}

// The final sweep of an iteration (or of the backward pass).  NEXT: it also leaves the residual and the row
// factors of the next iteration.
template <bool BWD, bool NEXT = false>
__global__ __launch_bounds__(256) void dense_final_sweep_kernel(const DenseArgs a)
{
    if (a.ctrl->stop) return;
    sweep_body<1, BWD, false, NEXT>(a, blockIdx.x);
}

// Chunk products and chunk-local sweeps need only d and r, and nothing of each
// other: one launch runs both.  The first n_sweep workgroups take the sweeps,
// whose sequential chains are bound by latency and so start first; the rest
// compose the chunk products, which keep the matrix cores busy meanwhile.
// PROD: how the chunk products are formed: 0 fp32, 1 three bf16 terms, 2 one bf16 term
template <bool BWD, int PROD>
__global__ __launch_bounds__(256, 2) void dense_products_sweep_kernel(const DenseArgs a, int n_sweep)
{
    if (a.ctrl->stop) return;
    if ((int)blockIdx.x < n_sweep) sweep_body<0, BWD>(a, blockIdx.x);
    else if (PROD == 0) chunk_products_body(a, (int)blockIdx.x - n_sweep);
    else chunk_products_bf16_body<PROD == 1 ? 3 : 1>(a, (int)blockIdx.x - n_sweep);
}

// process-wide choice of the product arithmetic of forward solves (pararnn_set_dense_products)
int g_dense_products = 0;
int g_dense_jacobian = 0;       // 0: the full Jacobian (Newton), 1: its diagonal (quasi-Newton)
int g_dense_one_launch = 1;     // 1: the first kDenseHead iterations as launches per phase, the rest in one persistent
                                // launch; 0: launches per phase throughout; 2: the persistent launch from the start
int g_dense_substitution = 1;   // 0: every linear system is solved by the chunked scan
constexpr int kDenseHead = 6;


void launch_products_sweep(int prod, int blocks, hipStream_t st, const DenseArgs &a, int n_sweep)
{
    if (prod == 1) hipLaunchKernelGGL((dense_products_sweep_kernel<false, 1>), dim3(blocks), dim3(256), 0, st, a, n_sweep);
    else if (prod == 2) hipLaunchKernelGGL((dense_products_sweep_kernel<false, 2>), dim3(blocks), dim3(256), 0, st, a, n_sweep);
    else hipLaunchKernelGGL((dense_products_sweep_kernel<false, 0>), dim3(blocks), dim3(256), 0, st, a, n_sweep);
}

// --------------------------------------------------------------------- carry
// x_c = A_c x_{c-1} + b_c for c = 0 .. n_c-2 (x_{-1} = 0, so x_0 = b_0), one
// workgroup per sequence.  Lane (row = lane / 4, q = lane % 4) of wave w holds
// columns 16j + 4q .. 16j + 4q + 3, j = 0..3, of row 16w + row of A_c (so that the
// four lanes of a quad load 64 contiguous bytes at a time): sixteen FMAs against x from
// LDS, two DPP adds across the quad, and the row's new value goes back to LDS.
// The matrices of the next DEPTH chunks are in flight meanwhile; the loop body
// is branch-free around the loads (indices are clamped) and its barrier orders
// LDS only, so those loads stay outstanding across steps.
__device__ __forceinline__ void carry_body(const DenseArgs &a, int b)
{
    constexpr int DEPTH = 8;
    __shared__ __attribute__((aligned(16))) float s_x[2][DH];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int row = 16 * w + (lane >> 2), q = lane & 3;
    const float *bcb = a.bc + (size_t)b * a.n_c * DH + row;
    float *xcb = a.xc + (size_t)b * a.n_c * DH + row;
    const float *Ab = a.Ac + ((size_t)b * a.n_c * DH + row) * DH + 4 * q;    // this lane's first columns, chunk 0
    const int last = a.n_c - 2;                       // last chunk whose end value is needed
    {
        const float x0 = bcb[0];
        if (q == 0) { s_x[0][row] = x0; xcb[0] = x0; }
    }
    if (last < 1) return;
    f4v buf[DEPTH][4];
    float bb[DEPTH];
#pragma unroll
    for (int k = 0; k < DEPTH; ++k) {
        const int c = min(1 + k, last);
#pragma unroll
        for (int j = 0; j < 4; ++j) buf[k][j] = *reinterpret_cast<const f4v *>(Ab + (size_t)c * DH * DH + 16 * j);
        bb[k] = bcb[(size_t)c * DH];
    }
    lds_barrier();
    int cur = 0;
    for (int base = 1; base <= last; base += DEPTH) {
#pragma unroll
        for (int k = 0; k < DEPTH; ++k) {
            const int c = base + k;
            const f4v *xs = reinterpret_cast<const f4v *>(&s_x[cur][4 * q]);
            f4v s = buf[k][0] * xs[0];
#pragma unroll
            for (int j = 1; j < 4; ++j) s = buf[k][j] * xs[4 * j] + s;
            float t = (s[0] + s[1]) + (s[2] + s[3]);
            t += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, t), 0xB1, 0xf, 0xf, false));
            t += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, t), 0x4E, 0xf, 0xf, false));
            const float xn = t + bb[k];
            // past the last chunk nothing is written and the buffers do not flip
            if (c <= last) {
                if (q == 0) { s_x[cur ^ 1][row] = xn; xcb[(size_t)c * DH] = xn; }
                cur ^= 1;
            }
            const int cn = min(c + DEPTH, last);
#pragma unroll
            for (int j = 0; j < 4; ++j) buf[k][j] = *reinterpret_cast<const f4v *>(Ab + (size_t)cn * DH * DH + 16 * j);
            bb[k] = bcb[(size_t)cn * DH];
            lds_barrier();
        }
    }
}

__global__ __launch_bounds__(256) void dense_carry_kernel(const DenseArgs a)
{
    if (a.ctrl->stop) return;
    carry_body(a, blockIdx.x);
}

// ------------------------------------------------- the whole solve in one launch
// Newton iterations of a forward solve in ONE persistent launch: the phases of an
// iteration (residual; chunk products + chunk-local sweeps; carry; final sweep) are
// separated by grid-wide barriers instead of kernel boundaries, the stopping test is
// taken by every workgroup from the same device-wide maximum right after the last
// barrier of an iteration, and the launch ends with the iteration that met the
// tolerance: no launch is enqueued for iterations that never run.  The grid is what
// the device holds at once (every workgroup is resident, so every barrier is reached
// by all of them); a barrier wait is bounded like the look-back waits of the scan
// kernels and ends the launch with status INTERNAL if it ever runs out.
//
// Words 16.. of the control block: [0], [1] max|delta| bits of odd / even iterations,
// [2] barrier arrivals (monotone), [3] ticket of the chunk-product workgroup items.
__device__ __forceinline__ bool grid_barrier(unsigned int *arrivals, unsigned int &generation, unsigned int spin_limit)
{
    __shared__ int s_ok;
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();                              // this workgroup's writes, before it arrives
        ++generation;
        const unsigned int target = generation * gridDim.x;
        atomicAdd(arrivals, 1u);
        unsigned int spins = 0;
        int ok = 1;
        while (__hip_atomic_load(arrivals, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target) {
            if (++spins >= spin_limit) { ok = 0; break; }
            __builtin_amdgcn_s_sleep(16);             // about half a microsecond: hundreds of workgroups poll one word
        }
        __threadfence();                              // the others' writes, after all have arrived
        s_ok = ok;
    }
    __syncthreads();
    return s_ok != 0;
}

// Each phase is a function of its own (not inlined): the phases keep W and their row addresses
// in registers in different layouts, and inlined into one body the compiler would carry all of
// them through the whole iteration loop and spill.  A phase reads the launch's arguments from the
// kernel-argument block and gets what changes per iteration by value.
__device__ __attribute__((noinline)) void phase_residual(const DenseArgs *ap, int mode)
{
    const DenseArgs a = *ap;
    residual_body(a, mode);
}

template <int PROD>
__device__ __attribute__((noinline)) void phase_products_sweeps(const DenseArgs *ap, unsigned int *ticket, int n_sweep,
                                                              int n_prod_blocks)
{
    __shared__ unsigned int s_t;
    const DenseArgs a = *ap;
    // chunk-local sweeps first (sequential chains, bound by latency), then the chunk products,
    // handed out by a ticket so that the workgroups that swept do not finish last
    for (int blk = blockIdx.x; blk < n_sweep; blk += gridDim.x) {
        sweep_body<0, false>(a, blk);
        __syncthreads();
    }
    for (;;) {
        if (threadIdx.x == 0) s_t = atomicAdd(ticket, 1u);
        __syncthreads();
        const unsigned int t = __builtin_amdgcn_readfirstlane(s_t);
        __syncthreads();
        if (t >= (unsigned int)n_prod_blocks) break;
        if (PROD == 0) chunk_products_body(a, (int)t);
        else chunk_products_bf16_body<PROD == 1 ? 3 : 1>(a, (int)t);
    }
}

__device__ __attribute__((noinline)) void phase_carry(const DenseArgs *ap)
{
    const DenseArgs a = *ap;
    for (int b = blockIdx.x; b < a.B; b += gridDim.x) {
        carry_body(a, b);
        __syncthreads();
    }
}

__device__ __attribute__((noinline)) void phase_final_sweep(const DenseArgs *ap, unsigned int *gmax, int n_sweep)
{
    DenseArgs a = *ap;
    a.gmax = gmax;
    for (int blk = blockIdx.x; blk < n_sweep; blk += gridDim.x) {
        sweep_body<1, false, true>(a, blk);
        __syncthreads();
    }
}

// k_first = 1: the solve from the initial guess; k_first > 1: iterations k_first .. max_iter of a
// solve whose earlier iterations ran as separate launches (nothing to do when one of them ended it).
template <int PROD>
__global__ __launch_bounds__(256, 2) void dense_newton_kernel(const DenseArgs a, int n_sweep, int n_prod_blocks,
                                                              int k_first)
{
    Ctrl *ctrl = a.ctrl;
    if (ctrl->stop) return;
    unsigned int *aux = reinterpret_cast<unsigned int *>(ctrl) + 16;
    unsigned int generation = 0;
    bool alive = true;
    if (k_first == 1) {
        // initial guess h^0_l = tanh(W h0 + u_l) (App. A); rows are independent
        phase_residual(&a, 1);
        alive = grid_barrier(aux + 2, generation, a.spin_limit);
    }
    int k = k_first;
    for (; alive && k <= a.max_iter; ++k) {
        unsigned int *gmax = aux + (k & 1);
        phase_residual(&a, 0);
        if (!(alive = grid_barrier(aux + 2, generation, a.spin_limit))) break;
        phase_products_sweeps<PROD>(&a, aux + 3, n_sweep, n_prod_blocks);
        if (!(alive = grid_barrier(aux + 2, generation, a.spin_limit))) break;
        phase_carry(&a);
        if (!(alive = grid_barrier(aux + 2, generation, a.spin_limit))) break;
        phase_final_sweep(&a, gmax, n_sweep);
        if (!(alive = grid_barrier(aux + 2, generation, a.spin_limit))) break;
        // every workgroup reads the same maximum and takes the same decision
        const float mk = __uint_as_float(__hip_atomic_load(gmax, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        int status, stop = 0;
        if (!(mk - mk == 0.0f)) { status = kStNonFinite; stop = 1; }
        else if (a.tol >= 0.0f && mk <= a.tol) { status = kStOk; stop = 1; }
        else status = a.tol < 0.0f ? kStOk : kStNotConverged;
        if (blockIdx.x == 0 && threadIdx.x == 0) {
            if (a.trace) a.trace[k - 1] = mk;
            a.iters_out[0] = k;
            a.iters_out[1] = status;
            ctrl->iters = k;
            ctrl->status = status;
            ctrl->stop = stop;
            // for the next iteration: its maximum slot was last read two iterations ago, and the
            // product ticket is not drawn again before two more barriers
            aux[(k + 1) & 1] = 0u;
            aux[3] = 0u;
        }
        if (stop) break;
    }
    if (!alive && threadIdx.x == 0) {
        atomicExch(&ctrl->status, kStInternal);
        a.iters_out[1] = kStInternal;
    }
}

void launch_newton(int prod, int grid, hipStream_t st, const DenseArgs &a, int n_sweep, int n_prod_blocks, int k_first)
{
    if (prod == 1) hipLaunchKernelGGL((dense_newton_kernel<1>), dim3(grid), dim3(256), 0, st, a, n_sweep, n_prod_blocks, k_first);
    else if (prod == 2) hipLaunchKernelGGL((dense_newton_kernel<2>), dim3(grid), dim3(256), 0, st, a, n_sweep, n_prod_blocks, k_first);
    else hipLaunchKernelGGL((dense_newton_kernel<0>), dim3(grid), dim3(256), 0, st, a, n_sweep, n_prod_blocks, k_first);
}

// workgroups of the one-launch solve: what the device holds at once
int newton_grid(int prod)
{
    static int cap[3] = {0, 0, 0};
    if (cap[prod] == 0) {
        int per_cu = 0;
        hipError_t e;
        if (prod == 1) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, dense_newton_kernel<1>, 256, 0);
        else if (prod == 2) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, dense_newton_kernel<2>, 256, 0);
        else e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, dense_newton_kernel<0>, 256, 0);
        if (e != hipSuccess || per_cu < 1) per_cu = 1;
        cap[prod] = per_cu * device_cu_count();
    }
    return cap[prod];
}

// ------------------------------------------- forward substitution, iterations as a wavefront
// The linear system of an iteration is block bi-diagonal: forward substitution solves it with one mat-vec
// W delta per timestep, 64 times fewer operations than composing the Jacobians, at the price of L sequential
// steps.  Iteration k at timestep l needs only iteration k-1 at timesteps l-1 and l, so the iterations of a
// block of kWaveIters run together, each one step behind the one before it: at step t, wave w of a sequence's
// workgroup is iteration w+1 of the block at timestep l = t - w, and a block costs L + kWaveIters - 1 steps
// whatever the number of its iterations.
//
// A step is the product z = W [delta of the four iterations], 64 x 64 x 4, on v_mfma_f32_4x4x1_16b_f32, and
//     F = tanh(y + u_l), d = 1 - F^2, delta = (F - h) + d z;   h += delta;   y_next = y + z
// for every row and iteration, with y = W h_{l-1} and h = h_l of the iterate before.  y advances by z = W delta as
// h does by delta, so W is applied to nothing but the updates and the initial guess, whose rows four more waves have ready
// group by group (guess_rows); later blocks continue from the y their predecessor left behind.
// What bounds a step is latency (LDS read, products, sum, LDS write, barrier), so it has one exchange: wave w owns
// rows 16 w .. 16 w + 15 and all of k.  The instruction's 16 blocks are four groups of four; a group covers the
// wave's 16 rows (4 columns of the B operand in each block: W) and one quarter of k, and the A operand (the four
// iterations' delta at that k) is broadcast inside the group, so 16 instructions cover k.  The four
// groups' partial sums meet by lane-row swaps that leave iteration i with lane group i: a lane is then one row of
// one iteration, and what an iteration hands to the next (h, y) moves up sixteen lanes within the wave.
// F and d are formed while the delta of the step before is on its way.  With one wave per SIMD every instruction counts (a vector instruction
// takes four cycles to issue, 1.8 ns), so the four waves touch no memory and compute no addresses: a fifth brings the
// rows of u (and, after the first block, h and y) in, sixteen bytes per lane, and takes the results out, by way of a ring of records in LDS, one
// per step, in which each iteration finds its inputs and leaves its results where the next one looks for them.
// Measured: see the rule at wavefront_plan().
constexpr int kWaveGroup = 8;         // steps per group: the mover wave brings in and takes out the rows of a group at a time
constexpr int kRing = 16;             // steps a ring in LDS holds: the group in use and the one that is ready

// tanh(y + u) of us = kTanhScale * u: one FMA into the exponential.
constexpr float kTanhScale = 2.8853900817779268f;
__device__ __forceinline__ float tanh_scaled(float y, float us)
{
    return fmaf(-2.0f, __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(fmaf(kTanhScale, y, us))), 1.0f);
}

// The first iterate and its y = W h, for every row at once, for sequences that are not cut: the initial guess
// h_l = tanh(W h0 + u_l) (App. A), written here; W h0 itself goes to a.r, one row per sequence.  Also clears the control block and the n_gm maxima.
__global__ __launch_bounds__(256) void dense_guess_kernel(const DenseArgs a, unsigned int *gm, int n_gm)
{
    if (blockIdx.x == 0) {
        if (threadIdx.x < 64) reinterpret_cast<unsigned int *>(a.ctrl)[threadIdx.x] = 0u;
        for (int i = threadIdx.x; i < n_gm; i += 256) gm[i] = 0u;
    }
    __shared__ f4v s_h[4][64];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n = lane & 15, g = lane >> 4;
    const int chn = 16 * w + 4 * g;
    const size_t rows = (size_t)a.B * a.L;
    const size_t n_items = (rows + 15) / 16;
    float wa[4][4];
    load_w_operand16(a.W, w, n, g, wa);
    const f4v zero = {0.0f, 0.0f, 0.0f, 0.0f};
    for (size_t item = blockIdx.x; item < n_items; item += gridDim.x) {
        const size_t row = item * 16 + n;
        const bool ok = row < rows;
        f4v uv = zero, c0 = zero;
        if (ok) uv = *reinterpret_cast<const f4v *>(a.u + row * DH + chn);
        if (a.h0) {
            const float *hp = a.h0 + (ok ? row / a.L : 0) * DH;
            f4v c1 = zero;
#pragma unroll
            for (int ww = 0; ww < 4; ww += 2) {
                const f4v xa = *reinterpret_cast<const f4v *>(hp + 16 * ww + 4 * g);
                const f4v xb = *reinterpret_cast<const f4v *>(hp + 16 * (ww + 1) + 4 * g);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    c0 = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[ww][v], xa[v], c0, 0, 0, 0);
                    c1 = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[ww + 1][v], xb[v], c1, 0, 0, 0);
                }
            }
            c0 = c0 + c1;
            if (ok && row % a.L == 0) *reinterpret_cast<f4v *>(a.r + (row / a.L) * DH + chn) = c0;
        }
        f4v hv;
#pragma unroll
        for (int v = 0; v < 4; ++v) hv[v] = tanh_scaled(c0[v], kTanhScale * uv[v]);
        if (ok) *reinterpret_cast<f4v *>(a.h + row * DH + chn) = hv;
        __syncthreads();                              // the previous item's reads of s_h
        s_h[w][lane] = hv;
        __syncthreads();
        f4v acc0 = zero, acc1 = zero;
#pragma unroll
        for (int ww = 0; ww < 4; ww += 2) {
            const f4v xa = s_h[ww][lane], xb = s_h[ww + 1][lane];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                acc0 = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[ww][v], xa[v], acc0, 0, 0, 0);
                acc1 = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[ww + 1][v], xb[v], acc1, 0, 0, 0);
            }
        }
        if (ok) *reinterpret_cast<f4v *>(a.d + row * DH + chn) = acc0 + acc1;
    }
}

// Waves of a workgroup: four for the chain, one that moves rows and, where the launch has them, four helpers, which make
// ahead of the chain what does not wait for it: the rows of the initial guess and their W h, or the row factors of the
// backward pass.  Without helpers that is a launch in front (dense_guess_kernel, dense_residual_kernel), which reads u and
// writes one or two more sets of rows.  us, with the launch / with helpers: forward 64 x 1024 97 / 87.5, 16 x 600 45.6 / 40.6, backward
// 64 x 1024 97 / 82, 256 x 256 83 / 70.  Forward solves that are not cut keep the launch (64 x 64 30 / 33, 256 x 256 109 / 110, both with a
// fence in every wave behind a block of iterations; with one of a workgroup the launch has 24 and 80), and so do backward passes of
// more sequences than units, where a unit's second workgroup has no room for so many waves (300 x 200 73 / 95).
constexpr int kChain = 4, kMover = 4, kHelpers = 5, kWaves = 9;
constexpr int kHelperUnits = 256;     // compute units
constexpr int wave_threads(bool help) { return (help ? kWaves : kHelpers) * kWave; }

// z of this lane's row from the exchanged vectors xv (lane 4 (4 s + m) + i, component g: row 16 s + 4 m + g of
// column i) and wr[4 m + g] = W[16 w + lane % 16][16 (lane / 16) + 4 m + g], as four partial sums over k:
// register i is column i, over the quarter lane / 16 of k.
__device__ __forceinline__ f4v wave_products(const f4v xv, const float (&wr)[16])
{
    f4v acc0 = {0.0f, 0.0f, 0.0f, 0.0f}, acc1 = acc0;
#define PARARNN_M(m)                                                                         \
    acc0 = __builtin_amdgcn_mfma_f32_4x4x1f32(xv[0], wr[4 * m + 0], acc0, 2, m, 0);          \
    acc1 = __builtin_amdgcn_mfma_f32_4x4x1f32(xv[1], wr[4 * m + 1], acc1, 2, m, 0);          \
    acc0 = __builtin_amdgcn_mfma_f32_4x4x1f32(xv[2], wr[4 * m + 2], acc0, 2, m, 0);          \
    acc1 = __builtin_amdgcn_mfma_f32_4x4x1f32(xv[3], wr[4 * m + 3], acc1, 2, m, 0);
    PARARNN_M(0) PARARNN_M(1) PARARNN_M(2) PARARNN_M(3)
#undef PARARNN_M
    return acc0 + acc1;
}

// x and y with the upper 32 lanes of x and the lower 32 of y exchanged, added up: lanes 0-31 hold x over both
// halves, lanes 32-63 y.  swap16: the same with the odd and even rows of 16 lanes.
__device__ __forceinline__ float swap32_add(float x, float y)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap16_add(float x, float y)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// the rows of one sequence, as a buffer whose bounds are the sequence's
__device__ __forceinline__ buf_rsrc seq_rsrc(const float *base, unsigned int bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(base), 0, bytes, 0x27000);
}

// Rows of one group of steps between memory and the mover wave's registers: sixteen lanes and 16 bytes each per row.
// row_of(t) is the row of the sequence that belongs to step t; rows outside it read zero and are not stored.
template <class F> __device__ __forceinline__ void rows_load(buf_rsrc r, f4v (&x)[2], int lane, int t, F row_of)
{
#pragma unroll
    for (int j = 0; j < 2; ++j)
        x[j] = __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(
                   r, (unsigned int)row_of(t + 4 * j + (lane >> 4)) * (DH * 4u) + 16u * (lane & 15), 0, 0));
}
// THROUGH: to memory, past the L2, for other workgroups of the launch.
constexpr int kThrough = 16;              // cache policy of such a buffer store: device scope
template <bool THROUGH, class F> __device__ __forceinline__ void rows_store(buf_rsrc r, const f4v (&x)[2], int lane, int t, F row_of)
{
#pragma unroll
    for (int j = 0; j < 2; ++j)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4v, x[j]), r,
                                               (unsigned int)row_of(t + 4 * j + (lane >> 4)) * (DH * 4u) + 16u * (lane & 15), 0, THROUGH ? kThrough : 0);
}
__device__ __forceinline__ void store_through(float *p, float x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void store_through(unsigned int *p, unsigned int x) { __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// The same rows in a ring of kRing records of N floats each: the row at float `at` of the records of steps t .. t + 3.
template <int N> __device__ __forceinline__ f4v *ring_slot(float (*ring)[N], int at, int lane, int t)
{
    return reinterpret_cast<f4v *>(&ring[(t + (lane >> 4)) & (kRing - 1)][at + 4 * (lane & 15)]);
}

// Stretches of a sequence.  The chain of L steps is what bounds a substitution, and most of the device has nothing to do
// meanwhile.  So a sequence is cut into n stretches that run side by side.  What enters a stretch is the update of its
// last step before, delta of every iteration, and nothing else (y and h come from it and the rows): a stretch starts
// kWarm steps early from delta = 0, and by its own first step a recurrence that contracts has forgotten that.  Whether it
// has is looked at: every stretch leaves the updates it reached at the step before its own first one, and at its last;
// where the two that belong together differ by more than kWarmTol (eight units of the last place; ten from the second iteration on) times the largest of the 64
// states at that step, at most 1, or by more than the tolerance of the solve, in any iteration and row, the stretch and all
// behind it are solved again as one chain, from the updates that the stretch before it ended with: kWarm steps
// more than one chain from the first step on.  Where they agree the states are those of one chain but for a rounding at a
// few steps.  The benchmark's W (0.8 N(0, 1/64)) agrees to 2e-7
// after 24-26 steps with u ~ N(0, 1), 52-64 with u a tenth to a third of that; 1.2 N(0, 1/64) after 50-61.
// Small states seldom agree even where all is forgotten: tanh and with it an update from the second iteration on
// has an absolute error of 6e-8.  Nor do any to a tolerance below kWarmTol: such solves have no stretches.
// (kWarm, the least length of a stretch and their number: dense_plan.h)
constexpr float kWarmTol = 4.8e-7f;
// From the second iteration on two histories that have forgotten everything still turn roundings of tanh over: up to 4.9e-7
// at 2880 borders of the benchmark's W (3.6e-7 in the first iteration, which is linear); one batch of 64 x 1024 in twenty and one of
// 16 x 600 in ten had a border above 4.8e-7, none of a hundred one above 6e-7.  What those iterations have not forgotten is
// less than in the first one, as their updates are.
constexpr float kWarmTolLater = 6e-7f;

struct DenseStretch {
    int n, len;                       // as in DensePlan
    float *edge;                      // [B][n][2][kWaveIters][64] updates at the step before the first one and at the last one
    unsigned int *top;                // [B][n][kWaveIters] max |delta|
    unsigned int *seen;               // [B][seen_words] how many iterations a sequence ran, and from word kWaveIters on max |delta| of each
    unsigned long long *count;        // [B + 1] tag + how many of a sequence's stretches have left what they leave; the last one of the sequences
    unsigned long long tag;           // of the call; the bits below kCountBits are zero
};
__host__ __device__ constexpr int seen_words(int max_iter) { return (kWaveIters + max_iter + 31) / 32 * 32; }       // whole lines

// The stretch of a sequence that is the last to end looks at its borders, in the same launch, and goes on with the sequence: nobody
// waits for another workgroup, so nothing rests on the order in which they start.  A count begins wherever the workspace stood:
// every workgroup puts the call's tag there when it starts, if nobody has (whoever of several comes second finds the word changed,
// and only this call changes it), and adds one when all it leaves is in memory.  The one that finds the others there clears the
// word for a replay of the launch, which has the same tag.
// Whatever others may read goes to memory past the L2 as it is stored: a fence in front of the count writes the L2 back, once for
// each workgroup, 1.2 us one after the other (40 us for 32 of them on each L2).
// As a launch of its own the look took 6.2 us forward and 4.5 backward.  us of a call, with that launch / in one: forward
// 64 x 1024 87.5 / 84.8, backward (with the terms of dL/dW) 82 / 70, training step 6 x 523 68.5 / 62.7.
constexpr int kCountBits = 9, kCountApart = 16;           // words: a line each (next to each other 16 x 600 took 1 us more)
static_assert(kStretches < 1 << kCountBits, "a count of all stretches");
__device__ __forceinline__ unsigned long long count_read(const DenseStretch &c, int which)
{
    return __hip_atomic_load(c.count + which * kCountApart, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void count_enters(const DenseStretch &c, int which, unsigned long long old)
{
    if (old >> kCountBits != c.tag >> kCountBits) atomicCAS(c.count + which * kCountApart, old, c.tag);
}
// One more of `all`; true for the last one, which clears the word when nothing waits for its stores.
__device__ __forceinline__ bool count_is_last(const DenseStretch &c, int which, int all)
{
    return (int)(atomicAdd(c.count + which * kCountApart, 1ull) & ((1u << kCountBits) - 1)) == all - 1;
}
__device__ __forceinline__ void count_clear(const DenseStretch &c, int which)
{
    __hip_atomic_store(c.count + which * kCountApart, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// What the unit's L1 and the L2 hold of memory that others, or other waves of the workgroup, have written is dropped: once for
// a workgroup, as every fence of a launch waits its turn (in every wave of 64 workgroups: 13 us more).
__device__ __forceinline__ void own_rows_fresh()
{
    if (threadIdx.x < kWave) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    __syncthreads();
}
// By all threads of a workgroup: true in the last stretch of sequence b to get here, which then finds what the others left.
__device__ __forceinline__ bool stretch_is_last(const DenseStretch &c, int b)
{
    __shared__ int s_last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this wave's stores; behind the barrier, every wave's
    __syncthreads();
    if (threadIdx.x == 0) s_last = count_is_last(c, b, c.n);
    __syncthreads();
    if (!s_last) return false;
    own_rows_fresh();
    if (threadIdx.x == kWave * (kWaves - 1)) count_clear(c, b);
    return true;
}

// The rows of a sequence that a block of iterations runs and leaves, and which: steps from `first` on are run, `start` to
// `end` count.
struct WaveRows {
    float *h, *y;                     // of the sequence
    int first, start, end;
};

constexpr int kWavePer = 3 * DH + 16, kWaveRec = kWaveIters * kWavePer + 2 * DH;
struct WaveLds {
    __attribute__((aligned(16))) float x[2][DH * kWaveIters];        // delta, in the order of wave_products
    __attribute__((aligned(16))) float rec[kRing][kWaveRec];
    f4v guess[DH / 4][16];                                           // rows of the initial guess, [channels 4 c ..][row % 16]
    unsigned int m[kWaveIters];
};

// W x for the 16 columns of a wave of helpers, rows 16 hw .. + 15, as sixteen products of four terms each in two sums: the
// MFMAs [from, to) of them.  One in a step of the chain, first thing behind its barrier, where the waves of the chain wait
// for LDS: in the way of the chain's own products (or, in the backward pass, of its vector instructions) they cost a step 40 ns.
struct HelperSums { f4v acc0, acc1; };
__device__ __forceinline__ void helper_products(int from, int to, const float (&wa)[4][4], const f4v (&x)[4], HelperSums &s)
{
#pragma unroll
    for (int m = 0; m < 16; ++m) {
        if (m < from || m >= to) continue;
        const int ww = (m & 1) + (m >= 8 ? 2 : 0), v = m >> 1 & 3;
        f4v &acc = m & 1 ? s.acc1 : s.acc0;
        if (m < 2) acc = f4v{0.0f, 0.0f, 0.0f, 0.0f};
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(wa[ww][v], x[ww][v], acc, 0, 0, 0);
    }
}
__device__ __forceinline__ void helper_barrier()
{
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier_keep_vmem();
    __builtin_amdgcn_sched_barrier(0);
}

// The sixteen MFMAs of two groups spread over sixteen steps less the two in which their operands are exchanged; `slot` counts
// from the first of those.
__device__ __forceinline__ void helper_products_at(int slot, const float (&wa)[4][4], const f4v (&x)[4], HelperSums &s)
{
    helper_products(slot < 10 ? slot - 2 : 2 * slot - 12, slot < 10 ? slot - 1 : 2 * slot - 10 < 16 ? 2 * slot - 10 : 16, wa, x, s);
}

// The initial guess h_l = tanh(W h0 + u_l) (App. A) and y_{l-1} = W h_{l-1} of it for the rows of a block's groups, by the
// four helping waves: wave hw has channels 16 hw .. + 15 of both, lane (n = lane % 16, g = lane / 16) channels 16 hw + 4 g ..
// + 3 of row n.  Two groups at a time, rows t - 1 .. t + 14 for those from t on, made while the two before the last one run;
// the first two in front of the chain, the next two during the first group.
__device__ __forceinline__ void guess_rows(const DenseArgs &a, int b, const WaveRows &q, WaveLds &s, int n_groups)
{
    const int lane = threadIdx.x & 63, hw = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) - kHelpers;
    const int n = lane & 15, g = lane >> 4, chn = 16 * hw + 4 * g;
    const buf_rsrc ru = seq_rsrc(a.u + (size_t)b * a.L * DH, (unsigned int)a.L * (DH * 4u));
    auto load_u = [&](int t, int i) {                      // of row t - 1 + i; outside the sequence zero
        return __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(ru, (unsigned int)(q.first + t - 1 + i) * (DH * 4u) + 4u * chn, 0, 0));
    };
    f4v uv = load_u(0, n), un = load_u(2 * kWaveGroup, n);
    float wa[4][4];
    load_w_operand16(a.W, hw, n, g, wa);
    f4v c0 = {0.0f, 0.0f, 0.0f, 0.0f}, hv = c0, x[4];      // c0: W h0
    HelperSums y;
    if (a.h0) {
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) x[ww] = *reinterpret_cast<const f4v *>(a.h0 + (size_t)b * DH + 16 * ww + 4 * g);
        hv = *reinterpret_cast<const f4v *>(a.h0 + (size_t)b * DH + chn);
        helper_products(0, 16, wa, x, y);
        c0 = y.acc0 + y.acc1;
    }
    if (q.first == 0 && n == 0) {                          // later blocks need it
#pragma unroll
        for (int v = 0; v < 4; ++v) store_through(a.r + (size_t)b * DH + chn + v, c0[v]);
    }
    auto guess = [&]() {
#pragma unroll
        for (int v = 0; v < 4; ++v) hv[v] = tanh_scaled(c0[v], kTanhScale * uv[v]);
    };
    auto fetch = [&]() {
#pragma unroll
        for (int ww = 0; ww < 4; ++ww) x[ww] = s.guess[4 * ww + g][n];
    };
    auto row_of = [&](int t) { return &s.rec[t & (kRing - 1)][chn]; };

    if (q.first + n > 0) guess();                          // else h0, in front of the sequence's first row
    s.guess[4 * hw + g][n] = hv;
    if (n > 0) *reinterpret_cast<f4v *>(row_of(n - 1)) = hv;
    helper_barrier();
    fetch();
    helper_products(0, 16, wa, x, y);
    *reinterpret_cast<f4v *>(row_of(n) + DH) = y.acc0 + y.acc1;
    helper_barrier();
    auto start = [&](int t) {                              // rows t - 1 .. t + 14; the ones after those are asked for
        uv = un;
        guess();
        s.guess[4 * hw + g][n] = hv;
        un = load_u(t + 2 * kWaveGroup, n);
        helper_barrier();
        fetch();
        helper_barrier();
    };
    f4v h_ready = hv, y_ready = c0;
    auto leave = [&](int t) {
        *reinterpret_cast<f4v *>(row_of(t - 1 + n)) = h_ready;
        *reinterpret_cast<f4v *>(row_of(t + n) + DH) = y_ready;
    };
    start(2 * kWaveGroup);
#pragma unroll
    for (int j = 0; j < kWaveGroup - 2; ++j) {
        helper_products(3 * j, 3 * j + 3, wa, x, y);
        helper_barrier();
    }
    for (int i = 1; i < n_groups; i += 2) {
        const int t = (i + 1) * kWaveGroup;                // of the two groups behind this one
        h_ready = hv;
        y_ready = y.acc0 + y.acc1;
        if (n < kWaveGroup) leave(t);
        start(t + 2 * kWaveGroup);
#pragma unroll
        for (int j = 2; j < kWaveGroup; ++j) {
            helper_products_at(j, wa, x, y);
            helper_barrier();
        }
        if (i + 1 == n_groups) break;
        if (n >= kWaveGroup) leave(t);
#pragma unroll
        for (int j = kWaveGroup; j < 2 * kWaveGroup; ++j) {
            helper_products_at(j, wa, x, y);
            helper_barrier();
        }
    }
    helper_barrier();
}

// A block of K iterations over the rows q of sequence b, by a whole workgroup; wr: W as wave_products wants it.  HELP: there
// are helpers; GUESS: they make the iterate that the block starts from, the initial guess, which is otherwise read from its rows.
// s.m[i]: max |delta| of iteration i.  KIND: kStretch leaves the updates that DenseStretch::edge holds in `edge`; kRest may find there
// what enters at the first row, the updates of the step before it (NULL: zero); kWhole starts from zero.
//
// Record of step t: for iteration i (0 ..) at timestep l = first + t - i three rows from float kWavePer i on: h_l and y_{l-1} of the
// iterate before (left there by iteration i - 1 in step t - 1, by the mover for i = 0), and kTanhScale * u_l.  The
// sixteen floats behind them put the four iterations of a wave's access into four different quarters of the banks.
// Steps before an iteration's first timestep find zeros there, which give delta = 0; the last of them, at the timestep before
// the first one, is where what enters takes its place.
enum { kWhole, kStretch, kRest };
template <int KIND, bool HELP, bool GUESS>
__device__ __forceinline__ void wavefront_block(const DenseArgs &a, int b, int K, const WaveRows &q, const float (&wr)[16], WaveLds &s,
                                                float *edge)
{
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int it = lane >> 4, r = lane & 15, row = 16 * (w & 3) + r;  // this lane: iteration `it` of the block, one row
    const int xw = 64 * (w & 3) + 16 * (r >> 2) + 4 * it + (r & 3);  // where this lane's delta goes
    const int L = q.end - q.first, lead = q.start - q.first;         // steps, of which the first do not count
    const int n_groups = (L + K - 1 + kWaveGroup - 1) / kWaveGroup;
    constexpr bool EDGE = KIND == kStretch;
    const bool enters = KIND == kRest && edge;
    if (w < kChain) s.x[0][xw] = enters && it == 0 ? edge[row] : 0.0f;
    if (threadIdx.x < kWaveIters) s.m[threadIdx.x] = 0u;
    if (HELP && w >= kHelpers) {
        if constexpr (GUESS) guess_rows(a, b, q, s, n_groups);
        else
            for (int i = 0; i < kWaveGroup * n_groups + 2; ++i) lds_barrier();
    } else if (w == kMover) {
        const unsigned int seq_bytes = (unsigned int)a.L * (DH * 4u);
        const buf_rsrc ru = seq_rsrc(a.u + (size_t)b * a.L * DH, seq_bytes), rh = seq_rsrc(q.h, seq_bytes), ry = seq_rsrc(q.y, seq_bytes);
        // results: the rows that count, y those before them
        const int y0 = q.start > 0 ? q.start - 1 : 0;
        const buf_rsrc oh = seq_rsrc(q.h + (size_t)q.start * DH, (unsigned int)(q.end - q.start) * (DH * 4u)),
                       oy = seq_rsrc(q.y + (size_t)y0 * DH, (unsigned int)(q.end - 1 - y0) * (DH * 4u));
        f4v xh[2], xy[2], xu[2];
        auto same = [&](int t) { return q.first + t; };
        auto before = [&](int t) { return q.first + t - 1; };
        auto bring = [&](int t) {
            if constexpr (!GUESS) {
                rows_load(rh, xh, lane, t, same);
                rows_load(ry, xy, lane, t, before);
            }
            rows_load(ru, xu, lane, t, same);
        };
        auto put = [&](int t) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if constexpr (!GUESS) {
                    *ring_slot(s.rec, 0, lane, t + 4 * j) = xh[j];
                    *ring_slot(s.rec, DH, lane, t + 4 * j) = xy[j];
                }
#pragma unroll
                for (int i = 0; i < kWaveIters; ++i) *ring_slot(s.rec, kWavePer * i + 2 * DH, lane, t + 4 * j + i) = xu[j] * kTanhScale;
            }
        };
        auto take = [&](int t) {                           // what iteration K - 1 left in the records t .. t + 7
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                xh[j] = *ring_slot(s.rec, kWavePer * K, lane, t + 4 * j);
                xy[j] = *ring_slot(s.rec, kWavePer * K + DH, lane, t + 4 * j);
            }
            rows_store<EDGE>(oh, xh, lane, t - K, [&](int l) { return l - lead; });
            rows_store<EDGE>(oy, xy, lane, t - K, [&](int l) { return q.first + l - 1 - y0; });
        };
#pragma unroll
        for (int i = 1; i < kWaveIters; ++i)
            for (int t = 0; t < i; ++t) s.rec[t][kWavePer * i + 2 * DH + lane] = 0.0f;
        bring(0);
        put(0);
        // y in front of the sequence's first row: W h0, the same for every iteration
        if (!GUESS && q.first == 0) s.rec[0][DH + lane] = a.h0 ? a.r[(size_t)b * DH + lane] : 0.0f;
        if constexpr (GUESS) lds_barrier();
        lds_barrier();
        for (int g = 0; g < n_groups; ++g) {
            const int t0 = g * kWaveGroup;
            lds_barrier();
            // a load is waited for behind the stores in front of it: those of rows that go to memory come after
            if constexpr (GUESS) bring(t0 + kWaveGroup);
            if (g > 0) take(t0 - kWaveGroup + 1);          // records t0 - 7 .. t0: complete with the first step of this group
            if constexpr (!GUESS) bring(t0 + kWaveGroup);
#pragma unroll 1
            for (int i = 1; i < kWaveGroup - 2; ++i) lds_barrier();
            put(t0 + kWaveGroup);                          // the group's last step reads the first of these records
            lds_barrier();
            lds_barrier();
        }
        lds_barrier();
        take((n_groups - 1) * kWaveGroup + 1);
    } else {
        float mymax = 0.0f, h_in, y_in, us;
        float *my_edge = EDGE ? edge + it * DH + row : nullptr;
        const float first_delta = enters ? edge[it * DH + row] : 0.0f;
        // what this lane's iteration leaves for the next one in record `rec`, and what it finds there itself
        auto hand_on = [&](float *record, float hn, float yn) {
            float *rec = record + kWavePer * it + row;
            rec[kWavePer] = hn;
            rec[kWavePer + DH] = yn;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the reader is in this wave
            __builtin_amdgcn_wave_barrier();
            h_in = rec[0];
            y_in = rec[DH];
            us = rec[2 * DH];
        };
        // kind 0: all timesteps count; 1: some do not, or it is one whose update is handed out; 2: none counts; 3: those before the
        // first one do not, and what enters is taken over
        auto step = [&](auto kind, int kB, float *next_rec, int t) {
            constexpr int kKind = decltype(kind)::value;
            const f4v xv = *reinterpret_cast<const f4v *>(&s.x[kB][4 * lane]);
            __builtin_amdgcn_sched_barrier(0);
            const float F = tanh_scaled(y_in, us), d = fmaf(-F, F, 1.0f), res = F - h_in;
            __builtin_amdgcn_sched_barrier(0);
            const f4v p = wave_products(xv, wr);
            const float z = swap16_add(swap32_add(p[0], p[2]), swap32_add(p[1], p[3]));
            float delta = fmaf(d, z, res);
            if constexpr (kKind == 3) {
                if (t - it == -1) delta = first_delta;
            }
            s.x[kB ^ 1][xw] = delta;
            __builtin_amdgcn_sched_barrier(0);
            hand_on(next_rec, fmaf(d, z, F), y_in + z);
            if constexpr (kKind == 1 || kKind == 3) {      // past the end too; a NaN has reached the last one
                const int l = t - it;
                if (l >= lead && l < L) mymax = nanmax(mymax, fabsf(delta));
                if constexpr (EDGE) {
                    if (l == lead - 1) store_through(my_edge, delta);
                    if (l == L - 1) store_through(my_edge + kWaveIters * DH, delta);
                }
            } else if constexpr (kKind == 0) {
                mymax = fmaxf(mymax, fabsf(delta));
            }
            // delta is written; the (at least three) LDS instructions of hand_on may be on their way still
            asm volatile("s_waitcnt lgkmcnt(3)\n\ts_barrier" ::: "memory");
        };
        if constexpr (GUESS) lds_barrier();
        lds_barrier();
        __builtin_amdgcn_s_setprio(3);
        hand_on(s.rec[0], 0.0f, 0.0f);
        int g = 0;
        if (enters) {
#pragma unroll
            for (int i = 0; i < kWaveGroup; ++i) step(std::integral_constant<int, 3>{}, i & 1, s.rec[i + 1], i);
            g = 1;
        }
        for (; g < n_groups; ++g) {
            const int t0 = g * kWaveGroup;
            float *rec = s.rec[t0 & (kRing - 1)], *rec_next = s.rec[(t0 + kWaveGroup) & (kRing - 1)];
            auto group = [&](auto kind) {
#pragma unroll
                for (int i = 0; i < kWaveGroup; ++i) step(kind, i & 1, i + 1 < kWaveGroup ? rec + kWaveRec * (i + 1) : rec_next, t0 + i);
            };
            if (t0 + kWaveGroup < L && (lead == 0 || t0 >= lead + kWaveIters - 1)) {
                group(std::integral_constant<int, 0>{});
            } else {
                if constexpr (EDGE) {
                    if (t0 + kWaveGroup < lead && t0 + kWaveGroup < L) { group(std::integral_constant<int, 2>{}); continue; }
                }
                group(std::integral_constant<int, 1>{});
            }
        }
        __builtin_amdgcn_s_setprio(0);
        lds_barrier();
        if (it < K) atomicMax(&s.m[it], __float_as_uint(mymax) & 0x7fffffffu);
    }
}

// W of this lane as wave_products wants it
__device__ __forceinline__ void load_w_wave(const float *W, float (&wr)[16])
{
    const int lane = threadIdx.x & 63, row = 16 * ((int)(threadIdx.x >> 6) & 3) + (lane & 15);
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        const f4v t = *reinterpret_cast<const f4v *>(W + row * DH + 16 * (lane >> 4) + 4 * m);
#pragma unroll
        for (int v = 0; v < 4; ++v) wr[4 * m + v] = t[v];
    }
}

// By one wave of the workgroup that is through with a sequence: the last of them reports the first iteration whose maximum over the
// sequences that ran it met the tolerance.  A lane has two sequences at most, and a block of their iterations at a time.
__device__ __forceinline__ void stretches_report(const DenseArgs &a, const DenseStretch &c)
{
    static_assert(kStretches / 2 <= 2 * kWave, "at least two stretches of a sequence");
    const int lane = threadIdx.x & 63;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // this sequence's words, which are this wave's
    int last = 0;
    if (lane == 0) last = count_is_last(c, a.B, a.B);
    if (!__builtin_amdgcn_readfirstlane(last)) return;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    int status = a.tol < 0.0f ? kStOk : kStNotConverged, k = 0;
    for (bool ended = false; k < a.max_iter && !ended;) {
        u4v top = {0u, 0u, 0u, 0u};
        for (int b = lane; b < a.B; b += kWave) {
            const unsigned int *row = c.seen + (size_t)b * seen_words(a.max_iter);
            const u4v m = *reinterpret_cast<const u4v *>(row + kWaveIters + k);
            const int ran = (int)row[0] - k;
#pragma unroll
            for (int i = 0; i < kWaveIters; ++i) top[i] = max(top[i], i < ran ? m[i] : 0u);
        }
#pragma unroll
        for (int i = 0; i < kWaveIters; ++i) {
            if (k == a.max_iter || ended) continue;
            const float mk = __uint_as_float(wave_max_u32(top[i]));
            if (a.trace && lane == 0) a.trace[k] = mk;
            ++k;
            if (!(mk - mk == 0.0f)) { status = kStNonFinite; ended = true; }
            else if (a.tol >= 0.0f && mk <= a.tol) { status = kStOk; ended = true; }
        }
    }
    if (lane == 0) {
        a.iters_out[0] = k;
        a.iters_out[1] = status;
        count_clear(c, a.B);
    }
}

// The solve of sequence b by a workgroup.  A sequence whose own update meets the tolerance at the end of a block is done:
// the blocks after it are run by the sequences that are not.  gm[k-1]: max |delta| of iteration k over the
// sequences that ran it.  The last workgroup to finish reports the first iteration whose maximum met the tolerance.
// CUT: there were stretches, and the maxima are in `seen`; it goes on behind the first block, or solves that again from the first border on where the
// updates differ.
template <bool CUT>
__device__ __forceinline__ void wavefront_sequence(const DenseArgs &a, unsigned int *gm, const DenseStretch &c, int b, WaveLds &s)
{
    __shared__ int s_held;
    const size_t seq = (size_t)b * a.L * DH;
    auto ended = [&](int K) {                              // the maxima in s.m are of a whole block
        bool met = false;
        for (int i = 0; i < K; ++i) {
            const float mk = __uint_as_float(s.m[i]);
            met = met || !(mk - mk == 0.0f) || (i == K - 1 && a.tol >= 0.0f && mk <= a.tol);
        }
        return met;
    };
    constexpr int kThreads = wave_threads(CUT), kTops = (kStretches * kWaveIters + kThreads - 1) / kThreads;
    unsigned int top[kTops];                               // of stretch (threadIdx.x + kThreads j) / kWaveIters
    int held = 0;                                          // stretches that are as they have to be
    if constexpr (CUT) {
        if (threadIdx.x == 0) s_held = c.n;
        if (threadIdx.x < kWaveIters) s.m[threadIdx.x] = 0u;
#pragma unroll
        for (int j = 0; j < kTops; ++j) {
            const int i = (int)threadIdx.x + kThreads * j;
            top[j] = i < c.n * kWaveIters ? c.top[(size_t)b * c.n * kWaveIters + i] : 0u;
        }
        lds_barrier();                                     // the loads stay on their way
        // A wave looks at the updates between two stretches, a quad a lane: the ones at the last step of stretch e, the ones that e + 1
        // started from, and the states that both belong to.
        constexpr int kQuads = kWaveIters * DH / 4, kBatch = 4;
        static_assert(kQuads == 64, "a quad per lane");
        const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
        const f4v *edge = reinterpret_cast<const f4v *>(c.edge) + (size_t)b * c.n * 2 * kQuads;
        const f4v *state = reinterpret_cast<const f4v *>(a.h + seq);
        const int K = min(kWaveIters, a.max_iter);
        for (int e0 = w; e0 < c.n - 1; e0 += kBatch * kWaves) {
            f4v there[kBatch], here[kBatch], hq[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                const int e = min(e0 + kWaves * j, c.n - 2);
                const f4v *at = edge + (size_t)e * 2 * kQuads + lane;
                there[j] = at[kQuads];
                here[j] = at[2 * kQuads];
                hq[j] = state[(size_t)((e + 1) * c.len - 1) * (DH / 4) + (lane & 15)];
            }
#pragma unroll
            for (int j = 0; j < kBatch; ++j) {
                unsigned int large = 0u;
#pragma unroll
                for (int v = 0; v < 4; ++v) large = max(large, __float_as_uint(hq[j][v]) & 0x7fffffffu);
                float bound = (lane < DH / 4 ? kWarmTol : kWarmTolLater) * fminf(__uint_as_float(wave_max_u32(large)), 1.0f);
                if (a.tol >= 0.0f) bound = fminf(bound, a.tol);
                if (lane >= K * (DH / 4)) continue;
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (!(fabsf(there[j][v] - here[j][v]) <= bound)) atomicMin(&s_held, min(e0 + kWaves * j, c.n - 2) + 1);
            }
        }
        __syncthreads();
        held = __builtin_amdgcn_readfirstlane(s_held);     // the same for the whole workgroup: buffers chosen by it are scalars
    }
    unsigned int *seen = CUT ? c.seen + (size_t)b * seen_words(a.max_iter) : nullptr;
    float wr[16];
    if (!CUT || held < c.n) load_w_wave(a.W, wr);
    for (int k0 = 0; k0 < a.max_iter; k0 += kWaveIters) {
        const int K = min(kWaveIters, a.max_iter - k0);
        if (!CUT || k0 > 0 || held < c.n) {
            const bool rest = CUT && k0 == 0;              // of the first block
            const int first = rest ? held * c.len : 0;
            const WaveRows q = {a.h + seq, a.d + seq, first, first, a.L};
            if (CUT && k0 == kWaveIters && held == c.n) load_w_wave(a.W, wr);
            float *enters = rest ? c.edge + ((size_t)(b * c.n + held - 1) * 2 + 1) * kWaveIters * DH : nullptr;
            if (CUT && k0 == 0) wavefront_block<kRest, CUT, CUT>(a, b, K, q, wr, s, enters);
            else wavefront_block<kWhole, CUT, false>(a, b, K, q, wr, s, nullptr);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the next block reads the rows that this one wrote
            __syncthreads();
            own_rows_fresh();
        }
        if (CUT && k0 == 0) {
#pragma unroll
            for (int j = 0; j < kTops; ++j) {
                const int i = (int)threadIdx.x + kThreads * j;
                if (i < held * kWaveIters) atomicMax(&s.m[i & (kWaveIters - 1)], top[j]);
            }
            __syncthreads();
        }
        const bool met = ended(K);
        if ((int)threadIdx.x < K) {
            if constexpr (CUT) store_through(seen + kWaveIters + k0 + threadIdx.x, s.m[threadIdx.x]);
            else atomicMax(&gm[k0 + threadIdx.x], s.m[threadIdx.x]);
        }
        if (CUT && threadIdx.x == 0) store_through(seen, (unsigned int)(k0 + K));
        __syncthreads();
        if (met) break;
    }
    if constexpr (CUT) {
        if (threadIdx.x < kWave) stretches_report(a, c);
    } else if (threadIdx.x == 0) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the maxima, which are this wave's
        if (atomicAdd(&a.ctrl->done, 1u) == (unsigned int)a.B - 1) {
            int status = a.tol < 0.0f ? kStOk : kStNotConverged, k = 1;
            for (; k <= a.max_iter; ++k) {
                const float mk = __uint_as_float(__hip_atomic_load(&gm[k - 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
                if (a.trace) a.trace[k - 1] = mk;
                if (!(mk - mk == 0.0f)) { status = kStNonFinite; break; }
                if (a.tol >= 0.0f && mk <= a.tol) { status = kStOk; break; }
            }
            a.iters_out[0] = min(k, a.max_iter);
            a.iters_out[1] = status;
        }
    }
}

// One workgroup per sequence, which is not cut.
__global__ __launch_bounds__(wave_threads(false)) void dense_wavefront_kernel(const DenseArgs a, unsigned int *gm)
{
    __shared__ WaveLds s;
    const DenseStretch c = {};
    wavefront_sequence<false>(a, gm, c, (int)blockIdx.x, s);
}

// One workgroup per stretch of a sequence for the first block of iterations; the last one of a sequence to end goes on with it.
__global__ __launch_bounds__(wave_threads(true)) void dense_stretch_kernel(const DenseArgs a, const DenseStretch c)
{
    __shared__ WaveLds s;
    const int b = (int)blockIdx.x / c.n, j = (int)blockIdx.x - b * c.n, K = min(kWaveIters, a.max_iter);
    const size_t seq = (size_t)b * a.L * DH;
    {
        // the count of the sequences by one workgroup of each: all of them at one word took 2 us of 64 x 1024
        const bool counts = threadIdx.x < (j == 0 ? 2 : 1);
        const int which = threadIdx.x == 0 ? b : a.B;
        unsigned long long old = 0;
        if (counts) old = count_read(c, which);
        float wr[16];
        load_w_wave(a.W, wr);
        __builtin_amdgcn_sched_barrier(0);                 // all of it on its way before anything is waited for
        if (counts) count_enters(c, which, old);
        const int start = j * c.len;
        const WaveRows q = {a.h + seq, a.d + seq, max(start - kWarm, 0), start, min(start + c.len, a.L)};
        wavefront_block<kStretch, true, true>(a, b, K, q, wr, s, c.edge + (size_t)blockIdx.x * 2 * kWaveIters * DH);
    }
    __syncthreads();
    if (threadIdx.x < kWaveIters) store_through(c.top + (size_t)blockIdx.x * kWaveIters + threadIdx.x, s.m[threadIdx.x]);
    if (stretch_is_last(c, b)) wavefront_sequence<true>(a, nullptr, c, b, s);
}

// Backward by substitution: mu_l = d_l (W^T mu_{l+1} + g_l), one workgroup per sequence.  The row factors
// d_l = 1 - tanh^2(W h_{l-1} + u_l) at the given states are the helpers' work (HELP) or in a.d.
// A single column leaves the matrix instruction's other three idle, and sixteen vector FMAs per lane (68 cycles)
// are quicker than sixteen of it (150): wave w owns rows 16 w .. + 15, lane group q the terms 16 q .. + 15 of their
// sums, which two lane-row swaps complete.  mu reaches the FMAs one value per lane, broadcast inside the lane row by
// the instruction itself (as 16-byte reads of all terms it cost 16 LDS transactions of 1 KB per step: 164 ns a step).  A fifth wave moves rows as in the forward kernel.  Ends with
// dL/dh0 = W^T mu_1.
//
// STRETCH: one workgroup per stretch of a sequence (DenseStretch: here from the last row down; what enters is one mu), which
// starts kWarm rows early from mu = 0 and leaves mu at the row behind its own last one in `edge`.  Otherwise a whole sequence, or
// what is run again behind the last border at which its stretches differ: rows 0 .. end - 1, with `x` entering.
//
// The helpers of a stretch leave the row factors in a.d, for a sequence that is run again.  GRADIENT: then they add up the terms of
// dL/dW of these rows instead, a group of steps behind the chain, each those of sixteen rows of the matrix, four rows of mu and h at
// a time on v_mfma_f32_16x16x4_f32, in sums of sixteen rows and a sum of those; `dw`: the matrix, and n_dw - 1 more behind it that the
// mover clears.  us of a pass whose sequences are run again, with row factors made anew and the terms added up behind the chain /
// so: 6 x 523 117 / 102, 16 x 600 137 / 120, 64 x 1024 218 / 197.
struct AdjointLds {
    // step t of the recurrence is row last - t; its record holds d and d g, and mu is in the slot of the same number
    __attribute__((aligned(16))) float rec[kRing][2 * DH], mu[kRing][DH];
};
template <bool STRETCH, bool HELP, bool GRADIENT = false>
__device__ __forceinline__ void adjoint_chain(const DenseArgs &a, float *dh0, int b, int start, int end, float x, float *edge, AdjointLds &lds,
                                              float *dw = nullptr, int n_dw = 0)
{
    static_assert(!GRADIENT || !HELP, "the helpers' work instead");
    auto &s_rec = lds.rec;
    auto &s_mu = lds.mu;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int q = lane >> 4, row = 16 * (w & 3) + (lane & 15);
    const unsigned int seq_bytes = (unsigned int)a.L * (DH * 4u);
    const int last = STRETCH ? min(end + kWarm, a.L) - 1 : end - 1, L = last + 1 - start, lead = last + 1 - end;
    auto rev = [last](int t) { return last - t; };
    float wr[16];                                          // W^T[row][16 q ..]
#pragma unroll
    for (int i = 0; i < 16; ++i) wr[i] = a.W[(16 * q + i) * DH + row];
    const int n_groups = (L + kWaveGroup - 1) / kWaveGroup;
    if (HELP && w >= kHelpers) {
        // lane (n = lane % 16, g = lane / 16) has channels 16 hw + 4 g .. + 3 of step n of two groups
        const int hw = w - kHelpers, n = lane & 15, g = lane >> 4, chn = 16 * hw + 4 * g;
        const buf_rsrc ru = seq_rsrc(a.u + (size_t)b * a.L * DH, seq_bytes), rh = seq_rsrc(a.h + (size_t)b * a.L * DH, seq_bytes),
                       rg = seq_rsrc(a.g + (size_t)b * a.L * DH, seq_bytes);
        float wa[4][4];
        load_w_operand16(a.W, hw, n, g, wa);
        auto load = [](buf_rsrc r, int row, int channel) {      // rows outside the sequence read zero
            return __builtin_bit_cast(f4v, __builtin_amdgcn_raw_buffer_load_b128(r, (unsigned int)row * (DH * 4u) + 4u * channel, 0, 0));
        };
        f4v xh[4], xu, xg, nh[4], nu, ng;                  // of the steps that are worked on, and of those after them
        HelperSums y;
        auto bring = [&](int t) {
            const int l = rev(t);
            nu = load(ru, l, chn);
            ng = load(rg, l, chn);
#pragma unroll
            for (int ww = 0; ww < 4; ++ww) nh[ww] = load(rh, l - 1, 16 * ww + 4 * g);
            if (l == 0 && a.h0) {
#pragma unroll
                for (int ww = 0; ww < 4; ++ww) nh[ww] = *reinterpret_cast<const f4v *>(a.h0 + (size_t)b * DH + 16 * ww + 4 * g);
            }
        };
        auto next = [&]() {
            xu = nu; xg = ng;
#pragma unroll
            for (int ww = 0; ww < 4; ++ww) xh[ww] = nh[ww];
        };
        f4v d, dg;
        auto finish = [&]() {
            const f4v p = y.acc0 + y.acc1 + xu;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float F = fast_tanh(p[v]);
                d[v] = fmaf(-F, F, 1.0f);
            }
            dg = d * xg;
        };
        // own rows: those behind them are another stretch's, steps past the last one come out in front
        const buf_rsrc rd = seq_rsrc(a.d + ((size_t)b * a.L + start) * DH, (unsigned int)(end - start) * (DH * 4u));
        auto put = [&](int t) {                            // the last readers of these records are done
            float *rec = s_rec[t & (kRing - 1)];
            *reinterpret_cast<f4v *>(rec + chn) = d;
            *reinterpret_cast<f4v *>(rec + DH + chn) = dg;
            if constexpr (STRETCH)
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4v, d), rd, (unsigned int)(rev(t) - start) * (DH * 4u) + 4u * chn, 0, kThrough);
        };
        // as guess_rows: two groups of steps at a time
        bring(n);
        next();
        bring(2 * kWaveGroup + n);
        helper_products(0, 16, wa, xh, y);
        finish();
        put(n);
        helper_barrier();
        next();
        bring(4 * kWaveGroup + n);
#pragma unroll
        for (int j = 0; j < kWaveGroup; ++j) {
            helper_products(2 * j, 2 * j + 2, wa, xh, y);
            helper_barrier();
        }
        for (int i = 1; i < n_groups; i += 2) {
            const int t = (i + 1) * kWaveGroup;            // of the two groups behind this one
            finish();
            if (n < kWaveGroup) put(t + n);
            next();
            helper_barrier();
            bring(t + 4 * kWaveGroup + n);
            helper_barrier();
#pragma unroll
            for (int j = 2; j < kWaveGroup; ++j) {
                helper_products_at(j, wa, xh, y);
                helper_barrier();
            }
            if (i + 1 == n_groups) break;
            if (n >= kWaveGroup) put(t + n);
#pragma unroll
            for (int j = kWaveGroup; j < 2 * kWaveGroup; ++j) {
                helper_products_at(j, wa, xh, y);
                helper_barrier();
            }
        }
        return;
    }
    if (GRADIENT && w >= kHelpers) {
        // Terms of dL/dW of group k: lane (n, g) has step 8 k + 4 i + g, channel 16 hw + n of mu and 16 j + n of h, in register 4 i + j.
        const int hw = w - kHelpers, n = lane & 15, g = lane >> 4;
        const buf_rsrc rh = seq_rsrc(a.h + (size_t)b * a.L * DH, seq_bytes);
        float mu[2], h[8], h_next[8];
        const f4v zero = {0.0f, 0.0f, 0.0f, 0.0f};
        f4v acc[8] = {zero, zero, zero, zero, zero, zero, zero, zero}, sum[4] = {zero, zero, zero, zero}, lost[4] = {zero, zero, zero, zero};
        auto bring = [&](int k) {                          // rows outside the sequence read zero
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int l = rev(k * kWaveGroup + 4 * i + g);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    h_next[4 * i + j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rh, (unsigned int)(l - 1) * (DH * 4u) + 4u * (16 * j + n), 0, 0));
                if (l == 0 && a.h0) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) h_next[4 * i + j] = a.h0[(size_t)b * DH + 16 * j + n];
                }
            }
        };
        auto take = [&](int k) {                           // mu of the group is complete; steps past the last one have none
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int t = k * kWaveGroup + 4 * i + g;
                mu[i] = t < L ? s_mu[t & (kRing - 1)][16 * hw + n] : 0.0f;
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) h[i] = h_next[i];
        };
        auto multiply = [&](int i) { acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(mu[i >> 2], h[i], acc[i], 0, 0, 0); };
        auto add = [&](int j) {                            // compensated: plain, the sums of 512 rows had a tenth more error than a tree of them
            const f4v y = acc[j] + acc[j + 4] - lost[j], s = sum[j] + y;
            lost[j] = (s - sum[j]) - y;
            sum[j] = s;
            acc[j] = acc[j + 4] = zero;
        };
        bring(0);
        helper_barrier();
        for (int k = 0; k < n_groups; ++k) {               // the terms of a group while the next one runs
#pragma unroll
            for (int j = 0; j < kWaveGroup; ++j) {
                if (k > 0) {
                    if (j == 0) { take(k - 1); bring(k); }
                    if (j < 4 && (k & 3) == 1) add(j);     // of 32 rows
                    multiply(j);
                }
                helper_barrier();
            }
        }
        take(n_groups - 1);
#pragma unroll
        for (int j = 0; j < 8; ++j) multiply(j);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            add(j);
#pragma unroll
            for (int v = 0; v < 4; ++v) dw[(16 * hw + 4 * g + v) * DH + 16 * j + n] = sum[j][v];
        }
        return;
    }
    if (w == kMover) {
        const buf_rsrc rd = seq_rsrc(a.d + (size_t)b * a.L * DH, seq_bytes), rg = seq_rsrc(a.g + (size_t)b * a.L * DH, seq_bytes),
                       ro = seq_rsrc(a.du + (size_t)b * a.L * DH, (unsigned int)end * (DH * 4u));   // rows behind the own ones are not stored
        f4v xd[2], xg[2], xm[2];
        auto bring = [&](int t) {
            if constexpr (!HELP) { rows_load(rd, xd, lane, t, rev); rows_load(rg, xg, lane, t, rev); }
        };
        auto put = [&](int t) {
            if constexpr (!HELP) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    *ring_slot(s_rec, 0, lane, t + 4 * j) = xd[j];
                    *ring_slot(s_rec, DH, lane, t + 4 * j) = xd[j] * xg[j];
                }
            }
        };
        auto take = [&](int t) {
#pragma unroll
            for (int j = 0; j < 2; ++j) xm[j] = *ring_slot(s_mu, 0, lane, t + 4 * j);
            rows_store<STRETCH>(ro, xm, lane, t, [&](int k) { return k < L ? last - k : -1; });
        };
        int k = DH * DH / 4 + lane;                        // quads to be cleared: up to four a lane and group, of 32 rows or more a matrix
        auto clear = [&]() {
            for (int i = 0; i < 4 && k < n_dw * (DH * DH / 4); ++i, k += kWave) reinterpret_cast<f4v *>(dw)[k] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
        };
        bring(0);
        put(0);
        lds_barrier();
        for (int g = 0; g < n_groups; ++g) {
            const int t0 = g * kWaveGroup;
            bring(t0 + kWaveGroup);
            if (g > 0) take(t0 - kWaveGroup);
            if constexpr (GRADIENT) clear();
#pragma unroll 1
            for (int i = 0; i < kWaveGroup - 2; ++i) lds_barrier();
            put(t0 + kWaveGroup);                          // the group's last step reads the first of these records
            lds_barrier();
            lds_barrier();
        }
        take((n_groups - 1) * kWaveGroup);
        return;
    }
    // W^T mu, this lane's row, of the wave's lanes holding mu: lane 16 q + i the term 16 q + i
    auto sum = [&](float x) {
        float s[4];
        // as one statement: the compiler makes a move and an FMA of each.  The wait states are those of a DPP source
        // that a vector instruction may just have written.
        asm("s_nop 1\n\t"
            "v_mul_f32_dpp %0, %4, %5 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
            "v_mul_f32_dpp %1, %4, %6 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
            "v_mul_f32_dpp %2, %4, %7 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
            "v_mul_f32_dpp %3, %4, %8 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %0, %4, %9 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %1, %4, %10 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %2, %4, %11 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %3, %4, %12 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %0, %4, %13 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %1, %4, %14 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %2, %4, %15 row_newbcast:10 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %3, %4, %16 row_newbcast:11 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %0, %4, %17 row_newbcast:12 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %1, %4, %18 row_newbcast:13 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %2, %4, %19 row_newbcast:14 row_mask:0xf bank_mask:0xf\n\t"
            "v_fmac_f32_dpp %3, %4, %20 row_newbcast:15 row_mask:0xf bank_mask:0xf"
            : "=&v"(s[0]), "=&v"(s[1]), "=&v"(s[2]), "=&v"(s[3])
            : "v"(x), "v"(wr[0]), "v"(wr[1]), "v"(wr[2]), "v"(wr[3]), "v"(wr[4]), "v"(wr[5]), "v"(wr[6]), "v"(wr[7]),
              "v"(wr[8]), "v"(wr[9]), "v"(wr[10]), "v"(wr[11]), "v"(wr[12]), "v"(wr[13]), "v"(wr[14]), "v"(wr[15]));
        const float p = (s[0] + s[1]) + (s[2] + s[3]);
        const float t = swap32_add(p, p);
        return swap16_add(t, t);
    };
    lds_barrier();
    __builtin_amdgcn_s_setprio(3);
    float d = s_rec[0][row], dg = s_rec[0][DH + row];
    for (int g = 0; g < n_groups; ++g) {
        const int s0 = (g * kWaveGroup) & (kRing - 1), s1 = (s0 + kWaveGroup) & (kRing - 1);
        float *mus = s_mu[s0];
        const float *rec = s_rec[s0], *rec_next = s_rec[s1];
#pragma unroll
        for (int i = 0; i < kWaveGroup; ++i) {
            const float mu = fmaf(d, sum(x), dg);
            mus[i * DH + row] = mu;                        // the four lane groups store the same value
            if constexpr (STRETCH) {
                if (g * kWaveGroup + i == lead - 1 && q == 0) store_through(edge + row, mu);
            }
            __builtin_amdgcn_sched_barrier(0);
            const float *nr = i + 1 < kWaveGroup ? rec + 2 * (i + 1) * DH : rec_next;
            d = nr[row];
            dg = nr[DH + row];
            // mu is written; the read of the next factors may be on its way still
            asm volatile("s_waitcnt lgkmcnt(1)\n\ts_barrier" ::: "memory");
            x = mus[i * DH + lane];
        }
    }
    if (dh0 && start == 0) {
        const float s = sum(s_mu[(L - 1) & (kRing - 1)][lane]);
        if (q == 0) store_through(dh0 + (size_t)b * DH + row, s);
    }
}

// The terms that rows first .. end - 1 of sequence b add to dL/dW = sum mu_l h_{l-1}^T, a matrix.  By eight waves: each has a quarter of
// it and every other batch of 32 rows, two at a time on v_mfma_f32_32x32x2_f32; the rows of a batch travel while the one before
// is multiplied.  In the launch of the stretches, where mu is at hand; as one of its own it took 6.6 us of a step of 6 x 523.
__device__ __forceinline__ void stretch_weight_gradient(const DenseArgs &a, int b, int first, int end, float (&s_half)[4][16][kWave], float *out)
{
    constexpr int kPairs = 16, kSums = 4;                  // sums of a wave: in one, 128 rows of 256 added up one by one, 1.5 to 2 times the error
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n = lane & 31, half = lane >> 5, mt = w & 1, nt = w >> 1 & 1, part = w >> 2;
    // rows past the end, and the one in front of the sequence, read zero
    const buf_rsrc rm = seq_rsrc(a.du + (size_t)b * a.L * DH, (unsigned int)end * (DH * 4u)),
                   rh = seq_rsrc(a.h + (size_t)b * a.L * DH, (unsigned int)(end - 1) * (DH * 4u));
    float m[kPairs], h[kPairs], mn[kPairs], hn[kPairs];
    auto bring = [&](int r) {
#pragma unroll
        for (int i = 0; i < kPairs; ++i) {
            const unsigned int at = (unsigned int)(r + 2 * i + half) * (DH * 4u) + 4u * n;
            mn[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rm, at + 128u * mt, 0, 0));
            hn[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rh, at - DH * 4u + 128u * nt, 0, 0));
        }
        if (r == 0 && half == 0 && a.h0) hn[0] = a.h0[(size_t)b * DH + 32 * nt + n];
    };
    f16v Qs[kSums], Q;
    if (w < 8) {
        int r = first + 2 * kPairs * part;
        bring(r);
#pragma unroll
        for (int k = 0; k < kSums; ++k)
#pragma unroll
            for (int v = 0; v < 16; ++v) Qs[k][v] = 0.0f;
        for (; r < end; r += 4 * kPairs) {
#pragma unroll
            for (int i = 0; i < kPairs; ++i) { m[i] = mn[i]; h[i] = hn[i]; }
            bring(r + 4 * kPairs);
#pragma unroll
            for (int i = 0; i < kPairs; ++i) Qs[i % kSums] = __builtin_amdgcn_mfma_f32_32x32x2f32(m[i], h[i], Qs[i % kSums], 0, 0, 0);
        }
        Q = (Qs[0] + Qs[1]) + (Qs[2] + Qs[3]);
        if (part == 1) {
#pragma unroll
            for (int v = 0; v < 16; ++v) s_half[w & 3][v][lane] = Q[v];
        }
    }
    lds_barrier();
    if (w < 4) {
#pragma unroll
        for (int v = 0; v < 16; ++v) store_through(out + (32 * mt + mfma_row(v, half)) * DH + 32 * nt + n, Q[v] + s_half[w][v][lane]);
    }
}

// One workgroup per sequence, which is not cut.
template <bool HELP>
__global__ __launch_bounds__(wave_threads(HELP)) void dense_adjoint_kernel(const DenseArgs a, float *dh0)
{
    __shared__ AdjointLds s;
    adjoint_chain<false, HELP>(a, dh0, (int)blockIdx.x, 0, a.L, 0.0f, nullptr, s);
}

// One workgroup per stretch; the last one of a sequence to end looks at the borders, where two mu may differ relative to the
// largest of the 64 values there, and runs on from the last one at which they do.  part: a matrix of terms of dL/dW per stretch.
// Those of rows that are run again are added up anew, in the first one; the other ones are zero.
__global__ __launch_bounds__(wave_threads(true)) void dense_adjoint_stretch_kernel(const DenseArgs a, float *dh0, const DenseStretch c, float *part)
{
    __shared__ AdjointLds s;
    __shared__ float s_half[4][16][kWave];
    __shared__ int s_apart;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int b = (int)blockIdx.x / c.n, j = (int)blockIdx.x - b * c.n;
    const int start = j * c.len, end = min(start + c.len, a.L);
    float *mine = part + (size_t)b * c.n * DH * DH;        // of this sequence
    auto written = [] {                                    // mu of these rows, for every wave
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    };
    if (threadIdx.x == 0) s_apart = 0;
    if (threadIdx.x == 0) count_enters(c, b, count_read(c, b));
    adjoint_chain<true, true>(a, dh0, b, start, end, 0.0f, c.edge + (size_t)blockIdx.x * DH, s);
    written();
    stretch_weight_gradient(a, b, start, end, s_half, mine + (size_t)j * DH * DH);
    if (!stretch_is_last(c, b)) return;
    for (int e = 1 + w; e < c.n; e += kWaves) {            // a wave looks at the 64 values between two stretches
        const float there = a.du[((size_t)b * a.L + (size_t)e * c.len) * DH + lane], here = c.edge[((size_t)b * c.n + e - 1) * DH + lane];
        const float top = __uint_as_float(wave_max_u32(__float_as_uint(there) & 0x7fffffffu));
        if (!(fabsf(there - here) <= kWarmTol * top)) atomicMax(&s_apart, e);
    }
    __syncthreads();
    const int e = __builtin_amdgcn_readfirstlane(s_apart), rows = e * c.len;
    if (e == 0) return;
    adjoint_chain<false, false, true>(a, dh0, b, 0, rows, a.du[((size_t)b * a.L + rows) * DH + lane], nullptr, s, mine, e);
}

DenseStretch planned(int B, int L, bool backward)
{
    const DensePlan p = g_dense_substitution ? wavefront_plan(B, L, backward) : DensePlan{0, 0};
    DenseStretch c;
    memset(&c, 0, sizeof(c));
    c.n = p.n; c.len = p.len;
    return c;
}

// ------------------------------------------------------------ backward extras
// Wt = W^T (16 KB)
__global__ __launch_bounds__(256) void dense_transpose_kernel(const float *W, float *Wt)
{
    for (int i = threadIdx.x; i < DH * DH; i += 256) Wt[(i % DH) * DH + i / DH] = W[i];
}

// dL/dh0[b] = W^T mu_{b,0}: thread j sums over the rows i of W
__global__ __launch_bounds__(64) void dense_dh0_kernel(const float *W, const float *mu, int L, float *dh0)
{
    const int b = blockIdx.x, j = threadIdx.x;
    const float *m = mu + (size_t)b * L * DH;
    float s = 0.0f;
    for (int i = 0; i < DH; ++i) s = fmaf(W[i * DH + j], m[i], s);
    dh0[(size_t)b * DH + j] = s;
}

// Partial sums of dL/dW = sum over rows (b, l) of mu_l h_{l-1}^T: wave p sums its
// contiguous share of the rows as 64 x 64 x (rows) products on
// v_mfma_f32_32x32x2_f32 (two rows per instruction: A = mu, B = h_{l-1}) and
// writes part[p][64][64]; the partials are added in a fixed order afterwards.
__global__ __launch_bounds__(256) void dense_dw_kernel(const DenseArgs a, float *part, int rows_per_wave)
{
    const int lane = threadIdx.x & 63, n = lane & 31, half = lane >> 5;
    const int p = blockIdx.x * 4 + (threadIdx.x >> 6);
    const size_t rows = (size_t)a.B * a.L;
    const size_t r0 = (size_t)p * rows_per_wave;
    const size_t r1 = r0 + rows_per_wave < rows ? r0 + rows_per_wave : rows;
    f16v Q[2][2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int v = 0; v < 16; ++v) Q[mt][nt][v] = 0.0f;
    // batches of eight rows: all their loads travel together
    constexpr int kPairs = 4;
    for (size_t r = r0; r < r1; r += 2 * kPairs) {
        float m0[kPairs], m1[kPairs], h0v[kPairs], h1v[kPairs];
#pragma unroll
        for (int i = 0; i < kPairs; ++i) {
            const unsigned int row = (unsigned int)r + 2 * i + half;   // this lane half's row of the pair (rows < 2^29)
            const bool ok = row < r1;
            const unsigned int rc = ok ? row : (unsigned int)rows - 1, bq = rc / (unsigned int)a.L;
            const bool first = rc == bq * (unsigned int)a.L, zero = !ok || (first && !a.h0);
            const float *hp = !first ? a.h + (size_t)(rc - 1) * DH : a.h0 ? a.h0 + (size_t)bq * DH : a.h;
            m0[i] = a.du[(size_t)rc * DH + n];
            m1[i] = a.du[(size_t)rc * DH + 32 + n];
            h0v[i] = hp[n];
            h1v[i] = hp[32 + n];
            if (!ok) { m0[i] = 0.0f; m1[i] = 0.0f; }
            if (zero) { h0v[i] = 0.0f; h1v[i] = 0.0f; }
        }
#pragma unroll
        for (int i = 0; i < kPairs; ++i) {
            Q[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(m0[i], h0v[i], Q[0][0], 0, 0, 0);
            Q[0][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(m0[i], h1v[i], Q[0][1], 0, 0, 0);
            Q[1][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(m1[i], h0v[i], Q[1][0], 0, 0, 0);
            Q[1][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(m1[i], h1v[i], Q[1][1], 0, 0, 0);
        }
    }
    float *out = part + (size_t)p * DH * DH;
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
        for (int nt = 0; nt < 2; ++nt)
#pragma unroll
            for (int v = 0; v < 16; ++v) out[(32 * mt + mfma_row(v, half)) * DH + 32 * nt + n] = Q[mt][nt][v];
}

size_t r256(size_t x) { return (x + 255) & ~(size_t)255; }

struct DenseLayout { size_t off_d, off_r, off_A, off_b, off_x, off_hend, total; int n_c; };

DenseLayout dense_layout(int B, int L)
{
    DenseLayout lo;
    lo.n_c = (L + CD - 1) / CD;
    size_t off = r256(sizeof(Ctrl));
    lo.off_d = off; off += r256((size_t)B * L * DH * 4);
    lo.off_r = off; off += r256((size_t)B * L * DH * 4);
    lo.off_A = off; off += r256((size_t)B * lo.n_c * DH * DH * 4);
    lo.off_b = off; off += r256((size_t)B * lo.n_c * DH * 4);
    lo.off_x = off; off += r256((size_t)B * lo.n_c * DH * 4);
    lo.off_hend = off; off += r256((size_t)B * lo.n_c * DH * 4);
    lo.total = off;
    return lo;
}

}  // namespace

int dense_chunk() { return CD; }

int dense_set_products(int mode)
{
    if (mode < 0 || mode > 2) return PARARNN_INVALID_ARG;
    g_dense_products = mode;
    return PARARNN_OK;
}

int dense_set_one_launch(int mode)
{
    if (mode < 0 || mode > 2) return PARARNN_INVALID_ARG;
    g_dense_one_launch = mode;
    return PARARNN_OK;
}

int dense_set_substitution(int enable)
{
    g_dense_substitution = enable ? 1 : 0;
    return PARARNN_OK;
}

int dense_set_jacobian(int mode)
{
    if (mode < 0 || mode > 1) return PARARNN_INVALID_ARG;
    g_dense_jacobian = mode;
    return PARARNN_OK;
}

int dense_chunk_products(const float *W, const float *d, int B, int L, int H, float *A, void *ctrl_scratch,
                         hipStream_t st)
{
    if (H != DH) return PARARNN_UNSUPPORTED;
    if (((uintptr_t)W | (uintptr_t)d | (uintptr_t)A) % 16) return PARARNN_UNSUPPORTED;
    DenseArgs a;
    memset(&a, 0, sizeof(a));
    a.W = W; a.d = const_cast<float *>(d); a.Ac = A;
    a.ctrl = static_cast<Ctrl *>(ctrl_scratch);
    a.B = B; a.L = L; a.n_c = (L + CD - 1) / CD;
    if (launch_reset(a.ctrl, nullptr, 0, nullptr, 0, st) != hipSuccess) return PARARNN_HIP_ERROR;
    const int n_prod = B * (a.n_c - 2);
    if (n_prod > 0)
        launch_products_sweep(g_dense_products, (n_prod + 3) / 4, st, a, 0);
    return hipGetLastError() == hipSuccess ? PARARNN_OK : PARARNN_HIP_ERROR;
}

// waves that share the rows of the dL/dW reduction (a multiple of 4: whole workgroups)
int dw_waves(int B, int L)
{
    const size_t rows = (size_t)B * L;
    size_t wv = (rows + 15) / 16;                 // at least 16 rows per wave: 52 waves for 3138 rows took 19 us, 197 take 7
    if (wv > 1024) wv = 1024;
    return (int)((wv + 3) / 4 * 4);
}

size_t dense_workspace_bytes(int dtype, int B, int L, int H, int backward)
{
    if (dtype != PARARNN_F32 || H != DH) return 256;
    const DenseLayout lo = dense_layout(B, L);
    if (!backward) return lo.total;
    // the forward layout, then W^T and the dL/dW partials
    return lo.total + r256((size_t)DH * DH * 4) + r256((size_t)dw_waves(B, L) * DH * DH * 4);
}

// dL/dW from mu (a.du) and the states
static int dense_weight_gradient(const DenseArgs &a, float *part, float *dW, hipStream_t st)
{
    const int wv = dw_waves(a.B, a.L);
    const size_t rows = (size_t)a.B * a.L;
    int rows_per_wave = (int)((rows + wv - 1) / wv);
    rows_per_wave += rows_per_wave & 1;           // pairs of rows
    hipLaunchKernelGGL(dense_dw_kernel, dim3(wv / 4), dim3(256), 0, st, a, part, rows_per_wave);
    if (hipGetLastError() != hipSuccess) return PARARNN_HIP_ERROR;
    return launch_param_reduce(part, dW, wv, DH * DH, st) == hipSuccess ? PARARNN_OK : PARARNN_HIP_ERROR;
}

int dense_backward(int dtype, const float *W, const void *u, const void *h0, const void *h, const void *g, int B,
                   int L, int H, void *du, float *dW, void *dh0, void *workspace, size_t workspace_bytes,
                   hipStream_t st)
{
    if (dtype != PARARNN_F32 || H != DH) return PARARNN_UNSUPPORTED;
    if (((uintptr_t)W | (uintptr_t)u | (uintptr_t)h | (uintptr_t)h0 | (uintptr_t)g | (uintptr_t)du) % 16)
        return PARARNN_UNSUPPORTED;
    if (workspace_bytes < dense_workspace_bytes(dtype, B, L, H, 1)) return PARARNN_WORKSPACE_TOO_SMALL;
    const DenseLayout lo = dense_layout(B, L);
    char *ws = static_cast<char *>(workspace);
    float *Wt = reinterpret_cast<float *>(ws + lo.total);
    float *part = reinterpret_cast<float *>(ws + lo.total + r256((size_t)DH * DH * 4));
    DenseArgs a;
    memset(&a, 0, sizeof(a));
    a.u = static_cast<const float *>(u); a.h0 = static_cast<const float *>(h0);
    a.h = const_cast<float *>(static_cast<const float *>(h));       // only read on this path
    a.d = reinterpret_cast<float *>(ws + lo.off_d);
    a.r = reinterpret_cast<float *>(ws + lo.off_r);
    a.Ac = reinterpret_cast<float *>(ws + lo.off_A);
    a.bc = reinterpret_cast<float *>(ws + lo.off_b);
    a.xc = reinterpret_cast<float *>(ws + lo.off_x);
    a.ctrl = reinterpret_cast<Ctrl *>(ws);
    a.g = static_cast<const float *>(g); a.du = static_cast<float *>(du);
    a.B = B; a.L = L; a.n_c = lo.n_c;
    DenseStretch c = planned(B, L, true);
    if (c.n > 0) {
        a.W = W;
        // what the stretches leave lies where the chunk products would: 256 bytes of each and 128 of a sequence, and they take 16 KB per 16 steps
        c.edge = a.Ac;
        if (B > kHelperUnits) {
            const size_t items = ((size_t)B * L + 15) / 16, most = (size_t)device_cu_count() * 8;
            hipLaunchKernelGGL(dense_residual_kernel, dim3((unsigned)(items < most ? items : most)), dim3(256), 0, st, a, 5);
            hipLaunchKernelGGL(dense_adjoint_kernel<false>, dim3(B), dim3(wave_threads(false)), 0, st, a, static_cast<float *>(dh0));
        } else if (c.n > 1) {
            // at most one matrix of terms per stretch, of which there are no more than waves that would share the rows
            c.count = reinterpret_cast<unsigned long long *>(c.edge + (size_t)B * c.n * DH);
            c.tag = call_nonce() << kCountBits;
            if (B * c.n > dw_waves(B, L)) return PARARNN_HIP_ERROR;
            hipLaunchKernelGGL(dense_adjoint_stretch_kernel, dim3(B * c.n), dim3(wave_threads(true)), 0, st, a, static_cast<float *>(dh0), c, part);
            if (hipGetLastError() != hipSuccess) return PARARNN_HIP_ERROR;
            return launch_param_reduce(part, dW, B * c.n, DH * DH, st) == hipSuccess ? PARARNN_OK : PARARNN_HIP_ERROR;
        } else {
            hipLaunchKernelGGL(dense_adjoint_kernel<true>, dim3(B), dim3(wave_threads(true)), 0, st, a, static_cast<float *>(dh0));
        }
        return dense_weight_gradient(a, part, dW, st);
    }
    if (launch_reset(a.ctrl, nullptr, 0, nullptr, 0, st) != hipSuccess) return PARARNN_HIP_ERROR;
    hipLaunchKernelGGL(dense_transpose_kernel, dim3(1), dim3(256), 0, st, W, Wt);
    // d_l = 1 - tanh^2(W h_{l-1} + u_l) at the given states (forward addressing, W itself)
    const size_t res_items = ((size_t)B * L + 15) / 16;
    const size_t res_cap = (size_t)device_cu_count() * 8;
    const int res_blocks = (int)(res_items < res_cap ? res_items : res_cap);
    a.W = W; a.rev = 0;
    hipLaunchKernelGGL(dense_residual_kernel, dim3(res_blocks), dim3(256), 0, st, a, 0);
    // the reverse scan with W^T
    a.W = Wt; a.rev = 1;
    const int n_prod = B * (lo.n_c - 2);
    const int n_sweep = (B * lo.n_c + 15) / 16;
    const int n_prod_blocks = n_prod > 0 ? (n_prod + 3) / 4 : 0;
    // always fp32 products: this is one linear solve, not an iteration that would correct an inexact one
    hipLaunchKernelGGL((dense_products_sweep_kernel<true, 0>), dim3(n_sweep + n_prod_blocks), dim3(256), 0, st, a, n_sweep);
    hipLaunchKernelGGL(dense_carry_kernel, dim3(B), dim3(256), 0, st, a);
    hipLaunchKernelGGL(dense_final_sweep_kernel<true>, dim3(n_sweep), dim3(256), 0, st, a);
    // step-local gradients
    if (dh0) hipLaunchKernelGGL(dense_dh0_kernel, dim3(B), dim3(64), 0, st, W, a.du, L, static_cast<float *>(dh0));
    return dense_weight_gradient(a, part, dW, st);
}

int dense_residual_norm(int dtype, const float *W, const void *u, const void *h0, const void *h, int B, int L, int H,
                        float *out, hipStream_t st)
{
    if (dtype != PARARNN_F32 || H != DH) return PARARNN_UNSUPPORTED;
    if (((uintptr_t)W | (uintptr_t)u | (uintptr_t)h | (uintptr_t)h0) % 16) return PARARNN_UNSUPPORTED;
    DenseArgs a;
    memset(&a, 0, sizeof(a));
    a.W = W; a.u = static_cast<const float *>(u); a.h0 = static_cast<const float *>(h0);
    a.h = const_cast<float *>(static_cast<const float *>(h));        // mode 2 only reads it
    a.B = B; a.L = L;
    a.norm = reinterpret_cast<unsigned int *>(out);
    if (launch_zero_words(a.norm, 1, st) != hipSuccess) return PARARNN_HIP_ERROR;
    const size_t res_items = ((size_t)B * L + 15) / 16;
    const size_t res_cap = (size_t)device_cu_count() * 4;
    const int res_blocks = (int)(res_items < res_cap ? res_items : res_cap);
    hipLaunchKernelGGL(dense_residual_kernel, dim3(res_blocks), dim3(256), 0, st, a, 2);
    return hipGetLastError() == hipSuccess ? PARARNN_OK : PARARNN_HIP_ERROR;
}

int dense_forward(int dtype, const float *W, const void *u, const void *h0, int B, int L, int H, float tol,
                  int max_iter, void *h, int *iters, float *delta_trace, void *workspace, size_t workspace_bytes,
                  hipStream_t st)
{
    if (dtype != PARARNN_F32 || H != DH) return PARARNN_UNSUPPORTED;
    if (((uintptr_t)W | (uintptr_t)u | (uintptr_t)h | (uintptr_t)h0) % 16) return PARARNN_UNSUPPORTED;
    const DenseLayout lo = dense_layout(B, L);
    if (workspace_bytes < lo.total) return PARARNN_WORKSPACE_TOO_SMALL;
    char *ws = static_cast<char *>(workspace);
    DenseArgs a;
    memset(&a, 0, sizeof(a));
    a.W = W; a.u = static_cast<const float *>(u); a.h0 = static_cast<const float *>(h0);
    a.h = static_cast<float *>(h);
    a.d = reinterpret_cast<float *>(ws + lo.off_d);
    a.r = reinterpret_cast<float *>(ws + lo.off_r);
    a.Ac = reinterpret_cast<float *>(ws + lo.off_A);
    a.bc = reinterpret_cast<float *>(ws + lo.off_b);
    a.xc = reinterpret_cast<float *>(ws + lo.off_x);
    a.hend = reinterpret_cast<float *>(ws + lo.off_hend);
    a.ctrl = reinterpret_cast<Ctrl *>(ws);
    a.iters_out = iters; a.trace = delta_trace;
    a.B = B; a.L = L; a.n_c = lo.n_c; a.k = 0; a.max_iter = max_iter; a.tol = tol;

    const int status0 = tol < 0.0f ? PARARNN_OK : PARARNN_NOT_CONVERGED;
    const size_t res_items = ((size_t)B * L + 15) / 16;           // one workgroup per 16 rows, a few rounds at most
    const size_t res_cap = (size_t)device_cu_count() * 8;
    const int res_blocks = (int)(res_items < res_cap ? res_items : res_cap);
    if (g_dense_jacobian == 1) {
        // Quasi-Newton: J_l is replaced by its diagonal (1 - F_l^2) * W_ii, so the linear solve is the
        // diagonal scan over 64 independent channels per sequence; no matrix products.  The scan adds
        // its result to h itself; its carry records live where the chunk products would (always
        // large enough).
        const CellInfo ci = {1, 1, 0, -1};
        const Layout sl = make_layout(ci, PARARNN_F32, B, L, DH, false, 4);
        unsigned long long *rec = reinterpret_cast<unsigned long long *>(ws + lo.off_A);
        if (lo.off_A + sl.n_rec * sizeof(unsigned long long) > lo.off_b) return PARARNN_WORKSPACE_TOO_SMALL;   // cannot happen: 24 B of records per 64 steps against 16 KB of products per 16
        if (launch_reset(a.ctrl, rec, sl.n_rec, iters, status0, st) != hipSuccess) return PARARNN_HIP_ERROR;
        hipLaunchKernelGGL(dense_residual_kernel, dim3(res_blocks), dim3(256), 0, st, a, 1);
        FwdArgs f;
        memset(&f, 0, sizeof(f));
        f.g = sl.g;
        f.u = a.r; f.jac = a.d; f.hit = a.h; f.raw_add = 1;
        f.rec = rec; f.ctrl = a.ctrl;
        f.iters_out = iters; f.trace = delta_trace;
        f.max_iter = max_iter; f.tol = tol;
        for (int k = 1; k <= max_iter; ++k) {
            hipLaunchKernelGGL(dense_residual_kernel, dim3(res_blocks), dim3(256), 0, st, a, 3);
            f.k = k;
            const hipError_t e = Kernels<RawScan<1>, float>::newton_iter(sl.cfg, f, false, st);
            if (e != hipSuccess) return PARARNN_HIP_ERROR;
        }
        return hipGetLastError() == hipSuccess ? PARARNN_OK : PARARNN_HIP_ERROR;
    }
    // the maxima of the iterations lie where the chunk products would (at least 4096 words)
    DenseStretch c = planned(B, L, false);
    if (g_dense_products == 0 && max_iter > 0 && max_iter <= DH * DH && c.n > 0) {
        unsigned int *gm = reinterpret_cast<unsigned int *>(ws + lo.off_A);
        if (tol >= 0.0f && tol < kWarmTol) { c.n = 1; c.len = L; }
        if (c.n > 1) {
            // 2.06 KB of each stretch of at least 32 steps and a word of each iteration; chunk products would take 1 KB per step
            c.edge = reinterpret_cast<float *>(gm);
            c.seen = reinterpret_cast<unsigned int *>(c.edge + (size_t)B * c.n * 2 * kWaveIters * DH);
            c.count = reinterpret_cast<unsigned long long *>(c.seen + (size_t)B * seen_words(max_iter));
            c.tag = call_nonce() << kCountBits;
            c.top = reinterpret_cast<unsigned int *>(c.count + (size_t)(B + 1) * kCountApart);
            if (reinterpret_cast<char *>(c.top + (size_t)B * c.n * kWaveIters) > ws + lo.off_b) { c.n = 1; c.len = L; }
        }
        if (c.n > 1) {
            hipLaunchKernelGGL(dense_stretch_kernel, dim3(B * c.n), dim3(wave_threads(true)), 0, st, a, c);
        } else {
            hipLaunchKernelGGL(dense_guess_kernel, dim3(res_blocks), dim3(256), 0, st, a, gm, max_iter);
            hipLaunchKernelGGL(dense_wavefront_kernel, dim3(B), dim3(wave_threads(false)), 0, st, a, gm);
        }
        return hipGetLastError() == hipSuccess ? PARARNN_OK : PARARNN_HIP_ERROR;
    }
    if (launch_reset(a.ctrl, nullptr, 0, iters, status0, st) != hipSuccess) return PARARNN_HIP_ERROR;
    const int n_prod = B * (lo.n_c - 2);
    const int n_prod_blocks = n_prod > 0 ? (n_prod + 3) / 4 : 0;
    const int n_sweep = (B * lo.n_c + 15) / 16;       // workgroups: 16 (sequence, chunk) columns each
    // Launch plan.  The first iterations run as separate launches per phase (each phase at the occupancy
    // that suits it: that is the fast way while the solve is running); what is left of max_iter runs in ONE
    // persistent launch that iterates on the device and returns at once when the solve has already ended.
    // A solve that converges within the head therefore costs one idle launch instead of four per
    // iteration up to max_iter.
    // A fixed-count solve (tol < 0) runs every iteration it is given: nothing is idle, so it stays on the fast path.
    const int head = g_dense_one_launch == 2 ? 0
                     : (g_dense_one_launch == 0 || tol < 0.0f) ? max_iter
                     : (max_iter < kDenseHead ? max_iter : kDenseHead);
    // the initial guess (all a solve of zero iterations returns); the persistent launch makes its own when it starts the solve
    if (max_iter == 0) hipLaunchKernelGGL(dense_residual_kernel, dim3(res_blocks), dim3(256), 0, st, a, 1);
    for (int k = 1; k <= head; ++k) {
        a.k = k;
        // the initial guess and the residual of iteration 1 in one launch; the final sweep of an iteration
        // leaves the next one's
        if (k == 1) hipLaunchKernelGGL(dense_residual_kernel, dim3(res_blocks), dim3(256), 0, st, a, 4);
        launch_products_sweep(g_dense_products, n_sweep + n_prod_blocks, st, a, n_sweep);
        hipLaunchKernelGGL(dense_carry_kernel, dim3(B), dim3(256), 0, st, a);
        if (k < max_iter) hipLaunchKernelGGL((dense_final_sweep_kernel<false, true>), dim3(n_sweep), dim3(256), 0, st, a);
        else hipLaunchKernelGGL((dense_final_sweep_kernel<false, false>), dim3(n_sweep), dim3(256), 0, st, a);
    }
    if (head < max_iter) {
        a.spin_limit = settings().spin_limit;
        const int cap = newton_grid(g_dense_products);
        const size_t most = res_items > (size_t)(n_sweep + n_prod_blocks) ? res_items : (size_t)(n_sweep + n_prod_blocks);
        const int grid = (int)(most < (size_t)cap ? (most < 1 ? 1 : most) : (size_t)cap);
        launch_newton(g_dense_products, grid, st, a, n_sweep, n_prod_blocks, head + 1);
    }
    return hipGetLastError() == hipSuccess ? PARARNN_OK : PARARNN_HIP_ERROR;
}

}  // namespace pararnn
