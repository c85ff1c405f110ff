// Input projection of the cells: u_g = B_g x + b_g for every gate g (the input
// terms of Eq. (7a) / (7b)), with multi-head, i.e. block-diagonal, B_g (App. C),
// and the derivatives of that map.  These are dense contractions and run on the
// matrix cores: operands rounded to bf16, fp32 accumulation
// (v_mfma_f32_32x32x16_bf16), the arithmetic of the paper's mixed-precision
// training set-up.  The bias add and the [B][L][G][H] layout of u are the GEMM's
// epilogue: u is written once, in the form the Newton kernels read.
//
//   forward   u[m][g][h]   = sum_j Wx[g][h][j] x[m][head(h) dh + j] + bias[g][h]
//   backward  dx[m][k dh+j] = sum_g sum_i du[m][g][k dh + i] Wx[g][k dh + i][j]
//             dWx[g][h][j] = sum_m du[m][g][h] x[m][head(h) dh + j]
//             dbias[g][h]  = sum_m du[m][g][h]
//
// forward and dx are "NT" products C[m][n] = sum_k A[m][k] B[n][k] with both
// operands contiguous in k (dx uses a transposed bf16 copy of the weights);
// dWx reduces over the rows m, which are the strided dimension of both of its
// operands, so its loader transposes on the way into LDS, and it is split over
// row ranges whose partial results are added in a fixed order afterwards.
//
// Tiles: 128 x 128 outputs per workgroup of four waves (64 x 64 per wave, four
// 32 x 32 accumulators), 64 k per step, both operand tiles in LDS in k-chunk-major
// order (fragment reads are contiguous), double buffered, the global loads of the
// next two steps in flight while a step is multiplied.
#include "pararnn.h"
#include "pararnn/common.h"
#include "pararnn/launch.h"
#include "proj.h"

#include <stdint.h>
#include <string.h>
#include <math.h>

namespace pararnn {

namespace {

typedef float f16v __attribute__((ext_vector_type(16)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf2v __attribute__((ext_vector_type(2)));
typedef __bf16 bf8v __attribute__((ext_vector_type(8)));
typedef unsigned int u4v __attribute__((ext_vector_type(4)));

constexpr int BM = 128, BN = 128, BK = 64;
// An operand tile in LDS: eight planes, one per 16-byte k-chunk, each holding that chunk of the
// 128 rows back to back, planes 16 bytes further apart than their size.
constexpr int PLANE = 128 * 8 + 8;       // bf16 elements from one plane to the next
constexpr int TILE = 8 * PLANE;          // bf16 elements of a tile

__device__ __forceinline__ unsigned int pack2(float x0, float x1)
{
    const bf2v p = {(__bf16)x0, (__bf16)x1};
    return __builtin_bit_cast(unsigned int, p);
}

// eight consecutive elements as fetched, and as packed bf16
struct Raw8f {
    f4v lo, hi;
};
__device__ __forceinline__ u4v load8(const unsigned short *p) { return *reinterpret_cast<const u4v *>(p); }
__device__ __forceinline__ Raw8f load8(const float *p)
{
    Raw8f r;
    r.lo = *reinterpret_cast<const f4v *>(p);
    r.hi = *reinterpret_cast<const f4v *>(p + 4);
    return r;
}
__device__ __forceinline__ u4v to_bf16x8(const u4v &v) { return v; }
__device__ __forceinline__ u4v to_bf16x8(const Raw8f &v)
{
    const u4v r = {pack2(v.lo[0], v.lo[1]), pack2(v.lo[2], v.lo[3]), pack2(v.hi[0], v.hi[1]), pack2(v.hi[2], v.hi[3])};
    return r;
}
template <typename AT> struct Raw8 { typedef u4v type; };
template <> struct Raw8<float> { typedef Raw8f type; };

// four consecutive outputs in the storage type
__device__ __forceinline__ void store4(float *p, const f4v &v) { *reinterpret_cast<f4v *>(p) = v; }
__device__ __forceinline__ void store4(unsigned short *p, const f4v &v)
{
    *reinterpret_cast<uint2 *>(p) = make_uint2(pack2(v[0], v[1]), pack2(v[2], v[3]));
}

__device__ __forceinline__ void store4(__attribute__((address_space(3))) float *p, const f4v &v)
{
    *(__attribute__((address_space(3))) f4v *)p = v;
}
__device__ __forceinline__ void store4(__attribute__((address_space(3))) unsigned short *p, const f4v &v)
{
    typedef unsigned int u2v __attribute__((ext_vector_type(2)));
    const u2v r = {pack2(v[0], v[1]), pack2(v[2], v[3])};
    *(__attribute__((address_space(3))) u2v *)p = r;
}

__device__ __forceinline__ int acc_row(int v, int half) { return 8 * (v >> 2) + 4 * half + (v & 3); }

// Element offset of 16-byte chunk `chunk` (0..7) of row `row` in an LDS operand tile.  A
// fragment read (32 consecutive rows, one chunk per lane half) is 512 contiguous bytes; the
// eight chunks of a row, stored by eight neighbouring lanes, fall into eight different
// 16-byte bank groups because of the 16 bytes between planes.
__device__ __forceinline__ int lds_off(int row, int chunk) { return chunk * PLANE + row * 8; }

// one 64-k step of a 64 x 64 wave tile from the LDS operand tiles.  PREFETCH: the fragments
// of the next 16 k are requested before the products of the current 16 k are issued (the
// scheduling barriers keep that order), so that LDS latency is paid once per step, not four
// times; it costs 16 registers, which only the bf16 NT kernel has to spare.
template <bool PREFETCH>
__device__ __forceinline__ void mma_step(const unsigned short *sa, const unsigned short *sb, int wm, int wn, int l32,
                                         int half, f16v (&acc)[2][2])
{
    auto read = [&](int kb, bf8v(&a)[2], bf8v(&b)[2]) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            a[i] = *reinterpret_cast<const bf8v *>(sa + lds_off(64 * wm + 32 * i + l32, 2 * kb + half));
            b[i] = *reinterpret_cast<const bf8v *>(sb + lds_off(64 * wn + 32 * i + l32, 2 * kb + half));
        }
    };
    if constexpr (PREFETCH) {
        bf8v fa[2][2], fb[2][2];
        read(0, fa[0], fb[0]);
#pragma unroll
        for (int kb = 0; kb < BK / 16; ++kb) {
            if (kb + 1 < BK / 16) read(kb + 1, fa[(kb + 1) & 1], fb[(kb + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                for (int ni = 0; ni < 2; ++ni)
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[kb & 1][mi], fb[kb & 1][ni], acc[mi][ni], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma unroll
        for (int kb = 0; kb < BK / 16; ++kb) {
            bf8v fa[2], fb[2];
            read(kb, fa, fb);
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                for (int ni = 0; ni < 2; ++ni)
                    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[mi], fb[ni], acc[mi][ni], 0, 0, 0);
        }
    }
}

// The step loop of both products.  Step t is multiplied from LDS buffer t % 2 while the
// global loads of steps t+1 and t+2 are outstanding in two register sets (memory latency
// is several times the duration of a step).  load(set) fetches the next step in stream
// order, store(buf, set) puts a fetched step into an LDS buffer (buf = -1: into none) and
// may publish through LDS what load() needs at its next call, compute(buf) multiplies.
// Loads and stores are issued unconditionally, also past the end of the stream (load()
// then has to deliver something harmless, which is stored and never multiplied): with
// no branch around them the compiler can wait for exactly the older register set while
// the younger loads stay in flight.  For the same reason load() must not touch what it
// fetched: conversion, zeroing of rows past the end and transposition happen in store().
// done() is asked after every step and must give every thread the same answer: the
// barriers are uniform.
template <class Stage, class Load, class Store, class Compute, class Done>
__device__ __forceinline__ void two_ahead(Load load, Store store, Compute compute, Done done)
{
    Stage r0, r1;
    load(r0);
    store(0, r0);
    __syncthreads();
    load(r1);
    store(-1, r1);            // nothing goes to a buffer: only what load() wants published through LDS
    __syncthreads();
    for (;;) {
        // a step from buffer 0; set 0 is free, set 1 holds the next step
        load(r0);
        compute(0);
        store(1, r1);
        __syncthreads();
        if (done()) break;
        // a step from buffer 1; set 1 is free, set 0 holds the next step
        load(r1);
        compute(1);
        store(0, r0);
        __syncthreads();
        if (done()) break;
    }
}

// The same with one register set: the loads of step t+1 are outstanding while step t is
// multiplied.  For stages too large to hold twice (fp32 rows before their transposition).
template <class Stage, class Load, class Store, class Compute, class Done>
__device__ __forceinline__ void one_ahead(Load load, Store store, Compute compute, Done done)
{
    Stage r;
    load(r);
    store(0, r);
    __syncthreads();
    for (int t = 0;; ++t) {
        load(r);
        compute(t & 1);
        store((t + 1) & 1, r);
        __syncthreads();
        if (done()) break;
    }
}

// ------------------------------------------------------------------ NT product
struct GemmArgs {
    const void *A;                 // [M][lda], storage type AT
    const unsigned short *Bw;      // bf16 [N][ldb]
    void *C;                       // [M][ldc], storage type CT
    const float *bias;             // indexed like the columns of C (same batch offsets), or NULL
    long long lda, ldb, ldc;
    int M, N, K;                   // K a multiple of BK
    int kseg;                      // k of A lives at (k / kseg) * kseg_stride + k % kseg; kseg a multiple of BK
    long long kseg_stride;
    int nz0, n_batch;              // batch index z = z1 * nz0 + z0
    long long a_off[2], b_off[2], c_off[2];     // element offsets per unit of z0, z1
    int tiles_m, tiles_n;
    int *tickets;                  // eight counters, zero at launch: the next tile number of each XCD
    int draw;                      // tile numbers taken per draw (copy-to-LDS kernel)
};

// first tile number of an XCD: an eighth of the grid each
__device__ __forceinline__ int xcd_first(const GemmArgs &a, int xcd)
{
    return (int)((long long)a.tiles_m * (a.tiles_n * a.n_batch) * xcd / 8);
}

// row block and (batch, column block) of tile number `no` in patch order
__device__ __forceinline__ void patch_tile(int no, int tiles_m, int inner_n, int &mt, int &inner)
{
    const int pm = no / (8 * inner_n), rem = no - pm * 8 * inner_n;
    const int hm = min(8, tiles_m - 8 * pm);                     // rows of this patch row
    const int pn = rem / (8 * hm), rem2 = rem - pn * 8 * hm;
    const int hn = min(8, inner_n - 8 * pn);                     // columns of this patch
    mt = 8 * pm + rem2 / hn;
    inner = 8 * pn + rem2 % hn;
}

// Persistent workgroups, each walking a list of output tiles; the (tile, k-step) pairs
// of that list form one flat stream of steps, so that the loads of a tile's first steps
// are in flight while the previous tile is still being multiplied.  Step t is multiplied
// from LDS buffer t % 2 while the global loads of steps t+1 and t+2 are outstanding in two
// register sets (memory latency is several times the duration of a step).
//
// Workgroups are dealt to the eight XCDs round-robin by the dispatcher; tile numbers are
// assigned so that each XCD works through a contiguous range, neighbours in time being
// the tiles that share a row block of A (all n tiles, gates and heads of it): they meet
// in one L2.
template <typename AT, typename CT, bool BIAS>
__global__ __launch_bounds__(256, 2) void proj_gemm_nt_kernel(const GemmArgs a)
{
    __shared__ __attribute__((aligned(16))) unsigned short s_a[2][TILE];
    __shared__ __attribute__((aligned(16))) unsigned short s_b[2][TILE];
    __shared__ int s_ring[8];
    const int xcd = blockIdx.x & 7;
    const int inner_n = a.tiles_n * a.n_batch;
    // The (row block, inner) grid is cut into patches of 8 x 8 tiles (smaller at the edges),
    // numbered one after the other; every XCD has an eighth of these numbers (an eighth of the
    // row blocks where there are many; whole row blocks per XCD left XCDs idle where there are
    // few), and its workgroups draw them from a counter: whatever their relative speed they are
    // inside one or two neighbouring patches at any time, whose 8 + 8 operand panels stay in
    // that XCD's L2.
    const int base = xcd_first(a, xcd), n_local = xcd_first(a, xcd + 1) - base;
    auto decode = [&](int local, int &mt, int &inner) { patch_tile(base + local, a.tiles_m, inner_n, mt, inner); };
    const int nk = a.K / BK;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, wm = w >> 1, wn = w & 1;
    const int half = lane >> 5, l32 = lane & 31;
    // Thread 0 draws the number of this workgroup's n-th tile and leaves it in s_ring[n % 8]
    // (n_local or more: the XCD's list is used up); everybody reads it after a later barrier.
    // At most three tiles are drawn ahead of the one being multiplied.
    if (tid == 0) s_ring[0] = atomicAdd(a.tickets + xcd, 1);
    __syncthreads();
    if (s_ring[0] >= n_local) return;

    struct Tile {
        const AT *A;
        const unsigned short *Bw;
        long long coff;
        int m0, n0;
    };
    auto tile_of = [&](int local) {
        int mt, inner;
        decode(local, mt, inner);
        const int nt = inner % a.tiles_n, z = inner / a.tiles_n;
        const int z0 = z % a.nz0, z1 = z / a.nz0;
        Tile t;
        t.A = static_cast<const AT *>(a.A) + z0 * a.a_off[0] + z1 * a.a_off[1];
        t.Bw = a.Bw + z0 * a.b_off[0] + z1 * a.b_off[1];
        t.coff = z0 * a.c_off[0] + z1 * a.c_off[1];
        t.m0 = mt * BM; t.n0 = nt * BN;
        return t;
    };
    // a thread stages four 16-byte pieces of each operand tile per step: piece q = tid + 256 i
    // is k-chunk q % 8 of the tile row below: eight lanes cover one row (eight bank groups), and
    // the two rows of sixteen consecutive lanes are eight apart (the other eight)
    auto piece_row = [](int q) { return ((q >> 4) & 7) + 8 * ((q >> 3) & 1) + 16 * (q >> 7); };
    const u4v zero4 = {0u, 0u, 0u, 0u};
    // the loading side: tile number ln of this workgroup, k-step lks of it; l_switch: the tile
    // is finished and the next load starts the tile drawn meanwhile; l_end: there was none
    Tile lt = tile_of(s_ring[0]);
    int ln = 0, lks = 0;
    bool l_switch = false, l_end = false;
    // the number drawn for tile ln + 1: requested when the last step of tile ln is fetched,
    // put into the ring by the store() that follows (the request's latency passes meanwhile)
    int drawn = 0;
    bool drawn_pending = false;
    struct Stage {
        typename Raw8<AT>::type a[4];
        u4v b[4];
        unsigned int valid;            // bit i: row of a[i] exists, bit 4 + i: row of b[i] exists
    };
    // per tile: where this thread's four pieces of each operand start (k = 0), and which of their
    // rows exist; rows past the end read the last row (valid memory) and are stored as zeros
    const AT *pa[4];
    const unsigned short *pb[4];
    unsigned int l_valid = 0u;
    auto point_at = [&](const Tile &t) {
        l_valid = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int q = tid + 256 * i, row = piece_row(q), c = q & 7;
            const int gm = t.m0 + row, gn = t.n0 + row;
            pa[i] = t.A + (long long)min(gm, a.M - 1) * a.lda + 8 * c;
            pb[i] = t.Bw + (long long)min(gn, a.N - 1) * a.ldb + 8 * c;
            l_valid |= (gm < a.M ? 1u : 0u) << i | (gn < a.N ? 16u : 0u) << i;
        }
    };
    point_at(lt);
    auto load_next = [&](Stage &r) {
        if (l_switch) {
            const int t = s_ring[(ln + 1) & 7];
            if (t >= n_local) {
                l_end = true;              // from here on the last step is fetched again (never multiplied)
            } else {
                lt = tile_of(t);
                point_at(lt);
                ++ln;
                lks = 0;
            }
            l_switch = false;
        }
        const bool last_step = !l_end && lks + 1 == nk;
        if (last_step && tid == 0) drawn = atomicAdd(a.tickets + xcd, 1);
        const int k0 = lks * BK;
        const long long kbase = (long long)(k0 / a.kseg) * a.kseg_stride + k0 % a.kseg;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            r.a[i] = load8(pa[i] + kbase);
            r.b[i] = load8(pb[i] + k0);
        }
        r.valid = l_valid;
        if (last_step) {
            drawn_pending = true;
            l_switch = true;
        } else if (!l_end) {
            ++lks;
        }
    };
    auto store_stage = [&](int buf, const Stage &r) {
        if (drawn_pending) {
            if (tid == 0) s_ring[(ln + 1) & 7] = drawn;
            drawn_pending = false;
        }
        if (buf < 0) return;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int q = tid + 256 * i, row = piece_row(q), c = q & 7;
            *reinterpret_cast<u4v *>(&s_a[buf][lds_off(row, c)]) = (r.valid >> i & 1u) ? to_bf16x8(r.a[i]) : zero4;
            *reinterpret_cast<u4v *>(&s_b[buf][lds_off(row, c)]) = (r.valid >> (4 + i) & 1u) ? r.b[i] : zero4;
        }
    };
    f16v acc[2][2];
    auto clear_acc = [&]() {
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.0f;
    };
    // The product is formed transposed, acc[ni][mi] = (W tile)(A tile)^T: a lane then owns one
    // ROW of C and, per group of four accumulator registers, four consecutive columns, so the
    // epilogue (bias, storage type, the caller's layout) stores 8 or 16 bytes per lane.
    Tile ct = lt;                      // tile being multiplied: number cn of this workgroup
    int cn = 0, cks = 0;
    bool c_end = false;
    auto finish_step = [&](int buf) {
        if (++cks < nk) return;
        // Epilogue.  The accumulators go through LDS so that a wave's global stores are whole
        // row segments (16 bytes per lane, neighbouring lanes neighbouring addresses): each
        // wave transposes its 64 x 64 part in two passes of 32 rows, in its own quarter of the
        // operand buffer that has just been multiplied (free once every wave is past this
        // step).  16-byte chunk c of row r sits at chunk position c ^ (r % chunks per row).
        __syncthreads();
        constexpr int EPC = 16 / (int)sizeof(CT);          // elements per 16-byte chunk
        constexpr int CPR = 64 / EPC;                      // chunks per 64-column row
        CT *stage = reinterpret_cast<CT *>(w < 2 ? s_a[buf] : s_b[buf]) + (w & 1) * (32 * 64);
        CT *C = static_cast<CT *>(a.C) + ct.coff;
        const int col0 = ct.n0 + 64 * wn;                  // N is a multiple of 64: all 64 columns exist or none
#pragma unroll
        for (int mi = 0; mi < 2; ++mi) {
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int col = 32 * ni + 8 * q + 4 * half;      // this lane's four columns, row l32
                    f4v o = {acc[ni][mi][4 * q], acc[ni][mi][4 * q + 1], acc[ni][mi][4 * q + 2], acc[ni][mi][4 * q + 3]};
                    if (BIAS) o += *reinterpret_cast<const f4v *>(a.bias + ct.coff + min(col0, a.N - 64) + col);
                    store4(stage + l32 * 64 + ((col / EPC) ^ (l32 & (CPR - 1))) * EPC + col % EPC, o);
                }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            constexpr int RPI = 64 / CPR;                  // rows per store instruction
#pragma unroll
            for (int it = 0; it < 32 / RPI; ++it) {
                const int r = it * RPI + lane / CPR, cc = lane % CPR;
                const u4v v = *reinterpret_cast<const u4v *>(stage + r * 64 + (cc ^ (r & (CPR - 1))) * EPC);
                const int row = ct.m0 + 64 * wm + 32 * mi + r;
                if (row < a.M && col0 < a.N) *reinterpret_cast<u4v *>(C + (long long)row * a.ldc + col0 + cc * EPC) = v;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        clear_acc();
        cks = 0;
        const int t = s_ring[++cn & 7];     // drawn at least one barrier ago
        if (t >= n_local) c_end = true;
        else ct = tile_of(t);
    };
    clear_acc();

    two_ahead<Stage>(load_next, store_stage,
                     [&](int buf) {
                         mma_step<sizeof(AT) == 2>(s_b[buf], s_a[buf], wn, wm, l32, half, acc);
                         finish_step(buf);
                     },
                     [&]() { return c_end; });
}

// ------------------------------- NT product, bf16 operands copied straight into LDS
// The same product for bf16 storage and K >= 128, built around buffer loads whose destination
// is LDS: operand tiles never pass through registers, and a step costs a wave eight copy
// instructions instead of loads, conversions and LDS stores.
//
//   tile     256 x 256 outputs per workgroup of eight waves (2 x 4; 128 rows x 64 columns per
//            wave = eight 32 x 32 accumulators), 64 k per step; one workgroup per CU
//   LDS      two stages of (256 + 256) rows x 128 bytes = 128 KB.  A copy instruction moves
//            64 x 16 bytes to consecutive LDS addresses, lane i to base + 16 i: 8 rows of a
//            stage, and 8 whole 128-byte lines of memory (with 32 k per step an instruction
//            took half of 16 lines, and the other half of every line was fetched again a step
//            later: the copies alone then took as long as the whole kernel does now).  Which
//            16-byte k-chunk of its row a lane fetches is free, and chosen so that chunk c of
//            row r lies at position c ^ swz(r) of the row: the eight lanes of a row still read
//            one line, and the fragment reads of the multiply (32 rows, one chunk each) spread
//            over all banks, whether 8 or 16 lanes are served per cycle.
//   step T   four rounds of (fragments of the next 16 k, eight products of the current 16 k);
//            before the last round: own copies of step T + 1 landed, own reads of step T done,
//            barrier; then the first fragments of step T + 1 are read and the copies of step
//            T + 2 start into the stage step T has just left.  One barrier per step, LDS
//            latency behind eight products, memory latency behind one step.
//   waits    the copies are issued from inline assembly, so the compiler neither knows nor
//            waits for them; at the one wait of a step the copies of step T + 1 are the only
//            loads the wave has outstanding, so the kernel waits for "no memory operation
//            outstanding", or for "at most sixteen" when the sixteen stores of an output tile
//            were issued after those copies: vector-memory operations of a wave complete in
//            issue order on this architecture (its single counter is used that way by every
//            compiled kernel), and waiting for the stores to drain cost a tenth of the time.
//   tiles    drawn from the per-XCD counters like above, a few consecutive numbers per draw
//            (the compiler waits for the atomic's result with every copy in flight, which
//            stalls the drawing wave; per draw, not per tile), and put into the ring one tile
//            ahead.
namespace dma {
constexpr int BM = 256, BN = 256, BK = 64;
constexpr int OP = 256 * BK;             // bf16 elements of one operand tile of a stage
constexpr int STAGE = 2 * OP;            // A tile, then W tile
}  // namespace dma

__device__ __forceinline__ int dma_swz(int row) { return (row & 7) ^ ((row >> 3) & 1); }

__device__ __forceinline__ unsigned int uniform(unsigned int v) { return __builtin_amdgcn_readfirstlane(v); }

// buffer descriptor words for the assembly forms: base, no stride, whole 4 GiB window
__device__ __forceinline__ u4v rsrc_words(const void *p)
{
    const unsigned long long v = (unsigned long long)p;
    const u4v r = {uniform((unsigned int)v), uniform((unsigned int)(v >> 32) & 0xffffu), 0xffffffffu, 0x27000u};
    return r;
}

__device__ __forceinline__ unsigned int lds_address(const void *p)
{
    return (unsigned int)(unsigned long long)(__attribute__((address_space(3))) const void *)p;
}

// 64 x 16 bytes (64 x 4 bytes) from rsrc + voff + soff to LDS lds_base + 16 (4) * lane.  The five wait
// states in front of the load are the ones a vector-memory instruction needs after a vector instruction
// (v_readfirstlane, v_readlane of a spilled value) has written one of its scalar operands; the compiler
// inserts them for its own instructions and not for what is inside an asm statement.  They also cover
// the wait state between the write of M0 and its use.
__device__ __forceinline__ void copy_to_lds_16(unsigned int lds_base, const u4v &rsrc, unsigned int voff, unsigned int soff)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(uniform(lds_base)), "v"(voff), "s"(rsrc), "s"(uniform(soff)) : "memory", "m0");
}
__device__ __forceinline__ void copy_to_lds_4(unsigned int lds_base, const u4v &rsrc, unsigned int voff, unsigned int soff)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dword %1, %2, %3 offen lds"
                 :: "s"(uniform(lds_base)), "v"(voff), "s"(rsrc), "s"(uniform(soff)) : "memory", "m0");
}

template <bool BIAS>
__global__ __launch_bounds__(512) void proj_gemm_nt_dma_kernel(const GemmArgs a)
{
    constexpr int BM = dma::BM, BN = dma::BN, BK = dma::BK, OP = dma::OP, STAGE = dma::STAGE;
    __shared__ __attribute__((aligned(16))) unsigned short s_op[2][STAGE];
    __shared__ __attribute__((aligned(16))) unsigned short s_epi[8][32 * 32];
    __shared__ __attribute__((aligned(16))) float s_bias[4][8][64];
    __shared__ int s_ring[8];
    const int xcd = blockIdx.x & 7;
    const int inner_n = a.tiles_n * a.n_batch;
    // an eighth of the (row block, inner) grid's patches of 8 x 8 tiles, as in proj_gemm_nt_kernel
    const int base = xcd_first(a, xcd), n_local = xcd_first(a, xcd + 1) - base;
    const int nk = a.K / BK;
    const int tid = threadIdx.x, lane = tid & 63, w = (int)uniform((unsigned int)tid >> 6), wm = w >> 2, wn = w & 3;
    const int half = lane >> 5, l32 = lane & 31;
    if (tid == 0) s_ring[0] = atomicAdd(a.tickets + xcd, a.draw);
    __syncthreads();
    const int first = (int)uniform((unsigned int)s_ring[0]);
    if (first >= n_local) return;

    struct Tile {
        const unsigned short *A, *Bw;
        long long coff;
        int m0, n0;
    };
    auto tile_of = [&](int local) {
        int mt, inner;
        patch_tile(base + local, a.tiles_m, inner_n, mt, inner);
        const int nt = inner % a.tiles_n, z = inner / a.tiles_n;
        const int z0 = z % a.nz0, z1 = z / a.nz0;
        Tile t;
        t.A = static_cast<const unsigned short *>(a.A) + z0 * a.a_off[0] + z1 * a.a_off[1];
        t.Bw = a.Bw + z0 * a.b_off[0] + z1 * a.b_off[1];
        t.coff = z0 * a.c_off[0] + z1 * a.c_off[1];
        t.m0 = mt * BM; t.n0 = nt * BN;
        return t;
    };

    // ---- the copying side: tile number ln of this workgroup, k-step lks of it.  A wave copies rows
    //      32 w .. 32 w + 31 of both operand tiles, eight rows (eight lanes each) per instruction.
    const unsigned int lds_op = lds_address(&s_op[0][0]);
    const int lrow = lane >> 3;
    u4v ra, rb, rbias;
    unsigned int va[4], vb[4], vbias = 0u;
    int ln = 0, lks = 0;
    long long seg_base = 0;                // element offset of the current k-segment in a row of A
    int kin = 0;                           // k within the segment
    bool l_end = false;
    auto point_at = [&](const Tile &t) {
        ra = rsrc_words(t.A + (long long)t.m0 * a.lda);
        rb = rsrc_words(t.Bw + (long long)t.n0 * a.ldb);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // rows past the end read the last row (valid memory); their products are never stored
            const int row = 32 * w + 8 * j + lrow;
            const unsigned int chunk = (unsigned int)((lane & 7) ^ dma_swz(8 * j + lrow));
            const int gm = min(t.m0 + row, a.M - 1) - t.m0, gn = min(t.n0 + row, a.N - 1) - t.n0;
            va[j] = (unsigned int)gm * (unsigned int)a.lda * 2u + chunk * 16u;
            vb[j] = (unsigned int)gn * (unsigned int)a.ldb * 2u + chunk * 16u;
        }
        if (BIAS) {
            rbias = rsrc_words(a.bias + t.coff);
            vbias = (unsigned int)min(t.n0 + 64 * wn + lane, a.N - 1) * 4u;
        }
        seg_base = 0; kin = 0;
    };
    // thread 0: the numbers drawn and not yet handed out
    int next_no = first + 1, left = a.draw - 1;
    auto draw = [&]() {
        // the number of tile ln + 1 goes into the ring; it is read after at least one barrier
        if (tid == 0) {
            if (left == 0) {
                next_no = atomicAdd(a.tickets + xcd, a.draw);
                left = a.draw;
            }
            s_ring[(ln + 1) & 7] = next_no++;
            --left;
        }
    };
    // the copies of the next step in stream order, into stage `buf`
    auto issue = [&](int buf) {
        if (lks == nk) {
            const int t = (int)uniform((unsigned int)s_ring[(ln + 1) & 7]);      // written at least a barrier ago
            if (t >= n_local) {
                l_end = true;
                return;
            }
            point_at(tile_of(t));
            ++ln;
            lks = 0;
        }
        if (lks == 0) {
            draw();
            if (BIAS) copy_to_lds_4(lds_address(&s_bias[ln & 3][w][0]), rbias, vbias, 0u);
        }
        const unsigned int soa = (unsigned int)((seg_base + kin) * 2), sob = (unsigned int)(lks * BK) * 2u;
        const unsigned int dst = lds_op + (unsigned int)buf * (STAGE * 2u) + (unsigned int)(32 * w) * (BK * 2u);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            copy_to_lds_16(dst + (unsigned int)j * (8u * BK * 2u), ra, va[j], soa);
            copy_to_lds_16(dst + OP * 2u + (unsigned int)j * (8u * BK * 2u), rb, vb[j], sob);
        }
        ++lks;
        kin += BK;
        if (kin == a.kseg) {
            kin = 0;
            seg_base += a.kseg_stride;
        }
    };

    // ---- the multiplying side
    // byte offset of this lane's fragment piece within a 32-row block, for the four 16-k rounds of a step
    unsigned int fo[4];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) fo[kb] = (unsigned int)l32 * 128u + (unsigned int)((2 * kb + half) ^ dma_swz(l32)) * 16u;
    auto read_frags = [&](int buf, int kb, bf8v (&fa)[4], bf8v (&fw)[2]) {
        const char *base = reinterpret_cast<const char *>(&s_op[buf][0]) + fo[kb];
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) fa[mi] = *reinterpret_cast<const bf8v *>(base + (128 * wm + 32 * mi) * (BK * 2));
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) fw[ni] = *reinterpret_cast<const bf8v *>(base + OP * 2 + (64 * wn + 32 * ni) * (BK * 2));
    };
    f16v acc[2][4];
    auto clear_acc = [&]() {
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int mi = 0; mi < 4; ++mi)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[ni][mi][v] = 0.0f;
    };
    // acc[ni][mi] = (W rows)(A rows)^T: a lane owns row l32 of the A block and, per four registers,
    // four consecutive columns
    auto multiply = [&](const bf8v (&fa)[4], const bf8v (&fw)[2]) {
#pragma unroll
        for (int mi = 0; mi < 4; ++mi)
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
                acc[ni][mi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[ni], fa[mi], acc[ni][mi], 0, 0, 0);
    };
    Tile ct = tile_of(first);
    int cn = 0, cks = 0;
    bool stores_behind = false;            // an output tile was stored after the copies the next wait is for
    auto epilogue = [&]() {
        // 16 rows x 64 columns at a time through this wave's LDS patch (2 KB), so that a global store
        // instruction writes eight whole 128-byte lines; 16-byte chunk c of patch row r sits at chunk
        // position c ^ (r % 8).  Rows and columns past the end fall outside the buffer descriptor and are
        // dropped, so the number of store instructions never depends on the data: sixteen.
        unsigned short *stage = &s_epi[w][0];
        const int rows_here = a.M - (ct.m0 + 128 * wm);                   // valid rows of this wave's part (may be <= 0)
        const bool cols_here = ct.n0 + 64 * wn < a.N;                     // N is a multiple of 64: all 64 columns or none
        unsigned short *C = static_cast<unsigned short *>(a.C) + ct.coff + (long long)(ct.m0 + 128 * wm) * a.ldc + ct.n0 + 64 * wn;
        const long long valid = (rows_here > 0 && cols_here) ? (long long)(min(rows_here, 128) - 1) * a.ldc * 2 + 128 : 0;
        const buf_rsrc rc = __builtin_amdgcn_make_buffer_rsrc(C, 0, (int)valid, 0x27000);
        const int r16 = l32 & 15;
        // this lane's bias values, read once: between the patch writes below the compiler keeps LDS
        // accesses in order, and every read would wait out the LDS latency by itself
        f4v bias4[2][4];
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f4v zero = {0.0f, 0.0f, 0.0f, 0.0f};
                bias4[ni][q] = BIAS ? *reinterpret_cast<const f4v *>(&s_bias[cn & 3][w][32 * ni + 8 * q + 4 * half]) : zero;
            }
#pragma unroll
        for (int mi = 0; mi < 4; ++mi)
#pragma unroll
            for (int ph = 0; ph < 2; ++ph) {                              // rows 16 ph .. 16 ph + 15 of the 32-row block
                if ((l32 >> 4) == ph) {
#pragma unroll
                    for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            f4v o = {acc[ni][mi][4 * q], acc[ni][mi][4 * q + 1], acc[ni][mi][4 * q + 2], acc[ni][mi][4 * q + 3]};
                            if (BIAS) o += bias4[ni][q];
                            store4(stage + r16 * 64 + ((4 * ni + q) ^ (r16 & 7)) * 8 + 4 * half, o);
                        }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    const int r = 8 * it + (lane >> 3), cc = lane & 7;
                    const u4v v = *reinterpret_cast<const u4v *>(stage + r * 64 + (cc ^ (r & 7)) * 8);
                    const unsigned int off = (unsigned int)(32 * mi + 16 * ph + r) * (unsigned int)a.ldc * 2u + (unsigned int)cc * 16u;
                    __builtin_amdgcn_raw_buffer_store_b128(v, rc, off, 0, 0);
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
    };

    // ---- prologue: two steps on their way, the first one landed
    point_at(ct);
    issue(0);
    issue(1);
    asm volatile("s_waitcnt vmcnt(8)" ::: "memory");       // the eight copies of the second step may be outstanding
    asm volatile("s_barrier" ::: "memory");
    bf8v fa0[4], fw0[2], fa1[4], fw1[2];
    read_frags(0, 0, fa0, fw0);
    clear_acc();

    for (int T = 0;; ++T) {
        const int buf = T & 1;
        read_frags(buf, 1, fa1, fw1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(fa0, fw0);
        __builtin_amdgcn_sched_barrier(0);
        read_frags(buf, 2, fa0, fw0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(fa1, fw1);
        __builtin_amdgcn_sched_barrier(0);
        read_frags(buf, 3, fa1, fw1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(fa0, fw0);
        __builtin_amdgcn_sched_barrier(0);
        // own copies of step T + 1 have landed, own reads of this stage are done; after the barrier
        // everybody's.  Behind those copies the wave has issued nothing, or the sixteen stores of an output tile.
        if (stores_behind) asm volatile("s_waitcnt vmcnt(16) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        stores_behind = false;
        read_frags(buf ^ 1, 0, fa0, fw0);
        if (!l_end) issue(buf);
        __builtin_amdgcn_sched_barrier(0);
        multiply(fa1, fw1);
        __builtin_amdgcn_sched_barrier(0);
        if (++cks == nk) {
            epilogue();
            stores_behind = true;
            clear_acc();
            cks = 0;
            const int nt = (int)uniform((unsigned int)s_ring[++cn & 7]);
            if (nt >= n_local) break;
            ct = tile_of(nt);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// ------------------------------- NT product, fp32 A and C, operands copied straight into LDS
// The kernel above for fp32 storage: rows of A arrive as fp32 (32 k = 128 bytes per row and step) and
// are rounded to bf16 when a lane reads its fragment (two 16-byte reads and four conversions per
// fragment); W is the bf16 copy, 32 k = 64 bytes per row and step, sixteen rows per copy instruction,
// 16-byte chunk c of row r at position c ^ (r / 4 % 4): sixteen rows of a fragment read then cover all
// banks once.  A step is two rounds of eight products; a stage is 32 KB of A and 16 KB of W.  A wave owns
// 64 rows of A x 128 rows of W (the fp32 fragments are the costly ones in registers: two per round instead
// of four).  With 32 k per step a step's products last a quarter of a microsecond, far less than a trip to
// memory, so there are three stages and the copies run two steps ahead; that takes all of LDS, and output
// tiles leave straight from the registers.
namespace dmaf {
constexpr int BK = 32;
constexpr int OPA = 256 * BK * 4;        // bytes of the A tile of a stage
constexpr int STAGE = OPA + 256 * BK * 2;  // A tile, then W tile
}  // namespace dmaf

__device__ __forceinline__ int dmaf_wswz(int row) { return (row >> 2) & 3; }

template <bool BIAS>
__global__ __launch_bounds__(512) void proj_gemm_nt_dma_f32_kernel(const GemmArgs a)
{
    constexpr int BM = dma::BM, BN = dma::BN, BK = dmaf::BK, OPA = dmaf::OPA, STAGE = dmaf::STAGE;
    __shared__ __attribute__((aligned(16))) unsigned char s_op[3][STAGE];
    __shared__ __attribute__((aligned(16))) float s_bias[2][8][128];
    __shared__ int s_ring[8];
    const int xcd = blockIdx.x & 7;
    const int inner_n = a.tiles_n * a.n_batch;
    // an eighth of the (row block, inner) grid's patches of 8 x 8 tiles, as in proj_gemm_nt_kernel
    const int base = xcd_first(a, xcd), n_local = xcd_first(a, xcd + 1) - base;
    const int nk = a.K / BK;
    const int tid = threadIdx.x, lane = tid & 63, w = (int)uniform((unsigned int)tid >> 6), wm = w & 3, wn = w >> 2;
    const int half = lane >> 5, l32 = lane & 31;
    if (tid == 0) s_ring[0] = atomicAdd(a.tickets + xcd, a.draw);
    __syncthreads();
    const int first = (int)uniform((unsigned int)s_ring[0]);
    if (first >= n_local) return;

    struct Tile {
        const float *A;
        const unsigned short *Bw;
        long long coff;
        int m0, n0;
    };
    auto tile_of = [&](int local) {
        int mt, inner;
        patch_tile(base + local, a.tiles_m, inner_n, mt, inner);
        const int nt = inner % a.tiles_n, z = inner / a.tiles_n;
        const int z0 = z % a.nz0, z1 = z / a.nz0;
        Tile t;
        t.A = static_cast<const float *>(a.A) + z0 * a.a_off[0] + z1 * a.a_off[1];
        t.Bw = a.Bw + z0 * a.b_off[0] + z1 * a.b_off[1];
        t.coff = z0 * a.c_off[0] + z1 * a.c_off[1];
        t.m0 = mt * BM; t.n0 = nt * BN;
        return t;
    };

    // ---- the copying side: tile number ln of this workgroup, k-step lks of it.  A wave copies rows
    //      32 w .. 32 w + 31 of both operand tiles: eight rows of A (eight lanes each) or sixteen rows
    //      of W (four lanes each) per instruction.
    const unsigned int lds_op = lds_address(&s_op[0][0]);
    const int lrow = lane >> 3;
    u4v ra, rb, rbias;
    unsigned int va[4], vb[2], vbias[2] = {0u, 0u};
    int ln = 0, lks = 0;
    long long seg_base = 0;                // element offset of the current k-segment in a row of A
    int kin = 0;                           // k within the segment
    bool l_end = false;
    auto point_at = [&](const Tile &t) {
        ra = rsrc_words(t.A + (long long)t.m0 * a.lda);
        rb = rsrc_words(t.Bw + (long long)t.n0 * a.ldb);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // rows past the end read the last row (valid memory); their products are never stored
            const int row = 32 * w + 8 * j + lrow;
            const unsigned int chunk = (unsigned int)((lane & 7) ^ dma_swz(8 * j + lrow));
            const int gm = min(t.m0 + row, a.M - 1) - t.m0;
            va[j] = (unsigned int)gm * (unsigned int)a.lda * 4u + chunk * 16u;
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int row = 32 * w + 16 * j + (lane >> 2);
            const unsigned int chunk = (unsigned int)((lane & 3) ^ dmaf_wswz(row));
            const int gn = min(t.n0 + row, a.N - 1) - t.n0;
            vb[j] = (unsigned int)gn * (unsigned int)a.ldb * 2u + chunk * 16u;
        }
        if (BIAS) {
            rbias = rsrc_words(a.bias + t.coff);
#pragma unroll
            for (int j = 0; j < 2; ++j) vbias[j] = (unsigned int)min(t.n0 + 128 * wn + 64 * j + lane, a.N - 1) * 4u;
        }
        seg_base = 0; kin = 0;
    };
    // thread 0: the numbers drawn and not yet handed out
    int next_no = first + 1, left = a.draw - 1;
    auto draw = [&]() {
        // the number of tile ln + 1 goes into the ring; it is read after at least one barrier
        if (tid == 0) {
            if (left == 0) {
                next_no = atomicAdd(a.tickets + xcd, a.draw);
                left = a.draw;
            }
            s_ring[(ln + 1) & 7] = next_no++;
            --left;
        }
    };
    // the copies of the next step in stream order, into stage `buf`
    auto issue = [&](int buf) {
        if (lks == nk) {
            const int t = (int)uniform((unsigned int)s_ring[(ln + 1) & 7]);      // written at least a barrier ago
            if (t >= n_local) {
                l_end = true;
                return;
            }
            point_at(tile_of(t));
            ++ln;
            lks = 0;
        }
        if (lks == 0) {
            draw();
            if (BIAS) {
#pragma unroll
                for (int j = 0; j < 2; ++j) copy_to_lds_4(lds_address(&s_bias[ln & 1][w][64 * j]), rbias, vbias[j], 0u);
            }
        }
        const unsigned int soa = (unsigned int)((seg_base + kin) * 4), sob = (unsigned int)(lks * BK) * 2u;
        const unsigned int dst = lds_op + (unsigned int)buf * (unsigned int)STAGE;
#pragma unroll
        for (int j = 0; j < 4; ++j) copy_to_lds_16(dst + (unsigned int)(32 * w + 8 * j) * 128u, ra, va[j], soa);
#pragma unroll
        for (int j = 0; j < 2; ++j) copy_to_lds_16(dst + OPA + (unsigned int)(32 * w + 16 * j) * 64u, rb, vb[j], sob);
        ++lks;
        kin += BK;
        if (kin == a.kseg) {
            kin = 0;
            seg_base += a.kseg_stride;
        }
    };

    // ---- the multiplying side
    // byte offsets of this lane's fragment pieces within a 32-row block, for the two 16-k rounds of a step:
    // eight fp32 of an A row (two chunks, rounded to bf16 here), eight bf16 of a W row (one chunk)
    unsigned int foa[2][2], fow[2];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
        for (int e = 0; e < 2; ++e) foa[kb][e] = (unsigned int)l32 * 128u + (unsigned int)((4 * kb + 2 * half + e) ^ dma_swz(l32)) * 16u;
        fow[kb] = (unsigned int)OPA + (unsigned int)l32 * 64u + (unsigned int)((2 * kb + half) ^ dmaf_wswz(l32)) * 16u;
    }
    auto read_frags = [&](int buf, int kb, bf8v (&fa)[2], bf8v (&fw)[4]) {
        const unsigned char *base = &s_op[buf][0];
#pragma unroll
        for (int mi = 0; mi < 2; ++mi) {
            const unsigned char *row = base + (64 * wm + 32 * mi) * 128;
            const f4v lo = *reinterpret_cast<const f4v *>(row + foa[kb][0]), hi = *reinterpret_cast<const f4v *>(row + foa[kb][1]);
            const u4v r = {pack2(lo[0], lo[1]), pack2(lo[2], lo[3]), pack2(hi[0], hi[1]), pack2(hi[2], hi[3])};
            fa[mi] = __builtin_bit_cast(bf8v, r);
        }
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) fw[ni] = *reinterpret_cast<const bf8v *>(base + fow[kb] + (128 * wn + 32 * ni) * 64);
    };
    f16v acc[4][2];
    auto clear_acc = [&]() {
#pragma unroll
        for (int ni = 0; ni < 4; ++ni)
#pragma unroll
            for (int mi = 0; mi < 2; ++mi)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[ni][mi][v] = 0.0f;
    };
    // acc[ni][mi] = (W rows)(A rows)^T: a lane owns row l32 of the A block and, per four registers,
    // four consecutive columns
    auto multiply = [&](const bf8v (&fa)[2], const bf8v (&fw)[4]) {
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int ni = 0; ni < 4; ++ni)
                acc[ni][mi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[ni], fa[mi], acc[ni][mi], 0, 0, 0);
    };
    Tile ct = tile_of(first);
    int cn = 0, cks = 0;
    auto epilogue = [&]() {
        // straight from the registers: a lane owns row l32 of each 32 x 32 block and, per four registers, four
        // consecutive columns, so a store instruction writes 32 bytes of 32 rows (all of LDS belongs to the
        // three stages).  Rows and columns past the end fall outside the buffer descriptor and are dropped, so
        // the number of store instructions never depends on the data: thirty-two.
        const int rows_here = a.M - (ct.m0 + 64 * wm);                    // valid rows of this wave's part (may be <= 0)
        const int cols_here = min(a.N - (ct.n0 + 128 * wn), 128);         // valid columns: a multiple of 64 (may be <= 0)
        float *C = static_cast<float *>(a.C) + ct.coff + (long long)(ct.m0 + 64 * wm) * a.ldc + ct.n0 + 128 * wn;
        const long long valid = (rows_here > 0 && cols_here > 0) ? (long long)(min(rows_here, 64) - 1) * a.ldc * 4 + 512 : 0;
        const buf_rsrc rc = __builtin_amdgcn_make_buffer_rsrc(C, 0, (int)valid, 0x27000);
        const unsigned int lane_off = (unsigned int)l32 * (unsigned int)a.ldc * 4u + (unsigned int)half * 16u;
        const float *bias_w = &s_bias[cn & 1][w][4 * half];
#pragma unroll
        for (int ni = 0; ni < 4; ++ni) {
            // columns past the end (a part that is only half there) go beyond the descriptor too
            const unsigned int col_off = 32 * ni < cols_here ? (unsigned int)(32 * ni) * 4u : 0x80000000u;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f4v zero = {0.0f, 0.0f, 0.0f, 0.0f};
                const f4v b4 = BIAS ? *reinterpret_cast<const f4v *>(bias_w + 32 * ni + 8 * q) : zero;
#pragma unroll
                for (int mi = 0; mi < 2; ++mi) {
                    f4v o = {acc[ni][mi][4 * q], acc[ni][mi][4 * q + 1], acc[ni][mi][4 * q + 2], acc[ni][mi][4 * q + 3]};
                    if (BIAS) o += b4;
                    const unsigned int off = lane_off + (unsigned int)(32 * mi) * (unsigned int)a.ldc * 4u + col_off + (unsigned int)(8 * q) * 4u;
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4v, o), rc, off, 0, 0);
                }
            }
        }
    };

    // ---- prologue: three steps on their way, the first one landed
    point_at(ct);
    issue(0);
    issue(1);
    issue(2);
    asm volatile("s_waitcnt vmcnt(12)" ::: "memory");      // the copies of the second and third step may be outstanding
    asm volatile("s_barrier" ::: "memory");
    bf8v fa0[2], fw0[4], fa1[2], fw1[4];
    read_frags(0, 0, fa0, fw0);
    clear_acc();

    // Step T is multiplied from stage T % 3 while the copies of steps T + 1 and T + 2 are under way; after the
    // barrier of step T its stage takes the copies of step T + 3.  At that barrier the copies of step T + 1 must
    // have landed; behind them the wave has issued the six copies of step T + 2 (unless the list of steps has
    // ended) and, for two steps after an output tile, its 32 stores.
    int st = 0;                            // T % 3
    int stores_behind = 0;                 // steps for which the stores of an output tile are still behind the copies waited for
    for (;;) {
        read_frags(st, 1, fa1, fw1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(fa0, fw0);
        __builtin_amdgcn_sched_barrier(0);
        if (stores_behind) {
            if (!l_end) asm volatile("s_waitcnt vmcnt(38) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(32) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            --stores_behind;
        } else {
            if (!l_end) asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)\n\ts_barrier" ::: "memory");
            else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        }
        // the copies first: the arithmetic of a tile change needs the registers the fp32 fragments would hold
        if (!l_end) issue(st);
        st = st == 2 ? 0 : st + 1;
        __builtin_amdgcn_sched_barrier(0);
        read_frags(st, 0, fa0, fw0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(fa1, fw1);
        __builtin_amdgcn_sched_barrier(0);
        if (++cks == nk) {
            epilogue();
            stores_behind = 2;
            clear_acc();
            cks = 0;
            const int nt = (int)uniform((unsigned int)s_ring[++cn & 7]);
            if (nt >= n_local) break;
            ct = tile_of(nt);
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}


// ------------------------------- forward product of narrow heads: the weights stay in registers
// u = W x + bias where a head is at most 256 wide (K = N = d_h = 64 KB).  The tiles of the kernels above then last four steps of
// 64 k or fewer: the first loads and the store of an output tile weigh as much as its products.  Here a workgroup keeps
// the d_h x d_h weights of one gate of one head in registers (a wave 64 of the output channels, 32 KB registers a lane) and
// rows of x stream past: a step is R rows, whole rows of the head, copied straight into LDS two or three steps ahead; a wave
// multiplies 32 of them by its weights and stores 32 x 64 outputs.  Bound by memory: 65536 rows, H = 1024, three gates in four
// heads of 256 in bf16 185 -> 138 us (3.9 TB/s), eight heads of 64 at H = 512 162 -> 43 (6.2 TB/s, x and u fit the last
// level of cache in part), 6993 rows of four heads of 192 with four gates in fp32 48 -> 28.
//
//   waves    MG row groups x KB column groups; R = 32 MG so that a stage is about 32 KB
//   LDS      NS stages; 16-byte chunk c of row r lies at c ^ (r & 7 ^ r / 8 & 1), in the low three bits: a copy instruction reads
//            whole lines, and eight rows of a fragment read cover all banks
//   waits    as above: operations of a wave complete in order.  A step issues N copies (for the step NS - 1 ahead, with nothing
//            to read past the end) and then N stores, so the number that may be outstanding at a step's one wait is known.
//   XCDs     a job is one head's share of the rows, on one XCD: its workgroups take the G gates of the same rows, and the
//            rows in turn, so that x comes from memory once; an XCD with several jobs runs them side by side.
template <typename AT, int KB> struct RowsShape {
    static constexpr int E = sizeof(AT), K = 64 * KB;
    static constexpr int MG = E == 2 ? (KB == 1 ? 8 : KB == 2 ? 4 : 2) : (KB == 1 ? 4 : KB == 4 ? 1 : 2);
    static constexpr int WAVES = MG * KB, R = 32 * MG, ROW = K * E, STAGE = R * ROW;
    static constexpr int NS = STAGE > 40 * 1024 ? 3 : 4;
    static constexpr int N = STAGE / 1024 / WAVES;          // copies of a wave per step; its stores: as many
    static_assert(N * 1024 * WAVES == STAGE && N == 2 * E && NS * STAGE + WAVES * 2048 <= 160 * 1024, "");
};

struct RowsArgs {
    const void *x;         // [M][H]
    const float *Wx;       // [G][H][dh]
    const float *bias;     // [G][H] or NULL
    void *u;               // [M][G][H]
    int M, H, G, heads;
    int log_parts;         // 2^log_parts shares of the rows
    int abreast, J;        // jobs an XCD runs side by side; workgroups of a job's gate
};

// 32 rows x 32 NI outputs of a wave to memory, rows and channels from `dst` on, `left` rows of them: 2 KB of rows at a time through
// the wave's patch of LDS, so that a store instruction writes pieces of rows that are as long as can be.  16-byte chunk c of patch
// row r sits at c ^ r in the low bits.  Rows past the end are dropped by the descriptor; always NI E stores.
template <typename AT, int NI, bool BIAS>
__device__ __forceinline__ void rows_out(const f16v (&acc)[NI], const f4v (&bias4)[NI][4], unsigned int lds_epi, unsigned char *dst,
                                         long long ldu, long long left, int lane)
{
    constexpr int E = sizeof(AT), PW = 32 * NI * E, PR = 2048 / PW, CH = PW / 16, SW = CH < 8 ? CH - 1 : 7;
    const int l32 = lane & 31, half = lane >> 5;
    const buf_rsrc rc = __builtin_amdgcn_make_buffer_rsrc(dst, 0, left > 0 ? (int)((min(left, 32ll) - 1) * ldu + PW) : 0, 0x27000);
    const int pr = l32 % PR, r0 = lane / CH;                               // patch row of this lane's outputs, and of its pieces to store
    unsigned int wr = lds_epi + (unsigned int)(pr * PW + (E == 2 ? 8 * half : 0)), wx = (unsigned int)((pr & SW) ^ (E == 4 ? half : 0)) * 16u;
    unsigned int rd = lds_epi + (unsigned int)(r0 * PW), rx = (unsigned int)((lane % CH) * 16), off = (unsigned int)r0 * (unsigned int)ldu + rx;
    asm volatile("" : "+v"(wr), "+v"(wx), "+v"(rd), "+v"(rx), "+v"(off));  // worked out here: there is no room to keep what follows from them
#pragma unroll
    for (int ph = 0; ph < 32 / PR; ++ph) {
        if (l32 / PR == ph) {
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    f4v o = {acc[ni][4 * q], acc[ni][4 * q + 1], acc[ni][4 * q + 2], acc[ni][4 * q + 3]};
                    if constexpr (BIAS) o += bias4[ni][q];
                    const unsigned int c = E == 2 ? 4 * ni + q : 8 * ni + 2 * q;
                    store4((__attribute__((address_space(3))) AT *)(unsigned long long)(wr + ((c * 16u) ^ wx)), o);
                }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            const unsigned int sw = (unsigned int)((r0 + it * (PR / 2)) & SW) * 16u;
            const u4v v = *(const __attribute__((address_space(3))) u4v *)(unsigned long long)(rd + it * (PR / 2) * PW + (rx ^ sw));
            __builtin_amdgcn_raw_buffer_store_b128(v, rc, off + (unsigned int)(PR * ph + it * (PR / 2)) * (unsigned int)ldu, 0, 0);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
}

template <typename AT, int KB, bool BIAS>
__global__ __launch_bounds__((64 * RowsShape<AT, KB>::WAVES)) void proj_rows_kernel(const RowsArgs a)
{
    typedef RowsShape<AT, KB> S;
    constexpr int E = S::E, K = S::K, R = S::R, ROW = S::ROW, NS = S::NS, N = S::N;
    __shared__ __attribute__((aligned(16))) unsigned char s_op[NS][S::STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s_epi[S::WAVES][2048];
    const int xcd = blockIdx.x & 7, wg = blockIdx.x >> 3, gate = wg % a.G, lane_job = wg / a.G % a.abreast, turn = wg / a.G / a.abreast;
    if (turn >= a.J) return;
    const int tid = threadIdx.x, lane = tid & 63, w = (int)uniform((unsigned int)tid >> 6), wm = w / KB, wn = w % KB;
    const int half = lane >> 5, l32 = lane & 31;
    const unsigned int lds_op = lds_address(&s_op[0][0]), lds_epi = lds_address(&s_epi[w][0]);
    const long long ldx = (long long)a.H * E, ldu = (long long)a.G * a.H * E;      // bytes
    // where this lane's 16 bytes of each copy come from, within a step
    unsigned int va[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int byte = (w * N + j) * 1024 + lane * 16, row = byte / ROW, c = byte % ROW / 16;
        va[j] = (unsigned int)row * (unsigned int)ldx + (unsigned int)(c ^ dma_swz(row)) * 16u;
    }
    // and this lane's pieces of the fragments: a row's position bits are those of its row within a block of 32
    unsigned int fo[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int c = E == 2 ? 2 * q + half : 4 * (q >> 1) + 2 * half + (q & 1);   // bf16: round q of four; fp32: piece q % 2 of round q / 2
        fo[q] = (unsigned int)(32 * wm + l32) * ROW + (unsigned int)(c ^ dma_swz(l32)) * 16u;
    }
    const int steps = (a.M + R - 1) / R, jobs = a.heads << a.log_parts;
    for (int job = xcd + 8 * lane_job; job < jobs; job += 8 * a.abreast) {
        const int head = job % a.heads, part = job / a.heads;
        const int s0 = (int)((long long)steps * part >> a.log_parts), s1 = (int)((long long)steps * (part + 1) >> a.log_parts);
        const int count = s1 - s0 > turn ? (s1 - s0 - turn + a.J - 1) / a.J : 0;   // steps s0 + turn + i J
        if (count == 0) continue;
        const unsigned long long x0 = (unsigned long long)a.x + (unsigned long long)head * ROW;
        auto issue = [&](int i, int stage) {
            const long long row = (long long)(s0 + turn + (long long)i * a.J) * R, left = a.M - row;
            const unsigned long long p = x0 + (unsigned long long)(row * ldx);
            // rows past the last one lie beyond the descriptor and arrive as zeros
            const unsigned int n = i < count ? (unsigned int)((min(left, (long long)R) - 1) * ldx + ROW) : 0u;
            const u4v rs = {uniform((unsigned int)p), uniform((unsigned int)(p >> 32) & 0xffffu), uniform(n), 0x27000u};
#pragma unroll
            for (int j = 0; j < N; ++j)
                copy_to_lds_16(lds_op + (unsigned int)stage * S::STAGE + (unsigned int)(w * N + j) * 1024u, rs, va[j], 0u);
        };
        // The weights come through the stages, as they are (fp32), 32 of every wave's 64 channels at a time or all of them
        // where they fit, in the same order of chunks: read from memory by the lanes that keep them they took 15 us at d_h = 256.
        const int o0 = gate * a.H + head * K + 64 * wn;                            // this wave's first output channel
        bf8v wf[2][4 * KB];
        f4v bias4[2][4];
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if constexpr (BIAS) bias4[ni][q] = *reinterpret_cast<const f4u *>(a.bias + o0 + 32 * ni + 8 * q + 4 * half);
        {
            constexpr int WB = 32 * KB * K * 4, PER = WB / 1024 / S::WAVES, AT_ONCE = 2 * WB <= NS * S::STAGE ? 2 : 1;
            static_assert(PER * 1024 * S::WAVES == WB && WB <= NS * S::STAGE, "");
            const unsigned long long p = (unsigned long long)(a.Wx + (size_t)(gate * a.H + head * K) * K);
            const u4v rs = {uniform((unsigned int)p), uniform((unsigned int)(p >> 32) & 0xffffu), (unsigned int)(K * K * 4), 0x27000u};
#pragma unroll
            for (int n0 = 0; n0 < 2; n0 += AT_ONCE) {
#pragma unroll
                for (int ni = n0; ni < n0 + AT_ONCE; ++ni)
#pragma unroll
                    for (int j = 0; j < PER; ++j) {
                        const int byte = (w * PER + j) * 1024 + lane * 16, row = byte / (4 * K), c = byte % (4 * K) / 16;
                        copy_to_lds_16(lds_op + (unsigned int)((ni - n0) * WB + (w * PER + j) * 1024), rs,
                                       (unsigned int)((row / 32 * 64 + 32 * ni + row % 32) * (4 * K) + (c ^ dma_swz(row)) * 16), 0u);
                    }
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
                for (int ni = n0; ni < n0 + AT_ONCE; ++ni)
#pragma unroll
                    for (int kb = 0; kb < 4 * KB; ++kb) {
                        const unsigned char *q = &s_op[0][0] + (ni - n0) * WB + (32 * wn + l32) * (4 * K) + kb / 2 * 128;
                        const int c = 4 * (kb & 1) + 2 * half;
                        Raw8f r;
                        r.lo = *reinterpret_cast<const f4v *>(q + (c ^ dma_swz(l32)) * 16);
                        r.hi = *reinterpret_cast<const f4v *>(q + ((c + 1) ^ dma_swz(l32)) * 16);
                        wf[ni][kb] = __builtin_bit_cast(bf8v, to_bf16x8(r));
                    }
#pragma unroll
                for (int ni = n0; ni < n0 + AT_ONCE; ++ni)
#pragma unroll
                    for (int kb = 0; kb < 4 * KB; ++kb) asm volatile("" : "+v"(wf[ni][kb]));    // read before what follows overwrites it
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            }
            if constexpr (BIAS) {
#pragma unroll
                for (int q = 0; q < 8; ++q) asm volatile("" : "+v"(bias4[q / 4][q % 4]));       // and waited for here, not in the loop
            }
        }
        // acc = (W rows)(x rows)^T: a lane owns row l32 of x and, per four registers, four consecutive channels
#pragma unroll
        for (int i = 0; i < NS - 1; ++i) issue(i, i);
        int stage = 0, behind = 0;
        for (int i = 0; i < count; ++i) {
            // the copies of this step have landed: behind them at most those of the steps after it, and stores
            asm volatile("" : "+s"(behind));                                       // (no copy of the loop for each of the first steps)
            if (behind >= NS - 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N * (2 * NS - 3)) : "memory");
            else if (behind == 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N * (NS - 2)) : "memory");
            else if (behind == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N * (NS - 1)) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N * NS) : "memory");
            ++behind;
            // everybody's have, and everybody has read the stage before it
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            issue(i + NS - 1, stage == 0 ? NS - 1 : stage - 1);
            const unsigned char *op = &s_op[stage][0];
            f16v acc[2];
#pragma unroll
            for (int ni = 0; ni < 2; ++ni)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[ni][v] = 0.0f;
            // the fragments of the next 32 k are read while those of the last are multiplied
            bf8v fa[2][2];
            auto read = [&](int g, bf8v(&f)[2]) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    if constexpr (E == 2) {
                        f[q] = *reinterpret_cast<const bf8v *>(op + fo[2 * (g & 1) + q] + (g >> 1) * 128);
                    } else {
                        Raw8f r;
                        r.lo = *reinterpret_cast<const f4v *>(op + fo[2 * q] + g * 128);
                        r.hi = *reinterpret_cast<const f4v *>(op + fo[2 * q + 1] + g * 128);
                        f[q] = __builtin_bit_cast(bf8v, to_bf16x8(r));
                    }
                }
            };
            read(0, fa[0]);
#pragma unroll
            for (int g = 0; g < 2 * KB; ++g) {
                if (g + 1 < 2 * KB) read(g + 1, fa[(g + 1) & 1]);
#pragma unroll
                for (int q = 0; q < 2; ++q)
#pragma unroll
                    for (int ni = 0; ni < 2; ++ni)
                        acc[ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[ni][2 * g + q], fa[g & 1][q], acc[ni], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            const long long row = (long long)(s0 + turn + (long long)i * a.J) * R + 32 * wm;
            rows_out<AT, 2, BIAS>(acc, bias4, lds_epi, static_cast<unsigned char *>(a.u) + row * ldu + (long long)o0 * E, ldu, a.M - row, lane);
            stage = stage + 1 == NS ? 0 : stage + 1;
        }
        // nothing of this job is in flight when the next one fills the stages
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
}


// ------------------------------- dx of narrow heads: the weights of all gates of a head stay in registers
// dx = sum over the gates of du_g W_g for heads of at most 256 channels, the same way: a workgroup keeps a head's G d_h x d_h
// weights (a wave 32 of the input channels j, 64 at d_h = 64), a step is R rows of one gate's du, and G steps add up to 32
// rows x channels of a row block per wave and turn.  Bound by memory: three gates, 65536 x 512 in heads of 64, bf16 73 -> 45 us
// (6.0 TB/s, in part from the last level of cache), 20000 x 768 in heads of 192 44 -> 27;
// fp32: 32768 x 1024 in heads of 256 130 -> 113, four gates of 6993 x 768 in heads of 192 35 -> 31.
//
//   W        arrives as fp32 rows i through two halves of the stages; a lane picks its column j of eight rows
//   waits    copies as above; the stores come with every G-th step: which of them lie between is known by the gate, but for
//            the first rows, which have none before them
template <typename AT, int KB, int G> struct DxShape {
    static constexpr int E = sizeof(AT), K = 64 * KB, ROW = K * E;
    static constexpr int NI = KB == 1 ? 2 : 1, NG = 2 * KB / NI;            // 32-channel blocks of a wave, groups of them
    static constexpr int MG = KB == 1 ? 16 / E : KB == 2 ? 2 : 1, RB = E == 2 && KB > 1 && KB * G < 12 ? 2 : 1;      // (192 registers of weights leave room for one row block)
    static constexpr int WAVES = MG * NG, R = 32 * MG * RB, STAGE = R * ROW, NS = STAGE <= 16384 ? 8 : STAGE < 32768 && E == 4 ? 6 : 4;
    static constexpr int N = STAGE / 1024 / WAVES, STORES = RB * NI * E;
    static constexpr int RW = NS * STAGE / 2 / (4 * K) < K ? NS * STAGE / 2 / (4 * K) : K;      // rows of W in half of the stages
    static constexpr int PER = RW * K * 4 / 1024 / WAVES;
    static_assert(N * 1024 * WAVES == STAGE && PER * 1024 * WAVES == RW * K * 4 && K % RW == 0 && RW % 16 == 0, "");
};

struct DxArgs {
    const void *du;        // [M][G][H]
    const float *Wx;       // [G][H][dh]
    void *dx;              // [M][H]
    int M, H, heads;
    int log_parts, abreast, J;
};

template <typename AT, int KB, int G>
__global__ __launch_bounds__((64 * DxShape<AT, KB, G>::WAVES)) void proj_dx_rows_kernel(const DxArgs a)
{
    typedef DxShape<AT, KB, G> S;
    constexpr int E = S::E, K = S::K, R = S::R, ROW = S::ROW, NS = S::NS, N = S::N, NI = S::NI, RB = S::RB;
    __shared__ __attribute__((aligned(128))) unsigned char s_op[NS * S::STAGE];
    __shared__ __attribute__((aligned(16))) unsigned char s_epi[S::WAVES][2048];
    const int xcd = blockIdx.x & 7, wg = blockIdx.x >> 3, lane_job = wg % a.abreast, turn = wg / a.abreast;
    if (turn >= a.J) return;
    const int tid = threadIdx.x, lane = tid & 63, w = (int)uniform((unsigned int)tid >> 6), wm = w / S::NG, wn = w % S::NG;
    const int half = lane >> 5, l32 = lane & 31;
    const unsigned int lds_op = lds_address(s_op), lds_epi = lds_address(&s_epi[w][0]);
    const long long ldu = (long long)G * a.H * E, ldx = (long long)a.H * E;        // bytes
    unsigned int va[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int byte = (w * N + j) * 1024 + lane * 16, row = byte / ROW, c = byte % ROW / 16;
        va[j] = (unsigned int)row * (unsigned int)ldu + (unsigned int)(c ^ dma_swz(row)) * 16u;
    }
    // of this lane's first fragment; the others of 128 bytes of a row are at this address with two of its bits changed
    const unsigned int fo = lds_op + (unsigned int)(32 * RB * wm + l32) * ROW + (unsigned int)(((E == 2 ? 1 : 2) * half) ^ dma_swz(l32)) * 16u;
    const int steps = (a.M + R - 1) / R, jobs = a.heads << a.log_parts;
    for (int job = xcd + 8 * lane_job; job < jobs; job += 8 * a.abreast) {
        const int head = job % a.heads, part = job / a.heads;
        const int s0 = (int)((long long)steps * part >> a.log_parts), s1 = (int)((long long)steps * (part + 1) >> a.log_parts);
        const int count = s1 - s0 > turn ? (s1 - s0 - turn + a.J - 1) / a.J : 0;   // row blocks s0 + turn + i J
        if (count == 0) continue;

        bf8v wf[NI][G][4 * KB];
        {
            constexpr int PER_GATE = K / S::RW, ROUNDS = G * PER_GATE;
            auto fetch = [&](int r) {
                const unsigned long long p = (unsigned long long)(a.Wx + ((size_t)(r / PER_GATE) * a.H + (size_t)head * K + (size_t)(r % PER_GATE) * S::RW) * K);
                const u4v rs = {uniform((unsigned int)p), uniform((unsigned int)(p >> 32) & 0xffffu), (unsigned int)(S::RW * K * 4), 0x27000u};
#pragma unroll
                for (int j = 0; j < S::PER; ++j) {
                    const unsigned int at = (unsigned int)((w * S::PER + j) * 1024);
                    copy_to_lds_16(lds_op + (unsigned int)((r & 1) * (NS * S::STAGE / 2)) + at, rs, (unsigned int)lane * 16u, at);
                }
            };
            fetch(0);
            if (ROUNDS > 1) fetch(1);
#pragma unroll
            for (int r = 0; r < ROUNDS; ++r) {
                if (r + 1 < ROUNDS) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(S::PER) : "memory");
                else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
                unsigned int w0 = lds_op + (unsigned int)((r & 1) * (NS * S::STAGE / 2) + (8 * half * K + 32 * NI * wn + l32) * 4);
                asm volatile("" : "+v"(w0));                                       // what is added is part of the instructions
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                    for (int k = 0; k < S::RW / 16; ++k) {
                        const __attribute__((address_space(3))) float *q = (const __attribute__((address_space(3))) float *)(unsigned long long)w0 + 16 * k * K + 32 * ni;
                        const u4v v = {pack2(q[0], q[K]), pack2(q[2 * K], q[3 * K]), pack2(q[4 * K], q[5 * K]), pack2(q[6 * K], q[7 * K])};
                        bf8v f = __builtin_bit_cast(bf8v, v);
                        asm volatile("" : "+v"(f));                                // read before what follows overwrites it
                        wf[ni][r / PER_GATE][r % PER_GATE * (S::RW / 16) + k] = f;
                        if (KB * G >= 12 && k % 2 == 1) asm volatile("" ::: "memory");      // registers for two fragments at a time
                    }
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                if (r + 2 < ROUNDS) fetch(r + 2);
            }
        }

        const unsigned long long u0 = (unsigned long long)a.du + (unsigned long long)head * ROW;
        // step t: gate t % G of row block t / G
        int ci = 0, cg = 0;                                                        // of the next copies
        auto issue = [&](int stage) {
            const long long row = (long long)(s0 + turn + (long long)ci * a.J) * R, left = a.M - row;
            const unsigned long long p = u0 + (unsigned long long)(row * ldu + (long long)cg * ldx);
            const unsigned int n = ci < count ? (unsigned int)((min(left, (long long)R) - 1) * ldu + ROW) : 0u;
            const u4v rs = {uniform((unsigned int)p), uniform((unsigned int)(p >> 32) & 0xffffu), uniform(n), 0x27000u};
#pragma unroll
            for (int j = 0; j < N; ++j)
                copy_to_lds_16(lds_op + (unsigned int)stage * S::STAGE + (unsigned int)(w * N + j) * 1024u, rs, va[j], 0u);
            if (++cg == G) {
                cg = 0;
                ++ci;
            }
        };
#pragma unroll
        for (int q = 0; q < NS - 1; ++q) issue(q);
        int stage = 0, before = 0;                                                 // row blocks stored before this one
        f16v acc[RB][NI];
        for (int i = 0; i < count; ++i) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[rb][ni][v] = 0.0f;
#pragma unroll
            for (int g = 0; g < G; ++g) {
                // the copies of this step have landed: behind them those of NS - 2 steps, and the stores at the ends of row blocks
                // among the NS - 1 steps before
                constexpr int COPIES = N * (NS - 2);
                constexpr int STORES = S::STORES;
                const int ends = g < NS - 1 ? (NS - 2 - g) / G + 1 : 0;
                if (ends > 0) {
                    asm volatile("" : "+s"(before));                               // (no copy of the loop for the first row blocks)
                    if (before < ends) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(COPIES) : "memory");
                    else if (ends == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(COPIES + STORES) : "memory");
                    else if (ends == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(COPIES + 2 * STORES) : "memory");
                    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(COPIES + 3 * STORES) : "memory");
                } else {
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(COPIES) : "memory");
                }
                asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
                issue(stage == 0 ? NS - 1 : stage - 1);
                // fragments are read two ahead of their products
                const unsigned int op = fo + (unsigned int)stage * S::STAGE;
                bf8v fa[3][RB];
                auto read = [&](int kb, bf8v(&f)[RB]) {
                    unsigned int at = op ^ (E == 2 ? 32u * (kb & 3) : 64u * (kb & 1));
                    if (KB * G >= 12) asm volatile("" : "+v"(at));                 // not kept for the next 128 bytes
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb) {
                        if constexpr (E == 2) {
                            f[rb] = *(const __attribute__((address_space(3))) bf8v *)(unsigned long long)(at + (kb >> 2) * 128 + rb * (32 * ROW));
                        } else {
                            Raw8f r;
                            r.lo = *(const __attribute__((address_space(3))) f4v *)(unsigned long long)(at + (kb >> 1) * 128 + rb * (32 * ROW));
                            r.hi = *(const __attribute__((address_space(3))) f4v *)(unsigned long long)((at ^ 16u) + (kb >> 1) * 128 + rb * (32 * ROW));
                            f[rb] = __builtin_bit_cast(bf8v, to_bf16x8(r));
                        }
                    }
                };
                read(0, fa[0]);
                read(1, fa[1]);
#pragma unroll
                for (int kb = 0; kb < 4 * KB; ++kb) {
                    if (kb + 2 < 4 * KB) read(kb + 2, fa[(kb + 2) % 3]);
#pragma unroll
                    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                        for (int ni = 0; ni < NI; ++ni)
                            acc[rb][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[ni][g][kb], fa[kb % 3][rb], acc[rb][ni], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                stage = stage + 1 == NS ? 0 : stage + 1;
            }
            const f4v none[NI][4] = {};
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) {
                const long long row = (long long)(s0 + turn + (long long)i * a.J) * R + 32 * (RB * wm + rb);
                rows_out<AT, NI, false>(acc[rb], none, lds_epi, static_cast<unsigned char *>(a.dx) + row * ldx + (long long)(head * K + 32 * NI * wn) * E, ldx, a.M - row, lane);
            }
            ++before;
        }
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
}

// --------------------------------------------------- dWx and dbias (TN product)
struct DwArgs {
    const void *du;        // [M][G][H], storage type AT
    const void *x;         // [M][H]
    float *part;           // [S][G][H][dh] partial sums of dWx
    float *dbpart;         // [S][G][H] partial sums of dbias, or NULL
    int M, H, G, heads, dh;
    int S, rows_per_split; // rows_per_split a multiple of BK
    int tiles;             // tiles per dh (128 wide; 256 wide for the copy-to-LDS kernel)
    int n_blocks, per_xcd; // tiles^2 * G * heads * S workgroups, an eighth of them (rounded up)
};

// Four adjacent channels of eight consecutive rows as fetched; transposed in registers into
// one 16-byte k-run per channel (rows that do not count become zeros), plus column sums.
template <typename AT> struct QuadRows;
template <> struct QuadRows<unsigned short> {
    uint2 v[8];
    int n_valid;
    __device__ __forceinline__ void load(const unsigned short *p, long long ld, int m, int m_last, int n_valid_)
    {
        // rows m .. m + 7, those past m_last replaced by m_last (valid memory, counted as zeros)
        const unsigned short *base = p + (long long)min(m, m_last) * ld;
        const int dm = max(m_last - m, 0), ldi = (int)ld;
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = *reinterpret_cast<const uint2 *>(base + min(r, dm) * ldi);
        n_valid = n_valid_;
    }
    __device__ __forceinline__ void transpose(u4v (&c)[4], float (&s)[4]) const
    {
        uint2 t[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) t[r] = r < n_valid ? v[r] : make_uint2(0u, 0u);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            c[0][k] = (t[2 * k].x & 0xffffu) | (t[2 * k + 1].x << 16);
            c[1][k] = (t[2 * k].x >> 16) | (t[2 * k + 1].x & 0xffff0000u);
            c[2][k] = (t[2 * k].y & 0xffffu) | (t[2 * k + 1].y << 16);
            c[3][k] = (t[2 * k].y >> 16) | (t[2 * k + 1].y & 0xffff0000u);
        }
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            s[0] += __builtin_bit_cast(float, t[r].x << 16);
            s[1] += __builtin_bit_cast(float, t[r].x & 0xffff0000u);
            s[2] += __builtin_bit_cast(float, t[r].y << 16);
            s[3] += __builtin_bit_cast(float, t[r].y & 0xffff0000u);
        }
    }
};
template <> struct QuadRows<float> {
    f4v v[8];
    int n_valid;
    __device__ __forceinline__ void load(const float *p, long long ld, int m, int m_last, int n_valid_)
    {
        const float *base = p + (long long)min(m, m_last) * ld;
        const int dm = max(m_last - m, 0), ldi = (int)ld;
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = *reinterpret_cast<const f4v *>(base + min(r, dm) * ldi);
        n_valid = n_valid_;
    }
    __device__ __forceinline__ void transpose(u4v (&c)[4], float (&s)[4]) const
    {
        const f4v zero = {0.0f, 0.0f, 0.0f, 0.0f};
        f4v t[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) t[r] = r < n_valid ? v[r] : zero;
#pragma unroll
        for (int ch = 0; ch < 4; ++ch)
#pragma unroll
            for (int k = 0; k < 4; ++k) c[ch][k] = pack2(t[2 * k][ch], t[2 * k + 1][ch]);
#pragma unroll
        for (int r = 0; r < 8; ++r)
#pragma unroll
            for (int ch = 0; ch < 4; ++ch) s[ch] += t[r][ch];
    }
};

// One workgroup: a 128 x 128 tile of dWx[g][head] for one row range.  Tile rows are
// the output channels i (operand du), tile columns the input channels j (operand x);
// k runs over the rows m of the range, 64 per step.  A thread stages channels
// 4 c4 .. 4 c4 + 3 of rows 8 rg .. 8 rg + 7 of the step for both operands.
template <typename AT>
__global__ __launch_bounds__(256, 2) void proj_dw_kernel(const DwArgs a)
{
    __shared__ __attribute__((aligned(16))) unsigned short s_a[2][TILE];
    __shared__ __attribute__((aligned(16))) unsigned short s_b[2][TILE];
    __shared__ float s_db[8][BM];
    // Workgroups go to the eight XCDs round-robin; numbering them so that each XCD works through a
    // contiguous range keeps the tiles that share operand panels (the tiles of one (head, range):
    // x is common to its gates, du to its column tiles) on one L2 at about the same time.
    int id = (int)(blockIdx.x & 7) * a.per_xcd + (int)(blockIdx.x >> 3);
    if (id >= a.n_blocks) return;
    const int tj = id % a.tiles; id /= a.tiles;
    const int ti = id % a.tiles; id /= a.tiles;
    const int g = id % a.G; id /= a.G;
    const int head = id % a.heads;
    const int s = id / a.heads;
    const int i0 = ti * BM, j0 = tj * BN;
    const int m_begin = s * a.rows_per_split;
    const int m_end = min(a.M, m_begin + a.rows_per_split);
    const long long ld_du = (long long)a.G * a.H, ld_x = a.H;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, wm = w >> 1, wn = w & 1;
    const int half = lane >> 5, l32 = lane & 31;
    const int c4 = tid & 31, rg = tid >> 5;
    // dh is a multiple of 64: a quad of channels is valid or not as a whole; an invalid one reads
    // the tile's first quad (valid memory) and counts as zeros
    const bool ok_a = i0 + 4 * c4 < a.dh, ok_b = j0 + 4 * c4 < a.dh;
    const AT *du = static_cast<const AT *>(a.du) + (long long)g * a.H + head * a.dh + i0 + (ok_a ? 4 * c4 : 0);
    const AT *x = static_cast<const AT *>(a.x) + head * a.dh + j0 + (ok_b ? 4 * c4 : 0);

    float sdb[4] = {0.0f, 0.0f, 0.0f, 0.0f}, unused[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    struct Stage {
        QuadRows<AT> a, b;
    };
    int m_next = m_begin;
    auto load_next = [&](Stage &r) {
        // past the end of the range the last step is fetched again and counts as zeros
        const bool real = m_next < m_end;
        const int m = (real ? m_next : m_next - BK) + 8 * rg;
        const int n_valid = real ? m_end - m : 0;      // rows of this thread's group that count
        r.a.load(du, ld_du, m, a.M - 1, ok_a ? n_valid : 0);
        r.b.load(x, ld_x, m, a.M - 1, ok_b ? n_valid : 0);
        if (real) m_next += BK;
    };
    auto store_stage = [&](int buf, const Stage &r) {
        if (buf < 0) return;
        u4v ca[4], cb[4];
        r.a.transpose(ca, sdb);
        r.b.transpose(cb, unused);
        // lane c4 stores its channels in the order ch = (i + c4 / 2) % 4: the eight neighbouring lanes
        // of a 16-byte store pass then hit eight different 16-byte bank groups
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ch = (i + (c4 >> 1)) & 3;
            const u4v va = ch == 0 ? ca[0] : ch == 1 ? ca[1] : ch == 2 ? ca[2] : ca[3];
            const u4v vb = ch == 0 ? cb[0] : ch == 1 ? cb[1] : ch == 2 ? cb[2] : cb[3];
            *reinterpret_cast<u4v *>(&s_a[buf][lds_off(4 * c4 + ch, rg)]) = va;
            *reinterpret_cast<u4v *>(&s_b[buf][lds_off(4 * c4 + ch, rg)]) = vb;
        }
    };
    f16v acc[2][2];
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.0f;

    const int nk = m_end > m_begin ? (m_end - m_begin + BK - 1) / BK : 0;
    int steps_done = 0;
    auto compute = [&](int buf) {
        mma_step<false>(s_a[buf], s_b[buf], wm, wn, l32, half, acc);
        ++steps_done;
    };
    auto done = [&]() { return steps_done >= nk; };
    if (nk > 0) {
        if constexpr (sizeof(AT) == 4) one_ahead<Stage>(load_next, store_stage, compute, done);
        else two_ahead<Stage>(load_next, store_stage, compute, done);
    }
    float *out = a.part + (((long long)s * a.G + g) * a.H + head * a.dh + i0) * a.dh + j0;
#pragma unroll
    for (int ni = 0; ni < 2; ++ni) {
        const int col = 64 * wn + 32 * ni + l32;
        if (j0 + col >= a.dh) continue;
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = 64 * wm + 32 * mi + acc_row(v, half);
                if (i0 + row < a.dh) out[(long long)row * a.dh + col] = acc[mi][ni][v];
            }
    }
    // column sums of du seen by this workgroup (the tj = 0 tiles cover every channel once)
    if (a.dbpart && tj == 0) {
#pragma unroll
        for (int ch = 0; ch < 4; ++ch) s_db[rg][4 * c4 + ch] = sdb[ch];
        __syncthreads();
        if (tid < BM && i0 + tid < a.dh) {
            float t = 0.0f;
#pragma unroll
            for (int q = 0; q < 8; ++q) t += s_db[q][tid];
            a.dbpart[((long long)s * a.G + g) * a.H + head * a.dh + i0 + tid] = t;
        }
    }
}

// ------------------------------- dWx and dbias, bf16 operands copied straight into LDS
// The same sums for bf16 storage and wide heads: 256 x 256 outputs per workgroup of eight waves
// (2 x 4; a wave owns 128 output channels i x 64 input channels j), 64 rows m per step, operand rows
// copied from memory to LDS as they are, 512 bytes of du and of x per row.
//
//   LDS      two stages of (64 + 64) rows x 512 bytes = 128 KB.  A copy instruction moves two rows;
//            16-byte chunk c of row r lies at position c ^ dw_swz(r) of its row.
//   reads    the products need, per lane, eight consecutive m of one channel: a column of the
//            stage.  ds_read_b64_tr_b16 hands a lane four of them: the sixteen lanes of a group read
//            8 bytes each, four lanes per row over four rows (32 bytes = 16 channels of a row), and
//            lane i of the group receives the i-th channel of the four rows.  With the chunk
//            positions above the four rows of a group lie in four different parts of the banks.
//   rows     past the end of a range lie beyond the buffer descriptor, which is rebuilt for every
//            step (base at the step's first row, extent to the end of the range): the copy writes
//            zeros for them, so they add nothing.  Tile columns past dh hold whatever follows in the
//            row (a neighbouring head or gate; zeros past the end of the tensor) and their sums are
//            not stored.
//   dbias    the column sums of du come from one more product per round, with an operand of ones,
//            in the tiles of the first column block; the wave with wn = mi does block mi.
namespace dwd {
constexpr int BT = 256, BK = 64;
constexpr int OP = BK * BT;              // bf16 elements of one operand's rows of a step
constexpr int STAGE = 2 * OP;            // du rows, then x rows
}  // namespace dwd

// position of 16-byte chunk c in stage row r: c ^ dw_swz(r).  Rows r .. r + 3 (r a multiple of four) get
// four different values both in bits 1-2 and in bits 2-3 of the chunk index: the four rows of a transposing
// read then lie in different 32-byte quarters of a 128-byte window and in different 64-byte quarters of a
// 256-byte window of the banks, whichever the LDS serves per cycle.
__device__ __forceinline__ int dw_swz(int row) { return (0xca60 >> (4 * (row & 3))) & 15; }       // 0, 6, 10, 12

typedef short s4v __attribute__((ext_vector_type(4)));
typedef short s8v __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) char *lds_char_ptr;
typedef __attribute__((address_space(3))) s4v *lds_s4v_ptr;

__global__ __launch_bounds__(512) void proj_dw_dma_kernel(const DwArgs a)
{
    constexpr int BT = dwd::BT, BK = dwd::BK, OP = dwd::OP, STAGE = dwd::STAGE;
    __shared__ __attribute__((aligned(16))) unsigned short s_op[2][STAGE];
    // Workgroups go to the eight XCDs round-robin and an XCD runs 32 of its contiguous range at a
    // time: the tiles of a (gate, head, range) are numbered in strips of four tile rows, down the strip's columns,
    // so that 32 consecutive ones cover 4 x 8 tiles (8 x panels, 4 du panels) where a head has that many.
    int id = (int)(blockIdx.x & 7) * a.per_xcd + (int)(blockIdx.x >> 3);
    if (id >= a.n_blocks) return;
    const int per_grid = a.tiles * a.tiles;
    const int in_grid = id % per_grid; id /= per_grid;
    const int strip = in_grid / (4 * a.tiles), in_strip = in_grid - strip * 4 * a.tiles;
    const int hs = min(4, a.tiles - 4 * strip);
    const int tj = in_strip / hs, ti = 4 * strip + in_strip % hs;
    const int g = id % a.G; id /= a.G;
    const int head = id % a.heads;
    const int s = id / a.heads;
    const int i0 = ti * BT, j0 = tj * BT;
    const int m_begin = s * a.rows_per_split;
    const int rows = min(a.M, m_begin + a.rows_per_split) - m_begin;
    const int nk = (rows + BK - 1) / BK;
    if (nk <= 0) return;
    const int tid = threadIdx.x, lane = tid & 63, w = (int)uniform((unsigned int)tid >> 6), wm = w >> 2, wn = w & 3;
    const int half = lane >> 5, l32 = lane & 31;
    const bool do_db = a.dbpart && tj == 0;

    // ---- the copying side: a wave copies rows 8 w .. 8 w + 7 of both operands' steps, two rows per instruction
    const long long ld_du = (long long)a.G * a.H, ld_x = a.H;
    const long long col_du = (long long)g * a.H + head * a.dh + i0, col_x = (long long)head * a.dh + j0;
    unsigned long long p_du = (unsigned long long)(static_cast<const unsigned short *>(a.du) + (long long)m_begin * ld_du + col_du);
    unsigned long long p_x = (unsigned long long)(static_cast<const unsigned short *>(a.x) + (long long)m_begin * ld_x + col_x);
    // bytes from there that belong to the range: whole rows, and the tile's columns of the last one
    long long rem_du = ((long long)(rows - 1) * ld_du + min((long long)BT, ld_du - col_du)) * 2;
    long long rem_x = ((long long)(rows - 1) * ld_x + min((long long)BT, ld_x - col_x)) * 2;
    unsigned int va[4], vb[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int row = 8 * w + 2 * j + (lane >> 5);
        const unsigned int chunk = (unsigned int)((lane & 31) ^ dw_swz(row));
        va[j] = (unsigned int)row * (unsigned int)ld_du * 2u + chunk * 16u;
        vb[j] = (unsigned int)row * (unsigned int)ld_x * 2u + chunk * 16u;
    }
    const unsigned int lds_op = lds_address(&s_op[0][0]);
    const lds_char_ptr lds_zero = (lds_char_ptr)&s_op[0][0] - lds_op;       // LDS address 0, as a pointer
    auto words = [&](unsigned long long p, long long rem) {
        const unsigned int n = rem <= 0 ? 0u : rem > 0xffffffffll ? 0xffffffffu : (unsigned int)rem;
        const u4v r = {uniform((unsigned int)p), uniform((unsigned int)(p >> 32) & 0xffffu), uniform(n), 0x27000u};
        return r;
    };
    auto issue = [&](int buf) {
        const u4v ra = words(p_du, rem_du), rb = words(p_x, rem_x);
        const unsigned int dst = lds_op + (unsigned int)buf * (STAGE * 2u) + (unsigned int)(8 * w) * (BT * 2u);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            copy_to_lds_16(dst + (unsigned int)j * (2u * BT * 2u), ra, va[j], 0u);
            copy_to_lds_16(dst + OP * 2u + (unsigned int)j * (2u * BT * 2u), rb, vb[j], 0u);
        }
        p_du += (unsigned long long)(BK * ld_du * 2); rem_du -= BK * ld_du * 2;
        p_x += (unsigned long long)(BK * ld_x * 2);   rem_x -= BK * ld_x * 2;
    };

    // ---- the multiplying side
    // this lane's place in a transposing read: row rr of the four, the 8 bytes at channel 16 hi + 4 (lane % 4) of
    // the 32-channel block.  The block's first chunk is a multiple of four and the lane's chunk within the block
    // is 2 hi + lo, so its position is (block chunk ^ high bits of the row's mask) + ((2 hi + lo) ^ low bits):
    // one lane offset per value of the block chunk's bits 2-3.
    const int rr = (lane & 15) >> 2, mask = dw_swz(rr);
    const int in_block = (2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ (mask & 3);
    const unsigned int rowpart = (unsigned int)(8 * half + rr) * (BT * 2u) + (unsigned int)(lane & 1) * 8u;
    unsigned int o_du[4], o_x[2];
#pragma unroll
    for (int mi = 0; mi < 4; ++mi)
        o_du[mi] = lds_op + rowpart + (unsigned int)(((16 * wm + 4 * mi) ^ (mask & 12)) + in_block) * 16u;
#pragma unroll
    for (int nj = 0; nj < 2; ++nj)
        o_x[nj] = lds_op + OP * 2u + rowpart + (unsigned int)(((8 * wn + 4 * nj) ^ (mask & 12)) + in_block) * 16u;
    auto read8 = [&](unsigned int addr) {
        const s4v q0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v_ptr)(lds_zero + addr));
        const s4v q1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v_ptr)(lds_zero + addr + 4u * BT * 2u));
        const s8v t = __builtin_shufflevector(q0, q1, 0, 1, 2, 3, 4, 5, 6, 7);
        return __builtin_bit_cast(bf8v, t);
    };
    auto read_frags = [&](int buf, int kb, bf8v (&fd)[4], bf8v (&fx)[2]) {
        const unsigned int base = (unsigned int)buf * (STAGE * 2u) + (unsigned int)(16 * kb) * (BT * 2u);
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) fd[mi] = read8(o_du[mi] + base);
#pragma unroll
        for (int nj = 0; nj < 2; ++nj) fx[nj] = read8(o_x[nj] + base);
    };
    f16v acc[2][4], accdb;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        accdb[v] = 0.0f;
#pragma unroll
        for (int nj = 0; nj < 2; ++nj)
#pragma unroll
            for (int mi = 0; mi < 4; ++mi) acc[nj][mi][v] = 0.0f;
    }
    const __bf16 one = (__bf16)1.0f;
    const bf8v ones = {one, one, one, one, one, one, one, one};
    // acc[nj][mi] = (x columns)^T (du columns): a lane owns channel l32 of the du block and, per four
    // registers, four consecutive channels of x
    auto multiply = [&](const bf8v (&fd)[4], const bf8v (&fx)[2]) {
#pragma unroll
        for (int mi = 0; mi < 4; ++mi) {
#pragma unroll
            for (int nj = 0; nj < 2; ++nj)
                acc[nj][mi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fx[nj], fd[mi], acc[nj][mi], 0, 0, 0);
            if (do_db && wn == mi) accdb = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, fd[mi], accdb, 0, 0, 0);
        }
    };

    // ---- two steps on their way, the first one landed
    issue(0);
    if (nk > 1) {
        issue(1);
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");   // the eight copies of the second step may be outstanding
    } else {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    asm volatile("s_barrier" ::: "memory");
    bf8v fd0[4], fx0[2], fd1[4], fx1[2];
    read_frags(0, 0, fd0, fx0);
    for (int T = 0; T < nk; ++T) {
        const int buf = T & 1;
        read_frags(buf, 1, fd1, fx1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(fd0, fx0);
        __builtin_amdgcn_sched_barrier(0);
        read_frags(buf, 2, fd0, fx0);
        __builtin_amdgcn_sched_barrier(0);
        multiply(fd1, fx1);
        __builtin_amdgcn_sched_barrier(0);
        read_frags(buf, 3, fd1, fx1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(fd0, fx0);
        __builtin_amdgcn_sched_barrier(0);
        // own copies of step T + 1 (the only memory operations outstanding) have landed, own reads of this
        // stage are done; after the barrier everybody's
        asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        read_frags(buf ^ 1, 0, fd0, fx0);                  // after the last step: stale rows, not used
        if (T + 2 < nk) issue(buf);
        __builtin_amdgcn_sched_barrier(0);
        multiply(fd1, fx1);
        __builtin_amdgcn_sched_barrier(0);
    }

    float *out = a.part + (((long long)s * a.G + g) * a.H + (long long)head * a.dh) * a.dh;
#pragma unroll
    for (int mi = 0; mi < 4; ++mi) {
        const int i = i0 + 128 * wm + 32 * mi + l32;
        if (i >= a.dh) continue;
#pragma unroll
        for (int nj = 0; nj < 2; ++nj)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int j = j0 + 64 * wn + 32 * nj + 8 * q + 4 * half;       // dh is a multiple of 4
                if (j >= a.dh) continue;
                const f4v o = {acc[nj][mi][4 * q], acc[nj][mi][4 * q + 1], acc[nj][mi][4 * q + 2], acc[nj][mi][4 * q + 3]};
                *reinterpret_cast<f4v *>(out + (long long)i * a.dh + j) = o;
            }
    }
    if (do_db && half == 0) {
        // every row of the product with ones holds the column sums
        const int i = i0 + 128 * wm + 32 * wn + l32;
        if (i < a.dh) a.dbpart[((long long)s * a.G + g) * a.H + (long long)head * a.dh + i] = accdb[0];
    }
}

// ------------------------------- dWx and dbias of narrow heads: a whole gate of a head per workgroup
// The same sums for heads of at most 256 channels: a workgroup holds all d_h x d_h sums of one gate of one head over a
// range of rows, so that du is read once and x once per gate, and no part of a tile lies idle (wider heads: below).  Rows go to LDS as they
// are, NS steps deep.  A wave owns IB x JB blocks of 32 x 32 sums; MS waves share a part and take the 16-row slices of a
// step in turn, their sums are added at the end.
//
//   bf16     columns come out of the stage by transposing reads, as above; chunk c of row r lies at c ^ DwRows::swz(r): within
//            128 bytes where a row is an odd number of those, for dw_swz does not fit it
//   fp32     a lane reads its channel of eight rows, 32 neighbouring channels at a time, and rounds them
//   dbias    is added up from the fragments of du (unrounded in fp32; eight rows before they join the sum); the waves that share a part's du blocks take one each
//   tiles    heads of more than 256 in four of half a head, 160 to 256 wide: no part of a tile idle, and du and x read twice, through the
//            L2 of one XCD; of three gates 15000 x 320 in fp32 60 -> 40 us, 60000 x 320 159 -> 119, four gates of two heads 15000 x 384
//            136 -> 86, bf16 142 -> 85 (four heads of 320), 160 -> 92 (of 384), fp32 448 and 512 (60000 x one head, three gates) 249 -> 214, 269 -> 226.  Bound by the
//            reads from LDS and the conversions of a 16-row slice, which nothing else of the wave overlaps
//   bound    by memory, and where ranges are many by their sums: three gates, 65536 x 512 in heads of 64, bf16: 110 -> 55 us (4.9 TB/s);
//            40000 x 512 in heads of 128, four gates: 67 -> 41; fp32: 16000 x 1024 in heads of 256 117 -> 100, 6993 x 768 in
//            heads of 192, four gates: 57 -> 35, of which the sums of 16 ranges, written and added, are half
template <typename AT, int NB> struct DwRows {              // tiles of 32 NB channels
    static constexpr int E = sizeof(AT), K = 32 * NB, ROW = K * E;
    static constexpr bool ODD = NB & 1;
    static constexpr int MS = NB == 2 ? (E == 2 ? 8 : 4) : NB == 4 ? 2 : 1;
    static constexpr int IB = ODD ? NB : NB >= 6 ? NB / 2 : 2, JB = ODD ? 1 : 2, WI = NB / IB, WJ = NB / JB, WAVES = MS * WI * WJ;
    static constexpr int R = E == 2 ? (NB == 2 ? 128 : NB == 4 ? 64 : 32) : (NB == 2 ? 64 : NB >= 7 ? 16 : 32);
    static constexpr int OP = R * ROW, STAGE = 2 * OP, NS = STAGE >= 40 * 1024 ? 3 : 4;
    static constexpr int N = OP / 1024 / WAVES;             // copies of each operand of a wave per step
    static constexpr int SLICES = R / 16 / MS;              // of a wave per step
    static constexpr int DB = (IB + WJ - 1) / WJ;           // du blocks of which a wave adds up the rows
    static_assert(N * 1024 * WAVES == OP && SLICES >= 1 && (MS == 1 || WAVES * 16384 <= NS * STAGE), "");
    // (rows of an odd number of 64 bytes lie in different parts of the banks by themselves)
    static __device__ __forceinline__ int swz(int row) { return E == 4 || ODD ? 0 : (NB & 2) ? 2 * (row & 3) : dw_swz(row); }
};

template <typename AT, int NB> __global__ __launch_bounds__((64 * DwRows<AT, NB>::WAVES)) void proj_dw_rows_kernel(const DwArgs a)
{
    typedef DwRows<AT, NB> S;
    constexpr int E = S::E, K = S::K, R = S::R, ROW = S::ROW, NS = S::NS, N = S::N, IB = S::IB, JB = S::JB, MS = S::MS, DB = S::DB;
    __shared__ __attribute__((aligned(16))) unsigned char s_op[NS * S::STAGE];
    __shared__ float s_db[MS][K];
    // numbered as above: the tiles and gates of a (head, range) on one XCD at a time
    int id = (int)(blockIdx.x & 7) * a.per_xcd + (int)(blockIdx.x >> 3);
    if (id >= a.n_blocks) return;
    const int tj = id % a.tiles; id /= a.tiles;
    const int ti = id % a.tiles; id /= a.tiles;
    const int g = id % a.G; id /= a.G;
    const int head = id % a.heads;
    const int s = id / a.heads;
    const int m_begin = s * a.rows_per_split;
    const int rows = min(a.M, m_begin + a.rows_per_split) - m_begin;
    if (rows <= 0) return;
    const int nk = (rows + R - 1) / R;
    const int tid = threadIdx.x, lane = tid & 63, w = (int)uniform((unsigned int)tid >> 6);
    const int ms = w % MS, part = w / MS, wi = part % S::WI, wj = part / S::WI;
    const int half = lane >> 5, l32 = lane & 31;
    const unsigned int lds_op = lds_address(s_op);

    // ---- the copying side
    const long long ld_du = (long long)a.G * a.H * E, ld_x = (long long)a.H * E;
    unsigned long long p_du = (unsigned long long)a.du + (unsigned long long)(m_begin * ld_du + ((long long)g * a.H + head * a.dh + ti * K) * E);
    unsigned long long p_x = (unsigned long long)a.x + (unsigned long long)(m_begin * ld_x + ((long long)head * a.dh + tj * K) * E);
    int left = rows;
    unsigned int va[N], vb[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int byte = (w * N + j) * 1024 + lane * 16, row = byte / ROW, c = (byte % ROW / 16) ^ S::swz(row);
        va[j] = (unsigned int)row * (unsigned int)ld_du + (unsigned int)c * 16u;
        vb[j] = (unsigned int)row * (unsigned int)ld_x + (unsigned int)c * 16u;
    }
    auto issue = [&](int stage) {
        // rows past the end of the range lie beyond the descriptors: the copy writes zeros for them
        const int n = min(left, R);
        const u4v ra = {uniform((unsigned int)p_du), uniform((unsigned int)(p_du >> 32) & 0xffffu), uniform(n > 0 ? (unsigned int)((n - 1) * ld_du + ROW) : 0u), 0x27000u};
        const u4v rb = {uniform((unsigned int)p_x), uniform((unsigned int)(p_x >> 32) & 0xffffu), uniform(n > 0 ? (unsigned int)((n - 1) * ld_x + ROW) : 0u), 0x27000u};
        const unsigned int dst = lds_op + (unsigned int)stage * S::STAGE + (unsigned int)(w * N) * 1024u;
#pragma unroll
        for (int j = 0; j < N; ++j) {
            copy_to_lds_16(dst + (unsigned int)j * 1024u, ra, va[j], 0u);
            copy_to_lds_16(dst + S::OP + (unsigned int)j * 1024u, rb, vb[j], 0u);
        }
        p_du += (unsigned long long)(R * ld_du);
        p_x += (unsigned long long)(R * ld_x);
        left -= R;
    };

    // ---- the multiplying side
    const int rr = (lane & 15) >> 2, mask = S::swz(rr);
    const unsigned int in_block = (unsigned int)((2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ (mask & 3));
    const lds_char_ptr lds_zero = (lds_char_ptr)s_op - lds_op;                     // LDS address 0, as a pointer
    auto place = [&](int block) {                                                  // of this lane's first element of a 32-channel block, in a slice
        if constexpr (E == 2) return (unsigned int)(8 * half + rr) * ROW + (unsigned int)(lane & 1) * 8u + (((unsigned int)(4 * block) ^ (unsigned int)(mask & 12)) + in_block) * 16u;
        else return (unsigned int)(8 * half) * ROW + (unsigned int)(32 * block + l32) * 4u;
    };
    unsigned int o_du[IB], o_x[JB];
#pragma unroll
    for (int i = 0; i < IB; ++i) o_du[i] = lds_op + place(IB * wi + i);
#pragma unroll
    for (int j = 0; j < JB; ++j) o_x[j] = lds_op + S::OP + place(JB * wj + j);
    float sdb[DB];
#pragma unroll
    for (int d = 0; d < DB; ++d) sdb[d] = 0.0f;
    auto read8 = [&](unsigned int addr, float *sum) {
        bf8v f;
        if constexpr (E == 2) {
            const s4v q0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v_ptr)(lds_zero + addr));
            const s4v q1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4v_ptr)(lds_zero + addr + 4u * ROW));
            f = __builtin_bit_cast(bf8v, __builtin_shufflevector(q0, q1, 0, 1, 2, 3, 4, 5, 6, 7));
            if (sum) *sum += (((float)f[0] + (float)f[1]) + ((float)f[2] + (float)f[3])) + (((float)f[4] + (float)f[5]) + ((float)f[6] + (float)f[7]));
        } else {
            Raw8f r;
#pragma unroll
            for (int q = 0; q < 8; ++q) (q < 4 ? r.lo : r.hi)[q & 3] = *(const __attribute__((address_space(3))) float *)(lds_zero + addr + (unsigned int)q * ROW);
            if (sum) *sum += ((r.lo[0] + r.lo[1]) + (r.lo[2] + r.lo[3])) + ((r.hi[0] + r.hi[1]) + (r.hi[2] + r.hi[3]));
            f = __builtin_bit_cast(bf8v, to_bf16x8(r));
        }
        return f;
    };
    const bool do_db = a.dbpart && tj == 0;
    f16v acc[JB][IB];
#pragma unroll
    for (int j = 0; j < JB; ++j)
#pragma unroll
        for (int i = 0; i < IB; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[j][i][v] = 0.0f;
    // Sums of 512 rows of a wave at a time, added up: a range here is up to four times as long as with the smaller tiles, and one
    // chain of roundings over it would be less exact.  Tiles of 224 and more have no registers for it; their ranges are no longer.
    constexpr bool TWO = NB < 7;
    f16v sum[TWO ? JB : 1][TWO ? IB : 1];
    if constexpr (TWO) {
#pragma unroll
        for (int j = 0; j < JB; ++j)
#pragma unroll
            for (int i = 0; i < IB; ++i) sum[j][i] = acc[j][i];
    }
    auto add_up = [&]() {
        if constexpr (TWO) {
#pragma unroll
            for (int j = 0; j < JB; ++j)
#pragma unroll
                for (int i = 0; i < IB; ++i)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        sum[j][i][v] += acc[j][i][v];
                        acc[j][i][v] = 0.0f;
                    }
        }
    };

#pragma unroll
    for (int q = 0; q < NS - 1; ++q) issue(q);
    int stage = 0;
    for (int T = 0; T < nk; ++T) {
        // own copies of this step have landed, behind them only those of the steps after it; after the barrier everybody's, and everybody
        // has read the stage before it
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(2 * N * (NS - 2)) : "memory");
        issue(stage == 0 ? NS - 1 : stage - 1);
#pragma unroll
        for (int sl = 0; sl < S::SLICES; ++sl) {
            const unsigned int at = (unsigned int)stage * S::STAGE + (unsigned int)(sl * MS + ms) * (16u * ROW);
            bf8v fd[IB], fx[JB];
#pragma unroll
            for (int j = 0; j < JB; ++j) fx[j] = read8(o_x[j] + at, nullptr);
#pragma unroll
            for (int i = 0; i < IB; ++i) fd[i] = read8(o_du[i] + at, nullptr);
#pragma unroll
            for (int i = 0; i < IB; ++i)
#pragma unroll
                for (int j = 0; j < JB; ++j) acc[j][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fx[j], fd[i], acc[j][i], 0, 0, 0);
            if (do_db) {
#pragma unroll
                for (int i = 0; i < IB; ++i)
                    if (i % S::WJ == wj || S::WJ == 1) (void)read8(o_du[i] + at, &sdb[i / S::WJ]);
            }
        }
        if (TWO && (T + 1) % (32 / S::SLICES) == 0) add_up();
        stage = stage + 1 == NS ? 0 : stage + 1;
    }
    // nothing is on its way into the stages any more
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if constexpr (TWO) {
        add_up();
#pragma unroll
        for (int j = 0; j < JB; ++j)
#pragma unroll
            for (int i = 0; i < IB; ++i) acc[j][i] = sum[j][i];
    }

    float *out = a.part + (((long long)s * a.G + g) * a.H + (long long)head * a.dh + ti * K) * a.dh + tj * K;
    auto put = [&](int i, int j, int q, const f4v &o) {
        const int row = 32 * (IB * wi + i) + l32, col = 32 * (JB * wj + j) + 8 * q + 4 * half;
        *reinterpret_cast<f4v *>(out + (long long)row * a.dh + col) = o;
    };
    if constexpr (MS > 1) {
        // the sums of the waves that share a part, [part][wave][four of its 64 registers][lane]; each wave adds up a share
        static_assert(IB * JB == 4, "");
        f4v *mine = reinterpret_cast<f4v *>(s_op) + (part * MS + ms) * (16 * 64) + lane;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const f16v &v = acc[q / 4 % JB][q / 4 / JB];
            const f4v o = {v[4 * (q % 4)], v[4 * (q % 4) + 1], v[4 * (q % 4) + 2], v[4 * (q % 4) + 3]};
            mine[q * 64] = o;
        }
        __syncthreads();
        const f4v *all = reinterpret_cast<const f4v *>(s_op) + part * MS * (16 * 64) + lane;
#pragma unroll
        for (int k = 0; k < 16 / MS; ++k) {
            const int q = ms * (16 / MS) + k;
            f4v o = all[q * 64];
#pragma unroll
            for (int r = 1; r < MS; ++r) o += all[(r * 16 + q) * 64];
            put(q / 4 / JB, q / 4 % JB, q % 4, o);
        }
    } else {
#pragma unroll
        for (int i = 0; i < IB; ++i)
#pragma unroll
            for (int j = 0; j < JB; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f4v o = {acc[j][i][4 * q], acc[j][i][4 * q + 1], acc[j][i][4 * q + 2], acc[j][i][4 * q + 3]};
                    put(i, j, q, o);
                }
    }
    if (do_db) {
#pragma unroll
        for (int d = 0; d < DB; ++d) {
            const float t = sdb[d] + __shfl_xor(sdb[d], 32);
            const int i = d * S::WJ + (S::WJ == 1 ? 0 : wj);
            if (half == 0 && i < IB) s_db[ms][32 * (IB * wi + i) + l32] = t;
        }
        __syncthreads();
        for (int c = tid; c < K; c += 64 * S::WAVES) {
            float t = 0.0f;
#pragma unroll
            for (int r = 0; r < MS; ++r) t += s_db[r][c];
            a.dbpart[((long long)s * a.G + g) * a.H + (long long)head * a.dh + ti * K + c] = t;
        }
    }
}

// ------------------------------------------------------------- weight copies
// Wb = bf16(Wx), same layout [G][H][dh]; n4 fours
__global__ __launch_bounds__(256) void proj_wb_kernel(const float *Wx, unsigned short *Wb, size_t n4, int *tickets)
{
    if (blockIdx.x == 0 && threadIdx.x < 8) tickets[threadIdx.x] = 0;      // for the product that follows
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += (size_t)gridDim.x * blockDim.x)
        store4(Wb + 4 * i, reinterpret_cast<const f4v *>(Wx)[i]);
}

// Wt[head][j][g dh + i] = bf16(Wx[g][head dh + i][j]): the B operand of the dx product.  One workgroup per 64 x 64 block
// of a head's matrix (dh is a multiple of 64), transposed through LDS so that memory is read and written in whole lines:
// 21 (43) -> 6 (8) us for 4 (8) million weights; read element by element along a column, a line was fetched several times.
constexpr int WT_PITCH = 36;             // dwords from one row of the LDS block to the next: 32 pairs and a pad of 16 bytes
__global__ __launch_bounds__(256) void proj_wt_kernel(const float *Wx, unsigned short *Wt, int G, int H, int dh,
                                                      int *tickets)
{
    __shared__ __attribute__((aligned(16))) unsigned int s_t[64 * WT_PITCH];      // [j][pair of i], bf16
    if (blockIdx.x == 0 && threadIdx.x < 8) tickets[threadIdx.x] = 0;      // for the product that follows
    const int nb = dh / 64;
    const int jb = blockIdx.x % nb, ib = (blockIdx.x / nb) % nb, gh = blockIdx.x / (nb * nb);
    const int g = gh % G, head = gh / G;
    const float *src = Wx + ((size_t)g * H + (size_t)head * dh + 64 * ib) * dh + 64 * jb;
    const int c = threadIdx.x & 15, r = threadIdx.x >> 4;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int p = r + 16 * q;                                           // rows 2 p and 2 p + 1, columns 4 c .. 4 c + 3
        const f4v v0 = *reinterpret_cast<const f4v *>(src + (size_t)(2 * p) * dh + 4 * c);
        const f4v v1 = *reinterpret_cast<const f4v *>(src + (size_t)(2 * p + 1) * dh + 4 * c);
#pragma unroll
        for (int k = 0; k < 4; ++k) s_t[(4 * c + k) * WT_PITCH + p] = pack2(v0[k], v1[k]);
    }
    __syncthreads();
    unsigned short *dst = Wt + ((size_t)head * dh + 64 * jb) * ((size_t)G * dh) + (size_t)g * dh + 64 * ib;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int j = (threadIdx.x >> 3) + 32 * q, ch = threadIdx.x & 7;
        *reinterpret_cast<u4v *>(dst + (size_t)j * ((size_t)G * dh) + 8 * ch) = *reinterpret_cast<const u4v *>(&s_t[j * WT_PITCH + 4 * ch]);
    }
}

size_t r256(size_t x) { return (x + 255) & ~(size_t)255; }

int g_proj_dma = 1;        // bf16 NT products use the copy-to-LDS kernel where it applies (proj_set_dma)

bool shapes_ok(int dtype, int B, int L, int H, int G, int n_heads)
{
    if (dtype != PARARNN_F32 && dtype != PARARNN_BF16) return false;
    if (B < 1 || L < 1 || H < 1 || G < 1 || G > 8 || n_heads < 1 || H % n_heads) return false;
    const double rows = (double)B * (double)L;
    return rows < 2.0e9 && rows * G * H < 3.0e10;
}

// up to this many rows are one range: a second one would save four steps (5 us) and cost a launch that adds the two
constexpr int dw_one_range = 8 * BK;

// row ranges of the dWx reduction: enough workgroups to fill the device, whole 64-row steps
void dw_split(int M, int base_tiles, int *S, int *rows_per_split)
{
    int want = (2048 + base_tiles - 1) / base_tiles;
    if (want < 1) want = 1;
    if (want > 64) want = 64;
    int rps = (M + want - 1) / want;
    rps = (rps + BK - 1) / BK * BK;
    if (rps < 4 * BK) rps = 4 * BK;
    if (M <= dw_one_range) rps = (M + BK - 1) / BK * BK;
    *rows_per_split = rps;
    *S = (M + rps - 1) / rps;
}

// The same for the copy-to-LDS kernel, one workgroup per compute unit: the number of ranges with the least
// estimated time, from the rounds of workgroups the device needs (a step of a 256 x 256 tile takes a compute
// unit about 2.3 us, a workgroup's start and output tile about 6 us) and the partial sums that have to be
// written and read again (about 4 TB/s); at least four steps per range.
void dw_dma_split(int M, int G, int H, int dh, int n_heads, int *S, int *rows_per_split)
{
    const int cus = device_cu_count() > 0 ? device_cu_count() : 256;
    const int tiles = (dh + dwd::BT - 1) / dwd::BT;
    const long long base_tiles = (long long)tiles * tiles * G * n_heads;
    const double nw = (double)G * H * dh;
    int best = 1;
    double best_us = 0.0;
    for (int s = 1; s <= 64; ++s) {
        int rps = (M + s - 1) / s;
        rps = (rps + dwd::BK - 1) / dwd::BK * dwd::BK;
        if (s > 1 && rps < 4 * dwd::BK) break;
        const int ranges = (M + rps - 1) / rps;
        const long long rounds = (base_tiles * ranges + cus - 1) / cus;
        const double us = (double)rounds * ((double)(rps / dwd::BK) * 2.3 + 6.0) + (ranges > 1 ? (double)ranges * nw * 8.0 / 4.0e6 : 0.0);
        if (s == 1 || us < best_us) { best_us = us; best = ranges; }
    }
    int rps = (M + best - 1) / best;
    rps = (rps + dwd::BK - 1) / dwd::BK * dwd::BK;
    *rows_per_split = rps;
    *S = (M + rps - 1) / rps;
}

// the copy-to-LDS kernel's 256-wide tiles against the 128-wide ones: taken where they cover dh with at most
// half as much again of idle tile area, and where the 128-wide ones are not all on the device at once in a single range
// (256 rows: 16 -> 11 us)
bool dw_dma_shape_ok(int M, int H, int G, int dh)
{
    const double t2 = (double)((dh + dwd::BT - 1) / dwd::BT * dwd::BT), t1 = (double)((dh + BM - 1) / BM * BM);
    return dh % 8 == 0 && H % 8 == 0 && (long long)G * H < (1 << 22) && t2 * t2 <= 1.5 * t1 * t1 &&
           !(M <= dw_one_range && (double)G * H / dh * (t1 / BM) * (t1 / BM) <= 2.0 * device_cu_count());
}

// The narrow-head kernel against the tiles of 128 and 256.  Up to 512 rows the tiles are one range and need no second launch
// (9 us against 10-26).  bf16: at least level from 600 rows on, up to 2.4 times faster, but for heads of 256, where the 256-wide tiles do the
// same.  fp32: more sums have to be written and added, for a range is all of a compute unit's work, and that pays
// with enough rows: by gates x heads x rows, heads of 128 and 192 24000 0.9-1.05 times as fast, 48000 1.1-1.2, a million
// 1.6; of 256, 96000 0.94, 128000 to a million 1.1-1.2; of 64, level at 600 rows; one or two gates in all never.
// Heads of 320 to 512 in four tiles of half a head, of the time with the tiles of 128 (bf16 from 448 on: those of 256, which are
// full), by gates x heads x rows: bf16 320 and 384 5000 0.98-1.09, 12000 0.89-1.02, 18000 0.77-0.8, 32000 and more 0.54-0.68; fp32 7000
// 1.03-1.2, 12000 0.99-1.06, 18000 0.88-0.92, 32000 and more 0.63-0.84; fp32 448 and 512 18000 1.17-1.2, 48000 0.94-1.08, 120000 and more 0.81-0.9.
int dw_rows_tiles(int dh) { return dh > 256 ? 2 : 1; }
bool dw_rows_shape_ok(int M, int H, int G, int dh, bool bf)
{
    if (dh % 64 || dh > 512 || M <= dw_one_range || (long long)G * H >= (1 << 22)) return false;
    const int units = G * (H / dh);
    if (dh > 256) return (bf ? dh <= 384 : true) && (double)units * M >= (bf ? 12000.0 : dh <= 384 ? 15000.0 : 60000.0);
    if (bf) return dh < 256;
    return dh == 64 || (units >= 3 && (double)units * M >= (dh == 256 ? 120000.0 : 40000.0));
}

// The ranges of the narrow-head kernel, one workgroup per compute unit: estimated as above, with 23 GB/s of rows per workgroup.
void dw_rows_split(int M, int G, int H, int dh, int n_heads, bool bf, int least, int *S, int *rows_per_split)
{
    const int cus = device_cu_count() > 0 ? device_cu_count() : 256;
    const int tiles = dw_rows_tiles(dh), width = dh / tiles;
    const int R = bf ? (dh == 64 ? 128 : dh == 128 ? 64 : 32) : (dh == 64 ? 64 : width >= 224 ? 16 : 32);
    const int units = G * n_heads * tiles * tiles;
    const double nw = (double)G * H * dh, row_us = 2.0 * width * (bf ? 2 : 4) / 23e3;
    double best_us = 0.0;
    if (width < 224) least = 1;                         // (wider tiles: no longer ranges than the smaller ones have)
    for (int s = least; s <= 96; ++s) {
        int rps = (M + s - 1) / s;
        rps = (rps + R - 1) / R * R;
        const int ranges = (M + rps - 1) / rps;
        const long long rounds = ((long long)units * ranges + cus - 1) / cus;
        const double us = (double)rounds * (rps * row_us + 6.0) + (ranges > 1 ? 3.0 + (double)ranges * nw * 8.0 / 4.0e6 : 0.0);
        if (s == least || us < best_us) { best_us = us; *rows_per_split = rps; *S = ranges; }
    }
}

struct ProjLayout {
    size_t off_tickets, off_w, off_part, off_db, total;
    int S, rows_per_split, tiles;
    int S3, rows_per_split3;               // the narrow-head dWx kernel's ranges (S3 = 0: not offered)
    int S2, rows_per_split2, tiles2;       // the copy-to-LDS dWx kernel's ranges and 256-wide tiles (S2 = 0: not offered)
};

ProjLayout proj_layout(int dtype, int B, int L, int H, int G, int n_heads, int backward)
{
    ProjLayout lo;
    const int dh = H / n_heads;
    const size_t nw = (size_t)G * H * dh;
    size_t off = 0;
    lo.off_tickets = off; off += 256;
    lo.off_w = off; off += r256(nw * sizeof(unsigned short));
    lo.tiles = (dh + BM - 1) / BM;
    lo.S = 0; lo.rows_per_split = 0;
    lo.S2 = 0; lo.rows_per_split2 = 0; lo.tiles2 = 0;
    lo.S3 = 0; lo.rows_per_split3 = 0;
    lo.off_part = lo.off_db = off;
    if (backward) {
        dw_split(B * L, lo.tiles * lo.tiles * G * n_heads, &lo.S, &lo.rows_per_split);
        // room for either kernel's partial sums, so that the size does not depend on proj_set_dma
        if (dw_dma_shape_ok(B * L, H, G, dh)) {
            lo.tiles2 = (dh + dwd::BT - 1) / dwd::BT;
            dw_dma_split(B * L, G, H, dh, n_heads, &lo.S2, &lo.rows_per_split2);
        }
        if (dw_rows_shape_ok(B * L, H, G, dh, dtype == PARARNN_BF16)) dw_rows_split(B * L, G, H, dh, n_heads, dtype == PARARNN_BF16, lo.S, &lo.S3, &lo.rows_per_split3);
        size_t s_max = (size_t)(lo.S > lo.S2 ? lo.S : lo.S2);
        if ((size_t)lo.S3 > s_max) s_max = (size_t)lo.S3;
        lo.off_part = off; off += r256(s_max * nw * sizeof(float));
        lo.off_db = off;   off += r256(s_max * G * H * sizeof(float));
    }
    lo.total = off < 256 ? 256 : off;
    return lo;
}

template <typename AT, typename CT> hipError_t launch_nt(GemmArgs &g, hipStream_t st)
{
    g.tiles_m = (g.M + BM - 1) / BM;
    g.tiles_n = (g.N + BN - 1) / BN;
    // two workgroups per compute unit (their LDS and registers allow no more), the same number on every XCD
    int slots = 2 * device_cu_count() / 8;
    if (slots < 1) slots = 1;
    if (slots > 64) slots = 64;                      // a patch of tiles has 64 members
    if (g.bias) hipLaunchKernelGGL((proj_gemm_nt_kernel<AT, CT, true>), dim3((unsigned)(8 * slots)), dim3(256), 0, st, g);
    else hipLaunchKernelGGL((proj_gemm_nt_kernel<AT, CT, false>), dim3((unsigned)(8 * slots)), dim3(256), 0, st, g);
    return hipGetLastError();
}

// Few output tiles: with the 128-wide ones all of them run at once, two to a compute unit at most, and a step of a tile
// takes half the time of a 256-wide one, which leaves three of four compute units idle (512 rows, dh = 512, four gates:
// dx 50 -> 38 us in bf16, 69 -> 44 in fp32 storage).  Two to a unit cost bf16 tiles of a few steps what the size gains
// (K = 768: 28 -> 30 us, K = 1024 and more: faster).
bool nt_few_tiles(const GemmArgs &g, bool bf)
{
    const long long tiles = (long long)((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN) * g.n_batch;
    const int cus = device_cu_count();
    return tiles <= cus || (tiles <= 2 * cus && (!bf || g.K >= 1024));
}

// the copy-to-LDS kernel: bf16 storage, at least two 64-k steps per tile, k-segments in whole steps, row
// offsets of a 256-row tile within 32 bits
bool nt_dma_ok(const GemmArgs &g)
{
    return !nt_few_tiles(g, true) && g.K >= 2 * dma::BK && g.K % dma::BK == 0 && g.kseg % dma::BK == 0 && g.N % 64 == 0 &&
           g.lda < (1 << 22) && g.ldb < (1 << 22) && g.ldc < (1 << 22) && g.lda % 8 == 0 && g.ldb % 8 == 0 && g.ldc % 8 == 0;
}

// the same for fp32 A and C: 32-k steps
bool nt_dma_f32_ok(const GemmArgs &g)
{
    return !nt_few_tiles(g, false) && g.K >= 3 * dmaf::BK && g.K % dmaf::BK == 0 && g.kseg % dmaf::BK == 0 && g.N % 64 == 0 &&
           g.lda < (1 << 22) && g.ldb < (1 << 22) && g.ldc < (1 << 22) && g.lda % 4 == 0 && g.ldb % 8 == 0 && g.ldc % 4 == 0;
}

hipError_t launch_nt_dma_f32(GemmArgs &g, hipStream_t st)
{
    g.tiles_m = (g.M + dma::BM - 1) / dma::BM;
    g.tiles_n = (g.N + dma::BN - 1) / dma::BN;
    int slots = device_cu_count() / 8;
    if (slots < 1) slots = 1;
    if (slots > 64) slots = 64;
    const long long per_wg = ((long long)(g.tiles_m + 7) / 8) * g.tiles_n * g.n_batch / slots;
    g.draw = per_wg >= 32 ? 4 : per_wg >= 16 ? 2 : 1;
    if (g.bias) hipLaunchKernelGGL((proj_gemm_nt_dma_f32_kernel<true>), dim3((unsigned)(8 * slots)), dim3(512), 0, st, g);
    else hipLaunchKernelGGL((proj_gemm_nt_dma_f32_kernel<false>), dim3((unsigned)(8 * slots)), dim3(512), 0, st, g);
    return hipGetLastError();
}

hipError_t launch_nt_dma(GemmArgs &g, hipStream_t st)
{
    g.tiles_m = (g.M + dma::BM - 1) / dma::BM;
    g.tiles_n = (g.N + dma::BN - 1) / dma::BN;
    // one workgroup per compute unit (its LDS allows no more), the same number on every XCD
    int slots = device_cu_count() / 8;
    if (slots < 1) slots = 1;
    if (slots > 64) slots = 64;
    // numbers per draw: about an eighth of a workgroup's share, four at most (the tail of a launch is then a few
    // tiles out of hundreds), one where a workgroup gets few tiles
    const long long per_wg = ((long long)(g.tiles_m + 7) / 8) * g.tiles_n * g.n_batch / slots;
    g.draw = per_wg >= 32 ? 4 : per_wg >= 16 ? 2 : 1;
    if (g.bias) hipLaunchKernelGGL((proj_gemm_nt_dma_kernel<true>), dim3((unsigned)(8 * slots)), dim3(512), 0, st, g);
    else hipLaunchKernelGGL((proj_gemm_nt_dma_kernel<false>), dim3((unsigned)(8 * slots)), dim3(512), 0, st, g);
    return hipGetLastError();
}

// The forward product with the weights in registers: every head of at most 256 channels, which is what a wave's registers hold
// (64 x 256 weights in 128 of them).  Also with few rows, where the launch that rounds W falls away: 604 problems of 1 to
// 60001 rows, 1 to 16 heads and 1 to 4 gates in both types take 1.8 times less on the geometric mean than with the kernels above, none
// more.  Row offsets of a step within 32 bits.
template <typename AT, int KB> hipError_t launch_rows_kb(const RowsArgs &a, int blocks, hipStream_t st)
{
    constexpr int T = 64 * RowsShape<AT, KB>::WAVES;
    if (a.bias) hipLaunchKernelGGL((proj_rows_kernel<AT, KB, true>), dim3((unsigned)blocks), dim3(T), 0, st, a);
    else hipLaunchKernelGGL((proj_rows_kernel<AT, KB, false>), dim3((unsigned)blocks), dim3(T), 0, st, a);
    return hipGetLastError();
}
template <typename AT> hipError_t launch_rows(const RowsArgs &a, int kb, int blocks, hipStream_t st)
{
    switch (kb) {
        case 1: return launch_rows_kb<AT, 1>(a, blocks, st);
        case 2: return launch_rows_kb<AT, 2>(a, blocks, st);
        case 3: return launch_rows_kb<AT, 3>(a, blocks, st);
        default: return launch_rows_kb<AT, 4>(a, blocks, st);
    }
}
// Jobs: every XCD gets the same number of them; side by side as many as take the least time, a job's weights at about two steps
// of R rows (with three heads one after the other, 300 rows took 22 us instead of 16).  `each`: workgroups that take the same rows.
void rows_jobs(int M, int n_heads, int each, int R, int slots, int *log_parts, int *abreast, int *J)
{
    *log_parts = 3;
    for (int h = n_heads; h % 2 == 0 && *log_parts > 0; h /= 2) --*log_parts;
    const int jobs = (n_heads << *log_parts) / 8;
    const double steps = (double)M / (1 << *log_parts) / R;
    double best = 0.0;
    for (int n = 1; n <= jobs && n * each <= slots; ++n) {
        const int j = slots / (n * each);
        const double t = (double)((jobs + n - 1) / n) * (2.0 + ceil(steps / j));
        if (n == 1 || t < best) { best = t; *abreast = n; *J = j; }
    }
}
bool rows_shape(int M, int H, int G, int n_heads, bool bf, RowsArgs *a, int *blocks)
{
    const int dh = H / n_heads, slots = device_cu_count() / 8;
    if (!g_proj_dma || dh % 64 || dh > 256 || slots < G || (long long)G * H >= (1 << 22)) return false;
    a->M = M; a->H = H; a->G = G; a->heads = n_heads;
    rows_jobs(M, n_heads, G, bf ? (dh <= 128 ? 16384 / dh : 64) : (dh == 64 ? 128 : dh == 256 ? 32 : 64), slots, &a->log_parts, &a->abreast, &a->J);
    *blocks = 8 * slots;
    return true;
}

// dx with the weights in registers: three and four gates of heads of at most 256 channels, as far as the weights fit (192 of a
// lane's registers: not four gates of 256).  792 problems of 1 to 60001 rows and 3 to 48 gates x heads, both types: 1.6 times less on the
// geometric mean than with the kernels above.  Heads of 256 take 10 us to load their weights, which 60001 x 256 or 16000 x 1024
// rows and channels (du and dx lie in the last level of cache and the tiles run at 3.5 TB/s) do not give back: 0.86-0.98
// in bf16, 0.93-1.16 in fp32; half of that 1.06-1.28.  Larger ones are faster by themselves (65536 x 1024 in bf16 142 -> 125 us),
// in fp32 1.1-1.2 times; in bf16 a training step gained 1 % on one device and lost 3 % on another, whose other kernels
// slowed down (the forward solve after it 366 -> 403 us): the tiles stay there.
template <typename AT> hipError_t launch_dx_rows(const DxArgs &a, int G, int kb, int blocks, hipStream_t st)
{
#define PARARNN_DX_ROWS(KB, G) hipLaunchKernelGGL((proj_dx_rows_kernel<AT, KB, G>), dim3((unsigned)blocks), dim3((64 * DxShape<AT, KB, G>::WAVES)), 0, st, a)
    switch (8 * kb + G) {
        case 8 + 3: PARARNN_DX_ROWS(1, 3); break;
        case 8 + 4: PARARNN_DX_ROWS(1, 4); break;
        case 16 + 3: PARARNN_DX_ROWS(2, 3); break;
        case 16 + 4: PARARNN_DX_ROWS(2, 4); break;
        case 24 + 3: PARARNN_DX_ROWS(3, 3); break;
        case 24 + 4: PARARNN_DX_ROWS(3, 4); break;
        default: PARARNN_DX_ROWS(4, 3);
    }
#undef PARARNN_DX_ROWS
    return hipGetLastError();
}
bool dx_rows_shape(int M, int H, int G, int n_heads, bool bf, DxArgs *a, int *blocks)
{
    const int dh = H / n_heads, slots = device_cu_count() / 8;
    if (!g_proj_dma || dh % 64 || dh > 256 || (G != 3 && G != 4) || (dh == 256 && G == 4) || slots < 1 || (long long)G * H >= (1 << 22)) return false;
    if (dh == 256 && (double)M * H > 10e6 && (bf || (double)M * H < 24e6)) return false;
    a->M = M; a->H = H; a->heads = n_heads;
    rows_jobs(M, n_heads, 1, bf ? (dh <= 128 ? 16384 / dh : dh * G < 768 ? 64 : 32) : dh == 64 ? 128 : dh == 128 ? 64 : 32, slots, &a->log_parts, &a->abreast, &a->J);
    *blocks = 8 * slots;
    return true;
}

template <typename AT> hipError_t launch_dw_rows(const DwArgs &a, int nb, int blocks, hipStream_t st)
{
#define PARARNN_DW_ROWS(NB) hipLaunchKernelGGL((proj_dw_rows_kernel<AT, NB>), dim3((unsigned)blocks), dim3((64 * DwRows<AT, NB>::WAVES)), 0, st, a)
    switch (nb) {
        case 2: PARARNN_DW_ROWS(2); break;
        case 4: PARARNN_DW_ROWS(4); break;
        case 5: PARARNN_DW_ROWS(5); break;
        case 6: PARARNN_DW_ROWS(6); break;
        case 7:
            if constexpr (sizeof(AT) == 4) PARARNN_DW_ROWS(7);
            break;
        default:
            if constexpr (sizeof(AT) == 4) PARARNN_DW_ROWS(8);
    }
#undef PARARNN_DW_ROWS
    return hipGetLastError();
}

int elementwise_blocks(size_t n)
{
    size_t blocks = (n + 255) / 256;
    const size_t cap = (size_t)device_cu_count() * 16;
    return (int)(blocks < cap ? blocks : cap);
}

}  // namespace

int proj_set_dma(int on)
{
    g_proj_dma = on ? 1 : 0;
    return PARARNN_OK;
}

size_t proj_workspace_bytes(int dtype, int B, int L, int H, int G, int n_heads, int backward)
{
    if (!shapes_ok(dtype, B, L, H, G, n_heads) || (H / n_heads) % BK) return 0;
    return proj_layout(dtype, B, L, H, G, n_heads, backward).total;
}

int proj_forward(int dtype, const void *x, const float *Wx, const float *bias, int B, int L, int H, int G,
                 int n_heads, void *u, void *workspace, size_t workspace_bytes, hipStream_t st)
{
    if (!shapes_ok(dtype, B, L, H, G, n_heads)) return PARARNN_INVALID_ARG;
    const int dh = H / n_heads;
    if (dh % BK) return PARARNN_UNSUPPORTED;
    if (((uintptr_t)x | (uintptr_t)Wx | (uintptr_t)u | (uintptr_t)workspace) % 16) return PARARNN_UNSUPPORTED;
    const ProjLayout lo = proj_layout(dtype, B, L, H, G, n_heads, 0);
    if (workspace_bytes < lo.total) return PARARNN_WORKSPACE_TOO_SMALL;
    RowsArgs r;
    int blocks;
    if (rows_shape(B * L, H, G, n_heads, dtype == PARARNN_BF16, &r, &blocks)) {
        r.x = x; r.Wx = Wx; r.bias = bias; r.u = u;
        const hipError_t e = dtype == PARARNN_BF16 ? launch_rows<unsigned short>(r, dh / 64, blocks, st) : launch_rows<float>(r, dh / 64, blocks, st);
        return e == hipSuccess ? PARARNN_OK : PARARNN_HIP_ERROR;
    }
    unsigned short *Wb = reinterpret_cast<unsigned short *>(static_cast<char *>(workspace) + lo.off_w);
    const size_t nw = (size_t)G * H * dh;
    int *tickets = reinterpret_cast<int *>(static_cast<char *>(workspace) + lo.off_tickets);
    hipLaunchKernelGGL(proj_wb_kernel, dim3(elementwise_blocks(nw / 4)), dim3(256), 0, st, Wx, Wb, nw / 4, tickets);
    GemmArgs g;
    memset(&g, 0, sizeof(g));
    g.A = x; g.Bw = Wb; g.C = u; g.bias = bias; g.tickets = tickets;
    g.lda = H; g.ldb = dh; g.ldc = (long long)G * H;
    g.M = B * L; g.N = dh; g.K = dh;
    g.kseg = dh; g.kseg_stride = 0;
    g.nz0 = G; g.n_batch = n_heads * G;                // z0 = gate, z1 = head: the tiles that read the same
    g.a_off[0] = 0; g.a_off[1] = dh;                   // columns of x (all gates of a head) are neighbours
    g.b_off[0] = (long long)H * dh; g.b_off[1] = (long long)dh * dh;
    g.c_off[0] = H; g.c_off[1] = dh;
    // fp32 storage: the copy-to-LDS kernel stores its output in 32-byte pieces, which costs more than its loads
    // gain once the output is four times the input (measured: 8-25 % faster with three gates, 1-9 % slower with four)
    const hipError_t e = dtype != PARARNN_BF16
                             ? ((g_proj_dma && nt_dma_f32_ok(g) && G <= 3) ? launch_nt_dma_f32(g, st) : launch_nt<float, float>(g, st))
                         : (g_proj_dma && nt_dma_ok(g)) ? launch_nt_dma(g, st) : launch_nt<unsigned short, unsigned short>(g, st);
    return e == hipSuccess ? PARARNN_OK : PARARNN_HIP_ERROR;
}

int proj_backward(int dtype, const void *x, const float *Wx, const void *du, int B, int L, int H, int G, int n_heads,
                  void *dx, float *dWx, float *dbias, void *workspace, size_t workspace_bytes, hipStream_t st)
{
    if (!shapes_ok(dtype, B, L, H, G, n_heads)) return PARARNN_INVALID_ARG;
    const int dh = H / n_heads;
    if (dh % BK) return PARARNN_UNSUPPORTED;
    if (((uintptr_t)x | (uintptr_t)Wx | (uintptr_t)du | (uintptr_t)dx | (uintptr_t)workspace) % 16) return PARARNN_UNSUPPORTED;
    const ProjLayout lo = proj_layout(dtype, B, L, H, G, n_heads, 1);
    if (workspace_bytes < lo.total) return PARARNN_WORKSPACE_TOO_SMALL;
    char *ws = static_cast<char *>(workspace);
    const size_t nw = (size_t)G * H * dh;
    const bool bf = dtype == PARARNN_BF16;
    hipError_t e = hipSuccess;
    DxArgs r;
    int blocks;
    if (dx && dx_rows_shape(B * L, H, G, n_heads, bf, &r, &blocks)) {
        r.du = du; r.Wx = Wx; r.dx = dx;
        if ((bf ? launch_dx_rows<unsigned short>(r, G, dh / 64, blocks, st) : launch_dx_rows<float>(r, G, dh / 64, blocks, st)) != hipSuccess) return PARARNN_HIP_ERROR;
    } else if (dx) {
        unsigned short *Wt = reinterpret_cast<unsigned short *>(ws + lo.off_w);
        int *tickets = reinterpret_cast<int *>(ws + lo.off_tickets);
        hipLaunchKernelGGL(proj_wt_kernel, dim3((unsigned)(nw / 4096)), dim3(256), 0, st, Wx, Wt, G, H, dh, tickets);
        GemmArgs g;
        memset(&g, 0, sizeof(g));
        g.A = du; g.Bw = Wt; g.C = dx; g.bias = nullptr; g.tickets = tickets;
        g.lda = (long long)G * H; g.ldb = (long long)G * dh; g.ldc = H;
        g.M = B * L; g.N = dh; g.K = G * dh;
        g.kseg = dh; g.kseg_stride = H;                 // k = (gate, i): gates are H apart in a row of du
        g.nz0 = n_heads; g.n_batch = n_heads;           // z0 = head
        g.a_off[0] = dh; g.b_off[0] = (long long)dh * G * dh; g.c_off[0] = dh;
        e = !bf ? ((g_proj_dma && nt_dma_f32_ok(g)) ? launch_nt_dma_f32(g, st) : launch_nt<float, float>(g, st))
            : (g_proj_dma && nt_dma_ok(g)) ? launch_nt_dma(g, st) : launch_nt<unsigned short, unsigned short>(g, st);
        if (e != hipSuccess) return PARARNN_HIP_ERROR;
    }
    if (dWx) {
        DwArgs a;
        memset(&a, 0, sizeof(a));
        a.du = du; a.x = x;
        a.part = reinterpret_cast<float *>(ws + lo.off_part);
        a.dbpart = dbias ? reinterpret_cast<float *>(ws + lo.off_db) : nullptr;
        a.M = B * L; a.H = H; a.G = G; a.heads = n_heads; a.dh = dh;
        const bool copy_kernel = bf && g_proj_dma && lo.S2 > 0;
        const bool rows_kernel = g_proj_dma && lo.S3 > 0;
        a.S = rows_kernel ? lo.S3 : copy_kernel ? lo.S2 : lo.S;
        if (a.S == 1) {                                 // one range: its sums are the results
            a.part = dWx;
            if (dbias) a.dbpart = dbias;
        }
        a.rows_per_split = rows_kernel ? lo.rows_per_split3 : copy_kernel ? lo.rows_per_split2 : lo.rows_per_split;
        a.tiles = rows_kernel ? dw_rows_tiles(dh) : copy_kernel ? lo.tiles2 : lo.tiles;
        a.n_blocks = a.tiles * a.tiles * n_heads * G * a.S;
        a.per_xcd = (a.n_blocks + 7) / 8;
        blocks = 8 * a.per_xcd;
        if (rows_kernel) {
            const int nb = dh / a.tiles / 32;
            if ((bf ? launch_dw_rows<unsigned short>(a, nb, blocks, st) : launch_dw_rows<float>(a, nb, blocks, st)) != hipSuccess) return PARARNN_HIP_ERROR;
        } else if (copy_kernel) hipLaunchKernelGGL(proj_dw_dma_kernel, dim3(blocks), dim3(512), 0, st, a);
        else if (bf) hipLaunchKernelGGL(proj_dw_kernel<unsigned short>, dim3(blocks), dim3(256), 0, st, a);
        else hipLaunchKernelGGL(proj_dw_kernel<float>, dim3(blocks), dim3(256), 0, st, a);
        if (hipGetLastError() != hipSuccess) return PARARNN_HIP_ERROR;
        if (a.S > 1) {
            if (((uintptr_t)dWx | (uintptr_t)dbias) % 16 == 0) {
                const ReducePair r = {{a.part, a.dbpart}, {dWx, dbias}, {(int)(nw / 4), dbias ? G * H / 4 : 0}, a.S};
                if (launch_param_reduce_pair(r, st) != hipSuccess) return PARARNN_HIP_ERROR;
            } else {
                if (launch_param_reduce(a.part, dWx, a.S, (int)nw, st) != hipSuccess) return PARARNN_HIP_ERROR;
                if (dbias && launch_param_reduce(a.dbpart, dbias, a.S, G * H, st) != hipSuccess) return PARARNN_HIP_ERROR;
            }
        }
    }
    return PARARNN_OK;
}

}  // namespace pararnn
