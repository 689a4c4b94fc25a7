// Mass-matrix solve with a polynomial preconditioner, for 2D problems: the solve
// that P2M_SOLVER_AUTO, P2M_SOLVER_RESIDENT_CHEB and the batches take.
//
// Mixed-precision iterative refinement as in every solve here (FP64 solution and
// residual outside, conjugate gradients in T with FP64 dot products inside), with an
// inner iteration built to need few grid barriers:
//
//  * the inner system is scaled symmetrically, A = D^-1/2 M D^-1/2 (unit diagonal,
//    so three stencil planes instead of four and no division), and preconditioned
//    by the polynomial p(A) of degree 2 (or 4) that makes 1 - l p(l) the scaled
//    Chebyshev polynomial T3 (T5) on [lo, hi].  Both are odd: beyond hi, 1 - l p(l) is
//    negative, below lo it lies in (0, 1), so l p(l) > 0 for every l > 0 and the
//    preconditioner is positive definite whatever the spectrum; [lo, hi] only
//    decides how fast it is (pcg_interval);
//  * Chronopoulos-Gear conjugate gradients: (r, u), (w, u) and (r, r) with u = p(A) r,
//    w = A u are reduced together, so an iteration has one grid barrier, and needs a
//    third (T5: a fifth) of the iterations of the diagonal preconditioner (T3: 5-6 for
//    15 at 8 particles per cell, 17 for 45 at 2);
//  * the three (five) stencil products of an iteration read r as many nodes outside the
//    tile.  A workgroup keeps its own copy of that ring's r and s (and, on the
//    innermost ring, p, d and x), advanced by the same operations on the same values
//    as their owners, so that per iteration only w crosses tiles: every tile publishes
//    the w of its border strip (device-coherent stores) and reads its ring's after
//    the barrier.
//
// A workgroup owns one tile for the whole solve and keeps its state in registers and
// its stencil in LDS; with more tiles than workgroups it owns several and streams
// their state from owner-only arrays.  The arithmetic and the order of every sum
// depend on the tile only, never on how the tiles are dealt, so a problem gives the
// same bits alone, in a batch, resident or streamed.
//
// Bound: the latency of one iteration (its LDS stencil products, a block sum, the
// grid barrier), not traffic, while one tile per workgroup fits the chip; the traffic of
// the streamed state beyond.  Whole mass assignment and interpolation, before (diagonal
// preconditioner, or the FP64 streaming solve) and now: 256 x 256 at 4 per cell, F = 1,
// 263 -> 108 us; 1024 x 1024 at 8 per cell, F = 3, 597 -> 403 us; 2048 x 2048
// 4.09 -> 2.39 ms; 512 x 512 FP64 at 8 per cell, F = 1, 1312 -> 193 us.  Two random particles
// per cell (50 to 440 iterations): 600 x 600, F = 1, 1.92 -> 1.65 ms, F = 3, 6.41 -> 5.91;
// 1400 x 1400, F = 3, 32.1 -> 29.4 ms.  What the large
// tile's 24 us iteration (F = 3) answered to: x kept as the start formula until a field
// needs a second correction (no FP64 x traffic in the usual two residual phases), border
// columns published transposed in one 16-byte store a lane and read 64 rows a wave
// (node-major columns cost 3 us of it), and no register spilled inside the loop.
#include <string.h>

#include <atomic>

#include "cg_common.hpp"

namespace p2m {

namespace {

// Tile of TX x TY nodes on NT threads; a thread owns OWN consecutive rows of one
// column (a column's stencil reads slide down the rows) and at most one ring slot.
template <int TX_, int TY_, int NT_, int PH_>
struct PTile {
    static constexpr int TX = TX_, TY = TY_, NT = NT_;
    static constexpr int PH = PH_;   // ring depth: one per stencil product of an iteration
    static constexpr int EX = TX + 2 * PH, EY = TY + 2 * PH, EN = EX * EY;
    static constexpr int OWN = TX * TY / NT;
    static constexpr int NRING = EN - TX * TY;
    static constexpr int NRP = (NRING + 63) / 64 * 64;
    static_assert(NT % TX == 0 && OWN * NT == TX * TY && NRING <= NT && EN % 4 == 0, "tile");
};
using TileS = PTile<32, 32, 1024, 5>;
using TileD = PTile<32, 32, 512, 3>;    // FP64 only (pcg_depth)
using TileL = PTile<64, 64, 1024, 3>;

constexpr int kStall = 40;

template <typename T>
struct PArgs {
    PolyInst one;          // the problem of a single solve
    const PolyInst* inst;  // the instances of a batch
    const int32_t* rmap;   // batch: tile -> instance
    const int32_t* order;  // batch: dealing order of the tiles
    int nprob, ntiles;
    T* coef;               // [4][nn] blocks at 4*no (orphan diagonals set to 1 here)
    T* b;                  // [F][nn] blocks at F*no (orphan entries set to 0 here)
    const T* w;            // [nn] blocks at no
    double* x64;           // [F][nn] blocks at F*no, owner-only
    T* pubR;               // [F][nn] blocks at F*no, published scaled residual of the row strips
    T* pubW[2];            // the same of w, by iteration parity
    T* colR;               // [F][2 PH ptx][ny] blocks at F*co, the column strips, a column's rows
    T* colW[2];            // adjacent (a wave reads and a lane writes whole runs)
    double* xring;         // [tile][F][NRP] ring copies of x, owner-only
    // streamed state (workgroups that own several tiles), by tile
    T* own;                // [tile][6][F][TX*TY]: p, d, s, r, w, u
    T* ring;               // [tile][5][F][NRP]: p, d, s, r, u
    T* rsd;                // [tile][TX*TY] inverse square roots of the diagonal
    T* cimg;               // [tile][3][EN] scaled stencil
    RSync sy;              // part: [2][3F][ntiles]; tot: [2][nprob][3F]
    int start;
    p2m_solve_opts opts;
};

__device__ __forceinline__ float mul_t(float a, float b) { return __fmul_rn(a, b); }
__device__ __forceinline__ double mul_t(double a, double b) { return __dmul_rn(a, b); }
__device__ __forceinline__ float fma_t(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __fma_rn(a, b, c); }
__device__ __forceinline__ double dot_t(double acc, float a, float b) { return dot_acc(acc, a, b); }
__device__ __forceinline__ double dot_t(double acc, double a, double b) { return __fma_rn(a, b, acc); }

// 1/sqrt of a diagonal entry; 1 for an orphan row (identity) and for a
// diagonal too small to invert (the row then decouples: its products with the
// neighbours are below its rounding)
// (the instruction and one Newton step, written out: the compiler lowers an FP32 square
// root with or without its refinement by context, and a ring copy has to equal its owner's
// value bit for bit)
__device__ __forceinline__ float rs_of(float d, bool orphan) {
    if (orphan || !(d >= 1.17549435e-38f)) return 1.0f;
    const float y = __builtin_amdgcn_rsqf(d);
    return fmaf(0.5f * y, fmaf(-d * y, y, 1.0f), y);
}
__device__ __forceinline__ double rs_of(double d, bool orphan) {
    return orphan || !(d >= 2.2250738585072014e-308) ? 1.0 : __ddiv_rn(1.0, __dsqrt_rn(d));
}
__device__ __forceinline__ float div_t(float a, float b) { return __fdiv_rn(a, b); }
__device__ __forceinline__ double div_t(double a, double b) { return __ddiv_rn(a, b); }

// Accesses at a 32-bit byte offset from a uniform base: one address register each
// (meshes are at most kPolyMaxNodes)
template <typename T>
__device__ __forceinline__ T ldo(const T* p, uint32_t i) {
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(p) + i * (uint32_t)sizeof(T));
}
template <typename T>
__device__ __forceinline__ T* ato(T* p, uint32_t i) {
    return reinterpret_cast<T*>(reinterpret_cast<char*>(p) + i * (uint32_t)sizeof(T));
}

// The value, opaque to the optimiser: addresses formed from it are formed where they are
// used.  Hoisted out of the solve's loops they take more registers than its state does.
template <typename V>
__device__ __forceinline__ V fresh(V v) {
    asm volatile("" : "+v"(v));
    return v;
}

// FP64 stencil product with coefficients of type T
template <typename T>
__device__ __forceinline__ double stencil_x(const T (&c)[7], double x0, double xe, double xw,
                                            double xn, double xs, double xne, double xsw) {
    double acc = __dmul_rn((double)c[0], x0);
    acc = __fma_rn((double)c[1], xe, acc);
    acc = __fma_rn((double)c[2], xw, acc);
    acc = __fma_rn((double)c[3], xn, acc);
    acc = __fma_rn((double)c[4], xs, acc);
    acc = __fma_rn((double)c[5], xne, acc);
    acc = __fma_rn((double)c[6], xsw, acc);
    return acc;
}

template <typename T, class TC, int F, bool BATCH, bool STREAM>
__global__ __launch_bounds__(TC::NT) void k_pcg(PArgs<T> a) {
    constexpr int PH = TC::PH;
    constexpr int NT = TC::NT, OWN = TC::OWN, EX = TC::EX, EN = TC::EN, NRP = TC::NRP;
    constexpr int NTN = TC::TX * TC::TY, NV = 3 * F, NW = NT / 64;
    // (two and) three fields resident on the large tile: their state does not fit 128 registers
    // (15 of them spilled and reloaded per iteration cost 5 us of 24), so two fields' d live in
    // LDS and the inverse square roots, needed in the residual phases only, are formed again.
    // Two fields give up the second exchange buffer for it: 700 x 700, whole pass 187 -> 183 us
    constexpr int DL = !STREAM && !BATCH && NT == 1024 && (F == 3 || (F == 2 && OWN > 1)) ? 2 : 0;
    // two exchange buffers per field where they fit (one workgroup barrier per stencil
    // product), else one (two barriers)
    constexpr size_t kTwo = ((size_t)(3 + 2 * F) * EN + (DL ? DL : 1) * NTN) * sizeof(T) + (BATCH ? 23000 : 1500);
    constexpr bool PP = kTwo <= (NT == 512 ? 80000u : 160000u);
    constexpr int UB = (PP ? 2 : 1) * F * EN;
    // One product and no u in memory where the active fields are all on the diagonal.  Two
    // fields streamed or in FP64 form every product: the branch costs them 1% of an ordinary
    // pass, and their stalled systems are faster than by the diagonal kernels as it is (1400 x
    // 1400, one particle per cell, 500 iterations: 26.1 ms by that one, 24.9)
    constexpr bool kSkip = F != 2 || (!STREAM && sizeof(T) == 4);
    constexpr int MAXP = BATCH ? kBatchMaxPairs : F, MAXK = BATCH ? kBatchMaxInstances : 1;

    __shared__ __align__(16) T cf[3 * EN];    // scaled E, N, NE of the tile and its ring
    __shared__ __align__(16) T ub[UB];        // exchange planes; x (FP64) in the residual phase
    __shared__ T rsl[DL ? 1 : NTN];           // inverse square roots of the own diagonal, by thread
    __shared__ T dl[DL ? DL * NTN : 1];
    __shared__ double red[NW * 4 * NV];
    __shared__ double vals[BATCH ? 3 * kBatchMaxPairs : NV];
    __shared__ double s_bb[MAXP], s_gam[MAXP], s_alpha[MAXP], s_relres[MAXP], s_target[MAXP];
    __shared__ T s_af[MAXP], s_bf[MAXP];
    __shared__ int s_iters[MAXP], s_refines[MAXP];
    __shared__ float s_best[MAXP];          // smallest (r,r) of the inner solve, and the
    __shared__ short s_since[MAXP];         // iterations since
    __shared__ unsigned char s_diag[MAXP];  // the polynomial has stalled: p(A) = 1 from here on
    __shared__ unsigned char s_done[MAXP], s_inner[MAXP], s_zero[MAXP];
    // corrections that are this solve's own doing and not on the caller's max_refine: bit 0 the
    // one after a stalled recurrence, bit 1 one after an inner solve that went for the goal (and
    // missed it: its norm is the scaled one, its recurrence perhaps FP32)
    __shared__ unsigned char s_more[MAXP];
    // x is held in x64 / xring (else it is the start, formed from b and w where needed);
    // the last inner solve went for the goal, so its residual is expected to be the last
    __shared__ unsigned char s_held[MAXP], s_last[MAXP];
    __shared__ uint32_t s_flags[MAXK];
    __shared__ int s_ok;

    const int G = gridDim.x, g = blockIdx.x, tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int col = tid % TC::TX, row0 = (tid / TC::TX) * OWN;
    const int o_q0 = (row0 + PH) * EX + col + PH;   // LDS index of the first own node
    constexpr bool keep = !STREAM;            // one tile per workgroup: its state stays here

    // ---- the current tile ----------------------------------------------------
    int k = 0, tile = 0, i0 = 0, j0 = 0, nx = 0, ny = 0, nn = 0, no = 0, co = 0, cl = 0, txa = 0, tya = 0;
    int o_g0 = 0, o_rg = 0, o_rq = 0, rdep = 0;   // first own node; ring slot: node, LDS index, depth (0: none)
    int o_rc = 0;                             // column-buffer element of a column ring slot, else -1
    int o_cc = 0;                             // column-buffer element of the first own node, else -1
    uint32_t am = 0, sm = 0;                  // own nodes inside the mesh; on the published row strips
    T pc[PH];
    T* out = nullptr;
    auto inst_of = [&](int kk) -> const PolyInst& {
        if constexpr (BATCH) return a.inst[kk];
        else return a.one;
    };
    auto set_tile = [&](int i) {
        tile = i;
        if constexpr (BATCH) {
            tile = __builtin_amdgcn_readfirstlane(a.order[i]);
            k = __builtin_amdgcn_readfirstlane(a.rmap[tile]);
        }
        const PolyInst& I = inst_of(k);
        const int lt = tile - I.pt;
        i0 = (lt % I.ptx) * TC::TX;
        j0 = (lt / I.ptx) * TC::TY;
        nx = I.m.nx;
        ny = I.m.ny;
        nn = I.m.nn;
        no = I.no;
        co = I.co;
        cl = 2 * PH * I.ptx * ny;
        out = (T*)I.out;
#pragma unroll
        for (int j = 0; j < PH; ++j) pc[j] = (T)I.pc[j];
        txa = min(TC::TX, nx - i0);
        tya = min(TC::TY, ny - j0);
        o_g0 = (j0 + row0) * nx + i0 + col;
        am = sm = 0;
#pragma unroll
        for (int o = 0; o < OWN; ++o) {
            const int r = row0 + o;
            if (!(col < txa && r < tya)) continue;
            am |= 1u << o;
            if (r < PH || r >= tya - PH) sm |= 1u << o;
        }
        // the published columns of a tile column: PH from the left, PH from the right
        const int tc = i0 / TC::TX;
        const int cs = col < PH ? col : (col >= txa - PH ? PH + col - (txa - PH) : -1);
        o_cc = col < txa && cs >= 0 ? (2 * PH * tc + cs) * ny + j0 + row0 : -1;
        // ring slots: PH rows below, PH above (corners included), PH columns left, right
        const int rw = txa + 2 * PH;
        int h = tid, lc = 0, lr = 0;
        const bool on = h < 2 * PH * rw + 2 * PH * tya;
        if (h < 2 * PH * rw) {
            const bool up = h >= PH * rw;
            if (up) h -= PH * rw;
            int rr = 0;
#pragma unroll
            for (int q = 1; q < PH; ++q) rr += h >= q * rw;
            lr = up ? tya + rr : rr - PH;
            lc = h - rr * rw - PH;
        } else {
            h -= 2 * PH * rw;
            const bool right = h >= PH * tya;
            if (right) h -= PH * tya;
            int cc = 0;
#pragma unroll
            for (int q = 1; q < PH; ++q) cc += h >= q * tya;
            lr = h - cc * tya;
            lc = cc + (right ? txa : -PH);
        }
        const int dx = lc < 0 ? -lc : (lc >= txa ? lc - txa + 1 : 0);
        const int dy = lr < 0 ? -lr : (lr >= tya ? lr - tya + 1 : 0);
        rdep = on ? max(dx, dy) : 0;
        int gc = (i0 + lc) % nx, gr = (j0 + lr) % ny;
        if (gc < 0) gc += nx;
        if (gr < 0) gr += ny;
        o_rg = on ? gc + nx * gr : 0;
        o_rc = -1;
        if (on && lr >= 0 && lr < tya) {   // a column slot: where its owner publishes it
            const int ot = gc / TC::TX, oc = gc - ot * TC::TX, ow = min(TC::TX, nx - ot * TC::TX);
            o_rc = (2 * PH * ot + (oc < PH ? oc : PH + oc - (ow - PH))) * ny + gr;
        }
        o_rq = on ? (lr + PH) * EX + lc + PH : 0;
    };
    auto inner_mask = [&]() {
        uint32_t mk = 0;
#pragma unroll
        for (int f = 0; f < F; ++f)
            if (s_inner[k * F + f]) mk |= 1u << f;
        return mk;
    };

    // ---- state of the current tile -------------------------------------------
    T vp[F][OWN], vd[F][OWN], vs[F][OWN], vr[F][OWN], vw[F][OWN];
    T np_[F], nd[F], ns[F], nr[F];            // ring copies of p, d, s, r
    // d is touched once an iteration: the first DL fields' in LDS
    auto d_get = [&](int f) {
        if (f < DL) {
#pragma unroll
            for (int o = 0; o < OWN; ++o) vd[f][o] = dl[(f * OWN + o) * NT + tid];
        }
    };
    auto d_put = [&](int f) {
        if (f < DL) {
#pragma unroll
            for (int o = 0; o < OWN; ++o) dl[(f * OWN + o) * NT + tid] = vd[f][o];
        }
    };
    struct Vec { T v[OWN]; };
    auto own_at = [&](int v, int f) {
        return ato(a.own + (((size_t)tile * 6 + v) * F + f) * NTN, tid * OWN);
    };
    auto ring_at = [&](int v, int f) {
        return ato(a.ring + (((size_t)tile * 5 + v) * F + f) * NRP, tid);
    };
    auto ld_own = [&](int v, int f, T (&x)[OWN]) {
        const Vec t = *reinterpret_cast<const Vec*>(__builtin_assume_aligned(own_at(v, f), OWN * sizeof(T)));
#pragma unroll
        for (int o = 0; o < OWN; ++o) x[o] = t.v[o];
    };
    auto st_own = [&](int v, int f, const T (&x)[OWN]) {
        Vec t;
#pragma unroll
        for (int o = 0; o < OWN; ++o) t.v[o] = x[o];
        *reinterpret_cast<Vec*>(__builtin_assume_aligned(own_at(v, f), OWN * sizeof(T))) = t;
    };
    auto load_img = [&]() {
        struct alignas(16) Q { unsigned u[4]; };
        constexpr int n = 3 * EN * (int)sizeof(T) / 16;
        const Q* src = reinterpret_cast<const Q*>(a.cimg + (size_t)tile * 3 * EN);
        Q* dst = reinterpret_cast<Q*>(cf);
        for (int i = tid; i < n; i += NT) dst[i] = src[i];
    };
    // the start at an own node from its b and w (a user's start is held from the set-up on)
    auto own_start = [&](T bk, T wk) -> double {
        if (a.start == P2M_START_ZERO || !(wk > (T)0)) return 0.0;
        return (double)div_t(bk, wk);
    };
    auto start_value = [&](int f, int kk) -> double {
        if (a.start == P2M_START_ZERO) return 0.0;
        const T wk = ldo(a.w + no, kk);
        if (!(wk > (T)0)) return 0.0;
        return a.start == P2M_START_FLIP
                   ? (double)div_t(ldo(a.b + (size_t)F * no + (size_t)f * nn, kk), wk)
                   : (double)ldo(out + (size_t)f * nn, kk);
    };

    unsigned epoch = 0;   // reductions done
    unsigned tep = 0;     // barrier passes done
    // block sums of the n values a thread holds (its sums over its nodes of the current
    // tile), in a fixed order, stored as the tile's partials of the next reduction
    static_assert(NW <= 16 && NV <= 16 && 16 * NV <= NT, "block sum layout");
    auto store_sums = [&](const double (&v)[NV], int n) {
        double mine = 0.0;
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            if (j >= n) break;
            const double r = row_sum16(v[j]);
            if ((lane & 15) == j) mine = r;
        }
        if ((lane & 15) < n) red[(wave * 4 + (lane >> 4)) * NV + (lane & 15)] = mine;
        __syncthreads();
        // value jv by one 16-lane row, lane l the four rows of wave l, then the row sum
        if (tid < ((16 * n + 63) & ~63)) {
            const int jv = tid >> 4, wv = tid & 15;
            double t = 0.0;
            if (jv < n && wv < NW) {
                const double* q = red + wv * 4 * NV + jv;
                t = (q[0] + q[NV]) + (q[2 * NV] + q[3 * NV]);
            }
            t = row_sum16(t);
            // value-major: the lanes that sum one value over the tiles read consecutive words
            if (jv < n && wv == 0)
                st_c(&a.sy.part[((size_t)((epoch + 1) & 1) * NV + jv) * a.ntiles + tile], t);
        }
        if (!keep) __syncthreads();
    };
    // totals over an instance's tiles [t0, t0 + nt) of nv values: value jv by the 32
    // lanes of one half wave, lane l over tiles l, l + 32, ..., then the two row sums
    auto sum_tiles = [&](int t0, int nt, int nv, auto put) {
        const double* part = a.sy.part + (size_t)(epoch & 1) * NV * a.ntiles;
        const int l = lane & 31;
        for (int jb = wave * 2; jb < nv; jb += NT / 32) {
            const int jv = jb + (lane >> 5);
            double acc = 0.0;
            if (jv < nv) {
                const double* p = part + (size_t)jv * a.ntiles + t0;
                for (int b0 = l; b0 < nt; b0 += 256) {
                    double v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) v[u] = b0 + 32 * u < nt ? ld_c(p + b0 + 32 * u) : 0.0;
#pragma unroll
                    for (int u = 0; u < 8; ++u)
                        if (b0 + 32 * u < nt) acc += v[u];
                }
            }
            const double r = row_sum16(acc);
            const double lo = readlane_d(r, 0) + readlane_d(r, 16);
            const double hi = readlane_d(r, 32) + readlane_d(r, 48);
            if (jv < nv && l == 0) put(jv, (lane & 32) ? hi : lo);
        }
    };
    auto barrier = [&]() -> bool {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        ++tep;
        if (tid == 0) {
            if (tree_arrive(a.sy, tep, G)) tree_release(a.sy, tep);
            s_ok = tree_wait(a.sy, tep) ? 1 : 0;
        }
        __syncthreads();
        return s_ok != 0;
    };
    // One reduction: every tile's partials are stored, then each workgroup sums them
    // itself (a single problem), or the workgroup assigned to an instance sums that
    // instance's and publishes the totals (a batch).  vals[kk * nv + j] on return.
    auto reduce = [&](int nv, auto after) -> bool {
        ++epoch;
        if (!barrier()) return false;
        after();
        if constexpr (BATCH) {
            double* tot = a.sy.tot + (size_t)(epoch & 1) * a.nprob * NV;
            for (int kk = g; kk < a.nprob; kk += G) {
                const PolyInst& I = a.inst[kk];
                sum_tiles(I.pt, I.npt, nv, [&](int jv, double v) { st_c(&tot[(size_t)kk * NV + jv], v); });
            }
            if (!barrier()) return false;
            for (int i = tid; i < a.nprob * nv; i += NT) {
                const int kk = i / nv, jv = i - kk * nv;
                vals[i] = ld_c(&tot[(size_t)kk * NV + jv]);
            }
        } else {
            sum_tiles(0, a.ntiles, nv, [&](int jv, double v) { vals[jv] = v; });
        }
        __syncthreads();
        return true;
    };

    for (int p = tid; p < a.nprob * F; p += NT) {
        s_iters[p] = 0; s_refines[p] = 0; s_done[p] = 0; s_inner[p] = 0; s_zero[p] = 0; s_diag[p] = 0;
        s_more[p] = 0;
        s_held[p] = a.start == P2M_START_USER; s_last[p] = 0;
        s_relres[p] = 0.0; s_bb[p] = 0.0;
    }
    for (int kk = tid; kk < a.nprob; kk += NT) s_flags[kk] = 0u;

    // ---- set-up: scaled stencil, orphan regularisation, start ------------------
    for (int i = g; i < a.ntiles; i += G) {
        set_tile(i);
        const int g0 = o_g0, q0 = o_q0, rg = o_rg, rq = o_rq;
        T* C = a.coef + (size_t)4 * no;
        const T* w = a.w + no;
        const bool user = a.start == P2M_START_USER;
        T dg[OWN], wg[OWN], e1[OWN], e2[OWN], e3[OWN], bg[F][OWN];
#pragma unroll
        for (int o = 0; o < OWN; ++o) {
            const int kk = (am & (1u << o)) ? g0 + o * nx : 0;
            dg[o] = ldo(C, kk);
            wg[o] = ldo(w, kk);
            e1[o] = ldo(C + nn, kk);
            e2[o] = ldo(C + (size_t)2 * nn, kk);
            e3[o] = ldo(C + (size_t)3 * nn, kk);
#pragma unroll
            for (int f = 0; f < F; ++f)
                bg[f][o] = user ? ldo(out + (size_t)f * nn, kk) : (T)0;
        }
        const T rd = ldo(C, rg), rw = ldo(w, rg), r1 = ldo(C + nn, rg), r2 = ldo(C + (size_t)2 * nn, rg),
                r3 = ldo(C + (size_t)3 * nn, rg);
#pragma unroll
        for (int f = 0; f < F; ++f)
            if (user && rdep == 1) a.xring[((size_t)tile * F + f) * NRP + tid] = start_value(f, rg);
        // the inverse square roots of the diagonal, in ub
        T rso[OWN];
        const T rsr = rs_of(rd, !(rw > (T)0));
#pragma unroll
        for (int o = 0; o < OWN; ++o) {
            const bool orphan = !(wg[o] > (T)0);
            rso[o] = rs_of(dg[o], orphan);
            if (!DL) rsl[o * NT + tid] = rso[o];
            if (am & (1u << o)) ub[q0 + o * EX] = rso[o];
        }
        if (rdep) ub[rq] = rsr;
        __syncthreads();
        // a coupling whose far node lies outside the ring is never used
#pragma unroll
        for (int o = 0; o < OWN; ++o) {
            if (!(am & (1u << o))) continue;
            const int q = q0 + o * EX;
            cf[q] = mul_t(mul_t(e1[o], rso[o]), ub[q + 1]);
            cf[EN + q] = mul_t(mul_t(e2[o], rso[o]), ub[q + EX]);
            cf[2 * EN + q] = mul_t(mul_t(e3[o], rso[o]), ub[q + EX + 1]);
        }
        if (rdep) {
            const int qc = rq % EX, qr = rq / EX;
            const bool ex = qc + 1 < txa + 2 * PH, ey = qr + 1 < tya + 2 * PH;
            cf[rq] = ex ? mul_t(mul_t(r1, rsr), ub[rq + 1]) : (T)0;
            cf[EN + rq] = ey ? mul_t(mul_t(r2, rsr), ub[rq + EX]) : (T)0;
            cf[2 * EN + rq] = ex && ey ? mul_t(mul_t(r3, rsr), ub[rq + EX + 1]) : (T)0;
        }
#pragma unroll
        for (int o = 0; o < OWN; ++o) {
            if (!(am & (1u << o))) continue;
            const int kk = g0 + o * nx;
            const bool orphan = !(wg[o] > (T)0);
            if (orphan) C[kk] = (T)1;
#pragma unroll
            for (int f = 0; f < F; ++f) {
                const size_t q = (size_t)F * no + (size_t)f * nn + kk;
                if (orphan) a.b[q] = (T)0;
                if (user) a.x64[q] = orphan ? 0.0 : (double)bg[f][o];
            }
            p2m_report* rep = inst_of(k).rep;
            if (orphan && rep) {
                atomicAdd(&rep->n_orphan, 1);
                atomicOr(&rep->flags, (uint32_t)P2M_FLAG_ORPHAN);
            }
        }
        __syncthreads();
        if (!keep) {
            struct alignas(16) Q { unsigned u[4]; };
            Q* dst = reinterpret_cast<Q*>(a.cimg + (size_t)tile * 3 * EN);
            const Q* s4 = reinterpret_cast<const Q*>(cf);
            for (int q = tid; q < 3 * EN * (int)sizeof(T) / 16; q += NT) dst[q] = s4[q];
            Vec t;
#pragma unroll
            for (int o = 0; o < OWN; ++o) t.v[o] = rso[o];
            *reinterpret_cast<Vec*>(a.rsd + (size_t)tile * NTN + (size_t)tid * OWN) = t;
            __syncthreads();
        }
    }
#pragma unroll
    for (int f = 0; f < F; ++f) {
#pragma unroll
        for (int o = 0; o < OWN; ++o) vp[f][o] = vd[f][o] = vs[f][o] = vr[f][o] = vw[f][o] = (T)0;
        np_[f] = nd[f] = ns[f] = nr[f] = (T)0;
    }
    __syncthreads();

    // A x at the own nodes (qo) and, with rn, at this thread's ring slot (qn), for the
    // fields in im; the same operations in the same order at either, so a ring value
    // equals its owner's bit for bit
    auto apply = [&](const T* U, uint32_t im, bool rn, T (&qo)[F][OWN], T (&qn)[F]) {
        // two rows at a time: a window slides down each column, and the coefficients of
        // more rows at once would not fit beside the state
        constexpr int R = OWN < 2 ? 1 : 2;
        static_assert(OWN % R == 0, "rows of a step");
#pragma unroll
        for (int h = 0; h < OWN; h += R) {
            const int q0 = fresh(o_q0) + h * EX;
            T cE[R], cW[R], cN[R + 1], cD[R], cS[R];
#pragma unroll
            for (int o = 0; o < R; ++o) {
                const int q = q0 + o * EX;
                cE[o] = cf[q];
                cW[o] = cf[q - 1];
                cN[o + 1] = cf[EN + q];
                cD[o] = cf[2 * EN + q];
                cS[o] = cf[2 * EN + q - EX - 1];
            }
            cN[0] = cf[EN + q0 - EX];
#pragma unroll
            for (int f = 0; f < F; ++f) {
                if (!(im & (1u << f))) continue;
                const T* L = U + f * EN + q0;
                T x[R + 2], e[R + 1], v[R + 1];
#pragma unroll
                for (int o = 0; o < R + 2; ++o) x[o] = L[(o - 1) * EX];
#pragma unroll
                for (int o = 0; o < R + 1; ++o) {
                    e[o] = L[o * EX + 1];
                    v[o] = L[(o - 1) * EX - 1];
                }
#pragma unroll
                for (int o = 0; o < R; ++o) {
                    T s = fma_t(cE[o], e[o], x[o + 1]);
                    s = fma_t(cW[o], v[o + 1], s);
                    s = fma_t(cN[o + 1], x[o + 2], s);
                    s = fma_t(cN[o], x[o], s);
                    s = fma_t(cD[o], e[o + 1], s);
                    qo[f][h + o] = fma_t(cS[o], v[o], s);
                }
            }
        }
        if (rn) {
            const int rq = fresh(o_rq);
            const T rE = cf[rq], rW = cf[rq - 1], rN = cf[EN + rq], rS = cf[EN + rq - EX],
                    rD = cf[2 * EN + rq], rM = cf[2 * EN + rq - EX - 1];
#pragma unroll
            for (int f = 0; f < F; ++f) {
                if (!(im & (1u << f))) continue;
                const T* L = U + f * EN + rq;
                T s = fma_t(rE, L[1], L[0]);
                s = fma_t(rW, L[-1], s);
                s = fma_t(rN, L[EX], s);
                s = fma_t(rS, L[-EX], s);
                s = fma_t(rD, L[EX + 1], s);
                qn[f] = fma_t(rM, L[-EX - 1], s);
            }
        }
    };
    T* const bA = ub;
    T* const bB = PP ? ub + F * EN : ub;
    auto put = [&](T* U, uint32_t im, const T (&xo)[F][OWN], bool rn, const T (&xn)[F]) {
        const int q0 = fresh(o_q0), rq = fresh(o_rq);
#pragma unroll
        for (int f = 0; f < F; ++f) {
            if (!(im & (1u << f))) continue;
#pragma unroll
            for (int o = 0; o < OWN; ++o)
                if (am & (1u << o)) U[f * EN + q0 + o * EX] = xo[f][o];
            if (rn) U[f * EN + rq] = xn[f];
        }
    };

    // the ring's published values
    auto ring_pub = [&](T* src, T* csrc, T (&x)[F]) {
        const int rg = fresh(o_rg), rc = fresh(o_rc);
#pragma unroll
        for (int f = 0; f < F; ++f) {
            x[f] = (T)0;
            if (rc >= 0) x[f] = ld_c(ato(csrc + (size_t)F * co + (size_t)f * cl, rc));
            else if (rdep) x[f] = ld_c(ato(src + (size_t)F * no + (size_t)f * nn, rg));
        }
    };
    // a thread's values of one field on the column strips: its rows are one run
    auto col_pub = [&](T* dst, int f, const T (&x)[OWN]) {
        const int cc = fresh(o_cc);
        if (cc < 0) return;
        T* const q = ato(dst + (size_t)F * co + (size_t)f * cl, cc);
        if (OWN * sizeof(T) == 16 && am == (1u << OWN) - 1) {   // one 16-byte store
            float v[4];
            __builtin_memcpy(v, &x[0], 16);
            st4f<kCoherent>(mkrs(dst + (size_t)F * co + (size_t)f * cl, (size_t)cl * sizeof(T)),
                            cc * (int)sizeof(T), 0, v);
            return;
        }
#pragma unroll
        for (int o = 0; o < OWN; ++o)
            if (am & (1u << o)) st_c(q + o, x[o]);
    };
    // p = u + beta p, d += alpha p, s = w + beta s, r -= alpha s, at the own nodes and the ring
    auto update = [&](uint32_t im, const T (&uo)[F][OWN], const T (&un)[F], const T (&wn)[F]) {
#pragma unroll
        for (int f = 0; f < F; ++f) {
            if (!(im & (1u << f))) continue;
            const T al = s_af[k * F + f], be = s_bf[k * F + f];
            d_get(f);
#pragma unroll
            for (int o = 0; o < OWN; ++o) {
                vp[f][o] = fma_t(be, vp[f][o], uo[f][o]);
                vd[f][o] = fma_t(al, vp[f][o], vd[f][o]);
                vs[f][o] = fma_t(be, vs[f][o], vw[f][o]);
                vr[f][o] = fma_t(-al, vs[f][o], vr[f][o]);
            }
            d_put(f);
            np_[f] = fma_t(be, np_[f], un[f]);
            nd[f] = fma_t(al, np_[f], nd[f]);
            ns[f] = fma_t(be, ns[f], wn[f]);
            nr[f] = fma_t(-al, ns[f], nr[f]);
        }
    };

    bool alive = true;
    int ex = 0;   // pubW parity written next
    for (int outer = 0; alive; ++outer) {
        // ---- residual phase: x += D^-1/2 d (outer > 0), r = D^-1/2 (b - M x), FP64 ----
        for (int i = g; i < a.ntiles; i += G) {
            if (!keep) set_tile(i);
            uint32_t todo = 0;
#pragma unroll
            for (int f = 0; f < F; ++f)
                if (!s_done[k * F + f]) todo |= 1u << f;
            if (!todo) continue;
            double pr[NV];   // ||r||^2, ||b||^2 (first pass), ||D^-1/2 r||^2
#pragma unroll
            for (int q = 0; q < NV; ++q) pr[q] = 0.0;
            double* const X = reinterpret_cast<double*>(ub);
            T c7[OWN][7], bo[F][OWN], wo[OWN], rb[F], rw = (T)1, rd = (T)1;
            {
                const int g0 = fresh(o_g0), rg = fresh(o_rg);
                const T* C = a.coef + (size_t)4 * no;
                const int dw = i0 + col == 0 ? nx - 1 : -1;
#pragma unroll
                for (int o = 0; o < OWN; ++o) {
                    const bool on = am & (1u << o);
                    const int kk = on ? g0 + o * nx : 0;
                    const int kw = on ? kk + dw : 0;
                    const int ds = j0 + row0 + o == 0 ? nn - nx : -nx;
                    const int ks = on ? kk + ds : 0, kd = on ? kw + ds : 0;
                    c7[o][0] = ldo(C, kk);
                    c7[o][1] = ldo(C + nn, kk);
                    c7[o][2] = ldo(C + nn, kw);
                    c7[o][3] = ldo(C + (size_t)2 * nn, kk);
                    c7[o][4] = ldo(C + (size_t)2 * nn, ks);
                    c7[o][5] = ldo(C + (size_t)3 * nn, kk);
                    c7[o][6] = ldo(C + (size_t)3 * nn, kd);
                    wo[o] = ldo(a.w + no, kk);
#pragma unroll
                    for (int f = 0; f < F; ++f) bo[f][o] = ldo(a.b + (size_t)F * no + (size_t)f * nn, kk);
                }
                if (rdep == 1) {
                    rw = ldo(a.w + no, rg);
                    rd = ldo(C, rg);
                }
#pragma unroll
                for (int f = 0; f < F; ++f)
                    rb[f] = rdep == 1 ? ldo(a.b + (size_t)F * no + (size_t)f * nn, rg) : (T)0;
                if (STREAM) {
                    const Vec t = *reinterpret_cast<const Vec*>(a.rsd + (size_t)tile * NTN +
                                                                (size_t)tid * OWN);
#pragma unroll
                    for (int o = 0; o < OWN; ++o) rsl[o * NT + tid] = t.v[o];
                }
            }
            const T rsr = rs_of(rd, !(rw > (T)0));
            T rso[OWN];
#pragma unroll
            for (int o = 0; o < OWN; ++o) rso[o] = DL ? rs_of(c7[o][0], false) : rsl[o * NT + tid];
#pragma unroll
            for (int f = 0; f < F; ++f) {
                if (!(todo & (1u << f))) {
#pragma unroll
                    for (int o = 0; o < OWN; ++o) vr[f][o] = (T)0;
                    continue;
                }
                const int p = k * F + f;
                const bool hf = s_held[p] != 0, st = outer > 0 && !s_last[p];
                const int g0 = fresh(o_g0), q0 = fresh(o_q0), rq = fresh(o_rq);
                const size_t qf = (size_t)F * no + (size_t)f * nn;
                double* const xr = a.xring + ((size_t)tile * F + f) * NRP + tid;
                double xo[OWN], xn = 0.0;
                if (hf) {
#pragma unroll
                    for (int o = 0; o < OWN; ++o)
                        xo[o] = ldo(a.x64 + qf, (am & (1u << o)) ? g0 + o * nx : 0);
                    if (rdep == 1) xn = *xr;
                } else {
                    xn = rdep == 1 ? own_start(rb[f], rw) : 0.0;
#pragma unroll
                    for (int o = 0; o < OWN; ++o) xo[o] = own_start(bo[f][o], wo[o]);
                }
                if (outer > 0) {
                    if (STREAM) {
                        ld_own(1, f, vd[f]);
                        if (rdep == 1) nd[f] = *ring_at(1, f);
                    }
                    d_get(f);
                    xn += (double)mul_t(nd[f], rsr);
#pragma unroll
                    for (int o = 0; o < OWN; ++o) xo[o] += (double)mul_t(vd[f][o], rso[o]);
                }
#pragma unroll
                for (int o = 0; o < OWN; ++o)
                    if (am & (1u << o)) X[q0 + o * EX] = xo[o];
                if (rdep == 1) X[rq] = xn;
                __syncthreads();
                if (outer > 0) {
                    if (st && rdep == 1) *xr = xn;
#pragma unroll
                    for (int o = 0; o < OWN; ++o) {
                        if (!(am & (1u << o))) continue;
                        if (st) *ato(a.x64 + qf, g0 + o * nx) = xo[o];
                        *ato(out + (size_t)f * nn, g0 + o * nx) = (T)xo[o];
                    }
                }
#pragma unroll
                for (int o = 0; o < OWN; ++o) {
                    const int q = q0 + o * EX;
                    const double mx = stencil_x(c7[o], xo[o], X[q + 1], X[q - 1], X[q + EX],
                                                X[q - EX], X[q + EX + 1], X[q - EX - 1]);
                    const bool on = am & (1u << o);
                    const double bk = on ? (double)bo[f][o] : 0.0;
                    const double r64 = on ? bk - mx : 0.0;
                    pr[f] = sq_acc(pr[f], r64);
                    if (outer == 0) pr[F + f] = sq_acc(pr[F + f], bk);
                    vr[f][o] = mul_t((T)r64, rso[o]);
                    const T rk = fresh(vr[f][o]);
                    pr[2 * F + f] = dot_t(pr[2 * F + f], rk, rk);
                    if (sm & (1u << o)) st_c(ato(a.pubR + qf, g0 + o * nx), vr[f][o]);
                }
                col_pub(a.colR, f, vr[f]);
                if (STREAM) st_own(3, f, vr[f]);
                __syncthreads();
            }
            store_sums(pr, NV);
        }
        T wn[F];   // the ring's published values, loaded beside the partials
        alive = reduce(NV, [&] {
            if (keep) ring_pub(a.pubR, a.colR, wn);
        });
        if (!alive) break;
        int more = 0;
        for (int p = tid; p < a.nprob * F; p += NT) {   // one thread per (instance, field)
            const int kk = BATCH ? p / F : 0, f = p - kk * F;
            if (s_done[p]) continue;
            s_refines[p] += 1;
            // (read here: in the comparison below it makes the 64 x 64 tile spill more, 2.40 ->
            // 2.43 ms at 2048^2 nodes)
            const int own = s_more[p], counted = outer - ((own + 1) >> 1);   // less its two bits
            const double rr = vals[kk * NV + f];
            if (outer == 0) s_bb[p] = vals[kk * NV + F + f];
            const double bb = s_bb[p];
            const double relres = bb == 0.0 ? 0.0 : sqrt(rr / bb);
            s_relres[p] = relres;
            if (bb == 0.0) {
                s_zero[p] = 1;
                s_done[p] = 1;
            } else if (relres <= a.opts.tol || counted >= a.opts.max_refine ||
                       s_iters[p] >= a.opts.maxit || !(relres == relres)) {
                s_done[p] = 1;
                if (!(relres <= a.opts.tol)) atomicOr(&s_flags[kk], (uint32_t)P2M_FLAG_NOT_CONVERGED);
            } else {
                // a goal within a thirtieth of the inner reduction is gone for at once:
                // a residual phase costs more than the last iteration it would save
                // (FP64: half of that again, as its answer's error is the residual's: a step of
                // five products may pass the goal only just)
                const double goal = (sizeof(T) == 8 ? 0.0625 : 0.25) * a.opts.tol * a.opts.tol * bb;
                const double rel = a.opts.inner_rtol * a.opts.inner_rtol * rr;
                const bool direct = goal * 900.0 >= rel;
                // the inner solve measures its residual in the scaled norm
                s_target[p] = (direct ? goal : rel) * (vals[kk * NV + 2 * F + f] / rr);
                // x + d was not stored if this residual was expected to be the last
                s_held[p] |= outer > 0 ? (s_last[p] ? 2 : 1) : 0;
                s_last[p] = direct;
                s_more[p] = own | (direct ? 2 : 0);
                s_inner[p] = 1;
                s_best[p] = 3.0e38f;
                s_since[p] = 0;
                more |= s_held[p] & 2 ? 3 : 1;
            }
        }
        const int left_out = __syncthreads_or(more & 2);   // (its result is 0 or 1)
        if (!__syncthreads_or(more)) break;
        // x += d where the residual phase left it out and the solve goes on after all
        if (left_out) {
            for (int i = g; i < a.ntiles; i += G) {
                if (!keep) set_tile(i);
                const int g0 = fresh(o_g0), rg = fresh(o_rg);
                const T* C = a.coef + (size_t)4 * no;
                const T* w = a.w + no;
                const T rsr = rdep == 1 ? rs_of(ldo(C, rg), !(ldo(w, rg) > (T)0)) : (T)1;
#pragma unroll
                for (int f = 0; f < F; ++f) {
                    const int p = k * F + f;
                    if (!s_inner[p] || !(s_held[p] & 2)) continue;
                    const bool hf = s_held[p] & 1;
                    d_get(f);
                    const size_t q = (size_t)F * no + (size_t)f * nn;
                    if (!keep) {
                        ld_own(1, f, vd[f]);
                        if (rdep == 1) nd[f] = *ring_at(1, f);
                    }
#pragma unroll
                    for (int o = 0; o < OWN; ++o) {
                        if (!(am & (1u << o))) continue;
                        const int kk = g0 + o * nx;
                        const double x = hf ? ldo(a.x64 + q, kk) : own_start(ldo(a.b + q, kk), ldo(w, kk));
                        *ato(a.x64 + q, kk) = x + (double)mul_t(vd[f][o], rs_of(ldo(C, kk), !(ldo(w, kk) > (T)0)));
                    }
                    if (rdep == 1) {
                        double* const xr = a.xring + ((size_t)tile * F + f) * NRP + tid;
                        *xr = (hf ? *xr : start_value(f, rg)) + (double)mul_t(nd[f], rsr);
                    }
                }
            }
            __syncthreads();
            for (int p = tid; p < a.nprob * F; p += NT)
                if (s_held[p] & 2) s_held[p] = 1;
            __syncthreads();
        }

        // ---- inner iterations; the first only forms u, w and their products ------
        if (keep) {
#pragma unroll
            for (int f = 0; f < F; ++f) {
                nr[f] = wn[f];
                np_[f] = nd[f] = ns[f] = (T)0;
#pragma unroll
                for (int o = 0; o < OWN; ++o) vp[f][o] = vd[f][o] = vs[f][o] = (T)0;
                d_put(f);
            }
        }
        uint32_t dm = 0;    // fields whose polynomial is 1
        bool poly = true;   // any active one's is not
        for (int it = 0;; ++it) {
            for (int i = g; i < a.ntiles; i += G) {
                if (!keep) set_tile(i);
                const uint32_t im = inner_mask();
                if (!im) continue;
                const int g0 = fresh(o_g0);
                if (!keep) load_img();
                if (STREAM) {
                    T uo[F][OWN], un[F];
                    ring_pub(it == 0 ? a.pubR : a.pubW[ex ^ 1], it == 0 ? a.colR : a.colW[ex ^ 1], wn);
#pragma unroll
                    for (int f = 0; f < F; ++f) {
                        np_[f] = nd[f] = ns[f] = un[f] = (T)0;
                        nr[f] = it == 0 ? wn[f] : (T)0;
#pragma unroll
                        for (int o = 0; o < OWN; ++o) vp[f][o] = vd[f][o] = vs[f][o] = (T)0;
                        if (!(im & (1u << f))) continue;
                        ld_own(3, f, vr[f]);
                        if (it == 0) continue;
                        ld_own(4, f, vw[f]);
                        if (rdep) nr[f] = *ring_at(3, f);
                        if (kSkip && s_diag[k * F + f]) {   // u = r
#pragma unroll
                            for (int o = 0; o < OWN; ++o) uo[f][o] = vr[f][o];
                            un[f] = nr[f];
                        } else {
                            ld_own(5, f, uo[f]);
                            if (rdep == 1) un[f] = *ring_at(4, f);
                        }
                        if (it == 1) continue;   // p = d = s = 0 so far
                        ld_own(0, f, vp[f]);
                        ld_own(1, f, vd[f]);
                        ld_own(2, f, vs[f]);
                        if (rdep) ns[f] = *ring_at(2, f);
                        if (rdep == 1) {
                            np_[f] = *ring_at(0, f);
                            nd[f] = *ring_at(1, f);
                        }
                    }
                    if (it > 0) update(im, uo, un, wn);
                }
                // u = p(A) r by Horner's rule (PH is odd: u ends in bA), w = A u
                static_assert(PH % 2 == 1, "u in bA");
                if (BATCH || STREAM || it == 0) {   // (a field stalls at the end of an inner solve)
                    dm = 0;
#pragma unroll
                    for (int f = 0; f < F; ++f)
                        if (s_diag[k * F + f]) dm |= 1u << f;
                    dm = __builtin_amdgcn_readfirstlane(dm);
                    if (F == 1) poly = dm == 0;
                }
                if (F > 1) poly = !kSkip || __builtin_amdgcn_readfirstlane(im & ~dm) != 0;
                T qo[F][OWN], qn[F];
                put(bA, im, vr, rdep != 0, nr);
                __syncthreads();
#pragma unroll
                for (int j = 1; j < PH; ++j) {
                    if (__builtin_expect(!poly, 0)) break;   // the products would only be multiplied by 0
                    const bool rn = rdep >= 1 && rdep <= PH - j;
                    apply(j & 1 ? bA : bB, im, rn, qo, qn);
#pragma unroll
                    for (int f = 0; f < F; ++f) {
                        if (!(im & (1u << f))) continue;
                        const bool one = dm & (1u << f);
                        const T cj = one ? (T)(j == PH - 1) : pc[PH - 1 - j], ct = one ? (T)0 : pc[PH - 1];
#pragma unroll
                        for (int o = 0; o < OWN; ++o)
                            qo[f][o] = j == 1 ? fma_t(ct, qo[f][o], mul_t(cj, vr[f][o]))
                                              : fma_t(cj, vr[f][o], qo[f][o]);
                        qn[f] = j == 1 ? fma_t(ct, qn[f], mul_t(cj, nr[f])) : fma_t(cj, nr[f], qn[f]);
                    }
                    if (!PP) __syncthreads();
                    put(j & 1 ? bB : bA, im, qo, rn, qn);
                    if (j < PH - 1) __syncthreads();
                }
                if (!keep) {
#pragma unroll
                    for (int f = 0; f < F; ++f) {
                        if (!(im & (1u << f))) continue;
                        if (!kSkip || !(dm & (1u << f))) {
                            st_own(5, f, qo[f]);
                            if (rdep == 1) *ring_at(4, f) = qn[f];
                        }
                        if (it > 0) {
                            st_own(0, f, vp[f]);
                            st_own(1, f, vd[f]);
                            st_own(2, f, vs[f]);
                            st_own(3, f, vr[f]);
                            if (rdep) *ring_at(2, f) = ns[f];
                            if (rdep == 1) {
                                *ring_at(0, f) = np_[f];
                                *ring_at(1, f) = nd[f];
                            }
                        }
                        if (rdep) *ring_at(3, f) = nr[f];
                    }
                }
                __syncthreads();
                apply(bA, im, false, qo, qn);
                const int q0 = fresh(o_q0);
                double pd[NV];
#pragma unroll
                for (int q = 0; q < NV; ++q) pd[q] = 0.0;
#pragma unroll
                for (int f = 0; f < F; ++f) {
                    if (!(im & (1u << f))) {
#pragma unroll
                        for (int o = 0; o < OWN; ++o) vw[f][o] = (T)0;
                        continue;
                    }
#pragma unroll
                    for (int o = 0; o < OWN; ++o) {
                        const bool on = am & (1u << o);
                        vw[f][o] = on ? qo[f][o] : (T)0;
                        if (sm & (1u << o))
                            st_c(ato(a.pubW[ex] + (size_t)F * no + (size_t)f * nn, g0 + o * nx), vw[f][o]);
                        const T uk = on ? bA[f * EN + q0 + o * EX] : (T)0;
                        // opaque: its conversion to FP64 is made here, not carried along with r
                        const T rk = fresh(vr[f][o]);
                        pd[f] = dot_t(pd[f], rk, uk);
                        pd[F + f] = dot_t(pd[F + f], vw[f][o], uk);
                        pd[2 * F + f] = dot_t(pd[2 * F + f], rk, rk);
                    }
                    col_pub(a.colW[ex], f, vw[f]);
                    if (!keep) st_own(4, f, vw[f]);
                }
                store_sums(pd, NV);
            }
            ex ^= 1;
            alive = reduce(NV, [&] {
                if (keep) ring_pub(a.pubW[ex ^ 1], a.colW[ex ^ 1], wn);
            });
            if (!alive) break;
            more = 0;
            for (int p = tid; p < a.nprob * F; p += NT) {
                const int kk = BATCH ? p / F : 0, f = p - kk * F;
                if (!s_inner[p]) continue;
                const double gam = vals[kk * NV + f], del = vals[kk * NV + F + f],
                             rho = vals[kk * NV + 2 * F + f];
                double den = del;
                double beta = 0.0;
                if (it > 0) {
                    s_iters[p] += 1;
                    // An ill-conditioned system's recurrence can stall above its target and
                    // then run away from the true residual.  When kStall iterations brought
                    // nothing, or the residual has grown by 10, it starts again from the true
                    // one, with the diagonal alone, whose rounding such systems bear.
                    // (As a ratio to the target: (r,r) itself may leave FP32's range.)
                    const float at = (float)(rho / s_target[p]);
                    if (at < s_best[p]) {
                        s_best[p] = at;
                        s_since[p] = 0;
                    } else if (!s_diag[p] && (++s_since[p] >= kStall ||
                                              (s_since[p] >= 8 && at > 100.f * s_best[p]))) {
                        s_diag[p] = 1;
                        s_more[p] |= 1;
                        s_inner[p] = 0;
                        continue;
                    }
                    if (!(rho > s_target[p]) || s_iters[p] >= a.opts.maxit) {
                        s_inner[p] = 0;
                        continue;
                    }
                    beta = gam / s_gam[p];
                    den = del - beta * gam / s_alpha[p];
                }
                if (!(den > 0.0) || !(gam > 0.0)) {
                    s_inner[p] = 0;
                    atomicOr(&s_flags[kk], (uint32_t)P2M_FLAG_BREAKDOWN);
                    if (it == 0) {
                        s_done[p] = 1;
                        atomicOr(&s_flags[kk], (uint32_t)P2M_FLAG_NOT_CONVERGED);
                    }
                    continue;
                }
                s_alpha[p] = gam / den;
                s_gam[p] = gam;
                s_af[p] = (T)s_alpha[p];
                s_bf[p] = (T)beta;
                more = 1;
            }
            if (!__syncthreads_or(more)) break;
            if (keep) {
                const uint32_t im = inner_mask();
                const int q0 = fresh(o_q0), rq = fresh(o_rq);
                T uo[F][OWN], un[F];
#pragma unroll
                for (int f = 0; f < F; ++f) {
#pragma unroll
                    for (int o = 0; o < OWN; ++o) uo[f][o] = bA[f * EN + q0 + o * EX];
                    un[f] = rdep == 1 ? bA[f * EN + rq] : (T)0;
                }
                update(im, uo, un, wn);
            }
        }
    }

    if (!alive)
        for (int kk = tid; kk < a.nprob; kk += NT)
            s_flags[kk] |= P2M_FLAG_BREAKDOWN | P2M_FLAG_NOT_CONVERGED;
    __syncthreads();
    // result of the fields that no later residual phase stored (solved by the start,
    // b == 0, an aborted solve): the FP64 solution rounded to T, 0 where b == 0
    for (int i = g; i < a.ntiles; i += G) {
        if (!keep) set_tile(i);
#pragma unroll
        for (int f = 0; f < F; ++f) {
            const int p = k * F + f;
            if (alive && s_refines[p] > 1) continue;
#pragma unroll
            for (int o = 0; o < OWN; ++o) {
                if (!(am & (1u << o))) continue;
                const int kk = fresh(o_g0) + o * nx;
                const size_t q = (size_t)F * no + (size_t)f * nn;
                const double x = s_held[p] ? ldo(a.x64 + q, kk)
                                           : own_start(ldo(a.b + q, kk), ldo(a.w + no, kk));
                *ato(out + (size_t)f * nn, kk) = s_zero[p] ? (T)0 : (T)x;
            }
        }
    }
    if (g == 0) {
        for (int kk = tid; kk < a.nprob; kk += NT) {
            p2m_report* rep = inst_of(kk).rep;
            if (!rep) continue;
            for (int f = 0; f < F; ++f) {
                rep->iters[f] = s_iters[kk * F + f];
                rep->refines[f] = s_refines[kk * F + f];
                rep->rel_residual[f] = s_relres[kk * F + f];
            }
            if (s_flags[kk]) atomicOr(&rep->flags, s_flags[kk]);
        }
    }
}

// barrier counters to zero; with rep, that report too (one launch for both)
__global__ void k_pcg_clear(unsigned* words, int n, p2m_report* rep) {
    for (int t = threadIdx.x; t < n; t += blockDim.x) words[t] = 0u;
    if (rep) {
        const int t = threadIdx.x;
        if (t < 8) {
            rep->iters[t] = 0;
            rep->refines[t] = 0;
            rep->rel_residual[t] = 0.0;
        }
        if (t == 0) {
            rep->flags = 0u;
            rep->n_orphan = 0;
            rep->n_invalid = 0;
            rep->reserved = 0;
        }
    }
}

constexpr int kSyncWords = 2 * kGroups * 32 + 2 * 32;

size_t al(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

template <typename T, class TC, bool BATCH, bool STREAM>
const void* pcg_kernel(int F) {
    switch (F) {
        case 1: return (const void*)k_pcg<T, TC, 1, BATCH, STREAM>;
        case 2: return (const void*)k_pcg<T, TC, 2, BATCH, STREAM>;
        case 3: return (const void*)k_pcg<T, TC, 3, BATCH, STREAM>;
    }
    return nullptr;
}
template <typename T>
const void* pcg_pick(bool small, int depth, bool batch, bool stream, int F) {
    if constexpr (sizeof(T) == 8) {
        if (!small || batch || stream) return nullptr;
        if (depth == TileD::PH) return pcg_kernel<T, TileD, false, false>(F);
        return F == 1 ? (const void*)k_pcg<T, TileS, 1, false, false> : nullptr;
    } else {
        if (depth != (small ? TileS::PH : TileL::PH)) return nullptr;
        if (small && batch)
            return stream ? pcg_kernel<T, TileS, true, true>(F) : pcg_kernel<T, TileS, true, false>(F);
        if (small) return stream ? nullptr : pcg_kernel<T, TileS, false, false>(F);
        if (batch)
            return stream ? pcg_kernel<T, TileL, true, true>(F) : pcg_kernel<T, TileL, true, false>(F);
        return stream ? pcg_kernel<T, TileL, false, true>(F) : pcg_kernel<T, TileL, false, false>(F);
    }
}

// what the host needs to know of a tile
struct TileInfo {
    int nt, own, en, nrp;
};
template <class C>
constexpr TileInfo tile_info() {
    return TileInfo{C::NT, C::TX * C::TY, C::EN, C::NRP};
}
TileInfo tile_of(bool small, int depth) {
    if (!small) return tile_info<TileL>();
    return depth == TileS::PH ? tile_info<TileS>() : tile_info<TileD>();
}

// streamed state per tile, bytes
size_t stream_bytes(int tsize, const TileInfo& t, int F, int ntiles) {
    const size_t n = (size_t)ntiles;
    return al(n * 6 * F * t.own * tsize) + al(n * 5 * F * t.nrp * tsize) + al(n * t.own * tsize) +
           al(n * 3 * t.en * tsize);
}

}  // namespace

// Stencil products of an iteration (the preconditioner's degree + 1).  The small tile takes
// five: at 4 particles per cell 4 iterations for 6 to the same residual, and the barrier,
// the sums and the ring exchange cost as much as two products.  256 x 256, F = 1: the solve
// 80 -> 65 us; 512 x 512 FP64, F = 1: 101 -> 85; two and three fields gain 0 to 2% of a
// pass.  In FP64 two and three fields do not fit the 128 registers of 1024 threads (384 x
// 384, F = 3: pass 224 us with three products on 512 threads, 255 with five); the ring of
// five on the large tile is more slots than it has threads.  FP64 meshes of more tiles than
// the device holds at 1024 threads each (256) take three, twice as many of which it holds.
int pcg_depth(int tsize, bool small, int F) { return small && (tsize == 4 || F == 1) ? 5 : 3; }

// Meshes of at most kPolyTiles small tiles (512 x 512) take the 32 x 32 tile, one per
// compute unit; larger ones the 64 x 64 tile, whose ring is a smaller share of it.  Past the
// line a quarter of the tiles hold four times the nodes and three products replace five, on
// 81 of 256 compute units at first: whole pass at 6 per cell, F = 1 / 3, 512 x 512 99 / 167 us,
// 520 x 520 125 / 265, 640 x 640 138 / 291, 960 x 960 (225 tiles) 189 / 350; by the diagonal
// solve 218 / 396, 220 / 409, 225 / 427, 280 / 498.
bool pcg_small(const Mesh& m) {
    return (int64_t)((m.nx + TileS::TX - 1) / TileS::TX) * ((m.ny + TileS::TY - 1) / TileS::TY) <=
           kPolyTiles;
}
int pcg_tiles(const Mesh& m, bool small, int* per_row) {
    const int tx = small ? TileS::TX : TileL::TX, ty = small ? TileS::TY : TileL::TY;
    const int px = (m.nx + tx - 1) / tx;
    if (per_row) *per_row = px;
    return px * ((m.ny + ty - 1) / ty);
}

void pcg_interval(const Mesh& m, int depth, double pc[5]) {
    const double ppc = (double)m.np / (double)m.nn;
    const double lo = ppc >= 6.0 ? 0.4 : (ppc >= 3.5 ? 0.28 : 0.18);
    const double hi = ppc >= 6.0 ? 2.1 : (ppc >= 3.5 ? 2.3 : 2.5);
    const double de = 0.5 * (hi - lo), s = (hi + lo) / (hi - lo);
    // 1 - l p(l) = T(s - l / de) / T(s), expanded at s
    if (depth == 5) {
        const double s2 = s * s, g = 1.0 / (s * (16.0 * s2 * s2 - 20.0 * s2 + 5.0));
        pc[0] = g * (80.0 * s2 * s2 - 60.0 * s2 + 5.0) / de;
        pc[1] = -g * s * (160.0 * s2 - 60.0) / (de * de);
        pc[2] = g * (160.0 * s2 - 20.0) / (de * de * de);
        pc[3] = -80.0 * g * s / (de * de * de * de);
        pc[4] = 16.0 * g / (de * de * de * de * de);
        return;
    }
    const double g = 1.0 / (4.0 * s * s * s - 3.0 * s);
    pc[0] = g * (12.0 * s * s - 3.0) / de;
    pc[1] = -12.0 * g * s / (de * de);
    pc[2] = 4.0 * g / (de * de * de);
}

namespace {

// Workgroups of a kernel the device holds at once, at most two per compute unit.  Kept per
// device and kernel after the first query (a batch asks once per instance).
constexpr int kMaxDevices = 16;
int resident_groups(const void* fn, int nt, int device, std::atomic<int>* known) {
    if (!fn) return 0;
    if (known) {
        const int v = known->load(std::memory_order_relaxed);
        if (v > 0) return v;
    }
    int cus = 0, per = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, nt, 0) != hipSuccess || per < 1)
        return 0;
    const int v = (per > 2 ? 2 : per) * cus;
    if (known) known->store(v, std::memory_order_relaxed);
    return v;
}

template <typename T>
SolveGrid grid_of(bool small, int depth, bool batch, int F, int ntiles, int device) {
    static std::atomic<int> known[kMaxDevices][2][2][2][2][kResidentMaxFields + 1];
    const int nt = tile_of(small, depth).nt;
    auto held = [&](bool stream) {
        std::atomic<int>* k = device >= 0 && device < kMaxDevices
                                  ? &known[device][small][depth == 5][batch][stream][F] : nullptr;
        return resident_groups(pcg_pick<T>(small, depth, batch, stream, F), nt, device, k);
    };
    const int h = held(false);
    return solve_grid(h, ntiles <= h ? 0 : held(true), ntiles);
}

}  // namespace

SolveGrid pcg_grid(int tsize, bool small, int depth, bool batch, int F, int ntiles, int device) {
    if (F < 1 || F > kResidentMaxFields) return {0, false};
    return tsize == 8 ? grid_of<double>(small, depth, batch, F, ntiles, device)
                      : grid_of<float>(small, depth, batch, F, ntiles, device);
}

int pcg_sync_words() { return kSyncWords; }

size_t pcg_column_elems(const Mesh& m, int depth, int per_row) {
    return (size_t)2 * depth * per_row * m.ny;
}

size_t pcg_workspace_bytes(int tsize, bool small, int depth, int F, int nprob, int ntiles,
                           size_t nodes, size_t cols, bool stream) {
    const TileInfo t = tile_of(small, depth);
    size_t s = al(kSyncWords * sizeof(unsigned)) + al((size_t)2 * 3 * F * ntiles * sizeof(double)) +
               al((size_t)2 * 3 * F * nprob * sizeof(double)) + al((size_t)F * nodes * sizeof(double)) +
               3 * al((size_t)F * nodes * tsize) + 3 * al((size_t)F * cols * tsize) +
               al((size_t)ntiles * F * t.nrp * sizeof(double));
    if (stream) s += stream_bytes(tsize, t, F, ntiles);
    return s;
}

template <typename T>
hipError_t launch_pcg(const PolySolve<T>& ps, int start, const p2m_solve_opts& opts, hipStream_t stream) {
    const bool batch = ps.inst != nullptr;
    const void* fn = pcg_pick<T>(ps.small, ps.depth, batch, ps.grid.stream, ps.F);
    if (!fn || ps.grid.groups < 1 || ps.nprob < 1 || (batch && ps.nprob * ps.F > kBatchMaxPairs))
        return hipErrorInvalidValue;
    const int F = ps.F;
    const TileInfo t = tile_of(ps.small, ps.depth);
    char* p = (char*)ps.ws;
    auto take = [&](size_t bytes) {
        char* q = p;
        p += al(bytes);
        return q;
    };
    PArgs<T> a;
    memset(&a, 0, sizeof(a));
    a.one = ps.one;
    a.inst = ps.inst;
    a.rmap = ps.rmap;
    a.order = ps.order;
    a.nprob = ps.nprob;
    a.ntiles = ps.ntiles;
    a.coef = ps.coef;
    a.b = ps.b;
    a.w = ps.w;
    a.start = start;
    a.opts = opts;
    unsigned* words = (unsigned*)take(kSyncWords * sizeof(unsigned));
    a.sy.ctr = words;
    a.sy.root = words + kGroups * 32;
    a.sy.rel = words + kGroups * 32 + 32;
    a.sy.abort = words + 2 * kGroups * 32 + 32;
    a.sy.part = (double*)take((size_t)2 * 3 * F * ps.ntiles * sizeof(double));
    a.sy.tot = (double*)take((size_t)2 * 3 * F * ps.nprob * sizeof(double));
    a.sy.spin = ps.spin;
    a.x64 = (double*)take((size_t)F * ps.nodes * sizeof(double));
    a.pubR = (T*)take((size_t)F * ps.nodes * sizeof(T));
    a.pubW[0] = (T*)take((size_t)F * ps.nodes * sizeof(T));
    a.pubW[1] = (T*)take((size_t)F * ps.nodes * sizeof(T));
    a.colR = (T*)take((size_t)F * ps.cols * sizeof(T));
    a.colW[0] = (T*)take((size_t)F * ps.cols * sizeof(T));
    a.colW[1] = (T*)take((size_t)F * ps.cols * sizeof(T));
    a.xring = (double*)take((size_t)ps.ntiles * F * t.nrp * sizeof(double));
    if (ps.grid.stream) {
        const size_t n = (size_t)ps.ntiles;
        a.own = (T*)take(n * 6 * F * t.own * sizeof(T));
        a.ring = (T*)take(n * 5 * F * t.nrp * sizeof(T));
        a.rsd = (T*)take(n * t.own * sizeof(T));
        a.cimg = (T*)take(n * 3 * t.en * sizeof(T));
    }
    if (!ps.cleared || ps.clear_rep) {
        hipLaunchKernelGGL(k_pcg_clear, dim3(1), dim3(256), 0, stream, words, kSyncWords, ps.clear_rep);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // An ordinary launch: the stream has finished every earlier kernel and the grid is
    // at most what the device holds at once (pcg_grid), so all its workgroups are
    // resident; the barrier is the kernel's own and every wait in it is bounded.
    void* args[] = {&a};
    return hipLaunchKernel(fn, dim3(ps.grid.groups), dim3(t.nt), args, 0, stream);
}
template hipError_t launch_pcg<float>(const PolySolve<float>&, int, const p2m_solve_opts&, hipStream_t);
template hipError_t launch_pcg<double>(const PolySolve<double>&, int, const p2m_solve_opts&, hipStream_t);

}  // namespace p2m
