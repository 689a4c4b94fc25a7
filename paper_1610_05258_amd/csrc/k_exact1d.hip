// The paper-exact 1D assignments (Table 1; Sec. 2.4 eq. (20); Appendix B), FP64.
//
// In 1D the particle "triangulation" of Sec. 2 is the order of the particles
// along the periodic segment, and the particle hat psi_mu is the P1 hat on the
// sorted particles (Sec. 3.1).  Every integral is the exact integral of that
// particle interpolant or of the mesh interpolant against the hats, either
// exactly (both factors are linear between merged breakpoints, so Simpson's
// rule on each piece is exact) or with the Appendix-B rule (on every gap of the
// target hats, the parabola through the source interpolant at both ends and the
// midpoint, integrated exactly against the two hats of the gap).
//
// The kernels, in call order (N, the number of located particles, stays on the device: a
// call has no host synchronisation; grids are sized for every particle):
//   k_x1d_sort     wrapped position of every binned particle (sort key); per cell,
//                  (position, particle number) order: cells of up to 32 particles by
//                  their own thread, larger ones by the whole workgroup with the merge
//                  network of the binning sort
//   k_x1d_setup    gaps g_k, volumes v_k = (g_{k-1} + g_k) / 2 (eq. (4)) and the
//                  values in sorted order
//   k_x1d_nodes    the particle interpolant at every node, with the Appendix-B rule
//                  c_j = int A psi_j (mesh hats), and the mesh mass matrix 2h/3, h/6
//   k_x1d_parts    the mesh interpolant at every particle, with the Appendix-B rule
//                  c'_mu = int Abar psi_mu (particle hats), and the particle mass matrix
//                  (g_{k-1} + g_k)/3, g_k/6 (cyclic tridiagonal)
//   k_x1d_c_exact / k_x1d_cp_exact + k_x1d_c_sum
//                  c and c' by exact overlaps instead
//   (k_x1d_small does binning, k_x1d_sort, k_x1d_setup and k_x1d_nodes or k_x1d_parts of a
//   small problem in one launch)
//   k_x1d_div / k_x1d_scatter
//                  lumped divisions and the result in caller order
// The mass solves themselves run in the streaming kernel (k_cg.hip, by cyclic reduction)
// on these stencils.
//
// Bound: launches.  64 cells, 256 particles, there and back: 20 launches and two host
// synchronisations took 158 us; 11 launches and none take 45 us.
#include "p2m_internal.hpp"

namespace p2m {

namespace {

constexpr int kB = 256;
constexpr int kSortSmall = 32;

inline int grid_of(size_t n) { return (int)((n + kB - 1) / kB); }

// position wrapped into [0, L): valid inputs satisfy 0 <= x < L + h
__device__ __forceinline__ double wrap_pos(double x, double L) { return x < L ? x : x - L; }

__device__ __forceinline__ bool pair_less(double ka, int ia, double kb, int ib) {
    return ka < kb || (ka == kb && ia < ib);
}

// Sort of one segment of (key, idx) pairs by the whole workgroup: the bitonic
// network whose comparators all put the smaller pair at the lower index (each
// merge first compares i with its mirror, then half-cleans), with comparators
// beyond the segment skipped (virtual +infinity padding never moves).
template <int BLOCK>
__device__ void block_sort_pairs(double* key, int32_t* idx, int n) {
    int P = 1;
    while (P < n) P <<= 1;
    for (int k = 2; k <= P; k <<= 1) {
        const int half = k >> 1;
        for (int q = threadIdx.x; q < P / 2; q += BLOCK) {
            const int blk = q / half, off = q - blk * half;
            const int i = blk * k + off, j = blk * k + k - 1 - off;
            if (j < n && pair_less(key[j], idx[j], key[i], idx[i])) {
                const double tk = key[i];
                const int ti = idx[i];
                key[i] = key[j];
                idx[i] = idx[j];
                key[j] = tk;
                idx[j] = ti;
            }
        }
        __syncthreads();
        for (int d = k >> 2; d >= 1; d >>= 1) {
            for (int q = threadIdx.x; q < P / 2; q += BLOCK) {
                const int blk = q / d;
                const int i = blk * 2 * d + (q - blk * d), j = i + d;
                if (j < n && pair_less(key[j], idx[j], key[i], idx[i])) {
                    const double tk = key[i];
                    const int ti = idx[i];
                    key[i] = key[j];
                    idx[i] = idx[j];
                    key[j] = tk;
                    idx[j] = ti;
                }
            }
            __syncthreads();
        }
    }
}

// insertion sort of the n (at most kSortSmall) pairs from s on
__device__ __forceinline__ void insertion_sort(double* key, int32_t* idx, int s, int n) {
    for (int i = s + 1; i < s + n; ++i) {
        const double kv = key[i];
        const int iv = idx[i];
        int j = i - 1;
        while (j >= s && pair_less(kv, iv, key[j], idx[j])) {
            key[j + 1] = key[j];
            idx[j + 1] = idx[j];
            --j;
        }
        key[j + 1] = kv;
        idx[j + 1] = iv;
    }
}

// Every cell's (key, idx) pairs in ascending (key, idx) order.
__global__ __launch_bounds__(kB) void k_x1d_sort(int ncells, const double* __restrict__ x, double L,
                                                 const int32_t* __restrict__ perm,
                                                 const int32_t* __restrict__ cs, double* key,
                                                 int32_t* idx) {
    __shared__ int big[kB];
    __shared__ int n_big;
    const int c0 = blockIdx.x * kB;
    const int last = cs[min(c0 + kB, ncells)];
    for (int k = cs[c0] + (int)threadIdx.x; k < last; k += kB) {
        const int p = perm[k];
        key[k] = wrap_pos(x[p], L);
        idx[k] = p;
    }
    const int c = c0 + (int)threadIdx.x;
    if (threadIdx.x == 0) n_big = 0;
    __syncthreads();
    int s = 0, n = 0;
    if (c < ncells) {
        s = cs[c];
        n = cs[c + 1] - s;
    }
    if (n > kSortSmall) {
        big[atomicAdd(&n_big, 1)] = c;   // any order: cells are independent
    } else if (n > 1) {
        insertion_sort(key, idx, s, n);
    }
    __syncthreads();
    const int nb = n_big;
    for (int k = 0; k < nb; ++k) {
        const int cc = big[k];
        const int bs = cs[cc];
        block_sort_pairs<kB>(key + bs, idx + bs, cs[cc + 1] - bs);
    }
}

// particle p was left out of the binning of N particles (N = 0: all were).  Asked before
// anything is written to the caller: a result may lie over the positions.
__device__ __forceinline__ bool left_out(const Mesh& m, const double* __restrict__ x, int p, int N) {
    int c;
    double xi;
    bool fin;
    return N == 0 || !locate_axis(x[p], m.nx, m.inv_hx, c, xi, fin);
}

__device__ __forceinline__ void setup_at(int k, int N, double L, const double* key, const int32_t* idx,
                                         const double* __restrict__ values, int F, int np, double* gap,
                                         double* vol_s, double* vol_c, double* As) {
    const double xk = key[k];
    const double g = (k + 1 < N) ? key[k + 1] - xk : (key[0] + L) - xk;
    const double gm = (k > 0) ? xk - key[k - 1] : (key[0] + L) - key[N - 1];
    gap[k] = g;
    const double v = 0.5 * (g + gm);
    vol_s[k] = v;
    const int p = idx[k];
    vol_c[p] = v;
    for (int f = 0; f < F; ++f) As[(size_t)f * N + k] = values[(size_t)f * np + p];
}

// gaps, volumes (eq. (4)) and values in sorted order; volumes also in caller order (NaN
// for the particles left out, where x is given)
__global__ void k_x1d_setup(Mesh m, const double* __restrict__ x, const int32_t* __restrict__ dN, double L, const double* __restrict__ key,
                            const int32_t* __restrict__ idx, const double* __restrict__ values,
                            int F, int np, double* __restrict__ gap, double* __restrict__ vol_s,
                            double* __restrict__ vol_c, double* __restrict__ As) {
    const int k = blockIdx.x * kB + threadIdx.x, N = *dN;
    if (x && k < np && left_out(m, x, k, N)) vol_c[k] = __builtin_nan("");
    if (k < N) setup_at(k, N, L, key, idx, values, F, np, gap, vol_s, vol_c, As);
}

// the periodic piecewise-linear interpolant through (key[k], A[k]) at y in [0, L)
__device__ __forceinline__ double interp_sorted(const double* key, const double* A, int N, double L,
                                                double y) {
    // a: the last knot with key <= y (none: the last knot, one period back)
    int lo = 0, hi = N;   // first index with key > y
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (key[mid] <= y) lo = mid + 1;
        else hi = mid;
    }
    const int a = lo - 1;
    double xa, xb, fa, fb;
    if (a < 0) {
        xa = key[N - 1] - L;
        fa = A[N - 1];
        xb = key[0];
        fb = A[0];
    } else {
        xa = key[a];
        fa = A[a];
        if (a + 1 < N) {
            xb = key[a + 1];
            fb = A[a + 1];
        } else {
            xb = key[0] + L;
            fb = A[0];
        }
    }
    const double slope = (fb - fa) / (xb - xa);
    return slope * (y - xa) + fa;
}

// node j at j h (h = L / n), its gap to the next node (the last one ends at L)
__device__ __forceinline__ double node_x(int j, double h) { return (double)j * h; }
__device__ __forceinline__ double node_gap(int j, int n, double h, double L) {
    return (j + 1 < n ? node_x(j + 1, h) : L) - node_x(j, h);
}

// Particle interpolant at node j, every field, to fn (if not null).  appb: the Appendix-B
// rule on the mesh hats, c_j = g_j/6 (f(x_j) + 2 f(m_j)) + g_{j-1}/6 (f(x_j) + 2 f(m_{j-1}))
// with m_j the midpoint of element j (both of a node's midpoints are evaluated here:
// cheaper than a launch between).  coef, w (if not null): the consistent mesh mass matrix
// of 1D P1 hats, 2h/3 on the diagonal, h/6 beside it; w = h (no orphans).
__device__ __forceinline__ void nodes_at(int j, int n, double h, double L, int N, const double* key,
                                         const double* As, int F, int appb, double* fn, double* c,
                                         double* coef, double* w) {
    const int jm = j > 0 ? j - 1 : n - 1;
    const double g = node_gap(j, n, h, L), gm = node_gap(jm, n, h, L);
    const double xj = node_x(j, h);
    for (int f = 0; f < F; ++f) {
        const double* A = As + (size_t)f * N;
        const double fj = N > 0 ? interp_sorted(key, A, N, L, xj) : 0.0;
        if (fn) fn[(size_t)f * n + j] = fj;
        if (!appb) continue;
        const double fm = N > 0 ? interp_sorted(key, A, N, L, wrap_pos(xj + 0.5 * g, L)) : 0.0;
        const double fmm =
            N > 0 ? interp_sorted(key, A, N, L, wrap_pos(node_x(jm, h) + 0.5 * gm, L)) : 0.0;
        const double own = g / 6.0 * (fj + 2.0 * fm);
        const double prev = gm / 6.0 * (fj + 2.0 * fmm);
        c[(size_t)f * n + j] = own + prev;
    }
    if (coef) {
        const double hh = L / (double)n;
        coef[j] = 2.0 * hh / 3.0;
        coef[(size_t)n + j] = hh / 6.0;
        w[j] = hh;
    }
}

__global__ void k_x1d_nodes(int n, double h, double L, const int32_t* __restrict__ dN,
                            const double* __restrict__ key, const double* __restrict__ As, int F,
                            int appb, double* __restrict__ fn, double* __restrict__ c,
                            double* __restrict__ coef, double* __restrict__ w) {
    const int j = blockIdx.x * kB + threadIdx.x;
    if (j < n) nodes_at(j, n, h, L, *dN, key, As, F, appb, fn, c, coef, w);
}

// Simpson on one piece [a, b] with f linear on it (fm its mean) against the two
// hats of the gap [left, right] that contains the piece
__device__ __forceinline__ void piece(double a, double b, double fa, double fb, double left,
                                      double right, double& to_left, double& to_right) {
    const double span = right - left;
    const double m = 0.5 * (a + b);
    const double fm = 0.5 * (fa + fb);
    const double la = (right - a) / span, lm = (right - m) / span, lb = (right - b) / span;
    const double h6 = (b - a) / 6.0;
    to_left += h6 * (fa * la + 4.0 * fm * lm + fb * lb);
    to_right += h6 * (fa * (1.0 - la) + 4.0 * fm * (1.0 - lm) + fb * (1.0 - lb));
}

// first index with key > y / with key >= y
__device__ __forceinline__ int upper_idx(const double* __restrict__ key, int N, double y) {
    int lo = 0, hi = N;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (key[mid] <= y) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}
__device__ __forceinline__ int lower_idx(const double* __restrict__ key, int N, double y) {
    int lo = 0, hi = N;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (key[mid] < y) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Exact overlaps with the mesh hats, element by element: element j is cut by the
// particles strictly inside it; er[j] goes to node j, el[j] to node j + 1.
__global__ void k_x1d_c_exact(int n, double h, double L, const int32_t* __restrict__ dN,
                              const double* __restrict__ key,
                              const double* __restrict__ As, int F, const double* __restrict__ fn,
                              double* __restrict__ to_lo, double* __restrict__ to_hi) {
    const int j = blockIdx.x * kB + threadIdx.x, N = *dN;
    if (j >= n) return;
    const double left = node_x(j, h);
    const double right = j + 1 < n ? node_x(j + 1, h) : L;
    const int k0 = upper_idx(key, N, left), k1 = lower_idx(key, N, right);
    for (int f = 0; f < F; ++f) {
        const double* A = As + (size_t)f * N;
        double lo = 0.0, hi = 0.0;
        double a = left, fa = fn[(size_t)f * n + j];
        for (int k = k0; k < k1; ++k) {
            piece(a, key[k], fa, A[k], left, right, lo, hi);
            a = key[k];
            fa = A[k];
        }
        piece(a, right, fa, fn[(size_t)f * n + (j + 1 < n ? j + 1 : 0)], left, right, lo, hi);
        to_lo[(size_t)f * n + j] = lo;
        to_hi[(size_t)f * n + j] = hi;
    }
}

// c_k = to_lo[k] + to_hi[k - 1] (periodic); K = *dK where dK is given
__global__ void k_x1d_c_sum(int K, const int32_t* __restrict__ dK, int F, const double* __restrict__ to_lo,
                            const double* __restrict__ to_hi, double* __restrict__ c) {
    const int k = blockIdx.x * kB + threadIdx.x;
    if (dK) K = *dK;
    if (k >= K) return;
    const int km = k > 0 ? k - 1 : K - 1;
    for (int f = 0; f < F; ++f) c[(size_t)f * K + k] = to_lo[(size_t)f * K + k] + to_hi[(size_t)f * K + km];
}

// the mesh interpolant of nodal values Ab at y in [0, L)
__device__ __forceinline__ double interp_mesh(const double* __restrict__ Ab, int n, double h,
                                              double inv_h, double L, double y) {
    int j = (int)floor(y * inv_h);
    if (j < 0) j = 0;
    if (j > n - 1) j = n - 1;
    while (j > 0 && node_x(j, h) > y) --j;
    while (j + 1 < n && node_x(j + 1, h) <= y) ++j;
    const double xa = node_x(j, h), xb = j + 1 < n ? node_x(j + 1, h) : L;
    const double fa = Ab[j], fb = Ab[j + 1 < n ? j + 1 : 0];
    const double slope = (fb - fa) / (xb - xa);
    return slope * (y - xa) + fa;
}

// Mesh interpolant at every sorted particle to fk (if not null).  appb: the Appendix-B rule
// on the particle hats (both of a particle's gap midpoints are evaluated here).  coef (if
// not null): the consistent particle mass matrix, (g_{k-1} + g_k)/3 and g_k/6.
__device__ __forceinline__ void parts_at(int k, int N, int n, double h, double inv_h, double L,
                                         const double* key, const double* gap, const double* Ab, int F,
                                         int appb, double* fk, double* c, double* coef) {
    const int km = k > 0 ? k - 1 : N - 1;
    const double xk = key[k], g = gap[k], gm = gap[km];
    const double mk = wrap_pos(xk + 0.5 * g, L), mm = wrap_pos(key[km] + 0.5 * gm, L);
    for (int f = 0; f < F; ++f) {
        const double* A = Ab + (size_t)f * n;
        const double fv = interp_mesh(A, n, h, inv_h, L, xk);
        if (fk) fk[(size_t)f * N + k] = fv;
        if (!appb) continue;
        const double own = g / 6.0 * (fv + 2.0 * interp_mesh(A, n, h, inv_h, L, mk));
        const double prev = gm / 6.0 * (fv + 2.0 * interp_mesh(A, n, h, inv_h, L, mm));
        c[(size_t)f * N + k] = own + prev;
    }
    if (coef) {
        coef[k] = gm / 3.0 + g / 3.0;
        coef[(size_t)N + k] = g / 6.0;
    }
}

__global__ void k_x1d_parts(const int32_t* __restrict__ dN, int n, double h, double inv_h, double L,
                            const double* __restrict__ key, const double* __restrict__ gap,
                            const double* __restrict__ Ab, int F, int appb, double* __restrict__ fk,
                            double* __restrict__ c, double* __restrict__ coef) {
    const int k = blockIdx.x * kB + threadIdx.x, N = *dN;
    if (k < N) parts_at(k, N, n, h, inv_h, L, key, gap, Ab, F, appb, fk, c, coef);
}

// Exact overlaps with the particle hats, gap by gap: gap k = [x_k, x_{k+1}] is cut
// by the nodes strictly inside it (the last gap runs past L to x_0 + L)
__global__ void k_x1d_cp_exact(const int32_t* __restrict__ dN, int n, double h, double inv_h, double L,
                               const double* __restrict__ key, const double* __restrict__ gap,
                               const double* __restrict__ Ab, const double* __restrict__ fk, int F,
                               double* __restrict__ to_lo, double* __restrict__ to_hi) {
    const int k = blockIdx.x * kB + threadIdx.x, N = *dN;
    if (k >= N) return;
    const double left = key[k];
    const double right = k + 1 < N ? key[k + 1] : key[0] + L;
    // node jj of the periodic continuation: node jj mod n, shifted by whole periods
    auto nodepos = [&](int jj) { return node_x(jj % n, h) + (double)(jj / n) * L; };
    // the first node strictly right of `left`
    int j = (int)floor(left * inv_h);
    if (j < 0) j = 0;
    while (j > 0 && nodepos(j) > left) --j;
    while (nodepos(j) <= left) ++j;
    const int kn = k + 1 < N ? k + 1 : 0;
    for (int f = 0; f < F; ++f) {
        const double* A = Ab + (size_t)f * n;
        double lo = 0.0, hi = 0.0;
        double a = left, fa = fk[(size_t)f * N + k];
        for (int jj = j;; ++jj) {
            const int jw = jj % n;
            const double xn = nodepos(jj);
            if (!(xn < right)) break;
            piece(a, xn, fa, A[jw], left, right, lo, hi);
            a = xn;
            fa = A[jw];
        }
        piece(a, right, fa, fk[(size_t)f * N + kn], left, right, lo, hi);
        to_lo[(size_t)f * N + k] = lo;
        to_hi[(size_t)f * N + k] = hi;
    }
}

// out[f][k] = c[f][k] / d[k] (d == nullptr: / s); K = *dK where dK is given
__global__ void k_x1d_div(int K, const int32_t* __restrict__ dK, int F, const double* __restrict__ c, const double* __restrict__ d,
                          double s, double* __restrict__ out) {
    const int k = blockIdx.x * kB + threadIdx.x;
    if (dK) K = *dK;
    if (k >= K) return;
    const double den = d ? d[k] : s;
    for (int f = 0; f < F; ++f) out[(size_t)f * K + k] = c[(size_t)f * K + k] / den;
}

// sorted-order values to caller order (k_x1d_out: the particles left out, whose volume is
// NaN, get NaN)
__global__ void k_x1d_fill_nan(size_t n, double* __restrict__ out) {
    const size_t i = (size_t)blockIdx.x * kB + threadIdx.x;
    if (i < n) out[i] = __builtin_nan("");
}
__global__ void k_x1d_scatter(int N, int F, int np, const int32_t* __restrict__ idx,
                              const double* __restrict__ xs, double* __restrict__ out) {
    const int k = blockIdx.x * kB + threadIdx.x;
    if (k >= N) return;
    const int p = idx[k];
    for (int f = 0; f < F; ++f) out[(size_t)f * np + p] = xs[(size_t)f * N + k];
}

__global__ void k_x1d_out(Mesh m, const double* __restrict__ vol_c, const int32_t* __restrict__ dN, int F,
                          const int32_t* __restrict__ idx, const double* __restrict__ xs,
                          double* __restrict__ out) {
    const int k = blockIdx.x * kB + threadIdx.x, N = *dN;
    if (k >= m.np) return;
    if (!(vol_c[k] == vol_c[k]))
        for (int f = 0; f < F; ++f) out[(size_t)f * m.np + k] = __builtin_nan("");
    if (k >= N) return;
    const int p = idx[k];
    for (int f = 0; f < F; ++f) out[(size_t)f * m.np + p] = xs[(size_t)f * N + k];
}

// Binning, order, setup and evaluation by one workgroup, for at most kSmallMax particles
// and cells: what k_bin_small, k_x1d_sort, k_x1d_setup and k_x1d_nodes or k_x1d_parts do
// (the particles' order by cell number is skipped: only the order along the line is
// used), with the keys in LDS.  The report is written whole.
// Bound: the launch and the dependent passes.  64 cells, 256 particles: 7.1 us instead of
// four launches of 12 us and their gaps (there and back 45 -> 33 us).  2048 particles,
// there and back: 67 us, by the general path 75; 4096: 86 and 83, so the line lies at 3072.
constexpr int kSmallBlock = 1024;
constexpr int kSmallItems = 3;
constexpr int kSmallMax = kSmallBlock * kSmallItems;

__global__ __launch_bounds__(kSmallBlock) void k_x1d_small(Mesh m, X1dSmall a, p2m_report* __restrict__ rep) {
    __shared__ double s_key[kSmallMax];
    __shared__ int32_t s_idx[kSmallMax], s_cs[kSmallMax + 1];
    __shared__ int s_wave[kSmallBlock / 64], s_big[kSmallBlock];
    __shared__ int s_nbig, s_inv;
    __shared__ uint32_t s_flags;
    const int tid = threadIdx.x, nc = m.nx, np = m.np;
    const double L = m.cell_measure * m.nx;
    double px[kSmallItems];
#pragma unroll
    for (int u = 0; u < kSmallItems; ++u) {
        const int i = tid + u * kSmallBlock;
        px[u] = i < np ? a.x[i] : 0.0;
    }
    for (int c = tid; c < nc; c += kSmallBlock) s_cs[c] = 0;
    if (tid == 0) {
        s_inv = 0;
        s_flags = 0u;
    }
    __syncthreads();
    int cell[kSmallItems], rank[kSmallItems];
#pragma unroll
    for (int u = 0; u < kSmallItems; ++u) {
        const int i = tid + u * kSmallBlock;
        cell[u] = -1;
        rank[u] = 0;
        if (i >= np) continue;
        int c;
        double xi;
        bool fin;
        if (locate_axis(px[u], m.nx, m.inv_hx, c, xi, fin)) {
            cell[u] = c;
            rank[u] = atomicAdd(&s_cs[c], 1);
        } else {
            atomicOr(&s_flags, fin ? (uint32_t)P2M_FLAG_RANGE : (uint32_t)P2M_FLAG_NONFINITE);
            atomicAdd(&s_inv, 1);
        }
    }
    __syncthreads();
    // exclusive scan of the counts in place, each thread a run of adjacent cells
    const int per = (nc + kSmallBlock - 1) / kSmallBlock;
    const int c0 = min(tid * per, nc), c1 = min(c0 + per, nc);
    int sum = 0;
    for (int c = c0; c < c1; ++c) sum += s_cs[c];
    int inc = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int u = __shfl_up(inc, d, 64);
        if ((tid & 63) >= d) inc += u;
    }
    if ((tid & 63) == 63) s_wave[tid >> 6] = inc;
    __syncthreads();
    int ex = inc - sum;
    for (int w = 0; w < (tid >> 6); ++w) ex += s_wave[w];
    for (int c = c0; c < c1; ++c) {
        const int n = s_cs[c];
        s_cs[c] = ex;
        ex += n;
    }
    if (tid == kSmallBlock - 1) s_cs[nc] = ex;
    __syncthreads();
    const int N = s_cs[nc];
#pragma unroll
    for (int u = 0; u < kSmallItems; ++u) {
        if (cell[u] < 0) continue;
        const int k = s_cs[cell[u]] + rank[u];
        s_key[k] = wrap_pos(px[u], L);
        s_idx[k] = tid + u * kSmallBlock;
    }
    if (tid == 0) *a.dN = N;
    __syncthreads();
    for (int b = 0; b < nc; b += kSmallBlock) {
        if (tid == 0) s_nbig = 0;
        __syncthreads();
        const int c = b + tid;
        if (c < nc) {
            const int s = s_cs[c], n = s_cs[c + 1] - s;
            if (n > kSortSmall) s_big[atomicAdd(&s_nbig, 1)] = c;
            else if (n > 1) insertion_sort(s_key, s_idx, s, n);
        }
        __syncthreads();
        const int nb = s_nbig;
        for (int q = 0; q < nb; ++q) {
            const int cc = s_big[q], s = s_cs[cc];
            block_sort_pairs<kSmallBlock>(s_key + s, s_idx + s, s_cs[cc + 1] - s);
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < kSmallItems; ++u) {
        const int k = tid + u * kSmallBlock;
        if (a.nan_volumes && k < np && cell[u] < 0) a.vol_c[k] = __builtin_nan("");
        if (k >= N) continue;
        a.key[k] = s_key[k];
        a.idx[k] = s_idx[k];
        setup_at(k, N, L, s_key, s_idx, a.values, a.values ? a.F : 0, np, a.gap, a.vol_s, a.vol_c, a.As);
    }
    report_clear(rep, s_flags, s_inv);
    __syncthreads();
    if (a.eval == X1dSmall::kNodes) {
        for (int j = tid; j < nc; j += kSmallBlock)
            nodes_at(j, nc, m.cell_measure, L, N, s_key, a.As, a.F, a.appb, a.f, a.c, a.coef, a.w);
    } else if (a.eval == X1dSmall::kParts) {
        for (int k = tid; k < N; k += kSmallBlock)
            parts_at(k, N, nc, m.cell_measure, m.inv_hx, L, s_key, a.gap, a.nodal, a.F, a.appb, a.f, a.c,
                     a.coef);
    }
}

}  // namespace

#define X1D_TRY(e)                                 \
    do {                                           \
        hipError_t e_ = (e);                       \
        if (e_ != hipSuccess) return e_;           \
    } while (0)

bool x1d_small_fits(const Mesh& m) { return m.np > 0 && m.np <= kSmallMax && m.nx <= kSmallMax; }

hipError_t x1d_small(const Mesh& m, const X1dSmall& a, p2m_report* rep, hipStream_t stream) {
    hipLaunchKernelGGL(k_x1d_small, dim3(1), dim3(kSmallBlock), 0, stream, m, a, rep);
    return hipGetLastError();
}

hipError_t x1d_sort(const Mesh& m, const double* x, const int32_t* perm, const int32_t* cs,
                    double* key, int32_t* idx, hipStream_t stream) {
    const double L = m.cell_measure * m.nx;
    hipLaunchKernelGGL(k_x1d_sort, dim3(grid_of(m.nx)), dim3(kB), 0, stream, m.nx, x, L, perm, cs, key,
                       idx);
    return hipGetLastError();
}

hipError_t x1d_setup(const Mesh& m, const double* x, const int32_t* dN, const double* key, const int32_t* idx,
                     const double* values, int F, double* gap, double* vol_s, double* vol_c,
                     double* As, hipStream_t stream) {
    if (m.np == 0) return hipSuccess;
    const double L = m.cell_measure * m.nx;
    hipLaunchKernelGGL(k_x1d_setup, dim3(grid_of(m.np)), dim3(kB), 0, stream, m, x, dN, L, key, idx,
                       values, F, m.np, gap, vol_s, vol_c, As);
    return hipGetLastError();
}

hipError_t x1d_p2m_overlap(const Mesh& m, const int32_t* dN, const double* key, const double* As,
                           int F, int quad, double* fn, double* t_lo, double* t_hi, double* c,
                           double* coef, double* w, bool evaluated, hipStream_t stream) {
    const int n = m.nx;
    const double h = m.cell_measure, L = h * n;
    const int appb = quad == P2M_QUAD_APPB && c ? 1 : 0;
    if (!evaluated) {
        hipLaunchKernelGGL(k_x1d_nodes, dim3(grid_of(n)), dim3(kB), 0, stream, n, h, L, dN, key, As, F,
                           appb, fn, c, coef, w);
        X1D_TRY(hipGetLastError());
    }
    if (appb || !c) return hipSuccess;
    hipLaunchKernelGGL(k_x1d_c_exact, dim3(grid_of(n)), dim3(kB), 0, stream, n, h, L, dN, key, As, F,
                       fn, t_lo, t_hi);
    X1D_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_x1d_c_sum, dim3(grid_of(n)), dim3(kB), 0, stream, n, (const int32_t*)nullptr,
                       F, t_lo, t_hi, c);
    return hipGetLastError();
}

hipError_t x1d_m2p_overlap(const Mesh& m, const int32_t* dN, const double* key, const double* gap,
                           const double* nodal, int F, int quad, double* fk, double* t_lo,
                           double* t_hi, double* c, double* coef, bool evaluated, hipStream_t stream) {
    if (m.np == 0) return hipSuccess;
    const int n = m.nx;
    const double h = m.cell_measure, L = h * n;
    const int appb = quad == P2M_QUAD_APPB ? 1 : 0;
    if (!evaluated) {
        hipLaunchKernelGGL(k_x1d_parts, dim3(grid_of(m.np)), dim3(kB), 0, stream, dN, n, h, m.inv_hx, L,
                           key, gap, nodal, F, appb, fk, c, coef);
        X1D_TRY(hipGetLastError());
    }
    if (appb) return hipSuccess;
    hipLaunchKernelGGL(k_x1d_cp_exact, dim3(grid_of(m.np)), dim3(kB), 0, stream, dN, n, h, m.inv_hx, L,
                       key, gap, nodal, fk, F, t_lo, t_hi);
    X1D_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_x1d_c_sum, dim3(grid_of(m.np)), dim3(kB), 0, stream, m.np, dN, F, t_lo, t_hi,
                       c);
    return hipGetLastError();
}

hipError_t x1d_div(int K, const int32_t* dK, int F, const double* c, const double* d, double s,
                   double* out, hipStream_t stream) {
    if (K == 0) return hipSuccess;
    hipLaunchKernelGGL(k_x1d_div, dim3(grid_of(K)), dim3(kB), 0, stream, K, dK, F, c, d, s, out);
    return hipGetLastError();
}

hipError_t x1d_fill_nan(size_t n, double* out, hipStream_t stream) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_x1d_fill_nan, dim3(grid_of(n)), dim3(kB), 0, stream, n, out);
    return hipGetLastError();
}

hipError_t x1d_out(const Mesh& m, const double* vol_c, const int32_t* dN, int F, const int32_t* idx,
                   const double* xs, double* out, hipStream_t stream) {
    if (m.np == 0) return hipSuccess;
    hipLaunchKernelGGL(k_x1d_out, dim3(grid_of(m.np)), dim3(kB), 0, stream, m, vol_c, dN, F, idx, xs, out);
    return hipGetLastError();
}

hipError_t x1d_scatter(int N, int F, int np, const int32_t* idx, const double* xs, double* out,
                       hipStream_t stream) {
    if (N == 0) return hipSuccess;
    hipLaunchKernelGGL(k_x1d_scatter, dim3(grid_of(N)), dim3(kB), 0, stream, N, F, np, idx, xs, out);
    return hipGetLastError();
}

}  // namespace p2m
