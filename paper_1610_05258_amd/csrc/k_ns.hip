// The mesh half of the particle fluid solver of Sec. 3.3 (Taylor-Green vortex
// sheet) on the periodic "/"-split P1 mesh with square cells of side h:
//
//   coef    : stencil arrays of the two symmetric systems the mass-matrix solver
//             takes (D, E, N, NE per node, and the diagonal as w):
//               viscous  I + s K, s = dt nu / h^2, K the P1 stiffness matrix, which
//                        on right isosceles triangles is the five-point Laplacian;
//               pressure K with node 0 held at 0 (its row and column replaced by
//                        the identity, which changes p by a constant only);
//   div     : right-hand side of the pressure system, -(1/dt) (D U*)_k with
//             (D U)_k = int psi_k div U_h;
//   correct : the projection U^{n+1} = U* - dt M_L^{-1} G p, (G p)_k = int psi_k
//             grad p_h, M_L = h^2 (row sums of the P1 mesh mass matrix);
//   advect  : mid-point advection of the particles, r* = r + (dt/2) a with a the
//             interpolated U^{n+1}, r <- r + dt U^{n+1}(r*), wrapped into [0, L).
//
// Every node sees the six triangles around it: of cell (i, j) both triangles
// (the node is their corner n00), of cell (i-1, j) the lower one (corner n10), of
// cell (i-1, j-1) both (corner n11) and of cell (i, j-1) the upper one (corner
// n01).  On a triangle the P1 derivatives are node differences over h; the
// integral of a hat over a triangle is h^2/6.  The node sums are formed in FP64
// and rounded once.
#include "p2m_internal.hpp"

namespace p2m {

namespace {

struct Nbr {
    int i, j, im, jm, ip, jp;
};

__device__ __forceinline__ Nbr nbr(int k, int nx, int ny) {
    Nbr q;
    q.i = k % nx;
    q.j = k / nx;
    q.im = q.i == 0 ? nx - 1 : q.i - 1;
    q.jm = q.j == 0 ? ny - 1 : q.j - 1;
    q.ip = q.i + 1 == nx ? 0 : q.i + 1;
    q.jp = q.j + 1 == ny ? 0 : q.j + 1;
    return q;
}

__global__ void k_ns_coef(int nx, int ny, float s, float* __restrict__ cv, float* __restrict__ wv,
                          float* __restrict__ cp, float* __restrict__ wp) {
    const int nn = nx * ny;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nn) return;
    const float dv = (float)(1.0 + 4.0 * (double)s);
    cv[k] = dv;
    cv[nn + k] = -s;
    cv[2 * nn + k] = -s;
    cv[3 * nn + k] = 0.f;
    wv[k] = dv;
    // node 0's couplings: its own E and N, the E of (nx-1, 0) and the N of (0, ny-1)
    const int i = k % nx, j = k / nx;
    const bool pin = k == 0;
    const bool e0 = pin || (i == nx - 1 && j == 0);
    const bool n0 = pin || (i == 0 && j == ny - 1);
    const float dp = pin ? 1.f : 4.f;
    cp[k] = dp;
    cp[nn + k] = e0 ? 0.f : -1.f;
    cp[2 * nn + k] = n0 ? 0.f : -1.f;
    cp[3 * nn + k] = 0.f;
    wp[k] = dp;
}

// sum of the six triangles' divergence differences of the velocity U [2][nn] around node
// (i, j) (lower triangle of cell c: u10 - u00 + v11 - v10; upper: u11 - u01 + v01 - v00)
__device__ __forceinline__ double div_sum(const float* __restrict__ U, int k, int nx, int ny) {
    const Nbr q = nbr(k, nx, ny);
    const float* u = U;
    const float* v = U + nx * ny;
    auto at = [&](const float* a, int ii, int jj) { return (double)a[ii + nx * jj]; };
    // cell (ci, cj) with upper-right corner (ci1, cj1)
    auto dl = [&](int ci, int cj, int ci1, int cj1) {
        return (at(u, ci1, cj) - at(u, ci, cj)) + (at(v, ci1, cj1) - at(v, ci1, cj));
    };
    auto du = [&](int ci, int cj, int ci1, int cj1) {
        return (at(u, ci1, cj1) - at(u, ci, cj1)) + (at(v, ci, cj1) - at(v, ci, cj));
    };
    return dl(q.i, q.j, q.ip, q.jp) + du(q.i, q.j, q.ip, q.jp) + dl(q.im, q.j, q.i, q.jp) +
           dl(q.im, q.jm, q.i, q.j) + du(q.im, q.jm, q.i, q.j) + du(q.i, q.jm, q.ip, q.j);
}

// rhs_k = scale * div_sum, scale = -(h/6)/dt, 0 at the held node 0
__global__ void k_ns_div(int nx, int ny, double scale, const float* __restrict__ U,
                         float* __restrict__ rhs) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nx * ny) return;
    rhs[k] = k == 0 ? 0.f : (float)(scale * div_sum(U, k, nx, ny));
}

// U^{n+1}_k = U*_k - factor * (sum of the six triangles' gradient differences),
// lower triangle of cell c: (p10 - p00, p11 - p10); upper: (p11 - p01, p01 - p00);
// factor = dt / (6 h)
__global__ void k_ns_correct(int nx, int ny, double factor, const float* __restrict__ Us,
                             const float* __restrict__ p, float* __restrict__ Un) {
    const int nn = nx * ny;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nn) return;
    const Nbr q = nbr(k, nx, ny);
    auto at = [&](int ii, int jj) { return (double)p[ii + nx * jj]; };
    double gx = 0.0, gy = 0.0;
    auto gl = [&](int ci, int cj, int ci1, int cj1) {
        gx += at(ci1, cj) - at(ci, cj);
        gy += at(ci1, cj1) - at(ci1, cj);
    };
    auto gu = [&](int ci, int cj, int ci1, int cj1) {
        gx += at(ci1, cj1) - at(ci, cj1);
        gy += at(ci, cj1) - at(ci, cj);
    };
    gl(q.i, q.j, q.ip, q.jp);
    gu(q.i, q.j, q.ip, q.jp);
    gl(q.im, q.j, q.i, q.jp);
    gl(q.im, q.jm, q.i, q.j);
    gu(q.im, q.jm, q.i, q.j);
    gu(q.i, q.jm, q.ip, q.j);
    Un[k] = (float)((double)Us[k] - factor * gx);
    Un[nn + k] = (float)((double)Us[nn + k] - factor * gy);
}

__device__ __forceinline__ double wrap(double x, double len) {
    return __dsub_rn(x, len * floor(x / len));
}

// U at an FP64 position (its triangle's three nodes, FP64 weights); false when the
// position cannot be located
__device__ __forceinline__ bool interp2(const Mesh& m, const float* __restrict__ U, double x,
                                        double y, double& ux, double& uy, bool& finite) {
    int cx = 0, cy = 0;
    double xi = 0.0, eta = 0.0;
    bool fx = true, fy = true;
    bool ok = locate_axis(x, m.nx, m.inv_hx, cx, xi, fx);
    ok = locate_axis(y, m.ny, m.inv_hy, cy, eta, fy) && ok;
    finite = fx && fy;
    if (!ok) return false;
    const int i1 = cx + 1 == m.nx ? 0 : cx + 1;
    const int j1 = cy + 1 == m.ny ? 0 : cy + 1;
    double c00, c10, c11, c01;
    corner_weights<double>(xi, eta, c00, c10, c11, c01);
    const int k00 = cx + m.nx * cy, k10 = i1 + m.nx * cy, k11 = i1 + m.nx * j1, k01 = cx + m.nx * j1;
    const float* v = U + m.nn;
    ux = c00 * U[k00] + c10 * U[k10] + c11 * U[k11] + c01 * U[k01];
    uy = c00 * v[k00] + c10 * v[k10] + c11 * v[k11] + c01 * v[k01];
    return true;
}

// x, y and xo, yo may be the same arrays (each thread reads its particle before
// writing it)
__global__ void k_ns_advect(Mesh m, double lx, double ly, double dt, const float* x,
                            const float* y, const float* __restrict__ a,
                            const float* __restrict__ U, float* xo, float* yo,
                            p2m_report* __restrict__ rep) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= m.np) return;
    const double x0 = x[i], y0 = y[i];
    const double xm = wrap(x0 + 0.5 * dt * (double)a[i], lx);
    const double ym = wrap(y0 + 0.5 * dt * (double)a[m.np + i], ly);
    double ux = 0.0, uy = 0.0;
    bool finite = true;
    if (!interp2(m, U, xm, ym, ux, uy, finite)) {
        if (rep) atomicOr(&rep->flags, finite ? (uint32_t)P2M_FLAG_RANGE : (uint32_t)P2M_FLAG_NONFINITE);
        xo[i] = NAN;
        yo[i] = NAN;
        return;
    }
    xo[i] = (float)wrap(x0 + dt * ux, lx);
    yo[i] = (float)wrap(y0 + dt * uy, ly);
}

// ---------------------------------------------------------------------------
// Direct solves of the mesh systems by the 2D discrete Fourier transform:
// I + s K and K are circulant on the periodic mesh, diagonal in the 2D discrete
// Fourier basis with eigenvalues 1 + s lam and lam, lam(kx, ky) = 4 - 2 cos(2 pi
// kx / nx) - 2 cos(2 pi ky / ny) (the five-point symbol); K's zero mode is the
// constant, left at 0 (zero-mean pressure).  FP64 in three launches:
//   k_fft_fwd   rows of the real right-hand side -> half spectrum (kx <= nx / 2; the
//               rest is its conjugate)
//   k_fft_cols  columns of the half spectrum: forward, divided by the symbol, inverse,
//               in place; a workgroup takes adjacent columns (64-byte pieces of a row)
//   k_fft_inv   rows back to real values
// Transforms run in LDS, several to a workgroup: Stockham radix 4 (one radix-2 pass if
// the length is an odd power), natural order in and out, twiddles from a table made once
// per workgroup; other lengths by Bluestein's algorithm over a power-of-two convolution.
// Bound: at the sizes of a time step (256 x 256) the chain of LDS passes and the launches,
// not memory (1 MB a field and pass).  Rows, columns (forward, division and inverse in one)
// and rows again over the half spectrum take three launches, 18.5 us for two fields at
// 256 x 256; separate transposes and division over the full spectrum, radix 2 and a sine and
// cosine per butterfly took seven and 34 us.
// ---------------------------------------------------------------------------
constexpr int kFftMaxN = 2048;   // a transform's buffers, twiddles and chirp: up to 96 KB of LDS
constexpr int kFftThreads = 256;

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// a * exp(-+ i 2 pi j / n) from the table tw[j] = exp(-i 2 pi j / n), j < n / 2
__device__ __forceinline__ double2 twist(double2 a, const double2* tw, int j, int half, bool inv) {
    double2 w = tw[j & (half - 1)];
    if (j & half) w = make_double2(-w.x, -w.y);
    if (inv) w.y = -w.y;
    return cmul(a, w);
}

__device__ __forceinline__ void fft_table(double2* tw, int n) {
    for (int t = threadIdx.x; t < n / 2; t += blockDim.x) {
        double sn, cs;
        sincospi(-2.0 * (double)t / (double)n, &sn, &cs);
        tw[t] = make_double2(cs, sn);
    }
}

// C transforms of length n = 2^logn, transform c at x + c n (y: scratch of the same
// size); the result ends in x (the two pointers are swapped per pass).  The workgroup's
// threads share the work; the caller synchronises before.
__device__ __forceinline__ void fft_lds(double2*& x, double2*& y, const double2* tw, int C, int n, int logn,
                                        bool inv) {
    const int half = n >> 1, quart = n >> 2;
    int ls = 0;
    if (logn & 1) {
        for (int t = threadIdx.x; t < C * half; t += blockDim.x) {
            const int c = t >> (logn - 1), j = t & (half - 1);
            const double2 a = x[c * n + j], b = x[c * n + j + half];
            y[c * n + 2 * j] = cadd(a, b);
            y[c * n + 2 * j + 1] = csub(a, b);
        }
        __syncthreads();
        double2* t = x;
        x = y;
        y = t;
        ls = 1;
    }
    for (; ls < logn; ls += 2) {
        const int ns = 1 << ls, ts = logn - 2 - ls;   // twiddle k r at index (k r) << ts
        for (int t = threadIdx.x; t < C * quart; t += blockDim.x) {
            const int c = t >> (logn - 2), j = t & (quart - 1), k = j & (ns - 1);
            const double2* xc = x + c * n + j;
            const double2 v0 = xc[0];
            const double2 v1 = twist(xc[quart], tw, k << ts, half, inv);
            const double2 v2 = twist(xc[2 * quart], tw, (2 * k) << ts, half, inv);
            const double2 v3 = twist(xc[3 * quart], tw, (3 * k) << ts, half, inv);
            const double2 s02 = cadd(v0, v2), d02 = csub(v0, v2), s13 = cadd(v1, v3);
            double2 d13 = csub(v1, v3);
            d13 = inv ? make_double2(-d13.y, d13.x) : make_double2(d13.y, -d13.x);   // +-i (v1 - v3)
            double2* yd = y + c * n + ((j >> ls) << (ls + 2)) + k;
            yd[0] = cadd(s02, s13);
            yd[ns] = cadd(d02, d13);
            yd[2 * ns] = csub(s02, s13);
            yd[3 * ns] = csub(d02, d13);
        }
        __syncthreads();
        double2* t = x;
        x = y;
        y = t;
    }
}

// A side of the mesh: its length n, the transform length m = 2^logm (n itself, or the
// convolution's >= 2n - 1) and, for Bluestein, the chirp's transform bhat: with
// c_j = exp(-i pi j^2 / n), the DFT is X_k = c_k sum_j (x_j c_j) conj(c_{k-j}), a
// circular convolution done by two power-of-two transforms.
struct FftSide {
    int n, m, logm;
    const double2* bhat;   // null: n is a power of two
};

__device__ __forceinline__ double2 chirp(int j, int n) {
    double sn, cs;
    sincospi(-(double)(((long long)j * j) % (2LL * n)) / (double)n, &sn, &cs);
    return make_double2(cs, sn);
}

// the DFT (inv: unnormalised inverse) of C sequences of length s.n at x + c s.m, in
// place as fft_lds; ch[0 .. n): the chirp.  Synchronises first.
__device__ void dft_lds(double2*& x, double2*& y, const double2* tw, const double2* ch, int C,
                        const FftSide& s, bool inv) {
    __syncthreads();
    if (!s.bhat) {
        fft_lds(x, y, tw, C, s.m, s.logm, inv);
        return;
    }
    for (int t = threadIdx.x; t < C * s.m; t += blockDim.x) {
        const int j = t & (s.m - 1);
        double2 v = make_double2(0.0, 0.0);
        if (j < s.n) {
            v = x[t];
            if (inv) v.y = -v.y;
            v = cmul(v, ch[j]);
        }
        x[t] = v;
    }
    __syncthreads();
    fft_lds(x, y, tw, C, s.m, s.logm, false);
    for (int t = threadIdx.x; t < C * s.m; t += blockDim.x) x[t] = cmul(x[t], s.bhat[t & (s.m - 1)]);
    __syncthreads();
    fft_lds(x, y, tw, C, s.m, s.logm, true);
    const double im = 1.0 / (double)s.m;
    for (int t = threadIdx.x; t < C * s.m; t += blockDim.x) {
        const int j = t & (s.m - 1);
        if (j >= s.n) continue;
        const double2 v = cmul(x[t], ch[j]);
        x[t] = make_double2(v.x * im, (inv ? -v.y : v.y) * im);
    }
    __syncthreads();
}

// LDS of a kernel on C transforms: two buffers, the twiddles, the chirp
struct FftLds {
    double2 *x, *y, *tw, *ch;
};
__device__ __forceinline__ FftLds fft_carve(double2* p, int C, const FftSide& s) {
    FftLds l;
    l.x = p;
    l.y = p + C * s.m;
    l.tw = p + 2 * C * s.m;
    l.ch = l.tw + s.m / 2;
    fft_table(l.tw, s.m);
    if (s.bhat)
        for (int t = threadIdx.x; t < s.n; t += blockDim.x) l.ch[t] = chirp(t, s.n);
    return l;
}
inline size_t fft_lds_bytes(int C, const FftSide& s) {
    return ((size_t)2 * C * s.m + s.m / 2 + (s.bhat ? s.n : 0)) * sizeof(double2);
}

// bhat = FFT_M(b), b_m = conj(c_m) for 0 <= m < n, b_{M-m} = conj(c_m) for
// 0 < m < n, 0 elsewhere; one workgroup a side
__global__ void k_fft_chirp(FftSide s0, FftSide s1, double2* out0, double2* out1) {
    extern __shared__ double2 fsh[];
    const FftSide s = blockIdx.x ? s1 : s0;
    double2* out = blockIdx.x ? out1 : out0;
    double2 *x = fsh, *y = fsh + s.m, *tw = fsh + 2 * s.m;
    fft_table(tw, s.m);
    for (int t = threadIdx.x; t < s.m; t += blockDim.x) {
        const int j = t < s.n ? t : (t > s.m - s.n ? s.m - t : -1);
        double2 v = make_double2(0.0, 0.0);
        if (j >= 0) {
            const double2 c = chirp(j, s.n);
            v = make_double2(c.x, -c.y);
        }
        x[t] = v;
    }
    __syncthreads();
    fft_lds(x, y, tw, 1, s.m, s.logm, false);
    for (int t = threadIdx.x; t < s.m; t += blockDim.x) out[t] = x[t];
}

// what the row transforms read: an array of reals, or the pressure's right-hand side
// formed from the velocity where it is read
template <typename R>
struct FftArray {
    const R* p;
    int nx;
    __device__ double operator()(size_t row, int i) const { return (double)p[row * nx + i]; }
};

struct FftDivergence {
    const float* U;   // [2][nn]
    int nx, ny;
    double scale;
    __device__ double operator()(size_t row, int i) const {
        return scale * div_sum(U, (int)row * nx + i, nx, ny);
    }
};

// C rows a workgroup of the nrows = nb ny real rows -> [row][nh], nh = nx / 2 + 1
template <typename Src>
__global__ __launch_bounds__(kFftThreads) void k_fft_fwd(Src src, double2* __restrict__ out, FftSide s,
                                                         int nrows, int C) {
    extern __shared__ double2 fsh[];
    FftLds l = fft_carve(fsh, C, s);
    const size_t r0 = (size_t)blockIdx.x * C;
    const int nh = s.n / 2 + 1;
    for (int t = threadIdx.x; t < C * s.m; t += blockDim.x) {
        const int c = t >> s.logm, i = t & (s.m - 1);
        l.x[t] = make_double2(i < s.n && r0 + c < (size_t)nrows ? src(r0 + c, i) : 0.0, 0.0);
    }
    dft_lds(l.x, l.y, l.tw, l.ch, C, s, false);
    for (int t = threadIdx.x; t < C * nh; t += blockDim.x) {
        const int c = t / nh, i = t - c * nh;
        if (r0 + c < (size_t)nrows) out[(r0 + c) * nh + i] = l.x[c * s.m + i];
    }
}

// the system's eigenvalue at (kx, ky): 1 + s lam (viscous), lam (pressure), or the
// consistent P1 mass matrix of the "/" split, s (1/2 + (cos tx + cos ty +
// cos(tx + ty)) / 6) with s = hx hy (mass)
__device__ __forceinline__ double fft_symbol(int kx, int ky, int nx, int ny, double s, int mode) {
    if (mode == kFftMass)
        return s * (0.5 + (cospi(2.0 * kx / nx) + cospi(2.0 * ky / ny) +
                           cospi(2.0 * kx / nx + 2.0 * ky / ny)) / 6.0);
    const double lam = 4.0 - 2.0 * cospi(2.0 * kx / nx) - 2.0 * cospi(2.0 * ky / ny);
    return mode == kFftPressure ? lam : 1.0 + s * lam;
}

// C columns a workgroup of [nb][ny][nh]; blockIdx.y: field
__global__ __launch_bounds__(kFftThreads) void k_fft_cols(double2* __restrict__ a, FftSide s, int nx, int nh,
                                                          int C, double sc, int mode) {
    extern __shared__ double2 fsh[];
    FftLds l = fft_carve(fsh, C, s);
    double2* p = a + (size_t)blockIdx.y * s.n * nh;
    const int c0 = blockIdx.x * C;
    for (int t = threadIdx.x; t < C * s.m; t += blockDim.x) {
        const int j = t / C, c = t - j * C;   // adjacent threads: adjacent columns
        l.x[c * s.m + j] = j < s.n && c0 + c < nh ? p[(size_t)j * nh + c0 + c] : make_double2(0.0, 0.0);
    }
    dft_lds(l.x, l.y, l.tw, l.ch, C, s, false);
    for (int t = threadIdx.x; t < C * s.n; t += blockDim.x) {
        const int c = t / s.n, ky = t - c * s.n, kx = c0 + c;
        const double2 v = l.x[c * s.m + ky];
        const double e = fft_symbol(kx, ky, nx, s.n, sc, mode);
        l.x[c * s.m + ky] = mode == kFftPressure && kx == 0 && ky == 0 ? make_double2(0.0, 0.0)
                                                                       : make_double2(v.x / e, v.y / e);
    }
    dft_lds(l.x, l.y, l.tw, l.ch, C, s, true);
    for (int t = threadIdx.x; t < C * s.n; t += blockDim.x) {
        const int j = t / C, c = t - j * C;
        if (c0 + c < nh) p[(size_t)j * nh + c0 + c] = l.x[c * s.m + j];
    }
}

// C rows a workgroup back to reals, times scale
template <typename R>
__global__ __launch_bounds__(kFftThreads) void k_fft_inv(const double2* __restrict__ a, R* __restrict__ out,
                                                         FftSide s, int nrows, int C, double scale) {
    extern __shared__ double2 fsh[];
    FftLds l = fft_carve(fsh, C, s);
    const size_t r0 = (size_t)blockIdx.x * C;
    const int nh = s.n / 2 + 1;
    for (int t = threadIdx.x; t < C * nh; t += blockDim.x) {
        const int c = t / nh, i = t - c * nh;
        const double2 v = r0 + c < (size_t)nrows ? a[(r0 + c) * nh + i] : make_double2(0.0, 0.0);
        l.x[c * s.m + i] = v;
        if (i > 0 && i < s.n - i) l.x[c * s.m + s.n - i] = make_double2(v.x, -v.y);
    }
    dft_lds(l.x, l.y, l.tw, l.ch, C, s, true);
    for (int t = threadIdx.x; t < C * s.n; t += blockDim.x) {
        const int c = t / s.n, i = t - c * s.n;
        if (r0 + c < (size_t)nrows) out[(r0 + c) * s.n + i] = (R)(l.x[c * s.m + i].x * scale);
    }
}

inline int grid_of(int n, int b) { return (n + b - 1) / b; }

inline int ilog2(int n) {
    int l = 0;
    while ((1 << l) < n) ++l;
    return l;
}

}  // namespace


// a side the row transforms take: a power of two up to kFftMaxN, or any length up
// to kFftMaxN / 2 (Bluestein, convolution length at most kFftMaxN)
static bool fft_side(int n) {
    return n >= 2 && (((n & (n - 1)) == 0 && n <= kFftMaxN) || 2 * n - 1 <= kFftMaxN);
}

bool fft_supported(const Mesh& m) { return m.dim == 2 && fft_side(m.nx) && fft_side(m.ny); }

// two complex planes of nb fields, then the chirp transforms of the two sides
size_t fft_workspace_bytes(const Mesh& m, int nb) {
    return ((size_t)2 * nb * m.nn + 2 * kFftMaxN) * sizeof(double2);
}

namespace {

template <typename Real, typename Src>
hipError_t fft_solve(const Mesh& m, int nb, double s, int mode, const Src& src, Real* x, void* ws,
                     hipStream_t stream) {
    const int nx = m.nx, ny = m.ny, nh = nx / 2 + 1;
    double2* fa = (double2*)ws;
    double2* tab = fa + (size_t)2 * nb * m.nn;
    auto side = [](int n, double2* bhat) {
        FftSide f;
        f.n = n;
        const bool pow2 = (n & (n - 1)) == 0;
        f.logm = ilog2(pow2 ? n : 2 * n - 1);
        f.m = 1 << f.logm;
        f.bhat = pow2 ? nullptr : bhat;
        return f;
    };
    const FftSide sx = side(nx, tab), sy = side(ny, nx == ny ? tab : tab + kFftMaxN);
    hipError_t e;
    if (sx.bhat || sy.bhat) {
        const FftSide& a = sx.bhat ? sx : sy;
        const int sides = sx.bhat && sy.bhat && nx != ny ? 2 : 1;
        const int mm = sides == 2 && sy.m > a.m ? sy.m : a.m;
        hipLaunchKernelGGL(k_fft_chirp, dim3(sides), dim3(kFftThreads), (size_t)(2 * mm + mm / 2) * sizeof(double2),
                           stream, a, sy, (double2*)a.bhat, (double2*)sy.bhat);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    // transforms a workgroup: as many as leave 256 workgroups (the chain of passes is as
    // long for one as for four), while its threads each have a radix-4 butterfly to do.
    // Always as many as that took 6.0 / 11.5 / 6.1 us for two fields at 256 x 256 instead of
    // 4.8 / 8.7 / 4.9, and 22 instead of 15 us for the 512 x 512 columns
    auto per = [](int transforms, const FftSide& f) {
        const int full = f.m >= 4 * kFftThreads ? 1 : 4 * kFftThreads / f.m;
        const int spread = transforms < 512 ? 1 : transforms / 256;
        return spread < full ? spread : full;
    };
    const int cr = per(nb * ny, sx), cc = per(nb * nh, sy);
    const int nrows = nb * ny;
    hipLaunchKernelGGL((k_fft_fwd<Src>), dim3(grid_of(nrows, cr)), dim3(kFftThreads), fft_lds_bytes(cr, sx),
                       stream, src, fa, sx, nrows, cr);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_fft_cols, dim3(grid_of(nh, cc), nb), dim3(kFftThreads), fft_lds_bytes(cc, sy), stream,
                       fa, sy, nx, nh, cc, s, mode);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL((k_fft_inv<Real>), dim3(grid_of(nrows, cr)), dim3(kFftThreads), fft_lds_bytes(cr, sx),
                       stream, fa, x, sx, nrows, cr, 1.0 / ((double)nx * ny));
    return hipGetLastError();
}

}  // namespace

template <typename Real>
hipError_t launch_fft_solve(const Mesh& m, int nb, double s, int mode, const Real* rhs, Real* x,
                            void* ws, hipStream_t stream) {
    return fft_solve<Real>(m, nb, s, mode, FftArray<Real>{rhs, m.nx}, x, ws, stream);
}
template hipError_t launch_fft_solve<double>(const Mesh&, int, double, int, const double*, double*,
                                             void*, hipStream_t);

hipError_t launch_ns_viscous(const Mesh& m, double s, const float* rhs, float* x, void* ws,
                             hipStream_t stream) {
    return launch_fft_solve<float>(m, 2, s, kFftViscous, rhs, x, ws, stream);
}

hipError_t launch_ns_pressure(const Mesh& m, double scale, const float* U, float* p, void* ws,
                              hipStream_t stream) {
    return fft_solve<float>(m, 1, 0.0, kFftPressure, FftDivergence{U, m.nx, m.ny, scale}, p, ws, stream);
}

hipError_t launch_ns_coef(const Mesh& m, float s, float* cv, float* wv, float* cp, float* wp,
                          hipStream_t stream) {
    hipLaunchKernelGGL(k_ns_coef, dim3(grid_of(m.nn, 256)), dim3(256), 0, stream, m.nx, m.ny, s,
                       cv, wv, cp, wp);
    return hipGetLastError();
}

hipError_t launch_ns_div(const Mesh& m, double scale, const float* U, float* rhs, hipStream_t stream) {
    hipLaunchKernelGGL(k_ns_div, dim3(grid_of(m.nn, 256)), dim3(256), 0, stream, m.nx, m.ny, scale, U,
                       rhs);
    return hipGetLastError();
}

hipError_t launch_ns_correct(const Mesh& m, double factor, const float* Us, const float* p,
                             float* Un, hipStream_t stream) {
    hipLaunchKernelGGL(k_ns_correct, dim3(grid_of(m.nn, 256)), dim3(256), 0, stream, m.nx, m.ny,
                       factor, Us, p, Un);
    return hipGetLastError();
}

hipError_t launch_ns_advect(const Mesh& m, double lx, double ly, double dt, const float* x,
                            const float* y, const float* a, const float* U, float* xo, float* yo,
                            p2m_report* rep, hipStream_t stream) {
    if (m.np == 0) return hipSuccess;
    hipLaunchKernelGGL(k_ns_advect, dim3(grid_of(m.np, 256)), dim3(256), 0, stream, m, lx, ly, dt,
                       x, y, a, U, xo, yo, rep);
    return hipGetLastError();
}

}  // namespace p2m
