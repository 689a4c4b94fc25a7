// Paper-exact 2D assignment (Sec. 3.2; Appendix B): P1 hats on the periodic
// Delaunay triangulation of the particles, all in FP64.
//
//   k_x2d_pos      binned order: wrapped positions, values and the cell of every
//                  located particle (slot k = position in the binned order)
//   k_x2d_star_quad, k_x2d_star  per particle, its Delaunay neighbours counter-clockwise by gift
//                  wrapping over the particles of the surrounding mesh cells, widened
//                  ring by ring until no particle outside the searched rings can
//                  change them (twice the largest circumradius within the searched
//                  radius); the volume int psi_mu is a third of the area of the
//                  triangles (mu, n_j, n_j+1).
//   k_x2d_check    every triangle (mu, a, b) must appear in the lists of a and b too
//   k_x2d_locate   the particle interpolant of eq. (1) at the points of a regular
//                  grid (mesh nodes, or nodes and edge midpoints): the triangle that
//                  holds the point is found by a walk from the nearest particle
//   k_x2d_rhs_mesh int A psi_j over the six mesh triangles around node j with the
//                  Appendix-B rule (A at vertices and midpoints from k_x2d_locate)
//   k_x2d_rhs_part int Abar psi_mu over the triangles around particle mu with the
//                  Appendix-B rule (Abar the mesh interpolant), and the consistent
//                  particle mass matrix in sparse-row form (diagonal, then the
//                  off-diagonal slots)
//   k_x2d_mmesh    the consistent mesh mass stencil (D, E, N, NE)
// The particle mass system is solved by k_pmass.hip, the mesh one by FFT (k_ns.hip) or the
// streaming CG (k_cg.hip).
#include "p2m_internal.hpp"

namespace p2m {

namespace {

constexpr int kB = 128;
constexpr int kCap = P2M_X2D_MAXDEG;   // neighbours per particle
constexpr int kRingMax = 8;            // mesh-cell rings searched around a particle
constexpr int kWalkMax = 1024;         // triangles a point-location walk may visit

constexpr int kCand = 40;              // candidates a quad keeps (about 28 are expected)
constexpr int kQuadRings = 4;          // mesh-cell rings a quad searches at most

// Neighbour lists: 2 kCap words a particle, entries in groups of four, the slots of a
// group and then their shifts, so that the list of an ordinary particle (at most eight
// neighbours) is one 64-byte piece whichever of its readers wants it.
__device__ __forceinline__ int at_slot(int i) { return (i >> 2) * 8 + (i & 3); }
__device__ __forceinline__ int at_shift(int i) { return (i >> 2) * 8 + 4 + (i & 3); }

inline int grid_of(size_t n) { return (int)((n + kB - 1) / kB); }

// a double's two halves through a quad permutation (every lane of the quad active)
template <int CTRL>
__device__ __forceinline__ double dpp_quad(double v) {
    const uint2 u = __builtin_bit_cast(uint2, v);
    uint2 r;
    r.x = (unsigned)__builtin_amdgcn_mov_dpp((int)u.x, CTRL, 0xF, 0xF, false);
    r.y = (unsigned)__builtin_amdgcn_mov_dpp((int)u.y, CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, r);
}

struct Geo {
    int nx, ny, N;
    int r0;   // first ring count the triangulation tries
    double lx, ly, hx, hy, inv_hx, inv_hy, inv_lx, inv_ly;
};

__device__ __forceinline__ int floor_div(int a, int n) {
    return a >= 0 ? a / n : -((-a + n - 1) / n);
}
__device__ __forceinline__ int pack_shift(int sx, int sy) { return (sx + 128) | ((sy + 128) << 8); }
__device__ __forceinline__ int shift_x(int s) { return (s & 255) - 128; }
__device__ __forceinline__ int shift_y(int s) { return ((s >> 8) & 255) - 128; }

__device__ __forceinline__ void flag(p2m_report* rep, uint32_t f) {
    if (rep) atomicOr(&rep->flags, f);
}

// ---------------------------------------------------------------------------
__global__ void k_x2d_pos(Geo g, const int32_t* __restrict__ perm, const double* __restrict__ x,
                          const double* __restrict__ y, const double* __restrict__ values, int F,
                          int np, double* __restrict__ xs, double* __restrict__ ys,
                          int32_t* __restrict__ cell, double* __restrict__ As,
                          int32_t* __restrict__ nleft) {
    const int k = blockIdx.x * kB + threadIdx.x;
    if (k == 0) *nleft = 0;   // of the triangulation's second kernel
    if (k >= g.N) return;
    const int p = perm[k];
    const double px = x[p], py = y[p];
    int cx, cy;
    double xi, eta;
    bool fx, fy;
    locate_axis(px, g.nx, g.inv_hx, cx, xi, fx);
    locate_axis(py, g.ny, g.inv_hy, cy, eta, fy);
    // a position in [L, L + h) belongs to cell 0 (the binning's wrap); move it there
    xs[k] = __dmul_rn(px, g.inv_hx) >= (double)g.nx ? px - g.lx : px;
    ys[k] = __dmul_rn(py, g.inv_hy) >= (double)g.ny ? py - g.ly : py;
    cell[k] = cx + g.nx * cy;
    if (values)
        for (int f = 0; f < F; ++f) As[(size_t)f * g.N + k] = values[(size_t)f * np + p];
}

// ---------------------------------------------------------------------------
// The Delaunay neighbours of slot k, counter-clockwise, by gift wrapping over the
// particles of the mesh cells within r rings of its own (coordinates relative to
// the particle).  The nearest particle is a Delaunay neighbour.  From a neighbour
// u, the next one is the particle c left of the edge (k, u) whose circle through
// k, u and c has its centre first along the edge's bisector: centre
// u / 2 + t (-u_y, u_x) with t = (|c|^2 - u.c) / (2 u x c), smallest t (an empty
// circle).  The centres are the Voronoi vertices; when twice the largest circle
// radius is within the searched radius (every particle left out is at least
// r min(hx, hy) away), no particle outside the rings can change the result;
// otherwise the search widens by a ring.
// One particle per group of G lanes: each lane scans every G-th cell of the
// search square, and the group agrees on the winner of every scan with a
// butterfly of lane exchanges (every lane ends with the same winner: the
// comparison of two candidates evaluates the same two products on both lanes).
struct Cand {
    double n, d;     // key n / d (d > 0)
    double vx, vy;   // position relative to the particle
    int q, s;        // slot and packed image shift; q < 0: none
};

// a before b: smaller key, ties to the smaller (slot, shift)
__device__ __forceinline__ bool before_cand(const Cand& a, const Cand& b) {
    if (a.q < 0) return false;
    if (b.q < 0) return true;
    const double l = a.n * b.d, r = b.n * a.d;
    if (l != r) return l < r;
    return a.q != b.q ? a.q < b.q : a.s < b.s;
}

// a found candidate before the wrap's best so far: one lane per particle scans in a
// fixed order, and equal keys there mean four points on one circle (a triangulation
// that is not unique), so the first found stands; a group breaks ties as above so
// that its winner does not depend on how the cells were dealt to its lanes
template <int G>
__device__ __forceinline__ bool before_wrap(const Cand& a, const Cand& b) {
    if constexpr (G == 1) return b.q < 0 || a.n * b.d < b.n * a.d;
    return before_cand(a, b);
}

template <int G>
__device__ __forceinline__ Cand group_min(Cand v) {
#pragma unroll
    for (int m = G / 2; m >= 1; m >>= 1) {
        Cand o;
        o.n = __shfl_xor(v.n, m, G);
        o.d = __shfl_xor(v.d, m, G);
        o.vx = __shfl_xor(v.vx, m, G);
        o.vy = __shfl_xor(v.vy, m, G);
        o.q = __shfl_xor(v.q, m, G);
        o.s = __shfl_xor(v.s, m, G);
        if (before_cand(o, v)) v = o;
    }
    return v;
}

template <int G>
__device__ __forceinline__ int group_or(int v) {
#pragma unroll
    for (int m = G / 2; m >= 1; m >>= 1) v |= __shfl_xor(v, m, G);
    return v;
}

// the particles of every G-th cell of the (2r + 1)^2 square around (cx, cy),
// starting at this lane's cell
template <int G, typename Fn>
__device__ __forceinline__ void for_lane_candidates(const Geo& g, const int32_t* __restrict__ cs,
                                                    int cx, int cy, int r, int lane, Fn&& fn) {
    if constexpr (G == 1) {   // row by row
        for (int dy = -r; dy <= r; ++dy) {
            const int ay = cy + dy;
            const int sy = floor_div(ay, g.ny);
            const int row = g.nx * (ay - sy * g.ny);
            for (int dx = -r; dx <= r; ++dx) {
                const int ax = cx + dx;
                const int sx = floor_div(ax, g.nx);
                const int cc = (ax - sx * g.nx) + row;
                const int q1 = cs[cc + 1];
                for (int q = cs[cc]; q < q1; ++q) fn(q, sx, sy);
            }
        }
    } else {   // cells lane, lane + G, ... of the square in row-major order
        const int side = 2 * r + 1, ncell = side * side;
        for (int ci = lane; ci < ncell; ci += G) {
            const int dyy = ci / side, dxx = ci - dyy * side;
            const int ax = cx + dxx - r, ay = cy + dyy - r;
            const int sx = floor_div(ax, g.nx), sy = floor_div(ay, g.ny);
            const int cc = (ax - sx * g.nx) + g.nx * (ay - sy * g.ny);
            const int q1 = cs[cc + 1];
            for (int q = cs[cc]; q < q1; ++q) fn(q, sx, sy);
        }
    }
}

template <int G>
__device__ void star_of(const Geo& g, int r0, int k, int lane, const double* __restrict__ xs,
                        const double* __restrict__ ys, const int32_t* __restrict__ cell,
                        const int32_t* __restrict__ cs, int32_t* __restrict__ deg,
                        int32_t* __restrict__ lst, double* __restrict__ vol, p2m_report* rep) {
    // plain rounding, no fused multiply-adds: the decisions below compare cross
    // products of nearly parallel vectors, and the same expression must give the
    // same result in every particle's computation
#pragma clang fp contract(off)
    const double px = xs[k], py = ys[k];
    const int c = cell[k];
    const int cy = c / g.nx, cx = c - cy * g.nx;
    const double hmin = g.hx < g.hy ? g.hx : g.hy;
    int32_t* nk = lst + (size_t)k * 2 * kCap;
    int n = 0;
    bool ok = false, bad = false;
    for (int r = r0; r <= kRingMax && !ok && !bad; ++r) {
        // the nearest particle image
        Cand b;
        b.q = -1;
        int dup = 0;
        for_lane_candidates<G>(g, cs, cx, cy, r, lane, [&](int q, int sx, int sy) {
            if (q == k && sx == 0 && sy == 0) return;
            Cand e;
            e.vx = (xs[q] - px) + sx * g.lx;
            e.vy = (ys[q] - py) + sy * g.ly;
            e.n = e.vx * e.vx + e.vy * e.vy;
            e.d = 1.0;
            e.q = q;
            e.s = pack_shift(sx, sy);
            if (!(e.n > 0.0)) dup = 1;   // two particles at one position
            if (before_cand(e, b)) b = e;
        });
        b = group_min<G>(b);
        bad = group_or<G>(dup) != 0;
        if (bad || b.q < 0) continue;
        const int q0 = b.q, s0 = b.s;
        int cq = q0, csh = s0;
        double ux = b.vx, uy = b.vy, rmax2 = 0.0;
        bool closed = false;
        n = 0;
        while (n < kCap) {
            if (lane == 0) {
                nk[at_slot(n)] = cq;
                nk[at_shift(n)] = csh;
            }
            ++n;
            // the particle left of (k, u) whose circle through k and u has its centre
            // first along the bisector: t = num / den, den = 2 u x c > 0
            Cand e;
            e.q = -1;
            for_lane_candidates<G>(g, cs, cx, cy, r, lane, [&](int q, int sx, int sy) {
                if (q == k && sx == 0 && sy == 0) return;
                const int sh = pack_shift(sx, sy);
                if (q == cq && sh == csh) return;   // the edge's own end
                const double rx = (xs[q] - px) + sx * g.lx;
                const double ry = (ys[q] - py) + sy * g.ly;
                const double cr = ux * ry - uy * rx;
                if (!(cr > 0.0)) return;
                Cand f;
                f.n = rx * rx + ry * ry - (ux * rx + uy * ry);
                f.d = 2.0 * cr;
                f.vx = rx;
                f.vy = ry;
                f.q = q;
                f.s = sh;
                if (before_wrap<G>(f, e)) e = f;
            });
            e = group_min<G>(e);
            if (e.q < 0) break;   // nothing on the left: the cell is open at this radius
            const double bt = e.n / e.d;
            const double ox = 0.5 * ux - bt * uy, oy = 0.5 * uy + bt * ux;
            const double rho2 = ox * ox + oy * oy;
            rmax2 = rho2 > rmax2 ? rho2 : rmax2;
            if (e.q == q0 && e.s == s0) {
                closed = true;
                break;
            }
            cq = e.q;
            csh = e.s;
            ux = e.vx;
            uy = e.vy;
        }
        const double reach = r * hmin * (1.0 - 1e-9);
        ok = closed && n >= 3 && 4.0 * rmax2 <= reach * reach;
    }
    if (!ok) {
        if (lane == 0) {
            deg[k] = 0;
            vol[k] = __builtin_nan("");
            flag(rep, P2M_FLAG_TRIANGULATION);
        }
        return;
    }
    if (lane != 0) return;
    deg[k] = n;
    double area2 = 0.0;
    double ax0 = 0.0, ay0 = 0.0, fx0 = 0.0, fy0 = 0.0;
    for (int i = 0; i < n; ++i) {
        const int q = nk[at_slot(i)], sh = nk[at_shift(i)];
        const double rx = (xs[q] - px) + shift_x(sh) * g.lx;
        const double ry = (ys[q] - py) + shift_y(sh) * g.ly;
        if (i == 0) {
            fx0 = rx;
            fy0 = ry;
        } else {
            area2 += ax0 * ry - ay0 * rx;
        }
        ax0 = rx;
        ay0 = ry;
    }
    area2 += ax0 * fy0 - ay0 * fx0;
    vol[k] = area2 / 6.0;   // a third of the triangles' total area (area2 / 2)
}

template <int G>
__global__ __launch_bounds__(kB) void k_x2d_star(Geo g, const double* __restrict__ xs,
                                                 const double* __restrict__ ys,
                                                 const int32_t* __restrict__ cell,
                                                 const int32_t* __restrict__ cs,
                                                 int32_t* __restrict__ deg, int32_t* __restrict__ lst,
                                                 double* __restrict__ vol, p2m_report* rep) {
    const int tid = blockIdx.x * kB + threadIdx.x;
    if (tid / G < g.N)   // the whole group
        star_of<G>(g, g.r0, tid / G, tid & (G - 1), xs, ys, cell, cs, deg, lst, vol, rep);
}

// The particles in left[0 .. *nleft): usually a few in a thousand, and then one
// particle's chain of scans is the kernel's time, so each gets a whole wave (16 lanes
// each took 79 us for 8,100 particles' few); 16 lanes where there are many.
constexpr int kFew = 4096;
__global__ __launch_bounds__(kB) void k_x2d_star_left(Geo g, const double* __restrict__ xs,
                                                      const double* __restrict__ ys,
                                                      const int32_t* __restrict__ cell,
                                                      const int32_t* __restrict__ cs,
                                                      int32_t* __restrict__ deg,
                                                      int32_t* __restrict__ lst,
                                                      double* __restrict__ vol,
                                                      const int32_t* __restrict__ nleft,
                                                      const int32_t* __restrict__ left,
                                                      p2m_report* rep) {
    const int tid = blockIdx.x * kB + threadIdx.x, n = *nleft;
    if (n <= kFew) {
        for (int at = tid / 64; at < n; at += gridDim.x * (kB / 64))
            star_of<64>(g, g.r0 + 1, left[at], tid & 63, xs, ys, cell, cs, deg, lst, vol, rep);
    } else {
        for (int at = tid / 16; at < n; at += gridDim.x * (kB / 16))
            star_of<16>(g, g.r0, left[at], tid & 15, xs, ys, cell, cs, deg, lst, vol, rep);
    }
}

// The same for almost every particle, four lanes each: the particles within a radius
// that is expected to hold 28 others (from the count of the 3 x 3 cells) are collected
// into LDS first, and the wrap scans those instead of whole cells; it stands when every
// circle's diameter is within that radius.  A particle whose list overflows or whose
// star is not closed that way goes to the general kernel's list.  1,048,576 particles at 4
// per cell: 100 candidates per scan, 2340 us, -> 28 and a one-off filter of the 100, 717 us.
// Bound: VALU issue, 4560 instructions a wave of 16 particles (cross products, key products
// and the quad's exchanges, more than their FP64 operations alone); they take two thirds of
// the SIMDs' cycles with 62% of the lanes on, at 2.4 waves a SIMD that wait 42% of the time
// (LDS conflicts: 2%).  Comparisons, rounding and ties as in the general
// kernel, so the lists and volumes are the same.
__device__ __forceinline__ double quad_move_d(double v, bool two) {
    return two ? dpp_quad<0x4E>(v) : dpp_quad<0xB1>(v);   // lanes two apart, or one
}

__global__ __launch_bounds__(kB) void k_x2d_star_quad(Geo g, const double* __restrict__ xs,
                                                      const double* __restrict__ ys,
                                                      const int32_t* __restrict__ cell,
                                                      const int32_t* __restrict__ cs,
                                                      int32_t* __restrict__ deg,
                                                      int32_t* __restrict__ lst,
                                                      double* __restrict__ vol,
                                                      int32_t* __restrict__ nleft,
                                                      int32_t* __restrict__ left) {
#pragma clang fp contract(off)
    constexpr int PB = kB / 4;
    __shared__ double2 s_r[PB][kCand];     // position relative to the particle
    __shared__ uint32_t s_id[PB][kCand];   // slot << 4 | image (ordered as slot, shift)
    const int lane = threadIdx.x & 3, p = threadIdx.x >> 2;
    const int k = blockIdx.x * PB + p;
    if (k >= g.N) return;   // the whole quad; no workgroup barrier below
    const double px = xs[k], py = ys[k];
    const int c = cell[k];
    const int cy = c / g.nx, cx = c - cy * g.nx;
    const double hmin = g.hx < g.hy ? g.hx : g.hy;
    // slots of columns [a, a + len) of row j (both may leave the mesh by less than it):
    // at most two runs
    auto runs = [&](int a, int len, int j, auto&& fn) {
        const int sy = j < 0 ? -1 : (j >= g.ny ? 1 : 0);
        const int32_t* row = cs + (size_t)g.nx * (j - sy * g.ny);
        while (len > 0) {
            const int sx = a < 0 ? -1 : (a >= g.nx ? 1 : 0);
            const int a0 = a - sx * g.nx, m = min(len, g.nx - a0);
            fn(row[a0], row[a0 + m], sx, sy);
            a += m;
            len -= m;
        }
    };
    int n9 = 0;
    for (int dy = -1; dy <= 1; ++dy)
        runs(cx - 1, 3, cy + dy, [&](int q0, int q1, int, int) { n9 += q1 - q0; });
    const double reach2 = 9.0 * g.hx * g.hy * (28.0 / 3.14159265358979) / (double)n9;
    double reach = sqrt(reach2);
    if (reach > kQuadRings * hmin) reach = kQuadRings * hmin;
    const double keep2 = reach * reach;
    int rx = (int)ceil(reach * (1.0 + 1e-9) * g.inv_hx), ry = (int)ceil(reach * (1.0 + 1e-9) * g.inv_hy);
    rx = rx > kQuadRings ? kQuadRings : rx;
    ry = ry > kQuadRings ? kQuadRings : ry;
    int cnt = 0;
    bool dup = false;
    const int wl = threadIdx.x & 63;
    for (int dy = -ry; dy <= ry; ++dy)
        runs(cx - rx, 2 * rx + 1, cy + dy, [&](int q0, int q1, int sx, int sy) {
            for (int q = q0; q < q1; q += 4) {   // the quad together
                const int i = q + lane;
                bool keep = false;
                double vx = 0.0, vy = 0.0;
                if (i < q1) {
                    vx = (xs[i] - px) + sx * g.lx;
                    vy = (ys[i] - py) + sy * g.ly;
                    const double n2 = vx * vx + vy * vy;
                    const bool self = i == k && sx == 0 && sy == 0;
                    keep = n2 <= keep2 && !self;
                    dup = dup || (!(n2 > 0.0) && !self);
                }
                const unsigned b = (unsigned)(__ballot(keep) >> (wl & ~3)) & 15u;
                const int at = cnt + __popc(b & ((1u << lane) - 1u));
                if (keep && at < kCand) {
                    s_r[p][at] = make_double2(vx, vy);
                    s_id[p][at] = ((uint32_t)i << 4) | (uint32_t)((sx + 1) + 3 * (sy + 1));
                }
                cnt += __popc(b);
            }
        });
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the quad reads what its lanes wrote
    const bool any_dup = ((unsigned)(__ballot(dup) >> (wl & ~3)) & 15u) != 0;
    bool ok = cnt <= kCand && cnt >= 3 && !any_dup;
    int nn = 0;
    double area2 = 0.0;
    if (ok) {
        // the winner of a scan over the quad: key n / d, ties to the smaller (slot, image)
        struct Best {
            double n, d;
            uint32_t id;
            int j;
        };
        auto before = [&](const Best& a, const Best& b) {
            if (a.j < 0) return false;
            if (b.j < 0) return true;
            const double l = a.n * b.d, r = b.n * a.d;
            if (l != r) return l < r;
            return a.id < b.id;
        };
        auto quad_min = [&](Best v) {
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                Best o;
                o.n = quad_move_d(v.n, m);
                o.d = quad_move_d(v.d, m);
                o.id = (uint32_t)(m ? __builtin_amdgcn_mov_dpp((int)v.id, 0x4E, 0xF, 0xF, false)
                                    : __builtin_amdgcn_mov_dpp((int)v.id, 0xB1, 0xF, 0xF, false));
                o.j = m ? __builtin_amdgcn_mov_dpp(v.j, 0x4E, 0xF, 0xF, false)
                        : __builtin_amdgcn_mov_dpp(v.j, 0xB1, 0xF, 0xF, false);
                if (before(o, v)) v = o;
            }
            return v;
        };
        Best b{0.0, 1.0, 0u, -1};
        for (int j = lane; j < cnt; j += 4) {
            const double2 v = s_r[p][j];
            const Best e{v.x * v.x + v.y * v.y, 1.0, s_id[p][j], j};
            if (before(e, b)) b = e;
        }
        b = quad_min(b);
        const int j0 = b.j;
        int cj = j0;
        const double2 first = s_r[p][j0];
        double ux = first.x, uy = first.y, rmax2 = 0.0;
        bool closed = false;
        int32_t* row = lst + (size_t)k * 2 * kCap;
        while (nn < kCap) {
            if (lane == 0) {
                const uint32_t id = s_id[p][cj];
                const int im = (int)(id & 15u);
                row[at_slot(nn)] = (int)(id >> 4);
                row[at_shift(nn)] = pack_shift(im % 3 - 1, im / 3 - 1);
            }
            ++nn;
            Best e{0.0, 1.0, 0u, -1};
            for (int j = lane; j < cnt; j += 4) {
                const double2 v = s_r[p][j];
                const double cr = ux * v.y - uy * v.x;
                if (!(cr > 0.0) || j == cj) continue;
                const Best f{v.x * v.x + v.y * v.y - (ux * v.x + uy * v.y), 2.0 * cr, s_id[p][j], j};
                if (before(f, e)) e = f;
            }
            e = quad_min(e);
            if (e.j < 0) break;   // nothing on the left: open within this radius
            const double bt = e.n / e.d;
            const double ox = 0.5 * ux - bt * uy, oy = 0.5 * uy + bt * ux;
            const double rho2 = ox * ox + oy * oy;
            rmax2 = rho2 > rmax2 ? rho2 : rmax2;
            const double2 v = s_r[p][e.j];
            area2 += ux * v.y - uy * v.x;
            if (e.j == j0) {
                closed = true;
                break;
            }
            cj = e.j;
            ux = v.x;
            uy = v.y;
        }
        const double lim = reach * (1.0 - 1e-9);
        ok = closed && nn >= 3 && 4.0 * rmax2 <= lim * lim;
    }
    if (lane != 0) return;
    if (!ok) {
        left[atomicAdd(nleft, 1)] = k;
        return;
    }
    deg[k] = nn;
    vol[k] = area2 / 6.0;   // a third of the triangles' total area (area2 / 2)
}

// position of neighbour (q, s) among the du entries of slot u's list, or -1 (a group of
// four entries is two 16-byte loads)
__device__ __forceinline__ int find_entry(const int32_t* __restrict__ lst, int du, int u, int q, int s) {
    const int4* l4 = (const int4*)(lst + (size_t)u * 2 * kCap);
    for (int j = 0; j < du; j += 4) {
        const int4 a = l4[j >> 1], b = l4[(j >> 1) + 1];
        if (a.x == q && b.x == s) return j;
        if (j + 1 < du && a.y == q && b.y == s) return j + 1;
        if (j + 2 < du && a.z == q && b.z == s) return j + 2;
        if (j + 3 < du && a.w == q && b.w == s) return j + 3;
    }
    return -1;
}

// ---------------------------------------------------------------------------
// Triangle (k, a, b) with a, b consecutive in k's list is (a, b, k) seen from a:
// in a's list, b must come right before k.  A failure marks the triangulation.  Four
// lanes a particle, each its own neighbours (a lane alone waits for them one by one).
__global__ void k_x2d_check(Geo g, const int32_t* __restrict__ deg, const int32_t* __restrict__ lst,
                            p2m_report* rep) {
    const size_t t = (size_t)blockIdx.x * kB + threadIdx.x;
    const int k = (int)(t >> 2);
    if (k >= g.N) return;
    const int d = deg[k];   // 0: flagged by the star kernel
    const int32_t* lk = lst + (size_t)k * 2 * kCap;
    bool ok = true;
    for (int i = (int)(t & 3); i < d && ok; i += 4) {
        const int a = lk[at_slot(i)], sa = lk[at_shift(i)];
        const int i1 = (i + 1 == d) ? 0 : i + 1;
        const int b = lk[at_slot(i1)], sb = lk[at_shift(i1)];
        const int da = deg[a];
        // k and b as seen from a's image
        const int sk = pack_shift(-shift_x(sa), -shift_y(sa));
        const int sba = pack_shift(shift_x(sb) - shift_x(sa), shift_y(sb) - shift_y(sa));
        const int j = find_entry(lst, da, a, k, sk);
        if (j < 0) {
            ok = false;
            break;
        }
        const int jp = (j == 0) ? da - 1 : j - 1;
        const int32_t* la = lst + (size_t)a * 2 * kCap;
        if (la[at_slot(jp)] != b || la[at_shift(jp)] != sba) ok = false;
    }
    if (!ok) flag(rep, P2M_FLAG_TRIANGULATION);
}

// ---------------------------------------------------------------------------
// The particle interpolant at grid point (I, J) of a gx x gy grid with spacing
// (dx, dy) (the nodes: the mesh itself; nodes and midpoints: half the spacing).
// out[f][J gx + I]; NaN where the walk fails.
struct Vtx {
    int q, sx, sy;
};

__global__ __launch_bounds__(kB) void k_x2d_locate(Geo g, int gx, int gy, double dx, double dy,
                                                   const double* __restrict__ xs,
                                                   const double* __restrict__ ys,
                                                   const int32_t* __restrict__ cs,
                                                   const int32_t* __restrict__ deg,
                                                   const int32_t* __restrict__ lst,
                                                   const double* __restrict__ As, int F,
                                                   double* __restrict__ out, p2m_report* rep) {
#pragma clang fp contract(off)   // orientation signs in plain rounding
    const int P = blockIdx.x * kB + threadIdx.x;
    if (P >= gx * gy) return;
    const int J = P / gx, I = P - J * gx;
    const double zx = I * dx, zy = J * dy;
    // cell of the point (points on a cell edge belong to the cell above / right)
    int cx = (int)floor(zx * g.inv_hx), cy = (int)floor(zy * g.inv_hy);
    cx = cx < 0 ? 0 : (cx >= g.nx ? g.nx - 1 : cx);
    cy = cy < 0 ? 0 : (cy >= g.ny ? g.ny - 1 : cy);
    const double hmin = g.hx < g.hy ? g.hx : g.hy;

    // nearest particle image
    double best = 1e300;
    Vtx a = {-1, 0, 0};
    for (int r = 0; r <= kRingMax; ++r) {
        for (int ddy = -r; ddy <= r; ++ddy) {
            const bool edge_row = (ddy == -r || ddy == r);
            const int step = edge_row ? 1 : 2 * r;
            for (int ddx = -r; ddx <= r; ddx += (step > 0 ? step : 1)) {
                const int ax = cx + ddx, ay = cy + ddy;
                const int sx = floor_div(ax, g.nx), sy = floor_div(ay, g.ny);
                const int cc = (ax - sx * g.nx) + g.nx * (ay - sy * g.ny);
                const int q1 = cs[cc + 1];
                for (int q = cs[cc]; q < q1; ++q) {
                    const double rx = (xs[q] - zx) + sx * g.lx;
                    const double ry = (ys[q] - zy) + sy * g.ly;
                    const double d2 = rx * rx + ry * ry;
                    if (d2 < best) {
                        best = d2;
                        a.q = q;
                        a.sx = sx;
                        a.sy = sy;
                    }
                }
                if (step == 0) break;
            }
        }
        const double reach = r * hmin;
        if (a.q >= 0 && best <= reach * reach) break;
    }
    bool ok = a.q >= 0 && deg[a.q] >= 3;
    double la = 0.0, lb = 0.0, lc = 0.0;
    Vtx b = {0, 0, 0}, c = {0, 0, 0};
    auto entry = [&](const Vtx& u, int j) -> Vtx {
        const int32_t* lu = lst + (size_t)u.q * 2 * kCap;
        const int s = lu[at_shift(j)];
        return Vtx{lu[at_slot(j)], u.sx + shift_x(s), u.sy + shift_y(s)};
    };
    auto rel = [&](const Vtx& v, double& rx, double& ry) {
        rx = (xs[v.q] - zx) + v.sx * g.lx;
        ry = (ys[v.q] - zy) + v.sy * g.ly;
    };
    // the neighbour that comes right before v in u's list (the third vertex of
    // the triangle across edge (u, v) from the current one)
    auto before = [&](const Vtx& u, const Vtx& v, Vtx& x) -> bool {
        const int du = deg[u.q];
        if (du < 3) return false;
        const int j = find_entry(lst, du, u.q, v.q, pack_shift(v.sx - u.sx, v.sy - u.sy));
        if (j < 0) return false;
        x = entry(u, j == 0 ? du - 1 : j - 1);
        return true;
    };
    if (ok) {
        b = entry(a, 0);
        c = entry(a, 1);
        ok = false;
        for (int step = 0; step < kWalkMax; ++step) {
            double ax_, ay_, bx_, by_, cx_, cy_;
            rel(a, ax_, ay_);
            rel(b, bx_, by_);
            rel(c, cx_, cy_);
            // twice the signed areas of (a, b, z), (b, c, z), (c, a, z) with z at 0
            const double oab = ax_ * by_ - ay_ * bx_;
            const double obc = bx_ * cy_ - by_ * cx_;
            const double oca = cx_ * ay_ - cy_ * ax_;
            Vtx x;
            if (oab < 0.0) {
                if (!before(a, b, x)) break;
                c = b;
                b = x;   // (a, x, b)
            } else if (obc < 0.0) {
                if (!before(b, c, x)) break;
                a = b;
                b = x;   // (b, x, c)
            } else if (oca < 0.0) {
                if (!before(c, a, x)) break;
                b = x;
                const Vtx t = a;
                a = c;
                c = t;   // (c, x, a)
            } else {
                const double s = oab + obc + oca;
                la = obc / s;
                lb = oca / s;
                lc = oab / s;
                ok = s > 0.0;
                break;
            }
        }
    }
    if (!ok) {
        for (int f = 0; f < F; ++f) out[(size_t)f * gx * gy + P] = __builtin_nan("");
        flag(rep, P2M_FLAG_TRIANGULATION);
        return;
    }
    for (int f = 0; f < F; ++f) {
        const double* A = As + (size_t)f * g.N;
        out[(size_t)f * gx * gy + P] = la * A[a.q] + lb * A[b.q] + lc * A[c.q];
    }
}

// ---------------------------------------------------------------------------
// Appendix-B rule on one triangle for its vertex a: |T| (Qa/30 - (Qb + Qc)/60 +
// 2 (Qab + Qac)/15 + Qbc/15)
__device__ __forceinline__ double appb(double area, double qa, double qb, double qc, double qab,
                                       double qac, double qbc) {
    return area * (qa * (1.0 / 30.0) - (qb + qc) * (1.0 / 60.0) + (qab + qac) * (2.0 / 15.0) +
                   qbc * (1.0 / 15.0));
}

// b_j over the six triangles of the "/" split around node (i, j); H [F][2ny][2nx]
// holds A on the half-spacing grid (node (i, j) at (2i, 2j)).
__global__ void k_x2d_rhs_mesh(Geo g, int F, const double* __restrict__ H, double* __restrict__ b) {
    const int k = blockIdx.x * kB + threadIdx.x;
    const int nn = g.nx * g.ny;
    if (k >= nn) return;
    const int j = k / g.nx, i = k - j * g.nx;
    const int gx = 2 * g.nx, gy = 2 * g.ny;
    // the other two vertices of each triangle, in half-spacing offsets
    const int ob[6][2] = {{2, 0}, {2, 2}, {-2, 0}, {-2, -2}, {-2, -2}, {0, -2}};
    const int oc[6][2] = {{2, 2}, {0, 2}, {0, 2}, {0, -2}, {-2, 0}, {2, 0}};
    const double area = 0.5 * g.hx * g.hy;
    for (int f = 0; f < F; ++f) {
        const double* Hf = H + (size_t)f * gx * gy;
        auto at = [&](int di, int dj) -> double {
            int I = 2 * i + di, Jj = 2 * j + dj;
            I = I < 0 ? I + gx : (I >= gx ? I - gx : I);
            Jj = Jj < 0 ? Jj + gy : (Jj >= gy ? Jj - gy : Jj);
            return Hf[(size_t)Jj * gx + I];
        };
        const double qa = at(0, 0);
        double s = 0.0;
#pragma unroll
        for (int t = 0; t < 6; ++t) {
            const int bx = ob[t][0], by = ob[t][1], cx = oc[t][0], cy = oc[t][1];
            s += appb(area, qa, at(bx, by), at(cx, cy), at(bx / 2, by / 2), at(cx / 2, cy / 2),
                      at((bx + cx) / 2, (by + cy) / 2));
        }
        b[(size_t)f * nn + k] = s;
    }
}

// the mesh interpolant (eq. (3) hats, "/" split) at a point of the plane
__device__ __forceinline__ double mesh_at(const Geo& g, const double* __restrict__ nodal, double x,
                                          double y) {
    x -= floor(x * g.inv_lx) * g.lx;
    y -= floor(y * g.inv_ly) * g.ly;
    int cx, cy;
    double xi, eta;
    bool fx, fy;
    locate_axis(x, g.nx, g.inv_hx, cx, xi, fx);
    locate_axis(y, g.ny, g.inv_hy, cy, eta, fy);
    double c00, c10, c11, c01;
    corner_weights<double>(xi, eta, c00, c10, c11, c01);
    const int i1 = (cx + 1 == g.nx) ? 0 : cx + 1, j1 = (cy + 1 == g.ny) ? 0 : cy + 1;
    return c00 * nodal[cx + g.nx * cy] + c10 * nodal[i1 + g.nx * cy] +
           c11 * nodal[i1 + g.nx * j1] + c01 * nodal[cx + g.nx * j1];
}

// c_mu over the triangles (mu, n_i, n_i+1) of slot k; c [F][N].  With coef, the same walk
// round the star writes the particle mass matrix in sparse-row form: coef[k] =
// sum |T| / 6; slot i of row k is the neighbour n_i with (|T_{i-1}| + |T_i|) / 12,
// T_i = (mu, n_i, n_i+1); a column of -1 ends the row (the solves read no slot behind it;
// clearing all 32 slots wrote 400 MB a million particles).
__global__ __launch_bounds__(kB) void k_x2d_rhs_part(Geo g, int F, const double* __restrict__ xs,
                               const double* __restrict__ ys, const int32_t* __restrict__ deg,
                               const int32_t* __restrict__ lst, const double* __restrict__ nodal,
                               double* __restrict__ c, double* __restrict__ coef,
                               int32_t* __restrict__ ecol) {
    const int k = blockIdx.x * kB + threadIdx.x;
    if (k >= g.N) return;
    const size_t N = (size_t)g.N;
    const int d = deg[k];
    const int nn = g.nx * g.ny;
    const double px = xs[k], py = ys[k];
    const int32_t* lk = lst + (size_t)k * 2 * kCap;
    auto rel = [&](int i, int& q, double& rx, double& ry) {
        const int sh = lk[at_shift(i)];
        q = lk[at_slot(i)];
        rx = (xs[q] - px) + shift_x(sh) * g.lx;
        ry = (ys[q] - py) + shift_y(sh) * g.ly;
    };
    for (int f = 0; f < F; ++f) {
        const double* Af = nodal + (size_t)f * nn;
        if (d == 0) {
            c[(size_t)f * N + k] = __builtin_nan("");
            continue;
        }
        const double qp = mesh_at(g, Af, px, py);
        double s = 0.0, ax, ay;
        int q;
        rel(d - 1, q, ax, ay);
        double qa = mesh_at(g, Af, px + ax, py + ay);
        double qpa = mesh_at(g, Af, px + 0.5 * ax, py + 0.5 * ay);
        double diag = 0.0, t0 = 0.0, tprev = 0.0;   // T_{d-1}, T_{i-1}
        int qprev = q;
        for (int i = 0; i < d; ++i) {
            double bx, by;
            rel(i, q, bx, by);
            const double qb = mesh_at(g, Af, px + bx, py + by);
            const double qpb = mesh_at(g, Af, px + 0.5 * bx, py + 0.5 * by);
            const double qab = mesh_at(g, Af, px + 0.5 * (ax + bx), py + 0.5 * (ay + by));
            const double area = 0.5 * (ax * by - ay * bx);   // triangle (mu, a, b) = T_{i-1}
            s += appb(area, qp, qa, qb, qpa, qpb, qab);
            if (coef && f == 0) {
                // entry i - 1 is complete once T_{i-1} is known; entry d - 1 after the loop
                if (i == 0) {
                    t0 = area;
                } else {
                    coef[N + (size_t)(i - 1) * N + k] = (tprev + area) * (1.0 / 12.0);
                    ecol[(size_t)(i - 1) * N + k] = qprev;
                }
                diag += area;
                tprev = area;
                qprev = q;
            }
            ax = bx;
            ay = by;
            qa = qb;
            qpa = qpb;
        }
        c[(size_t)f * N + k] = s;
        if (coef && f == 0) {
            coef[N + (size_t)(d - 1) * N + k] = (tprev + t0) * (1.0 / 12.0);
            ecol[(size_t)(d - 1) * N + k] = qprev;
            coef[k] = diag * (1.0 / 6.0);
        }
    }
    if (coef && d == 0) coef[k] = 0.0;
    if (coef && d < kCap) ecol[(size_t)d * N + k] = -1;
}

// consistent mesh mass stencil (Sec. 2.4 on the "/" split): D = hx hy / 2 and
// E = N = NE = hx hy / 12; w = hx hy (its row sums, the FLIP start's volumes)
__global__ void k_x2d_mmesh(int nn, double cm, double* __restrict__ coef, double* __restrict__ w) {
    const int k = blockIdx.x * kB + threadIdx.x;
    if (k >= nn) return;
    coef[k] = 0.5 * cm;
    coef[(size_t)nn + k] = cm / 12.0;
    coef[(size_t)2 * nn + k] = cm / 12.0;
    coef[(size_t)3 * nn + k] = cm / 12.0;
    w[k] = cm;
}

// caller-order triangulation (deg, neighbours as caller numbers, shifts)
__global__ void k_x2d_export(Geo g, const int32_t* __restrict__ perm, const int32_t* __restrict__ deg,
                             const int32_t* __restrict__ lst, int32_t* __restrict__ deg_out,
                             int32_t* __restrict__ nbr_out, int32_t* __restrict__ sh_out) {
    // a lane an entry: a particle's rows are written whole (entry numbers pass 2^31 from
    // 67,108,864 particles on)
    const size_t n = (size_t)g.N * kCap;
    for (size_t t = (size_t)blockIdx.x * kB + threadIdx.x; t < n; t += (size_t)gridDim.x * kB) {
        const int k = (int)(t / kCap), i = (int)(t % kCap);
        const int p = perm[k], d = deg[k];
        if (i == 0) deg_out[p] = d;
        const int32_t* lk = lst + (size_t)k * 2 * kCap;
        nbr_out[(size_t)p * kCap + i] = i < d ? perm[lk[at_slot(i)]] : -1;
        sh_out[(size_t)p * kCap + i] = i < d ? lk[at_shift(i)] : 0;
    }
}

__global__ void k_x2d_clear_export(int np, int32_t* __restrict__ deg_out,
                                   int32_t* __restrict__ nbr_out, int32_t* __restrict__ sh_out) {
    const int p = blockIdx.x * kB + threadIdx.x;
    if (p >= np) return;
    deg_out[p] = 0;
    for (int i = 0; i < kCap; ++i) {
        nbr_out[(size_t)p * kCap + i] = -1;
        sh_out[(size_t)p * kCap + i] = 0;
    }
}

Geo geo_of(const Mesh& m, int N, double lx, double ly) {
    Geo g;
    g.nx = m.nx;
    g.ny = m.ny;
    g.N = N;
    g.lx = lx;
    g.ly = ly;
    g.hx = lx / m.nx;
    g.hy = ly / m.ny;
    g.inv_hx = m.inv_hx;
    g.inv_hy = m.inv_hy;
    g.inv_lx = 1.0 / lx;
    g.inv_ly = 1.0 / ly;
    // dense particles (six or more per cell) usually close their cells within one
    // ring, sparser ones within two
    g.r0 = (m.nn > 0 && N >= 6 * (long)m.nn) ? 1 : 2;
    return g;
}

}  // namespace

#define X2D_TRY(e)                           \
    do {                                     \
        hipError_t e_ = (e);                 \
        if (e_ != hipSuccess) return e_;     \
    } while (0)

hipError_t x2d_triangulate(const X2dArgs& a, hipStream_t stream) {
    if (a.N == 0) return hipSuccess;
    const Geo g = geo_of(a.m, a.N, a.lx, a.ly);
    hipLaunchKernelGGL(k_x2d_pos, dim3(grid_of(a.N)), dim3(kB), 0, stream, g, a.perm, a.x, a.y,
                       a.values, a.F, a.m.np, a.xs, a.ys, a.cell, a.As, a.nleft);
    X2D_TRY(hipGetLastError());
    // Four lanes a particle over the candidates within a radius, then the general kernel
    // over what that left.  Meshes narrower than the quad's square (its images would
    // overlap) and counts beyond the candidates' 28-bit slots go to the general kernel
    // whole: 16 lanes a particle while that fits about 2^19 lanes (what 256 compute units
    // hold), else one.
    const bool quad = a.m.nx > 2 * kQuadRings && a.m.ny > 2 * kQuadRings && a.N < (1 << 28);
    if (quad) {
        hipLaunchKernelGGL(k_x2d_star_quad, dim3((a.N + kB / 4 - 1) / (kB / 4)), dim3(kB), 0, stream, g,
                           a.xs, a.ys, a.cell, a.cs, a.deg, a.lst, a.vol, a.nleft, a.left);
        X2D_TRY(hipGetLastError());
        const int most = 2048, need = grid_of((size_t)a.N * 64);
        hipLaunchKernelGGL(k_x2d_star_left, dim3(need < most ? need : most), dim3(kB), 0, stream, g,
                           a.xs, a.ys, a.cell, a.cs, a.deg, a.lst, a.vol, (const int32_t*)a.nleft,
                           (const int32_t*)a.left, a.rep);
    } else if ((size_t)a.N * 16 <= ((size_t)1 << 19)) {
        hipLaunchKernelGGL(k_x2d_star<16>, dim3(grid_of((size_t)a.N * 16)), dim3(kB), 0, stream, g, a.xs,
                           a.ys, a.cell, a.cs, a.deg, a.lst, a.vol, a.rep);
    } else {
        hipLaunchKernelGGL(k_x2d_star<1>, dim3(grid_of(a.N)), dim3(kB), 0, stream, g, a.xs, a.ys, a.cell,
                           a.cs, a.deg, a.lst, a.vol, a.rep);
    }
    X2D_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_x2d_check, dim3((a.N + kB / 4 - 1) / (kB / 4)), dim3(kB), 0, stream, g, a.deg,
                       a.lst, a.rep);
    return hipGetLastError();
}

hipError_t x2d_export(const X2dArgs& a, int32_t* deg_out, int32_t* nbr_out, int32_t* sh_out,
                      hipStream_t stream) {
    if (a.m.np > 0) {
        hipLaunchKernelGGL(k_x2d_clear_export, dim3(grid_of(a.m.np)), dim3(kB), 0, stream, a.m.np,
                           deg_out, nbr_out, sh_out);
        X2D_TRY(hipGetLastError());
    }
    if (a.N == 0) return hipSuccess;
    const Geo g = geo_of(a.m, a.N, a.lx, a.ly);
    const int most = 1 << 24, need = grid_of((size_t)a.N * kCap);   // a launch has at most 2^32 threads
    hipLaunchKernelGGL(k_x2d_export, dim3(need < most ? need : most), dim3(kB), 0, stream, g, a.perm,
                       a.deg, a.lst, deg_out, nbr_out, sh_out);
    return hipGetLastError();
}

hipError_t x2d_locate(const X2dArgs& a, bool half, double* out, hipStream_t stream) {
    const Geo g = geo_of(a.m, a.N, a.lx, a.ly);
    const int gx = half ? 2 * a.m.nx : a.m.nx, gy = half ? 2 * a.m.ny : a.m.ny;
    const double dx = half ? 0.5 * g.hx : g.hx, dy = half ? 0.5 * g.hy : g.hy;
    hipLaunchKernelGGL(k_x2d_locate, dim3(grid_of((size_t)gx * gy)), dim3(kB), 0, stream, g, gx, gy,
                       dx, dy, a.xs, a.ys, a.cs, a.deg, a.lst, a.As, a.F, out, a.rep);
    return hipGetLastError();
}

hipError_t x2d_rhs_mesh(const X2dArgs& a, const double* H, double* b, hipStream_t stream) {
    const Geo g = geo_of(a.m, a.N, a.lx, a.ly);
    hipLaunchKernelGGL(k_x2d_rhs_mesh, dim3(grid_of(a.m.nn)), dim3(kB), 0, stream, g, a.F, H, b);
    return hipGetLastError();
}

hipError_t x2d_mass_mesh(const X2dArgs& a, double* coef, double* w, hipStream_t stream) {
    hipLaunchKernelGGL(k_x2d_mmesh, dim3(grid_of(a.m.nn)), dim3(kB), 0, stream, a.m.nn,
                       a.m.cell_measure, coef, w);
    return hipGetLastError();
}

hipError_t x2d_rhs_part(const X2dArgs& a, const double* nodal, double* c, double* coef, int32_t* ecol,
                        hipStream_t stream) {
    if (a.N == 0) return hipSuccess;
    const Geo g = geo_of(a.m, a.N, a.lx, a.ly);
    hipLaunchKernelGGL(k_x2d_rhs_part, dim3(grid_of(a.N)), dim3(kB), 0, stream, g, a.F, a.xs, a.ys,
                       a.deg, a.lst, nodal, c, coef, ecol);
    return hipGetLastError();
}

}  // namespace p2m
