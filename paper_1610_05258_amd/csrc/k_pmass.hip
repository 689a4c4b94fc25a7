// Particle mass system of the paper-exact 2D M2P (eq. (20)): m_part x = c for F fields,
// m_part in sparse-row form (diagonal, then up to 32 slots a row, slot-major, ended by a
// column of -1), all in FP64.
//
// The spectrum is known: an element's mass matrix |T|/12 (I + J) against its diagonal
// |T|/6 I has the eigenvalues 1/2, 1/2 and 2, so every eigenvalue of D^-1 m_part lies in
// [1/2, 2] whatever the triangles, and the Chebyshev iteration on that interval converges
// at the rate 1/3 with no dot product: K = log3(4 / tol) steps, each one sparse product
// against the true residual (c - M x, not a recursion), then one residual check.  A step
// moves the row (12 bytes an entry) and 40 bytes of vectors; its neighbours' x come from
// L2, which is why each XCD takes one contiguous run of rows.
//
//  * many rows: one launch per step (the launch boundary is the cheapest grid-wide
//    ordering for vectors that are gathered through the L2s).  1,048,576 rows: 3.03 ms
//    (CG, two fenced grid barriers per iteration) -> 0.98 ms, 29.5 us a step.
//  * few rows (kSmallRows): one persistent kernel, a row per thread with its entries in
//    registers, x exchanged through device-coherent accesses and one counter-tree barrier
//    a step: a launch per step would cost more than the step.  8,100 rows: 383 -> 120 us.
//    Whole M2P by the one kernel and by the launches, F = 1: 8,100 rows 230 and 250 us, 32,761
//    rows 260 and 288, 65,536 rows 300 and 323; F = 3: 287 and 318, 322 and 352, 394 and 399,
//    90,000 rows 462 and 451.  The line at 32,768, below the crossing, keeps one workgroup on
//    every second compute unit, so that the grid is resident beside other work.
//
// A solve that does not reach tol, or that meets a row without a volume or a value that
// is not finite, leaves the word `ok` at 0; the streaming CG enqueued behind it then does
// the whole solve (and reports orphans and breakdowns), otherwise it returns at once.
#include "cg_common.hpp"

namespace p2m {

namespace {

constexpr int kPB = 256;
constexpr int kSmallRows = 32768;     // the persistent form: at most 128 workgroups
constexpr int kRegs = 8;              // row entries held in registers

struct PmArgs {
    int N, F, K;
    const double* coef;    // [N] diagonal, then slots
    const int32_t* ecol;   // [slot][N]
    const double* c;       // [F][N]
    const double* vol;     // [N] the start is c / vol
    double* x0;            // [F][N] iterates
    double* x1;
    double* d;             // [F][N] last step
    double* part;          // [2 F][blocks] residual and right-hand side partials
    double tol;
    int* ok;               // 1: x1 holds the solution
    int* bad;              // a row without a volume, or a value that is not finite
    double* out;
    p2m_report* rep;
    RSync sy;
};

// Chebyshev coefficients of step k on [1/2, 2]: theta = 5/4, delta = 3/4, sigma = 5/3;
// d <- a d + b D^-1 r
struct Step {
    double a, b;
};
__host__ __device__ inline void cheb_next(int k, double& rho, Step& s) {
    if (k == 0) {
        rho = 0.6;
        s.a = 0.0;
        s.b = 0.8;
        return;
    }
    const double rn = 1.0 / (10.0 / 3.0 - rho);
    s.a = rn * rho;
    s.b = 2.0 * rn / 0.75;
    rho = rn;
}

// workgroup of a step -> run of rows: the workgroups of one XCD (dealt round robin over
// the 8) take one contiguous range, so its L2 holds the x they gather
__device__ __forceinline__ int run_of(int b, int nb) {
    const int per = nb / 8, full = per * 8;
    return b < full ? (b & 7) * per + (b >> 3) : b;
}

__global__ __launch_bounds__(kPB) void k_pm_start(PmArgs a) {
    const int k = blockIdx.x * kPB + threadIdx.x;
    if (k >= a.N) return;
    const double v = a.vol[k];
    bool bad = !(v > 0.0);
    for (int f = 0; f < a.F; ++f) {
        const double x = a.c[(size_t)f * a.N + k] / v;
        bad = bad || !(x - x == 0.0);
        a.x0[(size_t)f * a.N + k] = x;
    }
    if (bad) *a.bad = 1;
}

// one step (CHECK false): x1 = x0 + d, d = s.a d + s.b D^-1 (c - M x0); or the residual of
// x0 into the partials
template <int F, bool CHECK>
__global__ __launch_bounds__(kPB) void k_pm_step(PmArgs a, const double* __restrict__ xin,
                                                 double* __restrict__ xout, Step s, int first) {
    const int k = run_of(blockIdx.x, gridDim.x) * kPB + threadIdx.x;
    const size_t N = (size_t)a.N;
    double rr[F], bb[F];
#pragma unroll
    for (int f = 0; f < F; ++f) rr[f] = bb[f] = 0.0;
    if (k < a.N) {
        const double D = a.coef[k];
        double m[F], x[F];
#pragma unroll
        for (int f = 0; f < F; ++f) {
            x[f] = xin[f * N + k];
            m[f] = D * x[f];
        }
        // four slots at a time: their loads are in flight together
        for (int j = 0; j < P2M_X2D_MAXDEG; j += 4) {
            int col[4];
            double e[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                col[u] = a.ecol[(size_t)(j + u) * N + k];
                e[u] = a.coef[(size_t)(j + u + 1) * N + k];
            }
            // entries end at the first -1; what lies behind it is not read into the sum
#pragma unroll
            for (int u = 1; u < 4; ++u)
                if (col[u - 1] < 0) col[u] = -1;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (col[u] < 0) continue;
#pragma unroll
                for (int f = 0; f < F; ++f) m[f] = fma(e[u], xin[f * N + col[u]], m[f]);
            }
            if (col[3] < 0) break;
        }
#pragma unroll
        for (int f = 0; f < F; ++f) {
            const double cf = a.c[f * N + k], r = cf - m[f];
            if (CHECK) {
                rr[f] = r * r;
                bb[f] = cf * cf;
                a.out[f * N + k] = x[f];
            } else {
                const double dn = s.a * (first ? 0.0 : a.d[f * N + k]) + s.b * (r / D);
                a.d[f * N + k] = dn;
                xout[f * N + k] = x[f] + dn;
            }
        }
    }
    if (CHECK) {
        __shared__ double lds[2][kPB / 64];
#pragma unroll
        for (int f = 0; f < F; ++f) {
            const double p = row_sum16(rr[f]), q = row_sum16(bb[f]);
            const double ps = (readlane_d(p, 0) + readlane_d(p, 16)) + (readlane_d(p, 32) + readlane_d(p, 48));
            const double qs = (readlane_d(q, 0) + readlane_d(q, 16)) + (readlane_d(q, 32) + readlane_d(q, 48));
            if ((threadIdx.x & 63) == 0) {
                lds[0][threadIdx.x >> 6] = ps;
                lds[1][threadIdx.x >> 6] = qs;
            }
            __syncthreads();
            if (threadIdx.x < 2) {
                const double* q4 = lds[threadIdx.x];
                a.part[(size_t)(2 * f + threadIdx.x) * gridDim.x + blockIdx.x] =
                    (q4[0] + q4[1]) + (q4[2] + q4[3]);
            }
            __syncthreads();
        }
    }
}

// one workgroup: totals in a fixed order, the report, and whether the solve stands
__device__ void pm_decide(const PmArgs& a, const double* part, int blocks) {
    __shared__ double tot[2 * kMaxFields];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int v = wave; v < 2 * a.F; v += kPB / 64) {
        double s = 0.0;
        for (int i = lane; i < blocks; i += 64) s += ld_c(part + (size_t)v * blocks + i);
        const double p = row_sum16(s);
        const double t = (readlane_d(p, 0) + readlane_d(p, 16)) + (readlane_d(p, 32) + readlane_d(p, 48));
        if (lane == 0) tot[v] = t;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        bool ok = *a.bad == 0;
        for (int f = 0; f < a.F; ++f) {
            const double bb = tot[2 * f + 1], rel = bb == 0.0 ? 0.0 : sqrt(tot[2 * f] / bb);
            ok = ok && rel <= a.tol;
        }
        if (ok && a.rep) {
            for (int f = 0; f < a.F; ++f) {
                const double bb = tot[2 * f + 1];
                a.rep->iters[f] = bb == 0.0 ? 0 : a.K;
                a.rep->refines[f] = 1;
                a.rep->rel_residual[f] = bb == 0.0 ? 0.0 : sqrt(tot[2 * f] / bb);
            }
        }
        *a.ok = ok ? 1 : 0;
    }
}

__global__ __launch_bounds__(kPB) void k_pm_decide(PmArgs a, int blocks) { pm_decide(a, a.part, blocks); }

// Few rows: the whole solve in one launch.  Row k of thread k; entries beyond kRegs stay
// in memory.  x is published with device-coherent stores, double-buffered by step parity
// (a workgroup overwrites step k's buffer two barriers later, when every workgroup has
// read it), and the last workgroup past the final barrier has every partial stored.
template <int F>
__global__ __launch_bounds__(kPB) void k_pm_small(PmArgs a) {
    const size_t N = (size_t)a.N;
    const int k = blockIdx.x * kPB + threadIdx.x, nb = gridDim.x;
    const bool on = k < a.N;
    __shared__ int s_ok;
    unsigned epoch = 0;
    auto sync = [&]() -> bool {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (nb == 1) return true;
        ++epoch;
        if (threadIdx.x == 0) {
            if (tree_arrive(a.sy, epoch, nb)) tree_release(a.sy, epoch);
            s_ok = tree_wait(a.sy, epoch) ? 1 : 0;
        }
        __syncthreads();
        return s_ok != 0;
    };
    int col[kRegs];
    double e[kRegs], D = 1.0, di = 1.0, x[F], d[F], c[F];
    bool more = on;
#pragma unroll
    for (int j = 0; j < kRegs; ++j) {
        col[j] = more ? a.ecol[(size_t)j * N + k] : -1;
        more = more && col[j] >= 0;
        if (!more) col[j] = -1;
        e[j] = more ? a.coef[(size_t)(j + 1) * N + k] : 0.0;
    }
    bool bad = false;
    if (on) {
        D = a.coef[k];
        di = 1.0 / D;
    }
#pragma unroll
    for (int f = 0; f < F; ++f) {
        c[f] = on ? a.c[f * N + k] : 0.0;
        const double v = on ? a.vol[k] : 1.0;
        x[f] = c[f] / v;
        d[f] = 0.0;
        bad = bad || !(v > 0.0) || !(x[f] - x[f] == 0.0);
        if (on) st_c(a.x0 + f * N + k, x[f]);
    }
    if (bad) __hip_atomic_store(a.bad, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    bool alive = sync();
    double rho = 0.0, r[F];
    for (int step = 0; alive; ++step) {
        const double* xin = step & 1 ? a.x1 : a.x0;
        double* xout = step & 1 ? a.x0 : a.x1;
        double g[F][kRegs];
#pragma unroll
        for (int f = 0; f < F; ++f)
#pragma unroll
            for (int j = 0; j < kRegs; ++j) g[f][j] = col[j] >= 0 ? ld_c(xin + f * N + col[j]) : 0.0;
#pragma unroll
        for (int f = 0; f < F; ++f) {
            double m = D * x[f];
#pragma unroll
            for (int j = 0; j < kRegs; ++j) m = fma(e[j], g[f][j], m);
            r[f] = m;
        }
        if (more)
            for (int j = kRegs; j < P2M_X2D_MAXDEG; ++j) {
                const int q = a.ecol[(size_t)j * N + k];
                if (q < 0) break;
                const double w = a.coef[(size_t)(j + 1) * N + k];
#pragma unroll
                for (int f = 0; f < F; ++f) r[f] = fma(w, ld_c(xin + f * N + q), r[f]);
            }
#pragma unroll
        for (int f = 0; f < F; ++f) r[f] = c[f] - r[f];
        if (step == a.K) break;
        Step s;
        cheb_next(step, rho, s);
#pragma unroll
        for (int f = 0; f < F; ++f) {
            d[f] = s.a * d[f] + s.b * (r[f] * di);
            x[f] += d[f];
            if (on) st_c(xout + f * N + k, x[f]);
        }
        alive = sync();
    }
    // residual partials of this workgroup, the result, and the decision by workgroup 0
    __shared__ double lds[2 * F][kPB / 64];
#pragma unroll
    for (int f = 0; f < F; ++f) {
        if (on) a.out[f * N + k] = x[f];
        const double p = row_sum16(on ? r[f] * r[f] : 0.0), q = row_sum16(on ? c[f] * c[f] : 0.0);
        const double ps = (readlane_d(p, 0) + readlane_d(p, 16)) + (readlane_d(p, 32) + readlane_d(p, 48));
        const double qs = (readlane_d(q, 0) + readlane_d(q, 16)) + (readlane_d(q, 32) + readlane_d(q, 48));
        if ((threadIdx.x & 63) == 0) {
            lds[2 * f][threadIdx.x >> 6] = ps;
            lds[2 * f + 1][threadIdx.x >> 6] = qs;
        }
    }
    __syncthreads();
    if (threadIdx.x < 2 * F) {
        const double* q4 = lds[threadIdx.x];
        st_c(a.part + (size_t)threadIdx.x * nb + blockIdx.x, (q4[0] + q4[1]) + (q4[2] + q4[3]));
    }
    if (!alive) return;   // every workgroup sees the abort; ok stays 0
    alive = sync();
    if (alive && blockIdx.x == 0) pm_decide(a, a.part, nb);
}

__global__ void k_pm_clear(unsigned* words, int n, int* ok, int* bad) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) words[i] = 0u;
    if (threadIdx.x == 0) {
        *ok = 0;
        *bad = 0;
    }
}

template <int F>
hipError_t run(PmArgs a, int blocks, hipStream_t stream) {
    if (a.N <= kSmallRows) {
        hipLaunchKernelGGL(k_pm_small<F>, dim3(blocks), dim3(kPB), 0, stream, a);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_pm_start, dim3(blocks), dim3(kPB), 0, stream, a);
    double rho = 0.0;
    double* in = a.x0;
    double* out = a.x1;
    for (int k = 0; k < a.K; ++k) {
        Step s;
        cheb_next(k, rho, s);
        hipLaunchKernelGGL(HIP_KERNEL_NAME(k_pm_step<F, false>), dim3(blocks), dim3(kPB), 0, stream, a,
                           in, out, s, k == 0 ? 1 : 0);
        double* t = in;
        in = out;
        out = t;
    }
    hipLaunchKernelGGL(HIP_KERNEL_NAME(k_pm_step<F, true>), dim3(blocks), dim3(kPB), 0, stream, a, in, out,
                       Step{0.0, 0.0}, 0);
    hipLaunchKernelGGL(k_pm_decide, dim3(1), dim3(kPB), 0, stream, a, blocks);
    return hipGetLastError();
}

}  // namespace

size_t pmass_sync_bytes() { return (size_t)(2 * kGroups * 32 + 2 * 32 + 64) * sizeof(unsigned); }

hipError_t launch_pmass(int N, int F, const double* coef, const int32_t* ecol, const double* c,
                        const double* vol, double* x0, double* x1, double* d, double* part, void* sync,
                        double tol, int maxit, long spin, double* out, p2m_report* rep, int** ok,
                        hipStream_t stream) {
    *ok = nullptr;
    // fields up to 3 share a row's entries; the residual of FP64 x cannot be asked below
    // its rounding, and a caller's iteration cap stays the CG's to honour
    const double k3 = log(4.0 / tol) / log(3.0);
    if (F > 3 || N < 1 || !(tol >= 4e-15) || k3 > (double)maxit) return hipSuccess;
    PmArgs a;
    a.N = N;
    a.F = F;
    a.K = (int)(k3 < 1.0 ? 1.0 : ceil(k3));
    a.coef = coef;
    a.ecol = ecol;
    a.c = c;
    a.vol = vol;
    a.x0 = x0;
    a.x1 = x1;
    a.d = d;
    a.part = part;
    a.tol = tol;
    a.out = out;
    a.rep = rep;
    unsigned* w = (unsigned*)sync;
    a.sy.ctr = w;
    a.sy.root = w + kGroups * 32;
    a.sy.rel = w + kGroups * 32 + 32;
    a.sy.abort = w + 2 * kGroups * 32 + 32;
    a.sy.part = nullptr;
    a.sy.tot = nullptr;
    a.sy.spin = spin;
    a.ok = (int*)(w + 2 * kGroups * 32 + 64);
    a.bad = a.ok + 32;
    hipLaunchKernelGGL(k_pm_clear, dim3(1), dim3(256), 0, stream, w, 2 * kGroups * 32 + 64, a.ok, a.bad);
    const int blocks = (N + kPB - 1) / kPB;
    hipError_t e = F == 1 ? run<1>(a, blocks, stream) : F == 2 ? run<2>(a, blocks, stream)
                                                               : run<3>(a, blocks, stream);
    *ok = a.ok;
    return e;
}

}  // namespace p2m
