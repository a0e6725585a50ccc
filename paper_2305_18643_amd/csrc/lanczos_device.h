// Device helpers shared by the single-solve and the batched Lanczos kernels
// (internal).  Both paths call exactly these functions, so a chain gives the
// same bits whichever path runs it.
#pragma once

#include <math.h>

#include <type_traits>

#include "lanczos_engine.h"

namespace qcm {

// LDS written by a wave's lanes is read by its others
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// x of lane l (wave-uniform)
__device__ __forceinline__ int64_t wave_read(int64_t x, int l) {
    return (int64_t)(uint32_t)__builtin_amdgcn_readlane((int)x, l) |
           ((int64_t)__builtin_amdgcn_readlane((int)(x >> 32), l) << 32);
}

template <typename T>
__device__ __forceinline__ double ldd(const T *p) {
    return (double)*p;
}

// Vectors and tables live in global memory, but a pointer read from a group
// table in memory (the batched engine) is generic to the compiler, which then
// emits flat accesses: those also count against the LDS counter, so every LDS
// wait waits for them too.  Cast to the global address space, the same
// accesses become global loads and stores.
template <typename T>
using gptr = __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ gptr<T> gp(T *p) {
    return (gptr<T>)p;
}
// Tables read with a wave-uniform index: through the constant address space
// they become scalar loads.
template <typename T>
using cptr = __attribute__((address_space(4))) const T *;
template <typename T>
__device__ __forceinline__ cptr<T> cp(const T *p) {
    return (cptr<T>)p;
}
template <typename T>
__device__ __forceinline__ double ldd(gptr<const T> p) {
    return (double)*p;
}
template <typename T>
__device__ __forceinline__ double ldd(gptr<T> p) {
    return (double)*p;
}

__device__ __forceinline__ double block_sum(double x, double *sh) {
    // 256 threads, fixed tree
    const int t = threadIdx.x;
    sh[t] = x;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (t < s) sh[t] += sh[t + s];
        __syncthreads();
    }
    double r = sh[0];
    __syncthreads();
    return r;
}

template <typename T>
__device__ __forceinline__ void st(T *p, double x) {
    *p = (T)x;
}

// One step of the Sturm sequence from (pm, pmm) = (p_{i-1}, p_{i-2}): counts
// the sign change and rescales the pair by a power of two when p_i leaves
// [2^-256, 2^256] (exact); a vanishing p_i becomes -2^-700 p_{i-1}.
__host__ __device__ inline void sturm_step(double ax, double bi, double &pm, double &pmm, int &cnt) {
    double p = fma(-bi, pmm, ax * pm);
    p = p == 0.0 ? -0x1p-700 * pm : p;
    cnt += (p < 0.0) != (pm < 0.0);
    const int e = ilogb(p);
    const int k = (e > 256 || e < -256) ? -e : 0;
    pmm = ldexp(pm, k);
    pm = ldexp(p, k);
}

__host__ __device__ inline uint32_t hi_word(double x) {
    uint64_t b;
    __builtin_memcpy(&b, &x, 8);
    return (uint32_t)(b >> 32);
}

// number of eigenvalues of T_M below x: the sign changes of the Sturm
// sequence p_i = (a_i - x) p_{i-1} - b_{i-1}^2 p_{i-2} (p_{-1} = 1, p_{-2} = 0),
// i.e. the negative pivots q_i = p_i / p_{i-1} of the LDL^T of T_M - x, counted
// without a division.  The pair (p_i, p_{i-1}) is rescaled by a power of two
// whenever p_i leaves [2^-256, 2^256] (exact), and a vanishing p_i becomes
// -2^-700 p_{i-1} (a pivot of -2^-700, so an eigenvalue at x counts as below
// it).  |p_{i-1}| lies in [2^-256, 2^256] there, so the replacement is a
// normal number and the rescale that follows brings the pair back into range
// (a replacement that underflowed to -0 would lose this and every later sign
// change).  b2[i] = b[i]^2.  Callable on the host too (for tests).
// Eight steps at a time are taken without the rescale, which is exact wherever
// it falls, so the count is the same: the chain of a step is then a product
// and an fma instead of seven dependent operations.  Where one of the eight
// leaves [2^-400, 2^400] (or vanishes) they are taken again one by one.
__host__ __device__ inline int sturm_below(int M, const double *__restrict__ a,
                                           const double *__restrict__ b2, double x) {
    constexpr int U = 8;
    int cnt = 0;
    double pm = 1.0, pmm = 0.0;
    int i = 0;
    double bp = 0.0;   // b_{i-1}^2
    for (; i + U <= M; i += U) {
        double p[U], c[U];
        uint32_t lo = 0xffffffffu, hi = 0, sg = hi_word(pm) >> 31;
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = b2[i + u];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double pa = u == 0 ? pm : p[u - 1], pb = u == 0 ? pmm : u == 1 ? pm : p[u - 2];
            p[u] = fma(-(u == 0 ? bp : c[u - 1]), pb, (a[i + u] - x) * pa);
            const uint32_t h = hi_word(p[u]), m = h & 0x7fffffffu;
            lo = m < lo ? m : lo;
            hi = m > hi ? m : hi;
            sg = (sg << 1) | (h >> 31);
        }
        if (lo >= (623u << 20) && hi < (1423u << 20)) {
#if defined(__HIP_DEVICE_COMPILE__)
            cnt += __popc((sg ^ (sg >> 1)) & 0xffu);
#else
            cnt += __builtin_popcount((sg ^ (sg >> 1)) & 0xffu);
#endif
            const int e = (int)((hi_word(p[U - 1]) >> 20) & 0x7ffu) - 1023;
            const int k = (e > 256 || e < -256) ? -e : 0;
            pmm = ldexp(p[U - 2], k);
            pm = ldexp(p[U - 1], k);
        } else {
#pragma unroll 1
            for (int u = 0; u < U; ++u) {
                sturm_step(a[i + u] - x, bp, pm, pmm, cnt);
                bp = b2[i + u];
            }
        }
        bp = c[U - 1];
    }
#pragma unroll 1
    for (; i < M; ++i) {
        sturm_step(a[i] - x, bp, pm, pmm, cnt);
        bp = b2[i];
    }
    return cnt;
}

// k-th smallest eigenvalue by 256-way multisection: every thread tests one
// point of the current bracket; 10 rounds narrow it by 257^10.  b2 = b^2.
// hint (k = 0 only): the lowest eigenvalue of a leading block of T, which
// can only lie above that of T; once a Sturm count confirms an eigenvalue
// below it (plus 1e-12 relative) it becomes the upper end, and the first
// round then spaces its points geometrically toward that end, where the
// eigenvalue of a converging recurrence lies.  Any hint is safe: one that
// the count does not confirm is ignored.  (The confirming count is taken
// beside the first round's counts.)
__device__ inline double tridiag_kth(int M, const double *a, const double *b, const double *b2,
                                     int k, double hint = NAN) {
    const int t = threadIdx.x;
    __shared__ double mn[4], mx[4];
    __shared__ int firsts[4];
    // Gershgorin bounds
    double lo0 = a[0], hi0 = a[0];
    for (int i = t; i < M; i += 256) {
        const double r = (i > 0 ? fabs(b[i - 1]) : 0.0) + (i < M - 1 ? fabs(b[i]) : 0.0);
        lo0 = fmin(lo0, a[i] - r);
        hi0 = fmax(hi0, a[i] + r);
    }
    for (int o = 32; o > 0; o >>= 1) {
        lo0 = fmin(lo0, __shfl_xor(lo0, o));
        hi0 = fmax(hi0, __shfl_xor(hi0, o));
    }
    if ((t & 63) == 0) {
        mn[t >> 6] = lo0;
        mx[t >> 6] = hi0;
    }
    __syncthreads();
    lo0 = fmin(fmin(mn[0], mn[1]), fmin(mn[2], mn[3]));
    hi0 = fmax(fmax(mx[0], mx[1]), fmax(mx[2], mx[3]));
    const double pad = 1e-12 * fmax(1.0, fmax(fabs(lo0), fabs(hi0)));
    double lo = lo0 - pad, hi = hi0 + pad;
    // the first point of the round with more than k eigenvalues below it (a
    // minimum, so the result does not rest on the counts being monotone)
    auto first_of = [&](int cnt) -> int {
        const unsigned long long m = __ballot(cnt > k);
        __syncthreads();
        if ((t & 63) == 0) firsts[t >> 6] = m ? (t & ~63) + __ffsll(m) - 1 : 256;
        __syncthreads();
        return min(min(firsts[0], firsts[1]), min(firsts[2], firsts[3]));
    };
    int round = 0;
    if (k == 0 && isfinite(hint)) {
        const double up = hint + 1e-12 * fmax(1.0, fabs(hint));
        if (up > lo && up < hi) {
            // point j of this round: up - (up - lo) 2^(-53 (j + 1) / 256)
            auto point = [&](int j) -> double {
                return up - (up - lo) * exp2(-53.0 * (double)(j + 1) / 256.0);
            };
            const bool go = up - lo > 4e-16 * fmax(fabs(lo), fabs(up));
            const int cu = sturm_below(M, a, b2, up);
            const int c = go ? sturm_below(M, a, b2, point(t)) : 0;
            if (cu > 0) {
                if (go) {
                    const int j = first_of(c);
                    const double nlo = j == 0 ? lo : point(j - 1);
                    hi = j == 256 ? up : point(j);
                    lo = nlo;
                } else {
                    hi = up;
                }
                round = go ? 1 : 10;
            }
        }
    }
    for (; round < 10; ++round) {
        // stop once the bracket is at the resolution of its end points
        if (!(hi - lo > 4e-16 * fmax(fabs(lo), fabs(hi)))) break;
        // uniform points
        auto point = [&](int j) -> double { return lo + (hi - lo) * (double)(j + 1) / 257.0; };
        const int j = first_of(sturm_below(M, a, b2, point(t)));
        const double nlo = j == 0 ? lo : point(j - 1);
        const double nhi = j == 256 ? hi : point(j);
        lo = nlo;
        hi = nhi;
    }
    return 0.5 * (lo + hi);
}

// Eigenvector for theta by inverse iteration: T - theta factored once by
// Gaussian elimination with row pivoting on the tridiagonal (multipliers in
// dl, swaps flagged in piv, reciprocal pivots in d, superdiagonals du, du2),
// then three solves in place on x, each normalised.  One wave calls it; the
// recurrences are every lane's (all lanes hold the same values, lane 0
// stores), eight rows at a time: the rows' operands are loaded together ahead
// of the chain, which would otherwise wait on a load per row.
__device__ inline void tridiag_vector(int M, const double *__restrict__ a, const double *__restrict__ b,
                                      double theta, double *x, double *d, double *du, double *du2,
                                      double *dl, double *piv) {
    const int lane = threadIdx.x & 63;
    typedef std::integral_constant<int, 8> Eight;
    typedef std::integral_constant<int, 1> One;
    double scale = 1.0;
    for (int i = lane; i < M; i += 64) scale = fmax(scale, fabs(a[i]));
    for (int o = 32; o > 0; o >>= 1) scale = fmax(scale, __shfl_xor(scale, o));
    const double tiny = 1e-15 * scale;
    auto wave_sync = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };
    // rows 0 .. n-1 in order, eight at a time
    auto rows = [](int n, auto &&f) {
        int i = 0;
        for (; i + 8 <= n; i += 8) f(i, Eight{});
        for (; i < n; ++i) f(i, One{});
    };
    // factorisation, the current row (di, dui) and the next one carried in
    // registers: row i is [di, dui, 0], row i+1 is [b_i, dn, dun]
    double di = a[0] - theta, dui = M > 1 ? b[0] : 0.0;
    rows(M - 1, [&](int i0, auto n_) {
        constexpr int U = decltype(n_)::value;
        double an[U], bn[U + 1], o[5][U];
#pragma unroll
        for (int u = 0; u < U; ++u) an[u] = a[i0 + u + 1];
#pragma unroll
        for (int u = 0; u < U; ++u) bn[u] = b[i0 + u];
        bn[U] = i0 + U < M - 1 ? b[i0 + U] : 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            double dli = bn[u];
            double dn = an[u] - theta;
            double dun = bn[u + 1];
            double du2i = 0.0;
            const bool sw = fabs(dli) > fabs(di);
            const double t0 = di, t1 = dui;
            di = sw ? dli : di;
            dli = sw ? t0 : dli;
            dui = sw ? dn : dui;
            dn = sw ? t1 : dn;
            du2i = sw ? dun : du2i;
            dun = sw ? 0.0 : dun;
            di = di == 0.0 ? tiny : di;
            const double inv = 1.0 / di;
            const double m = dli * inv;
            o[0][u] = inv;
            o[1][u] = dui;
            o[2][u] = du2i;
            o[3][u] = m;
            o[4][u] = sw ? 1.0 : 0.0;
            dn = fma(-m, dui, dn);
            dun = fma(-m, du2i, dun);
            di = dn;
            dui = dun;
        }
        if (lane == 0)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                d[i0 + u] = o[0][u];
                du[i0 + u] = o[1][u];
                du2[i0 + u] = o[2][u];
                dl[i0 + u] = o[3][u];
                piv[i0 + u] = o[4][u];
            }
    });
    if (di == 0.0) di = tiny;
    if (lane == 0) {
        d[M - 1] = 1.0 / di;
        du[M - 1] = du2[M - 1] = 0.0;
    }
    for (int i = lane; i < M; i += 64) x[i] = 1.0;
    wave_sync();
    for (int it = 0; it < 3; ++it) {
        // forward: the row swaps and multipliers, x_i carried
        double cur = x[0];
        rows(M - 1, [&](int i0, auto n_) {
            constexpr int U = decltype(n_)::value;
            double nx[U], pv[U], dm[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                nx[u] = x[i0 + u + 1];
                pv[u] = piv[i0 + u];
                dm[u] = dl[i0 + u];
            }
            double o[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool sw = pv[u] != 0.0;
                const double lo = sw ? nx[u] : cur, hi = sw ? cur : nx[u];
                o[u] = lo;
                cur = fma(-dm[u], lo, hi);
            }
            wave_sync();
            if (lane == 0)
#pragma unroll
                for (int u = 0; u < U; ++u) x[i0 + u] = o[u];
        });
        if (lane == 0) x[M - 1] = cur;
        wave_sync();
        // back substitution, x_{i+1} and x_{i+2} carried
        double x1 = 0.0, x2 = 0.0;
        rows(M, [&](int j0, auto n_) {
            constexpr int U = decltype(n_)::value;
            const int i0 = M - 1 - j0;   // rows i0, i0 - 1, ...
            double xs[U], u1[U], u2[U], dd[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                xs[u] = x[i0 - u];
                u1[u] = du[i0 - u];
                u2[u] = du2[i0 - u];
                dd[u] = d[i0 - u];
            }
            double o[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                double s = xs[u];
                if (j0 + u > 0) s = fma(-u1[u], x1, s);
                if (j0 + u > 1) s = fma(-u2[u], x2, s);
                const double xi = s * dd[u];
                o[u] = xi;
                x2 = x1;
                x1 = xi;
            }
            wave_sync();
            if (lane == 0)
#pragma unroll
                for (int u = 0; u < U; ++u) x[i0 - u] = o[u];
        });
        wave_sync();
        double nr = 0.0;
        rows(M, [&](int i0, auto n_) {
            constexpr int U = decltype(n_)::value;
            double xs[U];
#pragma unroll
            for (int u = 0; u < U; ++u) xs[u] = x[i0 + u];
#pragma unroll
            for (int u = 0; u < U; ++u) nr = fma(xs[u], xs[u], nr);
        });
        nr = 1.0 / sqrt(nr);
        for (int i = lane; i < M; i += 64) x[i] *= nr;
        wave_sync();
    }
    if (x[0] < 0.0) {
        wave_sync();
        for (int i = lane; i < M; i += 64) x[i] = -x[i];
    }
    wave_sync();
}

// Largest T_M whose coefficients and inverse-iteration arrays are staged in
// LDS by the ground-state test (every Sturm step and every elimination step
// then reads LDS instead of waiting on a cache round trip).
constexpr int kTriLds = 640;

__device__ __forceinline__ void tridiag_verdict(double bM, double xM, double tol, GsStatus *status) {
    const double est = bM * fabs(xM);
    status->est = est;
    status->converged = est <= tol * fmax(1.0, fabs(status->theta0)) ? 1 : 0;
}

// The test is a serial chain of FP64 operations (about 20 cycles each): what
// it costs is the length of that chain, not work.  Measured on T_M of a
// 12-orbital sector, M = 72: multisection 78 k cycles before the eight-step
// Sturm groups, 46 k now; inverse iteration 139 k cycles with a load, a store
// and a branch per row on the chain, 59 k now (94 -> 46 us in all; 126 us when
// every access was a flat one).
// The ground-state test of one workgroup (256 threads) on T_M: theta_0,
// theta_1 (only when want1; the convergence test does not need it, so the
// tests between steps skip it and the final one takes it), the eigenvector
// of theta_0 in svec, residual estimate beta[M-1] |s[M-1]| and the
// convergence flag, written to *status (which holds the previous test's
// result before).  Up to kTriLds steps the work happens
// in LDS; longer T_M use `work` (5 M doubles) and beta^2 in work + 5 M (M
// doubles).
__device__ inline void tridiag_status_block(const double *__restrict__ alpha,
                                            const double *__restrict__ beta, int M, double tol,
                                            double *__restrict__ work, double *__restrict__ svec,
                                            GsStatus *status, bool want1) {
    __shared__ double la[kTriLds], lb[kTriLds], lb2[kTriLds], lx[kTriLds], lw[5 * kTriLds];
    // (written out for LDS and for global memory: through one pointer to either
    // every access would be a flat one)
    auto test = [&](const double *a, const double *b, const double *b2, double *x, double *w, int S) {
        __syncthreads();
        // the previous test's theta_0 (of T_{M'}, M' <= M) as the hint
        const double hint = (status->M >= 1 && status->M <= M) ? status->theta0 : NAN;
        __syncthreads();
        double th0 = tridiag_kth(M, a, b, b2, 0, hint);
        double th1 = (want1 && M > 1) ? tridiag_kth(M, a, b, b2, 1) : NAN;
        if (threadIdx.x < 64) tridiag_vector(M, a, b, th0, x, w, w + S, w + 2 * S, w + 3 * S, w + 4 * S);
        if (threadIdx.x == 0) {
            status->theta0 = th0;
            status->theta1 = th1;
            status->M = M;
            tridiag_verdict(beta[M - 1], x[M - 1], tol, status);
        }
    };
    if (M <= kTriLds) {
        for (int i = threadIdx.x; i < M; i += blockDim.x) {
            la[i] = alpha[i];
            lb[i] = beta[i];
            lb2[i] = beta[i] * beta[i];
        }
        test(la, lb, lb2, lx, lw, kTriLds);
        __syncthreads();
        for (int i = threadIdx.x; i < M; i += blockDim.x) svec[i] = lx[i];
    } else {
        double *b2 = work + 5 * (size_t)M;
        for (int i = threadIdx.x; i < M; i += blockDim.x) b2[i] = beta[i] * beta[i];
        test(alpha, beta, b2, svec, work, M);
    }
}

// The same test as two independent parts, each one workgroup's: theta_0 of
// T_M into *status (from *prev, the previous test's record, as the hint) ...
__device__ inline void tridiag_theta_block(const double *__restrict__ alpha,
                                           const double *__restrict__ beta, int M,
                                           double *__restrict__ work, const GsStatus *prev,
                                           GsStatus *status) {
    __shared__ double la[kTriLds], lb[kTriLds], lb2[kTriLds];
    const double hint = (prev->M >= 1 && prev->M <= M) ? prev->theta0 : NAN;
    double th0;
    if (M <= kTriLds) {
        for (int i = threadIdx.x; i < M; i += blockDim.x) {
            la[i] = alpha[i];
            lb[i] = beta[i];
            lb2[i] = beta[i] * beta[i];
        }
        __syncthreads();
        th0 = tridiag_kth(M, la, lb, lb2, 0, hint);
    } else {
        for (int i = threadIdx.x; i < M; i += blockDim.x) work[i] = beta[i] * beta[i];
        __syncthreads();
        th0 = tridiag_kth(M, alpha, beta, work, 0, hint);
    }
    if (threadIdx.x == 0) {
        status->theta0 = th0;
        status->theta1 = NAN;
        status->M = M;
    }
}
// ... and the residual estimate of a T_M whose theta_0 stands in *status
// (work: 5 M doubles, svec: M, used where T_M does not fit LDS).
__device__ inline void tridiag_est_block(const double *__restrict__ alpha,
                                         const double *__restrict__ beta, int M, double tol,
                                         double *__restrict__ work, double *__restrict__ svec,
                                         GsStatus *status) {
    __shared__ double la[kTriLds], lb[kTriLds], lx[kTriLds], lw[5 * kTriLds];
    if (threadIdx.x >= 64) return;
    const double th0 = status->theta0;
    auto est = [&](const double *a, const double *b, double *x, double *w, int S) {
        tridiag_vector(M, a, b, th0, x, w, w + S, w + 2 * S, w + 3 * S, w + 4 * S);
        if (threadIdx.x == 0) tridiag_verdict(beta[M - 1], x[M - 1], tol, status);
    };
    if (M <= kTriLds) {
        for (int i = threadIdx.x; i < M; i += 64) {
            la[i] = alpha[i];
            lb[i] = beta[i];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        est(la, lb, lx, lw, kTriLds);
    } else {
        est(alpha, beta, svec, work, M);
    }
}

struct cplx {
    double re, im;
};

// One continued fraction at z, bottom floor first.  part 0 (electron):
// b0sq / (z + E0 - a0 - b1^2/(z + E0 - a1 - ...)); part 1 (hole):
// b0sq / (z - E0 + a0 - b1^2/(z - E0 + a1 - ...)).
__device__ inline cplx cf_value(const double *__restrict__ co, int len, int maxs, cplx z, double e0,
                         int part) {
    cplx r{0.0, 0.0};
    if (len <= 0 || co[0] == 0.0) return r;
    const double sg = part == 0 ? 1.0 : -1.0;
    const double zr = part == 0 ? z.re + e0 : z.re - e0;
    const double zi = z.im;
    const double *a = co + 1, *b2 = co + 1 + maxs;
    double gr = zr - sg * a[len - 1], gi = zi;
    for (int n = len - 2; n >= 0; --n) {
        double den = gr * gr + gi * gi;
        double qr = b2[n] * gr / den, qi = -b2[n] * gi / den;  // b2 / g
        gr = zr - sg * a[n] - qr;
        gi = zi - qi;
    }
    double den = gr * gr + gi * gi;
    r.re = co[0] * gr / den;
    r.im = -co[0] * gi / den;
    return r;
}

}  // namespace qcm
