// Lanczos recurrence on the device (paper: section "Exact diagonalizations",
// subsection "The Lanczos algorithm for the ground state", eqs. (Krylov),
// (LanczosRecursion), (tridiag)), in normalised form:
//   w = H v_n - beta_{n-1} v_{n-1};  alpha_n = <v_n, w>;  w -= alpha_n v_n;
//   beta_n = |w|;  v_{n+1} = w / beta_n          (beta_n^2 = paper's b_{n+1}^2)
//
// The engine runs nvec independent chains in one sector at once (vectors laid
// out consecutively), which is how the Green-function chains are batched.  A
// step is the three passes of lanczos_step.h.  Every dot product is a
// deterministic two-level sum (fixed blocks or chunks, then a fixed-order sum
// per chain), so results depend only on the inputs and the sector shape,
// never on launch timing or on other work sharing the GPU.
#include <math.h>

#include <string.h>

#include <algorithm>
#include <mutex>

#include "lanczos_step.h"

namespace qcm {

// ---------------------------------------------------------------- reductions

// partial[c][chunk] = sum over the chunk of x*y (vector c)
template <typename TX, typename TY>
__global__ void __launch_bounds__(256) k_dot_partial(const TX *__restrict__ x,
                                                     const TY *__restrict__ y, int64_t n,
                                                     int nchunks, double *__restrict__ partial) {
    __shared__ double sh[256];
    const int c = blockIdx.y;
    const int64_t base = (int64_t)blockIdx.x * kChunk;
    const TX *xc = x + (int64_t)c * n;
    const TY *yc = y + (int64_t)c * n;
    double acc = 0.0;
    for (int k = threadIdx.x; k < kChunk; k += 256) {
        int64_t i = base + k;
        if (i < n) acc = fma(ldd(xc + i), ldd(yc + i), acc);
    }
    double s = block_sum(acc, sh);
    if (threadIdx.x == 0) partial[(int64_t)c * nchunks + blockIdx.x] = s;
}

// Sum of the chunk partials of each chain.
// mode 2: out[c] = s (plain).
// mode 5: b0sq[c] = s, inv[c] = s > 0 ? 1/sqrt(s) : 0 (start-vector norm)
__global__ void __launch_bounds__(256) k_finish(const double *__restrict__ partial, int nchunks,
                                                int mode, ChainState cs, int n,
                                                double *__restrict__ out) {
    __shared__ double sh[256];
    const int c = blockIdx.x;
    double acc = 0.0;
    for (int k = threadIdx.x; k < nchunks; k += 256) acc += partial[(int64_t)c * nchunks + k];
    double s = block_sum(acc, sh);
    if (threadIdx.x != 0) return;
    (void)n;
    if (mode == 2) {
        out[c] = s;
    } else {
        cs.b0sq[c] = s;
        cs.inv[c] = s > 0.0 ? 1.0 / sqrt(s) : 0.0;
        if (!(s > 0.0)) {
            cs.done[c] = 1;
            cs.len[c] = 0;
        }
    }
}

// ---------------------------------------------------------------- vector updates

// x *= inv[c]
template <typename T>
__global__ void __launch_bounds__(256) k_scale(T *__restrict__ x, int64_t n_el, ChainState cs) {
    const int c = blockIdx.y;
    const double s = cs.inv[c];
    const int64_t off = (int64_t)c * n_el;
    const int64_t base = (int64_t)blockIdx.x * kChunk;
    for (int k = threadIdx.x; k < kChunk; k += 256) {
        int64_t i = base + k;
        if (i < n_el) st(x + off + i, ldd(x + off + i) * s);
    }
}

// psi += coef[n] * v  (psi FP64, one chain)
template <typename T>
__global__ void __launch_bounds__(256) k_accum(double *__restrict__ psi, const T *__restrict__ v,
                                               int64_t n_el, const double *__restrict__ coef,
                                               int n) {
    const double s = coef[n];
    const int64_t base = (int64_t)blockIdx.x * kChunk;
    for (int k = threadIdx.x; k < kChunk; k += 256) {
        int64_t i = base + k;
        if (i < n_el) psi[i] = fma(s, ldd(v + i), psi[i]);
    }
}

// SplitMix64 start vector, entry i = 2 (u_i >> 11) 2^-53 - 1 with
// u_i = mix(seed + (i+1) * golden gamma) (Steele, Lea & Flood 2014).
template <typename T>
__global__ void __launch_bounds__(256) k_splitmix(T *__restrict__ x, int64_t n, uint64_t seed) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint64_t z = seed + (uint64_t)(i + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    double u = (double)(z >> 11) * 0x1.0p-53;
    x[i] = (T)(2.0 * u - 1.0);
}

template <typename TI, typename TO>
__global__ void __launch_bounds__(256) k_convert(TO *__restrict__ o, const TI *__restrict__ in,
                                                 int64_t n) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) o[i] = (TO)in[i];
}

// partial sum of (w - theta psi)^2, FP64
__global__ void __launch_bounds__(256) k_resid_partial(const double *__restrict__ w,
                                                       const double *__restrict__ psi, double th,
                                                       int64_t n, int nchunks,
                                                       double *__restrict__ partial) {
    __shared__ double sh[256];
    const int64_t base = (int64_t)blockIdx.x * kChunk;
    double acc = 0.0;
    for (int k = threadIdx.x; k < kChunk; k += 256) {
        int64_t i = base + k;
        if (i < n) {
            double r = fma(-th, psi[i], w[i]);
            acc = fma(r, r, acc);
        }
    }
    double s = block_sum(acc, sh);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// ---------------------------------------------------------------- tridiagonal

// Ground-state test on T_M: theta_0, theta_1, the eigenvector s of theta_0
// (written to svec), and the residual estimate beta[M-1] |s[M-1]|.
__global__ void __launch_bounds__(256) k_tridiag_status(const double *__restrict__ alpha,
                                                        const double *__restrict__ beta, int M,
                                                        double tol, double *__restrict__ work,
                                                        double *__restrict__ svec,
                                                        GsStatus *status) {
    tridiag_status_block(alpha, beta, M, tol, work, svec, status, true);
}

// The tests between steps (no theta_1), each in two halves of about the same
// length that need not follow one another in one workgroup: workgroup 0 takes
// theta_0 of T_M (the next test's hint), workgroup 1 the residual estimate of
// the test before (T_Mv, theta_0 in *prev) and leaves its record, with whether
// the chain had stopped after step Mv - 1, in pinned host memory.  Mv = 0: no
// test before; M = 0: none after.
struct GsTest {
    GsStatus st;
    int32_t done, len;   // (len: steps recorded, when done)
};
__global__ void __launch_bounds__(256) k_tridiag_test(const double *__restrict__ alpha,
                                                      const double *__restrict__ beta, int M, int Mv,
                                                      double tol, double *work, double *work2,
                                                      double *svec, GsStatus *prev,
                                                      GsStatus *status, const int32_t *dlog,
                                                      const int32_t *len, GsTest *host) {
    if (blockIdx.x == 0) {
        if (M > 0) tridiag_theta_block(alpha, beta, M, work2, prev, status);
        return;
    }
    // (theta_0 of *prev is read by both workgroups, its estimate written here)
    tridiag_est_block(alpha, beta, Mv, tol, work, svec, prev);
    if (threadIdx.x == 0) {
        host->st = *prev;
        host->done = dlog[Mv - 1];
        host->len = *len;   // of a stopped chain: no later step changes it
    }
}

// A whole test in one workgroup (theta_0 of *prev as the hint), for tests several
// steps apart: its verdict does not wait for the next test's launch.
__global__ void __launch_bounds__(256) k_tridiag_whole(const double *__restrict__ alpha,
                                                       const double *__restrict__ beta, int M,
                                                       double tol, double *work, double *svec,
                                                       const GsStatus *prev, GsStatus *status,
                                                       const int32_t *dlog, const int32_t *len,
                                                       GsTest *host) {
    if (threadIdx.x == 0) *status = *prev;
    __syncthreads();
    tridiag_status_block(alpha, beta, M, tol, work, svec, status, false);
    if (threadIdx.x == 0) {
        host->st = *status;
        host->done = dlog[M - 1];
        host->len = *len;
    }
}

// psi_i = sum over n < M of svec[n] v_n[i] (FP64, in order of n) from kept
// vectors, vec elements apart
template <typename T>
__global__ void __launch_bounds__(256) k_psi(double *__restrict__ psi, const T *__restrict__ v,
                                             int64_t vec, int64_t n_el, int M,
                                             const double *__restrict__ svec) {
    const auto s = cp(svec);
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n_el; i += (int64_t)gridDim.x * 256) {
        const auto p = gp(v) + i;
        double acc = 0.0;
        int n = 0;
        for (; n + 8 <= M; n += 8) {
            T x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) x[u] = __builtin_nontemporal_load(p + (int64_t)(n + u) * vec);
#pragma unroll
            for (int u = 0; u < 8; ++u) acc = fma(s[n + u], (double)x[u], acc);
        }
        for (; n < M; ++n) acc = fma(s[n], (double)p[(int64_t)n * vec], acc);
        psi[i] = acc;
    }
}

// ---------------------------------------------------------------- side stream

struct SideRes {
    int dev = -1;
    hipStream_t s = nullptr;
    hipEvent_t ev[2 * SideLease::kEv + 2] = {};
    void *pinned = nullptr;
};
static std::mutex g_side_mu;
static std::vector<SideRes *> g_side_free;

int SideLease::lease() {
    int dev = -1;
    QCM_HIP(hipGetDevice(&dev));
    {
        std::lock_guard<std::mutex> lock(g_side_mu);
        for (size_t k = 0; k < g_side_free.size(); ++k)
            if (g_side_free[k]->dev == dev) {
                r = g_side_free[k];
                g_side_free.erase(g_side_free.begin() + k);
                break;
            }
    }
    if (!r) {
        SideRes *n = new SideRes();
        n->dev = dev;
        hipError_t e = hipStreamCreateWithFlags(&n->s, hipStreamNonBlocking);
        for (int k = 0; k < 2 * kEv + 2 && e == hipSuccess; ++k)
            e = hipEventCreateWithFlags(&n->ev[k], k < 2 * kEv ? hipEventDisableTiming
                                                               : hipEventDisableTiming |
                                                                     hipEventDisableSystemFence);
        if (e == hipSuccess) e = hipHostMalloc(&n->pinned, kSidePinned, hipHostMallocDefault);
        if (e != hipSuccess) {
            if (n->pinned) (void)hipHostFree(n->pinned);
            for (int k = 0; k < 2 * kEv + 2; ++k)
                if (n->ev[k]) (void)hipEventDestroy(n->ev[k]);
            if (n->s) (void)hipStreamDestroy(n->s);
            delete n;
            return fail(QCM_EHIP, "side stream: %s", hipGetErrorString(e));
        }
        r = n;
    }
    s = r->s;
    for (int k = 0; k < kEv; ++k) {
        ready[k] = r->ev[k];
        done[k] = r->ev[kEv + k];
    }
    for (int k = 0; k < 2; ++k) mark[k] = r->ev[2 * kEv + k];
    pinned = r->pinned;
    return QCM_OK;
}

SideLease::~SideLease() {
    if (!r) return;
    (void)hipStreamSynchronize(r->s);
    std::lock_guard<std::mutex> lock(g_side_mu);
    g_side_free.push_back(r);
}

// ---------------------------------------------------------------- engine

int engine_init(Engine &e, const HvOp &op, int prec, int nvec, int maxs, double btol, int reorth,
                Carver &cv) {
    e.op = op;
    e.prec = prec;
    e.nvec = nvec;
    e.dim = op.dim;
    e.maxs = maxs;
    e.reorth = reorth;
    size_t s = prec == QCM_FP64 ? 8 : 4;
    char *vecs = cv.take<char>(3 * s * (size_t)nvec * e.dim + 64);
    size_t vb = s * (size_t)nvec * e.dim;
    e.vbuf[0] = vecs;
    e.vbuf[1] = vecs + vb;
    e.vbuf[2] = vecs + 2 * vb;
    e.nchunks = (int)ceil_div(e.dim, kChunk);
    if (e.nchunks < 1) e.nchunks = 1;
    row_shape(op.up.d, op.dn.d, prec, &e.rows, &e.nblk);
    e.rg = side_rows(op.up.d, e.rows, prec);
    e.wgs = (int32_t)((e.nblk + e.rg - 1) / e.rg);
    e.fused = !op.split && !op.csr.rowptr && op.up.d < 65536 &&
              fused_lds(op.up.d, e.rows, prec, op.md.nbytes, op.md.u_uniform,
                        2 * op.md.nbond) <= kFusedLds;
    // alpha partials: per fused-product block, per row-mixing workgroup when
    // the step's first pass rides on the two-pass product, else per chunk
    e.na = e.fused ? e.nblk : (op.split ? (int32_t)split_pa_count(op) : e.nchunks);
    e.partial = cv.take<double>((size_t)nvec * e.nchunks);
    int64_t npa = e.nblk > e.nchunks ? e.nblk : e.nchunks;
    if (e.na > npa) npa = e.na;
    // five partial arrays (alpha and the norm dots of the fused or two-pass
    // product)
    e.pa = cv.take<double>((size_t)nvec * npa * 5);
    // norm partials, or the two-pass step's per-range dot sums
    e.pn = cv.take<double>((size_t)nvec * std::max<size_t>(3 * (size_t)e.nchunks, 5 * kDotBlocks));
    e.cs.maxs = maxs;
    e.cs.btol = btol;
    e.cs.alpha = cv.take<double>((size_t)nvec * maxs);
    e.cs.beta = cv.take<double>((size_t)nvec * maxs);
    double *sc = cv.take<double>((size_t)nvec * 7);
    e.cs.amax = sc;
    e.cs.inv = sc + nvec;
    e.cs.corr = sc + 2 * nvec;
    e.cs.corr2 = sc + 3 * nvec;
    e.cs.b0sq = sc + 4 * nvec;
    e.scratch = sc + 5 * nvec;
    e.cs.apre = sc + 6 * nvec;
    int32_t *ic = cv.take<int32_t>((size_t)nvec * 3);
    e.cs.len = ic;
    e.cs.done = ic + nvec;
    e.cs.renorm = ic + 2 * nvec;
    e.cs.dlog = cv.take<int32_t>(maxs);
    e.cs.stop = nullptr;
    e.ivp = 0;
    e.iv = 1;
    e.iw = 2;
    e.lazy = 0;
    e.pending = 0;
    e.vpold = nullptr;
    return QCM_OK;
}

int engine_reset(Engine &e, hipStream_t s) {
    QCM_HIP(hipMemsetAsync(e.cs.alpha, 0, sizeof(double) * e.nvec * e.maxs, s));
    QCM_HIP(hipMemsetAsync(e.cs.beta, 0, sizeof(double) * e.nvec * e.maxs, s));
    QCM_HIP(hipMemsetAsync(e.cs.amax, 0, sizeof(double) * e.nvec * 7, s));
    QCM_HIP(hipMemsetAsync(e.cs.len, 0, sizeof(int32_t) * e.nvec * 3, s));
    size_t sz = (e.prec == QCM_FP64 ? 8 : 4) * (size_t)e.nvec * e.dim;
    e.ivp = 0;
    e.iv = 1;
    e.iw = 2;
    e.pending = 0;
    QCM_HIP(hipMemsetAsync(e.vbuf[e.ivp], 0, sz, s));
    return QCM_OK;
}

void group_tables(const HvOp &op, BGroup *g) {
    g->d_up = op.up.d;
    g->d_dn = op.dn.d;
    g->dim = op.dim;
    g->su = op.up.states;
    g->sd = op.dn.states;
    g->eu = op.hu.ediag;
    g->ed = op.hd.ediag;
    g->nhu = op.hu.nh;
    g->nhd = op.hd.nh;
    g->cold = op.hd.col;
    g->cfd = op.hd.coef;
    g->wu = (op.hu.width + 3) / 4 * 4;   // slots of the packed list
    g->wd = op.hd.width;
    g->dslot = op.hd.rowmajor != 1;
    g->ulut = op.md.ulut;
    g->pku = op.hu.pk;
    g->ctab = op.md.ctab;
    g->nctab = 2 * op.md.nbond;
    g->t_uniform = op.md.t_is_uniform && op.md.nbond > 0;
    g->u_uniform = op.md.u_uniform;
    g->nbytes = op.md.nbytes;
}

BGroup engine_group(const Engine &e, int n) {
    BGroup g;
    memset(&g, 0, sizeof g);
    group_tables(e.op, &g);
    g.dim = e.dim;
    g.rg = e.rg;
    g.wgs = e.wgs;
    g.rows = e.rows;
    g.nblk = e.nblk;
    g.nvec = e.nvec;
    g.nchunks = e.nchunks;
    g.na = e.na;
    g.n = n;
    g.reorth = e.reorth;
    g.vp = e.vbuf[e.ivp];
    g.v = e.vbuf[e.iv];
    g.w = e.vbuf[e.iw];
    g.pa = e.pa;
    g.pstride = (int64_t)e.nvec * e.na;
    g.pn = e.pn;
    g.psi = nullptr;
    g.svec = nullptr;
    g.cs = e.cs;
    return g;
}

template <typename T>
static int step_t(Engine &e, int n, hipStream_t s) {
    const OneSrc src{engine_group(e, n)};
    const unsigned nk = (unsigned)e.nvec * e.nchunks;
    if (e.fused) {
        hv_step_launch<T>(src, (int64_t)e.nvec * e.wgs,
                          hv_lds(e.op.up.d, e.rows, e.rg, e.prec, e.op.md.nbytes,
                                 e.op.md.u_uniform, 2 * e.op.md.nbond),
                          s);
    } else if (e.op.split) {
        // the first pass (w -= beta' vp, partial <v, w>) inside the row-mixing
        // pass; a deferred update of the previous step inside the in-row pass
        SubPrev sp;
        sp.vp = e.vbuf[e.ivp];
        sp.beta = e.cs.beta;
        sp.maxs = e.cs.maxs;
        sp.n = n;
        sp.pa = e.pa;
        sp.pstride = (int64_t)e.nvec * e.na;
        sp.reorth = e.reorth;
        LazyUpd lz;
        if (e.pending) {
            // after the rotation: v_n is in ivp, v_{n-1} in iw (where W goes) or vpold
            lz.vold = e.vbuf[e.ivp];
            lz.vpold = e.vpold ? e.vpold : e.vbuf[e.iw];
            lz.apre = e.cs.apre;
            lz.corr = e.cs.corr;
            lz.corr2 = e.cs.corr2;
            lz.inv = e.cs.inv;
            lz.reorth = e.reorth;
        }
        QCM_TRY(hv_split_launch_sub(e.op, e.prec, e.vbuf[e.iv], e.vbuf[e.iw], e.nvec, sp,
                                    e.pending ? &lz : nullptr, s));
        e.pending = 0;
        // alpha, then beta from the product's dots: no norm pass
        ks_dots_stage<OneSrc><<<dim3(kDotBlocks, (unsigned)e.nvec), 256, 0, s>>>(src);
        ks_finish_dots<OneSrc><<<e.nvec, kDotBlocks, 0, s>>>(src);
        // chains whose beta the dots cannot resolve take the direct norm
        ks_norm<T, OneSrc><<<nk, 256, 0, s>>>(src, 1);
        ks_finish<OneSrc><<<e.nvec, 256, 0, s>>>(src, 4);
    } else {
        QCM_TRY(hv_launch(e.op, e.prec, e.vbuf[e.iv], e.vbuf[e.iw], e.nvec, s));
        ks_sub_prev<T, OneSrc><<<nk, 256, 0, s>>>(src);
    }
    if (e.fused) {
        // alpha and beta from the fused product's dots; the direct norm pass
        // only for chains whose beta the dots cannot resolve
        ks_finish_fused<T, OneSrc><<<e.nvec * finish_parts(e.nchunks), 256, 0, s>>>(src);
        if (e.nchunks > kFinishChunks) {
            ks_norm<T, OneSrc><<<nk, 256, 0, s>>>(src, 1);
            ks_finish<OneSrc><<<e.nvec, 256, 0, s>>>(src, 4);
        }
    } else if (!e.op.split) {
        ks_finish<OneSrc><<<e.nvec, 256, 0, s>>>(src, 0);
        ks_norm<T, OneSrc><<<nk, 256, 0, s>>>(src, 0);
        ks_finish<OneSrc><<<e.nvec, 256, 0, s>>>(src, 1);
    }
    if (e.op.split && e.lazy)
        e.pending = 1;   // the next step's in-row pass forms v_{n+1}
    else
        update_launch<T>(src, nk, s);
    QCM_LAUNCH_CHECK();
    // rotate: v_{n-1} <- v_n, v_n <- the new vector, next w <- old v_{n-1}
    int t = e.ivp;
    e.ivp = e.iv;
    e.iv = e.iw;
    e.iw = t;
    return QCM_OK;
}

int engine_step(Engine &e, int n, hipStream_t s) {
    if (e.prec == QCM_FP64) return step_t<double>(e, n, s);
    return step_t<float>(e, n, s);
}

// Coefficients of n steps from normalised start vectors, in one launch where
// the sector fits (*ran), by LDS and by the sums' layout: one norm chunk, at
// most 64 product blocks.  The vectors are left as they were.
int engine_run_chains(Engine &e, int n, int *ran, hipStream_t s) {
    *ran = 0;
    const HvOp &op = e.op;
    if (!e.fused || !op.hu.pk || e.nchunks != 1 || e.nblk > 64 || hv_one(op.up.d, e.rows)) return QCM_OK;
    const OneSrc src{engine_group(e, 0)};
    const int nlut = op.md.u_uniform >= 0.0 ? 0 : op.md.nbytes * 256;
    const size_t lds = chain_lds(op.up.d, op.dn.d, src.g.wu, (src.g.wd + 3) & ~3, src.g.nctab, nlut,
                                 e.reorth ? 5 : 3, e.nblk, e.prec == QCM_FP64 ? 8 : 4)
                           .bytes;
    if (lds > 158 * 1024) return QCM_OK;   // 160 KB less the kernel's own few words
    if (e.prec == QCM_FP64)
        ks_chain<double><<<e.nvec, kChainThreads, lds, s>>>(src, n);
    else
        ks_chain<float><<<e.nvec, kChainThreads, lds, s>>>(src, n);
    QCM_LAUNCH_CHECK();
    *ran = 1;
    return QCM_OK;
}

// The deferred update as its own pass (the update pass of the step before the
// rotation: w was its w, v its v, vp its vp).
template <typename T>
static int settle_t(Engine &e, hipStream_t s) {
    BGroup g = engine_group(e, 0);
    g.vp = e.vpold ? e.vpold : e.vbuf[e.iw];
    g.v = e.vbuf[e.ivp];
    g.w = e.vbuf[e.iv];
    const OneSrc src{g};
    update_launch<T>(src, (int64_t)e.nvec * e.nchunks, s);
    QCM_LAUNCH_CHECK();
    return QCM_OK;
}

int engine_settle(Engine &e, hipStream_t s) {
    if (!e.pending) return QCM_OK;
    e.pending = 0;
    if (e.prec == QCM_FP64) return settle_t<double>(e, s);
    return settle_t<float>(e, s);
}

// Normalise the current vectors v (chain start vectors), storing b0sq.
template <typename T>
static int normalize_t(Engine &e, hipStream_t s) {
    e.pending = 0;
    T *v = (T *)e.vbuf[e.iv];
    const dim3 g((unsigned)e.nchunks, (unsigned)e.nvec);
    k_dot_partial<T, T><<<g, 256, 0, s>>>(v, v, e.dim, e.nchunks, e.partial);
    k_finish<<<e.nvec, 256, 0, s>>>(e.partial, e.nchunks, 5, e.cs, 0, nullptr);
    k_scale<T><<<g, 256, 0, s>>>(v, e.dim, e.cs);
    QCM_LAUNCH_CHECK();
    return QCM_OK;
}

int engine_normalize(Engine &e, hipStream_t s) {
    if (e.prec == QCM_FP64) return normalize_t<double>(e, s);
    return normalize_t<float>(e, s);
}

int engine_seed(Engine &e, uint64_t seed, const void *v0, hipStream_t s) {
    e.pending = 0;
    void *v = e.vbuf[e.iv];
    size_t sz = (e.prec == QCM_FP64 ? 8 : 4) * (size_t)e.dim;
    if (v0) {
        QCM_HIP(hipMemcpyAsync(v, v0, sz, hipMemcpyDeviceToDevice, s));
    } else if (e.prec == QCM_FP64) {
        k_splitmix<double><<<ceil_div(e.dim, 256), 256, 0, s>>>((double *)v, e.dim, seed);
    } else {
        k_splitmix<float><<<ceil_div(e.dim, 256), 256, 0, s>>>((float *)v, e.dim, seed);
    }
    QCM_LAUNCH_CHECK();
    return QCM_OK;
}

int engine_accum(Engine &e, double *psi, const double *coef, int n, hipStream_t s) {
    QCM_TRY(engine_settle(e, s));
    const unsigned g = (unsigned)e.nchunks;
    if (e.prec == QCM_FP64)
        k_accum<double><<<g, 256, 0, s>>>(psi, (const double *)e.vbuf[e.iv], e.dim, coef, n);
    else
        k_accum<float><<<g, 256, 0, s>>>(psi, (const float *)e.vbuf[e.iv], e.dim, coef, n);
    QCM_LAUNCH_CHECK();
    return QCM_OK;
}

int tridiag_status(const double *alpha, const double *beta, int M, double tol, double *work,
                   double *svec, GsStatus *status, hipStream_t s) {
    k_tridiag_status<<<1, 256, 0, s>>>(alpha, beta, M, tol, work, svec, status);
    QCM_LAUNCH_CHECK();
    return QCM_OK;
}

// psi /= |psi| (FP64), through the chain state of chain 0 of e.
int psi_finalize(Engine &e, double *psi, hipStream_t s) {
    const int64_t dim = e.dim;
    int nch = (int)ceil_div(dim, kChunk);
    k_dot_partial<double, double><<<dim3(nch, 1), 256, 0, s>>>(psi, psi, dim, nch, e.partial);
    ChainState cs1 = e.cs;
    k_finish<<<1, 256, 0, s>>>(e.partial, nch, 5, cs1, 0, nullptr);
    k_scale<double><<<dim3(nch, 1), 256, 0, s>>>(psi, dim, cs1);
    QCM_LAUNCH_CHECK();
    return QCM_OK;
}

int residual_norm(const HvOp &op, const double *psi, double theta, double *w64, double *partial,
                  double *out, hipStream_t s) {
    QCM_TRY(hv_launch(op, QCM_FP64, psi, w64, 1, s));
    int nch = (int)ceil_div(op.dim, kChunk);
    k_resid_partial<<<nch, 256, 0, s>>>(w64, psi, theta, op.dim, nch, partial);
    ChainState dummy{};
    k_finish<<<1, 256, 0, s>>>(partial, nch, 2, dummy, 0, out);
    QCM_LAUNCH_CHECK();
    return QCM_OK;
}

}  // namespace qcm

using namespace qcm;

extern "C" void qcm_lanczos_default_opts(qcm_lanczos_opts *o) {
    if (!o) return;
    o->max_iter = 600;
    o->fixed_steps = 0;
    o->want_vector = 1;
    o->reorth = 0;
    o->prec = QCM_FP64;
    o->check_every = 1;
    o->tol = 1e-12;
    o->btol = 1e-13;
    o->seed = 1;
    o->d_v0 = nullptr;
}

namespace qcm {

int gs_run(const char *fn, const GsSetup &setup, int64_t dim, const qcm_lanczos_opts *o,
           double *h_alpha, double *h_beta, void *d_gs, qcm_gs_result *h_out, void *d_ws,
           size_t ws_bytes, size_t *ws_needed, void *stream) {
    if (!ws_needed || !o) return fail(QCM_EARG, "%s: NULL ws_needed or opts", fn);
    if (o->prec != QCM_FP64 && o->prec != QCM_FP32V)
        return fail(QCM_EARG, "%s: bad prec %d", fn, o->prec);
    if (o->max_iter < 1 && o->fixed_steps < 1)
        return fail(QCM_EARG, "%s: max_iter and fixed_steps both < 1", fn);
    if (o->want_vector && !d_gs && d_ws) return fail(QCM_EARG, "%s: want_vector needs d_gs", fn);
    if (dim < 1) return fail(QCM_EARG, "%s: empty sector", fn);
    const int limit = o->fixed_steps > 0 ? o->fixed_steps : o->max_iter;
    const int every = o->check_every > 0 ? o->check_every : 1;
    constexpr int kTests = SideLease::kEv;
    // the workspace is laid out by one function, run first without a base to
    // size it (no launch) and then on the workspace
    HvOp op;
    Engine e;
    double *svec = nullptr, *work = nullptr, *dscal = nullptr;
    GsStatus *status = nullptr;
    auto layout = [&](Carver &cv, hipStream_t st) -> int {
        QCM_TRY(setup(cv, st, &op));
        QCM_TRY(engine_init(e, op, o->prec, 1, limit, o->btol, o->reorth, cv));
        svec = cv.take<double>(limit);
        work = cv.take<double>((size_t)limit * 6);
        status = cv.take<GsStatus>(kTests);
        dscal = cv.take<double>(64);
        return QCM_OK;
    };
    Carver dry(nullptr);
    QCM_TRY(layout(dry, nullptr));
    const size_t need = dry.off + 256;
    *ws_needed = need;
    if (!d_ws) return QCM_OK;
    if (!h_out) return fail(QCM_EARG, "%s: h_out is NULL", fn);
    if (ws_bytes < need) return fail(QCM_EWORKSPACE, "%s: workspace %zu < %zu", fn, ws_bytes, need);
    hipStream_t s = as_stream(stream);
    Carver cv(d_ws);
    QCM_TRY(layout(cv, s));

    // Workspace beyond what is needed keeps the first pass's vectors v_0, v_1,
    // ..., so that the ground-state vector is summed from them instead of
    // running the recurrence again (12 orbitals, 72 steps: 4 ms of 26).
    const size_t vb = ((o->prec == QCM_FP64 ? 8 : 4) * (size_t)dim + 255) / 256 * 256;
    const size_t at = (cv.off + 255) / 256 * 256;
    int nkeep = 0;
    if (o->want_vector && d_gs && ws_bytes > at)
        nkeep = (int)std::min<size_t>((ws_bytes - at) / vb, (size_t)limit + 1);
    if (nkeep < 4) nkeep = 0;
    char *const keep = (char *)d_ws + at;
    // (a caller may have put its own vectors past what the call needs)
    auto within = [&](const void *p, size_t bytes) {
        return p && (const char *)p < keep + nkeep * vb && keep < (const char *)p + bytes;
    };
    if (within(d_gs, sizeof(double) * (size_t)dim) ||
        within(o->d_v0, (o->prec == QCM_FP64 ? 8 : 4) * (size_t)dim))
        nkeep = 0;
    void *const ring[3] = {e.vbuf[0], e.vbuf[1], e.vbuf[2]};
    auto slot = [&](int n) -> void * { return n < nkeep ? keep + (size_t)n * vb : ring[n % 3]; };
    // v_n is in slot(n); the product of step n goes where v_{n+1} will be.  The
    // ring's three buffers hold whatever comes after the kept vectors.
    auto aim = [&](int n) {
        e.vpold = e.vbuf[e.iw];
        e.vbuf[e.iw] = slot(n + 1);
    };

    // first pass: coefficients; the status starts empty (M = 0: no hint for
    // the first test, as in the batched engine)
    QCM_HIP(hipMemsetAsync(status, 0, kTests * sizeof(GsStatus), s));
    QCM_TRY(engine_reset(e, s));
    if (nkeep) e.vbuf[e.iv] = slot(0);
    QCM_TRY(engine_seed(e, o->seed, o->d_v0, s));
    QCM_TRY(engine_normalize(e, s));
    // the first pass needs the coefficients only: updates may be deferred
    e.lazy = 1;
    GsStatus hs{};
    int M = 0, conv = 0, brk = 0;
    // The tests run on a side stream beside the steps, some of which are
    // enqueued past a test whose verdict is not known yet: such a step is wasted
    // if the verdict ends the recurrence, but changes nothing (its coefficients
    // are not read).  Test t is launch t and has status record t mod kTests.
    // Tests after every step, or faster than whole ones can be taken: launch t
    // takes its theta_0 and, side by side, test t - 1's estimate, and two tests'
    // steps run ahead.  Tests further apart: launch t is the whole test, and as
    // many steps run ahead as take about that long, so that neither the steps
    // wait for it nor many are wasted (with the estimate left to the next launch,
    // 20 steps apart, up to 40 were: 14 orbitals (7,7) 59.8 -> 52.5 ms; tests 2
    // steps apart, 12 orbitals, whole 4.65 ms, pairs 4.39; 10 apart up to step
    // 1,000, whole 55 ms, pairs 37).  The times are those measured: a whole test
    // 45 us at 30 steps, 100 at 140, a step 25 us at 0.85 M states, 3.3 ms at 166 M.
    const double step_us = 20.0 + 20e-6 * (double)dim;
    auto ahead_of = [&](int Mt) { return (int)ceil((30.0 + 0.5 * Mt) / step_us); };
    SideLease side;
    QCM_TRY(side.lease());
    // With fixed steps there are no tests, but a chain that stops early (its
    // later steps are zero vectors, which its length leaves out) should not be
    // carried on for long: the finishing kernels leave its length in pinned
    // memory, where the host looks each time the steps up to the mark before the
    // last one are done.  A step or more is then always queued behind the
    // running one, so that the look costs nothing (a stream synchronisation each
    // step costs 15 us; one every 64 steps ran up to 63 steps past the end).  A
    // mark takes the stream 1 to 2 us, so short steps (under about 0.3 ms) have
    // one every second time to start with, and every eighth later.
    volatile int32_t *const stopped = (int32_t *)side.pinned;
    struct Drain {   // the steps in flight write to the leased memory
        hipStream_t s;
        bool on;
        ~Drain() {
            if (on) (void)hipStreamSynchronize(s);
        }
    } drain{s, o->fixed_steps > 0};
    int nmark = 0;
    if (o->fixed_steps > 0) {
        *stopped = 0;
        e.cs.stop = (int32_t *)side.pinned;
    }
    int ntest = 0, seen = 0, nlaunch = 0, tm[kTests] = {0};
    bool stop = false, pair[kTests] = {false};
    auto launch_test = [&](int Mt) -> int {
        const int k = nlaunch % kTests, kp = (nlaunch + kTests - 1) % kTests;
        QCM_HIP(hipEventRecord(side.ready[k], s));
        QCM_HIP(hipStreamWaitEvent(side.s, side.ready[k], 0));
        // (from whole tests to pairs only: ahead_of grows with the steps)
        const bool prev = nlaunch > 0 && pair[kp];
        pair[k] = prev || every == 1 || every <= ahead_of(Mt);
        if (pair[k])
            k_tridiag_test<<<prev ? 2 : 1, 256, 0, side.s>>>(
                e.cs.alpha, e.cs.beta, Mt, prev ? tm[kp] : 0, o->tol, work,
                work + 5 * (size_t)limit, svec, status + kp, status + k, e.cs.dlog, e.cs.len,
                (GsTest *)side.pinned + kp);
        else
            k_tridiag_whole<<<1, 256, 0, side.s>>>(e.cs.alpha, e.cs.beta, Mt, o->tol, work, svec,
                                                  status + kp, status + k, e.cs.dlog, e.cs.len,
                                                  (GsTest *)side.pinned + k);
        QCM_LAUNCH_CHECK();
        QCM_HIP(hipEventRecord(side.done[k], side.s));
        tm[k] = Mt;
        ++nlaunch;
        if (Mt > 0) ++ntest;
        return QCM_OK;
    };
    // the verdicts of the tests in order, until one ends the recurrence: those up
    // to t are waited for, later ones (of whole tests) taken if they are there
    auto verdicts = [&](int t) -> int {
        for (; seen < ntest && !stop; ++seen) {
            const bool p = pair[seen % kTests];
            if (seen > t && p) break;
            const hipEvent_t ev = side.done[(seen + (p ? 1 : 0)) % kTests];   // its verdict's launch
            // a short poll (it answers sooner: 1 % of a ground state of 12 orbitals),
            // then the runtime's own wait, which blocks or spins as the program chose
            hipError_t q = hipEventQuery(ev);
            for (int k = 0; k < 300 && q == hipErrorNotReady && seen <= t; ++k) q = hipEventQuery(ev);
            if (q == hipErrorNotReady && seen <= t) q = hipEventSynchronize(ev);
            if (q == hipErrorNotReady) break;
            QCM_HIP(q);
            const GsTest *g = (const GsTest *)side.pinned + seen % kTests;
            hs = g->st;
            M = hs.M;
            if (g->done) {
                // the chain stopped at len; steps after it carry zero vectors
                M = g->len;
                brk = conv = 1;
                stop = true;
            } else if (hs.converged) {
                conv = 1;
                stop = true;
            }
        }
        return QCM_OK;
    };
    for (int n = 0; n < limit && !stop; ++n) {
        if (nkeep) aim(n);
        QCM_TRY(engine_step(e, n, s));
        const bool last = n + 1 == limit, check = (n + 1) % every == 0 || last;
        if (o->fixed_steps > 0) {
            if (last) {
                QCM_HIP(hipStreamSynchronize(s));
            } else if ((n + 1) % (dim >= (1 << 24) ? 1 : n < 16 ? 2 : 8) == 0) {
                QCM_HIP(hipEventRecord(side.mark[nmark % 2], s));
                if (nmark++ > 0) QCM_HIP(hipEventSynchronize(side.mark[nmark % 2]));
            }
            M = n + 1;
            if (*stopped) {
                M = *stopped - 1;
                brk = conv = 1;
                stop = true;
            }
            continue;
        }
        if (check) QCM_TRY(launch_test(n + 1));
        if (last) {
            if (pair[(nlaunch - 1) % kTests]) QCM_TRY(launch_test(0));
            QCM_TRY(verdicts(ntest - 1));
        } else {
            // waited for: of pairs the last but two, of whole tests those as many
            // steps back as may run ahead
            int t = std::max(seen, ntest - 2);
            while (t < ntest && !pair[t % kTests] &&
                   tm[t % kTests] <= n + 1 - ahead_of(tm[t % kTests]))
                ++t;
            QCM_TRY(verdicts(t - 1));
        }
    }
    e.cs.stop = nullptr;
    // the record of the test that ended the recurrence (its theta_0 is the hint)
    GsStatus *const fin = status + (seen > 0 ? (seen - 1) % kTests : 0);
    if (nlaunch > 0) QCM_HIP(hipStreamWaitEvent(s, side.done[(nlaunch - 1) % kTests], 0));
    QCM_TRY(tridiag_status(e.cs.alpha, e.cs.beta, M, o->tol, work, svec, fin, s));
    QCM_HIP(hipMemcpyAsync(&hs, fin, sizeof hs, hipMemcpyDeviceToHost, s));
    QCM_HIP(hipStreamSynchronize(s));
    if (o->fixed_steps <= 0 && !brk) conv = hs.converged;

    qcm_gs_result r{};
    r.e0 = hs.theta0;
    r.residual_est = hs.est;
    r.theta1 = hs.theta1;
    r.n_iter = M;
    r.converged = conv;
    r.breakdown = brk;
    r.degenerate_suspect = degenerate_suspect(hs.theta0, hs.theta1);
    r.true_residual = -1.0;

    // the coefficients of the first pass go out before the second pass reruns
    // (and rewrites, with identical values) the recurrence
    if (h_alpha) QCM_HIP(hipMemcpy(h_alpha, e.cs.alpha, sizeof(double) * M, hipMemcpyDeviceToHost));
    if (h_beta) QCM_HIP(hipMemcpy(h_beta, e.cs.beta, sizeof(double) * M, hipMemcpyDeviceToHost));

    if (o->want_vector && d_gs) {
        // psi = sum_n s_n v_n: over the kept vectors, then (second pass) over
        // those of the identical recurrence, run again from where they end or
        // from the start
        double *psi = (double *)d_gs;
        e.lazy = 0;
        e.pending = 0;
        const int have = std::min(nkeep, M);
        if (have) {
            const unsigned g = (unsigned)std::min<size_t>(ceil_div((size_t)dim, 256), 1 << 23);
            const int64_t el = (int64_t)(vb / (o->prec == QCM_FP64 ? 8 : 4));
            if (o->prec == QCM_FP64)
                k_psi<double><<<g, 256, 0, s>>>(psi, (const double *)keep, el, dim, have, svec);
            else
                k_psi<float><<<g, 256, 0, s>>>(psi, (const float *)keep, el, dim, have, svec);
            QCM_LAUNCH_CHECK();
            if (have < M) {
                // from v_{have-2}, v_{have-1}: no step before M - 1 stopped
                // the chain, so its flags start clear
                QCM_HIP(hipMemsetAsync(e.cs.amax, 0, sizeof(double), s));
                QCM_HIP(hipMemsetAsync(e.cs.done, 0, sizeof(int32_t), s));
                e.ivp = 0;
                e.iv = 1;
                e.iw = 2;
                e.vbuf[0] = slot(have - 2);
                e.vbuf[1] = slot(have - 1);
                e.vbuf[2] = ring[have % 3];
                e.vpold = nullptr;
                for (int n = have - 1; n + 1 < M; ++n) {
                    e.vbuf[e.iw] = ring[(n + 1) % 3];
                    QCM_TRY(engine_step(e, n, s));
                    QCM_TRY(engine_accum(e, psi, svec, n + 1, s));
                }
            }
        } else {
            QCM_HIP(hipMemsetAsync(psi, 0, sizeof(double) * dim, s));
            QCM_TRY(engine_reset(e, s));
            QCM_TRY(engine_seed(e, o->seed, o->d_v0, s));
            QCM_TRY(engine_normalize(e, s));
            for (int n = 0; n < M; ++n) {
                QCM_TRY(engine_accum(e, psi, svec, n, s));
                if (n + 1 < M) QCM_TRY(engine_step(e, n, s));
            }
        }
        e.vbuf[0] = ring[0];
        e.vbuf[1] = ring[1];
        e.vbuf[2] = ring[2];
        // normalise psi and take the true residual, all FP64
        QCM_TRY(psi_finalize(e, psi, s));
        double *w64 = (double *)e.vbuf[0];  // 8*dim bytes: the first two FP32 or one FP64 vector
        QCM_TRY(residual_norm(op, psi, hs.theta0, w64, e.partial, dscal, s));
        double r2 = 0.0;
        QCM_HIP(hipMemcpyAsync(&r2, dscal, sizeof r2, hipMemcpyDeviceToHost, s));
        QCM_HIP(hipStreamSynchronize(s));
        r.true_residual = sqrt(r2);
    }
    *h_out = r;
    return QCM_OK;
}

}  // namespace qcm

extern "C" int qcm_lanczos_gs(const qcm_model *m, const qcm_basis *b, const qcm_lanczos_opts *o,
                              double *h_alpha, double *h_beta, void *d_gs, qcm_gs_result *h_out,
                              void *d_ws, size_t ws_bytes, size_t *ws_needed, void *stream) {
    if (!ws_needed || !o) return fail(QCM_EARG, "qcm_lanczos_gs: NULL ws_needed or opts");
    QCM_TRY(validate_model(m));
    QCM_TRY(check_basis(b, m->L));
    auto setup = [&](Carver &cv, hipStream_t st, HvOp *op) -> int {
        return hv_setup(m, b, cv, op, st);
    };
    return gs_run("qcm_lanczos_gs", setup, b->dim, o, h_alpha, h_beta, d_gs, h_out, d_ws,
                  ws_bytes, ws_needed, stream);
}

namespace qcm {

// Normalise the start vectors from norm partials already in e.partial.
int engine_normalize_from_partials(Engine &e, hipStream_t s) {
    e.pending = 0;
    const dim3 g((unsigned)e.nchunks, (unsigned)e.nvec);
    k_finish<<<e.nvec, 256, 0, s>>>(e.partial, e.nchunks, 5, e.cs, 0, nullptr);
    if (e.prec == QCM_FP64)
        k_scale<double><<<g, 256, 0, s>>>((double *)e.vbuf[e.iv], e.dim, e.cs);
    else
        k_scale<float><<<g, 256, 0, s>>>((float *)e.vbuf[e.iv], e.dim, e.cs);
    QCM_LAUNCH_CHECK();
    return QCM_OK;
}

}  // namespace qcm
