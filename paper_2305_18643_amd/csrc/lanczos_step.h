// One Lanczos step of a group of chains, as three passes over the vectors
// (internal; used by the single-solve engine and by the batched engine).
//
// A group is nvec chains in one sector (vectors [nvec][dim], consecutive).
// With v = v_n, vp = v_{n-1}, beta' = beta_{n-1}:
//   pass 1  w = H v - beta' vp, stored; partial sums of <v, w>
//           (fused into the product when rows of V fit in LDS, with the dots
//           <w, w>, <v, v> (<vp, w>, <vp, v>) that then replace pass 2;
//           otherwise the product runs first and a chunked pass subtracts and
//           sums);
//   finish  alpha_n = <v, w>;
//   pass 2  x = w - alpha_n v (not stored): partial sums of |x|^2 and, with
//           local reorthogonalisation, of <v, x> and <vp, x> (after the
//           two-pass product these come from dots its last pass already
//           summed, and this pass is skipped);
//   finish  c1 = <v, x>, c2 = <vp, x>; alpha_n += c1;
//           beta_n^2 = |x|^2 - c1^2 - c2^2 (the norm of x - c1 v - c2 vp for
//           unit v, vp orthogonal to each other, up to terms of order c^2 eps);
//   pass 3  v_{n+1} = (x - c1 v - c2 vp) / beta_n, rounded once to the storage
//           type (optionally also psi += s_n v_n for the ground-state replay).
// After the fused product one launch finishes a step: ks_finish_fused, which also
// takes the direct norm of pass 2 for short vectors where the dots cancel (longer
// ones: ks_norm and ks_finish).  The continued-fraction chains of a sector that
// fits LDS run all their steps in one launch (ks_chain), with the same sums.
// After the two-pass product the two finishes are ks_dots_stage and
// ks_finish_dots, and pass 3 may be deferred into the next step's in-row
// pass, which forms v_{n+1} element by element with the same operations when
// it stages a row.
// Every sum is a fixed-order two-level reduction (per block or per chunk of
// kChunk elements, then per chain), so results depend only on the inputs and
// the sector shape, not on the launch or on other groups sharing it.
#pragma once

#include <algorithm>
#include <type_traits>

#include "lanczos_device.h"

namespace qcm {

// Elements of V a product block stages in LDS (at least one whole row).
constexpr int64_t kTileElems = 2048;
// LDS a fused product block may use (row tile + lookup tables).
constexpr size_t kFusedLds = 144 * 1024;

// Vectors above this many bytes are taken one chain at a time by all XCDs, each
// a contiguous range of rows; smaller ones stay on one XCD each (its 4 MB L2).
constexpr int64_t kXcdChain = (int64_t)4 << 20;

// Everything a step kernel needs about one group.
struct BGroup {
    // sector and Hamiltonian (fused product)
    int64_t d_up, d_dn, dim;
    const uint32_t *su, *sd;
    const double *eu, *ed;
    const int32_t *nhu, *nhd, *cold;
    const double *cfd;     // down hops, row by row (hop s of row i at i * wd + s) or dslot
    const double *ulut;
    const uint32_t *pku;   // packed up hops (HopTables::pk)
    const double *ctab;    // hop coefficients by index (+-t_ab)
    double u_uniform;
    int32_t nbytes;
    int32_t nctab;
    int32_t wu, wd;    // widths of the hop lists
    int32_t dslot;     // down hops slot by slot: hop s of row i at s * d_dn + i
    int32_t rg;        // rows a product workgroup takes side by side (hv_one; else 1)
    int32_t wgs;       // product workgroups per vector
    int32_t t_uniform; // every bond has the same t (a coefficient is +-ctab[0])
    int32_t rows;      // rows of V per product block
    int32_t nblk;      // product blocks per vector
    int32_t nvec, nchunks;
    int32_t na;        // alpha partials per vector (nblk when fused, else nchunks)
    int64_t pstride;   // two-pass product: stride between its five partial arrays
    int32_t n;         // step index
    int32_t reorth;
    const void *vp, *v;
    void *w;
    double *pa;        // [nvec][na]
    double *pn;        // [nvec][3][nchunks]
    double *psi;       // ground-state replay: psi += svec[n] v_n in pass 3 (or NULL)
    const double *svec;
    ChainState cs;
};

__device__ __forceinline__ int find_group(const int64_t *__restrict__ begin, int ng, int64_t x) {
    int lo = 0, hi = ng - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (cp(begin)[mid] <= x)
            lo = mid;
        else
            hi = mid - 1;
    }
    return lo;
}

// Work sources: many groups through a table and prefix sums of their work
// items, or one group passed by value.
struct TabSrc {
    const BGroup *G;
    const int64_t *begin;
    int ng;
    int64_t base = 0;   // work item of workgroup 0
    __device__ __forceinline__ const BGroup &at(int64_t x, int64_t *local) const {
        x += base;
        const int g = find_group(begin, ng, x);
        *local = x - cp(begin)[g];
        return *(const BGroup *)cp(G + g);   // through the constant space: scalar loads
    }
};
struct OneSrc {
    BGroup g;
    int64_t base = 0;   // work item of workgroup 0
    __device__ __forceinline__ const BGroup &at(int64_t x, int64_t *local) const {
        *local = x + base;
        return g;
    }
};

// Launches of work items in slices: a launch takes fewer than 2^32 threads.
template <class Src, class F>
inline void each_slice(const Src &all, int64_t items, int64_t threads, F &&launch) {
    const int64_t most = 0xffffffffll / threads;
    if (items <= most) return launch(all, (unsigned)items);
    Src src = all;
    for (int64_t left = items; left > 0; left -= most, src.base += most)
        launch(src, (unsigned)std::min(left, most));
}

inline void row_shape(int64_t d_up, int64_t d_dn, int prec, int32_t *rows, int32_t *nblk) {
    (void)prec;
    int64_t r = kTileElems / (d_up > 0 ? d_up : 1);
    if (r < 1) r = 1;
    if (r > d_dn) r = d_dn;
    if (r < 1) r = 1;
    *rows = (int32_t)r;
    *nblk = (int32_t)((d_dn + r - 1) / r);
}

// LDS of a fused product block as its sector's path is decided: rows plus
// lookup tables.
inline size_t fused_lds(int64_t d_up, int32_t rows, int prec, int nbytes, double u_uniform,
                        int nctab) {
    const size_t lut = u_uniform >= 0.0 ? 0 : sizeof(double) * 256 * (size_t)nbytes;
    return lut + sizeof(double) * (size_t)nctab +
           (prec == QCM_FP64 ? 8 : 4) * (size_t)rows * (size_t)d_up;
}

constexpr int kSide = 2;

// Sectors of rows so long that a product block is one row (a sector with a
// single short row counts with the short ones).
inline bool hv_one(int64_t d_up, int32_t rows) { return rows == 1 && d_up > kTileElems / 2; }

// Rows of a one-row-per-block sector that a product workgroup takes side by
// side: their hop entries, coefficients and up-string data are then read once
// for all of them.  Bounded by LDS, so that two workgroups share a CU.
inline int32_t side_rows(int64_t d_up, int32_t rows, int prec) {
    if (!hv_one(d_up, rows)) return 1;
    const int64_t row = (d_up + 1) * (prec == QCM_FP64 ? 8 : 4);
    return kSide * row <= 64 * 1024 ? kSide : 1;
}

// How a product workgroup deals out its elements: tiles of 64 lanes along the
// rows, of a block of several rows or of one row per block, or, for rows too
// short for that, pairs of elements (one column of two rows) one after another.
// The line between the two for blocks of several rows: along rows of 45 the
// tiles leave more than half their lanes idle and the pairs are 1.02 to 1.4
// times as fast (10 orbitals (2,5), FP64 all-to-all hopping to FP32 chain); at
// 55 they are 0.88 to 1.2 times as fast, since each lane then loads its own
// down-hop lists.
enum { kHvRows = 0, kHvOne = 1, kHvShort = 2 };
constexpr int kShortRow = 48;
// The layout of the down-hop lists of a sector with one up string: slot by slot,
// as a lane has a row of its own and consecutive lanes then read side by side.
// Row by row each lane streams its own list, of which the L2 keeps nothing once
// the lists of the waves in flight exceed it (24 orbitals (0,12), 2,704,156 rows:
// a product 447 us row by row, 152 slot by slot).  Rows of more strings share a
// list, and slot by slot lose as often as they gain.
inline int dn_layout(int64_t d_up) { return d_up == 1 ? 2 : 1; }
inline int hv_form(int64_t d_up, int32_t rows) {
    return hv_one(d_up, rows) ? kHvOne : d_up <= kShortRow ? kHvShort : kHvRows;
}

// LDS of a product workgroup: lookup tables, the rows (interleaved in sets of
// rg, or kSide for blocks of several rows, each set with a zero slot), and for
// blocks of several rows the products awaiting the dots.
inline size_t hv_lds(int64_t d_up, int32_t rows, int32_t rg, int prec, int nbytes, double u_uniform,
                     int nctab) {
    const size_t s = prec == QCM_FP64 ? 8 : 4;
    const size_t lut = u_uniform >= 0.0 ? 0 : sizeof(double) * 256 * (size_t)nbytes;
    size_t t = (lut + sizeof(double) * (size_t)nctab + 15) & ~(size_t)15;
    const size_t dots = rg * 5 * 256 * sizeof(double);
    if (hv_one(d_up, rows)) return t + std::max(dots, s * (size_t)rg * (size_t)(d_up + 1));
    const size_t sets = (size_t)(rows + kSide - 1) / kSide;
    return t + std::max(dots, s * sets * kSide * (size_t)(d_up + 1) + s * (size_t)rows * (size_t)d_up);
}

// The group of chains of an engine at step n (vectors from its rotation).
BGroup engine_group(const Engine &e, int n);
// the sector and Hamiltonian fields of a group
void group_tables(const HvOp &op, BGroup *g);

// Workgroup x of n, renumbered so that each XCD (x mod 8) takes a contiguous
// range.
__device__ __forceinline__ int64_t xcd_chunk(int64_t x, int64_t n) {
    const int64_t k = x & 7, e = n >> 3, r = n & 7;
    return k * e + (k < r ? k : r) + (x >> 3);
}

// A wave-uniform value whose origin the compiler no longer sees: what derives
// from it (products, comparisons held as lane masks, loads through it) is
// formed where it is used instead of being kept in scalar registers, and
// spilled, over a loop.
template <typename X>
__device__ __forceinline__ X afresh(X x) {
    if constexpr (sizeof(X) == 4) {
        int y = __builtin_amdgcn_readfirstlane((int)x);
        asm volatile("" : "+s"(y));
        return (X)y;
    } else {
        const uint64_t b = (uint64_t)x;
        uint64_t y = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)b) |
                     (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(b >> 32)) << 32;
        asm volatile("" : "+s"(y));
        return (X)y;
    }
}

template <typename T, int RG>
struct alignas(sizeof(T) * RG) RowSet {
    T x[RG];
};
// adjacent columns of a row, aligned as one
template <typename T, int CW>
struct Cols {
    T x[CW];
};
template <typename C, typename P>
__device__ __forceinline__ C ld_cols(P p) {
    C c;
#pragma unroll
    for (int k = 0; k < (int)(sizeof(C) / sizeof(c.x[0])); ++k) c.x[k] = p[k];
    return c;
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void *p, int64_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes, 0x00020000);
}
template <typename T>
__device__ __forceinline__ T buf_load(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
    if constexpr (sizeof(T) == 16)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
    else if constexpr (sizeof(T) == 8)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
    else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
typedef int i32x4_t __attribute__((ext_vector_type(4), aligned(4)));
typedef double f64x4_t __attribute__((ext_vector_type(4), aligned(8)));

// pass 1, fused: w = H v - beta' vp for rows of V held in LDS.
//
// A wave takes 64 lanes x CW adjacent columns of RG rows at a time.  The rows
// lie interleaved in LDS ([column][row]), so one hop entry, one coefficient
// and one LDS gather serve RG rows, and one neighbour address serves CW
// columns.  The in-row loop runs to the largest hop count of the tile's
// strings (wave-uniform, no masking; groups of four): entries past a string's
// own hops read a zero slot after the row.  Row-mixing lists are wave-uniform
// (scalar loads of four columns and coefficients); the neighbours of a row's
// first eight hops and of its last one to three are in flight together for
// all RG rows.
//
// What bounds it: instruction issue and latency first (the earlier form, one
// element per thread with hop counts per lane, ran at 65 Gelements/s whatever
// the size or storage type, 142 VALU and 107 SALU instructions per 64
// elements; a variant whose neighbours all came from L2 ran no faster), then,
// for FP64 rows of 14 orbitals, the traffic of the neighbour rows between L2
// and memory.  Measured, the kernel alone on the same vectors again: 14-site
// chain (7,7) FP64 183 -> 102 us (a call between others 200 -> 116), ten chains
// of its (7,6) sector in FP32 1119 -> 566 us; 12-site ladder (6,6) FP64 40 -> 11.4
// us; ten vectors of a 10-orbital impurity in FP32 21 -> 9.4 us.
// Kept out: four rows side by side, neighbours loaded before the in-row hops
// (loads return in order, so the entries then wait for them; and the
// registers cost more in occupancy than the overlap gains in FP32).
//
// Sum order per element: diagonal, up hops in list order, down hops in list
// order, then -beta' vp; all FP64, rounded once.  pa != NULL: partial <v, w>,
// <w, w>, <v, v> (<vp, w>, <vp, v>) per block of q.rows rows, summed as 256
// threads taking the block's elements in turn, so that they do not depend on
// how the tiles are dealt out.
// FORM kHvOne: sectors of one row per block, q.rg blocks per workgroup (their
// products are read back for the dots); otherwise one block of several rows per
// workgroup, in sets of kSide (products kept in LDS for the dots).
constexpr int kHvThreads = 512;

// Waves per SIMD the product is compiled for, and adjacent columns per lane in
// blocks of several rows.  One group (a single solve): two columns, which
// halve the scalar work and the loads per element (3x4 (6,6) product 13.8 ->
// 11.7 us, 10 chains of 8 orbitals 11.4 -> 9.6 us); a batched round mixes
// short and long rows and is faster with one column and as many waves as fit
// (24 solves of 6 to 12 orbitals: 101 ms against 115).
template <typename T, class S, int FORM>
constexpr int hv_waves() {
    return FORM == kHvOne     ? (sizeof(T) == 8 ? 4 : 5)
           : FORM == kHvShort ? 6
                              : (std::is_same<S, OneSrc>::value ? 4 : 8);
}

// With two columns per lane and an odd row length d the last lane redoes column
// d - 2, with the hop count of its own tile, and stores it as the lane before
// does.  In a row of 128 k + 1 columns that lane would be in a tile of its own,
// whose hop count may be less than that column needs (which is in the tile before);
// no sector has such rows.
constexpr bool hv_rows_fit_pairs() {
    for (int L = 1; L <= 32; ++L)
        for (int N = 0; N <= L; ++N) {
            int64_t d = 1;
            for (int i = 1; i <= N; ++i) d = d * (L - N + i) / i;
            if (d > 1 && d < 65536 && d % 128 == 1) return false;
        }
    return true;
}
static_assert(hv_rows_fit_pairs(), "a row of 128 k + 1 columns: its last lane stores another tile's column");

template <typename T, class Src, int FORM, bool BIG>
__global__ void __launch_bounds__(kHvThreads, (hv_waves<T, Src, FORM>())) ks_hv(Src src) {
    constexpr bool ONE = FORM == kHvOne;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    int64_t local;
    const BGroup &q = src.at(blockIdx.x, &local);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int NT = FORM == kHvShort ? (int)blockDim.x : kHvThreads, NW = NT / 64;
    const int du = (int)q.d_up;
    const int64_t d_up = q.d_up, d_dn = q.d_dn;
    int64_t vec, wg;
    if (q.dim * (int64_t)sizeof(T) > kXcdChain) {
        // one chain at a time, each XCD a contiguous range of its rows
        vec = local / q.wgs;
        wg = xcd_chunk(local - vec * q.wgs, q.wgs);
    } else {
        // each XCD its own chains
        local = xcd_chunk(local, (int64_t)q.wgs * q.nvec);
        vec = local / q.wgs;
        wg = local - vec * q.wgs;
    }
    const int nlut = q.u_uniform >= 0.0 ? 0 : q.nbytes * 256;
    double *lut = reinterpret_cast<double *>(smem_raw);
    double *ct = lut + nlut;
    T *tile = reinterpret_cast<T *>(smem_raw + ((8 * (size_t)(nlut + q.nctab) + 15) & ~(size_t)15));
    // the partials of the dots, in the place of the rows once these are done
    double *sh = reinterpret_cast<double *>(tile);
    const auto v = gp((const T *)q.v) + vec * q.dim;
    const int sub = q.n > 0 && q.pa;
    const bool reo = q.reorth, dots = q.pa != nullptr;
    const double b = sub ? q.cs.beta[vec * q.cs.maxs + q.n - 1] : 0.0;
    for (int k = tid; k < nlut; k += NT) lut[k] = gp(q.ulut)[k];
    for (int k = tid; k < q.nctab; k += NT) ct[k] = gp(q.ctab)[k];
    const double tu = q.t_uniform ? q.ctab[0] : 0.0;
    // the vector's rows: through a buffer descriptor, a row's byte offset as the
    // scalar offset; vectors of 2 GB and more (BIG) through 64-bit row addresses
    const uint32_t rstep = (uint32_t)(du * (int)sizeof(T));
    const int64_t vbytes = q.dim * (int64_t)sizeof(T);
    const auto rv = buf_rsrc((const T *)q.v + vec * q.dim, BIG ? 0 : vbytes);
    auto row_at = [&](auto cw_, uint32_t i, int vo) {
        typedef Cols<T, decltype(cw_)::value> C;
        if constexpr (BIG)
            return ld_cols<C>((gptr<const T>)((gptr<const char>)v + (uint64_t)i * rstep + (uint32_t)vo));
        else
            return buf_load<C>(rv, vo, (int)(i * rstep));
    };
    const auto rpk = buf_rsrc(q.pku, (int64_t)q.wu * du * 4);
    const auto su = gp(q.su);
    const auto eu = gp(q.eu);
    const auto nhu = cp(q.nhu);
    const auto vpb = (gptr<const char>)gp((const T *)q.vp) + vec * vbytes;
    const auto wb = (gptr<char>)gp((T *)q.w) + vec * vbytes;
    const int W = q.wd;
    const double uu = q.u_uniform;
    const int tun = q.t_uniform, upc = __builtin_amdgcn_readfirstlane(uu >= 0.0);
    // the diagonal and the in-row hops of CW adjacent columns (from ic) of RG rows,
    // held interleaved at rs: nh hops, or as many more as fill a group of four
    auto in_row = [&](auto rg_, auto cw_, int ic, int nh, const T *rs, const auto &bd, const auto &ed,
                      auto &acc) {
        constexpr int RG = decltype(rg_)::value, CW = decltype(cw_)::value;
        typedef RowSet<T, RG> Set;
        const Set *row = reinterpret_cast<const Set *>(rs);
        const int du4 = afresh(du * 4);
        constexpr int kAhead = 8;   // entries loaded together
        Cols<uint32_t, CW> pe[kAhead];
        auto entries = [&](int s, int n) {
#pragma unroll
            for (int g = 0; g < kAhead; g += 4)
                if (s + g < n)
#pragma unroll
                    for (int u = g; u < g + 4; ++u)
                        pe[u] = buf_load<Cols<uint32_t, CW>>(rpk, ic * 4, (s + u) * du4);
        };
        entries(0, nh);
        const auto bu = ld_cols<Cols<uint32_t, CW>>(su + (uint32_t)ic);
        const auto eui = ld_cols<Cols<double, CW>>(eu + (uint32_t)ic);
#pragma unroll
        for (int c = 0; c < CW; ++c) {
            const Set own = row[ic + c];
#pragma unroll
            for (int r = 0; r < RG; ++r) {
                const uint32_t dbl = bu.x[c] & bd[r];
                double diag = eui.x[c] + ed[r];
                if (afresh(upc)) {
                    diag += uu * (double)__popc(dbl);
                } else {
                    for (int byte = 0; byte < q.nbytes; ++byte)
                        diag += lut[byte * 256 + ((dbl >> (8 * byte)) & 255u)];
                }
                acc[r][c] = diag * (double)own.x[r];
            }
        }
        // four hops: gathers, then sums in slot order; entries past a string's
        // own read the zero slot after the row
        auto group = [&](const Cols<uint32_t, CW> *p, auto tun_) {
#pragma unroll
            for (int c = 0; c < CW; ++c) {
                Set x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] = row[p[u].x[c] & 0xffffu];
                double cf[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if constexpr (decltype(tun_)::value)
                        cf[u] = __hiloint2double(
                            __double2hiint(tu) ^ (int)(p[u].x[c] & 0x80000000u), __double2loint(tu));
                    else
                        cf[u] = ct[(p[u].x[c] >> 16) & 0x3ffu];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u)
#pragma unroll
                    for (int r = 0; r < RG; ++r)
                        acc[r][c] = fma(cf[u], (double)x[u].x[r], acc[r][c]);
            }
        };
        auto hops = [&](auto tun_) {
            const int n = afresh(nh);
            for (int s = 0; s < n; s += kAhead) {
                if (s > 0) entries(s, n);
#pragma unroll
                for (int g = 0; g < kAhead; g += 4)
                    if (s + g < n) group(pe + g, tun_);
            }
        };
        if (afresh(tun))
            hops(std::true_type{});
        else
            hops(std::false_type{});
    };
    // the products of 64 CW up strings (tile tt; CW adjacent columns per lane)
    // in RG rows, held interleaved at rs; out(r, iu, w) takes element iu of row r
    auto tile_rows = [&](auto rg_, auto cw_, int tt, const auto &ri, const T *rs, auto &&out) {
        constexpr int RG = decltype(rg_)::value, CW = decltype(cw_)::value;
        typedef Cols<T, CW> C;
        // a lane past the row's end redoes the row's last columns
        const int iu = tt * (64 * CW) + lane * CW;
        const bool in = iu < du;
        const int ic = min(iu, du - CW);
        const int vo = ic * (int)sizeof(T);
        // the largest hop count of the tile's strings
        int nh = nhu[tt * (64 * CW)] >> 16;
        if constexpr (CW == 2) nh = max(nh, nhu[min(tt * 128 + 64, du - 1)] >> 16);
        double acc[RG][CW];
        in_row(rg_, cw_, ic, nh, rs, ri.bd, ri.ed, acc);
        // row-mixing neighbours: whole groups of four hops, the first kGr of
        // them and the last one to three hops loaded together for all rows
        constexpr int kGr = 2;
        C xm[RG][4 * kGr], xt[RG][3], pv[RG];
        cptr<int32_t> cl[RG];
        cptr<double> cf[RG];
#pragma unroll
        for (int r = 0; r < RG; ++r) {
            cl[r] = afresh(ri.cl[r]);
            cf[r] = afresh(ri.cf[r]);
            const int nhr = afresh(ri.nh[r]), nt = nhr & ~3;
#pragma unroll
            for (int t = 0; t < 4 * kGr; t += 4)
                if (t < nt) {
                    const i32x4_t c = *(cptr<i32x4_t>)(cl[r] + t);
#pragma unroll
                    for (int u = 0; u < 4; ++u) xm[r][t + u] = row_at(cw_, (uint32_t)c[u], vo);
                }
            if (nhr & 2) {
                xt[r][0] = row_at(cw_, (uint32_t)cl[r][nt], vo);
                xt[r][1] = row_at(cw_, (uint32_t)cl[r][nt + 1], vo);
            }
            if (nhr & 1) xt[r][2] = row_at(cw_, (uint32_t)cl[r][nhr - 1], vo);
            if (afresh(sub))
                pv[r] = ld_cols<C>((gptr<const T>)(vpb + (uint64_t)(uint32_t)ri.idn[r] * rstep + (uint32_t)vo));
        }
#pragma unroll
        for (int r = 0; r < RG; ++r) {
            auto add = [&](double c, const C &x) {
#pragma unroll
                for (int k = 0; k < CW; ++k) {
                    T xk = x.x[k];
                    // widened here, not where it was loaded
                    if constexpr (sizeof(T) == 4) asm("" : "+v"(xk));
                    acc[r][k] = fma(c, (double)xk, acc[r][k]);
                }
            };
            const int nhr = afresh(ri.nh[r]), nt = nhr & ~3;
#pragma unroll
            for (int t = 0; t < 4 * kGr; t += 4)
                if (t < nt) {
                    const f64x4_t c = *(cptr<f64x4_t>)(cf[r] + t);
#pragma unroll
                    for (int u = 0; u < 4; ++u) add(c[u], xm[r][t + u]);
                }
            for (int t = 4 * kGr; t < nt; t += 4) {
                const i32x4_t cc = *(cptr<i32x4_t>)(cl[r] + t);
                const f64x4_t c = *(cptr<f64x4_t>)(cf[r] + t);
                C x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] = row_at(cw_, (uint32_t)cc[u], vo);
#pragma unroll
                for (int u = 0; u < 4; ++u) add(c[u], x[u]);
            }
            if (nhr & 2) {
                add(cf[r][nt], xt[r][0]);
                add(cf[r][nt + 1], xt[r][1]);
            }
            if (nhr & 1) add(cf[r][nhr - 1], xt[r][2]);
            // -beta vp, round once, store
            if (afresh(sub)) add(-b, pv[r]);
            if (in && r < ri.nr) {
                C wt;
                const auto pw = (gptr<T>)(wb + (uint64_t)(uint32_t)ri.idn[r] * rstep + (uint32_t)vo);
#pragma unroll
                for (int k = 0; k < CW; ++k) {
                    wt.x[k] = (T)acc[r][k];
                    pw[k] = wt.x[k];
                }
                out(r, ic, wt);
            }
        }
    };
    // short rows: a lane takes one column of a set of RG rows; pair p is column
    // p mod du of set p / du (row_of).  Its rows' lists are its own, read four
    // hops at a time.  Tiles along the row left 64 - du lanes (or 128 - du of
    // two columns) idle: 16 orbitals (1,8), 29 vectors in FP64 230 -> 81 us;
    // (0,8), ten vectors 117 -> 9.5 us.
    auto short_rows = [&](auto rg_, int row0, int nr, int SR, auto &&row_of, auto &&out) {
        constexpr int RG = decltype(rg_)::value;
        int nh = 0;
        for (int k = 0; k < du; k += 64) nh = max(nh, nhu[k] >> 16);
        const int np = (nr + RG - 1) / RG * du;
        for (int p = tid; p < np; p += NT) {
            const int g = row_of(p), c = p - g * du;
            int idn[RG], nhr[RG];
            uint32_t bd[RG];
            double ed[RG], acc[RG][1];
            gptr<const int32_t> cl[RG];
            gptr<const double> cf[RG];
#pragma unroll
            for (int r = 0; r < RG; ++r) {
                const int i = row0 + min(g * RG + r, nr - 1);
                idn[r] = i;
                nhr[r] = gp(q.nhd)[i];
                bd[r] = gp(q.sd)[i];
                ed[r] = gp(q.ed)[i];
                cl[r] = gp(q.cold) + (int64_t)i * W;
                cf[r] = gp(q.cfd) + (int64_t)i * W;
            }
            in_row(rg_, std::integral_constant<int, 1>{}, c, nh, tile + g * SR, bd, ed, acc);
            auto neighbour = [&](int j) -> T {
                if constexpr (BIG)
                    return *(gptr<const T>)((gptr<const char>)v + (uint64_t)(uint32_t)j * rstep +
                                            (uint32_t)c * (uint32_t)sizeof(T));
                else
                    return buf_load<T>(rv, (j * du + c) * (int)sizeof(T), 0);
            };
            if (RG == 1 && q.dslot) {   // (a single up string)
#pragma unroll
                for (int r = 0; r < RG; ++r) {
                    const int n = nhr[r];
                    auto pc = gp(q.cold) + idn[r];
                    auto pf = gp(q.cfd) + idn[r];
                    int t = 0;
                    for (; t + 4 <= n; t += 4, pc += 4 * d_dn, pf += 4 * d_dn) {
                        double co[4];
                        T x[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            co[u] = pf[u * d_dn];
                            x[u] = neighbour(pc[u * d_dn]);
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u) acc[r][0] = fma(co[u], (double)x[u], acc[r][0]);
                    }
                    for (; t < n; ++t, pc += d_dn, pf += d_dn)
                        acc[r][0] = fma(*pf, (double)neighbour(*pc), acc[r][0]);
                }
            }
            // row by row: whole groups of four hops, then the last one to three together
#pragma unroll
            for (int r = 0; r < RG; ++r) {
                const int n = RG == 1 && q.dslot ? 0 : nhr[r], nt = n & ~3;
                for (int t = 0; t < nt; t += 4) {
                    const i32x4_t cc = *(gptr<const i32x4_t>)(cl[r] + t);
                    const f64x4_t co = *(gptr<const f64x4_t>)(cf[r] + t);
                    T x[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) x[u] = neighbour(cc[u]);
#pragma unroll
                    for (int u = 0; u < 4; ++u) acc[r][0] = fma(co[u], (double)x[u], acc[r][0]);
                }
                T x[3];
                double co[3];
                if (n & 2)
#pragma unroll
                    for (int u = 0; u < 2; ++u) {
                        co[u] = cf[r][nt + u];
                        x[u] = neighbour(cl[r][nt + u]);
                    }
                if (n & 1) {
                    co[2] = cf[r][n - 1];
                    x[2] = neighbour(cl[r][n - 1]);
                }
                if (n & 2) {
                    acc[r][0] = fma(co[0], (double)x[0], acc[r][0]);
                    acc[r][0] = fma(co[1], (double)x[1], acc[r][0]);
                }
                if (n & 1) acc[r][0] = fma(co[2], (double)x[2], acc[r][0]);
            }
#pragma unroll
            for (int r = 0; r < RG; ++r)
                if (g * RG + r < nr) {
                    const uint64_t at = (uint64_t)(uint32_t)idn[r] * rstep + (uint32_t)c * (uint32_t)sizeof(T);
                    if (sub) acc[r][0] = fma(-b, (double)*(gptr<const T>)(vpb + at), acc[r][0]);
                    const T wt = (T)acc[r][0];
                    *(gptr<T>)(wb + at) = wt;
                    out(g * RG + r, c, wt);
                }
        }
    };
    // what the tiles need of the nr (<= RG) rows from idn0
    auto row_info = [&](auto rg_, int idn0, int nr) {
        constexpr int RG = decltype(rg_)::value;
        struct {
            int nr, idn[RG], nh[RG];
            uint32_t bd[RG];
            double ed[RG];
            cptr<int32_t> cl[RG];
            cptr<double> cf[RG];
        } ri;
        ri.nr = nr;
#pragma unroll
        for (int r = 0; r < RG; ++r) {
            const int i = idn0 + min(r, nr - 1);
            ri.idn[r] = i;
            ri.nh[r] = cp(q.nhd)[i];
            ri.bd[r] = cp(q.sd)[i];
            ri.ed[r] = cp(q.ed)[i];
            ri.cl[r] = cp(q.cold) + (int64_t)i * W;
            ri.cf[r] = cp(q.cfd) + (int64_t)i * W;
        }
        return ri;
    };
    // sets of RG rows side by side: one set, each of whose rows is a block of
    // its own (ONE), or one block of several sets
    auto sets = [&](auto rg_) {
        constexpr int RG = decltype(rg_)::value;
        const int rows = ONE ? RG : q.rows;
        const int64_t row0 = wg * rows;
        const int nr = (int)min((int64_t)rows, d_dn - row0);
        const int nset = (nr + RG - 1) / RG;
        const int SR = RG * (du + 1);   // elements of a set
        T *wt_s = tile + (rows + RG - 1) / RG * SR;
        const bool by_row = FORM != kHvShort && (ONE || du >= NT);
        if (by_row)
            for (int r = 0; r < nset * RG; ++r) {
                T *t = tile + (r / RG) * SR + r % RG;
                const auto vr = v + (row0 + min(r, nr - 1)) * d_up;
                for (int k = tid; k < du; k += NT) t[k * RG] = vr[k];
            }
        for (int r = tid; r < nset * RG; r += NT) tile[(r / RG) * SR + du * RG + r % RG] = T(0);
        // e / du for e < 2^16: M = ceil(2^32 / du), and du = 1 apart
        const uint32_t M = 0xffffffffu / (uint32_t)du + 1u;
        auto row_of = [&](int e) { return du == 1 ? e : (int)__umulhi((uint32_t)e, M); };
        const int nel = nr * du;
        if (!by_row)
            for (int e = tid; e < nel; e += NT) {
                const int r = row_of(e), iu = e - r * du;
                tile[(r / RG) * SR + iu * RG + (r % RG)] = (v + row0 * d_up)[e];
            }
        __syncthreads();
        if constexpr (ONE) {
            const auto ri = row_info(rg_, (int)row0, nr);
            const int nt = (du + 127) >> 7;
            for (int tt = wave; tt < nt; tt += NW)
                tile_rows(rg_, std::integral_constant<int, 2>{}, tt, ri, tile, [](int, int, auto) {});
        } else if constexpr (FORM == kHvShort) {
            short_rows(rg_, (int)row0, nr, SR, row_of, [&](int r, int iu, T wt) {
                if (dots) wt_s[r * du + iu] = wt;
            });
        } else {
            auto tiles = [&](auto cw_) {
                constexpr int CW = decltype(cw_)::value;
                const int nt = (du + 64 * CW - 1) / (64 * CW);
                for (int u = wave; u < nset * nt; u += NW) {
                    const int g = u / nt, tt = u - g * nt;
                    const int rr = g * RG;
                    tile_rows(rg_, cw_, tt, row_info(rg_, (int)row0 + rr, min(RG, nr - rr)),
                              tile + g * SR, [&](int r, int iu, const auto &wt) {
                                  if (dots)
#pragma unroll
                                      for (int k = 0; k < CW; ++k)
                                          wt_s[(rr + r) * du + iu + k] = wt.x[k];
                              });
                }
            };
            if (std::is_same<Src, OneSrc>::value && du > 1)
                tiles(std::integral_constant<int, std::is_same<Src, OneSrc>::value ? 2 : 1>{});
            else
                tiles(std::integral_constant<int, 1>{});
        }
        if (!dots) return;
        // the dots: 256 threads per block take its elements in turn, the
        // products from LDS, or (one row per block) read back
        __syncthreads();
        const int t = tid & 255, blk = tid >> 8;   // thread and block
        double pa = 0.0, pww = 0.0, pvv = 0.0, ppw = 0.0, ppv = 0.0;
        const bool on = ONE ? blk < nr : blk == 0;
        if (on) {
            const int64_t e0 = (row0 + blk) * d_up;
            const int ne = ONE ? du : nel;
#pragma unroll 4
            for (int e = t; e < ne; e += 256) {
                double wd, vi;
                if (ONE) {
                    wd = (double)(gp((const T *)q.w) + vec * q.dim + e0)[e];
                    vi = (double)tile[e * RG + blk];
                } else {
                    const int r = row_of(e), iu = e - r * du;
                    wd = (double)wt_s[e];
                    vi = (double)tile[(r / RG) * SR + iu * RG + (r % RG)];
                }
                pa = fma(vi, wd, pa);
                pww = fma(wd, wd, pww);
                pvv = fma(vi, vi, pvv);
                if (reo) {
                    const double pv = sub ? (double)(gp((const T *)q.vp) + vec * q.dim + e0)[e] : 0.0;
                    ppw = fma(pv, wd, ppw);
                    ppv = fma(pv, vi, ppv);
                }
            }
        }
        __syncthreads();
        if (on) {
            double *x = sh + blk * 5 * 256 + t;
            x[0] = pa;
            x[256] = pww;
            x[512] = pvv;
            x[768] = ppw;
            x[1024] = ppv;
        }
        __syncthreads();
        // a tree over LDS (t + 128, t + 64, ..., t + 1), one wave per sum
        const int na = reo ? 5 : 3, nb = ONE ? nr : 1;
        for (int k = wave; k < na * nb; k += NW) {
            const int j = k / na, a = k - j * na;
            const double *x = sh + (j * 5 + a) * 256;
            double sum = (x[lane] + x[lane + 128]) + (x[lane + 64] + x[lane + 192]);
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) sum += __shfl_down(sum, o);
            if (lane == 0) q.pa[vec * q.na + (ONE ? row0 + j : wg) + a * q.pstride] = sum;
        }
    };
    if ((ONE && q.rg == 1) || (FORM == kHvShort && (q.rows * du <= 64 || q.dslot)))
        sets(std::integral_constant<int, 1>{});   // (short: a lane per element)
    else
        sets(std::integral_constant<int, kSide>{});
}

// Vectors whose byte offsets leave the 31 bits of a buffer load's offset.
inline bool hv_big(int64_t dim, size_t s) { return dim * (int64_t)s >= ((int64_t)1 << 31); }

// Threads of a product workgroup.  One of short rows takes no more waves than its
// pairs of elements fill, or four where they would fill five to seven, whose last
// waves run half empty (8 orbitals (1,4), 10,714 vectors: 79 us with five, 62);
// but at least the 256 of the dots, if there are any.  A tiny sector in many
// vectors is one workgroup per vector and bound by the waves it starts: 4
// orbitals (2,2), 166,666 vectors, 1082 us with eight waves each, 170 with one
// and pairs, 140 with one and a lane per element where a block has at most 64.
// Two waves where sums of U are staged (256 entries per eight orbitals).
inline unsigned hv_threads(int64_t d_up, int32_t rows, bool lut, bool dots) {
    if (hv_form(d_up, rows) != kHvShort) return kHvThreads;
    const int64_t n = ((rows + kSide - 1) / kSide * d_up + 63) / 64 * 64;
    if (n >= kHvThreads) return kHvThreads;
    return (unsigned)std::max<int64_t>(std::min<int64_t>(n, 256), dots ? 256 : lut ? 128 : 64);
}

// The fused product of one source of work, all of one form.
template <typename T, class Src>
inline void hv_form_launch(const Src &all, int form, bool big, int64_t items, unsigned threads,
                           size_t lds, hipStream_t s) {
    each_slice(all, items, threads, [&](const Src &src, unsigned wgs) {
        if (form == kHvOne && !big)
            ks_hv<T, Src, kHvOne, false><<<wgs, threads, lds, s>>>(src);
        else if (form == kHvOne)
            ks_hv<T, Src, kHvOne, true><<<wgs, threads, lds, s>>>(src);
        else if (form == kHvShort && !big)
            ks_hv<T, Src, kHvShort, false><<<wgs, threads, lds, s>>>(src);
        else if (form == kHvShort)
            ks_hv<T, Src, kHvShort, true><<<wgs, threads, lds, s>>>(src);
        else if (!big)
            ks_hv<T, Src, kHvRows, false><<<wgs, threads, lds, s>>>(src);
        else
            ks_hv<T, Src, kHvRows, true><<<wgs, threads, lds, s>>>(src);
    });
}
template <typename T>
inline void hv_step_launch(const OneSrc &src, int64_t wgs, size_t lds, hipStream_t s) {
    const BGroup &g = src.g;
    hv_form_launch<T>(src, hv_form(g.d_up, g.rows), hv_big(g.dim, sizeof(T)), wgs,
                      hv_threads(g.d_up, g.rows, g.u_uniform < 0.0, g.pa != nullptr), lds, s);
}

// chunk of a chunked pass
struct ChunkAt {
    int64_t vec, c, base;
};
__device__ __forceinline__ ChunkAt chunk_of(const BGroup &q, int64_t local) {
    ChunkAt r;
    r.vec = local / q.nchunks;
    r.c = local - r.vec * q.nchunks;
    r.base = r.c * kChunk;
    return r;
}

// pass 1, after a separate product: w -= beta' vp (n > 0); partial <v, w>
template <typename T, class Src>
__global__ void __launch_bounds__(256) ks_sub_prev(Src src) {
    __shared__ double sh[256];
    int64_t local;
    const BGroup &q = src.at(blockIdx.x, &local);
    const ChunkAt at = chunk_of(q, local);
    const int n = q.n;
    const double b = n > 0 ? q.cs.beta[at.vec * q.cs.maxs + n - 1] : 0.0;
    const int64_t off = at.vec * q.dim;
    const auto w = gp((T *)q.w) + off;
    const auto vp = gp((const T *)q.vp) + off;
    const auto v = gp((const T *)q.v) + off;
    double acc = 0.0;
    for (int k = threadIdx.x; k < kChunk; k += 256) {
        const int64_t i = at.base + k;
        if (i < q.dim) {
            double x = ldd(w + i);
            if (n > 0) {
                const T xt = (T)fma(-b, ldd(vp + i), x);
                w[i] = xt;
                x = (double)xt;
            }
            acc = fma(ldd(v + i), x, acc);
        }
    }
    const double s = block_sum(acc, sh);
    if (threadIdx.x == 0) q.pa[at.vec * q.na + at.c] = s;
}

// the direct norm pass of one chunk by one workgroup: |x|^2, <v, x>, <vp, x>
// with x = w - a v, a = alpha_n, summed over the 256 threads (every thread gets
// the sums)
template <typename T>
__device__ __forceinline__ void chunk_norm(const BGroup &q, int64_t vec, double a, int64_t base,
                                           double *sh, double *t) {
    const int64_t off = vec * q.dim;
    const auto w = gp((const T *)q.w) + off;
    const auto v = gp((const T *)q.v) + off;
    const auto vp = gp((const T *)q.vp) + off;
    double s0 = 0.0, s1 = 0.0, s2 = 0.0;
    if (q.reorth) {
        for (int k = threadIdx.x; k < kChunk; k += 256) {
            const int64_t i = base + k;
            if (i < q.dim) {
                const double vi = ldd(v + i);
                const double x = fma(-a, vi, ldd(w + i));
                s0 = fma(x, x, s0);
                s1 = fma(vi, x, s1);
                s2 = fma(ldd(vp + i), x, s2);
            }
        }
    } else {
        for (int k = threadIdx.x; k < kChunk; k += 256) {
            const int64_t i = base + k;
            if (i < q.dim) {
                const double x = fma(-a, ldd(v + i), ldd(w + i));
                s0 = fma(x, x, s0);
            }
        }
    }
    t[0] = block_sum(s0, sh);
    t[1] = q.reorth ? block_sum(s1, sh) : 0.0;
    t[2] = q.reorth ? block_sum(s2, sh) : 0.0;
}

// pass 2: partial |x|^2 (and <v, x>, <vp, x>) with x = w - alpha_n v; with
// cond, only for chains whose dot-based finish asked for it (cs.renorm)
template <typename T, class Src>
__global__ void __launch_bounds__(256) ks_norm(Src src, int cond) {
    __shared__ double sh[256];
    int64_t local;
    const BGroup &q = src.at(blockIdx.x, &local);
    const ChunkAt at = chunk_of(q, local);
    if (cond && !q.cs.renorm[at.vec]) return;
    double t[3];
    chunk_norm<T>(q, at.vec, q.cs.alpha[at.vec * q.cs.maxs + q.n], at.base, sh, t);
    if (threadIdx.x == 0) {
        double *pn = q.pn + at.vec * 3 * q.nchunks + at.c;
        pn[0] = t[0];
        if (q.reorth) {
            pn[q.nchunks] = t[1];
            pn[2 * q.nchunks] = t[2];
        }
    }
}

// sum over k = threadIdx.x, + 256, ... < n of p[k], added in that order; the
// loads go out eight at a time ahead of the additions
__device__ __forceinline__ double strided_sum(const double *__restrict__ p, int64_t n) {
    double acc = 0.0;
    int64_t k = threadIdx.x;
    for (; k + 7 * 256 < n; k += 8 * 256) {
        double x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) x[u] = p[k + u * 256];
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += x[u];
    }
    for (; k < n; k += 256) acc += p[k];
    return acc;
}

// The dots give |x|^2 = <w,w> - 2 a <v,w> + a^2 <v,v> with an absolute
// error of a few eps <w,w>; below kDotRel <w,w> (beta < 0.03 |w|) that is no
// longer beta to about 1e-12, and the chain takes the direct norm pass
// (cs.renorm) instead, as near a breakdown or an exhausted Krylov space.
constexpr double kDotRel = 1e-3;

// beta_n from |x|^2 and the reorthogonalisation terms c1 = <v, x>,
// c2 = <vp, x> of x = w - alpha_n v, and the chain's bookkeeping
__device__ __forceinline__ void finish_beta(const ChainState &cs, int c, int n, int reorth,
                                            double s0, double s1, double s2) {
    if (reorth) cs.alpha[(int64_t)c * cs.maxs + n] += s1;
    cs.corr[c] = s1;
    cs.corr2[c] = s2;
    const double bb = s0 - s1 * s1 - s2 * s2;
    const double b = sqrt(bb > 0.0 ? bb : 0.0);
    cs.beta[(int64_t)c * cs.maxs + n] = b;
    if (!cs.done[c]) {
        const double am = cs.amax[c] > 0.0 ? cs.amax[c] : 1.0;
        if (!(b >= cs.btol * am)) cs.done[c] = 1;
        cs.len[c] = n + 1;
    }
    cs.inv[c] = cs.done[c] ? 0.0 : 1.0 / b;
    if (c == 0) {
        cs.dlog[n] = cs.done[c];
        if (cs.stop && cs.done[c])
            __hip_atomic_store(cs.stop, 1 + cs.len[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// Vectors of at most this many chunks take the direct norm pass, when a chain
// asks for it, inside the finishing kernel: a step is then three launches
// instead of five (2.4 + 3.6 us less on a 12-orbital sector).  A chain then has a
// workgroup per chunk, each of which takes the sums of the dots by itself; more
// of them would make that count.  Every step asks for it where alpha is more
// than about 30 beta, as with a large constant in H: 120 steps of ten chains of
// 10 orbitals (5,5) then take 4.8 ms in FP64, and 60 of one chain of 213,444
// states 2.2 (12.9 and 18.0 with one workgroup per chain).
constexpr int kFinishChunks = 32;
__host__ __device__ inline int finish_parts(int nchunks) {
    return nchunks <= kFinishChunks ? nchunks : 1;
}

// x = w - a v with a = <v, w>: s = |x|^2, <v, x>, <vp, x> from the dots d
// (<v,w>, <w,w>, <v,v>, and with reorthogonalisation <vp,w>, <vp,v>); whether
// |x|^2 needs the direct norm instead
__device__ __forceinline__ bool dot_terms(const double *d, int reorth, double *s) {
    const double a = d[0], ww = d[1], vv = d[2];
    s[0] = fma(a * a, vv, fma(-2.0 * a, a, ww));
    s[1] = reorth ? fma(-a, vv, a) : 0.0;
    s[2] = reorth ? fma(-a, d[4], d[3]) : 0.0;
    return !(s[0] > kDotRel * ww);
}

// per-chain sums of the partials and the recurrence bookkeeping
// mode 0: alpha_n; mode 1: reorthogonalisation terms, beta_n, breakdown, from
// the norm pass; mode 4: mode 1 for the chains marked cs.renorm.
template <class Src>
__global__ void __launch_bounds__(256) ks_finish(Src src, int mode) {
    __shared__ double sh[256];
    int64_t local;
    const BGroup &q = src.at(blockIdx.x, &local);
    const int c = (int)local;
    if (c >= q.nvec) return;
    const ChainState &cs = q.cs;
    const int n = q.n;
    if (mode == 0) {
        const double *p = q.pa + (int64_t)c * q.na;
        double acc = strided_sum(p, q.na);
        const double s = block_sum(acc, sh);
        if (threadIdx.x == 0) {
            cs.alpha[(int64_t)c * cs.maxs + n] = s;
            cs.apre[c] = s;
            const double a = fabs(s);
            if (a > cs.amax[c]) cs.amax[c] = a;
        }
        return;
    }
    if (mode == 4 && !cs.renorm[c]) return;
    const double *p = q.pn + (int64_t)c * 3 * q.nchunks;
    const double s0 = block_sum(strided_sum(p, q.nchunks), sh);
    double s1 = 0.0, s2 = 0.0;
    if (q.reorth) {
        s1 = block_sum(strided_sum(p + q.nchunks, q.nchunks), sh);
        s2 = block_sum(strided_sum(p + 2 * q.nchunks, q.nchunks), sh);
    }
    if (threadIdx.x != 0) return;
    finish_beta(cs, c, n, q.reorth, s0, s1, s2);
}

// alpha_n and beta_n from the fused product's dots (q.na partials of each per
// chain), unless the dots cannot resolve beta: then the direct
// norm here (finish_parts workgroups per chain, a chunk each; the last one to
// finish its chunk, counted in cs.renorm, takes the sums), or, for longer
// vectors, by the norm pass for chains marked cs.renorm.
// The array sums are block_sum's trees, one wave per array.
template <typename T, class Src>
__global__ void __launch_bounds__(256) ks_finish_fused(Src src) {
    __shared__ double sh[5 * 256];
    __shared__ double tot[5];
    __shared__ int flag[2];   // direct norm wanted; this is the last workgroup
    int64_t local;
    const BGroup &q = src.at(blockIdx.x, &local);
    const uint32_t parts = finish_parts(q.nchunks), x0 = (uint32_t)local;
    const int c = parts == 1 ? x0 : x0 / parts, part = x0 - c * parts;
    const ChainState &cs = q.cs;
    const int n = q.n, t = threadIdx.x, lane = t & 63;
    const double *p = q.pa + (int64_t)c * q.na;
    const int na = q.reorth ? 5 : 3;
    for (int a = 0; a < na; ++a) sh[a * 256 + t] = strided_sum(p + a * q.pstride, q.na);
    __syncthreads();
    for (int a = t >> 6; a < na; a += 4) {
        const double *x = sh + a * 256;
        double s = (x[lane] + x[lane + 128]) + (x[lane + 64] + x[lane + 192]);
        for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o);
        if (lane == 0) tot[a] = s;
    }
    __syncthreads();
    const double a = tot[0];   // <v, w>
    if (t == 0) {
        double s[3];
        const bool rn = dot_terms(tot, q.reorth, s);
        flag[0] = rn && q.nchunks <= kFinishChunks;
        if (part == 0) {
            cs.alpha[(int64_t)c * cs.maxs + n] = a;
            cs.apre[c] = a;
            if (fabs(a) > cs.amax[c]) cs.amax[c] = fabs(a);
            if (q.nchunks > kFinishChunks) cs.renorm[c] = rn;
            if (!rn) finish_beta(cs, c, n, q.reorth, s[0], s[1], s[2]);
        }
    }
    __syncthreads();
    if (!flag[0]) return;
    double x[3];
    chunk_norm<T>(q, c, a, (int64_t)part * kChunk, sh, x);
    if (parts == 1) {
        if (t == 0) finish_beta(cs, c, n, q.reorth, x[0], x[1], x[2]);
        return;
    }
    double *pn = q.pn + (int64_t)c * 3 * q.nchunks;
    if (t == 0) {
        for (int k = 0; k < 3; ++k) pn[k * q.nchunks + part] = x[k];
        const int before = __hip_atomic_fetch_add(cs.renorm + c, 1, __ATOMIC_ACQ_REL,
                                                  __HIP_MEMORY_SCOPE_AGENT);
        flag[1] = before == (int)parts - 1;
    }
    __syncthreads();
    if (!flag[1]) return;
    const int m = q.nchunks;
    for (int k = 0; k < 3; ++k)
        x[k] = k == 0 || q.reorth ? block_sum(strided_sum(pn + k * m, m), sh) : 0.0;
    if (t == 0) {
        cs.renorm[c] = 0;
        finish_beta(cs, c, n, q.reorth, x[0], x[1], x[2]);
    }
}

// The two-pass product's partial arrays (three, five with
// reorthogonalisation, of q.na values per chain) are summed in two launches:
// ks_dots_stage sums contiguous ranges, one per workgroup of kDotBlocks, into
// q.pn ([chain][array][kDotBlocks]); ks_finish_dots sums those in order and
// records alpha_n and beta_n as ks_finish_fused does (the direct norm a pass of
// its own).  Each thread's
// share is summed in index order and each block's by a fixed tree.
constexpr int kDotBlocks = 64;

template <class Src>
__global__ void __launch_bounds__(256) ks_dots_stage(Src src) {
    constexpr int U = 8;
    __shared__ double sh[256];
    int64_t local;
    const BGroup &q = src.at(blockIdx.y, &local);
    const int c = (int)local;
    const int na = q.reorth ? 5 : 3;
    const int64_t len = (q.na + kDotBlocks - 1) / kDotBlocks;
    const int64_t k0 = (int64_t)blockIdx.x * len;
    const int64_t k1 = min((int64_t)q.na, k0 + len);
    const double *p = q.pa + (int64_t)c * q.na;
    double *o = q.pn + ((int64_t)c * 5) * kDotBlocks + blockIdx.x;
    for (int a = 0; a < na; ++a) {
        const double *pa = p + a * q.pstride;
        double acc = 0.0;
        int64_t k = k0 + threadIdx.x;
        for (; k + (U - 1) * 256 < k1; k += U * 256) {
            double x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = pa[k + u * 256];
#pragma unroll
            for (int u = 0; u < U; ++u) acc += x[u];
        }
        for (; k < k1; k += 256) acc += pa[k];
        const double t = block_sum(acc, sh);
        if (threadIdx.x == 0) o[a * kDotBlocks] = t;
    }
}

template <class Src>
__global__ void __launch_bounds__(kDotBlocks) ks_finish_dots(Src src) {
    __shared__ double sh[5][kDotBlocks];
    int64_t local;
    const BGroup &q = src.at(blockIdx.x, &local);
    const int c = (int)local;
    const ChainState &cs = q.cs;
    const int n = q.n;
    const int na = q.reorth ? 5 : 3;
    const int t = threadIdx.x;
    const double *p = q.pn + ((int64_t)c * 5) * kDotBlocks;
#pragma unroll
    for (int a = 0; a < 5; ++a) sh[a][t] = a < na ? p[a * kDotBlocks + t] : 0.0;
    __syncthreads();
    for (int s = kDotBlocks / 2; s > 0; s >>= 1) {
        if (t < s)
#pragma unroll
            for (int a = 0; a < 5; ++a) sh[a][t] += sh[a][t + s];
        __syncthreads();
    }
    if (t != 0) return;
    const double d[5] = {sh[0][0], sh[1][0], sh[2][0], sh[3][0], sh[4][0]};
    cs.alpha[(int64_t)c * cs.maxs + n] = d[0];
    cs.apre[c] = d[0];
    if (fabs(d[0]) > cs.amax[c]) cs.amax[c] = fabs(d[0]);
    double s3[3];
    cs.renorm[c] = dot_terms(d, q.reorth, s3);
    if (!cs.renorm[c]) finish_beta(cs, c, n, q.reorth, s3[0], s3[1], s3[2]);
}

// pass 3: w = (w - alpha v - c1 v - c2 vp) / beta_n; psi += svec[n] v (replay).
// Element by element, so a chunk is cut into kUpdParts workgroups: a vector of
// a few chunks would otherwise leave most of the chip idle (one workgroup took
// 9 us for 4,900 elements, 105 of them 15 us for 853,776).
constexpr int kUpdParts = 8;

template <typename T, class Src>
__global__ void __launch_bounds__(256) ks_update(Src src) {
    int64_t local;
    const BGroup &q = src.at(blockIdx.x / kUpdParts, &local);
    const ChunkAt at = chunk_of(q, local);
    const ChainState &cs = q.cs;
    const double a = cs.apre[at.vec], c1 = cs.corr[at.vec], c2 = cs.corr2[at.vec];
    const double s = cs.inv[at.vec];
    const int64_t off = at.vec * q.dim;
    const auto w = gp((T *)q.w) + off;
    const auto v = gp((const T *)q.v) + off;
    const auto vp = gp((const T *)q.vp) + off;
    const auto psi = gp(q.psi);
    const double sv = psi ? q.svec[q.n] : 0.0;
    constexpr int P = kChunk / kUpdParts;
    const int64_t base = at.base + (int64_t)(blockIdx.x % kUpdParts) * P;
#pragma unroll
    for (int k = 0; k < P; k += 256) {
        const int64_t i = base + k + threadIdx.x;
        if (i < q.dim) {
            const double vi = ldd(v + i);
            double x = fma(-a, vi, ldd(w + i));
            if (q.reorth) {
                x = fma(-c1, vi, x);
                x = fma(-c2, ldd(vp + i), x);
            }
            w[i] = (T)(x * s);
            if (psi) psi[i] = fma(sv, vi, psi[i]);
        }
    }
}

// Whole chains of a small sector in one launch: a workgroup runs the steps of
// one chain from LDS.
//
// A step of a sector of a few thousand states is otherwise three launches of
// 3 to 12 us each, all latency: 10 chains of 3,920 states (the Green function
// of an 8-orbital impurity) took 25 us a step.  Here the three vectors, the hop
// lists and the diagonal's tables stay in LDS and nothing is read from memory
// between the first and the last step.  Every sum is the one of the separate
// kernels (the element's terms in list order; the dots per product block over
// 256 threads and a tree; the direct norm over a chunk), so the coefficients
// are the same bit for bit: 7.6 us a step for the same chains, of which about 5
// are LDS reads (hop entry, neighbour, coefficient).  More workgroups per chain
// would have to exchange the vector through memory.  Rows lie du + 1 apart with a zero after each and a
// zero row at the end: hop lists are read four at a time, and entries past a
// string's own read a zero.
constexpr int kChainThreads = 1024;

struct ChainLds {
    size_t v, sh, part, ct, lut, su, eu, sd, ed, nu, nd, pk, cl, cf, bytes;
};
__host__ __device__ inline ChainLds chain_lds(int64_t du, int64_t dn, int wu, int wd, int nctab,
                                              int nlut, int na, int nblk, size_t s) {
    ChainLds l;
    size_t o = 0;
    auto take = [&](size_t n) {
        const size_t at = o;
        o = (o + n + 15) & ~(size_t)15;
        return at;
    };
    l.v = take(3 * s * (size_t)(dn + 1) * (size_t)(du + 1));
    l.sh = take(sizeof(double) * na * kChainThreads);
    l.part = take(sizeof(double) * na * nblk);
    l.ct = take(sizeof(double) * nctab);
    l.lut = take(sizeof(double) * nlut);
    l.eu = take(sizeof(double) * du);
    l.ed = take(sizeof(double) * dn);
    l.cf = take(sizeof(double) * wd * dn);
    l.cl = take(sizeof(int32_t) * wd * dn);
    l.pk = take(sizeof(uint32_t) * wu * du);
    l.su = take(sizeof(uint32_t) * du);
    l.sd = take(sizeof(uint32_t) * dn);
    l.nu = take(sizeof(int32_t) * du);
    l.nd = take(sizeof(int32_t) * dn);
    l.bytes = o;
    return l;
}

template <typename T>
__global__ void __launch_bounds__(kChainThreads) ks_chain(const OneSrc src, const int n1) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ double tot[5], sc[5];   // sums of the dots; a, c1, c2, inv, beta
    __shared__ int flag[2];            // direct norm wanted; chain stopped
    const BGroup &q = src.g;
    const int c = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    constexpr int NT = kChainThreads;
    const int du = (int)q.d_up, dn = (int)q.d_dn, d = (int)q.dim, wd = (q.wd + 3) & ~3, wu = q.wu;
    const int nlut = q.u_uniform >= 0.0 ? 0 : q.nbytes * 256, na = q.reorth ? 5 : 3;
    const ChainLds o = chain_lds(du, dn, wu, wd, q.nctab, nlut, na, q.nblk, sizeof(T));
    const int st = du + 1, vlen = (dn + 1) * st;
    T *bvp = reinterpret_cast<T *>(smem_raw + o.v), *bv = bvp + vlen, *bw = bv + vlen;
    double *sh = (double *)(smem_raw + o.sh), *part = (double *)(smem_raw + o.part);
    double *ct = (double *)(smem_raw + o.ct), *lut = (double *)(smem_raw + o.lut);
    double *eu = (double *)(smem_raw + o.eu), *ed = (double *)(smem_raw + o.ed);
    double *cf = (double *)(smem_raw + o.cf);
    int32_t *cl = (int32_t *)(smem_raw + o.cl), *nu = (int32_t *)(smem_raw + o.nu);
    int32_t *nd = (int32_t *)(smem_raw + o.nd);
    uint32_t *pk = (uint32_t *)(smem_raw + o.pk), *su = (uint32_t *)(smem_raw + o.su);
    uint32_t *sd = (uint32_t *)(smem_raw + o.sd);
    for (int k = tid; k < q.nctab; k += NT) ct[k] = q.ctab[k];
    for (int k = tid; k < nlut; k += NT) lut[k] = q.ulut[k];
    for (int k = tid; k < wu * du; k += NT) pk[k] = q.pku[k];
    for (int k = tid; k < du; k += NT) {
        su[k] = q.su[k];
        eu[k] = q.eu[k];
        nu[k] = q.nhu[k] & 0xffff;
    }
    for (int i = tid; i < dn; i += NT) {
        sd[i] = q.sd[i];
        ed[i] = q.ed[i];
        const int n = q.nhd[i];
        nd[i] = n;
        for (int s = 0; s < wd; ++s) {
            const int at = q.dslot ? s * dn + i : i * q.wd + s;
            cl[i * wd + s] = s < n ? q.cold[at] * st : dn * st;
            cf[i * wd + s] = s < n ? q.cfd[at] : 0.0;
        }
    }
    for (int k = tid; k < 3 * vlen; k += NT) bvp[k] = T(0);
    __syncthreads();
    // e / du for e < 2^16: M = ceil(2^32 / du), and du = 1 apart
    const uint32_t M = 0xffffffffu / (uint32_t)du + 1u;
    auto row_of = [&](int e) { return du == 1 ? e : (int)__umulhi((uint32_t)e, M); };
    const T *gv = (const T *)q.v + (int64_t)c * d;
    for (int e = tid; e < d; e += NT) bv[e + row_of(e)] = gv[e];
    const ChainState &cs = q.cs;
    double amax = 0.0;
    int done = 0, len = 0;
    if (tid == 0) {
        amax = cs.amax[c];
        done = cs.done[c];
        len = cs.len[c];
        flag[1] = done;
        sc[4] = 0.0;
    }
    const double uu = q.u_uniform;
    double *const al = cs.alpha + (int64_t)c * cs.maxs, *const be = cs.beta + (int64_t)c * cs.maxs;
    __syncthreads();
    for (int n = 0; n < n1; ++n) {
        if (flag[1]) break;   // nothing after a stopped chain's last step is read
        // w = H v - beta' vp
        const double b = sc[4];
        for (int e = tid; e < d; e += NT) {
            const int idn = row_of(e), iu = e - idn * du, at = e + idn;
            const T *row = bv + idn * st;
            const uint32_t dbl = su[iu] & sd[idn];
            double diag = eu[iu] + ed[idn];
            if (uu >= 0.0) {
                diag += uu * (double)__popc(dbl);
            } else {
                for (int byte = 0; byte < q.nbytes; ++byte)
                    diag += lut[byte * 256 + ((dbl >> (8 * byte)) & 255u)];
            }
            double acc = diag * (double)bv[at];
            const uint32_t *pe = pk + iu;
            const int nh = nu[iu];
            for (int s = 0; s < nh; s += 4) {
                uint32_t p[4];
                double x[4], cc[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) p[u] = pe[(s + u) * du];
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] = (double)row[p[u] & 0xffffu];
#pragma unroll
                for (int u = 0; u < 4; ++u) cc[u] = ct[(p[u] >> 16) & 0x3ffu];
#pragma unroll
                for (int u = 0; u < 4; ++u) acc = fma(cc[u], x[u], acc);
            }
            const T *col = bv + iu;
            const int nhd = nd[idn], l0 = idn * wd;
            for (int s = 0; s < nhd; s += 4) {
                double x[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) x[u] = (double)col[cl[l0 + s + u]];
#pragma unroll
                for (int u = 0; u < 4; ++u) acc = fma(cf[l0 + s + u], x[u], acc);
            }
            if (n > 0) acc = fma(-b, (double)bvp[at], acc);
            bw[at] = (T)acc;
        }
        __syncthreads();
        // the dots per product block
        for (int b0 = 0; b0 < q.nblk; b0 += NT / 256) {
            const int blk = b0 + (tid >> 8), t = tid & 255;
            double s5[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
            if (blk < q.nblk) {
                const int e0 = blk * q.rows * du, e1 = min(e0 + q.rows * du, d);
                for (int e = e0 + t; e < e1; e += 256) {
                    const int at = e + row_of(e);
                    const double wdv = (double)bw[at], vi = (double)bv[at];
                    s5[0] = fma(vi, wdv, s5[0]);
                    s5[1] = fma(wdv, wdv, s5[1]);
                    s5[2] = fma(vi, vi, s5[2]);
                    if (q.reorth) {
                        const double pv = n > 0 ? (double)bvp[at] : 0.0;
                        s5[3] = fma(pv, wdv, s5[3]);
                        s5[4] = fma(pv, vi, s5[4]);
                    }
                }
            }
            if (b0 > 0) __syncthreads();
            for (int a = 0; a < na; ++a) sh[a * NT + tid] = s5[a];
            __syncthreads();
            for (int k = wave; k < na * (NT / 256); k += NT / 64) {
                const int g = k / na, a = k - g * na;
                const double *x = sh + a * NT + g * 256;
                double t2 = (x[lane] + x[lane + 128]) + (x[lane + 64] + x[lane + 192]);
                for (int r = 32; r > 0; r >>= 1) t2 += __shfl_down(t2, r);
                if (lane == 0 && b0 + g < q.nblk) part[a * q.nblk + b0 + g] = t2;
            }
        }
        __syncthreads();
        if (wave < na) {   // nblk <= 64: the other leaves of the tree are zero
            double t2 = lane < q.nblk ? part[wave * q.nblk + lane] : 0.0;
            for (int r = 32; r > 0; r >>= 1) t2 += __shfl_down(t2, r);
            if (lane == 0) tot[wave] = t2;
        }
        __syncthreads();
        double a = 0.0, s0 = 0.0, s1 = 0.0, s2 = 0.0;
        // beta_n and the bookkeeping (finish_beta)
        auto beta_of = [&]() {
            if (q.reorth) al[n] = a + s1;
            const double bb = s0 - s1 * s1 - s2 * s2;
            const double bn = sqrt(bb > 0.0 ? bb : 0.0);
            be[n] = bn;
            const double am = amax > 0.0 ? amax : 1.0;
            if (!(bn >= cs.btol * am)) done = 1;
            len = n + 1;
            sc[0] = a;
            sc[1] = s1;
            sc[2] = s2;
            sc[3] = done ? 0.0 : 1.0 / bn;
            sc[4] = bn;
            flag[1] = done;
        };
        if (tid == 0) {
            a = tot[0];
            al[n] = a;
            if (fabs(a) > amax) amax = fabs(a);
            double s[3];
            flag[0] = dot_terms(tot, q.reorth, s);
            s0 = s[0];
            s1 = s[1];
            s2 = s[2];
            sc[0] = a;
            if (!flag[0]) beta_of();
        }
        __syncthreads();
        if (flag[0]) {
            // the direct norm (one chunk: d <= kChunk)
            double r[3] = {0.0, 0.0, 0.0};
            if (tid < 256) {
                const double an = sc[0];
                for (int e = tid; e < d; e += 256) {
                    const int at = e + row_of(e);
                    const double vi = (double)bv[at], x = fma(-an, vi, (double)bw[at]);
                    r[0] = fma(x, x, r[0]);
                    if (q.reorth) {
                        r[1] = fma(vi, x, r[1]);
                        r[2] = fma((double)bvp[at], x, r[2]);
                    }
                }
                for (int k = 0; k < 3; ++k) sh[k * NT + tid] = r[k];
            }
            __syncthreads();
            if (wave < 3) {
                const double *x = sh + wave * NT;
                double t2 = (x[lane] + x[lane + 128]) + (x[lane + 64] + x[lane + 192]);
                for (int k = 32; k > 0; k >>= 1) t2 += __shfl_down(t2, k);
                if (lane == 0) tot[wave] = t2;
            }
            __syncthreads();
            if (tid == 0) {
                s0 = tot[0];
                s1 = q.reorth ? tot[1] : 0.0;
                s2 = q.reorth ? tot[2] : 0.0;
                beta_of();
            }
            __syncthreads();
        }
        // v_{n+1} in the place of w
        const double an = sc[0], c1 = sc[1], c2 = sc[2], inv = sc[3];
        for (int e = tid; e < d; e += NT) {
            const int at = e + row_of(e);
            const double vi = (double)bv[at];
            double x = fma(-an, vi, (double)bw[at]);
            if (q.reorth) {
                x = fma(-c1, vi, x);
                x = fma(-c2, (double)bvp[at], x);
            }
            bw[at] = (T)(x * inv);
        }
        T *const t3 = bvp;
        bvp = bv;
        bv = bw;
        bw = t3;
        __syncthreads();
    }
    if (tid == 0) {
        cs.amax[c] = amax;
        cs.done[c] = done;
        cs.len[c] = len;
    }
}

template <typename T, class Src>
inline void update_launch(const Src &all, int64_t chunks, hipStream_t s) {
    each_slice(all, chunks, 256 * kUpdParts, [&](const Src &src, unsigned n) {
        ks_update<T, Src><<<n * kUpdParts, 256, 0, s>>>(src);
    });
}

// psi += svec[n] v_n alone (the last replay step)
template <typename T, class Src>
__global__ void __launch_bounds__(256) ks_accum(Src src) {
    int64_t local;
    const BGroup &q = src.at(blockIdx.x, &local);
    const ChunkAt at = chunk_of(q, local);
    const auto v = gp((const T *)q.v);
    const auto psi = gp(q.psi);
    const double sv = q.svec[q.n];
    for (int k = threadIdx.x; k < kChunk; k += 256) {
        const int64_t i = at.base + k;
        if (i < q.dim) psi[i] = fma(sv, ldd(v + i), psi[i]);
    }
}

}  // namespace qcm
