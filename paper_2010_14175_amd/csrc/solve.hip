// Group-per-row CSR products and the PCG iteration (Sec. 3 "miniwarp" SpMV; Sec. 5.2 PCG).
//
// SpMV: a group of GS lanes (GS in {4, 8, 16, 32, 64}, chosen from the average row length like
// the paper's miniwarps, but sized for 64-lane wavefronts) owns one row; lanes stride through
// the row's entries with coalesced, non-temporal loads of the matrix and cached loads of x;
// the group reduces with cross-lane shuffles in a fixed order.  Each block owns one
// contiguous range of rows and blocks are renumbered so that every XCD streams one contiguous
// part of the matrix (its L2 then holds the x entries its rows share).
//
// Batches: the solver always runs over a batch of independent systems (one system for
// pcg_solve).  Each system keeps its own scalars and done flag; every launch maps its blocks
// to (system, block within the system) with the block count a single-system solve of that
// system would use, and dot products are summed per system over exactly those blocks, so a
// system's iterates do not depend on its batch-mates (bit for bit).
//
// PCG: all scalars (rho, alpha, beta, ||r||) live on the device.  Dot products are fused into
// the kernel that produces one of their operands, which stores one partial sum per block.  With
// the fused products (small systems) every block of the kernel that needs the sum adds the
// partials itself, in block order (results do not depend on scheduling), and takes the scalar
// step in registers: three launches an iteration instead of six, the 20^3 solve 1.03 -> 0.82 ms.
// Larger systems have thousands of partials, added by one block per system in the same order.
// The scalars are kept in two buffers used in turn: a kernel that advances them reads one and
// its first block writes the other.  (A last-block-done reduction inside the producing kernel needs a device-scope
// release per block, which on this 8-XCD part writes back the L2 and cost more than the extra
// launch.)  A device flag ends the iteration: kernels that see it return at once, so the host
// enqueues chunks of iterations and reads the flag once per chunk, one chunk behind.
#include <unistd.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <mutex>
#include <vector>

#include "handle.hpp"

namespace afsai {

constexpr int kThreads = 256;
// automatic PCG form: fused products up to these entries of A and G (of one system; their second gather
// is paid per entry, the update kernels they save per row and per launch), and for the systems of a
// batch, where the launches are shared, up to these rows.  Microseconds an iteration, fused and
// separate: 7-point rows, 4.5 M entries 41.6, 48.9; 8.0 M 65.3, 65.8; 13 M 170, 94; 81-entry rows,
// 6.1 M 50.3, 55.0; 11 M 64.1, 63.8; 20 M 92.3, 87.3
constexpr int64_t kFusedEntries = 7 << 20;
constexpr int kFusedMaxRows = 200000;
constexpr int64_t kSmallBytes = 4 << 20;       // one-launch solve: matrix bytes of an iteration at most
constexpr int kSmallIters = 1024;              // and iterations of a launch
constexpr int kSmallPause = 64;                // solves that do not try it after one whose blocks did not meet
constexpr int64_t kGateEntries = 1 << 26;  // factors whose products look at r.r before they start
// resumable solver: iterations of the first chunk, least GPU time of a chunk and its share of
// the GPU time so far
constexpr int kFirstChunk = 4;
constexpr double kMinChunkUs = 100.0;
constexpr double kChunkShare = 0.125;

enum : int { FIN_NONE = 0, FIN_RHO0 = 3, FIN_INIT = 4, FIN_RESID = 6 };
enum : int { DONE_NO = 0, DONE_CONVERGED = 1, DONE_NOT_SPD = 2, DONE_MAXIT = 3, DONE_ZERO_RHS = 4 };

struct PcgScalars {  // 88 bytes: copied as 11 double words
    double rho;      // r.z of the current iterate
    double alpha;
    double beta;
    double rr;       // ||r||^2
    double bb;       // ||b||^2
    double tol;      // rtol * ||b||
    double rtol;
    int32_t it;      // iterations completed
    int32_t maxit;
    int32_t done;    // DONE_*
    int32_t plain;   // 1: M = I (z = r)
    double resid;    // ||b - A x||^2 of the final check
    int32_t fresh;   // 1: the scalar step after the last iteration has been taken
    int32_t pad;
};
static_assert(sizeof(PcgScalars) == 88, "PcgScalars is copied as 11 double words");

// Systems of a batch (device arrays; nullptr: one system covering everything)
struct Systems {
    const int32_t *row0 = nullptr;    // [nsys + 1] first row of each system
    const int32_t *slice0 = nullptr;  // [nsys + 1] first SELL slice of each system
};
// Blocks of one launch shape (device arrays; nullptr: one system, block b = its block b)
struct Map {
    const int32_t *blk_sys = nullptr;  // [nblocks] system of each (logical) block
    const int32_t *sys_b0 = nullptr;   // [nsys] first block of each system
    const int32_t *sys_nb = nullptr;   // [nsys] blocks of each system
};

struct Job {
    int k;   // system
    int lb;  // block within the system
    int nb;  // blocks of the system
    int gb;  // logical block of the launch (index of the partial sums)
};

__device__ __forceinline__ Job block_job(const Map &mp, int nxcd) {
    Job j;
    j.gb = xcd_block(blockIdx.x, gridDim.x, nxcd);
    if (mp.blk_sys) {
        j.k = mp.blk_sys[j.gb];
        j.lb = j.gb - mp.sys_b0[j.k];
        j.nb = mp.sys_nb[j.k];
    } else {
        j.k = 0;
        j.lb = j.gb;
        j.nb = gridDim.x;
    }
    return j;
}

// [lo, hi) of the `count` items starting at `base` that block lb of nb owns
__device__ __forceinline__ void block_range(int base, int count, int lb, int nb, int &lo, int &hi) {
    const int64_t per = ((int64_t)count + nb - 1) / nb;
    lo = base + (int)min<int64_t>(count, per * lb);
    hi = base + (int)min<int64_t>(count, per * (lb + 1));
}

__device__ __forceinline__ void sys_rows(const Systems &sy, int n, int k, int &r0, int &r1) {
    if (sy.row0) {
        r0 = sy.row0[k];
        r1 = sy.row0[k + 1];
    } else {
        r0 = 0;
        r1 = n;
    }
}

// ---------------------------------------------------------------------------------------
// block helpers
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ double block_sum(double v, double *sh /* >= kThreads/64 */) {
    v = wave_sum(v);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) sh[w] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x == 0)
        for (int k = 0; k < kThreads / 64; ++k) t += sh[k];
    __syncthreads();
    return t;  // valid in thread 0
}

// thread 0 stores this block's partial sums, slot k at partials[k * gridDim.x + gb], gb being
// the logical block (blocks of one system are consecutive and cover its rows in order)
__device__ __forceinline__ void store_partials(double *partials, int slots, const double *mine, int gb) {
    if (threadIdx.x == 0)
        for (int k = 0; k < slots; ++k) partials[(size_t)k * gridDim.x + gb] = mine[k];
}

// block_sum and store of one dot, or of two at once
template <bool TWO>
__device__ __forceinline__ void store_dots(double va, double vb, double *sh /* 2 * kThreads / 64 */, double *pa, double *pb,
                                           int gb) {
    va = wave_sum(va);
    if (TWO) vb = wave_sum(vb);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sh[w] = va;
        if (TWO) sh[kThreads / 64 + w] = vb;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double ta = 0.0, tb = 0.0;
        for (int k = 0; k < kThreads / 64; ++k) {
            ta += sh[k];
            if (TWO) tb += sh[kThreads / 64 + k];
        }
        pa[gb] = ta;
        if (TWO) pb[gb] = tb;
    }
}

// The partial sums that a launch of nblocks blocks stored (nblocks = 0: sums, one per system)
struct Parts {
    const double *p = nullptr;
    Map mp;
    int nblocks = 0;
};

// The sums of system k's partials of two launches, each in block order (every thread adds a
// contiguous run, then the runs are added in thread order); every thread of the block gets
// them.  b without partials: its sum is 0.  U: partials of each loaded before they are added, two by two (the
// lanes' runs lie apart, so that a block alone is bound by its loads' round trips and cache lines).
template <int U = 1>
__device__ __forceinline__ void parts_sum(const Parts &a, const Parts &b, int k, double *sh /* 2 * kThreads / 64 */,
                                          double &sa, double &sb) {
    if (a.nblocks == 0) {  // added before
        sa = a.p[k];
        sb = b.p ? b.p[k] : 0.0;
        return;
    }
    double v[2] = {0.0, 0.0};
    const double *p[2];
    int len[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const Parts &pt = q ? b : a;
        p[q] = pt.p;
        len[q] = 0;
        if (pt.p) {
            const int b0 = pt.mp.blk_sys ? pt.mp.sys_b0[k] : 0;
            const int np = pt.mp.blk_sys ? pt.mp.sys_nb[k] : pt.nblocks;
            const int per = (np + kThreads - 1) / kThreads;
            const int lo = threadIdx.x * per;
            p[q] += b0 + lo;
            len[q] = min(per, np - lo);
        }
        if (U == 1)
            for (int j = 0; j < len[q]; ++j) v[q] += p[q][j];
    }
    if constexpr (U > 1) {
        for (int j = 0; j < max(len[0], len[1]); j += U) {
            double t[2][U];
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int u = 0; u < U; u += 2) {
                    typedef double Two __attribute__((ext_vector_type(2), aligned(8)));
                    Two w = {0.0, 0.0};
                    if (j + u + 2 <= len[q]) w = *reinterpret_cast<const Two *>(p[q] + j + u);
                    else if (j + u < len[q]) w.x = p[q][j + u];
                    t[q][u] = w.x;
                    t[q][u + 1] = w.y;
                }
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int u = 0; u < U; ++u)
                    if (j + u < len[q]) v[q] += t[q][u];
        }
    }
    const int w = threadIdx.x >> 6;
    v[0] = wave_sum(v[0]);
    if (b.p) v[1] = wave_sum(v[1]);
    if ((threadIdx.x & 63) == 0) {
        sh[w] = v[0];
        sh[kThreads / 64 + w] = v[1];
    }
    __syncthreads();
    sa = sb = 0.0;
#pragma unroll
    for (int j = 0; j < kThreads / 64; ++j) {
        sa += sh[j];
        sb += sh[kThreads / 64 + j];
    }
    __syncthreads();
}

// The same, where few kernels or many blocks need a sum: one block per system stores the
// system's sums of one or two launches.  Two arrays of 547 partials (139,968 rows) are loaded at once before they are added
// (65.3 -> 64.0 us an iteration), of 4,096 too (5.1 -> 4.6 us a sum); between them the plain loop is as fast and shorter
// (2,391: 4.5, 4.1 us).
__global__ __launch_bounds__(kThreads) void k_reduce(Parts a, Parts b, double *oa, double *ob, const PcgScalars *scs) {
    const int k = blockIdx.x;
    const int done = scs[k].done;  // (loaded beside the partials)
    __shared__ double sh[2 * kThreads / 64];
    double sa, sb;
    const int na = a.mp.blk_sys ? a.mp.sys_nb[k] : a.nblocks, nb = b.mp.blk_sys ? b.mp.sys_nb[k] : b.nblocks;
    const int most = max(na, nb);
    if (most <= 4 * kThreads) parts_sum<4>(a, b, k, sh, sa, sb);
    else if (most <= 12 * kThreads) parts_sum<1>(a, b, k, sh, sa, sb);
    else parts_sum<16>(a, b, k, sh, sa, sb);
    if (threadIdx.x == 0 && !done) {
        oa[k] = sa;
        if (b.p) ob[k] = sb;
    }
}

// The scalar step after an iteration: rr = ||r||^2, rz = r.z (unused with M = I); bad: p.Ap <= 0
__device__ __forceinline__ void advance(PcgScalars &s, double rr, double rz, int bad) {
    s.fresh = 1;
    if (bad) {
        s.done = DONE_NOT_SPD;
        return;
    }
    s.rr = rr;
    s.it += 1;
    if (sqrt(rr) <= s.tol) {
        s.done = DONE_CONVERGED;
    } else if (s.it >= s.maxit) {
        s.done = DONE_MAXIT;
    } else {
        const double z = s.plain ? rr : rz;
        s.beta = z / s.rho;
        s.rho = z;
    }
}

// alpha = rho / p.q of the system, or false when p.q <= 0: the system's block 0 then marks it
__device__ __forceinline__ bool step_alpha(const PcgScalars &s, const Parts &pq, int k, int lb, int32_t *bad, double *sh,
                                           double &alpha) {
    double v, u;
    parts_sum(pq, Parts(), k, sh, v, u);
    if (!(v > 0.0) || !isfinite(v)) {
        if (lb == 0 && threadIdx.x == 0) bad[k] = 1;
        return false;
    }
    alpha = s.rho / v;
    return true;
}

// The scalars at the start, from b.b and r.r
__device__ __forceinline__ void init_scalars(PcgScalars &s, double bb, double rr) {
    s.bb = bb;
    s.rr = rr;
    s.tol = s.rtol * sqrt(bb);
    s.it = 0;
    if (bb == 0.0) s.done = DONE_ZERO_RHS;
    else if (sqrt(rr) <= s.tol) s.done = DONE_CONVERGED;
    else if (s.maxit == 0) s.done = DONE_MAXIT;
    if (s.plain) s.rho = rr;
}

// One block per system: the sums of the start and of the final check (partials of the previous
// launch; FIN_INIT has two of them, b.b and then r.r).
__global__ __launch_bounds__(kThreads) void k_finalize(Parts pa, Parts pb, int fin, PcgScalars *scs) {
    const int k = blockIdx.x;
    PcgScalars *sc = scs + k;
    if (fin == FIN_RHO0 && sc->done) return;
    __shared__ double sh[2 * kThreads / 64];
    double v, rr;
    parts_sum(pa, pb, k, sh, v, rr);
    if (threadIdx.x != 0) return;
    switch (fin) {
        case FIN_RHO0:
            sc->rho = v;
            break;
        case FIN_INIT:  // v = b.b, rr = r.r
            init_scalars(*sc, v, rr);
            break;
        case FIN_RESID:
            sc->resid = v;
            break;
        default:
            break;
    }
}

// ---------------------------------------------------------------------------------------
// CSR SpMV, one group of GS lanes per row; optional fused dot y.w (one system)
// ---------------------------------------------------------------------------------------
template <int GS, int U, typename VT, bool DOT>
__global__ __launch_bounds__(kThreads) void k_spmv(int n, const int32_t *__restrict__ rp,
                                                    const int32_t *__restrict__ ci,
                                                    const VT *__restrict__ val,
                                                    const double *__restrict__ x,
                                                    double *__restrict__ y,
                                                    const double *__restrict__ w,
                                                    double *__restrict__ partials,
                                                    PcgScalars *sc, int nxcd) {
    if (sc && sc->done) return;
    __shared__ double sh[kThreads / 64];
    const int lb = xcd_block(blockIdx.x, gridDim.x, nxcd);
    int r0, r1;
    block_range(0, n, lb, gridDim.x, r0, r1);
    const int lg = threadIdx.x % GS, grp = threadIdx.x / GS;
    constexpr int RPI = kThreads / GS;  // rows per block iteration
    double part = 0.0;
    for (int row = r0 + grp; row < r1; row += RPI) {
        const int a = rp[row], b = rp[row + 1];
        double acc = 0.0;
        for (int e0 = a + lg; e0 < b; e0 += GS * U) {
            int c[U];
            VT v[U];
            // all loads of a round are issued before any is used
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int e = e0 + u * GS;
                c[u] = -1;
                v[u] = VT(0);
                if (e < b) {
                    c[u] = __builtin_nontemporal_load(&ci[e]);
                    v[u] = __builtin_nontemporal_load(&val[e]);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (c[u] >= 0) acc = fma((double)v[u], x[c[u]], acc);
        }
#pragma unroll
        for (int off = GS / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, GS);
        if (lg == 0) {
            y[row] = acc;
            if (DOT) part = fma(acc, w[row], part);
        }
    }
    if (DOT) {
        const double bs = block_sum(part, sh);
        store_partials(partials, 1, &bs, lb);
    }
}

// rows [r0, r1) of SELL slice sl
__device__ __forceinline__ void sell_slice_rows(const int32_t *srow0, int n, int sl, int &r0, int &r1) {
    if (srow0) {
        r0 = srow0[sl];
        r1 = srow0[sl + 1];
    } else {
        r0 = sl * kSlice;
        r1 = min(n, r0 + kSlice);
    }
}

// The wavefront's index within its block, as a scalar: slice indices, their offsets and widths
// then stay in scalar registers and the per-lane loops over a slice run on scalar bounds
// (from the thread index the compiler would keep them in vector registers and guard every
// unrolled step with exec-mask branches).
__device__ __forceinline__ int wave_index() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

// Windows (kWin consecutive slices, one per wavefront of a block) of logical block lb of nb
// over nw windows: the blocks are grouped like the XCDs of xcd_block(); each group takes a
// contiguous part of the windows and deals it to its blocks in rounds of one window each, so
// that the blocks running at once on an XCD share one narrow band of rows and of the gathered
// vector (A's product at 150^3: 1,982 -> 1,928 us against one contiguous range per block).
// With one window per block (nb = nw) block lb takes window lb.  The walk depends only on
// (nw, lb, nb, nxcd): a system's partial sums are the same alone and in a batch, and the same
// for its natural and its length-ordered layouts.
__device__ __forceinline__ void window_walk(int nw, int lb, int nb, int nxcd, int &w0, int &w1, int &step) {
    const int ng = nxcd < 1 ? 1 : (nb < nxcd ? nb : nxcd);
    const int per = nb / ng, extra = nb % ng;
    int off, cnt;
    if (lb < extra * (per + 1)) {
        off = (lb / (per + 1)) * (per + 1);
        cnt = per + 1;
    } else {
        off = extra * (per + 1) + ((lb - extra * (per + 1)) / per) * per;
        cnt = per;
    }
    if (nw == nb) {
        w0 = lb;
        w1 = off + cnt;
    } else if (nw < (1 << 19) && nb <= (1 << 12)) {  // (a division of 64 bits takes some hundred instructions)
        w0 = (int)((uint32_t)nw * (uint32_t)off / (uint32_t)nb) + (lb - off);
        w1 = (int)((uint32_t)nw * (uint32_t)(off + cnt) / (uint32_t)nb);
    } else {
        w0 = (int)((int64_t)nw * off / nb) + (lb - off);
        w1 = (int)((int64_t)nw * (off + cnt) / nb);
    }
    step = cnt;
}

// A load of the matrix stream: NT (non-temporal) for matrices that no cache holds until the next
// iteration, so that they leave the gathered vectors in the L2
template <bool NT, typename T>
__device__ __forceinline__ T ldm(const T *p) {
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

// One lane's sum over `len` entries stored `stride` apart from base, continuing acc: one
// sequential fma chain in stored order.  Software pipeline: the columns and values of the
// next U entries are loaded before the gathers of the current U, so one round trip to memory
// serves both.
template <int U, int STRIDE, bool NT, typename VT>
__device__ __forceinline__ double lane_chain(const int32_t *__restrict__ col, const VT *__restrict__ val,
                                             const double *__restrict__ x, int64_t base, int len, double acc) {
    int c[U];
    VT v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        c[u] = 0;
        v[u] = VT(0);
        if (u < len) {
            const int64_t d = base + (int64_t)u * STRIDE;
            c[u] = ldm<NT>(&col[d]);
            v[u] = ldm<NT>(&val[d]);
        }
    }
    for (int k0 = 0; k0 < len; k0 += U) {
        int cn[U];
        VT vn[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            cn[u] = 0;
            vn[u] = VT(0);
            if (k0 + U + u < len) {
                const int64_t d = base + (int64_t)(k0 + U + u) * STRIDE;
                cn[u] = ldm<NT>(&col[d]);
                vn[u] = ldm<NT>(&val[d]);
            }
        }
        double xv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) xv[u] = (k0 + u < len) ? x[c[u]] : 0.0;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k0 + u < len) acc = fma((double)v[u], xv[u], acc);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            c[u] = cn[u];
            v[u] = vn[u];
        }
    }
    return acc;
}

// SELL-64 product: one wavefront per slice of 64 rows, one lane per row; entry k of the 64
// rows is one contiguous wave load.  Optional fused dots (DOT 1: y.w; 2: w.w too).  For the tail of a split layout
// (perm/rowmap set) the launch is not tied to systems (mp, sy empty, scs may be null).  With
// rows ordered by length (lens set, instance ORD) a block takes whole windows of kWin slices,
// its wavefronts taking the slices in turn, and the sums reach their natural rows through LDS,
// so that y is written and the dot summed in row order.  The ordered instance keeps twice as many entries in flight
// (its gathers are scattered over the window's rows and wait longest).
template <int U, typename VT, int DOT, bool NT, bool ORD = false>
__global__ __launch_bounds__(kThreads) void k_sell_spmv(int n, int nslices, const uint32_t *__restrict__ sptr,
                                                         const int32_t *__restrict__ srow0,
                                                         const int32_t *__restrict__ perm,
                                                         const int32_t *__restrict__ rowmap,
                                                         const uint64_t *__restrict__ init,
                                                         const int32_t *__restrict__ col,
                                                         const VT *__restrict__ val,
                                                         const double *__restrict__ x, double *__restrict__ y,
                                                         const double *__restrict__ w,
                                                         double *__restrict__ partials, PcgScalars *scs, Map mp,
                                                         Systems sy, int nxcd, const int32_t *__restrict__ lens,
                                                         const int32_t *__restrict__ wsl,
                                                         const int32_t *__restrict__ wofs,
                                                         const uint32_t *__restrict__ tsptr,
                                                         const int32_t *__restrict__ tcol,
                                                         const VT *__restrict__ tval,
                                                         const int32_t *__restrict__ toff,
                                                         const double *__restrict__ rr,
                                                         double *__restrict__ partials_ww) {
    const Job jb = block_job(mp, nxcd);
    if (scs && scs[jb.k].done) return;
    __shared__ double sh[2 * kThreads / 64];
    // converged by this iteration's r.r (one sum per system): the product is not needed
    if (rr && sqrt(rr[jb.k]) <= scs[jb.k].tol) return;
    const int sb = sy.slice0 ? sy.slice0[jb.k] : 0;
    const int sn = sy.slice0 ? sy.slice0[jb.k + 1] - sb : nslices;
    static_assert(kWin == kThreads / 64, "a window holds one slice per wavefront of a block");
    // (the ordered instance keeps the thread-derived index: measured faster there)
    const int wv = ORD ? (int)(threadIdx.x >> 6) : wave_index(), lane = threadIdx.x & 63;
    double part = 0.0, part_ww = 0.0;
    if constexpr (ORD) {
        static_assert(kWin * kSlice % kThreads == 0, "the wavefronts of a block take a window's slices in turn");
        constexpr int UO = U >= 8 ? 16 : U;
        __shared__ double sy_win[kWin * kSlice];
        // (slices of one system: window w holds slices kWin w to kWin w + kWin - 1, no look-ups)
        const bool one = !srow0;
        const int wa = one ? 0 : wofs[sb], wb = one ? (sn + kWin - 1) / kWin : wofs[sb + sn];
        int w0, w1, wstep;
        window_walk(wb - wa, jb.lb, jb.nb, nxcd, w0, w1, wstep);
        for (int wi = wa + w0; wi < wa + w1; wi += wstep) {
            const int ws = one ? wi * kWin : wsl[wi], we = one ? min(ws + kWin, sn) : wsl[wi + 1];
            int wr0, u0;
            sell_slice_rows(srow0, n, ws, wr0, u0);
            for (int sl = ws + wv; sl < we; sl += kThreads / 64) {
                const int64_t li = (int64_t)sl * kSlice + lane;
                const int r = perm[li];
                const int len = lens[li];
                const int64_t base = (int64_t)sptr[sl] * kSlice + lane;
                const double acc = lane_chain<UO, kSlice, NT>(col, val, x, base, len, 0.0);
                if (r >= 0) sy_win[r - wr0] = acc;
            }
            __syncthreads();
            for (int sl = ws + wv; sl < we; sl += kThreads / 64) {
                int r0, r1;
                sell_slice_rows(srow0, n, sl, r0, r1);
                const int rn = r0 + lane;
                if (rn < r1) {
                    const double an = sy_win[rn - wr0];
                    y[rn] = an;
                    if (DOT) part = fma(an, w[rn], part);
                    if (DOT == 2) part_ww = fma(w[rn], w[rn], part_ww);
                }
            }
            __syncthreads();
        }
        if (DOT) {
            store_dots<DOT == 2>(part, part_ww, sh, partials, partials_ww, jb.gb);
        }
        return;
    }
    int w0, w1, wstep;
    window_walk((sn + kWin - 1) / kWin, jb.lb, jb.nb, nxcd, w0, w1, wstep);
    for (int wi = w0; wi < w1; wi += wstep) {
        const int sl = sb + wi * kWin + wv;
        if (sl >= sb + sn) break;
        int r0, r1;
        sell_slice_rows(srow0, n, sl, r0, r1);
        int r = r0 + lane;
        if (perm) r = perm[sl * kSlice + lane];
        const bool valid = r >= 0 && r < (perm ? n : r1);
        const int ro = (valid && rowmap) ? rowmap[r] : r;
        const uint32_t c0 = sptr[sl];
        const int width = (int)(sptr[sl + 1] - c0);
        const int64_t base = (int64_t)c0 * kSlice + lane;
        // rows split between the two layouts start with their leading entries: run here from the
        // tail layout (tcol set; the slice's split rows are consecutive tail rows), or continue
        // the sum a separate tail product left in y
        double acc = 0.0;
        if (init && valid && ((init[sl] >> lane) & 1)) {
            if (tcol) {
                const int t = toff[sl] + __popcll(init[sl] & ((1ull << lane) - 1ull));
                const uint32_t tc0 = tsptr[t >> 6];
                const int tw = (int)(tsptr[(t >> 6) + 1] - tc0);
                const int64_t tb = (int64_t)tc0 * kSlice + (t & 63);
                for (int k = 0; k < tw; ++k) {
                    const int64_t d = tb + (int64_t)k * kSlice;
                    acc = fma((double)tval[d], x[tcol[d]], acc);
                }
            } else {
                acc = y[ro];
            }
        }
        acc = lane_chain<U, kSlice, NT>(col, val, x, base, width, acc);
        if (valid) {
            y[ro] = acc;
            if (DOT) part = fma(acc, w[ro], part);
            if (DOT == 2) part_ww = fma(w[ro], w[ro], part_ww);
        }
    }
    if (DOT) {
        store_dots<DOT == 2>(part, part_ww, sh, partials, partials_ww, jb.gb);
    }
}

// One lane's sum over `nr` runs of three consecutive columns (the layout with one column
// index per run): the values of run j are entries 3j..3j+2 of the lane, stored kSlice apart
// from vbase, its first column at rbase + j * kSlice.  The same sequential fma chain over the
// entries in stored order as lane_chain, with UR runs (3 UR entries) in flight.
template <int UR, bool NT, typename VT>
__device__ __forceinline__ double run_chain(const int32_t *__restrict__ col3, const VT *__restrict__ val,
                                            const double *__restrict__ x, int64_t rbase, int64_t vbase, int nr,
                                            double acc) {
    int c[UR];
    VT v[UR][3];
#pragma unroll
    for (int u = 0; u < UR; ++u) {
        c[u] = 0;
#pragma unroll
        for (int e = 0; e < 3; ++e) v[u][e] = VT(0);
        if (u < nr) {
            c[u] = ldm<NT>(&col3[rbase + (int64_t)u * kSlice]);
#pragma unroll
            for (int e = 0; e < 3; ++e) v[u][e] = ldm<NT>(&val[vbase + (int64_t)(3 * u + e) * kSlice]);
        }
    }
    for (int j0 = 0; j0 < nr; j0 += UR) {
        int cn[UR];
        VT vn[UR][3];
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            cn[u] = 0;
#pragma unroll
            for (int e = 0; e < 3; ++e) vn[u][e] = VT(0);
            if (j0 + UR + u < nr) {
                const int j = j0 + UR + u;
                cn[u] = ldm<NT>(&col3[rbase + (int64_t)j * kSlice]);
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    vn[u][e] = ldm<NT>(&val[vbase + (int64_t)(3 * j + e) * kSlice]);
            }
        }
        double xv[UR][3];
#pragma unroll
        for (int u = 0; u < UR; ++u)
#pragma unroll
            for (int e = 0; e < 3; ++e) xv[u][e] = (j0 + u < nr) ? x[c[u] + e] : 0.0;
#pragma unroll
        for (int u = 0; u < UR; ++u)
            if (j0 + u < nr) {
#pragma unroll
                for (int e = 0; e < 3; ++e) acc = fma((double)v[u][e], xv[u][e], acc);
            }
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            c[u] = cn[u];
#pragma unroll
            for (int e = 0; e < 3; ++e) v[u][e] = vn[u][e];
        }
    }
    return acc;
}

// SELL-64 product over the layout with one column index per run of three (plain layouts
// only: natural row order, no split): the walk, row sums, stores and fused dot of k_sell_spmv,
// so products and dots are identical to it bit for bit.
template <int UR, typename VT, bool DOT, bool NT>
__global__ __launch_bounds__(kThreads) void k_sell_spmv_runs(int n, const uint32_t *__restrict__ sptr,
                                                             const int32_t *__restrict__ srow0,
                                                             const int32_t *__restrict__ col3,
                                                             const VT *__restrict__ val,
                                                             const double *__restrict__ x, double *__restrict__ y,
                                                             const double *__restrict__ w,
                                                             double *__restrict__ partials, PcgScalars *scs, Map mp,
                                                             Systems sy, int nslices, int nxcd) {
    const Job jb = block_job(mp, nxcd);
    if (scs && scs[jb.k].done) return;
    __shared__ double sh[kThreads / 64];
    const int sb = sy.slice0 ? sy.slice0[jb.k] : 0;
    const int sn = sy.slice0 ? sy.slice0[jb.k + 1] - sb : nslices;
    const int wv = wave_index(), lane = threadIdx.x & 63;
    double part = 0.0;
    int w0, w1, wstep;
    window_walk((sn + kWin - 1) / kWin, jb.lb, jb.nb, nxcd, w0, w1, wstep);
    for (int wi = w0; wi < w1; wi += wstep) {
        const int sl = sb + wi * kWin + wv;
        if (sl >= sb + sn) break;
        int r0, r1;
        sell_slice_rows(srow0, n, sl, r0, r1);
        const int r = r0 + lane;
        const uint32_t c0 = sptr[sl];
        const int nr = (int)(sptr[sl + 1] - c0) / 3;
        const double acc = run_chain<UR, NT, VT>(col3, val, x, (int64_t)(c0 / 3u) * kSlice + lane,
                                             (int64_t)c0 * kSlice + lane, nr, 0.0);
        if (r < r1) {
            y[r] = acc;
            if (DOT) part = fma(acc, w[r], part);
        }
    }
    if (DOT) {
        const double bs = block_sum(part, sh);
        store_partials(partials, 1, &bs, jb.gb);
    }
}

// Fused PCG products (SELL-64, one lane per row, layouts without a tail).  The vector being
// multiplied is formed on the fly from two others with the same fma the separate update
// kernel would use, so the result is identical to update-then-multiply; the owner lane of
// each row also stores the updated entry.
//   FUSE_AP:  p_new = z + beta p_old (p_new = z on the first iteration); q = A p_new;
//             partial sums of p_new.q; takes the scalar step of the iteration before (pa: its
//             r.r, pb: its r.z) from s_in to s_out
//   FUSE_GR:  r_new = r_old - alpha q; x += alpha p_new; t = G r_new; partial sums of r_new.r_new
//             (pa: p.q)
enum : int { FUSE_AP = 1, FUSE_GR = 2 };

template <int U, typename VT, int MODE, bool NT>
__global__ __launch_bounds__(kThreads) void k_sell_fused(int n, int nslices, const uint32_t *__restrict__ sptr,
                                                          const int32_t *__restrict__ srow0,
                                                          const int32_t *__restrict__ col,
                                                          const VT *__restrict__ val,
                                                          const double *__restrict__ va,   // z | r_old
                                                          const double *__restrict__ vb,   // p_old | q
                                                          double *__restrict__ own_out,    // p_new | r_new
                                                          double *__restrict__ x,          // - | x
                                                          const double *__restrict__ pn,   // - | p_new
                                                          double *__restrict__ y,          // q | t
                                                          double *__restrict__ partials,
                                                          const PcgScalars *s_in, PcgScalars *s_out, int32_t *bad,
                                                          Parts pa, Parts pb, int first, Map mp, Systems sy,
                                                          int nxcd) {
    const Job jb = block_job(mp, nxcd);
    __shared__ double sh[2 * kThreads / 64];
    PcgScalars st = s_in[jb.k];
    double alpha = 0.0;
    if (MODE == FUSE_AP) {
        if (!st.done && !st.fresh) {
            double rr, rz;
            parts_sum(pa, pb, jb.k, sh, rr, rz);
            advance(st, rr, rz, bad[jb.k]);
        }
        if (!st.done) st.fresh = 0;
        if (jb.lb == 0 && threadIdx.x == 0) s_out[jb.k] = st;
        if (st.done) return;
    } else {
        if (st.done || !step_alpha(st, pa, jb.k, jb.lb, bad, sh, alpha)) return;
    }
    const double coef = (MODE == FUSE_AP) ? st.beta : -alpha;
    const int sb = sy.slice0 ? sy.slice0[jb.k] : 0;
    const int sn = sy.slice0 ? sy.slice0[jb.k + 1] - sb : nslices;
    const int wv = wave_index(), lane = threadIdx.x & 63;
    int w0, w1, wstep;
    window_walk((sn + kWin - 1) / kWin, jb.lb, jb.nb, nxcd, w0, w1, wstep);
    double part = 0.0;
    for (int wi = w0; wi < w1; wi += wstep) {
        const int sl = sb + wi * kWin + wv;
        if (sl >= sb + sn) break;
        int r0, r1;
        sell_slice_rows(srow0, n, sl, r0, r1);
        const int r = r0 + lane;
        const uint32_t c0 = sptr[sl];
        const int width = (int)(sptr[sl + 1] - c0);
        const int64_t base = (int64_t)c0 * kSlice + lane;
        double acc = 0.0;
        // software pipeline as in lane_chain: the next U columns and values are loaded before
        // the current gathers
        int c[U];
        VT v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            c[u] = 0;
            v[u] = VT(0);
            if (u < width) {
                const int64_t d = base + (int64_t)u * kSlice;
                c[u] = ldm<NT>(&col[d]);
                v[u] = ldm<NT>(&val[d]);
            }
        }
        for (int k0 = 0; k0 < width; k0 += U) {
            int cn[U];
            VT vn[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                cn[u] = 0;
                vn[u] = VT(0);
                if (k0 + U + u < width) {
                    const int64_t d = base + (int64_t)(k0 + U + u) * kSlice;
                    cn[u] = ldm<NT>(&col[d]);
                    vn[u] = ldm<NT>(&val[d]);
                }
            }
            double xa[U], xb[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const bool in = k0 + u < width;
                xa[u] = in ? va[c[u]] : 0.0;
                xb[u] = (in && !(MODE == FUSE_AP && first)) ? vb[c[u]] : 0.0;
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k0 + u < width) {
                    const double xv = (MODE == FUSE_AP && first) ? xa[u] : fma(coef, xb[u], xa[u]);
                    acc = fma((double)v[u], xv, acc);
                }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                c[u] = cn[u];
                v[u] = vn[u];
            }
        }
        if (r < r1) {
            const double own = (MODE == FUSE_AP && first) ? va[r] : fma(coef, vb[r], va[r]);
            own_out[r] = own;
            y[r] = acc;
            if (MODE == FUSE_AP) {
                part = fma(own, acc, part);
            } else {
                x[r] = fma(alpha, pn[r], x[r]);
                part = fma(own, own, part);
            }
        }
    }
    const double bs = block_sum(part, sh);
    store_partials(partials, 1, &bs, jb.gb);
}

// r = b - q ; partials of b.b and r.r ; finalisation checks ||b|| = 0 and ||r0|| <= tol
__global__ __launch_bounds__(kThreads) void k_init_residual(int n, const double *__restrict__ b,
                                                             const double *__restrict__ q,
                                                             double *__restrict__ r,
                                                             double *__restrict__ partials, Map mp, Systems sy,
                                                             int nxcd) {
    __shared__ double sh[kThreads / 64];
    const Job jb = block_job(mp, nxcd);
    int a0, a1, i0, i1;
    sys_rows(sy, n, jb.k, a0, a1);
    block_range(a0, a1 - a0, jb.lb, jb.nb, i0, i1);
    double pb = 0.0, pr = 0.0;
    for (int i = i0 + threadIdx.x; i < i1; i += kThreads) {
        const double bi = b[i], ri = bi - q[i];
        r[i] = ri;
        pb = fma(bi, bi, pb);
        pr = fma(ri, ri, pr);
    }
    double mine[2];
    mine[0] = block_sum(pb, sh);
    mine[1] = block_sum(pr, sh);
    store_partials(partials, 2, mine, jb.gb);
}

// x += alpha p ; r -= alpha q  (pq: the partials of p.q) ; SUM (M = I): partials of ||r||^2
template <bool SUM>
__global__ __launch_bounds__(kThreads) void k_update_xr(int n, double *__restrict__ x,
                                                         double *__restrict__ r,
                                                         const double *__restrict__ p,
                                                         const double *__restrict__ q,
                                                         double *__restrict__ partials,
                                                         const PcgScalars *scs, int32_t *bad, Parts pq, Map mp,
                                                         Systems sy, int nxcd) {
    const Job jb = block_job(mp, nxcd);
    const PcgScalars st = scs[jb.k];
    __shared__ double sh[2 * kThreads / 64];
    double alpha;
    if (st.done || !step_alpha(st, pq, jb.k, jb.lb, bad, sh, alpha)) return;
    int a0, a1, i0, i1;
    sys_rows(sy, n, jb.k, a0, a1);
    block_range(a0, a1 - a0, jb.lb, jb.nb, i0, i1);
    double pr = 0.0;
    for (int i = i0 + threadIdx.x; i < i1; i += kThreads) {
        x[i] = fma(alpha, p[i], x[i]);
        const double ri = fma(-alpha, q[i], r[i]);
        r[i] = ri;
        pr = fma(ri, ri, pr);
    }
    if (SUM) {
        const double bs = block_sum(pr, sh);
        store_partials(partials, 1, &bs, jb.gb);
    }
}

// With a preconditioner r.r is summed over the windows of a SELL product, block by block and row by row as
// k_sell_fused sums it, so that the forms, and a system alone and in a batch of another form, stop at the same iteration
// with the same ||r|| bit for bit (with M = I it is rho and keeps its order; only one form has it): by G^T's product, or
// here where the products wait for it.  (Here for every size: four times as many blocks, 612,000 rows of 7 10.01 -> 10.29 ms.)
__global__ __launch_bounds__(kThreads) void k_update_xr_win(int n, double *__restrict__ x, double *__restrict__ r,
                                                             const double *__restrict__ p, const double *__restrict__ q,
                                                             double *__restrict__ partials, const PcgScalars *scs,
                                                             int32_t *bad, Parts pq, Map mp, Systems sy, int nxcd) {
    static_assert(kWin * kSlice == kThreads, "one row of a window per thread");
    const Job jb = block_job(mp, nxcd);
    const double rho = scs[jb.k].rho, v = pq.p[jb.k];
    if (scs[jb.k].done) return;
    if (!(v > 0.0) || !isfinite(v)) {
        if (jb.lb == 0 && threadIdx.x == 0) bad[jb.k] = 1;
        return;
    }
    const double alpha = rho / v;
    __shared__ double sh[kThreads / 64];
    int a0, a1, w0, w1, step;
    sys_rows(sy, n, jb.k, a0, a1);
    const int64_t len = a1 - a0;
    window_walk((int)((len + kThreads - 1) / kThreads), jb.lb, jb.nb, nxcd, w0, w1, step);
    double pr = 0.0;
    for (int w = w0; w < w1; w += step) {
        const int64_t i = (int64_t)w * kThreads + threadIdx.x;
        if (i < len) {
            x[a0 + i] = fma(alpha, p[a0 + i], x[a0 + i]);
            const double ri = fma(-alpha, q[a0 + i], r[a0 + i]);
            r[a0 + i] = ri;
            pr = fma(ri, ri, pr);
        }
    }
    const double bs = block_sum(pr, sh);
    store_partials(partials, 1, &bs, jb.gb);
}

// The scalar step of the iteration (rr, rz: its partials) from s_in to s_out, then p = z + beta p
// (first = 1: no step, p = z)
__global__ __launch_bounds__(kThreads) void k_update_p(int n, double *__restrict__ p,
                                                        const double *__restrict__ z,
                                                        const PcgScalars *s_in, PcgScalars *s_out, const int32_t *bad,
                                                        Parts rr, Parts rz, int first, Map mp, Systems sy, int nxcd) {
    const Job jb = block_job(mp, nxcd);
    __shared__ double sh[2 * kThreads / 64];
    PcgScalars st = s_in[jb.k];
    if (!first) {
        if (!st.done) {
            double vr, vz;
            parts_sum(rr, rz, jb.k, sh, vr, vz);
            advance(st, vr, vz, bad[jb.k]);
        }
        if (jb.lb == 0 && threadIdx.x == 0) s_out[jb.k] = st;
    }
    if (st.done) return;
    const double beta = st.beta;
    int a0, a1, i0, i1;
    sys_rows(sy, n, jb.k, a0, a1);
    block_range(a0, a1 - a0, jb.lb, jb.nb, i0, i1);
    if (first)
        for (int i = i0 + threadIdx.x; i < i1; i += kThreads) p[i] = z[i];
    else
        for (int i = i0 + threadIdx.x; i < i1; i += kThreads) p[i] = fma(beta, p[i], z[i]);
}

// x = 0 for the systems whose right-hand side is zero
__global__ __launch_bounds__(kThreads) void k_zero_rhs(int n, double *__restrict__ x, const PcgScalars *scs, Map mp,
                                                       Systems sy, int nxcd) {
    const Job jb = block_job(mp, nxcd);
    if (scs[jb.k].done != DONE_ZERO_RHS) return;
    int a0, a1, i0, i1;
    sys_rows(sy, n, jb.k, a0, a1);
    block_range(a0, a1 - a0, jb.lb, jb.nb, i0, i1);
    for (int i = i0 + threadIdx.x; i < i1; i += kThreads) x[i] = 0.0;
}

// One block per system: takes the scalar step of the last iteration where no kernel has yet (the
// fused form takes it at the start of the next one), then copies the scalars into pinned
// host memory (mapped), where the host reads them once the chunk's event has completed; a
// kernel is cheaper here than a copy engine transfer of a few hundred bytes.
__global__ __launch_bounds__(kThreads) void k_publish(PcgScalars *scs, const int32_t *bad, Parts rr, Parts rz,
                                                      PcgScalars *__restrict__ host) {
    __shared__ double sh[2 * kThreads / 64];
    const int k = blockIdx.x;
    PcgScalars st = scs[k];
    if (!st.done && !st.fresh) {
        double vr, vz;
        parts_sum(rr, rz, k, sh, vr, vz);
        advance(st, vr, vz, bad[k]);
        if (threadIdx.x == 0) scs[k] = st;
    }
    if (threadIdx.x == 0) host[k] = st;
}

__global__ void k_set_scalars(PcgScalars *scs, int32_t *bad, int32_t *ctl, int nsys, double rtol, int maxit, int plain) {
    if (blockIdx.x == 0 && threadIdx.x < 4) ctl[threadIdx.x] = 0;
    for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < nsys; k += gridDim.x * blockDim.x) {
        PcgScalars s{};
        s.rtol = rtol;
        s.maxit = maxit;
        s.plain = plain;
        s.fresh = 1;
        scs[k] = s;
        bad[k] = 0;
    }
}

// true residual partials: ||b - Ax||^2 with q = A x
__global__ __launch_bounds__(kThreads) void k_resid_norm(int n, const double *__restrict__ b,
                                                          const double *__restrict__ q,
                                                          double *__restrict__ partials, Map mp, Systems sy,
                                                          int nxcd) {
    __shared__ double sh[kThreads / 64];
    const Job jb = block_job(mp, nxcd);
    int a0, a1, i0, i1;
    sys_rows(sy, n, jb.k, a0, a1);
    block_range(a0, a1 - a0, jb.lb, jb.nb, i0, i1);
    double pr = 0.0;
    for (int i = i0 + threadIdx.x; i < i1; i += kThreads) {
        const double d = b[i] - q[i];
        pr = fma(d, d, pr);
    }
    const double bs = block_sum(pr, sh);
    store_partials(partials, 1, &bs, jb.gb);
}

}  // namespace afsai

#include "pcg_small.hpp"

namespace afsai {

// ---------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------
// Lanes per row (the paper's miniwarp, Sec. 3) and independent loads per lane per round, from
// the average row length: about four entries per lane per round and at most 8 loads in flight
// per lane.
static void spmv_shape(double avg_nnz, int *gs, int *un) {
    int g = 4;
    while (g < 64 && g * 4 < avg_nnz) g <<= 1;
    int u = 1;
    while (u < 8 && g * u < avg_nnz) u <<= 1;
    if (option(AFSAI_OPT_SPMV_GROUP) > 0) g = (int)option(AFSAI_OPT_SPMV_GROUP);
    if (option(AFSAI_OPT_SPMV_UNROLL) > 0) u = (int)option(AFSAI_OPT_SPMV_UNROLL);
    *gs = g;
    *un = u;
}

static int blocks_for_rows(int n, int gs, const DeviceInfo &di) {
    const int64_t rows_per_iter = kThreads / gs;
    int64_t want = (n + rows_per_iter - 1) / rows_per_iter;
    int64_t cap = (int64_t)di.num_cus * 8;
    int64_t b = want < cap ? want : cap;
    return (int)(b < 1 ? 1 : b);
}

static int blocks_for_vec(int n, const DeviceInfo &di) {
    int64_t want = ((int64_t)n + kThreads * 4 - 1) / (kThreads * 4);
    int64_t cap = (int64_t)di.num_cus * 8;
    int64_t b = want < cap ? want : cap;
    return (int)(b < 1 ? 1 : b);
}

static int blocks_for_slices(int nslices, const DeviceInfo &di) {
    int64_t nb = ((int64_t)nslices + kThreads / 64 - 1) / (kThreads / 64);
    const int64_t cap = (int64_t)di.num_cus * 16;
    if (nb > cap) nb = cap;
    if (nb < 1) nb = 1;
    return (int)nb;
}

static std::atomic<int64_t> g_forms[4];  // afsai_pcg_form_counts

// the device's XCDs as bits of their hardware numbers (looked up on the first call)
static int xcc_mask(const DeviceInfo &di, hipStream_t s, uint32_t *mask) {
    constexpr int kMaxDev = 64;
    static std::mutex mu;
    static uint32_t known[kMaxDev] = {};
    *mask = 0;
    if (di.device < 0 || di.device >= kMaxDev) return AFSAI_OK;
    std::lock_guard<std::mutex> lk(mu);
    if (!known[di.device]) {
        DevBuf m;
        int rc;
        uint32_t h = 0;
        if ((rc = dalloc(m, sizeof(uint32_t), s))) return rc;
        AFSAI_HIP_TRY(hipMemcpyAsync(m.p, &h, sizeof h, hipMemcpyHostToDevice, s));
        hipLaunchKernelGGL(k_xcc_mask, dim3(di.num_cus * 4), dim3(64), 0, s, m.as<uint32_t>());
        AFSAI_HIP_TRY(hipMemcpyAsync(&h, m.p, sizeof h, hipMemcpyDeviceToHost, s));
        AFSAI_HIP_TRY(hipStreamSynchronize(s));
        known[di.device] = h;
    }
    *mask = known[di.device];
    return AFSAI_OK;
}

// The one-launch solves in flight on each XCD.  Two fit as a whole (pcg_small.hpp), and blocks of a third could keep
// each other and theirs out, so no more than two are let there; a further solve takes the ordinary launches.
// Where blocks did not meet all the same (another process on the device), the next kSmallPause solves of the
// device do not try.  A process's first XCD follows from its number, so that processes start on different ones.
class SmallPlaces {
  public:
    // an XCD of the mask for another solve: of those with the fewest solves the next in turn; -1: none
    int take(uint32_t mask) {
        std::lock_guard<std::mutex> lk(mu_);
        if (pause_ > 0) {
            --pause_;
            return -1;
        }
        int best = -1;
        for (int j = 0; j < 16; ++j) {
            const int x = (int)((turn_ + j) % 16);
            if ((mask >> x & 1) && used_[x] < 2 && (best < 0 || used_[x] < used_[best])) best = x;
        }
        if (best >= 0) {
            ++used_[best];
            turn_ = best + 1;
        }
        return best;
    }
    void give(int x, bool unmet) {
        std::lock_guard<std::mutex> lk(mu_);
        --used_[x];
        if (unmet) pause_ = kSmallPause;
    }

  private:
    std::mutex mu_;
    int used_[16] = {};
    unsigned turn_ = (unsigned)getpid();
    int pause_ = 0;
};
static SmallPlaces g_places[64];  // by device

struct Csr {
    int n = 0;
    int64_t nnz = 0;
    const int32_t *rp = nullptr, *ci = nullptr;
    const void *val = nullptr;
    bool f32 = false;
};

template <int GS, int U, typename VT>
static void launch_spmv_t(const Csr &A, const double *x, double *y, const double *w, double *partials,
                          PcgScalars *sc, int nb, int nxcd, hipStream_t s) {
    if (w)
        hipLaunchKernelGGL((k_spmv<GS, U, VT, true>), dim3(nb), dim3(kThreads), 0, s, A.n, A.rp, A.ci,
                           (const VT *)A.val, x, y, w, partials, sc, nxcd);
    else
        hipLaunchKernelGGL((k_spmv<GS, U, VT, false>), dim3(nb), dim3(kThreads), 0, s, A.n, A.rp, A.ci,
                           (const VT *)A.val, x, y, w, partials, sc, nxcd);
}

template <int GS, typename VT>
static void launch_spmv_u(const Csr &A, int un, const double *x, double *y, const double *w, double *partials,
                          PcgScalars *sc, int nb, int nxcd, hipStream_t s) {
    switch (un) {
        case 1: launch_spmv_t<GS, 1, VT>(A, x, y, w, partials, sc, nb, nxcd, s); break;
        case 2: launch_spmv_t<GS, 2, VT>(A, x, y, w, partials, sc, nb, nxcd, s); break;
        case 4: launch_spmv_t<GS, 4, VT>(A, x, y, w, partials, sc, nb, nxcd, s); break;
        default: launch_spmv_t<GS, 8, VT>(A, x, y, w, partials, sc, nb, nxcd, s); break;
    }
}

template <typename VT>
static void launch_spmv_v(const Csr &A, int gs, int un, const double *x, double *y, const double *w,
                          double *partials, PcgScalars *sc, int nb, int nxcd, hipStream_t s) {
    switch (gs) {
        case 4: launch_spmv_u<4, VT>(A, un, x, y, w, partials, sc, nb, nxcd, s); break;
        case 8: launch_spmv_u<8, VT>(A, un, x, y, w, partials, sc, nb, nxcd, s); break;
        case 16: launch_spmv_u<16, VT>(A, un, x, y, w, partials, sc, nb, nxcd, s); break;
        case 32: launch_spmv_u<32, VT>(A, un, x, y, w, partials, sc, nb, nxcd, s); break;
        default: launch_spmv_u<64, VT>(A, un, x, y, w, partials, sc, nb, nxcd, s); break;
    }
}

// blocks of the CSR product
static int spmv_blocks(const Csr &A, const DeviceInfo &di) {
    int gs, un;
    spmv_shape(A.n ? (double)A.nnz / A.n : 0.0, &gs, &un);
    return blocks_for_rows(A.n, gs, di);
}

// y = A x, CSR (one system; optionally fused dot y.w: one partial sum per block)
static void spmv(const char *name, const Csr &A, const double *x, double *y, const double *w,
                 double *partials, PcgScalars *sc, const DeviceInfo &di, hipStream_t s) {
    const double avg = A.n ? (double)A.nnz / A.n : 0.0;
    int gs, un;
    spmv_shape(avg, &gs, &un);
    const int nb = blocks_for_rows(A.n, gs, di);
    {
        ProfScope ps(name, s);
        if (A.f32)
            launch_spmv_v<float>(A, gs, un, x, y, w, partials, sc, nb, di.num_xcds, s);
        else
            launch_spmv_v<double>(A, gs, un, x, y, w, partials, sc, nb, di.num_xcds, s);
    }
}

// Block maps of a batch for the three launch shapes (SELL products, vector kernels), held on
// the device for one solve; empty for a single system.
struct Shape {
    Map mp;
    int nblocks = 0;
};
struct BatchMaps {
    int nsys = 1;
    Systems sy;
    Shape sell, vec;
    bool nt = true;  // the matrix stream is larger than the caches
    DevBuf buf;
};

static int make_batch_maps(int n, int nsys, const int32_t *row0, const DeviceInfo &di, hipStream_t s,
                           BatchMaps *bm) {
    bm->nsys = nsys;
    std::vector<int32_t> slice0(nsys + 1);
    Segments seg;
    seg.nsys = nsys;
    seg.row0 = row0;
    segment_slices(seg, n, slice0.data());
    if (nsys == 1) {
        bm->sell.nblocks = blocks_for_slices(slice0[1], di);
        bm->vec.nblocks = blocks_for_vec(n, di);
        return AFSAI_OK;
    }
    std::vector<int32_t> nb_sell(nsys), nb_vec(nsys);
    int64_t tot_sell = 0, tot_vec = 0;
    for (int k = 0; k < nsys; ++k) {
        nb_sell[k] = blocks_for_slices(slice0[k + 1] - slice0[k], di);
        nb_vec[k] = blocks_for_vec(row0[k + 1] - row0[k], di);
        tot_sell += nb_sell[k];
        tot_vec += nb_vec[k];
    }
    if (tot_sell >= (1 << 30) || tot_vec >= (1 << 30)) AFSAI_FAIL(AFSAI_ERR_TOO_LARGE, "batch: too many blocks");
    // layout: row0 | slice0 | sell: blk_sys, b0, nb | vec: blk_sys, b0, nb
    std::vector<int32_t> h;
    h.reserve((size_t)2 * (nsys + 1) + tot_sell + tot_vec + 4 * (size_t)nsys);
    h.insert(h.end(), row0, row0 + nsys + 1);
    h.insert(h.end(), slice0.begin(), slice0.end());
    size_t off_sell = h.size();
    for (int k = 0; k < nsys; ++k) h.insert(h.end(), nb_sell[k], k);
    size_t off_sell_b0 = h.size();
    int32_t acc = 0;
    for (int k = 0; k < nsys; ++k) {
        h.push_back(acc);
        acc += nb_sell[k];
    }
    size_t off_sell_nb = h.size();
    h.insert(h.end(), nb_sell.begin(), nb_sell.end());
    size_t off_vec = h.size();
    for (int k = 0; k < nsys; ++k) h.insert(h.end(), nb_vec[k], k);
    size_t off_vec_b0 = h.size();
    acc = 0;
    for (int k = 0; k < nsys; ++k) {
        h.push_back(acc);
        acc += nb_vec[k];
    }
    size_t off_vec_nb = h.size();
    h.insert(h.end(), nb_vec.begin(), nb_vec.end());
    int rc;
    if ((rc = dalloc(bm->buf, sizeof(int32_t) * h.size(), s))) return rc;
    AFSAI_HIP_TRY(hipMemcpyAsync(bm->buf.p, h.data(), sizeof(int32_t) * h.size(), hipMemcpyHostToDevice, s));
    AFSAI_HIP_TRY(hipStreamSynchronize(s));
    const int32_t *d = bm->buf.as<int32_t>();
    bm->sy.row0 = d;
    bm->sy.slice0 = d + nsys + 1;
    bm->sell.mp = Map{d + off_sell, d + off_sell_b0, d + off_sell_nb};
    bm->sell.nblocks = (int)tot_sell;
    bm->vec.mp = Map{d + off_vec, d + off_vec_b0, d + off_vec_nb};
    bm->vec.nblocks = (int)tot_vec;
    return AFSAI_OK;
}

// fused: a split layout's tail runs inside the slices' product (else the caller launched it)
template <int U, bool NT, typename VT>
static void launch_sell_t(const Sell &S, const double *x, double *y, const double *w, double *partials,
                          PcgScalars *scs, const Map &mp, const Systems &sy, int nb, int nxcd, hipStream_t s,
                          bool fused, const double *rr, double *ww) {
    const Sell *T = fused ? S.tail : nullptr;
    const uint32_t *tsp = T ? T->sptr : nullptr;
    const int32_t *tcl = T ? T->col : nullptr;
    const VT *tvl = T ? (const VT *)T->val : nullptr;
    const int32_t *tof = T ? S.toff : nullptr;
    if (S.col3) {
        // runs of three: about as many entries in flight as U
        constexpr int UR = U >= 8 ? 3 : 1;
        if (w)
            hipLaunchKernelGGL((k_sell_spmv_runs<UR, VT, true, NT>), dim3(nb), dim3(kThreads), 0, s, S.n, S.sptr,
                               S.srow0, S.col3, (const VT *)S.val, x, y, w, partials, scs, mp, sy, S.nslices, nxcd);
        else
            hipLaunchKernelGGL((k_sell_spmv_runs<UR, VT, false, NT>), dim3(nb), dim3(kThreads), 0, s, S.n, S.sptr,
                               S.srow0, S.col3, (const VT *)S.val, x, y, w, partials, scs, mp, sy, S.nslices, nxcd);
        return;
    }
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(nb), dim3(kThreads), 0, s, S.n, S.nslices, S.sptr, S.srow0, S.perm, S.rowmap, S.init,
                           S.col, (const VT *)S.val, x, y, w, partials, scs, mp, sy, nxcd, S.lens, S.wsl, S.wofs, tsp, tcl,
                           tvl, tof, rr, ww);
    };
    if (S.lens) {
        if (ww) go(k_sell_spmv<U, VT, 2, NT, true>);
        else if (w) go(k_sell_spmv<U, VT, 1, NT, true>);
        else go(k_sell_spmv<U, VT, 0, NT, true>);
    } else {
        if (ww) go(k_sell_spmv<U, VT, 2, NT>);
        else if (w) go(k_sell_spmv<U, VT, 1, NT>);
        else go(k_sell_spmv<U, VT, 0, NT>);
    }
}

// nt: non-temporal loads of the matrix (always with the unrolls of 1 and 2).  Also for few slices of long rows, whose
// vectors the ordinary loads drive out: 130,000 rows of 301 entries, a solve of 60 iterations 7.99, 7.09 ms; 60,000 of 601
// 7.66, 7.04
template <typename VT>
static void launch_sell_v(const Sell &S, int un, bool nt, const double *x, double *y, const double *w, double *partials,
                          PcgScalars *scs, const Map &mp, const Systems &sy, int nb, int nxcd, hipStream_t s,
                          bool fused = false, const double *rr = nullptr, double *ww = nullptr) {
    switch (un) {
        case 1: launch_sell_t<1, true, VT>(S, x, y, w, partials, scs, mp, sy, nb, nxcd, s, fused, rr, ww); break;
        case 2: launch_sell_t<2, true, VT>(S, x, y, w, partials, scs, mp, sy, nb, nxcd, s, fused, rr, ww); break;
        case 4:
            if (nt) launch_sell_t<4, true, VT>(S, x, y, w, partials, scs, mp, sy, nb, nxcd, s, fused, rr, ww);
            else launch_sell_t<4, false, VT>(S, x, y, w, partials, scs, mp, sy, nb, nxcd, s, fused, rr, ww);
            break;
        case 16:
            if (nt) launch_sell_t<16, true, VT>(S, x, y, w, partials, scs, mp, sy, nb, nxcd, s, fused, rr, ww);
            else launch_sell_t<16, false, VT>(S, x, y, w, partials, scs, mp, sy, nb, nxcd, s, fused, rr, ww);
            break;
        default:
            if (nt) launch_sell_t<8, true, VT>(S, x, y, w, partials, scs, mp, sy, nb, nxcd, s, fused, rr, ww);
            else launch_sell_t<8, false, VT>(S, x, y, w, partials, scs, mp, sy, nb, nxcd, s, fused, rr, ww);
            break;
    }
}

// Entries in flight per lane of a SELL product: 8 (16 in the length-ordered instance), or 4
// for matrices of at most 8 stored entries per row on average, whose lanes finish within one
// or two rounds anyway and gain more from the resident wavefronts the smaller register budget
// allows (a batch of short 7-point systems: its PCG 27.9 -> 25.0 ms).  Twice as many where there
// are at most two slices per SIMD: nothing else covers a round trip there (24,000 rows of 81
// entries: 52.5 -> 45.4 us an iteration, 107,811 rows 68 -> 64, 64,000 rows of 7 24.8 -> 22.4; the
// registers of 16 would cost the larger ones their second wavefront).  The sums do not depend on it.
static int sell_unroll(const Sell &S, const DeviceInfo &di) {
    if (option(AFSAI_OPT_SPMV_UNROLL) > 0) return (int)option(AFSAI_OPT_SPMV_UNROLL);
    const bool few = S.nslices <= 8 * di.num_cus;
    return ((S.n > 0 && S.entries <= 8 * (int64_t)S.n) ? 4 : 8) * (few ? 2 : 1);
}

// Matrix bytes of an iteration that the 256 MB memory-side cache still holds in the next one: up to
// there ordinary loads, else non-temporal ones.  Microseconds an iteration, ordinary and
// non-temporal: 78 MB 49.8, 53.6; 140 MB 66.7, 74.1; 227 MB 97.7, 98.7; 274 MB 92.3, 92.6; 403 MB
// 161.7, 152.1; 476 MB 147, 133; 1137 MB 285, 248.  Block products, K = 8, 143 MB of matrix: 67, 85 us;
// 478 MB: 200, 193.
constexpr int64_t kCachedBytes = (int64_t)256 << 20;
static int64_t stream_bytes(const Sell &S) { return S.entries * (4 + (S.f32 ? 4 : 8)); }

// y = S x for a SELL-64 matrix laid out for the batch (optionally fused dot y.w, and w.w with ww: one partial sum
// per block, finalised into the systems' scalars when fin says so); a split layout's tail is multiplied first
static void sell_spmv(const char *name, const Sell &S, const BatchMaps &bm, const double *x, double *y,
                      const double *w, double *partials, PcgScalars *scs, int fin, const DeviceInfo &di,
                      hipStream_t s, const double *rr = nullptr, double *ww = nullptr) {
    const int un = sell_unroll(S, di);
    // a split layout's tail runs in a launch of its own first; inside the slices' product when
    // asked for (measured slower: the lanes of long rows serialise their tails while the rest of
    // the wavefront waits)
    const bool fused = S.tail && S.toff && option(AFSAI_OPT_SELL_TAIL) == 1;
    if (S.tail && !fused) {
        const Sell &T = *S.tail;
        const int nbt = blocks_for_slices(T.nslices, di);
        // the tail's rows belong to any system: with one system it stops with it
        PcgScalars *tsc = (bm.nsys == 1) ? scs : nullptr;
        ProfScope ps("sell_tail", s);
        if (T.f32)
            launch_sell_v<float>(T, sell_unroll(T, di), bm.nt, x, y, nullptr, nullptr, tsc, Map(), Systems(), nbt, di.num_xcds, s);
        else
            launch_sell_v<double>(T, sell_unroll(T, di), bm.nt, x, y, nullptr, nullptr, tsc, Map(), Systems(), nbt, di.num_xcds,
                                  s);
    }
    const int nb = bm.sell.nblocks;
    {
        ProfScope ps(name, s);
        if (S.f32)
            launch_sell_v<float>(S, un, bm.nt, x, y, w, partials, scs, bm.sell.mp, bm.sy, nb, di.num_xcds, s, fused, rr, ww);
        else
            launch_sell_v<double>(S, un, bm.nt, x, y, w, partials, scs, bm.sell.mp, bm.sy, nb, di.num_xcds, s, fused, rr, ww);
    }
    if (w && fin != FIN_NONE)
        hipLaunchKernelGGL(k_finalize, dim3(bm.nsys), dim3(kThreads), 0, s, Parts{partials, bm.sell.mp, nb}, Parts(), fin,
                           scs);
}

// the scalars a fused product reads and writes
struct FusedScal {
    const PcgScalars *in = nullptr;
    PcgScalars *out = nullptr;
    int32_t *bad = nullptr;
    Parts pa, pb;
};

template <int U, bool NT, typename VT, int MODE>
static void launch_fused_t(const Sell &S, const double *va, const double *vb, double *own, double *x,
                           const double *pn, double *y, double *partials, const FusedScal &fs, int first,
                           const BatchMaps &bm, int nxcd, hipStream_t s) {
    hipLaunchKernelGGL((k_sell_fused<U, VT, MODE, NT>), dim3(bm.sell.nblocks), dim3(kThreads), 0, s, S.n, S.nslices,
                       S.sptr, S.srow0, S.col, (const VT *)S.val, va, vb, own, x, pn, y, partials, fs.in, fs.out, fs.bad,
                       fs.pa, fs.pb, first, bm.sell.mp, bm.sy, nxcd);
}

template <typename VT, int MODE>
static void launch_fused_v(const Sell &S, int un, const double *va, const double *vb, double *own, double *x,
                           const double *pn, double *y, double *partials, const FusedScal &fs, int first,
                           const BatchMaps &bm, int nxcd, hipStream_t s) {
    switch (un) {
        case 1: launch_fused_t<1, true, VT, MODE>(S, va, vb, own, x, pn, y, partials, fs, first, bm, nxcd, s); break;
        case 2: launch_fused_t<2, true, VT, MODE>(S, va, vb, own, x, pn, y, partials, fs, first, bm, nxcd, s); break;
        case 4:
            if (bm.nt) launch_fused_t<4, true, VT, MODE>(S, va, vb, own, x, pn, y, partials, fs, first, bm, nxcd, s);
            else launch_fused_t<4, false, VT, MODE>(S, va, vb, own, x, pn, y, partials, fs, first, bm, nxcd, s);
            break;
        case 16:
            if (bm.nt) launch_fused_t<16, true, VT, MODE>(S, va, vb, own, x, pn, y, partials, fs, first, bm, nxcd, s);
            else launch_fused_t<16, false, VT, MODE>(S, va, vb, own, x, pn, y, partials, fs, first, bm, nxcd, s);
            break;
        default:
            if (bm.nt) launch_fused_t<8, true, VT, MODE>(S, va, vb, own, x, pn, y, partials, fs, first, bm, nxcd, s);
            else launch_fused_t<8, false, VT, MODE>(S, va, vb, own, x, pn, y, partials, fs, first, bm, nxcd, s);
            break;
    }
}

template <int MODE>
static void sell_fused(const char *name, const Sell &S, const BatchMaps &bm, const double *va, const double *vb,
                       double *own, double *x, const double *pn, double *y, double *partials, const FusedScal &fs,
                       int first, const DeviceInfo &di, hipStream_t s) {
    const int un = sell_unroll(S, di);
    ProfScope ps(name, s);
    if (S.f32)
        launch_fused_v<float, MODE>(S, un, va, vb, own, x, pn, y, partials, fs, first, bm, di.num_xcds, s);
    else
        launch_fused_v<double, MODE>(S, un, va, vb, own, x, pn, y, partials, fs, first, bm, di.num_xcds, s);
}

struct MultiScal {
    double bb, rho, alpha, beta, rr, tr;
    int32_t done, iters, status, pad;
};

// every column of the block has stopped (sc null: there are no columns to ask)
template <int K>
__device__ __forceinline__ bool all_stopped(const MultiScal *sc) {
    if (!sc) return false;
    int done = 1;
#pragma unroll
    for (int j = 0; j < K; ++j) done &= sc[j].done;
    return done != 0;
}

// Y = A X for K vectors stored row by row (entry (i, j) at i * K + j): one wavefront per
// SELL-64 slice, one lane per row; every matrix entry is read once for the K vectors and the
// K values of a gathered row are contiguous.  Each output is the same sequential chain over
// the row's entries as in the single-vector product.  sc given: nothing is done when every column
// has stopped.
template <int K, typename VT, bool DOT, bool NT>
__global__ __launch_bounds__(kThreads) void k_sell_spmm(int n, int nslices, const uint32_t *__restrict__ sptr,
                                                         const int32_t *__restrict__ perm,
                                                         const int32_t *__restrict__ lens,
                                                         const int32_t *__restrict__ col,
                                                         const VT *__restrict__ val, const double *__restrict__ x,
                                                         double *__restrict__ y, int nxcd,
                                                         const double *__restrict__ w, double *__restrict__ partials,
                                                         const MultiScal *sc) {
    if (all_stopped<K>(sc)) return;
    constexpr int U = K <= 2 ? 8 : 4;  // entries in flight per lane (fewer for wide blocks: registers)
    __shared__ double sh[kThreads / 64];
    double part[K];
#pragma unroll
    for (int j = 0; j < K; ++j) part[j] = 0.0;
    const int lb = xcd_block(blockIdx.x, gridDim.x, nxcd);
    const int wv = wave_index(), lane = threadIdx.x & 63;
    int w0, w1, wstep;
    window_walk((nslices + kWin - 1) / kWin, lb, gridDim.x, nxcd, w0, w1, wstep);
    for (int wi = w0; wi < w1; wi += wstep) {
        const int sl = wi * kWin + wv;
        if (sl >= nslices) break;
        const uint32_t c0 = sptr[sl];
        int r = sl * kSlice + lane;
        bool valid = r < n;
        int len = (int)(sptr[sl + 1] - c0);
        if (lens) {
            r = perm[(int64_t)sl * kSlice + lane];
            len = lens[(int64_t)sl * kSlice + lane];
            valid = r >= 0;
        }
        const int64_t base = (int64_t)c0 * kSlice + lane;
        double acc[K];
#pragma unroll
        for (int j = 0; j < K; ++j) acc[j] = 0.0;
        // software pipeline as in lane_chain: the next U columns and values are loaded before
        // the current gathers
        int c[U];
        VT v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            c[u] = 0;
            v[u] = VT(0);
            if (u < len) {
                const int64_t d = base + (int64_t)u * kSlice;
                c[u] = ldm<NT>(&col[d]);
                v[u] = ldm<NT>(&val[d]);
            }
        }
        for (int k0 = 0; k0 < len; k0 += U) {
            int cn[U];
            VT vn[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                cn[u] = 0;
                vn[u] = VT(0);
                if (k0 + U + u < len) {
                    const int64_t d = base + (int64_t)(k0 + U + u) * kSlice;
                    cn[u] = ldm<NT>(&col[d]);
                    vn[u] = ldm<NT>(&val[d]);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (k0 + u < len) {
                    const double *xc = x + (int64_t)c[u] * K;
#pragma unroll
                    for (int j = 0; j < K; ++j) acc[j] = fma((double)v[u], xc[j], acc[j]);
                }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                c[u] = cn[u];
                v[u] = vn[u];
            }
        }
        if (valid) {
#pragma unroll
            for (int j = 0; j < K; ++j) {
                y[(int64_t)r * K + j] = acc[j];
                if (DOT) part[j] = fma(acc[j], w[(int64_t)r * K + j], part[j]);
            }
        }
    }
    if (DOT) {
        // per column j: this block's partial sum at partials[j * gridDim.x + lb]
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const double bs = block_sum(part[j], sh);
            if (threadIdx.x == 0) partials[(size_t)j * gridDim.x + lb] = bs;
        }
    }
}

// Block product over the layout with one column index per run of three (plain layouts: no
// length ordering): a lane reads a run's index and its three values and the 3K consecutive
// entries of X's rows c..c+2; per column the sum is the same chain over the entries in stored
// order as k_sell_spmm's, so Y and the partial sums are identical to it bit for bit.
template <int K, bool DOT, bool NT>
__global__ __launch_bounds__(kThreads) void k_sell_spmm_runs(int n, int nslices, const uint32_t *__restrict__ sptr,
                                                              const int32_t *__restrict__ col3,
                                                              const double *__restrict__ val,
                                                              const double *__restrict__ x, double *__restrict__ y,
                                                              int nxcd, const double *__restrict__ w,
                                                              double *__restrict__ partials, const MultiScal *sc) {
    if (all_stopped<K>(sc)) return;
    constexpr int UR = K <= 2 ? 3 : 1;  // runs in flight per lane (9 or 3 entries)
    __shared__ double sh[kThreads / 64];
    double part[K];
#pragma unroll
    for (int j = 0; j < K; ++j) part[j] = 0.0;
    const int lb = xcd_block(blockIdx.x, gridDim.x, nxcd);
    const int wv = wave_index(), lane = threadIdx.x & 63;
    int w0, w1, wstep;
    window_walk((nslices + kWin - 1) / kWin, lb, gridDim.x, nxcd, w0, w1, wstep);
    for (int wi = w0; wi < w1; wi += wstep) {
        const int sl = wi * kWin + wv;
        if (sl >= nslices) break;
        const uint32_t c0 = sptr[sl];
        const int r = sl * kSlice + lane;
        const int nr = (int)(sptr[sl + 1] - c0) / 3;
        const int64_t rbase = (int64_t)(c0 / 3u) * kSlice + lane, vbase = (int64_t)c0 * kSlice + lane;
        double acc[K];
#pragma unroll
        for (int j = 0; j < K; ++j) acc[j] = 0.0;
        int c[UR];
        double v[UR][3];
#pragma unroll
        for (int u = 0; u < UR; ++u) {
            c[u] = 0;
#pragma unroll
            for (int e = 0; e < 3; ++e) v[u][e] = 0.0;
            if (u < nr) {
                c[u] = ldm<NT>(&col3[rbase + (int64_t)u * kSlice]);
#pragma unroll
                for (int e = 0; e < 3; ++e) v[u][e] = ldm<NT>(&val[vbase + (int64_t)(3 * u + e) * kSlice]);
            }
        }
        for (int j0 = 0; j0 < nr; j0 += UR) {
            int cn[UR];
            double vn[UR][3];
#pragma unroll
            for (int u = 0; u < UR; ++u) {
                cn[u] = 0;
#pragma unroll
                for (int e = 0; e < 3; ++e) vn[u][e] = 0.0;
                if (j0 + UR + u < nr) {
                    const int jr = j0 + UR + u;
                    cn[u] = ldm<NT>(&col3[rbase + (int64_t)jr * kSlice]);
#pragma unroll
                    for (int e = 0; e < 3; ++e)
                        vn[u][e] = ldm<NT>(&val[vbase + (int64_t)(3 * jr + e) * kSlice]);
                }
            }
#pragma unroll
            for (int u = 0; u < UR; ++u)
                if (j0 + u < nr) {
                    const double *xc = x + (int64_t)c[u] * K;
#pragma unroll
                    for (int e = 0; e < 3; ++e)
#pragma unroll
                        for (int j = 0; j < K; ++j) acc[j] = fma(v[u][e], xc[e * K + j], acc[j]);
                }
#pragma unroll
            for (int u = 0; u < UR; ++u) {
                c[u] = cn[u];
#pragma unroll
                for (int e = 0; e < 3; ++e) v[u][e] = vn[u][e];
            }
        }
        if (r < n) {
#pragma unroll
            for (int j = 0; j < K; ++j) {
                y[(int64_t)r * K + j] = acc[j];
                if (DOT) part[j] = fma(acc[j], w[(int64_t)r * K + j], part[j]);
            }
        }
    }
    if (DOT) {
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const double bs = block_sum(part[j], sh);
            if (threadIdx.x == 0) partials[(size_t)j * gridDim.x + lb] = bs;
        }
    }
}

// Block product over A in 3 x 3 blocks (sell_node_blocks): a lane takes the three rows of a node (L
// lanes share a node, K / L columns each), so that one gathered block row of X serves nine
// entries.  The products with a lane per row are bound by the bytes the L1 returns: 64 gathered
// bytes per entry for K = 8; here 21, and 8.4 bytes of matrix instead of 9.3 or 12.  K = 8 at 680,943
// rows (54 M entries): 231 -> 187 us, 2.5 TB/s of matrix; L = 1 spills and L = 4 takes 249 us (the
// columns and values come four times); four lanes on one row with two columns each, 423 us.  Per
// column and row the sum is the chain of k_sell_spmm_runs: Y is identical bit for bit.
template <int K, int L, bool NT>
__global__ __launch_bounds__(kThreads) void k_node_spmm(int n, int nslices, const uint32_t *__restrict__ bptr,
                                                        const int32_t *__restrict__ bcol,
                                                        const double *__restrict__ bval, const double *__restrict__ x,
                                                        double *__restrict__ y, int nxcd, const MultiScal *sc) {
    constexpr int C = K / L;
    if (all_stopped<K>(sc)) return;
    const int lb = xcd_block(blockIdx.x, gridDim.x, nxcd);
    const int wv = wave_index(), lane = threadIdx.x & 63;
    int w0, w1, wstep;
    window_walk((nslices * L + kWin - 1) / kWin, lb, gridDim.x, nxcd, w0, w1, wstep);
    for (int wi = w0; wi < w1; wi += wstep) {
        const int unit = wi * kWin + wv, sl = unit / L;
        if (sl >= nslices) break;
        const int l = (unit % L) * (64 / L) + lane / L;  // node of the slice
        const int r = 3 * (sl * kSlice + l);
        const int b0 = (int)bptr[sl], b1 = (int)bptr[sl + 1];
        const double *xj = x + (lane % L) * C;
        double acc[3][C];
#pragma unroll
        for (int d = 0; d < 3; ++d)
#pragma unroll
            for (int j = 0; j < C; ++j) acc[d][j] = 0.0;
        // the next block's index and values are loaded behind this one's gathers
        int c = 0, cn;
        double v[9], vn[9];
        if (b0 < b1) {
            c = ldm<NT>(&bcol[(int64_t)b0 * kSlice + l]);
#pragma unroll
            for (int q = 0; q < 9; ++q) v[q] = ldm<NT>(&bval[((int64_t)b0 * 9 + q) * kSlice + l]);
        }
        cn = c;
        for (int b = b0; b < b1; ++b) {
            const double *xc = xj + (int64_t)(c < 0 ? 0 : c) * K;
            double xv[3][C];
#pragma unroll
            for (int e = 0; e < 3; ++e)
#pragma unroll
                for (int j = 0; j < C; ++j) xv[e][j] = xc[e * K + j];
            if (b + 1 < b1) {
                cn = ldm<NT>(&bcol[(int64_t)(b + 1) * kSlice + l]);
#pragma unroll
                for (int q = 0; q < 9; ++q) vn[q] = ldm<NT>(&bval[((int64_t)(b + 1) * 9 + q) * kSlice + l]);
            }
            if (c >= 0) {
#pragma unroll
                for (int e = 0; e < 3; ++e)
#pragma unroll
                    for (int d = 0; d < 3; ++d)
#pragma unroll
                        for (int j = 0; j < C; ++j) acc[d][j] = fma(v[3 * d + e], xv[e][j], acc[d][j]);
            }
            c = cn;
#pragma unroll
            for (int q = 0; q < 9; ++q) v[q] = vn[q];
        }
        // the zeros times x that the rows' plain slices hold (k_node_fill)
        if (c < -1)
#pragma unroll
            for (int d = 0; d < 3; ++d)
                if ((-1 - c) >> d & 1)
#pragma unroll
                    for (int j = 0; j < C; ++j) acc[d][j] = fma(0.0, xj[(int64_t)(r + d) * K + j], acc[d][j]);
        if (r < n)
#pragma unroll
            for (int d = 0; d < 3; ++d)
#pragma unroll
                for (int j = 0; j < C; ++j) y[(int64_t)(r + d) * K + (lane % L) * C + j] = acc[d][j];
    }
}

// per column the partial sums of y.w over the windows of 256 rows, in the order of k_sell_spmm's dots
template <int K>
__global__ __launch_bounds__(kThreads) void k_window_dot(int n, int nslices, const double *__restrict__ y,
                                                         const double *__restrict__ w, double *__restrict__ partials,
                                                         int nxcd, const MultiScal *sc) {
    __shared__ double sh[kThreads / 64];
    if (all_stopped<K>(sc)) return;
    double part[K];
#pragma unroll
    for (int j = 0; j < K; ++j) part[j] = 0.0;
    const int lb = xcd_block(blockIdx.x, gridDim.x, nxcd);
    int w0, w1, wstep;
    window_walk((nslices + kWin - 1) / kWin, lb, gridDim.x, nxcd, w0, w1, wstep);
    for (int wi = w0; wi < w1; wi += wstep) {
        const int r = wi * kWin * kSlice + threadIdx.x;
        if (r < n)
#pragma unroll
            for (int j = 0; j < K; ++j) part[j] = fma(y[(int64_t)r * K + j], w[(int64_t)r * K + j], part[j]);
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const double bs = block_sum(part[j], sh);
        if (threadIdx.x == 0) partials[(size_t)j * gridDim.x + lb] = bs;
    }
}

// ---------------------------------------------------------------------------------------
// PCG over a block of K right-hand sides (x0 = 0): K independent recurrences with their own
// scalars and stopping tests; the vectors are n x K row-major blocks and every product reads
// its matrix once for the K columns.
// ---------------------------------------------------------------------------------------
enum : int { MF_BB = 0, MF_RHO0 = 1, MF_PQ = 2, MF_RR = 3, MF_RZ = 4, MF_TRUE = 5 };

// the columns' scalars into pinned host memory
__global__ void k_multi_publish(int k, const MultiScal *__restrict__ sc, MultiScal *__restrict__ host) {
    if ((int)threadIdx.x < k) host[threadIdx.x] = sc[threadIdx.x];
}

// One block per column: the column's partial sums (nb per column) added in block order, then
// the scalar step of the textbook recurrence for that column.
__global__ __launch_bounds__(kThreads) void k_fin_multi(const double *__restrict__ partials, int nb, int mode,
                                                         double rtol, int maxit, MultiScal *sc) {
    __shared__ double sh[kThreads / 64];
    const int j = blockIdx.x;
    const int per = (nb + kThreads - 1) / kThreads;
    const int lo = threadIdx.x * per, hi = min(nb, lo + per);
    double v = 0.0;
    for (int b = lo; b < hi; ++b) v += partials[(size_t)j * nb + b];
    const double t = block_sum(v, sh);
    if (threadIdx.x != 0) return;
    MultiScal &m = sc[j];
    switch (mode) {
        case MF_BB:
            m.bb = t;
            m.rr = t;
            m.iters = 0;
            m.done = 0;
            m.status = AFSAI_ERR_NOT_CONVERGED;
            if (t == 0.0 || sqrt(t) <= rtol * sqrt(t)) {
                m.done = 1;  // b = 0 (x = 0) or converged at x0
                m.status = AFSAI_OK;
            } else if (maxit <= 0) {
                m.done = 1;
            }
            break;
        case MF_RHO0: m.rho = t; break;
        case MF_PQ:
            if (!m.done) {
                if (!(t > 0.0)) {
                    m.done = 1;
                    m.status = AFSAI_ERR_NOT_SPD;
                } else {
                    m.alpha = m.rho / t;
                }
            }
            break;
        case MF_RR:
            if (!m.done) {
                m.rr = t;
                m.iters += 1;
                if (sqrt(t) <= rtol * sqrt(m.bb)) {
                    m.done = 1;
                    m.status = AFSAI_OK;
                } else if (m.iters >= maxit) {
                    m.done = 1;
                }
            }
            break;
        case MF_RZ:
            if (!m.done) {
                m.beta = t / m.rho;
                m.rho = t;
            }
            break;
        default: m.tr = t; break;
    }
}

// The vector kernels take one thread per entry of the n x K block: block b covers the
// entries of rows [i0, i1) (contiguous, in block order) and, since kThreads is a multiple of
// K, thread t always meets column t % K, so every thread sums one column in a fixed order.
template <int K>
__device__ __forceinline__ void multi_range(int n, int64_t &e0, int64_t &e1) {
    int i0, i1;
    block_range(0, n, blockIdx.x, gridDim.x, i0, i1);
    e0 = (int64_t)i0 * K;
    e1 = (int64_t)i1 * K;
}

// this block's per-column sums of part (thread t holding column t % K) at
// partials[j * gridDim.x + block]: lanes of one column added by shuffles, then the
// wavefronts in order
template <int K>
__device__ __forceinline__ void multi_store(double part, double *sh /* kThreads / 64 * K */, double *partials) {
    static_assert(kThreads % K == 0 && 64 % K == 0, "a thread keeps one column");
#pragma unroll
    for (int off = 32; off >= K; off >>= 1) part += __shfl_xor(part, off, 64);
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane < K) sh[w * K + lane] = part;
    __syncthreads();
    if (threadIdx.x < K) {
        double t = 0.0;
        for (int k = 0; k < kThreads / 64; ++k) t += sh[k * K + threadIdx.x];
        partials[(size_t)threadIdx.x * gridDim.x + blockIdx.x] = t;
    }
}

// x = 0, r = b; partial sums of b.b per column
template <int K>
__global__ __launch_bounds__(kThreads) void k_multi_init(int n, const double *__restrict__ b, double *__restrict__ x,
                                                          double *__restrict__ r, double *__restrict__ partials) {
    __shared__ double sh[kThreads / 64 * K];
    int64_t e0, e1;
    multi_range<K>(n, e0, e1);
    double part = 0.0;
    for (int64_t e = e0 + threadIdx.x; e < e1; e += kThreads) {
        const double be = b[e];
        x[e] = 0.0;
        r[e] = be;
        part = fma(be, be, part);
    }
    multi_store<K>(part, sh, partials);
}

// partial sums of a.b per column (and copy = a when given)
template <int K>
__global__ __launch_bounds__(kThreads) void k_multi_dot(int n, const double *__restrict__ a, const double *__restrict__ b,
                                                         double *__restrict__ copy, double *__restrict__ partials) {
    __shared__ double sh[kThreads / 64 * K];
    int64_t e0, e1;
    multi_range<K>(n, e0, e1);
    double part = 0.0;
    for (int64_t e = e0 + threadIdx.x; e < e1; e += kThreads) {
        const double ae = a[e];
        if (copy) copy[e] = ae;
        part = fma(ae, b[e], part);
    }
    multi_store<K>(part, sh, partials);
}

// columns still running: x += alpha p, r -= alpha q; partial sums of r.r per column
template <int K>
__global__ __launch_bounds__(kThreads) void k_multi_xr(int n, double *__restrict__ x, double *__restrict__ r,
                                                        const double *__restrict__ p, const double *__restrict__ q,
                                                        const MultiScal *__restrict__ sc, double *__restrict__ partials) {
    __shared__ double sh[kThreads / 64 * K];
    if (all_stopped<K>(sc)) return;
    int64_t e0, e1;
    multi_range<K>(n, e0, e1);
    const int j = threadIdx.x % K;
    const bool run = !sc[j].done;
    const double alpha = sc[j].alpha;
    double part = 0.0;
    for (int64_t e = e0 + threadIdx.x; e < e1; e += kThreads) {
        double re = r[e];
        if (run) {
            x[e] = fma(alpha, p[e], x[e]);
            re = fma(-alpha, q[e], re);
            r[e] = re;
        }
        part = fma(re, re, part);
    }
    multi_store<K>(part, sh, partials);
}

// columns still running: p = z + beta p
template <int K>
__global__ __launch_bounds__(kThreads) void k_multi_p(int n, const double *__restrict__ z, double *__restrict__ p,
                                                       const MultiScal *__restrict__ sc) {
    int64_t e0, e1;
    multi_range<K>(n, e0, e1);
    const int j = threadIdx.x % K;
    if (sc[j].done) return;
    const double beta = sc[j].beta;
    for (int64_t e = e0 + threadIdx.x; e < e1; e += kThreads) p[e] = fma(beta, p[e], z[e]);
}

// partial sums of (b - q).(b - q) per column
template <int K>
__global__ __launch_bounds__(kThreads) void k_multi_resid(int n, const double *__restrict__ b,
                                                           const double *__restrict__ q, double *__restrict__ partials) {
    __shared__ double sh[kThreads / 64 * K];
    int64_t e0, e1;
    multi_range<K>(n, e0, e1);
    double part = 0.0;
    for (int64_t e = e0 + threadIdx.x; e < e1; e += kThreads) {
        const double d = b[e] - q[e];
        part = fma(d, d, part);
    }
    multi_store<K>(part, sh, partials);
}

// Whether the block form is the faster one.  Up to four columns its wavefronts, a third as many, only wait longer
// while the form with a row to a lane has all its windows on the CUs at once: `windows` of them to each (1: 65,536 rows
// here).  Calls of the prepared product, microseconds with blocks and without: K = 1, 52,728 rows 31.8, 28.3; 98,304 rows
// 32.4, 33.2; K = 2 32.6, 28.3; 33.4, 33.6; K = 4 35.0, 34.6; 36.0, 38.6; K = 8, 1,536 rows 30.4, 35.7.
// pcg_solve_multi, which also converts the matrix, milliseconds (2 windows): K = 1, 98,304 rows 3.96, 3.82; 192,000 rows 6.12,
// 6.60; K = 4 5.44, 5.42; 9.10, 9.95.
static bool blocks_pay(int K, int n, int windows, const DeviceInfo &di) {
    return K > 4 || n / (kSlice * kWin) >= windows * di.num_cus;
}

// nt: non-temporal loads of the matrix
template <int K, bool DOT, bool NT>
static void spmm_launch_t(const Sell &S, const double *x, double *y, const double *w, double *partials, int nb,
                          const DeviceInfo &di, hipStream_t s, const MultiScal *sc) {
    const dim3 bt(kThreads);
    if (S.bptr && (!S.val || blocks_pay(K, S.n, 1, di))) {
        constexpr int L = K >= 8 ? 2 : 1;
        const int nsl = (S.n / 3 + kSlice - 1) / kSlice;
        hipLaunchKernelGGL((k_node_spmm<K, L, NT>), dim3(blocks_for_slices(nsl * L, di)), bt, 0, s, S.n, nsl, S.bptr,
                           S.bcol, S.bval, x, y, di.num_xcds, sc);
        if (DOT)
            hipLaunchKernelGGL((k_window_dot<K>), dim3(nb), bt, 0, s, S.n, (S.n + kSlice - 1) / kSlice, y, w, partials,
                               di.num_xcds, sc);
    } else if (S.col3 && !S.f32 && !S.lens)
        hipLaunchKernelGGL((k_sell_spmm_runs<K, DOT, NT>), dim3(nb), bt, 0, s, S.n, S.nslices, S.sptr, S.col3,
                           (const double *)S.val, x, y, di.num_xcds, w, partials, sc);
    else if (S.f32)
        hipLaunchKernelGGL((k_sell_spmm<K, float, DOT, NT>), dim3(nb), bt, 0, s, S.n, S.nslices, S.sptr, S.perm, S.lens,
                           S.col, (const float *)S.val, x, y, di.num_xcds, w, partials, sc);
    else
        hipLaunchKernelGGL((k_sell_spmm<K, double, DOT, NT>), dim3(nb), bt, 0, s, S.n, S.nslices, S.sptr, S.perm, S.lens,
                           S.col, (const double *)S.val, x, y, di.num_xcds, w, partials, sc);
}

template <int K, bool DOT>
static void spmm_launch(const Sell &S, bool nt, const double *x, double *y, const double *w, double *partials, int nb,
                        const DeviceInfo &di, hipStream_t s, const MultiScal *sc = nullptr) {
    if (nt) spmm_launch_t<K, DOT, true>(S, x, y, w, partials, nb, di, s, sc);
    else spmm_launch_t<K, DOT, false>(S, x, y, w, partials, nb, di, s, sc);
}

static int check_csr_arg(const afsai_csr *A, const char *who) {
    if (!A) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "%s: A is NULL", who);
    if (A->n <= 0 || A->nnz < A->n) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "%s: n = %d, nnz = %d", who, A->n, A->nnz);
    if (!A->row_ptr || !A->col_idx || !A->val) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "%s: null CSR array", who);
    return AFSAI_OK;
}

static Csr csr_of(const afsai_csr *A) {
    Csr c;
    c.n = A->n;
    c.nnz = A->nnz;
    c.rp = A->row_ptr;
    c.ci = A->col_idx;
    c.val = A->val;
    return c;
}

// work vectors of the solver: r, r', z, p, p', q, t
constexpr int kWorkVectors = 7;

// A solve in progress: PCG (Sec. 5.2) over a batch of nsys independent systems (row0: host,
// nsys + 1 entries; one system when nsys == 1).  begin() enqueues the start and two chunks of
// iterations; advance() reads the state after the oldest chunk in flight (waiting for it when
// `block`, else returning at once if it is not there yet) and enqueues the next chunk, sized from
// the slowest system's convergence rate so that few iterations are queued past convergence
// (those return at once on the device flags); finish() computes the true residuals and the
// results.  All work goes to one stream; any number of runs may be in progress on different
// streams (the serving loop advances many of them from one host thread).
// A stream per thread and device on which iterations are captured into graphs (never run).
static hipStream_t capture_stream(int device) {
    struct Streams {
        hipStream_t s[64] = {};
        ~Streams() {
            for (hipStream_t &x : s)
                if (x) (void)hipStreamDestroy(x);
        }
    };
    thread_local Streams ts;
    if (device < 0 || device >= 64) return nullptr;
    if (!ts.s[device] && hipStreamCreateWithFlags(&ts.s[device], hipStreamNonBlocking) != hipSuccess) {
        (void)hipGetLastError();
        ts.s[device] = nullptr;
    }
    return ts.s[device];
}

class PcgRun {
  public:
    // prepared: A's SELL layout converted beforehand (one system; not owned), else converted
    // by begin() for this solve
    PcgRun(const afsai_csr &A, afsai_precond P, int nsys, const int32_t *row0, const double *b, double *x,
           double rtol, int32_t maxit, hipStream_t s, const Sell *prepared = nullptr)
        : A_(A), P_(P), nsys_(nsys), b_(b), x_(x), rtol_(rtol), maxit_(maxit), s_(s), prepared_(prepared) {
        if (nsys > 1 && row0) row0_.assign(row0, row0 + nsys + 1);
        else row0_ = {0, A.n};
    }
    ~PcgRun() {
        if (started_) (void)hipStreamSynchronize(s_);
        leave_place(false);
        for (int k = 0; k < 2; ++k) {
            if (gexec_[k]) (void)hipGraphExecDestroy(gexec_[k]);
            if (graph_[k]) (void)hipGraphDestroy(graph_[k]);
        }
        if (!prepared_) sell_free(&As_);
        for (hipEvent_t e : {t0_, t1_, ev_[0], ev_[1], ev_[2], ev_[3]})
            if (e) (void)hipEventDestroy(e);
        pinned_free(hsc_);
    }
    PcgRun(const PcgRun &) = delete;
    PcgRun &operator=(const PcgRun &) = delete;

    int begin() {
        const int n = A_.n;
        int rc;
        if ((rc = device_info(&di_))) return rc;
        AFSAI_HIP_TRY(hipEventCreate(&t0_));
        AFSAI_HIP_TRY(hipEventCreate(&t1_));
        for (hipEvent_t &e : ev_) AFSAI_HIP_TRY(hipEventCreate(&e));
        // the host copies of the scalars (cached pinned blocks: no hipHostMalloc per solve)
        hsc_ = (PcgScalars *)pinned_alloc(2 * sizeof(PcgScalars) * (size_t)nsys_);
        if (!hsc_) return set_error_code(AFSAI_ERR_NO_MEMORY, "pcg: out of pinned host memory");
        hs_[0] = hsc_;
        hs_[1] = hsc_ + nsys_;
        AFSAI_HIP_TRY(hipHostGetDevicePointer((void **)&dhs_[0], hsc_, 0));
        dhs_[1] = dhs_[0] + nsys_;
        AFSAI_HIP_TRY(hipEventRecord(t0_, s_));
        started_ = true;
        if ((rc = make_batch_maps(n, nsys_, row0_.data(), di_, s_, &bm_))) return rc;
        Segments seg;
        seg.nsys = nsys_;
        seg.row0 = row0_.data();

        // partial sums: p.q, r.r and r.z (the start and the final check use them in turn); scalars: two
        // buffers and the marks of systems with p.Ap <= 0
        const size_t maxb = std::max(bm_.sell.nblocks, std::max(bm_.vec.nblocks, di_.num_cus * 16));
        const size_t nsc_elems = (2 * (sizeof(PcgScalars) / sizeof(double)) + 3) * (size_t)nsys_ + ((size_t)nsys_ + 1) / 2 + 2;
        const size_t need = (size_t)kWorkVectors * n + 3 * maxb + nsc_elems;
        double *ws = nullptr;
        if (P_ && P_->work_elems >= need) {
            ws = P_->work;
        } else {
            if ((rc = dalloc(own_, need * sizeof(double), s_))) return rc;
            ws = own_.as<double>();
        }
        r_ = ws;
        r2_ = ws + n;
        z_ = ws + 2 * (size_t)n;
        p_ = ws + 3 * (size_t)n;
        p2_ = ws + 4 * (size_t)n;
        q_ = ws + 5 * (size_t)n;
        t_ = ws + 6 * (size_t)n;
        partials_ = ws + kWorkVectors * (size_t)n;
        pa_rr_ = partials_ + maxb;
        pa_rz_ = partials_ + 2 * maxb;
        sc_ = (PcgScalars *)(partials_ + 3 * maxb);
        red_ = (double *)(sc_ + 2 * (size_t)nsys_);
        ctl_ = (int32_t *)(red_ + 3 * (size_t)nsys_);  // control words of the one-launch solve
        bad_ = ctl_ + 4;

        // A in the SELL-64 layout for the iteration (one conversion per solve); CSR only for one
        // system when asked for
        use_sell_ = option(AFSAI_OPT_PCG_CSR_A) == 0 || nsys_ > 1 || prepared_;
        if (prepared_) {
            As_ = *prepared_;
        } else if (use_sell_) {
            ProfScope ps("sell_A", s_);
            if ((rc = sell_from_csr(n, A_.nnz, A_.row_ptr, A_.col_idx, A_.val, false, false, &As_, di_, s_, seg)))
                return rc;
        }
        // fused products where launches dominate (small systems), separate updates where the
        // fused products' second gather costs more than the update kernels; the fused kernels
        // need layouts without a tail
        const int64_t form = option(AFSAI_OPT_PCG_FORM);
        int nmax = 0;
        for (int k = 0; k < nsys_; ++k) nmax = std::max(nmax, row0_[k + 1] - row0_[k]);
        const bool small = nsys_ > 1 ? nmax < kFusedMaxRows : As_.entries + (P_ ? P_->sg.entries : 0) <= kFusedEntries;
        const bool want_fused = form == 2 || (form == 0 && small);
        fused_ = P_ && use_sell_ && want_fused && !As_.tail && !P_->sg.tail && !As_.perm && !P_->sg.perm;
        bm_.nt = stream_bytes(As_) + (P_ ? stream_bytes(P_->sg) + stream_bytes(P_->sgt) : 0) > kCachedBytes;
        if ((rc = choose_small())) return rc;
        if (!small_) return start();
        ++g_forms[AFSAI_PCG_ONE_LAUNCH];
        return enqueue_small();
    }

    // The start of the iteration and its first chunk
    int start() {
        const int n = A_.n;
        int rc;
        ++g_forms[fused_ ? AFSAI_PCG_FUSED : AFSAI_PCG_SEPARATE];
        const dim3 gv(bm_.vec.nblocks), gs(bm_.nsys);
        const int plain = P_ ? 0 : 1;
        hipLaunchKernelGGL(k_set_scalars, dim3((nsys_ + 255) / 256), dim3(256), 0, s_, sc_, bad_, ctl_, nsys_, rtol_,
                           maxit_, plain);
        // r0 = b - A x0
        spmv_A("spmv_A", x_, q_, nullptr, nullptr);
        hipLaunchKernelGGL(k_init_residual, gv, dim3(kThreads), 0, s_, n, b_, q_, r_, partials_, bm_.vec.mp, bm_.sy,
                           di_.num_xcds);
        hipLaunchKernelGGL(k_finalize, gs, dim3(kThreads), 0, s_, vec_parts(partials_),
                           vec_parts(partials_ + bm_.vec.nblocks), (int)FIN_INIT, sc_);
        // z0 = M^-1 r0, rho0 = r0.z0, p0 = z0
        zz_ = z_;
        if (P_) {
            sell_spmv("spmv_G", P_->sg, bm_, r_, t_, nullptr, nullptr, sc_, FIN_NONE, di_, s_);
            sell_spmv("spmv_GT_dot", P_->sgt, bm_, t_, z_, r_, pa_rz_, sc_, FIN_RHO0, di_, s_);
        } else {
            zz_ = r_;
        }
        // A's product with one column index per run of three consecutive columns where every
        // row is made of such runs (3 x 3 blocks): 9.3 instead of 12 bytes per FP64 entry, the
        // same sums (the fused kernels keep the plain layout)
        if (use_sell_ && !prepared_ && !fused_ && option(AFSAI_OPT_SELL_RUNS) != 1) {
            ProfScope ps("sell_A_runs", s_);
            if ((rc = sell_group_runs(&As_, di_, s_))) return rc;
        }
        // iterations replayed from captured graphs only when asked for (never while the kernel
        // timer is on: its events would be captured); on MI355X with ROCm 7 enqueuing the
        // kernels measured faster than replaying graphs at every size tried
        use_graph_ = !profiling_on() && option(AFSAI_OPT_PCG_GRAPH) == 2;
        if (!fused_)
            hipLaunchKernelGGL(k_update_p, gv, dim3(kThreads), 0, s_, n, p_, zz_, sc_, (PcgScalars *)nullptr, bad_,
                               Parts(), Parts(), 1, bm_.vec.mp, bm_.sy, di_.num_xcds);
        return start_chunks();
    }

    // The launches of the fused form from iteration `done` on, an even number of iterations after the start: p and r
    // are in the first of their buffers, the scalars, with the last step taken, too
    int go_on(int done) {
        static_assert(kSmallIters % 2 == 0, "the buffers of a continued solve");
        ++g_forms[AFSAI_PCG_FUSED];
        iter_no_ = enqueued_ = done;
        return start_chunks();
    }

    int start_chunks() {
        int rc;
        mark0_ = prof_mark();
        prev_it_.assign(nsys_, 0);
        prev_rr_.assign(nsys_, 0.0);
        rate_.assign(nsys_, 0.0);
        tol_.assign(nsys_, 0.0);
        have_prev_.assign(nsys_, 0);
        // the state after the start (a chunk of no iterations) and a first chunk in flight
        // before any state is read
        if ((rc = enqueue_chunk(0))) return rc;
        if ((rc = enqueue_chunk(kFirstChunk))) return rc;
        return AFSAI_OK;
    }

    // Returns AFSAI_OK and sets *finished; with block == false returns at once (finished
    // false) when the oldest chunk in flight has not completed.
    int advance(bool block, bool *finished) {
        *finished = false;
        if (done_) {
            *finished = true;
            return AFSAI_OK;
        }
        if (small_) return advance_small(block, finished);
        const int slot = (c_ - 2) & 1;  // state after the oldest chunk in flight
        hipEvent_t ev = ev_[(c_ - 2) & 3];
        if (!block) {
            const hipError_t q = hipEventQuery(ev);
            if (q == hipErrorNotReady) return AFSAI_OK;
            if (q != hipSuccess) AFSAI_HIP_TRY(q);
        } else {
            AFSAI_HIP_TRY(hipEventSynchronize(ev));
        }
        // GPU time of that chunk (from the end of the chunk before it)
        if (c_ >= 3 && its_[(c_ - 2) & 3] > 0) {
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, ev_[(c_ - 3) & 3], ev) == hipSuccess && ms > 0.f) {
                gpu_us_ += 1e3 * ms;
                it_us_ = 1e3 * ms / its_[(c_ - 2) & 3];
            } else {
                (void)hipGetLastError();
            }
        }
        const PcgScalars *st = hs_[slot];
        bool all_done = true;
        for (int k = 0; k < nsys_; ++k) {
            if (st[k].done != DONE_NO) continue;
            all_done = false;
            tol_[k] = st[k].tol;
            if (have_prev_[k] && st[k].it > prev_it_[k] && st[k].rr > 0.0 && prev_rr_[k] > 0.0) {
                const double rt = std::log(st[k].rr / prev_rr_[k]) / (st[k].it - prev_it_[k]);
                if (rt < 0.0) rate_[k] = rt;
            }
            if (st[k].rr > 0.0) {
                prev_rr_[k] = st[k].rr;
                prev_it_[k] = st[k].it;
                have_prev_[k] = 1;
            }
        }
        if (all_done || enqueued_ >= maxit_) {
            done_ = true;
            *finished = true;
            return AFSAI_OK;
        }
        // Chunk size: enough GPU work to cover the host's turnaround (two chunks are in flight)
        // and a fixed share of the time so far, so that the iterations enqueued past
        // convergence stay a small part of the solve; capped by the iterations the slowest
        // active system still needs at its observed rate.
        int todo = kFirstChunk;
        if (it_us_ > 0.0) {
            const double window_us = std::max(kMinChunkUs, gpu_us_ * kChunkShare);
            todo = (int)std::min(64.0, std::max(1.0, std::ceil(window_us / it_us_)));
        }
        int need_max = -1;
        for (int k = 0; k < nsys_; ++k) {
            if (st[k].done != DONE_NO) continue;
            if (!(rate_[k] < 0.0 && have_prev_[k])) {
                need_max = -1;
                break;
            }
            const double need_it = std::ceil(std::log(tol_[k] * tol_[k] / prev_rr_[k]) / rate_[k]);
            need_max = std::max(need_max, (int)need_it - (enqueued_ - prev_it_[k]) + 1);
        }
        if (need_max >= 0) todo = std::min(todo, std::max(1, need_max));
        return enqueue_chunk(todo);
    }

    int finish(afsai_pcg_info *info) {
        const int n = A_.n;
        AFSAI_HIP_TRY(hipStreamSynchronize(s_));
        std::vector<PcgScalars> fin_s(nsys_);
        const size_t scbytes = sizeof(PcgScalars) * (size_t)nsys_;
        float ms = 0.f;
        if (small_) {  // the launch has left the final scalars and the true residual
            fin_s[0] = hs_[0][0];
            AFSAI_HIP_TRY(hipEventElapsedTime(&ms, t0_, ev_[0]));
            return report(fin_s, ms, info);
        }
        AFSAI_HIP_TRY(hipMemcpyAsync(fin_s.data(), scal(iter_no_), scbytes, hipMemcpyDeviceToHost, s_));
        AFSAI_HIP_TRY(hipStreamSynchronize(s_));
        int it_max = 0;
        for (int k = 0; k < nsys_; ++k) it_max = std::max(it_max, (int)fin_s[k].it);
        {
            const int keep_to = it_max >= 1 && it_max <= (int)marks_.size() ? marks_[it_max - 1] : mark0_;
            prof_drop(keep_to, prof_mark());
        }
        const dim3 gv(bm_.vec.nblocks), gs(bm_.nsys);
        hipLaunchKernelGGL(k_zero_rhs, gv, dim3(kThreads), 0, s_, n, x_, scal(iter_no_), bm_.vec.mp, bm_.sy,
                           di_.num_xcds);
        // true residuals ||b - A x||
        spmv_A("spmv_A", x_, q_, nullptr, nullptr);
        hipLaunchKernelGGL(k_resid_norm, gv, dim3(kThreads), 0, s_, n, b_, q_, partials_, bm_.vec.mp, bm_.sy,
                           di_.num_xcds);
        hipLaunchKernelGGL(k_finalize, gs, dim3(kThreads), 0, s_, vec_parts(partials_), Parts(), (int)FIN_RESID,
                           scal(iter_no_));
        AFSAI_HIP_TRY(hipMemcpyAsync(hs_[0], scal(iter_no_), scbytes, hipMemcpyDeviceToHost, s_));
        AFSAI_HIP_TRY(hipEventRecord(t1_, s_));
        AFSAI_HIP_TRY(hipStreamSynchronize(s_));
        AFSAI_HIP_TRY(hipGetLastError());
        AFSAI_HIP_TRY(hipEventElapsedTime(&ms, t0_, t1_));
        prof_flush();
        return report(fin_s, ms, info);
    }

  private:
    // status and results from the final scalars (the true residuals in the host copy)
    int report(const std::vector<PcgScalars> &fin_s, float ms, afsai_pcg_info *info) {
        int status = AFSAI_OK;
        for (int k = 0; k < nsys_ && status == AFSAI_OK; ++k) {
            const PcgScalars &f = fin_s[k];
            if (f.done == DONE_NOT_SPD) {
                if (nsys_ == 1)
                    set_error("pcg_solve: p.Ap <= 0 at iteration %d (matrix or preconditioner not SPD)", f.it + 1);
                else
                    set_error("pcg_solve_batched: system %d: p.Ap <= 0 at iteration %d (not SPD)", k, f.it + 1);
                status = AFSAI_ERR_NOT_SPD;
            } else if (f.done == DONE_MAXIT || f.done == DONE_NO) {
                if (nsys_ == 1) set_error("pcg_solve: not converged in %d iterations", f.it);
                else set_error("pcg_solve_batched: system %d not converged in %d iterations", k, f.it);
                status = AFSAI_ERR_NOT_CONVERGED;
            }
        }
        if (info) {
            for (int k = 0; k < nsys_; ++k) {
                const PcgScalars &f = fin_s[k];
                const double nb = sqrt(f.bb);
                info[k].iters = f.it;
                info[k].converged = (f.done == DONE_CONVERGED || f.done == DONE_ZERO_RHS) ? 1 : 0;
                info[k].relres = nb > 0 ? sqrt(f.rr) / nb : 0.0;
                info[k].true_relres = (nb > 0 && f.done != DONE_ZERO_RHS) ? sqrt(hs_[0][k].resid) / nb : 0.0;
                info[k].ms = ms;
            }
        }
        return status;
    }

    // The one-launch solve for systems that one XCD reads faster than the launches of an iteration
    // take (whole solves, launches and this: 8,000 rows of 7 0.84, 0.47 ms; 15,625 rows 0.99, 0.73 ms; at
    // 17,576 rows, past one window per group, 23 and 27 us an iteration), when the automatic forms are in force and the kernel timer is off
    int choose_small() {
        small_ = false;
        if (!fused_ || P_->sgt.tail || nsys_ != 1 || option(AFSAI_OPT_PCG_FORM) != 0 || option(AFSAI_OPT_PCG_GRAPH) == 2 || profiling_on())
            return AFSAI_OK;
        const int vb = P_->sg.f32 ? 4 : 8;
        if (12 * As_.entries + (4 + vb) * (P_->sg.entries + P_->nnz_g) > kSmallBytes || P_->sgt.entries > (1 << 24))
            return AFSAI_OK;
        uint32_t mask = 0;
        int rc;
        if ((rc = xcc_mask(di_, s_, &mask))) return rc;
        const int nx = __builtin_popcount(mask);
        if (nx < 1) return AFSAI_OK;
        const int cus = std::max(1, di_.num_cus / nx), nw = (As_.nslices + kWin - 1) / kWin;
        const int ng = std::min(kSmallWin, (nw + cus - 1) / cus);
        const int blocks = std::min(cus, (nw + ng - 1) / ng);
        if (nw > blocks * ng) return AFSAI_OK;
        const int xcc = g_places[di_.device].take(mask);
        if (xcc < 0) return AFSAI_OK;
        place_ = xcc;
        sa_ = SmallArgs{A_.n, As_.nslices, (int)As_.entries, (int)P_->sg.entries, (int)P_->sgt.entries, As_.sptr, P_->sg.sptr, P_->sgt.sptr, As_.col, P_->sg.col, P_->sgt.col,
                        (const double *)As_.val, P_->sg.val, P_->sgt.val, P_->sgt.perm, P_->sgt.lens, b_, x_, r_, r2_, z_,
                        p_, p2_, q_, t_, partials_, pa_rr_, pa_rz_, sc_, dhs_[0], (SmallCtl *)ctl_, blocks, xcc,
                        bm_.vec.nblocks, 0, kSmallIters, 0, 0};
        if (option(AFSAI_OPT_PCG_ONE_LAUNCH) == 3) sa_.xcc = __builtin_ctz(~mask);  // (bit 16 at the latest)
        small_grid_ = dim3((unsigned)(blocks * nx));
        small_block_ = dim3((unsigned)(ng * kThreads));
        small_ = true;
        return AFSAI_OK;
    }

    void leave_place(bool unmet) {
        if (place_ >= 0) g_places[di_.device].give(place_, unmet);
        place_ = -1;
    }

    // up to kSmallIters iterations from sa_.iter0 on
    int enqueue_small() {
        // the record comes from a cache and may hold an earlier solve's end: marked, so that a launch
        // of which no block reached the XCD is seen (its stream is idle here)
        hs_[0][0] = PcgScalars{};
        hs_[0][0].pad = SMALL_ABSENT;
        sa_.miss = option(AFSAI_OPT_PCG_ONE_LAUNCH) == (sa_.iter0 == 0 ? 1 : 2);
        sa_.late = option(AFSAI_OPT_PCG_ONE_LAUNCH) == 4 && sa_.iter0 > 0;
        if (sa_.iter0 == 0)
            hipLaunchKernelGGL(k_set_scalars, dim3(1), dim3(256), 0, s_, sc_, bad_, ctl_, 1, rtol_, maxit_, 0);
        else
            hipLaunchKernelGGL(k_small_again, dim3(1), dim3(64), 0, s_, (SmallCtl *)ctl_);
        const bool ord = sa_.t_perm != nullptr;
        if (P_->sg.f32) {
            if (ord) hipLaunchKernelGGL((k_pcg_small<float, true>), small_grid_, small_block_, 0, s_, sa_);
            else hipLaunchKernelGGL((k_pcg_small<float, false>), small_grid_, small_block_, 0, s_, sa_);
        } else {
            if (ord) hipLaunchKernelGGL((k_pcg_small<double, true>), small_grid_, small_block_, 0, s_, sa_);
            else hipLaunchKernelGGL((k_pcg_small<double, false>), small_grid_, small_block_, 0, s_, sa_);
        }
        AFSAI_HIP_TRY(hipGetLastError());
        AFSAI_HIP_TRY(hipEventRecord(ev_[0], s_));
        return AFSAI_OK;
    }

    int advance_small(bool block, bool *finished) {
        if (block) {
            AFSAI_HIP_TRY(hipEventSynchronize(ev_[0]));
        } else {
            const hipError_t q = hipEventQuery(ev_[0]);
            if (q == hipErrorNotReady) return AFSAI_OK;
            if (q != hipSuccess) AFSAI_HIP_TRY(q);
        }
        const PcgScalars &st = hs_[0][0];
        // no block ran, or they did not come together: the usual launches, from the start or from the
        // iteration where the launch before ended
        if (st.pad == SMALL_UNMET || st.pad == SMALL_ABSENT) {
            small_ = false;
            leave_place(true);
            ++g_forms[AFSAI_PCG_UNMET];
            return sa_.iter0 == 0 ? start() : go_on(sa_.iter0);
        }
        if (st.pad != SMALL_RAN) AFSAI_FAIL(AFSAI_ERR_HIP, "pcg_solve: the blocks of a one-launch solve lost each other");
        if (st.done != DONE_NO) {
            leave_place(false);
            done_ = true;
            *finished = true;
            return AFSAI_OK;
        }
        sa_.iter0 += sa_.iters;
        return enqueue_small();
    }

    // the scalars before iteration it (0-based): two buffers in turn
    PcgScalars *scal(int it) const { return sc_ + (size_t)(it & 1) * nsys_; }
    Parts sell_parts(const double *p) const { return Parts{p, bm_.sell.mp, bm_.sell.nblocks}; }
    Parts vec_parts(const double *p) const { return Parts{p, bm_.vec.mp, bm_.vec.nblocks}; }
    Parts red_parts(int j) const { return Parts{red_ + (size_t)j * nsys_, Map(), 0}; }
    // partials of r.r (over the windows but with M = I, see k_update_xr_win) and of r.z
    Parts rr_parts() const { return P_ ? sell_parts(pa_rr_) : vec_parts(pa_rr_); }
    Parts rz_parts() const { return P_ ? sell_parts(pa_rz_) : Parts(); }

    // products inside the iteration stop with their system (gate: its scalars); the first and the
    // final A x run for every system
    void spmv_A(const char *name, const double *xin, double *yout, const double *w, PcgScalars *gate) {
        if (use_sell_) sell_spmv(name, As_, bm_, xin, yout, w, w ? partials_ : nullptr, gate, FIN_NONE, di_, s_);
        else spmv(name, csr_of(&A_), xin, yout, w, w ? partials_ : nullptr, gate, di_, s_);
    }

    // One iteration: from the captured graph of its buffer parity (captured at its first use;
    // the first fused iteration, which forms p = z, always runs directly), else enqueued.
    // Capture runs on a private stream of this thread (the caller's stream may be the null
    // stream, which cannot capture); nothing executes there, the graph is launched on s_.
    int launch_iteration() {
        const int par = iter_no_ & 1;
        if (!use_graph_ || (fused_ && iter_no_ == 0)) {
            enqueue_iteration();
            return AFSAI_OK;
        }
        if (!gexec_[par]) {
            hipStream_t cs = capture_stream(di_.device);
            hipGraph_t g = nullptr;
            hipError_t e = cs ? hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal) : hipErrorUnknown;
            if (e == hipSuccess) {
                const int it0 = iter_no_;
                const size_t nmarks = marks_.size();
                hipStream_t keep = s_;
                s_ = cs;
                enqueue_iteration();
                s_ = keep;
                iter_no_ = it0;
                marks_.resize(nmarks);
                e = hipStreamEndCapture(cs, &g);
            }
            if (e == hipSuccess && g) e = hipGraphInstantiate(&gexec_[par], g, nullptr, nullptr, 0);
            if (e != hipSuccess || !gexec_[par]) {
                // capture not available: enqueue directly from here on
                (void)hipGetLastError();
                if (g) (void)hipGraphDestroy(g);
                gexec_[par] = nullptr;
                use_graph_ = false;
                enqueue_iteration();
                return AFSAI_OK;
            }
            graph_[par] = g;
        }
        AFSAI_HIP_TRY(hipGraphLaunch(gexec_[par], s_));
        marks_.push_back(prof_mark());
        ++iter_no_;
        return AFSAI_OK;
    }

    void enqueue_iteration() {
        const int n = A_.n;
        const dim3 gv(bm_.vec.nblocks), gs(nsys_);
        PcgScalars *s_in = scal(iter_no_), *s_out = scal(iter_no_ + 1);
        if (fused_) {
            // p and r are double-buffered: the products read neighbours' old entries while
            // owners store the new ones
            const bool odd = (iter_no_ & 1) == 0;  // iteration 1, 3, ...: p -> p2, r -> r2
            double *p_old = odd ? p_ : p2_, *p_new = odd ? p2_ : p_;
            double *r_old = odd ? r_ : r2_, *r_new = odd ? r2_ : r_;
            sell_fused<FUSE_AP>("spmv_A_dot", As_, bm_, z_, p_old, p_new, nullptr, nullptr, q_, partials_,
                                FusedScal{s_in, s_out, bad_, rr_parts(), rz_parts()}, iter_no_ == 0 ? 1 : 0, di_, s_);
            sell_fused<FUSE_GR>("spmv_G_upd", P_->sg, bm_, r_old, q_, r_new, x_, p_new, t_, pa_rr_,
                                FusedScal{s_out, nullptr, bad_, sell_parts(partials_), Parts()}, 0, di_, s_);
            marks_.push_back(prof_mark());
            sell_spmv("spmv_GT_dot", P_->sgt, bm_, t_, z_, r_new, pa_rz_, s_out, FIN_NONE, di_, s_);
            ++iter_no_;
            return;
        }
        // the sums are added by launches of their own here: thousands of blocks would each read
        // thousands of partials (121^3: 23.4 -> 25.9 ms)
        spmv_A("spmv_A_dot", p_, q_, p_, s_in);
        const Parts pq = use_sell_ ? sell_parts(partials_) : Parts{partials_, Map(), spmv_blocks(csr_of(&A_), di_)};
        hipLaunchKernelGGL(k_reduce, gs, dim3(kThreads), 0, s_, pq, Parts(), red_, (double *)nullptr, s_in);
        // the iteration that converges needs no z: with a large G (the two products cost more than a
        // launch per iteration) r.r is summed before them and they return; else by G^T's product, which has r for r.z
        const bool gate = P_ && P_->sg.entries >= kGateEntries;
        {
            ProfScope ps("update_xr", s_);
            if (gate)
                hipLaunchKernelGGL(k_update_xr_win, dim3(bm_.sell.nblocks), dim3(kThreads), 0, s_, n, x_, r_, p_, q_, pa_rr_,
                                   s_in, bad_, red_parts(0), bm_.sell.mp, bm_.sy, di_.num_xcds);
            else if (P_)
                hipLaunchKernelGGL(k_update_xr<false>, gv, dim3(kThreads), 0, s_, n, x_, r_, p_, q_, (double *)nullptr, s_in,
                                   bad_, red_parts(0), bm_.vec.mp, bm_.sy, di_.num_xcds);
            else
                hipLaunchKernelGGL(k_update_xr<true>, gv, dim3(kThreads), 0, s_, n, x_, r_, p_, q_, pa_rr_, s_in, bad_,
                                   red_parts(0), bm_.vec.mp, bm_.sy, di_.num_xcds);
        }
        marks_.push_back(prof_mark());
        if (gate)
            hipLaunchKernelGGL(k_reduce, gs, dim3(kThreads), 0, s_, rr_parts(), Parts(), red_ + nsys_,
                               (double *)nullptr, s_in);
        if (P_) {
            const double *rr = gate ? red_ + nsys_ : nullptr;
            sell_spmv("spmv_G", P_->sg, bm_, r_, t_, nullptr, nullptr, s_in, FIN_NONE, di_, s_, rr);
            sell_spmv("spmv_GT_dot", P_->sgt, bm_, t_, z_, r_, pa_rz_, s_in, FIN_NONE, di_, s_, rr, gate ? nullptr : pa_rr_);
        }
        if (gate)
            hipLaunchKernelGGL(k_reduce, gs, dim3(kThreads), 0, s_, rz_parts(), Parts(), red_ + 2 * (size_t)nsys_,
                               (double *)nullptr, s_in);
        else
            hipLaunchKernelGGL(k_reduce, gs, dim3(kThreads), 0, s_, rr_parts(), rz_parts(), red_ + nsys_,
                               red_ + 2 * (size_t)nsys_, s_in);
        {
            ProfScope ps("update_p", s_);
            hipLaunchKernelGGL(k_update_p, gv, dim3(kThreads), 0, s_, n, p_, zz_, s_in, s_out, bad_, red_parts(1),
                               P_ ? red_parts(2) : Parts(), 0, bm_.vec.mp, bm_.sy, di_.num_xcds);
        }
        ++iter_no_;
    }

    // todo iterations (at most what maxit leaves), then a copy of the scalars into the host
    // slot of this chunk and its event
    int enqueue_chunk(int todo) {
        if (todo > maxit_ - enqueued_) todo = maxit_ - enqueued_;
        for (int k = 0; k < todo; ++k) {
            int rc;
            if ((rc = launch_iteration())) return rc;
        }
        enqueued_ += todo;
        const int slot = c_ & 1;
        hipLaunchKernelGGL(k_publish, dim3(nsys_), dim3(kThreads), 0, s_, scal(iter_no_), bad_, rr_parts(), rz_parts(),
                           dhs_[slot]);
        its_[c_ & 3] = todo;
        AFSAI_HIP_TRY(hipEventRecord(ev_[c_ & 3], s_));
        ++c_;
        return AFSAI_OK;
    }

    const afsai_csr A_;
    afsai_precond P_;
    int nsys_;
    std::vector<int32_t> row0_;
    const double *b_;
    double *x_;
    double rtol_;
    int32_t maxit_;
    hipStream_t s_;
    DeviceInfo di_;
    BatchMaps bm_;
    DevBuf own_;
    const Sell *prepared_ = nullptr;
    Sell As_;
    bool use_sell_ = true, fused_ = false, started_ = false, done_ = false, use_graph_ = false;
    hipGraph_t graph_[2] = {nullptr, nullptr};
    hipGraphExec_t gexec_[2] = {nullptr, nullptr};
    double *r_ = nullptr, *r2_ = nullptr, *z_ = nullptr, *p_ = nullptr, *p2_ = nullptr, *q_ = nullptr, *t_ = nullptr;
    const double *zz_ = nullptr;
    double *partials_ = nullptr, *pa_rr_ = nullptr, *pa_rz_ = nullptr;
    double *red_ = nullptr;     // [3][nsys]: the sums p.q, r.r, r.z of the separate form
    PcgScalars *sc_ = nullptr;  // [2][nsys]
    int32_t *bad_ = nullptr;    // [nsys]
    int32_t *ctl_ = nullptr;
    bool small_ = false;        // the whole solve in one launch (pcg_small.hpp)
    int place_ = -1;            // its XCD among g_places
    SmallArgs sa_{};
    dim3 small_grid_, small_block_;
    PcgScalars *hsc_ = nullptr;
    PcgScalars *hs_[2] = {nullptr, nullptr};
    PcgScalars *dhs_[2] = {nullptr, nullptr};  // device addresses of hs_
    hipEvent_t t0_ = nullptr, t1_ = nullptr, ev_[4] = {nullptr, nullptr, nullptr, nullptr};
    int its_[4] = {0, 0, 0, 0};
    double gpu_us_ = 0.0, it_us_ = 0.0;
    int iter_no_ = 0, enqueued_ = 0, c_ = 0, mark0_ = 0;
    std::vector<int> marks_, prev_it_;
    std::vector<double> prev_rr_, rate_, tol_;
    std::vector<char> have_prev_;
};

struct PcgTask {
    PcgRun run;
    PcgTask(const afsai_csr &A, afsai_precond P, const double *b, double *x, double rtol, int32_t maxit,
            hipStream_t s)
        : run(A, P, 1, nullptr, b, x, rtol, maxit, s) {}
};

int pcg_task_begin(const afsai_csr &A, afsai_precond P, const double *b, double *x, double rtol, int32_t maxit,
                   hipStream_t stream, PcgTask **out) {
    *out = nullptr;
    PcgTask *t = new PcgTask(A, P, b, x, rtol, maxit, stream);
    const int rc = t->run.begin();
    if (rc) {
        delete t;
        return rc;
    }
    *out = t;
    return AFSAI_OK;
}
int pcg_task_advance(PcgTask *t, bool block, bool *finished) { return t->run.advance(block, finished); }
int pcg_task_finish(PcgTask *t, afsai_pcg_info *info) { return t->run.finish(info); }
void pcg_task_free(PcgTask *t) { delete t; }

static int pcg_batch(const afsai_csr *A, afsai_precond P, int nsys, const int32_t *row0, const double *b, double *x,
                     double rtol, int32_t maxit, hipStream_t s, afsai_pcg_info *info, const Sell *prepared = nullptr) {
    PcgRun run(*A, P, nsys, row0, b, x, rtol, maxit, s, prepared);
    int rc = run.begin();
    if (rc) return rc;
    bool fin = false;
    while (!fin)
        if ((rc = run.advance(true, &fin))) return rc;
    return run.finish(info);
}

}  // namespace afsai

using namespace afsai;

extern "C" {

int afsai_pcg_form_counts(int64_t counts[4]) {
    if (!counts) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "afsai_pcg_form_counts: null argument");
    for (int k = 0; k < 4; ++k) counts[k] = g_forms[k].load(std::memory_order_relaxed);
    return AFSAI_OK;
}

int afsai_spmv(const afsai_csr *A, const double *x, double *y, void *stream) {
    int rc = check_csr_arg(A, "afsai_spmv");
    if (rc) return rc;
    if (!x || !y) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "afsai_spmv: null vector");
    DeviceInfo di;
    if ((rc = device_info(&di))) return rc;
    hipStream_t s = (hipStream_t)stream;
    spmv("spmv_A", csr_of(A), x, y, nullptr, nullptr, nullptr, di, s);
    AFSAI_HIP_TRY(hipGetLastError());
    return AFSAI_OK;
}

}  // extern "C"

namespace afsai {

template <int K>
static int pcg_multi(const afsai_csr *A, afsai_precond P, const double *B, double *X, double rtol, int32_t maxit,
                     hipStream_t s, const DeviceInfo &di, afsai_pcg_info *info) {
    const int n = A->n;
    int rc;
    Sell SA;
    struct Free {
        Sell *S;
        ~Free() { sell_free(S); }
    } free_sa{&SA};
    if (blocks_pay(K, n, 2, di) && option(AFSAI_OPT_SELL_RUNS) != 1 && option(AFSAI_OPT_SELL_WIDTH) == 0 && n % 3 == 0) {
        // 3 x 3 blocks, unless the rows would be ordered by length (the dots of that layout are
        // summed in another order)
        ProfScope ps("sell_A_blocks", s);
        bool ordered = true;
        if ((rc = sell_ordered(n, A->nnz, A->row_ptr, &ordered, di, s))) return rc;
        if (!ordered && (rc = sell_node_blocks(n, A->nnz, A->row_ptr, A->col_idx, A->val, false, &SA, di, s))) return rc;
    }
    if (!SA.bptr) {
        {
            ProfScope ps("sell_A", s);
            if ((rc = sell_from_csr(n, A->nnz, A->row_ptr, A->col_idx, A->val, false, false, &SA, di, s))) return rc;
        }
        if (SA.tail) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve_multi: split SELL layouts are not supported");
        if (option(AFSAI_OPT_SELL_RUNS) != 1) {
            ProfScope ps("sell_A_runs", s);
            if ((rc = sell_group_runs(&SA, di, s))) return rc;
        }
    }
    const bool nt = (SA.bptr ? SA.bentries * 9 : stream_bytes(SA)) +
                        (P ? stream_bytes(P->sg) + stream_bytes(P->sgt) : 0) > kCachedBytes;
    const int nbA = blocks_for_slices((n + kSlice - 1) / kSlice, di), nbv = blocks_for_vec(n, di);
    const int nbG = P ? blocks_for_slices(P->sg.nslices, di) : 0;
    const int nbGT = P ? blocks_for_slices(P->sgt.nslices, di) : 0;
    const int nbmax = std::max(std::max(nbA, nbv), std::max(nbG, nbGT));
    const size_t blk = (size_t)n * K;
    DevBuf work, parts, scb;
    if ((rc = dalloc(work, sizeof(double) * blk * 5, s))) return rc;
    if ((rc = dalloc(parts, sizeof(double) * (size_t)K * nbmax, s))) return rc;
    if ((rc = dalloc(scb, sizeof(MultiScal) * K, s))) return rc;
    double *R = work.as<double>(), *Z = R + blk, *Pv = Z + blk, *Q = Pv + blk, *T = Q + blk;
    double *pa = parts.as<double>();
    MultiScal *sc = scb.as<MultiScal>();
    auto fin = [&](int nb, int mode) {
        hipLaunchKernelGGL(k_fin_multi, dim3(K), dim3(kThreads), 0, s, pa, nb, mode, rtol, (int)maxit, sc);
    };
    // Z = M R with partial sums of R.Z; returns the blocks of that launch
    auto precond = [&](const MultiScal *gate) {
        if (P) {
            spmm_launch<K, false>(P->sg, nt, R, T, nullptr, nullptr, nbG, di, s, gate);
            spmm_launch<K, true>(P->sgt, nt, T, Z, R, pa, nbGT, di, s, gate);
            return nbGT;
        }
        hipLaunchKernelGGL((k_multi_dot<K>), dim3(nbv), dim3(kThreads), 0, s, n, R, R, Z, pa);
        return nbv;
    };
    // the scalars after each iteration, in pinned host memory (two slots in turn)
    struct Host {
        MultiScal *h = nullptr, *d = nullptr;
        hipEvent_t ev[2] = {nullptr, nullptr};
        hipStream_t s;
        ~Host() {
            (void)hipStreamSynchronize(s);
            for (hipEvent_t e : ev)
                if (e) (void)hipEventDestroy(e);
            pinned_free(h);
        }
    } host;
    host.s = s;
    host.h = (MultiScal *)pinned_alloc(2 * K * sizeof(MultiScal));
    if (!host.h) return set_error_code(AFSAI_ERR_NO_MEMORY, "pcg_solve_multi: out of pinned host memory");
    AFSAI_HIP_TRY(hipHostGetDevicePointer((void **)&host.d, host.h, 0));
    for (hipEvent_t &e : host.ev) AFSAI_HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    hipLaunchKernelGGL((k_multi_init<K>), dim3(nbv), dim3(kThreads), 0, s, n, B, X, R, pa);
    fin(nbv, MF_BB);
    fin(precond(nullptr), MF_RHO0);
    AFSAI_HIP_TRY(hipMemcpyAsync(Pv, Z, sizeof(double) * blk, hipMemcpyDeviceToDevice, s));
    // The host reads the scalars one iteration behind (waiting for each iteration before the next
    // left the GPU idle for about 45 us of 300 at 250,000 rows); the iteration that is then queued past the
    // last column's end returns at once
    for (int it = 0; it < maxit; ++it) {
        spmm_launch<K, true>(SA, nt, Pv, Q, Pv, pa, nbA, di, s, sc);
        fin(nbA, MF_PQ);
        hipLaunchKernelGGL((k_multi_xr<K>), dim3(nbv), dim3(kThreads), 0, s, n, X, R, Pv, Q, sc, pa);
        fin(nbv, MF_RR);
        fin(precond(sc), MF_RZ);
        hipLaunchKernelGGL((k_multi_p<K>), dim3(nbv), dim3(kThreads), 0, s, n, Z, Pv, sc);
        hipLaunchKernelGGL(k_multi_publish, dim3(1), dim3(64), 0, s, K, sc, host.d + (it & 1) * K);
        AFSAI_HIP_TRY(hipGetLastError());
        AFSAI_HIP_TRY(hipEventRecord(host.ev[it & 1], s));
        if (it == 0) continue;
        AFSAI_HIP_TRY(hipEventSynchronize(host.ev[(it - 1) & 1]));
        bool all = true;
        for (int j = 0; j < K; ++j) all = all && host.h[((it - 1) & 1) * K + j].done;
        if (all) break;
    }
    // true residuals ||b - A x|| per column
    spmm_launch<K, false>(SA, nt, X, Q, nullptr, nullptr, nbA, di, s);
    hipLaunchKernelGGL((k_multi_resid<K>), dim3(nbv), dim3(kThreads), 0, s, n, B, Q, pa);
    fin(nbv, MF_TRUE);
    std::vector<MultiScal> h(K);
    AFSAI_HIP_TRY(hipGetLastError());
    AFSAI_HIP_TRY(hipMemcpyAsync(h.data(), sc, sizeof(MultiScal) * K, hipMemcpyDeviceToHost, s));
    AFSAI_HIP_TRY(hipStreamSynchronize(s));
    int worst = AFSAI_OK;
    for (int j = 0; j < K; ++j) {
        const MultiScal &m = h[j];
        if (info) {
            info[j].iters = m.iters;
            info[j].converged = m.status == AFSAI_OK ? 1 : 0;
            info[j].relres = m.bb > 0.0 ? std::sqrt(m.rr / m.bb) : 0.0;
            info[j].true_relres = m.bb > 0.0 ? std::sqrt(m.tr / m.bb) : 0.0;
        }
        if (m.status == AFSAI_ERR_NOT_SPD) worst = AFSAI_ERR_NOT_SPD;
        else if (m.status != AFSAI_OK && worst == AFSAI_OK) worst = m.status;
    }
    if (worst == AFSAI_ERR_NOT_SPD) set_error("pcg_solve_multi: p.Ap <= 0 in a column (A not SPD)");
    else if (worst != AFSAI_OK) set_error("pcg_solve_multi: a column did not converge");
    return worst;
}

}  // namespace afsai

extern "C" {

int pcg_solve_multi(const afsai_csr *A, afsai_precond P, int32_t k, const double *B, double *X, double rtol,
                    int32_t maxit, void *stream, afsai_pcg_info *info) {
    if (k != 1 && k != 2 && k != 4 && k != 8)
        AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve_multi: k = %d (1, 2, 4 or 8)", k);
    int rc = check_csr_arg(A, "pcg_solve_multi");
    if (rc) return rc;
    if (!B || !X || B == X) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve_multi: null or aliased blocks");
    if (!(rtol > 0.0) || maxit < 0) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve_multi: rtol = %g, maxit = %d", rtol, maxit);
    if (P && (P->n != A->n || !P->seg_row0.empty() || P->sg.tail || P->sgt.tail))
        AFSAI_FAIL(AFSAI_ERR_INVALID_ARG,
                   "pcg_solve_multi: the preconditioner must be a single system of A's size without split layouts");
    DeviceInfo di;
    if ((rc = device_info(&di))) return rc;
    hipStream_t s = (hipStream_t)stream;
    const auto t0 = std::chrono::steady_clock::now();
    switch (k) {
        case 1: rc = pcg_multi<1>(A, P, B, X, rtol, maxit, s, di, info); break;
        case 2: rc = pcg_multi<2>(A, P, B, X, rtol, maxit, s, di, info); break;
        case 4: rc = pcg_multi<4>(A, P, B, X, rtol, maxit, s, di, info); break;
        default: rc = pcg_multi<8>(A, P, B, X, rtol, maxit, s, di, info); break;
    }
    const double ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    if (info)
        for (int j = 0; j < k; ++j) info[j].ms = ms;
    return rc;
}

}  // extern "C"

namespace afsai {

// Y = A X with A's SELL layout S (no split layout), k in {1, 2, 4, 8}; synchronous on s
static int spmm_sell(const Sell &S, int32_t k, const double *X, double *Y, const DeviceInfo &di, hipStream_t s) {
    {
        ProfScope ps("spmm_A", s);
        const int nb = blocks_for_slices(S.nslices, di);
        const bool nt = (S.bptr && blocks_pay(k, S.n, 1, di) ? S.bentries * 9 : stream_bytes(S)) > kCachedBytes;
        switch (k) {
            case 1: spmm_launch<1, false>(S, nt, X, Y, nullptr, nullptr, nb, di, s); break;
            case 2: spmm_launch<2, false>(S, nt, X, Y, nullptr, nullptr, nb, di, s); break;
            case 4: spmm_launch<4, false>(S, nt, X, Y, nullptr, nullptr, nb, di, s); break;
            default: spmm_launch<8, false>(S, nt, X, Y, nullptr, nullptr, nb, di, s); break;
        }
    }
    const hipError_t le = hipGetLastError();
    const hipError_t se = hipStreamSynchronize(s);
    if (le != hipSuccess || se != hipSuccess) AFSAI_FAIL(AFSAI_ERR_HIP, "afsai_spmm: %s", hipGetErrorString(le != hipSuccess ? le : se));
    return AFSAI_OK;
}

static int spmm_args(int32_t k, const double *X, double *Y, const char *who) {
    if (k != 1 && k != 2 && k != 4 && k != 8) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "%s: k = %d (1, 2, 4 or 8)", who, k);
    if (!X || !Y) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "%s: null block", who);
    if (X == Y) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "%s: X and Y alias", who);
    return AFSAI_OK;
}

}  // namespace afsai

extern "C" {

int afsai_spmm(const afsai_csr *A, int32_t k, const double *X, double *Y, void *stream) {
    int rc = spmm_args(k, X, Y, "afsai_spmm");
    if (rc) return rc;
    if ((rc = check_csr_arg(A, "afsai_spmm"))) return rc;
    DeviceInfo di;
    if ((rc = device_info(&di))) return rc;
    hipStream_t s = (hipStream_t)stream;
    Sell S;
    {
        ProfScope ps("sell_A", s);
        if ((rc = sell_from_csr(A->n, A->nnz, A->row_ptr, A->col_idx, A->val, false, false, &S, di, s))) return rc;
    }
    if (S.tail || S.srow0) {
        sell_free(&S);
        AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "afsai_spmm: split SELL layouts (AFSAI_OPT_SELL_UNEVEN = 1) are not supported");
    }
    rc = spmm_sell(S, k, X, Y, di, s);
    sell_free(&S);
    return rc;
}

int afsai_matrix_prepare(const afsai_csr *A, void *stream, afsai_matrix *out) {
    clear_error();
    if (out) *out = nullptr;
    if (!out) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "afsai_matrix_prepare: null handle pointer");
    int rc = check_csr_arg(A, "afsai_matrix_prepare");
    if (rc) return rc;
    DeviceInfo di;
    if ((rc = device_info(&di))) return rc;
    hipStream_t s = (hipStream_t)stream;
    afsai_matrix M = new afsai_matrix_s();
    M->device = di.device;
    M->A = *A;
    {
        ProfScope ps("sell_A", s);
        rc = sell_from_csr(A->n, A->nnz, A->row_ptr, A->col_idx, A->val, false, false, &M->S, di, s);
        // run indices for pcg_solve_prepared's products, the per-entry columns kept for the
        // block products
        if (rc == AFSAI_OK && option(AFSAI_OPT_SELL_RUNS) != 1) rc = sell_group_runs(&M->S, di, s, true);
        // and 3 x 3 blocks for the block products
        if (rc == AFSAI_OK && option(AFSAI_OPT_SELL_RUNS) != 1)
            rc = sell_node_blocks(A->n, A->nnz, A->row_ptr, A->col_idx, A->val, true, &M->S, di, s);
    }
    if (rc == AFSAI_OK && hipStreamSynchronize(s) != hipSuccess) rc = set_error_code(AFSAI_ERR_HIP, "afsai_matrix_prepare: synchronisation failed");
    if (rc != AFSAI_OK) {
        sell_free(&M->S);
        delete M;
        return rc;
    }
    *out = M;
    return AFSAI_OK;
}

void afsai_matrix_destroy(afsai_matrix M) {
    if (!M) return;
    (void)hipDeviceSynchronize();
    sell_free(&M->S);
    delete M;
}

int afsai_spmm_prepared(afsai_matrix M, int32_t k, const double *X, double *Y, void *stream) {
    if (!M) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "afsai_spmm_prepared: null matrix");
    int rc = spmm_args(k, X, Y, "afsai_spmm_prepared");
    if (rc) return rc;
    if (M->S.tail || M->S.srow0)
        AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "afsai_spmm_prepared: split SELL layouts (AFSAI_OPT_SELL_UNEVEN = 1) are not supported");
    DeviceInfo di;
    if ((rc = device_info(&di))) return rc;
    if (di.device != M->device)
        AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "afsai_spmm_prepared: matrix prepared on device %d, current device %d",
                   M->device, di.device);
    return spmm_sell(M->S, k, X, Y, di, (hipStream_t)stream);
}

int pcg_solve_prepared(afsai_matrix M, afsai_precond P, const double *b, double *x, double rtol, int32_t maxit,
                       void *stream, afsai_pcg_info *info) {
    clear_error();
    if (!M) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve_prepared: null matrix");
    if (!b || !x) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve_prepared: null b or x");
    if (!(rtol > 0.0) || maxit < 0)
        AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve_prepared: rtol = %g, maxit = %d", rtol, maxit);
    if (P && P->n != M->A.n)
        AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve_prepared: preconditioner has n = %d, A has n = %d", P->n, M->A.n);
    if (P && P->seg_row0.size() > 2)
        AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve_prepared: the preconditioner is for a batch");
    if (M->S.tail || M->S.srow0)
        AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve_prepared: split SELL layouts are not supported for A");
    DeviceInfo di;
    int rc = device_info(&di);
    if (rc) return rc;
    if (di.device != M->device || (P && P->device != M->device))
        AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve_prepared: matrix prepared on device %d, current device %d",
                   M->device, di.device);
    return pcg_batch(&M->A, P, 1, nullptr, b, x, rtol, maxit, (hipStream_t)stream, info, &M->S);
}

int afsai_apply(afsai_precond P, const double *r, double *z, void *stream) {
    if (!P || !r || !z) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "afsai_apply: null argument");
    if (r == z) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "afsai_apply: r and z alias");
    DeviceInfo di;
    int rc = device_info(&di);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    double *t = P->work;  // first n entries
    // products only (no dots): the whole matrix as one system
    BatchMaps bm;
    if ((rc = make_batch_maps(P->sg.nslices * kSlice, 1, nullptr, di, s, &bm))) return rc;
    bm.nt = stream_bytes(P->sg) + stream_bytes(P->sgt) > kCachedBytes;
    bm.sell.nblocks = blocks_for_slices(P->sg.nslices, di);
    sell_spmv("spmv_G", P->sg, bm, r, t, nullptr, nullptr, nullptr, FIN_NONE, di, s);
    bm.sell.nblocks = blocks_for_slices(P->sgt.nslices, di);
    sell_spmv("spmv_GT", P->sgt, bm, t, z, nullptr, nullptr, nullptr, FIN_NONE, di, s);
    AFSAI_HIP_TRY(hipGetLastError());
    return AFSAI_OK;
}

}  // extern "C"

namespace afsai {

// Scratch of afsai_apply_noalloc: the intermediate t = G r of one application, for up to
// kNoAllocMaxRows rows (128 MiB of doubles, held by every GPU the library runs on until the
// process ends).  Host code never passes `scratch` itself to a kernel: each device's address
// of the array is taken once with hipGetSymbolAddress (with that device current) and kept.
constexpr int64_t kNoAllocMaxRows = (int64_t)1 << 24;
static __device__ __align__(256) double scratch[kNoAllocMaxRows];

// address of `scratch` on the current device, looked up on the first call there
static int scratch_ptr(double **out) {
    constexpr int kMaxDev = 64;
    static std::mutex mu;
    static double *ptr[kMaxDev] = {};
    int dev = -1;
    AFSAI_HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDev) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "afsai_apply_noalloc: device %d", dev);
    std::lock_guard<std::mutex> lk(mu);
    if (!ptr[dev]) {
        void *p = nullptr;
        AFSAI_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) AFSAI_FAIL(AFSAI_ERR_HIP, "afsai_apply_noalloc: no device address for the scratch array");
        ptr[dev] = (double *)p;
    }
    *out = ptr[dev];
    return AFSAI_OK;
}

}  // namespace afsai

extern "C" {

int afsai_apply_noalloc(afsai_precond P, const double *r, double *z, void *stream) {
    if (!P || !r || !z) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "afsai_apply_noalloc: null argument");
    if (r == z) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "afsai_apply_noalloc: r and z alias");
    if ((int64_t)P->n > kNoAllocMaxRows)
        AFSAI_FAIL(AFSAI_ERR_TOO_LARGE, "afsai_apply_noalloc: n = %d exceeds the scratch limit of %lld rows", P->n,
                   (long long)kNoAllocMaxRows);
    DeviceInfo di;
    int rc = device_info(&di);
    if (rc) return rc;
    double *t = nullptr;
    if ((rc = scratch_ptr(&t))) return rc;
    hipStream_t s = (hipStream_t)stream;
    // the products of afsai_apply, the whole matrix as one system (no device block maps)
    BatchMaps bm;
    bm.nt = stream_bytes(P->sg) + stream_bytes(P->sgt) > kCachedBytes;
    bm.sell.nblocks = blocks_for_slices(P->sg.nslices, di);
    sell_spmv("spmv_G", P->sg, bm, r, t, nullptr, nullptr, nullptr, FIN_NONE, di, s);
    bm.sell.nblocks = blocks_for_slices(P->sgt.nslices, di);
    sell_spmv("spmv_GT", P->sgt, bm, t, z, nullptr, nullptr, nullptr, FIN_NONE, di, s);
    AFSAI_HIP_TRY(hipGetLastError());
    return AFSAI_OK;
}

int pcg_solve(const afsai_csr *A, afsai_precond P, const double *b, double *x, double rtol, int32_t maxit,
              void *stream, afsai_pcg_info *info) {
    clear_error();
    int rc = check_csr_arg(A, "pcg_solve");
    if (rc) return rc;
    if (!b || !x) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve: null b or x");
    if (!(rtol > 0.0) || maxit < 0) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve: rtol = %g, maxit = %d", rtol, maxit);
    if (P && P->n != A->n) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve: preconditioner has n = %d, A has n = %d", P->n, A->n);
    if (P && P->seg_row0.size() > 2)
        AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve: the preconditioner is for a batch; use pcg_solve_batched");
    return pcg_batch(A, P, 1, nullptr, b, x, rtol, maxit, (hipStream_t)stream, info);
}

int pcg_solve_batched(const afsai_csr *A, afsai_precond P, int32_t nsys, const int32_t *offsets, const double *b,
                      double *x, double rtol, int32_t maxit, void *stream, afsai_pcg_info *info) {
    clear_error();
    int rc = check_csr_arg(A, "pcg_solve_batched");
    if (rc) return rc;
    if (!b || !x || !offsets || nsys < 1) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve_batched: null argument or nsys < 1");
    if (!(rtol > 0.0) || maxit < 0)
        AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve_batched: rtol = %g, maxit = %d", rtol, maxit);
    if (offsets[0] != 0 || offsets[nsys] != A->n)
        AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve_batched: offsets must run from 0 to n = %d", A->n);
    for (int k = 0; k < nsys; ++k)
        if (offsets[k + 1] <= offsets[k])
            AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve_batched: system %d is empty or offsets decrease", k);
    if (P) {
        if (P->n != A->n) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve_batched: preconditioner has n = %d, A has n = %d", P->n, A->n);
        const bool same = (nsys == 1 && P->seg_row0.size() <= 2) ||
                          (P->seg_row0.size() == (size_t)nsys + 1 &&
                           std::equal(P->seg_row0.begin(), P->seg_row0.end(), offsets));
        if (!same) AFSAI_FAIL(AFSAI_ERR_INVALID_ARG, "pcg_solve_batched: the preconditioner was set up for other systems");
    }
    return pcg_batch(A, P, nsys, offsets, b, x, rtol, maxit, (hipStream_t)stream, info);
}

}  // extern "C"
