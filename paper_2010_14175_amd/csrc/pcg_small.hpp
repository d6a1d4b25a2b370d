// A whole PCG solve of a small system in one launch, on the CUs of one XCD.
//
// Why: a solve of a small system is bound by its launches.  At 20^3
// (8,000 rows) an iteration is three kernels of 1.5 us of work each, but 6.5 us apart (start, cold
// caches, scalar loads, end): 0.83 ms for 34 iterations.  Blocks that stay and meet at a barrier
// need 1.1 us for it when they share an L2 (32 blocks, measured; kernels of the whole chip would have
// to write their L2s back at each barrier), and the matrix stays in that L2: 0.47 ms.
//
// The blocks: the launch puts as many on every XCD (blocks are dealt round robin); those that
// find themselves on the chosen XCD (its number is read from the hardware register, not assumed) take
// a rank each, the others return.  Vectors are written with plain stores, which reach the shared
// L2 before a thread arrives at the barrier (vmcnt(0)), and read with agent-scope loads, which pass
// the CU's own L1 by and hit in that L2.  Every wait is bounded: a block that waits too
// long gives up, all others then do, and the host solves the system the usual way.
//
// The arithmetic is the fused products' (k_sell_fused, k_sell_spmv): the same windows of four
// slices (one partial sum each), the same vector blocks at the start and for the final
// residual, the same order of every sum, so the iterates are theirs bit for bit.
#pragma once

namespace afsai {

constexpr int kSmallWin = 2;                        // windows of a block at most (8 wavefronts)
// Longest waits, in ticks of the 100 MHz clock.  At a launch's first barrier, where blocks that found no room may be
// missing (three solves' blocks on one XCD can keep each other out) and giving up costs nothing: 10 ms.  At
// the later ones all blocks are there and run; only a stopped queue is waited for: 20 s.
constexpr long long kSmallMeet = 1000000;
constexpr long long kSmallWait = 20LL * 100000000;

// what a launch leaves in the record's last word; the host puts SMALL_ABSENT there before it
enum : int { SMALL_RAN = 0, SMALL_UNMET = 1, SMALL_LOST = 2, SMALL_ABSENT = 3 };

// control words of a solve (zeroed before its launch)
struct SmallCtl {
    int32_t ticket;   // ranks given out
    uint32_t arrive;  // arrivals at the barriers
    int32_t dead;     // a block gave up
    int32_t pad;
};

struct SmallArgs {
    int n, nslices, a_entries, g_entries, t_entries;
    const uint32_t *a_sptr, *g_sptr, *t_sptr;
    const int32_t *a_col, *g_col, *t_col;
    const double *a_val;
    const void *g_val, *t_val;
    const int32_t *t_perm, *t_lens;  // G^T ordered by length in its windows (or null)
    const double *b;
    double *x, *r, *r2, *z, *p, *p2, *q, *t;
    double *pq, *rr, *rz;  // partial sums
    PcgScalars *sc, *host;
    SmallCtl *ctl;
    int blocks, xcc, nbv;  // blocks that take part, their XCD, vector blocks
    int iter0, iters;      // iterations done before this launch, and most of it
    int miss;              // arrivals that the first barrier waits for and nobody makes (0 but in tests)
    int late;              // the last block comes after the others have given up (tests)
};

// pointers in the global address space (a flat load would also wait for LDS)
template <typename T>
using Glob = __attribute__((address_space(1))) T *;
template <typename T>
__device__ __forceinline__ Glob<T> glob(T *p) { return (Glob<T>)p; }
__device__ __forceinline__ double ld_agent(const double *p) {
    return __hip_atomic_load(glob(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// a vector read by index with agent scope (buffer loads, cache policy bit sc1): scheduled like
// ordinary loads, one offset register each
struct SharedVec {
    __amdgpu_buffer_rsrc_t rs;
    __device__ __forceinline__ SharedVec(const double *p, int n)
        : rs(__builtin_amdgcn_make_buffer_rsrc((void *)p, 0, n * 8, 0x00027000)) {}
    __device__ __forceinline__ double operator()(int c) const {
        const auto w = __builtin_amdgcn_raw_buffer_load_b64(rs, c * 8, 0, 16);
        return __hiloint2double((int)w[1], (int)w[0]);
    }
};
__device__ __forceinline__ int xcc_id() { return __builtin_amdgcn_s_getreg((3 << 11) | 20) & 15; }  // HW_REG_XCC_ID

// which XCDs there are: bit k for XCD k
__global__ void k_xcc_mask(uint32_t *mask) {
    if (threadIdx.x == 0) atomicOr(mask, 1u << xcc_id());
}

// the control words before another launch of a solve
__global__ void k_small_again(SmallCtl *ctl) {
    if (threadIdx.x == 0) *ctl = SmallCtl{};
}

// A SELL-64 matrix behind buffer descriptors (32-bit offsets: one register an address)
template <typename VT>
struct SmallMat {
    __amdgpu_buffer_rsrc_t cr, vr;
    __device__ __forceinline__ SmallMat(const int32_t *col, const void *val, int entries)
        : cr(__builtin_amdgcn_make_buffer_rsrc((void *)col, 0, entries * 4, 0x00027000)),
          vr(__builtin_amdgcn_make_buffer_rsrc((void *)val, 0, entries * (int)sizeof(VT), 0x00027000)) {}
    __device__ __forceinline__ int col(int e) const { return (int)__builtin_amdgcn_raw_buffer_load_b32(cr, e * 4, 0, 0); }
    __device__ __forceinline__ double val(int e) const {
        if constexpr (sizeof(VT) == 4) return (double)__uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(vr, e * 4, 0, 0));
        const auto w = __builtin_amdgcn_raw_buffer_load_b64(vr, e * 8, 0, 0);
        return __hiloint2double((int)w[1], (int)w[0]);
    }
};

// A lane's row in a slice: its first entry, the slice's width (a scalar), its own length, and the
// columns of its first U entries, which stay in registers for the whole solve
template <int U>
struct SmallRow {
    int base, width, len;
    int c[U];
    template <typename M>
    __device__ __forceinline__ void init(const M &m, const uint32_t *sptr, const int32_t *lens, int sl, bool on) {
        const int lane = threadIdx.x & 63;
        base = width = len = 0;
        if (!on) return;
        const uint32_t c0 = glob(sptr)[sl];
        base = (int)c0 * kSlice + lane;
        width = __builtin_amdgcn_readfirstlane((int)(glob(sptr)[sl + 1] - c0));
        len = lens ? glob(lens)[(int64_t)sl * kSlice + lane] : width;
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = width > 0 ? m.col(base + min(u, width - 1) * kSlice) : 0;
    }
};

// The fma chain over the row (lane_chain's order), the gathered entry given by f(column).  The
// columns are loaded one round ahead, the values with the gathers; loads past the width repeat
// the last entry (no branches around them) and are not added.
template <int U, typename M, typename F>
__device__ __forceinline__ double small_chain(const SmallRow<U> &row, const M &m, F f) {
    double acc = 0.0;
    if (row.width <= 0) return acc;
    int c[U];
#pragma unroll
    for (int u = 0; u < U; ++u) c[u] = row.c[u];
    for (int k0 = 0; k0 < row.width; k0 += U) {
        int cn[U];
        double v[U], xv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            v[u] = m.val(row.base + min(k0 + u, row.width - 1) * kSlice);
            cn[u] = 0;
        }
        if (k0 + U < row.width)
#pragma unroll
            for (int u = 0; u < U; ++u) cn[u] = m.col(row.base + min(k0 + U + u, row.width - 1) * kSlice);
#pragma unroll
        for (int u = 0; u < U; ++u) xv[u] = f(c[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double t = fma(v[u], xv[u], acc);
            acc = k0 + u < row.len ? t : acc;
            c[u] = cn[u];
        }
    }
    return acc;
}

// Two blocks of 8 wavefronts fit a CU at 128 registers, so that two solves on one XCD can both
// be resident as a whole.
template <typename VT, bool ORD>
__global__ __launch_bounds__(kSmallWin * kThreads) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_pcg_small(SmallArgs a) {
    constexpr int U = 8;
    __shared__ int s_rank, s_dead;
    __shared__ double sh[kSmallWin * 4], sh2[kSmallWin * 4], s_sum[8];
    __shared__ double win[ORD ? kSmallWin * kThreads : 1];
    if (xcc_id() != a.xcc) return;
    if (threadIdx.x == 0) s_rank = __hip_atomic_fetch_add(glob(&a.ctl->ticket), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int rank = s_rank;
    if (rank >= a.blocks) return;

    const int lane = threadIdx.x & 63;
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int ng = blockDim.x / kThreads, grp = wid >> 2, wv = wid & 3;  // groups of four wavefronts
    // this group's window (one vector block too, where there are as many) and the wavefront's slice
    const int w = rank * ng + grp, sl = w * kWin + wv, r = sl * kSlice + lane;
    const int nw = (a.nslices + kWin - 1) / kWin;
    const bool on = sl < a.nslices, has = on && r < a.n;
    SmallRow<U> ra, rg, rt;
    const SmallMat<double> ma(a.a_col, a.a_val, a.a_entries);
    const SmallMat<VT> mg(a.g_col, a.g_val, a.g_entries), mt(a.t_col, a.t_val, a.t_entries);
    ra.init(ma, a.a_sptr, nullptr, sl, on);
    rg.init(mg, a.g_sptr, nullptr, sl, on);
    rt.init(mt, a.t_sptr, ORD ? a.t_lens : nullptr, sl, on);
    int rperm = -1;  // with ordered windows: the row this lane multiplies
    if (ORD && on) rperm = glob(a.t_perm)[(int64_t)sl * kSlice + lane];
    uint32_t phase = 0;
    if (a.late && rank == a.blocks - 1)
        for (const long long t0 = wall_clock64(); wall_clock64() - t0 < 3 * kSmallMeet;) __builtin_amdgcn_s_sleep(64);

    // all blocks' stores before it are in the L2 after it; false: given up.  A block that gives up takes its
    // arrival back, if the barrier is still short of one: then it stays short for every block, also for one that
    // comes late, and either all pass a barrier or none does.
    auto barrier = [&]() __attribute__((always_inline)) -> bool {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        ++phase;
        if (threadIdx.x == 0) {
            __hip_atomic_fetch_add(glob(&a.ctl->arrive), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t want = phase * (uint32_t)a.blocks + (phase == 1 ? (uint32_t)a.miss : 0u);
            const long long longest = phase == 1 ? kSmallMeet : kSmallWait;
            int dead = 0;
            // (the clock and the other blocks' state only now and then: both are slow to read)
            long long t0 = 0;
            for (uint32_t spin = 1;
                 __hip_atomic_load(glob(&a.ctl->arrive), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < want; ++spin) {
                if (spin % 1024) continue;
                const long long now = wall_clock64();
                if (t0 == 0) t0 = now;
                if (__hip_atomic_load(glob(&a.ctl->dead), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ||
                    now - t0 > longest) {
                    uint32_t seen = __hip_atomic_load(glob(&a.ctl->arrive), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    while (seen < want && !dead)  // (a failed exchange reads seen anew)
                        dead = __hip_atomic_compare_exchange_strong(glob(&a.ctl->arrive), &seen, seen - 1, __ATOMIC_RELAXED,
                                                                    __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (dead) __hip_atomic_store(glob(&a.ctl->dead), 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
            }
            s_dead = dead;
        }
        __syncthreads();
        return s_dead == 0;
    };
    // sums of two partial arrays in parts_sum's order (256 threads, runs of `per`)
    auto sums = [&](const double *pa, const double *pb, int np, double &sa, double &sb) __attribute__((always_inline)) {
        double va = 0.0, vb = 0.0;
        if (threadIdx.x < kThreads) {
            const int per = (np + kThreads - 1) / kThreads;
            const int lo = threadIdx.x * per, hi = min(np, lo + per);
            for (int j = lo; j < hi; ++j) {
                va += ld_agent(pa + j);
                if (pb) vb += ld_agent(pb + j);
            }
            va = wave_sum(va);
            vb = wave_sum(vb);
            if (lane == 0) {
                s_sum[wid] = va;
                s_sum[4 + wid] = vb;
            }
        }
        __syncthreads();
        sa = sb = 0.0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            sa += s_sum[j];
            sb += s_sum[4 + j];
        }
        __syncthreads();
    };
    // the four wavefronts' parts of a group to one partial sum (two of them with pb) at w < count
    auto store_parts = [&](double va, double vb, int count, double *pa, double *pb) __attribute__((always_inline)) {
        va = wave_sum(va);
        if (pb) vb = wave_sum(vb);
        if (lane == 0) {
            sh[wid] = va;
            sh2[wid] = vb;
        }
        __syncthreads();
        if (wv == 0 && lane == 0 && w < count) {
            double ta = 0.0, tb = 0.0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                ta += sh[grp * 4 + j];
                tb += sh2[grp * 4 + j];
            }
            glob(pa)[w] = ta;
            if (pb) glob(pb)[w] = tb;
        }
    };
    // y = M x (plain order)
    auto product = [&](const SmallRow<U> &row, const auto &m, const double *xin, double *y) __attribute__((always_inline)) {
        const double acc = small_chain<U>(row, m, SharedVec(xin, a.n));
        if (has) glob(y)[r] = acc;
    };
    // z = G^T t and the partial sums of z.v
    auto product_t = [&](const double *v) __attribute__((always_inline)) {
        double zn = small_chain<U>(rt, mt, SharedVec(a.t, a.n)), part = 0.0;
        if constexpr (ORD) {  // the row sums go to their natural rows through LDS
            if (rperm >= 0) win[grp * kThreads + rperm - w * kWin * kSlice] = zn;
            __syncthreads();
            zn = win[grp * kThreads + wv * kSlice + lane];
        }
        if (has) {
            glob(a.z)[r] = zn;
            part = fma(zn, ld_agent(v + r), part);
        }
        store_parts(part, 0.0, nw, a.rz, nullptr);
    };
    // rows of vector block w, where there is one
    int i0 = 0, i1 = 0;
    if (w < a.nbv) block_range(0, a.n, w, a.nbv, i0, i1);
    i0 += threadIdx.x & (kThreads - 1);

    PcgScalars st = *a.sc;
    auto solve = [&]() __attribute__((always_inline)) -> bool {
        if (a.iter0 == 0) {
            // r = b - A x0; b.b, r.r over the vector blocks
            product(ra, ma, a.x, a.q);
            if (!barrier()) return false;
            double pb = 0.0, pr = 0.0;
            for (int j = i0; j < i1; j += kThreads) {
                const double bj = glob(a.b)[j], rj = bj - ld_agent(a.q + j);
                glob(a.r)[j] = rj;
                pb = fma(bj, bj, pb);
                pr = fma(rj, rj, pr);
            }
            store_parts(pb, pr, a.nbv, a.pq, a.rr);
            if (!barrier()) return false;
            double bb, rr;
            sums(a.pq, a.rr, a.nbv, bb, rr);
            init_scalars(st, bb, rr);
            if (!st.done) {
                product(rg, mg, a.r, a.t);
                if (!barrier()) return false;
                product_t(a.r);
                if (!barrier()) return false;
                double rz, u;
                sums(a.rz, nullptr, nw, rz, u);
                st.rho = rz;
            }
        }
        for (int it = 0; it < a.iters && !st.done; ++it) {
            const int no = a.iter0 + it;
            const bool odd = no & 1;
            const double *p_old = odd ? a.p2 : a.p, *r_old = odd ? a.r2 : a.r;
            double *p_new = odd ? a.p : a.p2, *r_new = odd ? a.r : a.r2;
            const SharedVec zv(a.z, a.n), pov(p_old, a.n), rov(r_old, a.n), qv(a.q, a.n);
            // p = z + beta p (p = z first), q = A p, p.q
            const double beta = st.beta;
            const auto pv = [&](int c) __attribute__((always_inline)) { return fma(beta, pov(c), zv(c)); };
            double part = 0.0, own = 0.0;
            double acc = no == 0 ? small_chain<U>(ra, ma, zv) : small_chain<U>(ra, ma, pv);
            if (has) {
                own = no == 0 ? zv(r) : pv(r);
                glob(p_new)[r] = own;
                glob(a.q)[r] = acc;
                part = fma(own, acc, part);
            }
            const double p_r = own;
            store_parts(part, 0.0, nw, a.pq, nullptr);
            if (!barrier()) return false;
            double pq, u;
            sums(a.pq, nullptr, nw, pq, u);
            if (!(pq > 0.0) || !isfinite(pq)) {
                st.done = DONE_NOT_SPD;
                break;
            }
            // r -= alpha q, x += alpha p, t = G r, r.r
            const double alpha = st.rho / pq;
            const auto rv = [&](int c) __attribute__((always_inline)) { return fma(-alpha, qv(c), rov(c)); };
            acc = small_chain<U>(rg, mg, rv);
            part = 0.0;
            if (has) {
                own = rv(r);
                glob(r_new)[r] = own;
                glob(a.t)[r] = acc;
                glob(a.x)[r] = fma(alpha, p_r, glob(a.x)[r]);
                part = fma(own, own, part);
            }
            store_parts(part, 0.0, nw, a.rr, nullptr);
            if (!barrier()) return false;
            product_t(r_new);
            if (!barrier()) return false;
            double rr, rz;
            sums(a.rr, a.rz, nw, rr, rz);
            advance(st, rr, rz, 0);
        }
        if (st.done) {
            // x = 0 for a zero right-hand side; the true residual ||b - A x||^2
            if (st.done == DONE_ZERO_RHS && has) glob(a.x)[r] = 0.0;
            if (!barrier()) return false;
            product(ra, ma, a.x, a.q);
            if (!barrier()) return false;
            double pr = 0.0;
            for (int j = i0; j < i1; j += kThreads) {
                const double d = glob(a.b)[j] - ld_agent(a.q + j);
                pr = fma(d, d, pr);
            }
            store_parts(pr, 0.0, a.nbv, a.pq, nullptr);
            if (!barrier()) return false;
            double rs, u;
            sums(a.pq, nullptr, a.nbv, rs, u);
            st.resid = rs;
        }
        return true;
    };
    const bool ok = solve();
    if (threadIdx.x == 0 && (rank == 0 || !ok)) {
        // given up: UNMET while x, r, z, p and the scalars are those from before the launch (its first
        // barrier; of the first launch, which can be begun anew, the start's four)
        st.pad = ok ? SMALL_RAN : (phase <= (a.iter0 == 0 ? 4u : 1u) ? SMALL_UNMET : SMALL_LOST);
        *a.sc = st;
        *a.host = st;
    }
}

}  // namespace afsai
