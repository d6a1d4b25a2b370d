// The per-row adaptive FSAI setup (Sec. 2) in inverse-factor form (rows_w.hpp) for matrices
// whose rows are made of aligned runs of three columns (3c, 3c+1, 3c+2), as a discretisation
// with three unknowns per node gives: the candidate table holds runs, not columns.
//
// Why: k_rows_w is bound by instruction issue (0.81 of the VALU limit at 64^3) and spends half
// of it on one table lookup and one slot per matrix entry.  A row of 81 entries is 27 runs, so
// 32 lanes take a whole row of A: one lookup, one slot byte and one 24-byte load per lane
// serve three entries.  Patterns of up to 32 positions put two rows on a wavefront (32 lanes
// each); larger ones keep one row per wavefront, whose halves take two member rows (and two
// gathered rows) at once.  The slot bytes need 6 registers where k_rows_w keeps 24 (48).
// Measured: this kernel takes 10.2 ms at 64^3 (21 positions) and 571 ms at 150^3 (46 positions),
// k_rows_w 20.4 and 985 ms before.  Now bound by the LDS (0.7 of its cycles in use at 64^3, half of
// that for the gradients' additions) and instruction issue (0.7) alike, with 16 and 11 wavefronts
// per CU by LDS; a tenth fewer vector instructions alone changed nothing.
//
// Layout of one row group (LDS): per table slot the run's first column, a word with one byte
// per column (0: candidate, p + 1: member at position p) and three gradients (one plane per
// column of the run, so that a lane-wise scan is free of bank conflicts); then W as in
// rows_w.hpp.  A table slot is the run's place in the hash table (buckets of four keys).
//
// Results are those of k_rows_w bit for bit: every gradient receives its terms in the same
// order (member rows in turn, the second half of the wavefront after the first, the columns of
// one member row distinct), the selection takes the same maximum and the same smallest
// column in the band, and extend_w is shared, over the same blocks of new rows.
#pragma once

#include "rows_w.hpp"

#pragma clang fp contract(off)

namespace afsai {
namespace bform {

using wform::gred;
using wform::Memb;
using wform::OpMax;
using wform::OpMinU;
using wform::wsync;
using wform::wu;

constexpr int kEmpty = 0x7FFFFFF0;  // above every column, and so is kEmpty + 2
constexpr int kRunRow = 32;         // runs of a row of A at most (one per lane of 32)

template <int GS, int MMAX, int CAPT, int NB>
struct Layout {
    static constexpr int VALB = 3 * CAPT * 8;
    static constexpr int LDV = MMAX + 2;  // rows of NR and LV (see rows_w.hpp)
    static constexpr int ALV = 2 * NB * LDV + NB;  // NR, LV, NAI in doubles
    static constexpr int O_KEY = 0;
    static constexpr int O_INF = CAPT * 4;
    static constexpr int O_VAL = CAPT * 8;
    static constexpr int O_MS = O_VAL + VALB;  // Memb[MMAX] (product pass)
    static constexpr int O_SEL = O_MS;         // sel, row start, row end [MMAX] (from the selection on)
    static constexpr int FIXED = wform::al16(O_MS + MMAX * 16);
    // between the selection and the next product pass the gradient planes hold the gathered rows
    // and product vectors
    static_assert(ALV * 8 <= VALB, "the step's vectors fit in the gradient planes");
    static_assert(CAPT % 4 == 0 && CAPT <= 256, "buckets of four keys, slots in a byte");
    // (the first of the 8 doubles after W is the matrix products' zero)
    // rows of W kept for patterns of at most mm positions grown s at a time: all but the last block
    // of the last step
    static __host__ __device__ constexpr int w_rows(int mm, int s) { return mm > 1 ? mm - 1 - ((s - 1) % NB + 1) : 0; }
    static __host__ __device__ constexpr int bytes(int mm, int s) {
        return FIXED + wform::al16((wform::tri_w(w_rows(mm, s)) + 8) * 8);
    }
};

// Finds the run starting at column c, inserting it when absent if `add`; its slot, or -1 (when
// the table is full, or the run is absent and not to be added).  Two lanes looking up one new run at once (two gathered rows) get the same slot:
// one claim wins, the other returns the slot that now holds its run.
template <int CAPT>
__device__ __forceinline__ int bfind(int32_t *hkey, int c, bool add) {
    constexpr int NBK = CAPT / 4;
    uint32_t b = __umulhi((uint32_t)c * 2654435761u, (uint32_t)NBK);
    for (int probe = 0; probe < NBK;) {
        const int4 k4 = *reinterpret_cast<const int4 *>(&hkey[4 * b]);
        const int kk[4] = {k4.x, k4.y, k4.z, k4.w};
        int empty = -1, hit = -1;
#pragma unroll
        for (int e = 3; e >= 0; --e) {
            empty = kk[e] == kEmpty ? e : empty;
            hit = kk[e] == c ? e : hit;
        }
        if (hit >= 0) return (int)(4 * b) + hit;
        if (empty < 0) {
            b = b + 1 < (uint32_t)NBK ? b + 1 : 0u;
            ++probe;
            continue;
        }
        if (!add) return -1;
        const int old = atomicCAS(&hkey[4 * b + empty], kEmpty, c);
        if (old == kEmpty || old == c) return (int)(4 * b) + empty;
    }
    return -1;
}

// The two largest |gradient| of this lane's table entries and their places (4 * scan step +
// column of the run); members, empty slots and columns from i on hold NaN, which counts as -1
template <int GS, int CAPT>
__device__ __forceinline__ void btop2(const double *hval, int gl, double &a1, double &a2, int &i1, int &i2) {
    a1 = -1.0;
    a2 = -1.0;
    i1 = i2 = 0;
#pragma unroll
    for (int jj = 0; jj < (CAPT + GS - 1) / GS; ++jj) {
        const int e = gl + GS * jj;
        double v[3];
#pragma unroll
        for (int x = 0; x < 3; ++x) v[x] = (CAPT % GS == 0 || e < CAPT) ? hval[x * CAPT + e] : -1.0;
#pragma unroll
        for (int x = 0; x < 3; ++x) {
            const bool in = CAPT % GS == 0 || e < CAPT;
            const double a = in ? fmax(fabs(v[x]), -1.0) : -1.0;
            const bool g1 = a > a1, g2 = a > a2;
            i2 = g1 ? i1 : (g2 ? 4 * jj + x : i2);
            i1 = g1 ? 4 * jj + x : i1;
            a2 = fmax(a2, fmin(a1, a));
            a1 = fmax(a1, a);
        }
    }
}

template <int GS, int MMAX, int CAPT, int NB, int WPE>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WPE, 8))) void k_rows_b(
    int n, const int32_t *__restrict__ rp, const int32_t *__restrict__ ci, const double *__restrict__ av,
    const float *__restrict__ /*av32*/, const double *__restrict__ diag, const int32_t *__restrict__ dlo, int kmax, int s,
    double eps, double tau, int /*gmax*/, const int32_t *__restrict__ list, int nlist, int32_t *__restrict__ counters,
    int nxcd, int claim, int32_t *__restrict__ ell_col, double *__restrict__ ell_val, int ldell,
    int32_t *__restrict__ m_out, double *__restrict__ psi_out, int32_t *__restrict__ steps_out,
    int32_t *__restrict__ reason_out, int8_t *__restrict__ status_out, int32_t *__restrict__ ovf_count,
    int32_t *__restrict__ ovf_list) {
    using LY = Layout<GS, MMAX, CAPT, NB>;
    static_assert(GS == 32 || GS == 64, "32 lanes take a row of A");
    static_assert(MMAX <= GS, "one lane per pattern position");
    constexpr int RPW = 64 / GS;                   // rows per wavefront
    constexpr int LDV = LY::LDV;
    constexpr int HPG = GS / 32;                   // rows of A a group takes at once
    constexpr int SPL = (CAPT + GS - 1) / GS;      // table slots per lane
    constexpr int NGR = (NB + HPG - 1) / HPG;      // rounds of gathered rows
    constexpr int NSL = (MMAX / HPG + 3) / 4;      // slot registers (four bytes each)
    static_assert(MMAX % (4 * HPG) == 0, "whole rounds");

    extern __shared__ __align__(16) unsigned char lds_w[];
    __shared__ int32_t s_row;
    const int lane = threadIdx.x;
    const int gl = lane & (GS - 1), grp = lane / GS;
    const int hl = lane & 31, half = HPG == 2 ? lane >> 5 : 0;
    const int mmx = kmax > 0 ? 1 + kmax * s : 1;  // largest pattern
    const int wrows = LY::w_rows(mmx, s), gbytes = LY::bytes(mmx, s);
    unsigned char *gbase = lds_w + grp * gbytes;
    int32_t *hkey = reinterpret_cast<int32_t *>(gbase + LY::O_KEY);
    uint32_t *hinf = reinterpret_cast<uint32_t *>(gbase + LY::O_INF);
    double *hval = reinterpret_cast<double *>(gbase + LY::O_VAL);  // [3][CAPT]
    double *Wm = reinterpret_cast<double *>(gbase + LY::FIXED);
    Memb *memb = reinterpret_cast<Memb *>(gbase + LY::O_MS);        // [MMAX], lengths in runs
    int32_t *sel = reinterpret_cast<int32_t *>(gbase + LY::O_SEL);  // [MMAX] selected columns
    int32_t *selb = sel + MMAX;                                     // [MMAX] their row starts
    int32_t *sele = selb + MMAX;                                    // [MMAX] their row ends
    double *NR = hval;                                              // [NB][LDV]
    double *LV = NR + NB * LDV;                                     // [NB][LDV]
    double *NAI = LV + NB * LDV;                                    // [NB]: a_{u,i}
    const uint64_t gm = wform::group_bits<GS>(grp);
    const int zslot = wform::tri_w(wrows);  // of the padding after W, zero for the matrix products
    if (gl == 0) Wm[zslot] = 0.0;
    const double kNaN = __longlong_as_double(0x7FF8000000000000ll);

    const int x = blockIdx.x % nxcd;
    const int64_t per = ((int64_t)nlist + nxcd - 1) / nxcd;
    const int q0 = (int)min<int64_t>(nlist, per * x), q1 = (int)min<int64_t>(nlist, per * (x + 1));
    const int take = claim * RPW;

    int qn = 0, qe = 0;
    for (;;) {
        if (qn >= qe) {
            if (lane == 0) s_row = q0 + atomicAdd(&counters[x], take);
            __syncthreads();
            qn = __builtin_amdgcn_readfirstlane(s_row);  // the block is one wavefront: a scalar
            __syncthreads();
            if (qn >= q1) break;
            qe = min(qn + take, q1);
        }
        const int qi = qn + grp;
        qn += RPW;
        const bool have = qi < qe;
        const int i = have ? (list ? list[qi] : qi) : 0;

        // ---- row state (uniform inside the group) and per-position registers
        int8_t status = ROW_OK;
        int32_t reason = STOP_KMAX;
        int steps = 0, m_o = 0;
        double aii = 1.0;
        int ibeg = 0, ilen = 0;
        if (have) {
            aii = diag[i];
            ibeg = rp[i];
            ilen = (dlo[i] + 2) / 3;  // runs that start left of column i
        }
        bool act = have;
        if (act && (!(aii > 0.0) || !isfinite(aii))) {
            status = ROW_NOT_SPD;
            act = false;
        }
        double psi = aii;
        const double psi0 = aii;
        double gi = act ? 1.0 / sqrt(aii) : 0.0;
        int r_col = 0, r_beg = 0, r_len = 0;
        double r_g = 0.0, r_ai = 0.0;
        double yi = 0.0;  // lane j: (W^T l_i)_j
        // slot of this lane's run in member row q (0: row i, q: position q - 1): byte q / HPG, in
        // the half q % HPG
        uint32_t slr[NSL];
#pragma unroll
        for (int r = 0; r < NSL; ++r) slr[r] = 0u;
#pragma unroll
        for (int jj = 0; jj < SPL; ++jj) {
            const int e = gl + GS * jj;
            if (CAPT % GS == 0 || e < CAPT) {
                hkey[e] = kEmpty;
                hinf[e] = 0u;
            }
        }
        wsync();
        if (act && kmax > 0) {
            // row i's runs left of the diagonal: the first candidates
            bool bad = ilen > kRunRow;
            if (half == 0 && hl < ilen) {
                const int slot = bfind<CAPT>(hkey, ci[ibeg + 3 * hl], true);
                if (slot < 0) bad = true;
                else slr[0] |= (uint32_t)slot;
            }
            if (__ballot(bad) & gm) {
                status = ROW_OVERFLOW;
                act = false;
            }
        }

        for (int k = 1; k <= kmax; ++k) {
            if (!__ballot(act)) break;

            // ---- 1. product pass
            if (wu<GS>(act)) {
                // zero gradients; NaN for members, columns from i on and empty slots
#pragma unroll
                for (int jj = 0; jj < SPL; ++jj) {
                    const int e = gl + GS * jj;
                    if (CAPT % GS == 0 || e < CAPT) {
                        const int c0 = hkey[e];
                        const uint32_t f = hinf[e];
#pragma unroll
                        for (int y = 0; y < 3; ++y)
                            hval[y * CAPT + e] = (c0 + y >= i || (f & (0xFFu << (8 * y)))) ? kNaN : 0.0;
                    }
                }
                if (gl == 0) memb[0] = Memb{ibeg, ilen, gi};
                if (gl < m_o) memb[gl + 1] = Memb{r_beg, r_len, r_g};
            }
            wsync();
            const int mo_u = wu<GS>(m_o);
            if (wu<GS>(act)) {
                // four member rows (of each half) at a time; lanes without a run load the row's first
                // (loads under a condition made the ones behind them wait: 150^3 590 -> 571 ms; the next
                // rows' loads between the additions: 581)
                double aa[4][3], gg[4];
                int len[4];
                auto load = [&](int q, int u) __attribute__((always_inline)) {
                    const Memb mb = memb[min(q, mo_u)];
                    len[u] = q <= mo_u ? mb.len : 0;
                    gg[u] = mb.g;
                    const double *a = av + mb.beg + (hl < len[u] ? 3 * hl : 0);
#pragma unroll
                    for (int y = 0; y < 3; ++y) aa[u][y] = a[y];
                };
#pragma unroll
                for (int qb = 0; qb < MMAX; qb += 4 * HPG) {
                    if (qb <= mo_u) {
#pragma unroll
                        for (int u = 0; u < 4; ++u) load(qb + u * HPG + half, u);
                        const uint32_t sw = slr[qb / (4 * HPG)];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            double *h = hval + ((sw >> (8 * u)) & 0xFFu);
                            // the halves in turn: a slot's terms in the order of the members
#pragma unroll
                            for (int hh = 0; hh < HPG; ++hh) {
                                if (half == hh && hl < len[u]) {
#pragma unroll
                                    for (int y = 0; y < 3; ++y)
                                        __hip_atomic_fetch_add(h + y * CAPT, aa[u][y] * gg[u], __ATOMIC_RELAXED,
                                                               __HIP_MEMORY_SCOPE_WORKGROUP);
                                }
                                if constexpr (HPG > 1) wsync();
                            }
                        }
                    }
                }
            }
            wsync();

            // ---- 2. selection (as in k_rows_w, over the runs' columns)
            int ns = 0;
            int r_js = 0, r_nb = 0, r_ne = 0;  // lane v: v-th column selected in this step, its row extents
            if (wu<GS>(act)) {
                double a1, a2;
                int i1, i2;
                btop2<GS, CAPT>(hval, gl, a1, a2, i1, i2);
                const double M = gred<GS, OpMax>(a1);
                // (beside an infinite gradient none is eligible: the row stops)
                if (wu<GS>(M > 0.0 && M < INFINITY)) {
                    const double thr = 0x1.0p-40 * M;
                    bool partial = false;
                    for (int round = 0; round < s; ++round) {
                        const double v1 = a1 > thr ? a1 : -1.0;
                        const double v2 = a2 > thr ? a2 : -1.0;
                        const double Mp = round == 0 ? M : gred<GS, OpMax>(v1);
                        if (!wu<GS>(Mp > 0.0)) break;
                        const double band = (1.0 - tau) * Mp;
                        const bool slow = (__ballot(v2 >= band || (partial && v1 >= band)) & gm) != 0;
                        uint32_t lb = wform::kEmptyKey;
                        int le = 0, ly = 0;
                        if (!slow) {
                            if (v1 >= band) {
                                le = gl + GS * (i1 >> 2);
                                ly = i1 & 3;
                                lb = (uint32_t)(hkey[le] + ly);
                            }
                        } else {
#pragma unroll 2
                            for (int jj = 0; jj < SPL; ++jj) {
                                const int e = gl + GS * jj;
                                if (CAPT % GS == 0 || e < CAPT) {
                                    const uint32_t c0 = (uint32_t)hkey[e];
                                    for (int y = 0; y < 3; ++y) {
                                        const double a = fabs(hval[y * CAPT + e]);
                                        if (a > thr && a >= band && c0 + y < lb) {
                                            lb = c0 + y;
                                            le = e;
                                            ly = y;
                                        }
                                    }
                                }
                            }
                        }
                        const uint32_t js = gred<GS, OpMinU>(lb);
                        const bool won = lb == js && js != wform::kEmptyKey;
                        if (won) {
                            hinf[le] |= (uint32_t)(m_o + ns + 1) << (8 * ly);
                            hval[ly * CAPT + le] = kNaN;
                        }
                        if (!slow) {
                            a1 = won ? a2 : a1;
                            i1 = won ? i2 : i1;
                            a2 = won ? -1.0 : a2;
                            partial = partial || won;
                        } else {
                            wsync();
                            btop2<GS, CAPT>(hval, gl, a1, a2, i1, i2);
                            partial = false;
                        }
                        // the new row's extents, loaded while the next rounds run
                        if (gl == ns) {
                            r_js = (int)js;
                            r_nb = rp[js];
                            r_ne = rp[js + 1];
                        }
                        ++ns;
                    }
                }
                if (ns == 0) {
                    reason = STOP_NOCAND;
                    act = false;
                }
            }
            wsync();
            // the selected columns in the place of the member records (no longer read this step)
            if (act && gl < ns) {
                sel[gl] = r_js;
                selb[gl] = r_nb;
                sele[gl] = r_ne;
            }
            wsync();

            // ---- 3./4. gather the new rows and extend W, NB rows at a time
            bool spd = true;
            int nsd = 0;
            // the last step's rows are looked up but not entered: no product pass follows
            const bool more = k < kmax;
            const int nsw = GS == 64 ? wu<GS>(ns)
                                     : __builtin_amdgcn_readfirstlane((int)gred<64, OpMax>((double)(act ? ns : 0)));
            for (int nw = 0; nw < nsw; nw += NB) {
                // old positions of this block (earlier blocks of the step included)
                const int mwb = GS == 64 ? wu<GS>(m_o)
                                         : __builtin_amdgcn_readfirstlane((int)gred<64, OpMax>((double)(act ? m_o : 0)));
                const int mo = wu<GS>(m_o);  // this row's old positions (a scalar with 64 lanes)
                const bool blk = wu<GS>(act && nsd < ns);
                const int nbk = wu<GS>(blk ? min(NB, ns - nsd) : 0);
                if (blk) {
#pragma unroll
                    for (int jj = 0; jj < (NB * LDV + GS - 1) / GS; ++jj)
                        if (gl + GS * jj < NB * LDV) NR[gl + GS * jj] = 0.0;
                    if (gl < NB) NAI[gl] = 0.0;
                }
                wsync();
                bool bad = false;
                // new row v is member mo + v + 1: the half with that parity takes it
                const int flip = HPG == 2 ? (half ^ ((mo + 1) & 1)) : 0;
                if (blk) {
                    int gc[NGR];
                    double ga[NGR][3];
#pragma unroll
                    for (int w = 0; w < NGR; ++w) {
                        const int v = w * HPG + flip;
                        gc[w] = kEmpty;
#pragma unroll
                        for (int y = 0; y < 3; ++y) ga[w][y] = 0.0;
                        if (v < nbk) {
                            const int nb = selb[nsd + v], ln = sele[nsd + v] - nb;
                            if (ln > 3 * kRunRow) bad = true;
                            if (3 * hl < ln) {
                                gc[w] = ci[nb + 3 * hl];
                                const double *a = av + nb + 3 * hl;
#pragma unroll
                                for (int y = 0; y < 3; ++y) ga[w][y] = a[y];
                            }
                        }
                    }
                    int mylen = 0;  // lane mo + v: runs of new row v left of column i
#pragma unroll
                    for (int w = 0; w < NGR; ++w) {
                        const int v = w * HPG + flip;
                        const int c0 = gc[w];
                        const bool lo = c0 < i;
                        if (c0 <= i && i < c0 + 3) NAI[v] = c0 == i ? ga[w][0] : (c0 + 1 == i ? ga[w][1] : ga[w][2]);
                        int slot = 0;
                        if (lo) {
                            slot = bfind<CAPT>(hkey, c0, more);
                            if (slot < 0) {
                                bad = bad || more;
                            } else {
                                const uint32_t f = hinf[slot];
#pragma unroll
                                for (int y = 0; y < 3; ++y) {
                                    const int ps = (int)((f >> (8 * y)) & 0xFFu);
                                    if (ps) NR[v * LDV + ps - 1] = ga[w][y];
                                }
                            }
                        }
                        const uint32_t sb = lo && slot >= 0 ? (uint32_t)slot : 0u;
                        // byte of the member in this half's registers
                        const int qi8 = (mo + v + 1) / HPG;
#pragma unroll
                        for (int r = 0; r < NSL; ++r) slr[r] |= (qi8 >> 2) == r ? sb << (8 * (qi8 & 3)) : 0u;
                        // (the columns left of i are the first of the row)
                        const uint64_t bl = __ballot(lo);
#pragma unroll
                        for (int h = 0; h < HPG; ++h) {
                            const int vh = HPG == 2 ? w * HPG + (h ^ ((mo + 1) & 1)) : w;
                            const int cnt = __popc((uint32_t)(HPG == 2 ? bl >> (32 * h) : bl >> (32 * grp)));
                            if (gl == mo + vh && vh < nbk) mylen = cnt;
                        }
                    }
                    if (gl >= mo && gl < mo + nbk) {
                        r_beg = selb[nsd + gl - mo];
                        r_col = sel[nsd + gl - mo];
                        r_len = mylen;
                    }
                }
                if (__ballot(bad) & gm) {
                    if (blk) {
                        status = ROW_OVERFLOW;
                        act = false;
                    }
                }
                wsync();
                const bool go = blk && act;
                // a_{u,i} of the new positions
                if (go && gl >= mo && gl < mo + nbk) r_ai = NAI[gl - mo];
                wform::extend_w<GS, MMAX, NB, LDV>(go, mo, mwb, nbk, gl, gbytes / 8, zslot, wrows, Wm, NR, LV, r_ai, yi, psi,
                                                   spd, status, act);
                if (blk) {
                    m_o += nbk;
                    nsd += nbk;
                }
                wsync();
            }

            // ---- 5. g, psi and the exit test
            if (wu<GS>(act)) {
                if (!(psi > 0.0) || !isfinite(psi)) {
                    status = ROW_NOT_SPD;
                    act = false;
                } else {
                    const double dinv = wform::rsqrt_nr(psi);
                    gi = dinv;
                    r_g = gl < m_o ? -(yi * dinv) : 0.0;
                    steps = k;
                    if (psi <= eps * psi0) {
                        reason = STOP_EPS;
                        act = false;
                    }
                }
            }
        }

        // ---- outputs: the row with ascending columns (i, the largest, last)
        if (wu<GS>(have && status == ROW_OK)) {
            const int col = gl < m_o ? r_col : (gl == m_o ? i : 0x7fffffff);
            if (gl <= m_o) sel[gl] = col;
            wsync();
            int rank = 0;
            const int mo_u = wu<GS>(m_o);
            for (int t = 0; t <= mo_u; ++t) rank += (sel[t] < col) ? 1 : 0;
            if (gl <= m_o) {
                ell_col[(size_t)i * ldell + rank] = col;
                ell_val[(size_t)i * ldell + rank] = gl < m_o ? r_g : gi;
            }
        } else {
            wsync();
        }
        if (have && gl == 0) {
            m_out[i] = (status == ROW_OK) ? m_o + 1 : 0;
            psi_out[i] = psi;
            steps_out[i] = steps;
            reason_out[i] = reason;
            status_out[i] = status;
            if (status == ROW_OVERFLOW) {
                const int pos = atomicAdd(ovf_count, 1);
                ovf_list[pos] = i;
            }
        }
        wsync();
    }
}

}  // namespace bform
}  // namespace afsai
