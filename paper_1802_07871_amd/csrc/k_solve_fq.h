// k_solve_fq.h -- the nonlinear charge solve of the charge coupling (k_fq.h) in
// one launch, for the systems that take the one-launch linear solve.
//
// The multi-launch form takes nine dependent launches per iteration (18,086
// atoms: 73 us; five MD steps 11.4 ms, 4.25 with this solve, which takes 0.44
// ms).  Here, as in k_solve.h, a block keeps its rows' matrix
// entries in registers and exchanges through agent-scope slots that are their
// own flags.  An iteration exchanges p once: the block keeps the charges of
// its halo in LDS and advances them with the same step as their owners
// (q += alpha p, bit for bit), so the line search and the coupling's gradient,
// whose bonds reach rows of the halo only, need no other exchange.  Three sums
// over the system remain: the two Newton steps on the step length and the
// residual's.  Bound, like k_solve, by its exchanges: four round trips past
// the L2s per iteration, each with the wait for the slowest block.
#pragma once
#include "k_fq.h"
#include "k_solve.h"

namespace ctbop {

constexpr int SVF_NW = SV_T / 64;
constexpr int SVF_REG_BONDS = 2;            // bonds a lane keeps in registers

// Each bond's position in the block's halo, 16 bits, row-major (Wb per row):
// in the second half of the block's rows of S.hsidx, whose first half is more
// than the halo list takes and whose last word is the list's length (room for
// both where Wl > Wb, which the host asks for).
__device__ __forceinline__ uint16_t *svf_bonds(const Seg &S, int row0, int rb)
{
    return reinterpret_cast<uint16_t *>(S.hsidx + (size_t)row0 * S.Wl) + (size_t)rb * S.Wl;
}

// Sums 0 .. K-1 of the products of two row arrays, a wave each, as in
// k_solve: the block's into tot, every block's into red.  Round `ex` of the
// exchange.  false: a wait ran out.
template <int K, int RB>
__device__ __forceinline__ bool svf_sum(const double (*va)[RB], unsigned long long fa, unsigned long long fb, int wv,
                                        int wl, int nblk, int blk, int ex,
                                        __attribute__((address_space(1))) unsigned long long *slots_p, double *tot,
                                        double (*red)[SV_LINE], const int *pabort)
{
    static_assert(K <= SVF_NW, "a sum per wave");
    if (wv < K) {
        const double *a = va[(fa >> (4 * wv)) & 15], *b = va[(fb >> (4 * wv)) & 15];
        double v = 0.0;
#pragma unroll
        for (int k = 0; k < RB; k += 64) v += a[k + wl] * b[k + wl];
        v = wave_sum(v);
        if (wl == 0) tot[wv] = v;
    }
    if (nblk == 1) return true;
    __syncthreads();
    if (wv == 0) sv_put(sv_line(slots_p, ex % 3, nblk, blk, wl), tot[wl & 15]);
    return sv_collect<SVF_NW>(slots_p, ex % 3, nblk, blk, red, wv, wl, pabort);
}

// empty this block's sums of the round before (every block has read them)
__device__ __forceinline__ void svf_clear(int wv, int wl, int nblk, int blk, int ex,
                                          __attribute__((address_space(1))) unsigned long long *slots_p)
{
    if (nblk > 1 && wv == 1) sv_clear(sv_line(slots_p, (ex + 2) % 3, nblk, blk, wl));
}

template <int LPR, typename R>
__global__ void __launch_bounds__(SV_T, 2) k_solve_fq(const Tile *tiles, Seg *segs, SolveCtl ctl)
{
    constexpr int RB = sv_rows(LPR), EPT = BK / LPR, E = sv_regs<R, LPR, 2>(), NB = SVF_REG_BONDS;
    int seg;
    const int row0 = sv_row0<RB>(tiles, segs, seg);
    if (row0 < 0) return;
    const Seg &S = segs[seg];
    if (uni(S.sst->pabort)) return;
    __shared__ double hp[SV_HALO], hq[SV_HALO];
    __shared__ uint16_t hl[SV_HALO];
    // the rows' arrays: r, y, H p, q, m1, r of the iteration before, p, the
    // quadratic residual, ones, the line search's A and B, J
    enum { R_ = 0, Y_, S_, Q_, M_, RO_, P_, RL_, ONE_, A_, B_, J_, NV_ };
    __shared__ double va[NV_][RB];
    __shared__ double tot[SV_LINE], red[SVF_NW][SV_LINE];
    __shared__ SegState st;
    __shared__ int sab, nslot;
    const int tid = threadIdx.x, rl = tid / LPR, lane = tid % LPR, row = row0 + rl, wv = uni(tid >> 6), wl = tid & 63;
    const int n = uni(S.n), Wl = uni(S.Wl), Wb = uni(S.Wb), blk = row0 / RB, nblk = (n + RB - 1) / RB;
    const bool live = row < n;
    const double Q = S.Q, kq = S.fqk;
    SegState *const sst = uni(S.sst);
    int *const pabort = &sst->pabort;
    const auto slots_y0 = sv_slots(uni(S.y)), slots_y1 = sv_slots(uni(S.hz)), slots_p = sv_slots(uni((double *)S.H));
    const uint32_t *region = S.hsidx + (size_t)row0 * Wl;
    const int nh = uni((int)region[(size_t)RB * Wl - 1]);
    {
        const auto list = gbl(reinterpret_cast<const uint16_t *>(region));
        const auto qg = gbl(S.q);
        for (int k = tid; k < nh; k += SV_T) {
            const uint16_t j = list[k];
            hl[k] = j;
            hq[k] = qg[j];
        }
    }
    const int cnt = live ? gbl(S.hcnt)[row] : 0;
    const auto vals = gbl(uni(reinterpret_cast<const R *>(S.Hr)) + (size_t)row0 * Wl);
    const auto poss = gbl(uni(S.hs16) + (size_t)row0 * Wl);
    const unsigned rowe = (unsigned)(rl * Wl);
    R hv[E];
    uint32_t hj[E / 2];
#pragma unroll
    for (int k0 = 0; k0 < E; k0 += 8) {
        uint32_t a[8];
#pragma unroll
        for (int u = 0; u < 8; u++) {
            const int e = (k0 + u) * LPR + lane;
            hv[k0 + u] = vals[rowe + (unsigned)(e < cnt ? e : 0)];
            a[u] = poss[rowe + (unsigned)(e < cnt ? e : 0)];
        }
#pragma unroll
        for (int u = 0; u < 8; u++) {
            const bool in = (k0 + u) * LPR + lane < cnt;
            hv[k0 + u] = in ? hv[k0 + u] : (R)0;
            a[u] = in ? a[u] : 0u;
            if (u & 1) hj[(k0 + u) / 2] = a[u - 1] | (a[u] << 16);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    int mxc = cnt;
#pragma unroll
    for (int o = 32; o >= LPR; o >>= 1) mxc = max(mxc, __shfl_xor(mxc, o, 64));
    const int nch = uni((mxc + 8 * LPR - 1) / (8 * LPR));
    float bv[EPT];
#pragma unroll
    for (int u = 0; u < EPT; u++) bv[u] = (float)gbl(S.binv + (size_t)row * BK)[lane * EPT + u];
    // the row's bonds: lane l takes bonds l, l + LPR, ..., the first NB in registers
    const int nb = live ? gbl(S.bcnt)[row] : 0;
    const auto wqs = gbl(S.wq + slice_base(row, Wb));
    const auto bps = gbl(svf_bonds(S, row0, RB) + (size_t)rl * Wb);
    double bw[NB];
    int bp[NB];
#pragma unroll
    for (int u = 0; u < NB; u++) {
        const int e = lane + u * LPR;
        bw[u] = e < nb ? wqs[(size_t)e * SLICE] : 0.0;
        bp[u] = e < nb ? (int)bps[e] : 0;
    }
    // f over the row's bonds: (weight, halo position of the partner)
    auto bonds = [&](auto f) {
#pragma unroll
        for (int u = 0; u < NB; u++)
            if (lane + u * LPR < nb) f(bw[u], bp[u]);
        for (int e = lane + NB * LPR; e < nb; e += LPR) f(wqs[(size_t)e * SLICE], (int)bps[e]);
    };
    static_assert(sizeof(SegState) % 4 == 0 && sizeof(SegState) / 4 <= SV_T, "a word per thread");
    if (tid < (int)(sizeof(SegState) / 4)) reinterpret_cast<int *>(&st)[tid] = reinterpret_cast<const int *>(sst)[tid];
    if (tid == 0) {
        sab = ctl.way & 1;
        nslot = 0;
    }
    if (tid < SV_LINE) tot[tid] = 0.0;
    if (lane == 0) {
        va[Q_][rl] = live ? S.q[row] : 0.0;
        va[RL_][rl] = live ? S.r[row] : 0.0;
        va[M_][rl] = live ? S.m1[row] : 0.0;
        va[J_][rl] = live ? S.jd[row] : 0.0;
        va[ONE_][rl] = 1.0;
        va[Y_][rl] = va[S_][rl] = va[RO_][rl] = va[P_][rl] = va[R_][rl] = va[A_][rl] = va[B_][rl] = 0.0;
    }
    __syncthreads();
    int ex = 0;
    // r = the quadratic residual less the coupling's gradient at the charges
    // of the halo; y = M r
    auto residual = [&]() {
        double g = 0.0;
        const double qm = va[Q_][rl];
        bonds([&](double w, int j) { g -= w * fq_d1(kq, qm - hq[j]); });
        g = row_sum<LPR>(g);
        if (lane == 0) va[R_][rl] = live ? va[RL_][rl] - g : 0.0;
    };
    auto precond = [&]() {
        double y = 0.0;
#pragma unroll
        for (int u = 0; u < EPT; u++) y += (double)bv[u] * va[R_][(rl & ~(BK - 1)) + lane * EPT + u];
        y = row_sum<LPR>(y);
        if (lane == 0) va[Y_][rl] = y;
    };
    // first pass over the starting residual: its shift (r m1, m1, entries)
    residual();
    if (lane == 0) va[A_][rl] = (double)cnt;
    sv_slot_count<E, LPR>(nch, cnt, lane, wl, &nslot, tot);
    __syncthreads();
    bool ok = svf_sum<3, RB>(va, 0x940ull, 0x884ull, wv, wl, nblk, blk, ex, slots_p, tot, red, pabort);
    if (!ok) sab = 1;
    __syncthreads();
    if (!sab) {
        if (wv == 0) {
            const double mine = sv_total<SVF_NW>(tot, red, nblk, wl);
            double t[3];
            for (int k = 0; k < 3; k++) t[k] = sv_lane(mine, k);
            const double slots = sv_lane(mine, SV_SLOTS);
            if (wl == 0) {
                st.sdinv = t[1];
                st.w = t[0] / t[1];
                st.nnz_coul = t[2];
                st.nnz_wide = 0.0;
                st.nnz_halo = t[2];
                st.nnz_slots = slots;
                st.mshift = st.mu_prev - st.w;
                st.iters = 0;
                st.qshift = 0.0;
            }
        }
        svf_clear(wv, wl, nblk, blk, ex, slots_p);
        ex++;
        __syncthreads();
        if (lane == 0 && live) {
            va[R_][rl] -= st.w;
            va[RL_][rl] -= st.w;
        }
        // second pass: the shift left, r^T z and the norm (r m1, r y, r, r r)
        __syncthreads();
        precond();
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        ok = svf_sum<4, RB>(va, 0x0000ull, 0x0814ull, wv, wl, nblk, blk, ex, slots_p, tot, red, pabort);
        if (!ok) sab = 1;
        __syncthreads();
    }
    if (!sab) {
        if (wv == 0) {
            const double mine = sv_total<SVF_NW>(tot, red, nblk, wl);
            double t[4];
            for (int k = 0; k < 4; k++) t[k] = sv_lane(mine, k);
            if (wl == 0) {
                const double w = t[0] / st.sdinv, res2 = (t[3] - t[2] * t[2] / n) / n;
                st.w = w;
                st.rho = t[1] - w * t[0];
                st.beta = 0.0;
                st.res = sqrt(fmax(res2, 0.0));
                st.res0 = st.res;
                st.mshift -= w;
                st.done = st.res < ctl.tol ? 1 : 0;
            }
        }
        svf_clear(wv, wl, nblk, blk, ex, slots_p);
        ex++;
        __syncthreads();
    }
    const bool run = !sab;
    for (int it = 0; run && !st.done; it++) {
#pragma unroll
        for (int k = 0; k < E; k++) asm volatile("" : "+v"(hv[k]));
#pragma unroll
        for (int k = 0; k < E / 2; k++) asm volatile("" : "+v"(hj[k]));
        // the direction: r -= w, p = (y - w m1) + beta p
        const auto ps = (it & 1) ? slots_y1 : slots_y0;
        if (lane == 0) {
            double p = 0.0;
            if (live) {
                const double w = st.w;
                va[R_][rl] -= w;
                va[RL_][rl] -= w;
                p = (va[Y_][rl] - w * va[M_][rl]) + st.beta * va[P_][rl];
            }
            va[P_][rl] = p;
            sv_put(ps + row, p);
        }
        // (every thread has read the loop's condition)
        __syncthreads();
        ok = true;
        for (int k0 = tid; k0 < nh + tid && ok; k0 += 4 * SV_T) {
            int k[4];
            unsigned long long v[4];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                k[u] = min(k0 + u * SV_T, nh - 1);
                v[u] = sv_get(ps + (unsigned)hl[k[u]]);
            }
#pragma unroll
            for (int u = 0; u < 4; u++) {
                ok = ok && sv_wait(ps + (unsigned)hl[k[u]], v[u], pabort);
                hp[k[u]] = __longlong_as_double((long long)v[u]);
            }
        }
        if (!ok) sab = 1;
        __syncthreads();
        if (sab) break;
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = 0; k < E; k += 8)
            if (k < 8 * nch) {
#pragma unroll
                for (int u = 0; u < 8; u++) acc[u & 3] += (double)hv[k + u] * hp[half16(hj[(k + u) / 2], u)];
                __builtin_amdgcn_sched_barrier(0);
            }
        for (int e0 = E * LPR + lane; e0 < cnt; e0 += 4 * LPR) {
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int e = e0 + u * LPR;
                if (e < cnt) acc[u] += (double)vals[rowe + (unsigned)e] * hp[poss[rowe + (unsigned)e]];
            }
        }
        const double hs = row_sum<LPR>((acc[0] + acc[1]) + (acc[2] + acc[3]));
        // the line search's sums A(alpha), B(alpha) of the row
        const double qm = va[Q_][rl], pm = va[P_][rl];
        auto line = [&](double al) {
            double A = 0.0, B = 0.0;
            bonds([&](double w, int j) {
                const double d = pm - hp[j], t = (qm - hq[j]) + al * d;
                A -= 0.5 * w * d * fq_d1(kq, t);
                B -= 0.5 * w * d * d * fq_d2(kq, t);
            });
            A = row_sum<LPR>(A);
            B = row_sum<LPR>(B);
            if (lane == 0) {
                va[A_][rl] = A;
                va[B_][rl] = B;
            }
        };
        line(0.0);
        if (lane == 0) va[S_][rl] = va[J_][rl] * pm + hs;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        // p H p, p r, A, B
        ok = svf_sum<4, RB>(va, 0xa966ull, 0x8802ull, wv, wl, nblk, blk, ex, slots_p, tot, red, pabort);
        if (!ok) sab = 1;
        __syncthreads();
        if (sab) break;
        if (wv == 0) {
            const double mine = sv_total<SVF_NW>(tot, red, nblk, wl);
            double t[4];
            for (int k = 0; k < 4; k++) t[k] = sv_lane(mine, k);
            if (wl == 0) {
                st.ps = t[0];
                st.pr = t[1];
                st.A0 = t[2];
                st.alpha = 0.0;
                const double d2 = t[0] + t[3];
                if (!(d2 > 0.0) || !(st.ps > 0.0)) {
                    st.status |= ST_NOT_PD;
                    st.done = 1;
                } else {
                    st.alpha = t[1] / d2;
                }
            }
        }
        // (every block has staged p)
        if (lane == 0) sv_clear(ps + row);
        svf_clear(wv, wl, nblk, blk, ex, slots_p);
        ex++;
        __syncthreads();
        if (st.done) break;
        line(st.alpha);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        ok = svf_sum<2, RB>(va, 0xa9ull, 0x88ull, wv, wl, nblk, blk, ex, slots_p, tot, red, pabort);
        if (!ok) sab = 1;
        __syncthreads();
        if (sab) break;
        if (wv == 0) {
            const double mine = sv_total<SVF_NW>(tot, red, nblk, wl);
            double t[2];
            for (int k = 0; k < 2; k++) t[k] = sv_lane(mine, k);
            if (wl == 0) {
                const double d1 = -st.pr + st.alpha * st.ps + (t[0] - st.A0), d2 = st.ps + t[1];
                if (!(d2 > 0.0)) {
                    st.status |= ST_NOT_PD;
                    st.done = 1;
                    st.alpha = 0.0;
                } else {
                    st.alpha -= d1 / d2;
                }
            }
        }
        svf_clear(wv, wl, nblk, blk, ex, slots_p);
        ex++;
        __syncthreads();
        if (st.done) break;
        // the step: q, the halo's q, the quadratic residual
        const double al = st.alpha;
        for (int k = tid; k < nh; k += SV_T) hq[k] += al * hp[k];
        if (lane == 0) {
            va[Q_][rl] += al * va[P_][rl];
            va[RL_][rl] -= al * va[S_][rl];
            va[RO_][rl] = va[R_][rl];
        }
        __syncthreads();
        residual();
        __syncthreads();
        precond();
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        // r m1, r y, r, r r, q, y r_old, m1 r_old
        ok = svf_sum<7, RB>(va, 0x4130000ull, 0x5580814ull, wv, wl, nblk, blk, ex, slots_p, tot, red, pabort);
        if (!ok) sab = 1;
        __syncthreads();
        if (sab) break;
        if (wv == 0) {
            const double mine = sv_total<SVF_NW>(tot, red, nblk, wl);
            double t[7];
            for (int k = 0; k < 7; k++) t[k] = sv_lane(mine, k);
            if (wl == 0) {
                const double w = t[0] / st.sdinv;
                const double rho = t[1] - w * t[0], cross = t[5] - w * t[6];
                const double res2 = (t[3] - t[2] * t[2] / n) / n;
                const double beta = (rho - cross) / st.rho;
                st.beta = beta > 0.0 ? beta : 0.0;
                st.rho = rho;
                st.w = w;
                st.mshift -= w;
                st.res = sqrt(fmax(res2, 0.0));
                st.iters += 1;
                st.iters_total += 1;
                st.qshift = (Q - t[4]) / n;
                if (st.res < ctl.tol) {
                    st.done = 1;
                } else if (st.iters >= ctl.maxit) {
                    st.done = 1;
                    st.status |= ST_NOCONV;
                }
            }
        }
        svf_clear(wv, wl, nblk, blk, ex, slots_p);
        ex++;
        __syncthreads();
    }
    if (sab || ((ctl.way & 2) && blk == nblk - 1)) {
        if (tid == 0) __hip_atomic_store(pabort, PA_WAIT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    if (lane == 0 && live) S.q[row] = va[Q_][rl];
    if (blk == 0 && tid == 0) {
        SegState *o = sst;
        o->sdinv = st.sdinv;
        o->w = st.w;
        o->nnz_coul = st.nnz_coul;
        o->nnz_wide = st.nnz_wide;
        o->nnz_halo = st.nnz_halo;
        o->nnz_slots = st.nnz_slots;
        o->mshift = st.mshift;
        o->iters = st.iters;
        o->iters_total = st.iters_total;
        o->qshift = st.qshift;
        o->rho = st.rho;
        o->alpha = st.alpha;
        o->beta = st.beta;
        o->res = st.res;
        o->res0 = st.res0;
        const int bad = st.status & (ST_NOCONV | ST_NOT_PD);
        if (bad) atomicOr(&o->status, bad);
        o->done = 1;
    }
}

// After the preparation: each bond's position in the block's halo, found in
// the halo list by bisection.  A partner that the list does not hold (bonds
// reaching past the Coulomb cutoff) sends the system to the multi-launch solve.
template <int LPR>
__global__ void __launch_bounds__(TILE) k_solve_fq_bonds(const Tile *tiles, Seg *segs)
{
    constexpr int RB = sv_rows(LPR);
    const Tile T = my_tile(tiles);
    const Seg &S = segs[T.seg];
    const int s = T.row0 + threadIdx.x;
    if (s >= S.n || S.sst->pabort) return;
    const int row0 = s / RB * RB, nb = S.bcnt[s];
    const uint32_t *region = S.hsidx + (size_t)row0 * S.Wl;
    const int nh = (int)region[(size_t)RB * S.Wl - 1];
    const auto list = gbl(reinterpret_cast<const uint16_t *>(region));
    const auto bidx = gbl(S.bidx);
    const auto out = gblw(svf_bonds(S, row0, RB) + (size_t)(s - row0) * S.Wb);
    for (int e = 0; e < nb; e++) {
        const int j = (int)(bidx[sliced(s, e, S.Wb)] & J_MASK);
        int lo = 0, hi = nh - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if ((int)list[mid] < j) lo = mid + 1;
            else hi = mid;
        }
        if (nh == 0 || (int)list[lo] != j) {
            atomicOr(&S.sst->pabort, PA_BOND);
            return;
        }
        out[e] = (uint16_t)lo;
    }
}

} // namespace ctbop
