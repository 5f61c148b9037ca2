// k_tersoff.h -- covalent part: bond pass and atomic-free force gather.
//
// Bond pass (one lane per bond): for every bond (i -> j), i.e. every
// covalent-list entry inside the cutoff S_ij, the environment sums of the two channels
//     zeta_l,ij = sum_{k != j} fc(r_ik) w_l(cos theta_ijk) exp[(alpha_l (r_ij - r_ik))^3]
// (Methods, Eq. 2, one per channel), the vectorised bond order
//     b_ij = G (sum_l (g_l + zeta_l^n_l)^-p)^(1/(2 sigma p))       (Eqs. 3-5, 7)
// and the bond energy 1/2 fc (fR - b fA).  Per entry it stores b_ij, the
// coefficients P_l = dE/dzeta_l,ij = -1/2 fc fA db/dzeta_l and the bond's
// attraction c_ij = fc b fA (which the charge coupling f_q scales).
//
// Force gather (two work items per bond of m) writes only F_m: every covalent
// term that moves with x_m, read back from the stored coefficients:
//   m as the centre i  : its own bonds (pair term) and their k environments;
//   m as the partner j : bonds (i -> m) of each neighbour i, found through the
//                        reverse-slot index, with i's environment k;
//   m as environment k : bonds (i -> k) of each neighbour i, with m in them.
// No atomics: each F_m is a plain sum in a fixed order (deterministic).
#pragma once
#include "ctbop_dev.h"

namespace ctbop {

template <typename R> struct R3 { R x, y, z; };

template <typename R>
__device__ __forceinline__ R dev_sqrt(R v) { return sqrt(v); }

// Reciprocal and square root of the covalent force terms: with FP32 terms the
// hardware instructions (~1 ulp, as close as the FP32 terms themselves),
// otherwise the correctly rounded operations.
__device__ __forceinline__ float term_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
template <typename R>
__device__ __forceinline__ R term_rcp(R x) { return (R)1 / x; }
__device__ __forceinline__ float term_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
template <typename R>
__device__ __forceinline__ R term_sqrt(R x) { return dev_sqrt(x); }

__device__ __forceinline__ void dev_sincos(float a, float *s, float *c) { sincosf(a, s, c); }
__device__ __forceinline__ void dev_sincos(double a, double *s, double *c) { sincos(a, s, c); }

template <typename R>
__device__ __forceinline__ R cutoff(R r, R Rc, R Sc, R piSR, R &dfc)
{
    if (r <= Rc) { dfc = (R)0; return (R)1; }
    if (r >= Sc) { dfc = (R)0; return (R)0; }
    R sn, cs;
    dev_sincos(piSR * (r - Rc), &sn, &cs);
    dfc = (R)-0.5 * piSR * sn;
    return (R)0.5 + (R)0.5 * cs;
}

// angular function of channel l for centre species t (and d/dcos):
// w = gam (1 + (c^2/d^2) x^2 / (d^2 + x^2)), x = h - cos, one division
template <typename R>
__device__ __forceinline__ R angular(const Params<R> &P, int t, int l, R cs, R &dw)
{
    const R x = P.h[t][l] - cs;
    const R iden = term_rcp(P.d2[t][l] + x * x);
    const R w = P.gam[t][l] * ((R)1 + P.c2d2[t][l] * x * x * iden);
    dw = -P.gam[t][l] * P.c2[t][l] * (R)2 * x * iden * iden;
    return w;
}

template <typename R>
__device__ __forceinline__ R radial(const Params<R> &P, int t, int l, R dl, R &de)
{
    R a = P.alpha[t][l] * dl;
    R e = exp(a * a * a);
    de = (R)3 * P.alpha[t][l] * a * a * e;
    return e;
}

// vectorised bond order and its derivatives in zeta_1, zeta_2
template <typename R>
__device__ __forceinline__ R bond_order(const Params<R> &P, int t, R z1, R z2, R &db1, R &db2)
{
    R zn1 = z1 > (R)0 ? pow(z1, P.nn[t][0]) : (R)0;
    R zn2 = z2 > (R)0 ? pow(z2, P.nn[t][1]) : (R)0;
    R zh1 = P.g[t][0] + zn1, zh2 = P.g[t][1] + zn2;
    R a1, a2, S, b;
    if (P.p_is_2) {
        R i1 = (R)1 / zh1, i2 = (R)1 / zh2;
        a1 = i1 * i1;
        a2 = i2 * i2;
        S = a1 + a2;
        b = P.G[t] * pow(S, P.inv2sig[t] * (R)0.5);
        a1 *= i1;                    // zh^-p-1
        a2 *= i2;
    } else {
        a1 = pow(zh1, -P.p);
        a2 = pow(zh2, -P.p);
        S = a1 + a2;
        b = P.G[t] * pow(S, P.inv2sig[t] / P.p);
        a1 /= zh1;
        a2 /= zh2;
    }
    R k = -b * P.inv2sig[t] / S;
    db1 = z1 > (R)0 ? k * P.nn[t][0] * (zn1 / z1) * a1 : (R)0;
    db2 = z2 > (R)0 ? k * P.nn[t][1] * (zn2 / z2) * a2 : (R)0;
    return b;
}

// Gradients w.r.t. the bond partner (gj) and the environment atom (gk) of the
// zeta_l term of a triplet: centre species tc, bond vector db (length rb),
// environment vector de (length re), environment cutoff pair penv.
template <typename R>
__device__ __forceinline__ void trip_grad(const Params<R> &P, int tc, int penv, const R3<R> &db, R rb,
                                          const R3<R> &de, R re, R3<R> gj[2], R3<R> gk[2])
{
    const R ib = term_rcp(rb), ie = term_rcp(re);
    const R3<R> ub = {db.x * ib, db.y * ib, db.z * ib};
    const R3<R> ue = {de.x * ie, de.y * ie, de.z * ie};
    const R cs = ub.x * ue.x + ub.y * ue.y + ub.z * ue.z;
    const R3<R> cb = {(ue.x - cs * ub.x) * ib, (ue.y - cs * ub.y) * ib, (ue.z - cs * ub.z) * ib};
    const R3<R> ce = {(ub.x - cs * ue.x) * ie, (ub.y - cs * ue.y) * ie, (ub.z - cs * ue.z) * ie};
    R dfe;
    const R fe = cutoff(re, P.Rc[penv], P.Sc[penv], P.piSR[penv], dfe);
#pragma unroll
    for (int l = 0; l < 2; l++) {
        R dw, de_ = (R)0, ex = (R)1;
        const R w = angular(P, tc, l, cs, dw);
        if (!P.alpha_zero[tc]) ex = radial(P, tc, l, rb - re, de_);
        const R a = fe * dw * ex, bcoef = fe * w * de_, c = dfe * w * ex;
        gj[l].x = a * cb.x + bcoef * ub.x;
        gj[l].y = a * cb.y + bcoef * ub.y;
        gj[l].z = a * cb.z + bcoef * ub.z;
        gk[l].x = c * ue.x + a * ce.x - bcoef * ue.x;
        gk[l].y = c * ue.y + a * ce.y - bcoef * ue.y;
        gk[l].z = c * ue.z + a * ce.z - bcoef * ue.z;
    }
}

template <typename R>
__device__ __forceinline__ R3<R> pair_vec(const typename Vec4<R>::type &a, const typename Vec4<R>::type &b,
                                          const typename Vec4<R>::type &D)
{
    R3<R> v = {(b.x - a.x) + D.x, (b.y - a.y) + D.y, (b.z - a.z) + D.z};
    return v;
}

template <typename R>
__device__ __forceinline__ void load_dtab2(const Seg &S, typename Vec4<R>::type *tab)
{
    for (int c = threadIdx.x; c < NCODE; c += blockDim.x) {
        int d0 = c / 49 - 3, d1 = (c / 7) % 7 - 3, d2 = c % 7 - 3;
        typename Vec4<R>::type v;
        v.x = (R)(d0 * S.cw[0][0] + d1 * S.cw[1][0] + d2 * S.cw[2][0]);
        v.y = (R)(d0 * S.cw[0][1] + d1 * S.cw[1][1] + d2 * S.cw[2][1]);
        v.z = (R)(d0 * S.cw[0][2] + d1 * S.cw[1][2] + d2 * S.cw[2][2]);
        v.w = 0;
        tab[c] = v;
    }
    __syncthreads();
}

// The parameters in LDS: the triplet loops index them by species, and
// per-lane indexed reads of the kernel-argument copy go through the vector
// memory path (and are read again in every iteration for want of registers).
template <typename P>
__device__ __forceinline__ void stage_params(const P &src, P &dst)
{
    static_assert(sizeof(P) % 4 == 0, "parameter block of whole words");
    const int *a = reinterpret_cast<const int *>(&src);
    int *b = reinterpret_cast<int *>(&dst);
    for (int k = threadIdx.x; k < (int)(sizeof(P) / 4); k += blockDim.x) b[k] = a[k];
}

// Work items of the covalent kernels: the bonds of a block's rows, numbered
// row after row, so that a lane takes a bond rather than an atom.  With an
// atom per lane the loops over bonds and bond pairs ran one after another in
// a lane (and 64 atoms with different bond counts shared a wave: 30 % of the
// lanes active); a small system's time was that chain.  Rows go in order of
// decreasing bond count (a counting sort; their order among equals, taken
// by atomics, moves no sum), so that a wave's loops over a row's bonds have
// similar lengths.  Items go in chunks of at most CAP, whole rows each.
constexpr int COV_ROWS = 128, COV_FINE = 32;    // rows per block: large and small launches
template <int ROWS> constexpr int cov_cap() { return ROWS == COV_FINE ? 256 : 768; }

template <int ROWS, int CAP>
struct RowItems {
    static constexpr int STEP = CAP - WB + 1;   // items per chunk before a row may start the next one
    int count[WB + 1], first[WB + 1], items[WB + 1];
    int total;
    int start[ROWS];                            // a row's first item
    uint8_t nb[ROWS];
    uint8_t row[CAP];                           // chunk: an item's row
    uint8_t used[CAP];

    // start[] of every row from nb[] (all threads of the block; nb is set,
    // ends with a barrier)
    __device__ __forceinline__ void number()
    {
        const int tid = threadIdx.x;
        if (tid <= WB) count[tid] = 0;
        __syncthreads();
        int place = 0;
        if (tid < ROWS) place = atomicAdd(&count[nb[tid]], 1);
        __syncthreads();
        if (tid <= WB) {
            int r = 0;
            for (int k = tid + 1; k <= WB; k++) r += count[k] * k;
            items[tid] = r;
            if (tid == 0) total = r;
        }
        __syncthreads();
        if (tid < ROWS) start[tid] = items[nb[tid]] + place * nb[tid];
        __syncthreads();
    }
    __device__ __forceinline__ int chunks() const { return (total + STEP - 1) / STEP; }
    // the rows and items of chunk c (ends with a barrier); its items are
    // numbers below len(c), those in use flagged
    __device__ __forceinline__ void open(int c)
    {
        const int tid = threadIdx.x;
        for (int k = tid; k < CAP; k += TILE) used[k] = 0;
        __syncthreads();
        if (tid < ROWS && in_chunk(tid, c)) {
            const int at = start[tid] - c * STEP;
            for (int e = 0; e < nb[tid]; e++) {
                row[at + e] = (uint8_t)tid;
                used[at + e] = 1;
            }
        }
        __syncthreads();
    }
    __device__ __forceinline__ int len(int c) const { return min(CAP, total - c * STEP); }
    __device__ __forceinline__ bool in_chunk(int r, int c) const
    {
        return nb[r] > 0 && start[r] >= c * STEP && start[r] < (c + 1) * STEP;
    }
};

// D(code), the offset of a list entry's cell (what the tables hold)
__device__ __forceinline__ R3<double> code_offset(const Seg &S, int c)
{
    const int d0 = c / 49 - 3, d1 = (c / 7) % 7 - 3, d2 = c % 7 - 3;
    R3<double> v = {d0 * S.cw[0][0] + d1 * S.cw[1][0] + d2 * S.cw[2][0],
                    d0 * S.cw[0][1] + d1 * S.cw[1][1] + d2 * S.cw[2][1],
                    d0 * S.cw[0][2] + d1 * S.cw[1][2] + d2 * S.cw[2][2]};
    return v;
}

// Bond pass.  First the bonds of the step: the covalent-list entries inside
// S_ij, by the FP64 distance used below, compacted in list order (so every
// loop over bonds and triplets runs over bonds only; the skin shell of the
// covalent list, e.g. the twelve second neighbours of Si in SiC, drops out),
// with the slot map that lets the force gather find each bond's reverse.
// The bond pass runs in FP64 from the FP64 local coordinates: it is a small
// share of the step (a few bonds per atom), and FP64 keeps the energy free of
// FP32 rounding in zeta, b and the large, cancelling fR and b fA terms.  The
// coefficients are stored in the pair precision R for the force gather.
//
// Eight lanes take a row's list entries (their places by ballots); then a
// lane takes a bond, its row's bonds in LDS.  Bound by latency and FP64
// transcendentals: 512 atoms 68 -> 13 us, 20,000 atoms 195 -> 37, a chunk of
// 131,072 atoms of the 1M-atom slab beside the solve 273 -> 185.
template <typename R, int ROWS>
__global__ void __launch_bounds__(TILE) k_bond(const Tile *tiles, Seg *segs, Params<double> Pk)
{
    using V4 = typename Vec4<R>::type;
    constexpr int CAP = cov_cap<ROWS>(), LB = 8;
    const Tile T = my_rows<ROWS>(tiles);
    const Seg &S = segs[T.seg];
    __shared__ Params<double> P;
    __shared__ RowItems<ROWS, CAP> it;
    // the chunk's bonds: vector over length, length, cutoff value, pair type
    __shared__ double gx[CAP], gy[CAP], gz[CAP], gr[CAP], gf[CAP];
    __shared__ uint8_t gp[CAP];
    stage_params(Pk, P);
    if (threadIdx.x < ROWS) it.nb[threadIdx.x] = 0;
    __syncthreads();
    const double4 *xs = S.xs64;
    const int Wb = S.Wb, Ws = S.Ws;
    {
        const int lane = threadIdx.x % LB;
        const unsigned below = (1u << lane) - 1u;
        const auto sidx = gbl(S.sidx);
        const auto srev = gbl(S.srev);
        const auto bidx = gblw(S.bidx);
        const auto bsrev = gblw(S.bsrev);
        const auto cmap = gblw(S.cmap);
        for (int k = threadIdx.x / LB; k < ROWS; k += TILE / LB) {
            const int s = T.row0 + k;
            if (s >= S.n) {
                if (s < S.npad && lane == 0) {
                    S.ecov[s] = 0.0;
                    S.bcnt[s] = 0;
                }
                continue;                        // the whole group skips together
            }
            const double4 li = ld4<double>(xs, s);
            const int ti = (int)li.w;
            const int ns = S.scnt[s];
            const size_t rl = (size_t)s * Ws, ob = slice_base(s, Wb), oc = slice_base(s, Ws);
            int nb = 0;
            for (int e0 = 0; e0 < ns; e0 += LB) {
                const int e = e0 + lane;
                bool in = false;
                uint32_t ent = 0;
                if (e < ns) {
                    ent = sidx[rl + e];
                    const double4 lj = ld4<double>(xs, ent & J_MASK);
                    const int pp = ti * 2 + (int)lj.w;
                    const R3<double> D = code_offset(S, (int)(ent >> CODE_SHIFT));
                    const R3<double> d = {(lj.x - li.x) + D.x, (lj.y - li.y) + D.y, (lj.z - li.z) + D.z};
                    in = d.x * d.x + d.y * d.y + d.z * d.z < P.Sc[pp] * P.Sc[pp];
                }
                const unsigned gm = group_ballot<LB>(in);
                const int at = nb + __popc(gm & below);
                const bool kept = in && at < Wb;
                if (kept) {
                    bidx[ob + (size_t)at * SLICE] = ent;
                    bsrev[ob + (size_t)at * SLICE] = srev[rl + e];
                }
                if (e < ns) cmap[oc + (size_t)e * SLICE] = kept ? (uint8_t)at : (uint8_t)255;
                nb += __popc(gm);
            }
            if (lane == 0) {
                if (nb > Wb) atomicOr(&S.sst->status, ST_OVERFLOW);
                nb = min(nb, Wb);
                S.bcnt[s] = nb;
                it.nb[k] = (uint8_t)nb;
            }
        }
    }
    __syncthreads();
    it.number();
    double ecov = 0.0;
    for (int c = 0; c < it.chunks(); c++) {
        it.open(c);
        const int len = it.len(c);
        for (int i = threadIdx.x; i < len; i += TILE) {
            if (!it.used[i]) continue;
            const int lr = it.row[i], s = T.row0 + lr, e = i - (it.start[lr] - c * it.STEP);
            const uint32_t ent = gbl(S.bidx)[sliced(s, e, Wb)];
            const double4 li = ld4<double>(xs, s), lj = ld4<double>(xs, ent & J_MASK);
            const int pp = (int)li.w * 2 + (int)lj.w;
            const R3<double> D = code_offset(S, (int)(ent >> CODE_SHIFT));
            const R3<double> d = {(lj.x - li.x) + D.x, (lj.y - li.y) + D.y, (lj.z - li.z) + D.z};
            const double r = sqrt(d.x * d.x + d.y * d.y + d.z * d.z), ir = 1.0 / r;
            double dummy;
            gx[i] = d.x * ir;
            gy[i] = d.y * ir;
            gz[i] = d.z * ir;
            gr[i] = r;
            gf[i] = cutoff<double>(r, P.Rc[pp], P.Sc[pp], P.piSR[pp], dummy);
            gp[i] = (uint8_t)pp;
        }
        __syncthreads();
        double eb[(CAP + TILE - 1) / TILE];      // the energies of this lane's bonds
#pragma unroll
        for (int u = 0; u < (CAP + TILE - 1) / TILE; u++) {
            const int i = threadIdx.x + u * TILE;
            eb[u] = 0.0;
            if (i >= len || !it.used[i]) continue;
            const int lr = it.row[i], i0 = it.start[lr] - c * it.STEP, nb = it.nb[lr];
            const int pp = gp[i], ti = pp >> 1;
            const double ux = gx[i], uy = gy[i], uz = gz[i], r = gr[i], fc = gf[i];
            double z1 = 0, z2 = 0;
            for (int k = i0; k < i0 + nb; k++) {
                if (k == i) continue;
                const double cs = ux * gx[k] + uy * gy[k] + uz * gz[k], fk = gf[k];
                double dw, dex;
                double w1 = angular<double>(P, ti, 0, cs, dw), w2 = angular<double>(P, ti, 1, cs, dw);
                if (!P.alpha_zero[ti]) {
                    w1 *= radial<double>(P, ti, 0, r - gr[k], dex);
                    w2 *= radial<double>(P, ti, 1, r - gr[k], dex);
                }
                z1 += fk * w1;
                z2 += fk * w2;
            }
            double db1, db2;
            const double b = bond_order<double>(P, ti, z1, z2, db1, db2);
            const double fR = P.A[pp] * exp(-P.lam1[pp] * r), fA = P.B[pp] * exp(-P.lam2[pp] * r);
            eb[u] = 0.5 * fc * (fR - b * fA);
            V4 out;
            out.x = (R)b;
            out.y = (R)(-0.5 * fc * fA * db1);
            out.z = (R)(-0.5 * fc * fA * db2);
            out.w = (R)(fc * b * fA);            // the charge-free attraction (f_q coupling)
            st4<R>(reinterpret_cast<V4 *>(S.slot), sliced(T.row0 + lr, i - i0, Wb), out);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < (CAP + TILE - 1) / TILE; u++) {
            const int i = threadIdx.x + u * TILE;
            if (i < len) gr[i] = eb[u];
        }
        __syncthreads();
        if (threadIdx.x < ROWS && it.in_chunk(threadIdx.x, c)) {
            const int i0 = it.start[threadIdx.x] - c * it.STEP;
            for (int e = 0; e < it.nb[threadIdx.x]; e++) ecov += gr[i0 + e];
        }
        __syncthreads();
    }
    if (threadIdx.x < ROWS && T.row0 + (int)threadIdx.x < S.n) S.ecov[T.row0 + threadIdx.x] = ecov;
}

// Bond index, in the partner i's row, of the reverse of bond (m, e)
__device__ __forceinline__ int reverse_bond(const Seg &S, int m, int e, int i)
{
    return S.cmap[sliced(i, S.bsrev[sliced(m, e, S.Wb)], S.Ws)];
}

// pair-term derivative dV/dr of 1/2 fc (fR - b fA) at fixed b
template <typename R>
__device__ __forceinline__ R pair_dvdr(const Params<R> &P, int pp, R r, R b)
{
    R dfc;
    const R fc = cutoff(r, P.Rc[pp], P.Sc[pp], P.piSR[pp], dfc);
    const R fR = P.A[pp] * exp(-P.lam1[pp] * r), fA = P.B[pp] * exp(-P.lam2[pp] * r);
    return (R)0.5 * (dfc * (fR - b * fA) + fc * (-P.lam1[pp] * fR + b * P.lam2[pp] * fA));
}

// Two work items per bond (m, e): the bond with m as its centre (the pair
// term and m's environment), and, of the same pair, the bond of the
// neighbour i in which m is the partner, with i's other bonds, in which m
// is the environment.  An item's FP32 terms are added in the order of the
// bonds; an atom's items in FP64, bond by bond.  512 atoms 107 -> 20 us,
// 20,000 atoms 519 -> 47, a chunk of 131,072 atoms of the 1M-atom slab beside
// the solve 293 -> 241.
template <typename R, int ROWS>
__global__ void __launch_bounds__(TILE) k_force_cov(const Tile *tiles, Seg *segs, Params<R> Pk)
{
    using V4 = typename Vec4<R>::type;
    constexpr int CAP = cov_cap<ROWS>() / (sizeof(R) / 4);
    const Tile T = my_rows<ROWS>(tiles);
    const Seg &S = segs[T.seg];
    // serving: only segments whose charge solve finished and whose forces are pending
    __shared__ V4 dtab[NCODE];
    __shared__ Params<R> P;
    __shared__ RowItems<ROWS, CAP> it;
    // the chunk's bonds: vector, length, list entry, pair type; forces of the items
    __shared__ R gx[CAP], gy[CAP], gz[CAP], gr[CAP];
    __shared__ uint32_t ge[CAP];
    __shared__ uint8_t gp[CAP];
    __shared__ R fo[2][3][CAP];
    const auto bcnt = gbl(S.bcnt);
    if (threadIdx.x < ROWS) {
        const int m = T.row0 + threadIdx.x;
        it.nb[threadIdx.x] = (uint8_t)(m < S.n ? bcnt[m] : 0);
    }
    stage_params(Pk, P);
    load_dtab2<R>(S, dtab);                 // (ends with a barrier)
    it.number();
    const V4 *xs = reinterpret_cast<const V4 *>(S.xs);
    const V4 *slot = reinterpret_cast<const V4 *>(S.slot);
    const int Wb = S.Wb, Ws = S.Ws;
    const auto bidx = gbl(S.bidx);
    const auto bsrev = gbl(S.bsrev);
    const auto cmap = gbl(S.cmap);
    double fx = 0, fy = 0, fz = 0;
    for (int c = 0; c < it.chunks(); c++) {
        it.open(c);
        const int len = it.len(c), len64 = (len + 63) & ~63;
        for (int i = threadIdx.x; i < len; i += TILE) {
            if (!it.used[i]) continue;
            const int lr = it.row[i], m = T.row0 + lr, e = i - (it.start[lr] - c * it.STEP);
            const uint32_t ent = bidx[sliced(m, e, Wb)];
            const V4 lm = ld4<R>(xs, m), lj = ld4<R>(xs, ent & J_MASK);
            const R3<R> d = pair_vec<R>(lm, lj, dtab[ent >> CODE_SHIFT]);
            gx[i] = d.x;
            gy[i] = d.y;
            gz[i] = d.z;
            gr[i] = term_sqrt(d.x * d.x + d.y * d.y + d.z * d.z);
            ge[i] = ent;
            gp[i] = (uint8_t)((int)lm.w * 2 + (int)lj.w);
        }
        __syncthreads();
        // (whole waves of either kind)
        for (int w = threadIdx.x; w < 2 * len64; w += TILE) {
            const bool partner = w < len64;
            const int i = partner ? w : w - len64;
            if (i >= len || !it.used[i]) continue;
            const int lr = it.row[i], i0 = it.start[lr] - c * it.STEP, e = i - i0, nb = it.nb[lr];
            const int m = T.row0 + lr;
            const R r = gr[i];
            R ax = (R)0, ay = (R)0, az = (R)0;
            if (!partner) {
                // m as the centre of its own bond
                const R3<R> d = {gx[i], gy[i], gz[i]};
                const int pp = gp[i], tm = pp >> 1;
                const R ir = term_rcp(r);
                const V4 sv = ld4<R>(slot, sliced(m, e, Wb));
                const R dv = pair_dvdr(P, pp, r, sv.x) * ir;
                ax = dv * d.x;
                ay = dv * d.y;
                az = dv * d.z;
                if (sv.y != (R)0 || sv.z != (R)0) {
                    for (int k = i0; k < i0 + nb; k++) {
                        if (k == i) continue;
                        const R3<R> dk = {gx[k], gy[k], gz[k]};
                        R3<R> gj[2], gk[2];
                        trip_grad(P, tm, (int)gp[k], d, r, dk, gr[k], gj, gk);
                        ax += sv.y * (gj[0].x + gk[0].x) + sv.z * (gj[1].x + gk[1].x);
                        ay += sv.y * (gj[0].y + gk[0].y) + sv.z * (gj[1].y + gk[1].y);
                        az += sv.z * (gj[1].z + gk[1].z) + sv.y * (gj[0].z + gk[0].z);
                    }
                }
            } else {
                // m as the partner j or the environment k of its neighbour's bonds
                const uint32_t ent = ge[i];
                const int nbr = (int)(ent & J_MASK), tm = gp[i] >> 1, ti = gp[i] & 1, pp = ti * 2 + tm;
                const int ni = bcnt[nbr];
                // bond (i -> m) in row i (a reverse always exists)
                const int rv = cmap[slice_base(nbr, Ws) + (size_t)bsrev[sliced(m, e, Wb)] * SLICE];
                if (rv < ni) {
                    const V4 li = ld4<R>(xs, nbr);
                    const R ir = term_rcp(r);
                    const R3<R> d = {-gx[i], -gy[i], -gz[i]};            // i -> m
                    const size_t sli = slice_base(nbr, Wb);
                    const V4 sv = ld4<R>(slot, sli + (size_t)rv * SLICE);
                    const R dv = pair_dvdr(P, pp, r, sv.x) * ir;
                    ax = -dv * d.x;
                    ay = -dv * d.y;
                    az = -dv * d.z;
                    const auto rowi = bidx + sli;
                    for (int t = 0; t < ni; t++) {
                        if (t == rv) continue;
                        const uint32_t ent2 = rowi[(size_t)t * SLICE];
                        const V4 sk = ld4<R>(slot, sli + (size_t)t * SLICE);   // bond (i -> k)
                        const V4 lk = ld4<R>(xs, ent2 & J_MASK);
                        const int pk = ti * 2 + (int)lk.w;
                        const R3<R> dk = pair_vec<R>(li, lk, dtab[ent2 >> CODE_SHIFT]);   // i -> k
                        const R rk = term_sqrt(dk.x * dk.x + dk.y * dk.y + dk.z * dk.z);
                        R3<R> gj[2], gk[2];
                        if (sv.y != (R)0 || sv.z != (R)0) {
                            // bond (i -> m), environment k: m is the partner j
                            trip_grad(P, ti, pk, d, r, dk, rk, gj, gk);
                            ax -= sv.y * gj[0].x + sv.z * gj[1].x;
                            ay -= sv.y * gj[0].y + sv.z * gj[1].y;
                            az -= sv.y * gj[0].z + sv.z * gj[1].z;
                        }
                        if (sk.y != (R)0 || sk.z != (R)0) {
                            // bond (i -> k), environment m: m is the environment atom
                            trip_grad(P, ti, pp, dk, rk, d, r, gj, gk);
                            ax -= sk.y * gk[0].x + sk.z * gk[1].x;
                            ay -= sk.y * gk[0].y + sk.z * gk[1].y;
                            az -= sk.y * gk[0].z + sk.z * gk[1].z;
                        }
                    }
                }
            }
            fo[partner][0][i] = ax;
            fo[partner][1][i] = ay;
            fo[partner][2][i] = az;
        }
        __syncthreads();
        if (threadIdx.x < ROWS && it.in_chunk(threadIdx.x, c)) {
            const int i0 = it.start[threadIdx.x] - c * it.STEP, i1 = i0 + it.nb[threadIdx.x];
#pragma unroll
            for (int h = 0; h < 2; h++)
                for (int i = i0; i < i1; i++) {
                    fx += (double)fo[h][0][i];
                    fy += (double)fo[h][1][i];
                    fz += (double)fo[h][2][i];
                }
        }
        __syncthreads();
    }
    const int m = T.row0 + (int)threadIdx.x;
    if (threadIdx.x < ROWS && m < S.n) {
        S.Fcov[m] = fx;
        S.Fcov[S.npad + m] = fy;
        S.Fcov[2 * S.npad + m] = fz;
    }
}

} // namespace ctbop
