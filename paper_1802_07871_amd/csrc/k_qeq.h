// k_qeq.h -- charge equilibration and the Coulomb terms.
//
// The charges minimise the energy at every call (Methods).  With the
// self energy chi q + J q^2/2 and the Coulomb kernel C_ij, the energy is
// quadratic in q, so the minimiser solves  H q + chi = mu 1,  sum q = Q,
// H = diag(J) + [C_ij summed over images].  It is found by projected
// block-Jacobi-preconditioned conjugate gradients:
//   z = M (r - w 1),  w = (1^T M r) / (1^T M 1),
// which keeps every direction on sum z = 0; M is the inverse of the diagonal
// blocks of H over BK consecutive sorted rows (atoms of one or two cells,
// which carry the strongest couplings).  The residual r is stored shifted
// by the running w (r = -(Hq + chi) + const), so it never carries the large
// multiplier mu, whose rounding would otherwise swamp r^T z.  Vectors,
// dot products and the projection are FP64; the matrix entries are stored in
// the pair precision (FP32 in the mixed build).
//
// Assembly and the force gather give each row LPR consecutive lanes, which
// read consecutive entries (neighbours in one cell, so their coordinates are
// gathered together) and combine by a fixed butterfly.  The charge-solve
// product runs one row per lane over a sliced copy of the rows, made once per
// step, where entry e of 64 consecutive rows is one contiguous segment.
#pragma once
#include "ctbop_dev.h"
#include "k_tersoff.h"

namespace ctbop {

// Shielded, tapered Coulomb kernel C(r) = ke T(r/rc) (r^3 + g3)^(-1/3) and
// (dC/dr)/r, evaluated in FP64 for a given distance: an FP32 seed of the
// reciprocal cube root and one Newton step, y <- y (4 - u y^3) / 3, leave a
// relative error of ~1e-13, so the only error left in the matrix entries is
// the (unbiased) rounding of r itself and of the stored FP32 value.
// The radial derivative comes divided by r, without a division: with
// T'(x) = -140 x^3 (1-x)^3 and x = r/rc,
//   (dC/dr)/r = ke [ -140 x^2 (1-x)^3 y / rc^2 - T r y^4 ].
__device__ __forceinline__ double rcbrt64(double u)
{
    // u^(-1/3) for u = r^3 + g3 > 0 (pairs are never closer than 0.5 A): the
    // hardware FP32 log2/exp2 seed (~1e-7) and one FP64 Newton step
    const double y = (double)__builtin_amdgcn_exp2f(-0.333333343f * __builtin_amdgcn_logf((float)u));
    return y * (4.0 - u * y * y * y) * (1.0 / 3.0);
}

// g3 = gamma_ij^-3 of the pair
__device__ __forceinline__ double coul64_g(const Params<double> &P, double g3, double r, double &dCr)
{
    const double x = r * P.inv_rc, x2 = x * x, x3 = x2 * x;
    const double om = 1.0 - x, om2 = om * om;
    const double T = om2 * om2 * (1.0 + 4.0 * x + 10.0 * x2 + 20.0 * x3);
    const double u = r * r * r + g3;
    const double y = rcbrt64(u);
    const double y2 = y * y;
    dCr = P.ke * (-140.0 * P.inv_rc * P.inv_rc * x2 * om2 * om * y - T * r * y2 * y2);
    return P.ke * T * y;
}

__device__ __forceinline__ double coul64(const Params<double> &P, int pp, double r, double &dCr)
{
    return coul64_g(P, P.g3[pp], r, dCr);
}

// The same in FP32 (the mixed build's force gather): the hardware log2/exp2
// seed and one FP32 Newton step leave ~1 ulp in y; the pair's energy and
// force terms are then summed in FP64.  Per pair ~1e-7 relative, against the
// 1e-6 eV/atom and 1e-5 relative-force budget.
__device__ __forceinline__ float coul32_g(float ke, float inv_rc, float g3, float r, float &dCr)
{
    const float x = r * inv_rc, x2 = x * x, x3 = x2 * x;
    const float om = 1.0f - x, om2 = om * om;
    const float T = om2 * om2 * (1.0f + 4.0f * x + 10.0f * x2 + 20.0f * x3);
    const float u = r * r * r + g3;
    float y = __builtin_amdgcn_exp2f(-0.333333343f * __builtin_amdgcn_logf(u));
    y = y * (4.0f - u * y * y * y) * 0.333333343f;
    const float y2 = y * y;
    dCr = ke * (-140.0f * inv_rc * inv_rc * x2 * om2 * om * y - T * r * y2 * y2);
    return ke * T * y;
}

__device__ __forceinline__ double coul64_val_g(const Params<double> &P, double g3, double r)
{
    const double x = r * P.inv_rc, x2 = x * x, x3 = x2 * x;
    const double om = 1.0 - x, om2 = om * om;
    const double T = om2 * om2 * (1.0 + 4.0 * x + 10.0 * x2 + 20.0 * x3);
    const double u = r * r * r + g3;
    const double y = rcbrt64(u);
    return P.ke * T * y;
}

__device__ __forceinline__ double coul64_val(const Params<double> &P, int pp, double r)
{
    return coul64_val_g(P, P.g3[pp], r);
}

struct CgCtl {
    double tol;
    int maxit;
};

// Distance of a list entry, in the pair precision R and then widened: every
// kernel that tests it against rc computes it this one way, so all of them
// agree on which entries lie inside.
template <typename R>
__device__ __forceinline__ double entry_r(const typename Vec4<R>::type &li, const typename Vec4<R>::type &lj,
                                          const typename Vec4<R>::type &D, R3<R> &d)
{
    d = pair_vec<R>(li, lj, D);
    return (double)dev_sqrt(d.x * d.x + d.y * d.y + d.z * d.z);
}

// Assemble the Coulomb rows of the step: the list entries inside rc, in list
// order, into hidx/Hr (group ballots give each lane its place), and the
// starting residual r = -(H q0 + chi) + mu_prev.  A row is flagged (hwide)
// when one of its entries lies further from the tile than a 16-bit offset
// from any slice of the tile reaches (which keeps it in the halo window too).
//
// ROWS rows per block: a tile per block where the launch fills the chip, FINE
// rows where it does not (a group then takes one row instead of sixteen one
// after another: the rows' loads, not the chip, set the time: 512 atoms 166 ->
// 16 us, 20,000 atoms 202 -> 27 us).
template <typename R, int LPR, int ROWS>
__global__ void __launch_bounds__(TILE) k_assemble(const Tile *tiles, Seg *segs, Params<double> PD)
{
    using V4 = typename Vec4<R>::type;
    const Tile T = my_rows<ROWS>(tiles);
    const Seg &S = segs[T.seg];
    __shared__ V4 dtab[NCODE];
    load_dtab2<R>(S, dtab);
    const V4 *xs = reinterpret_cast<const V4 *>(S.xs);
    const auto qv = gbl(S.q);
    R *Hr = reinterpret_cast<R *>(S.Hr);
    const double mprev = S.sst->mu_prev;
    constexpr int G = TILE / LPR;
    const int lane = threadIdx.x % LPR;
    const unsigned below = (1u << lane) - 1u;
    // Each group stages its kept entries in LDS and writes them out FL at a
    // time: whole 128-byte lines of hidx (rows start on 2 KB boundaries), so
    // no line of the output is written in pieces.
    constexpr int FL = 32;
    __shared__ uint32_t bidx_lds[G][FL + LPR];
    __shared__ R bval_lds[G][FL + LPR];
    uint32_t *bi = bidx_lds[threadIdx.x / LPR];
    R *bv = bval_lds[threadIdx.x / LPR];
    for (int k = threadIdx.x / LPR; k < ROWS; k += G) {
        const int s = T.row0 + k;
        if (s >= S.n) {
            if (s < S.npad && lane == 0) {
                S.hcnt[s] = 0;
                S.hwide[s] = 0;
            }
            continue;                          // the whole group skips together
        }
        const V4 li = xs[s];
        const int ti = (int)li.w;
        const double g3_0 = PD.g3[ti * 2], g3_1 = PD.g3[ti * 2 + 1];
        const int cnt = S.lcnt[s];
        const auto row = gbl(S.lidx + (size_t)s * S.Wl);
        const auto hrow = gblw(S.hidx + (size_t)s * S.Wl);
        const auto vrow = gblw(Hr + (size_t)s * S.Wl);
        double acc = 0.0;
        int nbuf = 0, done = 0;
        bool wide = false;
        const int tbase = s & ~(TILE - 1);      // the row may take any slice of its tile
        for (int e0 = 0; e0 < cnt; e0 += LPR) {
            const int e = e0 + lane;
            bool in = false;
            uint32_t ent = 0;
            int j = 0, tj = 0;
            double r = 0.0, qj = 0.0;
            if (e < cnt) {
                ent = row[e];
                j = (int)(ent & J_MASK);
                const V4 lj = ld4<R>(xs, j);
                qj = qv[j];                      // loaded beside the position (most entries are kept)
                tj = (int)lj.w;
                R3<R> d;
                r = entry_r<R>(li, lj, dtab[ent >> CODE_SHIFT], d);
                in = r < PD.rc;
            }
            const unsigned gm = group_ballot<LPR>(in);
            double cv = 0.0;
            if (in) {
                const int at = nbuf + __popc(gm & below);
                const R c = (R)coul64_val_g(PD, tj ? g3_1 : g3_0, r);
                bi[at] = ent;
                bv[at] = c;
                cv = (double)c;
                const int off = j - tbase;
                wide = wide || off - (TILE - SLICE) < -32768 || off > 32767;
            }
            acc += cv * qj;
            nbuf += __popc(gm);
            __builtin_amdgcn_wave_barrier();
            if (nbuf >= FL) {
                for (int t = lane; t < FL; t += LPR) {
                    hrow[done + t] = bi[t];
                    vrow[done + t] = bv[t];
                }
                const int rest = nbuf - FL;      // < LPR
                uint32_t ri = 0;
                R rv = (R)0;
                if (lane < rest) {
                    ri = bi[FL + lane];
                    rv = bv[FL + lane];
                }
                __builtin_amdgcn_wave_barrier();
                if (lane < rest) {
                    bi[lane] = ri;
                    bv[lane] = rv;
                }
                __builtin_amdgcn_wave_barrier();
                done += FL;
                nbuf = rest;
            }
        }
        for (int t = lane; t < nbuf; t += LPR) {
            hrow[done + t] = bi[t];
            vrow[done + t] = bv[t];
        }
        __builtin_amdgcn_wave_barrier();
        acc = group_sum<LPR>(acc);
        wide = group_ballot<LPR>(wide) != 0u;
        if (lane == 0) {
            const double qs = S.q[s];
            S.hcnt[s] = done + nbuf;
            S.hwide[s] = wide ? 1 : 0;
            S.jd[s] = PD.J[ti];
            S.r[s] = -(PD.J[ti] * qs + acc + PD.chi[ti]) + mprev;
            S.p[s] = 0.0;
        }
    }
}

// Sliced copy (hsidx, H) of the step's rows (hidx, Hr) for the charge-solve
// product, and the block-Jacobi preconditioner.  Each block first orders its
// tile's rows by decreasing length (the slot order, hperm), then transposes
// the tile one slice (SLICE slots) at a time through LDS, in chunks of HS_CH
// entries per row: four lanes read one row's chunk, 16 bytes each, of hidx
// and Hr (chunks of 16 rather than 32 entries keep the block's LDS under
// 40 KB, four blocks per CU: 736 -> 693 us), and add the entries whose
// neighbour lies in the row's own BK-row block into that block row in LDS,
// the four lanes in turn (so the additions keep list order); then every lane
// writes entries of its slot as slice columns (64 lanes store contiguous
// memory).  The tile's blocks (J on the diagonal) are then inverted in LDS by
// Gauss-Jordan elimination in FP32 (H is SPD and its blocks well conditioned,
// so no pivoting; the preconditioner only has to be symmetric positive
// definite, its accuracy sets the iteration count, not the solution),
// symmetrised and written with their row sums; the tile's partial sums of
// r m1 and m1 start the projection.
constexpr int HS_CH = 16;                // entries per row and chunk (4 lanes x 4)
constexpr int HS_E = HS_CH / 4;
constexpr int HS_LPR = 4;                // lanes reading one row's chunk

// entries e0 .. e0+N-1 of a row-major row (fewer when the row ends first)
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
template <int N, typename T>
__device__ __forceinline__ void loadN(const __attribute__((address_space(1))) T *row, int e0, int cnt, bool vec,
                                      T (&out)[N])
{
    if (vec && e0 + N <= cnt) {
        const __attribute__((address_space(1))) u32x4 *src = (const __attribute__((address_space(1))) u32x4 *)(row + e0);
        u32x4 w[N * sizeof(T) / 16];
#pragma unroll
        for (int k = 0; k < (int)(N * sizeof(T) / 16); k++) w[k] = src[k];
        memcpy(out, w, sizeof out);
    } else {
#pragma unroll
        for (int k = 0; k < N; k++) out[k] = e0 + k < cnt ? row[e0 + k] : (T)0;
    }
}

template <typename R>
__global__ void __launch_bounds__(TILE) k_hslice(const Tile *tiles, Seg *segs)
{
    const Tile T = my_tile(tiles);
    const Seg &S = segs[T.seg];
    __shared__ uint32_t ci[SLICE][HS_CH + 1];
    __shared__ R cv[SLICE][HS_CH + 1];
    __shared__ float A[TILE / BK][BK][BK + 1];
    __shared__ int cnt_lds[TILE];
    __shared__ int slot_row[TILE];
    __shared__ int slot_cnt[TILE];
    __shared__ uint8_t wide_row[TILE];
    __shared__ uint8_t sw[TILE / SLICE];
    __shared__ double lds[4 * 6];
    __shared__ unsigned long long hbm[HALO_WORDS];
    __shared__ uint16_t hpre[HALO_WORDS];
    const int tid = threadIdx.x;
    const int own = T.row0 + tid;
    const bool live = own < S.n;
    const int own_cnt = live ? S.hcnt[own] : 0;
    cnt_lds[tid] = own_cnt;
    float *Af = &A[0][0][0];
    for (int w = tid; w < TILE / BK * BK * (BK + 1); w += TILE) Af[w] = 0.0f;
    wide_row[tid] = (live && S.hwide[own] != 0) ? 1 : 0;
    // the tile's halo bitmap: an entry's place in the halo is the set bits before its own
    const int tl = T.row0 / TILE;
    const bool hfit = S.nhalo[tl] <= HALO_MAX;
    if (hfit) {
        for (int w = tid; w < HALO_WORDS; w += TILE) {
            hbm[w] = S.hbits[(size_t)tl * HALO_WORDS + w];
            hpre[w] = S.hpre[(size_t)tl * HALO_WORDS + w];
        }
    }
    __syncthreads();
    // slot of each row: longer rows first, ties by row
    int rank = 0;
    for (int k = 0; k < TILE; k++) {
        const int c = cnt_lds[k];
        rank += (c > own_cnt || (c == own_cnt && k < tid)) ? 1 : 0;
    }
    slot_row[rank] = tid;
    slot_cnt[rank] = own_cnt;
    __syncthreads();
    // thread tid's slot is tid (row rk); a wave is a slice: the full form
    // when one of its rows needs it, else halo positions when the halo fits,
    // else 16-bit offsets from the slice's first slot
    const int rk = slot_row[tid];
    const int rrow = T.row0 + rk;
    S.hperm[own] = (uint8_t)rk;
    const uint8_t smode = __ballot(wide_row[rk] != 0) != 0ull ? SL_FULL : !hfit ? SL_OFF16
                          : slot_cnt[tid & ~(SLICE - 1)] <= (S.Wl & ~(GRP - 1)) ? SL_HALO : SL_HALO16;
    if ((tid & (SLICE - 1)) == 0) {
        S.swide[own / SLICE] = smode;
        sw[tid / SLICE] = smode;
    }
    // slots padded to the slice's longest row (its first slot)
    const double slots = (tid & (SLICE - 1)) == 0 ? (double)SLICE * (double)slot_cnt[tid] : 0.0;
    __syncthreads();                         // every slice's form (sw) is set
    const R *Hr = reinterpret_cast<const R *>(S.Hr);
    const auto H = gblw(reinterpret_cast<R *>(S.H));
    const auto hsidx = gblw(S.hsidx);
    const auto hs16 = gblw(S.hs16);
    const bool vec = (S.Wl & 3) == 0;        // rows start on 16-byte boundaries
    for (int sl = 0; sl < TILE / SLICE; sl++) {
        const int slot0 = sl * SLICE;
        const int sbase = T.row0 + slot0;
        const int mlen = slot_cnt[slot0];
        const int mode = sw[sl];
        // reading: lanes 4l .. 4l+3 take slot l's row
        const int rl = tid / HS_LPR, rq = tid % HS_LPR;
        const int rrk = slot_row[slot0 + rl];
        const int rcnt = slot_cnt[slot0 + rl];
        const int rbb = (T.row0 + rrk) & ~(BK - 1);
        const auto irow = gbl(S.hidx + (size_t)(T.row0 + rrk) * S.Wl);
        const auto vrow = gbl(Hr + (size_t)(T.row0 + rrk) * S.Wl);
        // writing: lane l of wave w takes entries w, w+4, ... of slot l's chunk
        const int wl = tid % SLICE, wq = tid / SLICE;
        const int wcnt = slot_cnt[slot0 + wl];
        const size_t b0 = slice_base(sbase + wl, S.Wl);
        float *arow = &A[rrk / BK][rrk % BK][0];
        for (int E0 = 0; E0 < mlen; E0 += HS_CH) {
            const int e0 = E0 + rq * HS_E;
            if (e0 < rcnt) {
                uint32_t ie[HS_E];
                R ve[HS_E];
                loadN<HS_E>(irow, e0, rcnt, vec, ie);
                loadN<HS_E>(vrow, e0, rcnt, vec, ve);
#pragma unroll
                for (int k = 0; k < HS_E; k++) {
                    ci[rl][rq * HS_E + k] = ie[k];
                    cv[rl][rq * HS_E + k] = ve[k];
                }
                // entries whose neighbour lies in the row's own block, added
                // into its block row by the row's four lanes in turn (the
                // lanes of one wave: their LDS accesses stay in order), so
                // the additions keep list order
                for (int q4 = 0; q4 < HS_LPR; q4++) {
                    if (rq == q4) {
#pragma unroll
                        for (int k = 0; k < HS_E; k++) {
                            const unsigned col = (unsigned)((int)(ie[k] & J_MASK) - rbb);
                            if (e0 + k < rcnt && col < (unsigned)BK) arow[col] += (float)ve[k];
                        }
                    }
                    __builtin_amdgcn_wave_barrier();
                }
            }
            __syncthreads();
            // an entry's place in the halo
            auto place = [&](uint32_t ent) {
                const int hw = (int)(ent & J_MASK) - T.row0 + HALO_WIN / 2;
                const unsigned long long below = (1ull << (hw & 63)) - 1ull;
                return (unsigned)(hpre[hw >> 6] + __popcll(hbm[hw >> 6] & below));
            };
            if (mode == SL_HALO) {
                // wave w takes entries 4w .. 4w+3 of the chunk, half a group
                // (past the row's end, up to a whole group, zeros)
                static_assert(HS_CH == 16 && GRP == 8, "four waves, half a group each");
                const int e = E0 + 4 * wq, g = e / GRP, h = (e / 4) & 1;
                if (g * GRP < wcnt) {
                    typedef R rv4 __attribute__((ext_vector_type(4)));
                    rv4 v;
                    unsigned long long w = 0ull;
#pragma unroll
                    for (int k = 0; k < 4; k++) {
                        const bool in = e + k < wcnt;
                        v[k] = in ? cv[wl][4 * wq + k] : (R)0;
                        w |= (unsigned long long)(in ? place(ci[wl][4 * wq + k]) : 0u) << (12 * k);
                    }
                    const size_t at = hs_group(sbase + wl, g, S.Wl) + 3 * h;
#pragma unroll
                    for (int k = 0; k < 3; k++) hs16[at + k] = (uint16_t)(w >> (16 * k));
                    constexpr int V = 16 / sizeof(R);
                    typedef R rv __attribute__((ext_vector_type(V)));
#pragma unroll
                    for (int k = 0; k < 4 / V; k++) {
                        rv o;
#pragma unroll
                        for (int t = 0; t < V; t++) o[t] = v[k * V + t];
                        *(__attribute__((address_space(1))) rv *)(H + hs_plane<R>(sbase + wl, g, h * (4 / V) + k,
                                                                                 S.Wl)) = o;
                    }
                }
            } else
#pragma unroll
            for (int k = 0; k < HS_CH / 4; k++) {
                const int c = wq + 4 * k;
                const int e = E0 + c;
                if (e < wcnt) {
                    const uint32_t ent = ci[wl][c];
                    if (mode == SL_HALO16) {
                        hs16[b0 + (size_t)e * SLICE] = (uint16_t)place(ent);
                    } else if (mode == SL_OFF16) {
                        hs16[b0 + (size_t)e * SLICE] = (uint16_t)((int)(ent & J_MASK) - sbase + 32768);
                    } else {
                        hsidx[b0 + (size_t)e * SLICE] = ent;
                    }
                    H[b0 + (size_t)e * SLICE] = cv[wl][c];
                }
            }
            __syncthreads();
        }
    }
    __syncthreads();
    // the tile's BK x BK blocks ([block][row][col]) hold the block rows; add
    // J on the diagonal (identity rows past n), then one row per thread in row order
    {
        const bool rlive = rrow < S.n;
        const int rb = rk / BK, ri = rk % BK;
        if (rlive) {
            A[rb][ri][ri] += (float)S.jd[rrow];
        } else {
#pragma unroll
            for (int t = 0; t < BK; t++) A[rb][ri][t] = (t == ri ? 1.0f : 0.0f);
        }
    }
    __syncthreads();
    const int blk = tid / BK, i = tid % BK;
    // in-place Gauss-Jordan inversion, thread i updates row i
    for (int k = 0; k < BK; k++) {
        const float piv = 1.0f / A[blk][k][k];
        const float aik = A[blk][i][k];
        float rowk[BK];
#pragma unroll
        for (int t = 0; t < BK; t++) rowk[t] = A[blk][k][t];
        __syncthreads();
        if (i == k) {
#pragma unroll
            for (int t = 0; t < BK; t++) A[blk][k][t] = (t == k) ? piv : rowk[t] * piv;
        } else {
            const float f = aik * piv;
#pragma unroll
            for (int t = 0; t < BK; t++) A[blk][i][t] = (t == k) ? -f : A[blk][i][t] - f * rowk[t];
        }
        __syncthreads();
    }
    // row i of the block (symmetrised), rounded to FP16 and stored as the
    // row's 16 entries; the row sum m1 is taken from the rounded entries, so
    // that the projection uses exactly the preconditioner that is applied
    double m1 = 0.0;
    _Float16 *bo = S.binv + (size_t)(T.row0 + blk * BK + i) * BK;
#pragma unroll
    for (int t = 0; t < BK; t++) {
        const _Float16 b = (_Float16)(0.5f * (A[blk][i][t] + A[blk][t][i]));
        bo[t] = b;
        m1 += (double)(float)b;
    }
    double v[6] = {0, 0, 0, 0, 0, 0};
    if (live) {
        S.m1[own] = m1;
        v[0] = S.r[own] * m1;
        v[1] = (double)own_cnt;
        v[2] = sw[rank / SLICE] == SL_FULL ? (double)own_cnt : 0.0;
        v[4] = m1;
        v[5] = sw[rank / SLICE] == SL_HALO || sw[rank / SLICE] == SL_HALO16 ? (double)own_cnt : 0.0;
    } else if (own < S.npad) {
        S.m1[own] = 0.0;
    }
    v[3] = slots;
    tile_partials<6>(S, T.row0 / TILE, v, lds);
}

// y = M r for row s: the row of s's block inverse (16 FP16 entries, two
// 16-byte loads) against the block's r, exchanged by shuffles within the BK
// lanes of the block (every lane of the block must call it; rows past n pass
// r = 0).  The inverse only sets the iteration count: symmetric and positive
// definite after rounding (its entries move by ~5e-4 relative, its smallest
// eigenvalues are ~1e-2 of its largest), so the solution is unchanged.
__device__ __forceinline__ double block_apply(const _Float16 *binv, int s, double r)
{
    static_assert(BK == 16, "a row of the block is two 16-byte words");
    typedef _Float16 h8 __attribute__((ext_vector_type(8)));
    const auto B = gbl(reinterpret_cast<const h8 *>(binv + (size_t)s * BK));
    const h8 b0 = B[0], b1 = B[1];
    double y = 0.0;
#pragma unroll
    for (int t = 0; t < 8; t++) y += (double)(float)b0[t] * __shfl(r, t, BK);
#pragma unroll
    for (int t = 0; t < 8; t++) y += (double)(float)b1[t] * __shfl(r, 8 + t, BK);
    return y;
}

// First pass over the starting residual: its M-weighted mean w0 = 1^T M r /
// 1^T M 1, and the start of the single-reduction solve, whose first update
// shifts r by w0 (the shift left by rounding is measured by its first
// finalize and removed with the next update's shift; the charge coupling's
// solve and the adjoint take a second pass instead, k_shift_stats and
// k_fin_assemble, which set the state again).
__global__ void k_fin_w0(const int *seg_ids, Seg *segs)
{
    const Seg &S = segs[seg_ids[blockIdx.x]];
    __shared__ double lds[4 * 6];
    double tot[6];
    seg_total<6>(S, lds, tot);
    if (threadIdx.x == 0) {
        SegState *st = S.sst;
        st->sdinv = tot[4];
        st->w = tot[0] / tot[4];
        st->nnz_coul = tot[1];
        st->nnz_wide = tot[2];
        st->nnz_slots = tot[3];
        st->nnz_halo = tot[5];
        st->mshift = st->mu_prev - st->w;
        st->iters = 0;
        st->qshift = 0.0;
        st->cg_first = 1;
        st->cg_last = 0;
        st->par = 0;
    }
}

// Second pass: r <- r - w0 and the sums of the shifted residual.  Forming
// r^T z and the projected norm from one-pass sums of the unshifted residual
// cancels catastrophically when r is nearly constant (for instance a
// single-species input, whose exact residual is constant).
__global__ void __launch_bounds__(TILE) k_shift_stats(const Tile *tiles, Seg *segs)
{
    const Tile T = my_tile(tiles);
    const Seg &S = segs[T.seg];
    __shared__ double lds[4 * 4];
    const int s = T.row0 + threadIdx.x;
    const bool live = s < S.n;
    // the segment's pointers in registers before the first store
    const auto rv = gblw(S.r);
    const auto yv = gblw(S.y);
    const auto m1 = gbl(S.m1);
    const _Float16 *binv = S.binv;
    double r = 0.0;
    if (live) {
        const double w = S.sst->w;
        r = rv[s] - w;
        rv[s] = r;
        if (S.rl) S.rl[s] -= w;              // f_q coupling: the quadratic part too
    }
    const double y = block_apply(binv, s, r);
    double v[4] = {0, 0, 0, 0};
    if (live) {
        yv[s] = y;
        v[0] = r * m1[s];
        v[1] = r * y;
        v[2] = r;
        v[3] = r * r;
    }
    tile_partials<4>(S, T.row0 / TILE, v, lds);
}

__global__ void k_fin_assemble(const int *seg_ids, Seg *segs, CgCtl ctl)
{
    const Seg &S = segs[seg_ids[blockIdx.x]];
    __shared__ double lds[4 * 4];
    double tot[4];
    seg_total<4>(S, lds, tot);
    if (threadIdx.x == 0) {
        SegState *st = S.sst;
        const double w0 = st->w;
        const double w = tot[0] / st->sdinv;          // residual shift left after the first pass
        const double res2 = (tot[3] - tot[2] * tot[2] / S.n) / S.n;
        st->w = w;
        st->rho = tot[1] - w * tot[0];
        st->beta = 0.0;
        st->res = sqrt(fmax(res2, 0.0));
        st->res0 = st->res;
        st->mshift = st->mu_prev - w0 - w;
        st->iters = 0;
        st->qshift = 0.0;
        st->cg_first = 1;
        st->cg_last = 0;
        st->done = (st->res < ctl.tol) ? 1 : 0;
    }
}

// r <- r - w,  p <- M (r - w 1) + beta p = (y - w m1) + beta p (the charge
// coupling's nonlinear solve; the linear solves use the single-reduction form)
__global__ void __launch_bounds__(TILE) k_cg_dir(const Tile *tiles, Seg *segs)
{
    const Tile T = my_tile(tiles);
    const Seg &S = segs[T.seg];
    if (S.sst->done) return;
    const int s = T.row0 + threadIdx.x;
    if (s >= S.n) return;
    const double w = S.sst->w, beta = S.sst->beta;
    const auto rv = gblw(S.r);
    const auto pv = gblw(S.p);
    const double y = gbl(S.y)[s], m1 = gbl(S.m1)[s], p = pv[s];
    const double r = rv[s] - w;
    rv[s] = r;
    pv[s] = (y - w * m1) + beta * p;
    if (S.rl) S.rl[s] -= w;                  // f_q coupling: the quadratic part too
}

// s = H p and the tile's share of p^T s, one row per lane; U entries of the
// row are loaded before their products are summed, so U gathers of p are in
// flight per lane (U accumulators, combined in a fixed order at the end).
template <typename R, int U, typename IDX>
__device__ __forceinline__ double spmv_row(const double *p_, const IDX *row_, const R *hrow_, int cnt, int jbase)
{
    const auto p = gbl(p_);
    const auto row = gbl(row_);
    const auto hrow = gbl(hrow_);
    double acc[U];
#pragma unroll
    for (int u = 0; u < U; u++) acc[u] = 0.0;
    int e = 0;
    for (; e + U <= cnt; e += U) {
        IDX jj[U];
        R hh[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            jj[u] = __builtin_nontemporal_load(row + (size_t)(e + u) * SLICE);
            hh[u] = __builtin_nontemporal_load(hrow + (size_t)(e + u) * SLICE);
        }
#pragma unroll
        for (int u = 0; u < U; u++) acc[u] += (double)hh[u] * p[jbase + (int)(jj[u] & J_MASK)];
    }
    for (; e < cnt; e++)
        acc[0] += (double)__builtin_nontemporal_load(hrow + (size_t)e * SLICE) *
                  p[jbase + (int)(__builtin_nontemporal_load(row + (size_t)e * SLICE) & J_MASK)];
    double a = 0.0;
#pragma unroll
    for (int u = 0; u < U; u++) a += acc[u];
    return a;
}

// A slot of a 12-bit halo slice: 8 entries per group, 5.5 bytes each (FP32),
// three loads per group and the next group's in flight meanwhile.  Bound by
// HBM: 1,008,640 atoms 202 us with 16-bit positions and sixteen loads per 8
// entries, 192 now (beside the covalent kernels in part).
template <typename R>
__device__ __forceinline__ double spmv_row_group(const double *hp, const uint16_t *hs16, const R *H, int slot, int cnt,
                                                 int W)
{
    constexpr int V = 16 / sizeof(R), NP = GRP / V;
    typedef R rv __attribute__((ext_vector_type(V)));
    const auto pos = gbl(reinterpret_cast<const unsigned *>(hs16 + hs_group(slot, 0, W)));
    const auto val = (const __attribute__((address_space(1))) rv *)gbl(H + hs_plane<R>(slot, 0, 0, W));
    const int ng = (cnt + GRP - 1) / GRP;
    double acc[GRP];
#pragma unroll
    for (int u = 0; u < GRP; u++) acc[u] = 0.0;
    unsigned w[2][3];
    rv v[2][NP];
    auto load = [&](int b, int g) {
#pragma unroll
        for (int k = 0; k < 3; k++) w[b][k] = __builtin_nontemporal_load(pos + (size_t)g * (SLICE * 3) + k);
#pragma unroll
        for (int k = 0; k < NP; k++) v[b][k] = __builtin_nontemporal_load(val + ((size_t)g * NP + k) * SLICE);
    };
    auto use = [&](int b) {
        const unsigned long long lo = ((unsigned long long)w[b][1] << 32) | w[b][0],
                                 hi = ((unsigned long long)w[b][2] << 32) | w[b][1];
        const unsigned p[GRP] = {(unsigned)lo & 4095u,         (unsigned)(lo >> 12) & 4095u,
                                 (unsigned)(lo >> 24) & 4095u, (unsigned)(lo >> 36) & 4095u,
                                 (unsigned)(hi >> 16) & 4095u, (unsigned)(hi >> 28) & 4095u,
                                 (unsigned)(hi >> 40) & 4095u, (unsigned)(hi >> 52) & 4095u};
#pragma unroll
        for (int u = 0; u < GRP; u++) acc[u] += (double)v[b][u / V][u % V] * hp[p[u]];
    };
    if (ng > 0) load(0, 0);
    for (int g = 0; g < ng; g += 2) {
        if (g + 1 < ng) load(1, g + 1);
        use(0);
        if (g + 2 < ng) load(0, g + 2);
        if (g + 1 < ng) use(1);
    }
    double a = 0.0;
#pragma unroll
    for (int u = 0; u < GRP; u++) a += acc[u];
    return a;
}

// The same with p of the tile's halo staged in LDS (hp) and the row's
// entries as 16-bit halo positions; products and sums in the same order.
template <typename R, int U>
__device__ __forceinline__ double spmv_row_halo(const double *hp, const uint16_t *row_, const R *hrow_, int cnt)
{
    const auto row = gbl(row_);
    const auto hrow = gbl(hrow_);
    double acc[U];
#pragma unroll
    for (int u = 0; u < U; u++) acc[u] = 0.0;
    int e = 0;
    for (; e + U <= cnt; e += U) {
        uint16_t jj[U];
        R hh[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            jj[u] = __builtin_nontemporal_load(row + (size_t)(e + u) * SLICE);
            hh[u] = __builtin_nontemporal_load(hrow + (size_t)(e + u) * SLICE);
        }
#pragma unroll
        for (int u = 0; u < U; u++) acc[u] += (double)hh[u] * hp[jj[u]];
    }
    for (; e < cnt; e++)
        acc[0] += (double)__builtin_nontemporal_load(hrow + (size_t)e * SLICE) *
                  hp[__builtin_nontemporal_load(row + (size_t)e * SLICE)];
    double a = 0.0;
#pragma unroll
    for (int u = 0; u < U; u++) a += acc[u];
    return a;
}

// What the product kernel computes: for the f_q coupling's nonlinear solve
// s = H p with p^T s and p^T r (the line search); for the single-reduction
// solve H y of y = M r, into hz, with the six sums its finalize needs.
enum SpmvMode { SP_FQ = 1, SP_CG1 = 2 };
constexpr int P_UPD = 0;    // single-reduction solve: partials 0..7 from the update,
constexpr int P_PRD = 8;    // 8..13 from the product
constexpr int P_CG1 = 14;   // partials the finalize adds up

// s = H p and the tile's share of p^T s, one slot (row) per lane over the
// sliced copy; U entries of the row are loaded before their products are
// summed (U accumulators, combined in a fixed order at the end).  The block
// first stages p of its tile's halo in LDS; a slice of halo positions then
// reads 5.5 bytes per entry from memory and p from LDS.  Slices of 16-bit
// offsets (the halo did not fit) or full entries gather p from memory.
template <typename R, int U, int MODE>
__global__ void __launch_bounds__(TILE) k_spmv(const Tile *tiles, Seg *segs)
{
    const Tile T = my_tile(tiles);
    const Seg &S = segs[T.seg];
    if (S.sst->done || (MODE == SP_CG1 && S.sst->cg_last)) return;
    __shared__ double lds[4 * 6];
    __shared__ double hp[HALO_MAX];
    const double *x = MODE == SP_CG1 ? S.y : S.p;
    // rows in order (the epilogue's loads and stores coalesce), loaded
    // first so that their latency hides behind the staging and the rows
    // (also in the FP64 kernel, where they cost a wave per SIMD: loading
    // them after the rows was slower)
    const int row = T.row0 + threadIdx.x;
    const bool live = row < S.n;
    double xs = 0.0, jd = 0.0, m1s = 0.0, rs = 0.0, ss = 0.0;
    if (live) {
        xs = x[row];
        jd = S.jd[row];
        if (MODE == SP_CG1) {
            m1s = S.m1[row];
            rs = S.r[row];
            ss = S.s[row];
        }
        if (MODE == SP_FQ) rs = S.r[row];
    }
    const int tl = T.row0 / TILE;
    const int nh = S.nhalo[tl];
    if (nh <= HALO_MAX) {
        const auto hl = gbl(S.halo + (size_t)tl * HALO_MAX);
        const auto pg = gbl(x);
        for (int k = threadIdx.x; k < nh; k += TILE) hp[k] = pg[hl[k]];
    }
    __syncthreads();
    // lane = slot: its row's off-diagonal sum, handed to the row's lane in LDS
    const int slot = T.row0 + threadIdx.x;
    const int rl = S.hperm[slot];
    const int s = T.row0 + rl;
    double a = 0.0;
    if (s < S.n) {
        const size_t b0 = slice_base(slot, S.Wl);
        const R *hrow = reinterpret_cast<const R *>(S.H) + b0;
        const int cnt = S.hcnt[s];
        const int mode = S.swide[slot / SLICE];
        a = mode == SL_HALO ? spmv_row_group<R>(hp, S.hs16, reinterpret_cast<const R *>(S.H), slot, cnt, S.Wl)
            : mode == SL_HALO16 ? spmv_row_halo<R, U>(hp, S.hs16 + b0, hrow, cnt)
            : mode == SL_FULL ? spmv_row<R, U, uint32_t>(x, S.hsidx + b0, hrow, cnt, 0)
                              : spmv_row<R, U, uint16_t>(x, S.hs16 + b0, hrow, cnt, (slot & ~(SLICE - 1)) - 32768);
    }
    __syncthreads();
    hp[rl] = a;
    __syncthreads();
    double v[6] = {0, 0, 0, 0, 0, 0};
    if (live) {
        const double y = jd * xs + hp[threadIdx.x];
        if (MODE == SP_CG1) {
            S.hz[row] = y;
            v[0] = xs * y;                   // y^T H y
            v[1] = m1s * y;                  // m1^T H y
            v[2] = rs * y;                   // r^T H y
            v[3] = y * y;
            v[4] = ss * y;                   // s_old^T H y
            v[5] = y;
        } else {
            S.s[row] = y;
            v[0] = xs * y;
            v[1] = xs * rs;
        }
    }
    if (MODE == SP_CG1) {
        tile_partials_at<6>(S, tl, v, lds, P_PRD);
    } else {
        double w[2] = {v[0], v[1]};
        tile_partials<2>(S, tl, w, lds);
    }
}

// ---------------------------------------------------------------------------
// Systems of up to SPLIT_TILES tiles that no one-launch solve takes (or whose
// own gave up), where the host finds that it pays (split_iteration): the product
// with eight waves per row slice, and the finalize in the update (two launches
// per iteration instead of four).  There a lane per row leaves most of the card idle and an
// iteration is a chain of launches that each wait for memory once or twice:
// with 36,864 atoms 50 us (product 29.5, its sums 8.8, update 4.5, gaps) and
// 31 this way (18, 7.3, gaps), ten MD steps 19.4 and 12.8 ms (8.2 in one launch).
// ---------------------------------------------------------------------------
constexpr int SPLIT_TILES = 256;
static_assert(sizeof(SegState) <= 16 * FIN_SPLIT * sizeof(double) && sizeof(SegState) / 4 <= TILE, "scratch, a word per thread");
constexpr int SPLIT = TILE / SLICE;         // blocks per tile: one per slice

// scratch of the split iteration: the product's partials (k of block b at k
// * blocks + b) where the list build keeps an order, the solver's state at
// the product in the group sums' place
__device__ __forceinline__ double *split_part(const Seg &S) { return reinterpret_cast<double *>(S.perm_tmp); }
__device__ __forceinline__ SegState *split_state(const Seg &S)
{
    return reinterpret_cast<SegState *>(S.part + (size_t)NPART * S.ntile);
}

constexpr int SPLIT_T = 512, SPLIT_W = SPLIT_T / 64;

// One wave's share of a row: entries in groups of GRP, every SPLIT_W-th
// group (the first is loaded before y is staged).
template <typename R>
struct SplitRow {
    static constexpr int V = 16 / sizeof(R), NP = GRP / V;
    typedef R rv __attribute__((ext_vector_type(V)));
    const __attribute__((address_space(1))) unsigned *pos;
    const __attribute__((address_space(1))) rv *val;
    int ng, g;
    unsigned w[3];
    rv v[NP];
    __device__ __forceinline__ void load()
    {
        if (g >= ng) return;
#pragma unroll
        for (int k = 0; k < 3; k++) w[k] = pos[(size_t)g * (SLICE * 3) + k];
#pragma unroll
        for (int k = 0; k < NP; k++) v[k] = val[((size_t)g * NP + k) * SLICE];
    }
    __device__ __forceinline__ double sum(const double *hp)
    {
        double acc[GRP];
#pragma unroll
        for (int u = 0; u < GRP; u++) acc[u] = 0.0;
        while (g < ng) {
            const unsigned long long lo = ((unsigned long long)w[1] << 32) | w[0],
                                     hi = ((unsigned long long)w[2] << 32) | w[1];
            const unsigned p[GRP] = {(unsigned)lo & 4095u,         (unsigned)(lo >> 12) & 4095u,
                                     (unsigned)(lo >> 24) & 4095u, (unsigned)(lo >> 36) & 4095u,
                                     (unsigned)(hi >> 16) & 4095u, (unsigned)(hi >> 28) & 4095u,
                                     (unsigned)(hi >> 40) & 4095u, (unsigned)(hi >> 52) & 4095u};
#pragma unroll
            for (int u = 0; u < GRP; u++) acc[u] += (double)v[u / V][u % V] * hp[p[u]];
            g += SPLIT_W;
            load();
        }
        double a = 0.0;
#pragma unroll
        for (int u = 0; u < GRP; u++) a += acc[u];
        return a;
    }
};

// The same of entries that are not grouped: positions idx(e) into x.
template <typename R, typename X, typename I>
__device__ __forceinline__ double spmv_part(X x, const R *hrow_, int cnt, int wv, I idx)
{
    const auto hrow = gbl(hrow_);
    double acc[GRP];
#pragma unroll
    for (int u = 0; u < GRP; u++) acc[u] = 0.0;
    for (int e0 = wv * GRP; e0 < cnt; e0 += SPLIT_W * GRP) {
        int j[GRP];
        R h[GRP];
#pragma unroll
        for (int u = 0; u < GRP; u++) {
            const int e = min(e0 + u, cnt - 1);
            j[u] = idx(e);
            h[u] = hrow[(size_t)e * SLICE];
        }
#pragma unroll
        for (int u = 0; u < GRP; u++)
            if (e0 + u < cnt) acc[u] += (double)h[u] * x[j[u]];
    }
    double a = 0.0;
#pragma unroll
    for (int u = 0; u < GRP; u++) a += acc[u];
    return a;
}

// H y of one slice (a lane per row, SPLIT_W waves sharing its entries), and
// the six sums the finalize needs; also copies the solver's state for the
// update.  Bound by latency (five loads that wait for one another, 38 MB of
// entries at 2.1 TB/s beside them): what does not wait for y (the halo list,
// the first entries) is loaded before the test for the end of the solve, and
// three blocks fit on a CU, so that 65,536 atoms run in two rounds (four
// waves per slice 22 us, eight with up to four groups in flight 18.4 to 19.3,
// one group in flight 17.8).
template <typename R>
__global__ void __launch_bounds__(SPLIT_T, sizeof(R) == 8 ? 4 : 6) k_spmv_split(const Tile *tiles, Seg *segs)
{
    constexpr int NHL = HALO_MAX / SPLIT_T;
    static_assert(HALO_MAX % SPLIT_T == 0, "whole rounds of the staging");
    const Tile T = tiles[blockIdx.x / SPLIT];
    const int sl = blockIdx.x % SPLIT, wv = __builtin_amdgcn_readfirstlane(threadIdx.x / SLICE),
              wl = threadIdx.x % SLICE;
    const Seg &S = segs[T.seg];
    const int tl = T.row0 / TILE;
    const int slot = T.row0 + sl * SLICE + wl;
    const int rl = gbl(S.hperm)[slot];
    const int nh = S.nhalo[tl], mode = S.swide[slot / SLICE], over = S.sst->done | S.sst->cg_last;
    const auto hl = gbl(S.halo + (size_t)tl * HALO_MAX);
    int j[NHL];
#pragma unroll
    for (int u = 0; u < NHL; u++) j[u] = (int)hl[threadIdx.x + u * SPLIT_T];
    if (tl == 0 && sl == 0 && threadIdx.x < sizeof(SegState) / 4)
        reinterpret_cast<int *>(split_state(S))[threadIdx.x] = reinterpret_cast<const int *>(S.sst)[threadIdx.x];
    if (over) return;
    __shared__ double hp[HALO_MAX];
    __shared__ double sum[SPLIT_W][SLICE];
    const int s = T.row0 + rl;
    const bool live = s < S.n;
    const auto x = gbl(S.y);
    const int cnt = live ? gbl(S.hcnt)[s] : 0;
    double xs = 0.0, jd = 0.0, m1s = 0.0, rs = 0.0, ss = 0.0;
    if (wv == 0 && live) {
        xs = x[s];
        jd = gbl(S.jd)[s];
        m1s = gbl(S.m1)[s];
        rs = gbl(S.r)[s];
        ss = gbl(S.s)[s];
    }
    double v[NHL];
    const bool staged = nh <= HALO_MAX;
    if (staged) {
#pragma unroll
        for (int u = 0; u < NHL; u++)
            if ((int)threadIdx.x + u * SPLIT_T < nh) v[u] = x[j[u]];
    }
    SplitRow<R> row;
    row.pos = gbl(reinterpret_cast<const unsigned *>(S.hs16 + hs_group(slot, 0, S.Wl)));
    row.val = (const __attribute__((address_space(1))) typename SplitRow<R>::rv *)gbl(
        reinterpret_cast<const R *>(S.H) + hs_plane<R>(slot, 0, 0, S.Wl));
    row.ng = mode == SL_HALO ? (cnt + GRP - 1) / GRP : 0;
    row.g = wv;
    row.load();
    if (staged) {
#pragma unroll
        for (int u = 0; u < NHL; u++)
            if ((int)threadIdx.x + u * SPLIT_T < nh) hp[threadIdx.x + u * SPLIT_T] = v[u];
    }
    __syncthreads();
    double a = 0.0;
    if (mode == SL_HALO) {
        a = row.sum(hp);
    } else if (live) {
        const size_t b0 = slice_base(slot, S.Wl);
        const R *hrow = reinterpret_cast<const R *>(S.H) + b0;
        const auto h16 = gbl(S.hs16 + b0);
        const auto h32 = gbl(S.hsidx + b0);
        const int jb = (slot & ~(SLICE - 1)) - 32768;
        if (mode == SL_HALO16)
            a = spmv_part<R>((const double *)hp, hrow, cnt, wv, [&](int e) { return (int)h16[(size_t)e * SLICE]; });
        else if (mode == SL_FULL)
            a = spmv_part<R>(x, hrow, cnt, wv, [&](int e) { return (int)(h32[(size_t)e * SLICE] & J_MASK); });
        else
            a = spmv_part<R>(x, hrow, cnt, wv, [&](int e) { return jb + (int)h16[(size_t)e * SLICE]; });
    }
    sum[wv][wl] = a;
    __syncthreads();
    if (wv != 0) return;
    double y = 0.0;
    if (live) {
        double t = sum[0][wl];
#pragma unroll
        for (int k = 1; k < SPLIT_W; k++) t += sum[k][wl];
        y = jd * xs + t;
        S.hz[s] = y;
    }
    const double p[6] = {xs * y, m1s * y, rs * y, y * y, ss * y, y};
    const auto out = gblw(split_part(S));
    const int nb = S.ntile * SPLIT, blk = tl * SPLIT + sl;
#pragma unroll
    for (int k = 0; k < 6; k++) {
        const double t = wave_sum(p[k]);
        if (wl == 0) out[(size_t)k * nb + blk] = t;
    }
}

// ---------------------------------------------------------------------------
// The same projected PCG with one reduction per iteration (Chronopoulos and
// Gear's rearrangement of conjugate gradients): the product is taken of
// y = M r, the unprojected preconditioned residual, and the direction's
// product follows by recurrence, s = H y + beta s.  The projection enters as
// the shift c of the residual, r <- r - c 1 with c = m1^T r / 1^T M 1, so that
// y = M r is the projected preconditioned residual; c of the next residual is
// known one step ahead from m1^T r and m1^T s.  The finalize also takes the
// projected norm of the next residual, |r|^2 - 2 alpha r^T s + alpha^2 |s|^2
// (each minus its mean part), from sums of the two kernels, so the solve
// stops after the update that meets the tolerance without a further product.
// An iteration is four launches: product (k_spmv, SP_CG1), the finalize's two
// stages (k_cg1_sum, k_cg1_fin), update; of up to SPLIT_TILES tiles it is two,
// k_spmv_split and k_cg1_step.
// ---------------------------------------------------------------------------

// p <- y + beta p, s <- H y + beta s, q <- q + alpha p, r <- r - alpha s - c,
// y <- M r, and the tile's sums for the finalize.  FIRST: the solve's start,
// which only shifts r (by the shift left after the second pass) and clears
// p and s.
template <bool FIRST>
__global__ void __launch_bounds__(TILE) k_cg1_update(const Tile *tiles, Seg *segs)
{
    const Tile T = my_tile(tiles);
    const Seg &S = segs[T.seg];
    if (S.sst->done) return;
    __shared__ double lds[4 * 8];
    const int s = T.row0 + threadIdx.x;
    const bool live = s < S.n;
    const double alpha = S.sst->alpha, beta = S.sst->beta, c = S.sst->w;
    // the segment's pointers in registers before the first store
    const auto qv = gblw(S.q);
    const auto rv = gblw(S.r);
    const auto yv = gblw(S.y);
    const auto pv = gblw(S.p);
    const auto sv = gblw(S.s);
    const auto hz = gbl(S.hz);
    const _Float16 *binv = S.binv;
    double q = 0.0, r = 0.0, sn = 0.0;
    if (live) {
        if (FIRST) {
            q = qv[s];
            r = rv[s] - c;
            pv[s] = 0.0;
            sv[s] = 0.0;
        } else {
            const double p = yv[s] + beta * pv[s];
            sn = hz[s] + beta * sv[s];
            q = qv[s] + alpha * p;
            r = (rv[s] - alpha * sn) - c;
            pv[s] = p;
            sv[s] = sn;
            qv[s] = q;
        }
        rv[s] = r;
    }
    const double y = block_apply(binv, s, r);
    double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (live) {
        yv[s] = y;
        v[0] = y;                // 1^T M r = m1^T r (M symmetric)
        v[1] = r * y;
        v[2] = r;
        v[3] = r * r;
        v[4] = q;
        v[5] = r * sn;
        v[6] = sn * sn;
        v[7] = sn;
    }
    tile_partials_at<8>(S, T.row0 / TILE, v, lds, P_UPD);
}

// First stage of the finalize: FIN_SPLIT blocks per segment, each summing
// the 14 partials over its range of tiles.
__global__ void __launch_bounds__(TILE) k_cg1_sum(const int *seg_ids, Seg *segs)
{
    const Seg &S = segs[seg_ids[blockIdx.x / FIN_SPLIT]];
    if (S.sst->done) return;
    __shared__ double lds[4 * P_CG1];
    seg_group_sum<P_CG1>(S, blockIdx.x % FIN_SPLIT, lds);
}

// The scalar step of an iteration from its 14 sums: the residual after the
// last update and the stop test; then gamma = r^T y, delta = y^T H y, beta =
// gamma / gamma_old, alpha = gamma / (delta - beta gamma / alpha_old) (= gamma
// / p^T H p), the next shift c and the projected norm of the next residual,
// which marks the coming update as the last when it meets the tolerance.
// Returns the status bits of a failed solve.  inv_n = 1/n and inv_sd = 1 /
// 1^T M 1: one thread takes the step between two kernels (or two halves of an
// iteration), so its divisions are the two that depend on the sums, and the
// root of the residual is taken at the start and the end only.
__device__ __forceinline__ int cg1_step(SegState &st, double inv_n, double inv_sd, double Q,
                                        const double (&t)[P_CG1], double tol, int maxit)
{
    const double rr = t[P_UPD + 3] - t[P_UPD + 2] * t[P_UPD + 2] * inv_n;
    const double res2 = fmax(rr * inv_n, 0.0);
    const bool first = st.cg_first != 0;
    if (!first) {
        st.iters += 1;
        st.iters_total += 1;
    }
    const bool met = st.cg_last || res2 <= tol * tol, out = st.iters >= maxit;
    const double gam = t[P_UPD + 1], del = t[P_PRD + 0];
    const double beta = first ? 0.0 : gam / st.rho;
    const double den = first ? del : del - beta * beta * st.den;   // (beta gamma / alpha_old)
    const bool bad = !(den > 0.0) || !(gam > 0.0);
    if (first) st.res0 = sqrt(res2);
    if (met || out || bad) {
        st.res = sqrt(res2);
        st.qshift = (Q - t[P_UPD + 4]) * inv_n;
        st.done = 1;
        return met ? 0 : out ? ST_NOCONV : ST_NOT_PD;
    }
    const double alpha = gam / den;
    // sums of the new s = H y + beta s_old (m1^T s by its own recurrence:
    // an error in it only leaves m1^T r of the next residual slightly off
    // zero, and the next shift, from the measured m1^T r, removes that)
    const double m1s = first ? t[P_PRD + 1] : t[P_PRD + 1] + beta * st.m1s;
    const double rs = t[P_PRD + 2] + beta * t[P_UPD + 5];
    const double ss = t[P_PRD + 3] + 2.0 * beta * t[P_PRD + 4] + beta * beta * t[P_UPD + 6];
    const double sum_s = t[P_PRD + 5] + beta * t[P_UPD + 7];
    const double c = (t[P_UPD + 0] - alpha * m1s) * inv_sd;
    const double rs_p = rs - t[P_UPD + 2] * sum_s * inv_n;
    const double ss_p = ss - sum_s * sum_s * inv_n;
    const double next2 = (rr - 2.0 * alpha * rs_p + alpha * alpha * ss_p) * inv_n;
    st.cg_first = 0;
    st.m1s = m1s;
    st.rho = gam;
    st.den = den;
    st.alpha = alpha;
    st.beta = beta;
    st.w = c;
    st.mshift -= c;
    if (next2 < tol * tol) st.cg_last = 1;
    return 0;
}

__global__ void __launch_bounds__(TILE) k_cg1_fin(const int *seg_ids, Seg *segs, CgCtl ctl)
{
    const Seg &S = segs[seg_ids[blockIdx.x]];
    if (S.sst->done) return;
    __shared__ double lds[FIN_SPLIT * P_CG1];
    double t[P_CG1];
    seg_total_groups<P_CG1>(S, lds, t);
    if (threadIdx.x == 0) {
        const int bad = cg1_step(*S.sst, 1.0 / S.n, 1.0 / S.sst->sdinv, S.Q, t, ctl.tol, ctl.maxit);
        if (bad) atomicOr(&S.sst->status, bad);
    }
}

// The split iteration's second launch: every block adds up the partials of
// all blocks and takes the scalar step itself, then updates its tile's rows
// as k_cg1_update does.  The state it reads is the product's copy and the
// first block stores the new one, and the update's partials have two sets
// (SegState::par), so no block reads what another writes.  36,864 atoms: 7.3 us
// against 13.3 and two launch gaps in three launches.
__global__ void __launch_bounds__(TILE) k_cg1_step(const Tile *tiles, Seg *segs, CgCtl ctl)
{
    const Tile T = my_tile(tiles);
    const Seg &S = segs[T.seg];
    const SegState *const old = split_state(S);
    __shared__ double lds[4 * 8];
    __shared__ double tot[16];
    __shared__ SegState st;
    constexpr int NW = TILE / 64;
    const int tid = threadIdx.x, wv = __builtin_amdgcn_readfirstlane(tid / 64), wl = tid % 64;
    if (tid < (int)(sizeof(SegState) / 4)) reinterpret_cast<int *>(&st)[tid] = reinterpret_cast<const int *>(old)[tid];
    // the row, in flight beside the sums
    const int s = T.row0 + tid, nt = S.ntile, par = old->par;
    const bool live = s < S.n;
    const auto qv = gblw(S.q);
    const auto rv = gblw(S.r);
    const auto yv = gblw(S.y);
    const auto pv = gblw(S.p);
    const auto sv = gblw(S.s);
    const auto hz = gbl(S.hz);
    const auto part = gblw(S.part);
    const _Float16 *binv = S.binv;
    double q = 0.0, r = 0.0, y = 0.0, p = 0.0, sn = 0.0, h = 0.0;
    if (live) {
        q = qv[s];
        r = rv[s];
        y = yv[s];
        p = pv[s];
        sn = sv[s];
        h = hz[s];
    }
    // sums wv, wv + NW, ...: 0..7 of the update (a partial per tile), 8..13
    // of the product (SPLIT per tile)
    const auto prd = gbl(split_part(S));
    constexpr int NU = SPLIT_TILES / 64, NP = SPLIT_TILES * SPLIT / 64;
    const int nb = nt * SPLIT, kp = 2 - wv / 2;      // the wave's sums of the product: 2, 2, 1, 1
    double xu[2][NU], xp[2][NP];
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
        for (int i = 0; i < NP; i++)
            if (i * 64 < nb) xp[h][i] = prd[(size_t)min(wv + h * NW, 5) * nb + min(i * 64 + wl, nb - 1)];
#pragma unroll
    for (int h = 0; h < 2; h++)
#pragma unroll
        for (int i = 0; i < NU; i++) xu[h][i] = part[(size_t)(8 * par + wv + h * NW) * nt + min(i * 64 + wl, nt - 1)];
    if (old->done) return;
#pragma unroll
    for (int h = 0; h < 2; h++) {
        double t = 0.0, u = 0.0;
#pragma unroll
        for (int i = 0; i < NU; i++) t += i * 64 + wl < nt ? xu[h][i] : 0.0;
#pragma unroll
        for (int i = 0; i < NP; i++)
            if (i * 64 < nb) u += i * 64 + wl < nb ? xp[h][i] : 0.0;
        t = wave_sum(t);
        u = wave_sum(u);
        if (wl == 0) {
            tot[P_UPD + wv + h * NW] = t;
            if (h < kp) tot[P_PRD + wv + h * NW] = u;
        }
    }
    __syncthreads();
    if (wv == 0) {
        const double mine = tot[wl & 15];
        double t[P_CG1];
#pragma unroll
        for (int k = 0; k < P_CG1; k++)
            t[k] = __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(mine), k),
                                    __builtin_amdgcn_readlane(__double2loint(mine), k));
        if (wl == 0) {
            const int bad = cg1_step(st, 1.0 / S.n, 1.0 / st.sdinv, S.Q, t, ctl.tol, ctl.maxit);
            if (T.row0 == 0) {
                SegState *o = S.sst;
                o->par = par ^ 1;
                o->iters = st.iters;
                o->iters_total = st.iters_total;
                o->cg_first = st.cg_first;
                o->cg_last = st.cg_last;
                o->w = st.w;
                o->rho = st.rho;
                o->alpha = st.alpha;
                o->beta = st.beta;
                o->res = st.res;
                o->res0 = st.res0;
                o->mshift = st.mshift;
                o->qshift = st.qshift;
                o->m1s = st.m1s;
                o->den = st.den;
                if (bad) atomicOr(&o->status, bad);
                o->done = st.done;
            }
        }
    }
    __syncthreads();
    if (st.done) return;
    if (live) {
        p = y + st.beta * p;
        sn = h + st.beta * sn;
        q = q + st.alpha * p;
        r = (r - st.alpha * sn) - st.w;
        pv[s] = p;
        sv[s] = sn;
        qv[s] = q;
        rv[s] = r;
    }
    y = block_apply(binv, s, r);
    double v[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (live) {
        yv[s] = y;
        v[0] = y;
        v[1] = r * y;
        v[2] = r;
        v[3] = r * r;
        v[4] = q;
        v[5] = r * sn;
        v[6] = sn * sn;
        v[7] = sn;
    }
    double u[8];
    block_sum<8>(v, lds, u);
    if (tid == 0) {
#pragma unroll
        for (int k = 0; k < 8; k++) part[(size_t)(8 * (par ^ 1) + k) * nt + T.row0 / TILE] = u[k];
    }
}

// Coulomb forces and energy at the equilibrated charges, plus the covalent
// forces and energies: writes F, q (user order) and the tile's energy.
// With ROWS < TILE (small launches, as in the assembly: 20,000 atoms 137 ->
// 18 us) the blocks' sums go to S.s, free after the solve.
template <typename R, int LPR, int ROWS>
__global__ void __launch_bounds__(TILE) k_force_coul(const Tile *tiles, Seg *segs, Params<double> PD, int gate)
{
    using V4 = typename Vec4<R>::type;
    const Tile T = my_rows<ROWS>(tiles);
    const Seg &S = segs[T.seg];
    if (gate && (!S.sst->done || S.sst->pabort || S.sst->forces_done)) return;
    __shared__ V4 dtab[NCODE];
    __shared__ double lds[4 * 3];
    load_dtab2<R>(S, dtab);
    const V4 *xs = reinterpret_cast<const V4 *>(S.xs);
    const auto qv = gbl(S.q);
    const double qsh = S.sst->qshift;
    const bool keep_hist = S.q_ring != nullptr;
    const int push = (S.sst->qhead + 1) % NHIST;       // ring slot that takes the previous solution
    constexpr int G = TILE / LPR;
    const int lane = threadIdx.x % LPR;
    const float ke32 = (float)PD.ke, irc32 = (float)PD.inv_rc;
    double esum = 0.0;
    // bond statistics of the step (for the measurement): bonds and ordered bond pairs
    double nb = 0.0, nt = 0.0;
    if ((int)threadIdx.x < ROWS && T.row0 + (int)threadIdx.x < S.n) {
        nb = (double)S.bcnt[T.row0 + threadIdx.x];
        nt = nb * (nb - 1.0);
    }
    for (int k = threadIdx.x / LPR; k < ROWS; k += G) {
        const int s = T.row0 + k;
        if (s >= S.n) continue;
        const V4 li = xs[s];
        const int ti = (int)li.w;
        const double g3_0 = PD.g3[ti * 2], g3_1 = PD.g3[ti * 2 + 1];
        const float g3f_0 = (float)g3_0, g3f_1 = (float)g3_1;
        const int cnt = S.hcnt[s];
        const auto row = gbl(S.hidx + (size_t)s * S.Wl);
        double ec = 0.0, fx = 0.0, fy = 0.0, fz = 0.0;
        for (int e = lane; e < cnt; e += LPR) {
            const uint32_t ent = row[e];
            const int j = (int)(ent & J_MASK);
            const V4 lj = ld4<R>(xs, j);
            const double qj = qv[j] + qsh;
            // every entry lies inside rc: the rows were selected by the
            // assembly's distance test (entry_r).  With FP32 pair terms the
            // distance is taken with the hardware square root (~1 ulp, as
            // close as the FP32 pair function itself) and needs no test; the
            // FP64 build keeps the test, as a select rather than a branch so
            // that the loop body stays one block and the charge load issues
            // beside the position load
            R3<R> d;
            double r;
            if constexpr (sizeof(R) == 4) {
                d = pair_vec<R>(li, lj, dtab[ent >> CODE_SHIFT]);
                r = (double)__builtin_amdgcn_sqrtf(d.x * d.x + d.y * d.y + d.z * d.z);
            } else {
                r = entry_r<R>(li, lj, dtab[ent >> CODE_SHIFT], d);
            }
            const bool in = sizeof(R) == 4 ? true : r < PD.rc;
            double dCr, c;
            if constexpr (sizeof(R) == 4) {
                float d32;
                c = (double)coul32_g(ke32, irc32, (int)lj.w ? g3f_1 : g3f_0, (float)r, d32);
                dCr = (double)d32;
            } else {
                c = coul64_g(PD, (int)lj.w ? g3_1 : g3_0, r, dCr);
            }
            c = in ? c : 0.0;
            dCr = in ? dCr : 0.0;
            ec += c * qj;
            if (j != s) {
                const double g = qj * dCr;
                fx += g * (double)d.x;
                fy += g * (double)d.y;
                fz += g * (double)d.z;
            }
        }
        ec = group_sum<LPR>(ec);
        fx = group_sum<LPR>(fx);
        fy = group_sum<LPR>(fy);
        fz = group_sum<LPR>(fz);
        if (lane == 0) {
            const double qs = S.q[s] + qsh;
            const int i = S.perm[s];
            S.F[i] = qs * fx + S.Fcov[s];
            S.F[S.n + i] = qs * fy + S.Fcov[S.npad + s];
            S.F[2 * S.n + i] = qs * fz + S.Fcov[2 * S.npad + s];
            S.q_out[i] = qs;
            if (keep_hist) S.q_ring[(size_t)push * S.n + i] = S.q_state[i];
            S.q_state[i] = qs;
            esum += PD.E0[ti] + PD.chi[ti] * qs + 0.5 * PD.J[ti] * qs * qs + 0.5 * qs * ec + S.ecov[s];
        }
    }
    double v[3] = {esum, nb, nt};
    if constexpr (ROWS == TILE) {
        tile_partials<3>(S, T.row0 / TILE, v, lds);
    } else {
        double tot[3];
        block_sum<3>(v, lds, tot);
        if (threadIdx.x == 0) {
#pragma unroll
            for (int k = 0; k < 3; k++) S.s[(size_t)k * (S.npad / ROWS) + T.row0 / ROWS] = tot[k];
        }
    }
}

template <int ROWS>
__global__ void k_fin_energy(const int *seg_ids, Seg *segs, int gate)
{
    const Seg &S = segs[seg_ids[blockIdx.x]];
    if (gate && (!S.sst->done || S.sst->pabort || S.sst->forces_done)) return;
    __shared__ double lds[4 * 3];
    double tot[3];
    if constexpr (ROWS == TILE) seg_total<3>(S, lds, tot);
    else block_total<3>(S.s, S.npad / ROWS, lds, tot);
    if (threadIdx.x == 0) {
        SegState *st = S.sst;
        st->energy = tot[0];
        st->nbond = tot[1];
        st->ntrip = tot[2];
        if (S.E_out) *S.E_out = tot[0];
        st->mu_prev = st->mshift;
        st->nhist = st->nhist < NHIST + 1 ? st->nhist + 1 : NHIST + 1;
        if (S.q_ring) st->qhead = (st->qhead + 1) % NHIST;
        st->forces_done = 1;
    }
}

// serving: per-segment flags (done, forces_done, status, iterations)
__global__ void k_collect(const int *seg_ids, Seg *segs, int nseg, int4 *out)
{
    int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= nseg) return;
    const SegState *st = segs[seg_ids[k]].sst;
    out[k] = make_int4(st->done && !st->pabort, st->pabort ? -st->pabort : st->forces_done, st->status, st->iters);
}

} // namespace ctbop
