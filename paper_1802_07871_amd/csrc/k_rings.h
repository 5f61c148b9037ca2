// k_rings.h -- ring statistics of the carbon bond graph: shortest-path rings
// (Franzblau 1991) of at most RING_MAX members, the bonds on no ring (chain
// bonds) and the in-plane orientation of every 6-membered ring, the analysis
// the paper draws for its growth and anneal runs (rings by size, chains, a
// 6-ring hue that repeats every 60 degrees).
//
// Bonds: two C atoms with an image of one within r_bond of the other, taken
// from the covalent list (complete up to S_CC at the current positions), one
// edge per atom pair.  Rings: those whose smallest user index is atom s are
// found from the pairs of s's neighbours (a, b) with larger indices: a ring
// leaves s by a and returns by b, so two half-paths grow from a and b and meet
// in a bond or a common neighbour.  A shortest-path ring has no shortcut: for
// every two ring vertices at ring distance d (at most 4), no path of fewer
// than d bonds joins them in the whole graph; the parts of that which the
// growing half-paths already break end them early, and a ring found is tested
// whole.  The cell must be at least max_size * r_bond wide in every periodic
// direction, so neither a cycle nor a shortcut can wind around it (and an atom
// pair has at most one edge).
//
// Bound by dependent, irregular reads: an atom's degree, user index and
// neighbours are one 64-byte record, read as one line, and the search meets in
// the middle instead of walking every path depth first (~10 times fewer
// atoms visited on a sheet).  1,000,000-atom sheet with 400 Stone-Wales
// defects: 8.6 ms depth first, 0.74 now (0.98 with each ring tested where it
// was found); 250,000-atom random network 4.4 -> 1.0 ms; 4,800-atom sheet
// 1.84 -> 0.17 ms.
#pragma once
#include "ctbop_dev.h"
#include "k_tersoff.h"

namespace ctbop {

constexpr int RING_DEG = 12;       // C neighbours per atom at most
constexpr int RING_MAX = 8;        // largest ring
constexpr int RING_C = 1;          // type index of carbon
// an atom's record: degree, user index, neighbours as covalent-list entries
// (row | image code; RING_NONE: none)
constexpr int REC = 16, REC_NB = 2;
constexpr uint32_t RING_NONE = 0xffffffffu;
constexpr int RING_HB = 256;       // histogram bins that a block counts in LDS

// counter slots
enum : int {
    RC_BONDS = 9,                  // 0..8: rings by size
    RC_CHAIN = 10,
    RC_LISTED = 11,                // rings found (listed up to the caller's capacity)
    RC_HIST = 12,                  // 6-rings that entered the histogram
    RC_OVERFLOW = 13,              // atoms with more than RING_DEG C neighbours
    RC_N = 16
};

struct RingWs {
    uint32_t *rec;                 // [npad * REC]
    uint32_t *mark;                // [npad] bit k: bond k lies on a ring
    unsigned long long *cnt;       // [RC_N]
    unsigned long long *hist;      // [nbins]
    int32_t *list;                 // [cap * 9] (size, user indices in ring order, -1 padding) or null
    double *orient;                // [cap] (6-rings: orientation in degrees; others: -1) or null
    long long cap;
};

struct RingCfg {
    double rb2;                    // r_bond^2
    int max_size;
    int nbins;
    double n[3], u[3], w[3];       // plane normal, reference direction in the plane, n x u
    double cos_tilt_min;           // rings whose normal is within the tilt limit; < -1: no limit
};

// The records of all atoms (degree 0 but for C atoms) and the cleared bond
// marks; four lanes take an atom's covalent list, the records leave through
// LDS as whole lines.
constexpr int ADJ_L = 4, ADJ_ROWS = TILE / ADJ_L;
__global__ void __launch_bounds__(TILE) k_ring_adj(const Tile *tiles, Seg *segs, RingWs W, RingCfg c)
{
    const Tile T = my_rows<ADJ_ROWS>(tiles);
    const Seg &S = segs[T.seg];
    __shared__ uint32_t out[ADJ_ROWS * REC];
    for (int k = threadIdx.x; k < ADJ_ROWS * REC; k += TILE) out[k] = RING_NONE;
    __syncthreads();
    const int lr = threadIdx.x / ADJ_L, lane = threadIdx.x % ADJ_L, s = T.row0 + lr;
    int nd = 0;
    if (s < S.n) {
        const double4 li = ld4<double>(S.xs64, s);
        if ((int)li.w == RING_C) {
            const auto sidx = gbl(S.sidx + (size_t)s * S.Ws);
            const int ns = S.scnt[s];
            for (int e0 = 0; e0 < ns; e0 += ADJ_L) {
                const int e = e0 + lane;
                bool in = false;
                uint32_t ent = 0;
                if (e < ns) {
                    ent = sidx[e];
                    const int j = (int)(ent & J_MASK);
                    const double4 lj = ld4<double>(S.xs64, j);
                    const R3<double> D = code_offset(S, (int)(ent >> CODE_SHIFT));
                    const R3<double> d = {(lj.x - li.x) + D.x, (lj.y - li.y) + D.y, (lj.z - li.z) + D.z};
                    in = j != s && (int)lj.w == RING_C && d.x * d.x + d.y * d.y + d.z * d.z < c.rb2;
                }
                const unsigned gm = group_ballot<ADJ_L>(in);
                const int at = nd + __popc(gm & ((1u << lane) - 1u));
                if (in && at < RING_DEG) out[lr * REC + REC_NB + at] = ent;
                nd += __popc(gm);
            }
            if (nd > RING_DEG) {
                if (lane == 0) atomicAdd(&W.cnt[RC_OVERFLOW], 1ull);
                nd = RING_DEG;
            }
        }
    }
    if (lane == 0) {
        out[lr * REC] = (uint32_t)nd;
        out[lr * REC + 1] = s < S.n ? (uint32_t)S.perm[s] : 0u;
        W.mark[s] = 0u;
    }
    __syncthreads();
    const auto rec = gblw(W.rec + (size_t)T.row0 * REC);
    for (int k = threadIdx.x; k < ADJ_ROWS * REC; k += TILE) rec[k] = out[k];
}

// An atom's record as the search holds it: neighbour rows (the first six;
// RING_NONE's row is no atom's).
struct RingAtom {
    int deg, perm;
    int nb[6];
};
__device__ __forceinline__ RingAtom ring_atom(const RingWs &W, int v)
{
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const auto r = (const __attribute__((address_space(1))) u32x4 *)(W.rec + (size_t)v * REC);
    const u32x4 a = r[0], b = r[1];
    RingAtom o;
    o.deg = (int)a[0];
    o.perm = (int)a[1];
    o.nb[0] = (int)(a[2] & J_MASK);
    o.nb[1] = (int)(a[3] & J_MASK);
    o.nb[2] = (int)(b[0] & J_MASK);
    o.nb[3] = (int)(b[1] & J_MASK);
    o.nb[4] = (int)(b[2] & J_MASK);
    o.nb[5] = (int)(b[3] & J_MASK);
    return o;
}
__device__ __forceinline__ uint32_t ring_entry(const RingWs &W, int v, int k)
{
    return gbl(W.rec)[(size_t)v * REC + REC_NB + k];
}
__device__ __forceinline__ int ring_nb(const RingWs &W, int v, int k) { return (int)(ring_entry(W, v, k) & J_MASK); }

// is w a neighbour of atom v (record A)?
__device__ __forceinline__ bool ring_has(const RingWs &W, int v, const RingAtom &A, int w)
{
    bool f = false;
#pragma unroll
    for (int k = 0; k < 6; k++) f = f || A.nb[k] == w;
    for (int k = 6; k < A.deg && !f; k++) f = ring_nb(W, v, k) == w;
    return f;
}
// does atom v (record A) have a neighbour in common with w (record B), or w itself?
__device__ __forceinline__ bool ring_near(const RingWs &W, int v, const RingAtom &A, int w, const RingAtom &B)
{
    bool f = false;
#pragma unroll
    for (int k = 0; k < 6; k++) f = f || (k < A.deg && (A.nb[k] == w || ring_has(W, w, B, A.nb[k])));
    for (int k = 6; k < A.deg && !f; k++) {
        const int t = ring_nb(W, v, k);
        f = t == w || ring_has(W, w, B, t);
    }
    return f;
}
// the bond of v that leads to w (they are bonded)
__device__ __forceinline__ int ring_bond_to(const RingWs &W, int v, int w)
{
    int k = 0;
    while (k < RING_DEG - 1 && ring_nb(W, v, k) != w) k++;
    return k;
}

// a path of fewer than d bonds (2 <= d <= 4) from a to b?
__device__ bool ring_shortcut(const RingWs &W, int a, int b, int d)
{
    const RingAtom A = ring_atom(W, a);
    if (ring_has(W, a, A, b)) return true;
    if (d <= 2) return false;
    const RingAtom B = ring_atom(W, b);
    if (ring_near(W, a, A, b, B)) return true;                     // a - c - b
    if (d <= 3) return false;
    for (int k = 0; k < A.deg; k++) {                              // a - c - e - b
        const int cv = ring_nb(W, a, k);
        const RingAtom C = ring_atom(W, cv);
        for (int m = 0; m < C.deg; m++) {
            const int e = ring_nb(W, cv, m);
            if (e != a && ring_has(W, b, B, e)) return true;
        }
    }
    return false;
}

// Orientation (degrees in [0, 60)) and |cos| of the tilt of the 6-ring whose
// vertices, unwrapped along its bonds, are p[0..5].
__device__ double ring_orientation(const R3<double> *p, const RingCfg &c, double &cos_tilt)
{
    double cx = 0, cy = 0, cz = 0;
    for (int k = 0; k < 6; k++) {
        cx += p[k].x;
        cy += p[k].y;
        cz += p[k].z;
    }
    cx /= 6.0;
    cy /= 6.0;
    cz /= 6.0;
    double nx = 0, ny = 0, nz = 0;
    for (int k = 0; k < 6; k++) {
        const int l = (k + 1) % 6;
        const double ax = p[k].x - cx, ay = p[k].y - cy, az = p[k].z - cz;
        const double bx = p[l].x - cx, by = p[l].y - cy, bz = p[l].z - cz;
        nx += ay * bz - az * by;
        ny += az * bx - ax * bz;
        nz += ax * by - ay * bx;
    }
    cos_tilt = ::fabs(nx * c.n[0] + ny * c.n[1] + nz * c.n[2]) / ::sqrt(nx * nx + ny * ny + nz * nz);
    double zr = 0.0, zi = 0.0;
    for (int k = 0; k < 3; k++) {
        const double dx = p[k + 3].x - p[k].x, dy = p[k + 3].y - p[k].y, dz = p[k + 3].z - p[k].z;
        const double th = ::atan2(dx * c.w[0] + dy * c.w[1] + dz * c.w[2], dx * c.u[0] + dy * c.u[1] + dz * c.u[2]);
        double sn, cs;
        ::sincos(6.0 * th, &sn, &cs);
        zr += cs;
        zi += sn;
    }
    double ang = ::atan2(zi, zr) * (180.0 / M_PI) / 6.0;
    if (ang < 0.0) ang += 60.0;
    return ang;
}

// Cycles found by the search wait in LDS (column i of path: the vertices in
// ring order, second below the last, RING_CAND of them and one column per
// thread for those that find no room), so that the whole test runs with
// every lane on one.
constexpr int RING_CAND = 512, RING_COLS = RING_CAND + TILE;

// Cycle tx of path, L atoms: the whole test, then counts, marks, orientation
// and the list.
__device__ __noinline__ void ring_emit(const Seg &S, const RingWs &W, const RingCfg &c,
                                       const int (*path)[RING_COLS], int tx, int L, unsigned *count, unsigned *hist)
{
    for (int a = 0; a < L; a++)
        for (int b = a + 2; b < L; b++) {
            const int d = min(b - a, L - (b - a));
            if (d >= 2 && ring_shortcut(W, path[a][tx], path[b][tx], d)) return;
        }
    atomicAdd(&count[L], 1u);
    R3<double> p[6];
    p[0] = {0.0, 0.0, 0.0};
    for (int m = 0; m < L; m++) {
        const int v = path[m][tx], w = path[m + 1 < L ? m + 1 : 0][tx], k = ring_bond_to(W, v, w);
        atomicOr(&W.mark[v], 1u << k);
    }
    double ang = -1.0;
    if (L == 6) {
#pragma unroll
        for (int m = 0; m < 5; m++) {
            const int v = path[m][tx], w = path[m + 1][tx];
            const uint32_t ent = ring_entry(W, v, ring_bond_to(W, v, w));
            const double4 lv = ld4<double>(S.xs64, v), lw = ld4<double>(S.xs64, w);
            const R3<double> D = code_offset(S, (int)(ent >> CODE_SHIFT));
            p[m + 1] = {p[m].x + ((lw.x - lv.x) + D.x), p[m].y + ((lw.y - lv.y) + D.y), p[m].z + ((lw.z - lv.z) + D.z)};
        }
        double ct;
        ang = ring_orientation(p, c, ct);
        if (c.cos_tilt_min < -1.0 || ct >= c.cos_tilt_min) {
            int bin = (int)(ang / 60.0 * c.nbins);
            bin = bin < 0 ? 0 : (bin >= c.nbins ? c.nbins - 1 : bin);
            if (c.nbins <= RING_HB) atomicAdd(&hist[bin], 1u);
            else atomicAdd(&W.hist[bin], 1ull);
            atomicAdd(&count[RING_MAX + 1], 1u);
        }
    }
    if (W.list) {
        const unsigned long long slot = atomicAdd(&W.cnt[RC_LISTED], 1ull);
        if ((long long)slot < W.cap) {
            int32_t *o = W.list + (size_t)slot * 9;
            o[0] = L;
            for (int m = 0; m < RING_MAX; m++) o[1 + m] = m < L ? S.perm[path[m][tx]] : -1;
            if (W.orient) W.orient[slot] = ang;
        }
    }
}

// Work items: the pairs (a, b) of an atom's neighbours with larger user
// indices, a's below b's, numbered over the block's atoms (half of a sheet's
// atoms have none) and taken by its threads in chunks of at most RING_ITEMS.
constexpr int RING_ITEMS = 1024, RING_PAIRS = RING_DEG * (RING_DEG - 1) / 2;
__global__ void __launch_bounds__(TILE) k_rings(const Tile *tiles, Seg *segs, RingWs W, RingCfg c)
{
    const Tile T = my_tile(tiles);
    const Seg &S = segs[T.seg];
    constexpr int STEP = RING_ITEMS - RING_PAIRS + 1;
    __shared__ int path[RING_MAX][RING_COLS];
    __shared__ uint8_t size[RING_CAND];
    __shared__ int ncand;
    __shared__ uint16_t item[RING_ITEMS];      // row | a's bond | b's bond
    __shared__ uint8_t used[RING_ITEMS];
    __shared__ unsigned hist[RING_HB];
    __shared__ unsigned count[RING_MAX + 2];   // rings by size, histogram entries
    __shared__ int scan[4], total;
    const int tx = threadIdx.x;
    for (int k = tx; k < RING_HB; k += TILE) hist[k] = 0u;
    if (tx < RING_MAX + 2) count[tx] = 0u;
    int big = 0, pairs = 0;                    // bonds to larger user indices
    {
        const int s = T.row0 + tx;
        if (s < S.n) {
            const RingAtom A = ring_atom(W, s);
            for (int k = 0; k < A.deg; k++)
                if ((int)gbl(W.rec)[(size_t)ring_nb(W, s, k) * REC + 1] > A.perm) big |= 1 << k;
            const int m = __popc((unsigned)big);
            pairs = m * (m - 1) / 2;
        }
    }
    const int start = block_excl_scan(pairs, scan);
    if (tx == TILE - 1) total = start + pairs;
    __syncthreads();
    for (int c0 = 0; c0 < total; c0 += STEP) {
        for (int k = tx; k < RING_ITEMS; k += TILE) used[k] = 0;
        if (tx == 0) ncand = 0;
        __syncthreads();
        if (pairs > 0 && start >= c0 && start < c0 + STEP) {
            const int s = T.row0 + tx;
            int at = start - c0;
            for (int ka = 0; ka < RING_DEG; ka++) {
                if (!((big >> ka) & 1)) continue;
                for (int kb = ka + 1; kb < RING_DEG; kb++) {
                    if (!((big >> kb) & 1)) continue;
                    const int a = ring_nb(W, s, ka), b = ring_nb(W, s, kb);
                    const bool ab = gbl(W.rec)[(size_t)a * REC + 1] < gbl(W.rec)[(size_t)b * REC + 1];
                    item[at] = (uint16_t)(tx | (ab ? ka : kb) << 8 | (ab ? kb : ka) << 12);
                    used[at] = 1;
                    at++;
                }
            }
        }
        __syncthreads();
        const int len = min(RING_ITEMS, total - c0);
        for (int i = tx; i < len; i += TILE) {
            if (!used[i]) continue;
            const int s = T.row0 + (item[i] & 255);
            const RingAtom A0 = ring_atom(W, s);
            const int u0 = A0.perm;
            const int a = ring_nb(W, s, (item[i] >> 8) & 15), b = ring_nb(W, s, item[i] >> 12);
            const RingAtom A = ring_atom(W, a), B = ring_atom(W, b);
            auto found = [&](int L, int v2, int v3, int v4, int v5, int v6, int v7) {
                int at = atomicAdd(&ncand, 1);
                const bool room = at < RING_CAND;
                if (!room) at = RING_CAND + tx;
                path[0][at] = s;
                path[1][at] = a;
                path[2][at] = v2;
                path[3][at] = v3;
                path[4][at] = v4;
                path[5][at] = v5;
                path[6][at] = v6;
                path[7][at] = v7;
                if (room) size[at] = (uint8_t)L;
                else ring_emit(S, W, c, path, at, L, count, hist);
            };
            if (ring_has(W, a, A, b)) {
                found(3, b, 0, 0, 0, 0, 0);
                continue;                        // (a and b at distance 2 in any longer ring)
            }
            if (c.max_size < 4) continue;
            for (int ix = 0; ix < A.deg; ix++) {
                const int x = ring_nb(W, a, ix);
                if (x == s) continue;
                const RingAtom X = ring_atom(W, x);
                if (X.perm < u0 || ring_has(W, s, A0, x)) continue;
                if (ring_has(W, x, X, b)) {      // s a x b
                    found(4, x, b, 0, 0, 0, 0);
                    continue;
                }
                if (c.max_size < 5) continue;
                for (int iy = 0; iy < B.deg; iy++) {
                    const int y = ring_nb(W, b, iy);
                    if (y == s || y == x) continue;
                    const RingAtom Y = ring_atom(W, y);
                    if (Y.perm < u0 || ring_has(W, s, A0, y) || ring_has(W, y, Y, a)) continue;
                    if (ring_has(W, x, X, y)) {  // s a x y b
                        found(5, x, y, b, 0, 0, 0);
                        continue;
                    }
                    if (c.max_size < 6) continue;
                    for (int ip = 0; ip < X.deg; ip++) {
                        const int p = ring_nb(W, x, ip);
                        if (p == a) continue;
                        const RingAtom P = ring_atom(W, p);
                        // p lies three bonds from s, two from a (and, past a
                        // ring of six, two or more from b)
                        if (P.perm < u0 || p == b || ring_has(W, p, P, b) || ring_near(W, p, P, s, A0)) continue;
                        if (ring_has(W, p, P, y)) {   // s a x p y b
                            found(6, x, p, y, b, 0, 0);
                            continue;
                        }
                        if (c.max_size < 7) continue;
                        for (int iq = 0; iq < Y.deg; iq++) {
                            const int q = ring_nb(W, y, iq);
                            if (q == b || q == p || q == x) continue;
                            const RingAtom Qa = ring_atom(W, q);
                            if (Qa.perm < u0 || ring_has(W, q, Qa, a) || ring_has(W, q, Qa, x) ||
                                ring_near(W, q, Qa, s, A0))
                                continue;
                            if (ring_has(W, p, P, q)) {   // s a x p q y b
                                found(7, x, p, q, y, b, 0);
                                continue;
                            }
                            if (c.max_size < 8) continue;
                            for (int iz = 0; iz < P.deg; iz++) {
                                const int z = ring_nb(W, p, iz);
                                if (z == x || !ring_has(W, q, Qa, z)) continue;
                                const RingAtom Z = ring_atom(W, z);
                                if (Z.perm < u0) continue;
                                found(8, x, p, z, q, y, b);
                            }
                        }
                    }
                }
            }
        }
        __syncthreads();
        for (int i = tx; i < min(ncand, RING_CAND); i += TILE) ring_emit(S, W, c, path, i, size[i], count, hist);
        __syncthreads();
    }
    __syncthreads();
    // the block's counts
    if (tx <= RING_MAX && count[tx]) {
        atomicAdd(&W.cnt[tx], (unsigned long long)count[tx]);
        if (!W.list) atomicAdd(&W.cnt[RC_LISTED], (unsigned long long)count[tx]);
    }
    if (tx == RING_MAX + 1 && count[tx]) atomicAdd(&W.cnt[RC_HIST], (unsigned long long)count[tx]);
    if (c.nbins <= RING_HB)
        for (int k = tx; k < c.nbins; k += TILE)
            if (hist[k]) atomicAdd(&W.hist[k], (unsigned long long)hist[k]);
}

// bonds (each once) and the bonds on no ring
__global__ void __launch_bounds__(TILE) k_ring_chain(const Tile *tiles, Seg *segs, RingWs W)
{
    const Tile T = my_tile(tiles);
    const Seg &S = segs[T.seg];
    __shared__ unsigned tot[2];
    if (threadIdx.x < 2) tot[threadIdx.x] = 0u;
    __syncthreads();
    const int s = T.row0 + threadIdx.x;
    unsigned nb = 0, nc = 0;
    if (s < S.n) {
        const RingAtom A = ring_atom(W, s);
        const unsigned mark = W.mark[s];
        for (int k = 0; k < A.deg; k++) {
            const int t = ring_nb(W, s, k);
            if ((int)gbl(W.rec)[(size_t)t * REC + 1] < A.perm) continue;
            nb++;
            if (!((mark >> k) & 1u) && !((W.mark[t] >> ring_bond_to(W, t, s)) & 1u)) nc++;
        }
    }
    if (nb) atomicAdd(&tot[0], nb);
    if (nc) atomicAdd(&tot[1], nc);
    __syncthreads();
    if (threadIdx.x == 0) {
        if (tot[0]) atomicAdd(&W.cnt[RC_BONDS], (unsigned long long)tot[0]);
        if (tot[1]) atomicAdd(&W.cnt[RC_CHAIN], (unsigned long long)tot[1]);
    }
}

} // namespace ctbop
