// k_solve.h -- the charge solve of a small or middling system in one launch.
//
// The multi-launch solve (k_qeq.h) takes four dependent launches per
// iteration, each a few microseconds of launch gap and fill, and gives a row
// to a lane: at 20,000 atoms its product ran 79 blocks on 256 CUs and an
// iteration took 48 us for about 3 us of matrix data.  Here every block
// keeps sv_rows(LPR) rows for the whole solve: the rows' matrix entries, block
// inverses and solver vectors stay in registers, and an iteration exchanges
// only y = M r (each block stages the y of its rows' neighbours in LDS) and
// 14 partial sums.
//
// Blocks of one system exchange these through memory with loads and stores
// at agent scope (they go past the L2s, which are not coherent between
// XCDs), and a value is its own flag: a slot holds SV_EMPTY (a NaN pattern
// no result has) until its owner stores the value, so a reader loads until
// it is something else, and no counter, fence or second round trip is
// needed.  Slots are emptied again by their owner, y after the sums of the
// same iteration have been read (every block has then staged it; two
// buffers), sums one iteration later (three buffers).
//
// No block may wait forever: the blocks of one system are at most the CUs of
// the device and hold at most one CU each, later blocks of a launch are
// never waited for by earlier systems, the host lets no more solves of the
// process run at once than fit (solve_turn.h), and every wait is bounded
// (SV_WAIT); a wait that runs out (the device shared with other processes, or
// with kernels that long) marks the system (SegState::pabort), all its blocks leave, and the host takes
// the multi-launch path from the starting charges on.  A wait can run out in one
// block when the others have finished, charges, state and status written, so
// nothing that a solve leaves counts unless pabort is clear.
#pragma once
#include "ctbop_dev.h"
#include "k_qeq.h"

namespace ctbop {

constexpr int SV_T = 512;                   // threads per block
constexpr int SV_MAX_ATOMS = 127 * TILE;    // blocks of SV_T threads (the bitmap of all rows, a word per thread)
constexpr int SV_HALO = 6144;               // distinct neighbours a block stages at most
// Blocks of SV_TW threads keep 256 rows each.
constexpr int SV_TW = 1024;
constexpr int SV_MAX_ATOMS_W = 192 * TILE;
constexpr unsigned long long SV_EMPTY = ~0ull;
constexpr unsigned long long SV_NAN = 0x7ff8000000000000ull;
constexpr long long SV_WAIT = 1000000;      // ticks of the 100 MHz clock: 10 ms per wait
constexpr int SV_NSUM = 14;
constexpr int SV_SLOTS = SV_NSUM;           // and, in the first iteration, the slots that a product reads
constexpr int SV_MAX_BLOCKS = 256;          // blocks of one system
constexpr int SV_LINE = 16;                 // a block's sums: one 128-byte line,
constexpr int SV_REP = 4;                   // in as many copies, a quarter of the blocks reading each
constexpr int SV_MIN_WL = 8;                // list strides whose copy of the rows holds the lines

// rows of a block, LPR lanes each
constexpr int sv_rows(int lpr, int t = SV_T) { return t / lpr; }
// matrix entries of a row that each of its lanes keeps in registers (longer
// rows stream the rest)
template <typename R, int LPR, int OCC, int T = SV_T> constexpr int sv_regs()
{
    return LPR == 8 || (sizeof(R) == 8 && OCC == 4) ? 24 : sizeof(R) == 8 ? 32 : OCC == 4 ? (T == SV_T ? 40 : 32) : 48;
}

__device__ __forceinline__ void sv_put(__attribute__((address_space(1))) unsigned long long *p, double v)
{
    unsigned long long b = (unsigned long long)__double_as_longlong(v);
    if (b == SV_EMPTY) b = SV_NAN;
    __hip_atomic_store(p, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void sv_clear(__attribute__((address_space(1))) unsigned long long *p)
{
    __hip_atomic_store(p, SV_EMPTY, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long sv_get(const __attribute__((address_space(1))) unsigned long long *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Load a slot until its value is there; false when the wait ran out or
// another block of the system gave up.
__device__ __forceinline__ bool sv_wait(const __attribute__((address_space(1))) unsigned long long *p,
                                        unsigned long long &v, const int *pabort)
{
    if (v != SV_EMPTY) return true;
    const long long t0 = wall_clock64();
    for (int k = 0;; k++) {
        v = sv_get(p);
        if (v != SV_EMPTY) return true;
        __builtin_amdgcn_s_sleep(1);
        if ((k & 63) == 63) {
            if (__hip_atomic_load(pabort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return false;
            if (wall_clock64() - t0 > SV_WAIT) return false;
        }
    }
}

// half u & 1 of a packed pair of 16-bit numbers
__device__ __forceinline__ uint32_t half16(uint32_t w, int u) { return (u & 1) ? w >> 16 : w & 0xffffu; }

// block-uniform values read from memory, in scalar registers
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
template <typename T> __device__ __forceinline__ T *uni(T *p)
{
    const unsigned long long b = (unsigned long long)p;
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)b);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(b >> 32));
    return (T *)(((unsigned long long)hi << 32) | lo);
}

// Entry slots that a product of the block's rows reads, into tot[SV_SLOTS]: of
// every wave the groups of eight per lane of its longest row, and what longer
// rows than the registers hold stream.  All threads; n is zero before.
template <int E, int LPR>
__device__ __forceinline__ void sv_slot_count(int nch, int cnt, int lane, int wl, int *n, double *tot)
{
    if (wl == 0) atomicAdd(n, 64 * min(8 * nch, E));
    if (lane == 0 && cnt > E * LPR) atomicAdd(n, cnt - E * LPR);
    __syncthreads();
    if (threadIdx.x == 0) tot[SV_SLOTS] = (double)*n;
}

// sum over the LPR lanes of a row, in every lane (DPP moves within 16 lanes)
template <int LPR>
__device__ __forceinline__ double row_sum(double v)
{
    v = dpp_add<0xb1>(v);
    v = dpp_add<0x4e>(v);
    if (LPR >= 8) v = dpp_add<0x141>(v);
    if (LPR >= 16) v = dpp_add<0x140>(v);
    return v;
}

// The block's place: rows row0 .. row0 + RB - 1 of the segment of tile
// blockIdx / SUB (SUB = TILE / RB blocks per tile), or none (row0 < 0).
template <int RB>
__device__ __forceinline__ int sv_row0(const Tile *tiles, const Seg *segs, int &seg)
{
    constexpr int SUB = TILE / RB;
    const Tile T = tiles[blockIdx.x / SUB];
    const int r = T.row0 + (int)(blockIdx.x % SUB) * RB;
    seg = uni(T.seg);
    return uni(r < segs[T.seg].n ? r : -1);
}

// scratch of the solve in arrays that only the multi-launch path uses: the
// y buffers are S.y and S.hz, the sums the head of S.H (three buffers of
// SV_REP lines per block), the block's halo list the head of its rows in
// S.hsidx, with its length in the last word of them
__device__ __forceinline__ __attribute__((address_space(1))) unsigned long long *sv_slots(double *p)
{
    return (__attribute__((address_space(1))) unsigned long long *)p;
}

// empty the exchange slots of a row (before a solve)
__device__ __forceinline__ void sv_clear_row(const Seg &S, int s)
{
    reinterpret_cast<unsigned long long *>(S.y)[s] = SV_EMPTY;
    reinterpret_cast<unsigned long long *>(S.hz)[s] = SV_EMPTY;
}

// The sums of a block, loc[0 .. 15], into its line of a buffer, by one wave:
// one 128-byte store per copy.  (A slot per sum and block, [sum][block],
// made 14 narrow stores into lines that 16 blocks share and all blocks read:
// 20,000 atoms, 8000 cycles from the first store to the last sum.)
__device__ __forceinline__ __attribute__((address_space(1))) unsigned long long *
sv_line(__attribute__((address_space(1))) unsigned long long *slots, int buf, int nblk, int blk, int wl)
{
    static_assert(SV_REP * SV_LINE == 64, "a lane per word");
    return slots + (unsigned)(((buf * SV_REP + (wl >> 4)) * nblk + blk) * SV_LINE + (wl & 15));
}

// The waves' shares of every block's sums into red (wave w takes blocks 4 w
// .. 4 w + 3 of every 4 NW); false when a wait ran out.
template <int NW>
__device__ __forceinline__ bool sv_collect(__attribute__((address_space(1))) unsigned long long *slots, int buf, int nblk,
                                           int blk, double (*red)[SV_LINE], int wv, int wl, const int *pabort)
{
    constexpr int PB = SV_MAX_BLOCKS / (4 * NW);
    const auto line = slots + (unsigned)((buf * SV_REP + (blk & (SV_REP - 1))) * nblk * SV_LINE + (wl & 15));
    unsigned long long x[PB];
#pragma unroll
    for (int i = 0; i < PB; i++)
        if ((i * NW + wv) * 4 < nblk)
            x[i] = sv_get(line + (unsigned)(min((i * NW + wv) * 4 + (wl >> 4), nblk - 1) * SV_LINE));
    bool ok = true;
    double t = 0.0;
#pragma unroll
    for (int i = 0; i < PB; i++)
        if ((i * NW + wv) * 4 < nblk) {
            const int b = (i * NW + wv) * 4 + (wl >> 4);
            ok = ok && sv_wait(line + (unsigned)(min(b, nblk - 1) * SV_LINE), x[i], pabort);
            t += b < nblk ? __longlong_as_double((long long)x[i]) : 0.0;
        }
    t += __shfl_xor(t, 16, 64);
    t += __shfl_xor(t, 32, 64);
    if (wl < SV_LINE) red[wv][wl] = t;
    return ok;
}

// sum wl & 15 of the system, from the waves' shares (one block: its own)
template <int NW>
__device__ __forceinline__ double sv_total(const double *loc, const double (*red)[SV_LINE], int nblk, int wl)
{
    if (nblk == 1) return loc[wl & 15];
    double t = red[0][wl & 15];
#pragma unroll
    for (int w = 1; w < NW; w++) t += red[w][wl & 15];
    return t;
}
__device__ __forceinline__ double sv_lane(double v, int k)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), k),
                            __builtin_amdgcn_readlane(__double2loint(v), k));
}

// Before the multi-launch solve of a system whose one-launch solve gave up: the
// state and the status of a part of its blocks that may have finished.
__global__ void k_solve_retry(const int *seg_ids, Seg *segs)
{
    SegState *st = segs[seg_ids[blockIdx.x]].sst;
    st->done = 0;
    st->iters = 0;
    st->pabort = 0;
    st->status &= ~(ST_NOCONV | ST_NOT_PD);
}

// What the solve needs of the assembled rows: the block's halo (the distinct
// rows its entries name, ascending), each entry's position in it (hs16, row-
// major like hidx), the inverses of the BK x BK diagonal blocks (as k_hslice
// makes them) with their row sums, and the sums of the first shift.  Also
// empties the exchange slots.  A block of more than `most` neighbours (SV_HALO
// at most) sends the system to the multi-launch solve.  Bound by latency (two passes over the rows, a
// scan, 16 elimination steps).
template <int LPR, typename R, int T>
__global__ void __launch_bounds__(T) k_solve_prep(const Tile *tiles, Seg *segs, int most)
{
    constexpr int RB = sv_rows(LPR, T), EPT = BK / LPR;
    static_assert(LPR == 4 || LPR == 8 || LPR == 16, "a row's lanes share a 16-lane DPP row");
    int seg;
    const int row0 = sv_row0<RB>(tiles, segs, seg);
    if (row0 < 0) return;
    const Seg &S = segs[seg];
    __shared__ unsigned long long bm[T];
    __shared__ uint16_t pre[T];
    __shared__ unsigned long long A64[RB * BK];
    __shared__ float A[RB][BK + 1];
    __shared__ int wsum[T / 64];
    __shared__ double lds[T / 64 * 3];
    const int tid = threadIdx.x, rl = tid / LPR, lane = tid % LPR, row = row0 + rl;
    const int n = S.n, Wl = S.Wl;
    const bool live = row < n;
    const auto hcnt = gbl(S.hcnt);
    const int cnt = live ? hcnt[row] : 0;
    const auto ent = gbl(S.hidx + (size_t)row * Wl);
    const auto val = gbl(reinterpret_cast<const R *>(S.Hr) + (size_t)row * Wl);
    for (int w = tid; w < T; w += T) bm[w] = 0ull;
    for (int w = tid; w < RB * BK; w += T) A64[w] = 0ull;
    __syncthreads();
    // Entries of the row's own block are added as 2^-40 fixed point: exact
    // in any order (an atom and several images of a neighbour in a small
    // cell), and finer than the FP32 inversion needs
    // (eight entries of a lane in flight; the indices of the row's first 192
    // stay in registers for the positions below: ten MD steps of 36,864 atoms
    // 8.43 ms reading them again, 8.00; 32 removal energies 9.97, 9.50)
    constexpr int U = 8, NK = 192 / LPR;
    int kept[NK];
    auto mark = [&](int j, R v) {
        // (most neighbours are marked already, and marks of one word wait for each other)
        const unsigned long long bit = 1ull << (j & 63);
        if (!(bm[j >> 6] & bit)) atomicOr(&bm[j >> 6], bit);
        if ((j & ~(BK - 1)) == (row & ~(BK - 1)))
            atomicAdd(&A64[rl * BK + (j & (BK - 1))], (unsigned long long)(long long)((double)v * 1099511627776.0));
    };
#pragma unroll
    for (int k0 = 0; k0 < NK; k0 += U) {
        const int e0 = lane + k0 * LPR;
        if (e0 >= cnt) break;
        R v[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int e = min(e0 + u * LPR, cnt - 1);
            kept[k0 + u] = (int)(ent[e] & J_MASK);
            v[u] = val[e];
        }
#pragma unroll
        for (int u = 0; u < U; u++)
            if (e0 + u * LPR < cnt) mark(kept[k0 + u], v[u]);
    }
    for (int e0 = lane + NK * LPR; e0 < cnt; e0 += U * LPR) {
        int j[U];
        R v[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int e = min(e0 + u * LPR, cnt - 1);
            j[u] = (int)(ent[e] & J_MASK);
            v[u] = val[e];
        }
#pragma unroll
        for (int u = 0; u < U; u++)
            if (e0 + u * LPR < cnt) mark(j[u], v[u]);
    }
    __syncthreads();
    // positions: set bits before each word (threads 0 .. T-1, one word each)
    const unsigned long long mine = bm[tid];
    const int c = __popcll(mine);
    int inc = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(inc, o, 64);
        if ((tid & 63) >= o) inc += t;
    }
    if ((tid & 63) == 63) wsum[tid >> 6] = inc;
    __syncthreads();
    int before = inc - c, total = 0;
    for (int w = 0; w < T / 64; w++) {
        if (w < (tid >> 6)) before += wsum[w];
        total += wsum[w];
    }
    pre[tid] = (uint16_t)before;
    uint32_t *region = S.hsidx + (size_t)row0 * Wl;
    uint16_t *list = reinterpret_cast<uint16_t *>(region);
    {
        unsigned long long b = mine;
        int at = before;
        while (b) {
            const int bit = __ffsll((long long)b) - 1;
            list[at++] = (uint16_t)(64 * tid + bit);
            b &= b - 1;
        }
    }
    if (tid == 0) {
        region[(size_t)RB * Wl - 1] = (uint32_t)total;
        if (total > most) atomicOr(&S.sst->pabort, PA_CROWDED);   // (before the solve has changed anything)
    }
    // the FP32 block row, J on the diagonal; identity rows past n
    {
        const int i = row & (BK - 1);
#pragma unroll
        for (int u = 0; u < EPT; u++) {
            const int t = lane * EPT + u;
            float a = (float)((double)(long long)A64[rl * BK + t] * (1.0 / 1099511627776.0));
            if (t == i) a = live ? a + (float)S.jd[row] : 1.0f;
            A[rl][t] = a;
        }
    }
    __syncthreads();
    const auto pos = gblw(S.hs16 + (size_t)row * Wl);
    auto place = [&](int j) {
        return (uint16_t)(pre[j >> 6] + __popcll(bm[j >> 6] & ((1ull << (j & 63)) - 1ull)));
    };
#pragma unroll
    for (int k = 0; k < NK; k++)
        if (lane + k * LPR < cnt) pos[lane + k * LPR] = place(kept[k]);
    for (int e0 = lane + NK * LPR; e0 < cnt; e0 += U * LPR) {
        int j[U];
#pragma unroll
        for (int u = 0; u < U; u++) j[u] = (int)(ent[min(e0 + u * LPR, cnt - 1)] & J_MASK);
#pragma unroll
        for (int u = 0; u < U; u++)
            if (e0 + u * LPR < cnt) pos[e0 + u * LPR] = place(j[u]);
    }
    // Gauss-Jordan, in place: a row's lanes hold EPT of its columns
    const int b0 = rl & ~(BK - 1), i = rl & (BK - 1);
    for (int k = 0; k < BK; k++) {
        const float piv = 1.0f / A[b0 + k][k];
        const float f = A[rl][k] * piv;
        float out[EPT];
#pragma unroll
        for (int u = 0; u < EPT; u++) {
            const int t = lane * EPT + u;
            const float rk = A[b0 + k][t], own = A[rl][t];
            out[u] = i == k ? (t == k ? piv : rk * piv) : (t == k ? -f : own - f * rk);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < EPT; u++) A[rl][lane * EPT + u] = out[u];
        __syncthreads();
    }
    double m1 = 0.0;
    const auto bo = gblw(S.binv + (size_t)row * BK);
#pragma unroll
    for (int u = 0; u < EPT; u++) {
        const int t = lane * EPT + u;
        const _Float16 b = (_Float16)(0.5f * (A[rl][t] + A[b0 + t][i]));
        bo[t] = b;
        m1 += (double)(float)b;
    }
    m1 = row_sum<LPR>(m1);
    if (lane == 0) {
        S.m1[row] = live ? m1 : 0.0;
        sv_clear_row(S, row);
    }
    if (tid < 3 * 64) *sv_line(sv_slots((double *)S.H), tid / 64, (n + RB - 1) / RB, row0 / RB, tid % 64) = SV_EMPTY;
    // partial sums of the block: r m1, m1 and the entries
    double v[3] = {0.0, 0.0, 0.0};
    if (live && lane == 0) {
        v[0] = S.r[row] * m1;
        v[1] = m1;
        v[2] = (double)cnt;
    }
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const double s = wave_sum(v[k]);
        if ((tid & 63) == 0) lds[(tid >> 6) * 3 + k] = s;
    }
    __syncthreads();
    if (tid < 3) {
        double s = 0.0;
        for (int w = 0; w < T / 64; w++) s += lds[w * 3 + tid];
        S.part[(size_t)(row0 / RB) * 3 + tid] = s;
    }
}

// Tolerance of a solve; relative: times the starting residual (the adjoint,
// whose source has the caller's scale).  way, on request alone: the solve gives
// up in its first iteration (1), or its last block does at the end, when the
// others have finished (2).
struct SolveCtl {
    double tol;
    int maxit;
    int relative;
    int way;
};

// The whole projected PCG of one system (the single-reduction form of
// k_cg1_update, k_spmv and k_cg1_fin, whose scalar step it shares), blocks
// of RB rows.  An iteration is bound by its two exchanges (a round trip past
// the L2s each, with the wait for the slowest block) and the gathers from
// LDS: at 20,000 atoms in cycles ~1100 y = M r, ~3700 staging y, ~3900
// products (352 wave gathers), ~1200 block sums, ~4000 their exchange, ~2600
// the scalar step.
// 20,000 atoms: an iteration 48 -> 8.5 us, a cold solve 2.2 -> 0.41 ms; 512
// atoms 26 -> 5.2 us; 36,864 atoms (SV_TW) 31 in two launches -> 11.5 us.
// OCC 4 keeps two blocks on a CU in half the registers,
// for launches with more blocks than CUs.
template <int LPR, typename R, int OCC, int T>
__global__ void __launch_bounds__(T, OCC) k_solve(const Tile *tiles, Seg *segs, SolveCtl ctl)
{
    constexpr int RB = sv_rows(LPR, T), EPT = BK / LPR, E = sv_regs<R, LPR, OCC, T>();
    constexpr int NW = T / 64, NH = (SV_NSUM + NW - 1) / NW;
    static_assert(E % 8 == 0, "entries are loaded and used by eight");
    int seg;
    const int row0 = sv_row0<RB>(tiles, segs, seg);
    if (row0 < 0) return;
    const Seg &S = segs[seg];
    if (uni(S.sst->pabort)) return;
    __shared__ double hp[SV_HALO];
    __shared__ uint16_t hl[SV_HALO];
    // the rows' r, y, s, q, m1 and H y, ones, p and J (a row's first lane
    // takes its vector steps; the registers are the matrix's)
    __shared__ double va[9][RB];
    double *const vr = va[0], *const vy = va[1], *const vs = va[2], *const vq = va[3], *const vh = va[5],
           *const vp = va[7], *const vj = va[8];
    __shared__ double tot[SV_LINE], red[NW][SV_LINE];   // the block's sums, the waves' shares of all blocks'
    __shared__ SegState st;
    __shared__ int sab, nslot;
    const int tid = threadIdx.x, rl = tid / LPR, lane = tid % LPR, row = row0 + rl, wv = uni(tid >> 6), wl = tid & 63;
    const int n = uni(S.n), Wl = uni(S.Wl), blk = row0 / RB, nblk = (n + RB - 1) / RB;
    const bool live = row < n;
    const double Q = S.Q;
    SegState *const sst = uni(S.sst);
    int *const pabort = &sst->pabort;
    const auto slots_y0 = sv_slots(uni(S.y)), slots_y1 = sv_slots(uni(S.hz)), slots_p = sv_slots(uni((double *)S.H));
    // the block's halo rows
    const uint32_t *region = S.hsidx + (size_t)row0 * Wl;
    const int nh = uni((int)region[(size_t)RB * Wl - 1]);
    const auto list = gbl(reinterpret_cast<const uint16_t *>(region));
    for (int k = tid; k < nh; k += T) hl[k] = list[k];
    // the row's entries
    const int cnt = live ? gbl(S.hcnt)[row] : 0;
    const auto vals = gbl(uni(reinterpret_cast<const R *>(S.Hr)) + (size_t)row0 * Wl);
    const auto poss = gbl(uni(S.hs16) + (size_t)row0 * Wl);
    const unsigned rowe = (unsigned)(rl * Wl);   // the row's first entry
    R hv[E];
    uint32_t hj[E / 2];
    // (eight at a time: all loads of a group in flight, no more registers)
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
    // chunks of eight entries per lane that this wave's rows need
    int mxc = cnt;
#pragma unroll
    for (int o = 32; o >= LPR; o >>= 1) mxc = max(mxc, __shfl_xor(mxc, o, 64));
    const int nch = uni((mxc + 8 * LPR - 1) / (8 * LPR));
    float bv[EPT];
#pragma unroll
    for (int u = 0; u < EPT; u++) bv[u] = (float)gbl(S.binv + (size_t)row * BK)[lane * EPT + u];
    static_assert(sizeof(SegState) % 4 == 0 && sizeof(SegState) / 4 <= T, "a word per thread");
    if (tid < (int)(sizeof(SegState) / 4)) reinterpret_cast<int *>(&st)[tid] = reinterpret_cast<const int *>(sst)[tid];
    if (tid == 0) {
        sab = ctl.way & 1;
        nslot = 0;
    }
    if (tid < SV_LINE) tot[tid] = 0.0;
    if (lane == 0) {
        vr[rl] = live ? S.r[row] : 0.0;
        vq[rl] = live ? S.q[row] : 0.0;
        va[4][rl] = live ? S.m1[row] : 0.0;
        vj[rl] = live ? S.jd[row] : 0.0;
        va[6][rl] = 1.0;
        vy[rl] = vs[rl] = vh[rl] = vp[rl] = 0.0;
    }
    // the first shift, from the sums of k_solve_prep
    if (wv == 0) {
        double v[3] = {0.0, 0.0, 0.0};
        const auto part = gbl(S.part);
        for (int b = wl; b < nblk; b += 64) {
#pragma unroll
            for (int k = 0; k < 3; k++) v[k] += part[(size_t)b * 3 + k];
        }
#pragma unroll
        for (int k = 0; k < 3; k++) {
            v[k] = wave_sum(v[k]);
            if (wl == 0) tot[k] = v[k];
        }
    }
    __syncthreads();
    if (tid == 0) {
        st.sdinv = tot[1];
        st.w = tot[0] / tot[1];
        st.nnz_coul = tot[2];
        st.nnz_wide = 0.0;
        st.nnz_halo = tot[2];
        st.mshift = st.mu_prev - st.w;
        st.iters = 0;
        st.qshift = 0.0;
        // (a relative tolerance needs the shift that rounding left removed
        // before the first step too: the source may be constant but for it)
        st.cg_first = ctl.relative ? 2 : 1;
        st.cg_last = 0;
        st.rho = st.alpha = st.beta = st.m1s = 0.0;
    }
    sv_slot_count<E, LPR>(nch, cnt, lane, wl, &nslot, tot);
    __syncthreads();
    if (lane == 0 && live) vr[rl] -= st.w;
    const double inv_n = 1.0 / n, inv_sd = 1.0 / st.sdinv;
    double tol = ctl.tol;
    // sum w is of the products of two row arrays (0..7 of the last update: y,
    // r y, r, r r, q, r s, s s, s; 8..13 of the product: y h, m1 h, r h, h h,
    // s h, h), three bits each
    constexpr unsigned long long FA = 01ull | 01ull << 3 | 00ull << 6 | 00ull << 9 | 03ull << 12 | 02ull << 15 |
                                      02ull << 18 | 02ull << 21 | 01ull << 24 | 04ull << 27 | 00ull << 30 |
                                      05ull << 33 | 02ull << 36 | 05ull << 39;
    constexpr unsigned long long FB = 06ull | 00ull << 3 | 06ull << 6 | 00ull << 9 | 06ull << 12 | 00ull << 15 |
                                      02ull << 18 | 06ull << 21 | 05ull << 24 | 05ull << 27 | 05ull << 30 |
                                      05ull << 33 | 05ull << 36 | 06ull << 39;
    for (int it = 0;; it++) {
        const bool last = st.cg_last != 0;
        // the values kept in registers stay as they are loaded: nothing
        // derived from them (addresses, FP64 copies) is kept across iterations
#pragma unroll
        for (int k = 0; k < E; k++) asm volatile("" : "+v"(hv[k]));
#pragma unroll
        for (int k = 0; k < E / 2; k++) asm volatile("" : "+v"(hj[k]));
        // y = M r: the row's lanes share the block row
        __syncthreads();
        if (!last) {
            double y = 0.0;
#pragma unroll
            for (int u = 0; u < EPT; u++) y += (double)bv[u] * vr[(rl & ~(BK - 1)) + lane * EPT + u];
            y = row_sum<LPR>(y);
            const auto ys = (it & 1) ? slots_y1 : slots_y0;
            if (lane == 0) {
                sv_put(ys + row, y);
                vy[rl] = y;
            }
            // stage the halo, four loads in flight per thread (past its end
            // the last one again)
            bool ok = true;
            for (int k0 = tid; k0 < nh + tid && ok; k0 += 4 * T) {
                int k[4];
                unsigned long long v[4];
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    k[u] = min(k0 + u * T, nh - 1);
                    v[u] = sv_get(ys + (unsigned)hl[k[u]]);
                }
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    ok = ok && sv_wait(ys + (unsigned)hl[k[u]], v[u], pabort);
                    hp[k[u]] = __longlong_as_double((long long)v[u]);
                }
            }
            if (!ok) sab = 1;
            __syncthreads();
            if (sab) break;
            // hz = H y
            double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int k = 0; k < E; k += 8)
                if (k < 8 * nch) {
#pragma unroll
                    for (int u = 0; u < 8; u++)
                        acc[u & 3] += (double)hv[k + u] * hp[half16(hj[(k + u) / 2], u)];
                    __builtin_amdgcn_sched_barrier(0);
                }
            // the rest of longer rows, in the same order
            for (int e0 = E * LPR + lane; e0 < cnt; e0 += 4 * LPR) {
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const int e = e0 + u * LPR;
                    if (e < cnt) acc[u] += (double)vals[rowe + (unsigned)e] * hp[poss[rowe + (unsigned)e]];
                }
            }
            const double a = row_sum<LPR>((acc[0] + acc[1]) + (acc[2] + acc[3]));
            if (lane == 0) vh[rl] = vj[rl] * vy[rl] + a;   // (rows past n: 0)
        }
        // (emptied slots are in place before this block's sums say so)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        // sums wv and wv + NW: the block's share, then every block's
        double v[NH];
#pragma unroll
        for (int h = 0; h < NH; h++) {
            const int w = min(wv + h * NW, SV_NSUM - 1);
            const double *a = va[(FA >> (3 * w)) & 7], *b = va[(FB >> (3 * w)) & 7];
            v[h] = 0.0;
#pragma unroll
            for (int k = 0; k < RB; k += 64) v[h] += a[k + wl] * b[k + wl];
        }
#pragma unroll
        for (int h = 0; h < NH; h++) {
            v[h] = wave_sum(v[h]);
            if (wl == 0 && wv + h * NW < SV_NSUM) tot[wv + h * NW] = v[h];
        }
        if (nblk > 1) {
            __syncthreads();
            if (wv == 0) sv_put(sv_line(slots_p, it % 3, nblk, blk, wl), tot[wl & 15]);
            if (!sv_collect<NW>(slots_p, it % 3, nblk, blk, red, wv, wl, pabort)) sab = 1;
        }
        __syncthreads();
        if (sab) break;
        if (wv == 0) {
            // the scalar step, on the sums in scalar registers
            const double mine = sv_total<NW>(tot, red, nblk, wl);
            double t[P_CG1];
#pragma unroll
            for (int k = 0; k < P_CG1; k++) t[k] = sv_lane(mine, k);
            if (wl == SV_SLOTS) st.nnz_slots = mine;
            if (wl == 0 && st.cg_first == 2) {
                st.w = t[P_UPD + 0] * inv_sd;
                st.mshift -= st.w;
                st.cg_first = 1;
            } else if (wl == 0) {
                if (ctl.relative && st.cg_first) {
                    const double rr = t[P_UPD + 3] - t[P_UPD + 2] * t[P_UPD + 2] * inv_n;
                    tol = fmax(ctl.tol * sqrt(fmax(rr * inv_n, 0.0)), 1e-300);
                }
                st.status |= cg1_step(st, inv_n, inv_sd, Q, t, tol, ctl.maxit);
            }
        }
        // empty this iteration's y and the previous one's sums
        if (!last && lane == 0) sv_clear(((it & 1) ? slots_y1 : slots_y0) + row);
        if (nblk > 1 && wv == 1) sv_clear(sv_line(slots_p, (it + 2) % 3, nblk, blk, wl));
        __syncthreads();
        if (st.done) break;
        if (lane == 0 && live) {
            const double alpha = st.alpha, beta = st.beta, c = st.w;
            const double p = vy[rl] + beta * vp[rl], s = vh[rl] + beta * vs[rl];
            vp[rl] = p;
            vs[rl] = s;
            vq[rl] += alpha * p;
            vr[rl] = (vr[rl] - alpha * s) - c;
        }
    }
    if (sab || ((ctl.way & 2) && blk == nblk - 1)) {
        if (tid == 0) __hip_atomic_store(pabort, PA_WAIT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    if (lane == 0 && live) S.q[row] = vq[rl];
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
        o->cg_first = st.cg_first;
        o->cg_last = st.cg_last;
        o->rho = st.rho;
        o->alpha = st.alpha;
        o->beta = st.beta;
        o->m1s = st.m1s;
        o->res = st.res;
        o->res0 = st.res0;
        const int bad = st.status & (ST_NOCONV | ST_NOT_PD);
        if (bad) atomicOr(&o->status, bad);
        o->done = 1;
    }
}

} // namespace ctbop
