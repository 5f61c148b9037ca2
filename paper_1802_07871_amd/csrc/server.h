// server.h -- continuous-batching serving engine (host side), included by
// ctbop.hip after the single-system path.
//
// Every admitted request is a segment: one region of the caller's arena holds
// its inputs, outputs and the same per-system layout the single-system path
// uses, and one entry of a device table holds its descriptor.  A scheduler
// thread runs ticks on one stream:
//   1. admit pending requests in arrival order while slots and arena bytes
//      allow (a request that does not fit waits; retained systems are evicted
//      least recently used first), and send their inputs in one launch;
//   2. set-up kernels (bins, lists, bond pass, Coulomb assembly) over the new
//      segments' tiles, all in one launch per kernel;
//   3. the one-launch charge solve of the new segments that take it, then K
//      iterations over the tiles of the others, again one launch per kernel;
//      each segment stops on its own test;
//   4. force and energy kernels over the same tiles, gated per segment on
//      "solve finished, forces pending";
//   5. read the per-segment flags and, by one launch into pinned memory, the
//      finished results, copy these to the caller's host buffers and free (or
//      retain) their regions.
// Requests that arrive during a tick join at the next one, so work of
// requests of any size and phase overlaps on the device.  Each segment's
// arithmetic and reduction order do not depend on the other segments (but for a
// one-launch solve that gives up because work outside this process, or a
// kernel that holds the CUs for 10 ms, keeps its blocks waiting), so a
// result is bitwise the same alone and in the mix.
#pragma once
#include <chrono>
#include <condition_variable>
#include <deque>
#include <map>
#include <mutex>
#include <thread>

namespace {

double now_s()
{
    using namespace std::chrono;
    return duration<double>(steady_clock::now().time_since_epoch()).count();
}

struct SrvReq {
    long ticket;
    int n;
    std::vector<double> pos;
    std::vector<int32_t> types;
    double box[9];
    int pbc[3];
    double Q;
    long sys_id;
    std::vector<double> q0;         // starting charges (user order), or empty
    // or: the atoms of a system in device memory but one, with its charges as
    // the starting charges (removal energies); read when the request is admitted
    const double *x_dev = nullptr, *q_dev = nullptr;
    const int32_t *types_dev = nullptr;
    int skip = -1;
    double *E_out, *F_out, *q_out;
    double t_submit, t_admit;
};

enum SlotState { FREE = 0, ACTIVE = 1, RETAINED = 2 };

struct SrvSlot {
    int state = FREE;
    SrvReq req;
    size_t off = 0, bytes = 0;      // region in the arena
    Layout L;
    size_t io_off = 0;              // I/O arrays at the start of the region
    int phase = 0;                  // 0 = needs set-up, 1 = solving/finishing
    bool placed = false;            // placed since the last tick, its inputs not yet on the device
    bool fresh = false;             // in a new region
    bool many = false;              // its one-launch solve gave up: multi-launch solve
    int kind = 0;                   // of its solve, from its set-up on (solve_kind)
    long sys_id = -1;
    double last_use = 0;
    Sig sig;
};

} // namespace

namespace ctbop {

// An admitted request for k_admit, in pinned memory: its descriptor and where
// its inputs are (pinned or device memory; x null: copied by themselves;
// skip >= 0: those of a system of n + 1 atoms without atom skip).
struct SrvAdmit {
    Seg seg;
    const double *x, *q0;
    const int32_t *type;
    int slot, n, skip, fresh, warm;
};
// Where k_deliver puts the results of an active request (pinned memory or null).
struct SrvOut {
    double *F, *q;
    int slot, n;
};

// Inputs, descriptors and start states of the requests admitted to a tick, a
// column of blocks each, read across PCIe from pinned memory (or, for removal
// energies, from the full system's arrays on the device).  Bound by that link.
// A request took three to five copies and launches by itself: 48 requests of 8
// to 20,000 atoms 6.6 ms, 3.7 with this and k_deliver; 32 removal energies of
// 18,086 atoms 13.0 ms with inputs put together on the host, 10.7 with a
// launch per system that makes them here, 9.7 now.
__global__ void __launch_bounds__(TILE) k_admit(const SrvAdmit *adm, Seg *segs)
{
    const SrvAdmit &A = adm[blockIdx.x];
    const int tid = threadIdx.x, n = A.n, skip = A.skip, ns = skip >= 0 ? n + 1 : n;
    if (A.x) {
        const double *x = A.x, *q0 = A.q0;
        const int32_t *type = A.type;
        double *xo = const_cast<double *>(A.seg.x), *qo = A.seg.q_state;
        int32_t *to = const_cast<int32_t *>(A.seg.type);
        for (int i = blockIdx.y * TILE + tid; i < n; i += gridDim.y * TILE) {
            const int j = i + (skip >= 0 && i >= skip ? 1 : 0);
            const double x0 = x[j], x1 = x[(size_t)ns + j], x2 = x[2 * (size_t)ns + j], q = q0 ? q0[j] : 0.0;
            const int32_t t = type[j];
            xo[i] = x0;
            xo[(size_t)n + i] = x1;
            xo[2 * (size_t)n + i] = x2;
            to[i] = t;
            if (q0) qo[i] = q;
        }
    }
    if (blockIdx.y != 0) return;
    static_assert(sizeof(Seg) % 4 == 0 && sizeof(SegState) % 4 == 0, "copied as words");
    for (int w = tid; w < (int)(sizeof(Seg) / 4); w += TILE)
        reinterpret_cast<int *>(segs + A.slot)[w] = reinterpret_cast<const int *>(&A.seg)[w];
    SegState *st = A.seg.sst;
    if (A.fresh)
        for (int w = tid; w < (int)(sizeof(SegState) / 4); w += TILE) reinterpret_cast<int *>(st)[w] = 0;
    __syncthreads();
    if (tid == 0) st->warm = A.warm;
}

// Forces, charges and energies of the finished requests into pinned memory.
__global__ void __launch_bounds__(TILE) k_deliver(const SrvOut *out, const Seg *segs, double *E)
{
    const SrvOut &o = out[blockIdx.x];
    const Seg &S = segs[o.slot];
    if (!S.sst->forces_done) return;
    const int i0 = blockIdx.y * TILE + threadIdx.x, step = gridDim.y * TILE, n = o.n;
    if (o.F) {
        double *F = o.F;
        for (int i = i0; i < 3 * n; i += step) F[i] = S.F[i];
    }
    if (o.q) {
        double *q = o.q;
        for (int i = i0; i < n; i += step) q[i] = S.q_out[i];
    }
    if (i0 == 0) E[blockIdx.x] = *S.E_out;
}

} // namespace ctbop

struct ctbop_server {
    ctbop_ctx *ctx = nullptr;
    char *arena = nullptr;
    size_t arena_bytes = 0;
    int max_slots = 0;
    int cg_per_tick = 8;
    int iters_hint = 0;      // solver iterations of the last finished request (tick thread only)
    int device = 0;
    hipStream_t stream = nullptr;
    // the covalent kernels of newly set-up systems run on a stream of the
    // server's own beside the assembly and the solve, joined before the
    // Coulomb forces (as the single-system path does)
    hipStream_t side = nullptr;
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    int turn_dev = -1;                // device of join_turn
    // device tables at the head of the arena
    Seg *dsegs = nullptr;
    Tile *dtiles_setup = nullptr, *dtiles_act = nullptr;
    int *dids_setup = nullptr, *dids_act = nullptr;
    int4 *dflags = nullptr;
    int max_tiles = 0;
    // host mirrors (pinned)
    Tile *htiles = nullptr;
    int *hids = nullptr;
    int4 *hflags = nullptr;
    double *hE = nullptr;             // after hflags, as the next two
    SrvAdmit *hadm = nullptr;
    SrvOut *hout = nullptr;
    // pinned room for the inputs, then the results, of a tick (tick thread
    // only); allocated with the server, so that a tick allocates nothing
    char *stage = nullptr;
    size_t stage_bytes = 0;
    // regions
    std::map<size_t, size_t> free_ranges;   // offset -> size
    std::vector<SrvSlot> slots;
    std::deque<SrvReq> pending;
    std::deque<ctbop_result> done;
    long next_ticket = 1;
    size_t max_pending = 1 << 20;
    // thread
    std::thread th;
    std::mutex mu;
    std::condition_variable cv;
    bool stop = false;
    int error = 0;
    std::string errmsg;
    // statistics
    long ticks = 0, admitted = 0, completed = 0;
    double busy_s = 0;
    size_t peak_bytes = 0, used_bytes = 0;
};

namespace {

size_t io_bytes(int n) { return align_up(8 * 3 * (size_t)n, 256) + align_up(4 * (size_t)n, 256) +
                                align_up(8 * 3 * (size_t)n, 256) + align_up(8 * (size_t)n, 256) + 256; }

bool range_alloc(ctbop_server *S, size_t bytes, size_t &off)
{
    for (auto it = S->free_ranges.begin(); it != S->free_ranges.end(); ++it) {
        if (it->second >= bytes) {
            off = it->first;
            size_t rest = it->second - bytes;
            S->free_ranges.erase(it);
            if (rest) S->free_ranges[off + bytes] = rest;
            S->used_bytes += bytes;
            S->peak_bytes = std::max(S->peak_bytes, S->used_bytes);
            return true;
        }
    }
    return false;
}

void range_free(ctbop_server *S, size_t off, size_t bytes)
{
    S->used_bytes -= bytes;
    auto it = S->free_ranges.emplace(off, bytes).first;
    auto nx = std::next(it);
    if (nx != S->free_ranges.end() && it->first + it->second == nx->first) {
        it->second += nx->second;
        S->free_ranges.erase(nx);
    }
    if (it != S->free_ranges.begin()) {
        auto pv = std::prev(it);
        if (pv->first + pv->second == it->first) {
            pv->second += it->second;
            S->free_ranges.erase(it);
        }
    }
}

Sig req_sig(const ctbop_ctx *ctx, const SrvReq &r, size_t bytes)
{
    Sig g;
    memset(&g, 0, sizeof g);
    g.n = r.n;
    memcpy(g.box, r.box, sizeof g.box);
    for (int a = 0; a < 3; a++) g.pbc[a] = r.pbc[a] ? 1 : 0;
    g.fp64 = ctx->opts.fp64;
    g.bytes = bytes;
    return g;
}

// place a request into a slot and its region (the next tick sends its
// descriptor and inputs).  Returns false if it does not fit right now.
int admit_one(ctbop_server *S, SrvReq &r, bool &placed)
{
    placed = false;
    ctbop_ctx *ctx = S->ctx;
    // a retained system with the same id and geometry keeps its lists and charges
    int reuse = -1, freeslot = -1;
    for (int k = 0; k < S->max_slots; k++) {
        SrvSlot &sl = S->slots[k];
        if (sl.state == RETAINED && r.sys_id >= 0 && sl.sys_id == r.sys_id) reuse = k;
        if (sl.state == FREE && freeslot < 0) freeslot = k;
    }
    Layout L;
    int rc = make_layout(ctx, r.n, r.box, r.pbc, nullptr, L);
    if (rc) return rc;
    const size_t iob = io_bytes(r.n);
    const size_t need = iob + L.bytes;
    Sig sg = req_sig(ctx, r, L.bytes);
    int k = -1;
    bool fresh = true;
    if (reuse >= 0 && S->slots[reuse].sig == sg) {
        k = reuse;
        fresh = false;
    } else {
        if (reuse >= 0) {                  // same id, new geometry: drop the old state
            range_free(S, S->slots[reuse].off, S->slots[reuse].bytes);
            S->slots[reuse].state = FREE;
            if (freeslot < 0) freeslot = reuse;
        }
        size_t off;
        while (!range_alloc(S, need, off)) {
            // evict the least recently used retained system, if any
            int lru = -1;
            for (int j = 0; j < S->max_slots; j++)
                if (S->slots[j].state == RETAINED && (lru < 0 || S->slots[j].last_use < S->slots[lru].last_use)) lru = j;
            if (lru < 0) return CTBOP_OK;  // wait for running requests to finish
            range_free(S, S->slots[lru].off, S->slots[lru].bytes);
            S->slots[lru].state = FREE;
            if (freeslot < 0) freeslot = lru;
        }
        if (freeslot < 0) {
            range_free(S, off, need);
            return CTBOP_OK;
        }
        k = freeslot;
        S->slots[k].off = off;
        S->slots[k].bytes = need;
    }
    SrvSlot &sl = S->slots[k];
    char *base = S->arena + sl.off;
    rc = make_layout(ctx, r.n, r.box, r.pbc, base + iob, sl.L);
    if (rc) return rc;
    sl.io_off = 0;
    sl.sig = sg;
    sl.sys_id = r.sys_id;
    sl.state = ACTIVE;
    sl.phase = 0;
    sl.many = false;
    sl.req = std::move(r);
    sl.req.t_admit = now_s();
    sl.last_use = sl.req.t_admit;
    sl.placed = true;
    sl.fresh = fresh;
    S->admitted++;
    placed = true;
    return CTBOP_OK;
}

// Device arrays of a slot's request.
struct SrvArrays {
    double *x;
    int32_t *type;
    double *F, *q, *E;
};
SrvArrays slot_arrays(const ctbop_server *S, const SrvSlot &sl)
{
    const size_t n = (size_t)sl.req.n;
    SrvArrays a;
    a.x = (double *)(S->arena + sl.off);
    a.type = (int32_t *)((char *)a.x + align_up(8 * 3 * n, 256));
    a.F = (double *)((char *)a.type + align_up(4 * n, 256));
    a.q = (double *)((char *)a.F + align_up(8 * 3 * n, 256));
    a.E = (double *)((char *)a.q + align_up(8 * n, 256));
    return a;
}

// Send the inputs and descriptors of the requests placed since the last tick,
// through the pinned room; inputs that do not fit it are copied by themselves.
int send_placed(ctbop_server *S, const std::vector<int> &act)
{
    hipStream_t st = S->stream;
    std::vector<int> fresh;
    for (int k : act)
        if (S->slots[k].placed) fresh.push_back(k);
    if (fresh.empty()) return CTBOP_OK;
    size_t at = 0;
    int tiles = 1, m = 0;
    for (int k : fresh) {
        SrvSlot &sl = S->slots[k];
        const size_t n = (size_t)sl.req.n;
        const SrvArrays a = slot_arrays(S, sl);
        SrvAdmit &A = S->hadm[m++];
        A.seg = sl.L.seg;
        A.seg.x = a.x;
        A.seg.type = a.type;
        A.seg.F = a.F;
        A.seg.q_out = a.q;
        A.seg.E_out = a.E;
        A.seg.Q = sl.req.Q;
        A.slot = k;
        A.n = sl.req.n;
        A.skip = sl.req.skip;
        A.fresh = sl.fresh ? 1 : 0;
        // starting charges given with the request replace the warm-start
        // state; a retained system otherwise starts from its last charges
        const bool q0 = !sl.req.q0.empty();
        A.warm = sl.fresh && !q0 && !sl.req.x_dev ? 0 : 1;
        A.x = sl.req.x_dev;
        A.type = sl.req.types_dev;
        A.q0 = sl.req.q_dev;
        const size_t b = align_up(28 * n, 8) + (q0 ? 8 * n : 0);
        if (!sl.req.x_dev && at + b <= S->stage_bytes) {
            char *p = S->stage + at;
            at += b;
            memcpy(p, sl.req.pos.data(), 24 * n);
            A.x = (const double *)p;
            p += 24 * n;
            if (q0) {
                memcpy(p, sl.req.q0.data(), 8 * n);
                A.q0 = (const double *)p;
                p += 8 * n;
            }
            memcpy(p, sl.req.types.data(), 4 * n);
            A.type = (const int32_t *)p;
        } else if (!sl.req.x_dev) {
            HIPCHK(hipMemcpyAsync(a.x, sl.req.pos.data(), 24 * n, hipMemcpyHostToDevice, st));
            HIPCHK(hipMemcpyAsync(a.type, sl.req.types.data(), 4 * n, hipMemcpyHostToDevice, st));
            if (q0) HIPCHK(hipMemcpyAsync(A.seg.q_state, sl.req.q0.data(), 8 * n, hipMemcpyHostToDevice, st));
        }
        if (A.x) tiles = std::max(tiles, sl.L.ntile);
        sl.placed = false;
    }
    hipLaunchKernelGGL(k_admit, dim3(m, std::min(tiles, 64)), dim3(TILE), 0, st, S->hadm, S->dsegs);
    HIPCHK(hipGetLastError());
    return CTBOP_OK;
}

// One tick: set up the newly admitted systems, run cg_iters solver
// iterations over every active system, then the (gated) force kernels and
// the harvest.  With poll set (nobody waiting for admission when the tick
// began) the iterations go in chunks, the first as long as the last finished
// request needed, then cg_check each, with a convergence check after each
// chunk: the tick goes on until an active system has converged (or the
// iteration limit), so that it is harvested at once, unless a request
// arrives, which ends it at the next check once cg_iters have run.  A lone
// request is then served in one tick, like a plain call.  Systems solved in one
// launch have converged by then: a tick that holds one does not poll, so that
// its result does not wait for a large system's solve.
template <typename R>
int server_tick(ctbop_server *S, const Params<R> &prm, int cg_iters, bool poll)
{
    ctbop_ctx *ctx = S->ctx;
    hipStream_t st = S->stream;
    // tables: set-up tiles/ids and active tiles/ids
    int nts = 0, nis = 0, nta = 0, nia = 0;
    std::vector<int> act;
    for (int k = 0; k < S->max_slots; k++) {
        SrvSlot &sl = S->slots[k];
        if (sl.state != ACTIVE) continue;
        act.push_back(k);
    }
    if (act.empty()) return CTBOP_OK;
    SolvePass pass;
    // the largest first: of a batch that fills the device more than once the
    // last systems to run are then the smallest
    std::stable_sort(act.begin(), act.end(), [&](int a, int b) { return S->slots[a].req.n > S->slots[b].req.n; });
    const int src = send_placed(S, act);
    if (src) return src;
    int total_tiles = 0;
    for (int k : act) total_tiles += S->slots[k].L.ntile;
    if (total_tiles > S->max_tiles) return fail(CTBOP_E_NOMEM, "server tile table too small");
    Tile *hts = S->htiles, *hta = S->htiles + S->max_tiles;
    int *his = S->hids, *hia = S->hids + S->max_slots;
    // Set-up tables: the systems of each one-launch kind, then those of the
    // multi-launch solve.  Active tables: the multi-launch systems first,
    // which the iterations below run over.
    constexpr int NCLS = 4, CLS[NCLS] = {8, 4, SV_WIDE, 0};
    int cls_tiles[NCLS] = {0, 0, 0, 0}, nis_many = 0, nta_many = 0, nia_many = 0;
    for (int k : act) {
        SrvSlot &sl = S->slots[k];
        if (sl.phase != 0) continue;
        sl.kind = sl.many ? 0 : solve_kind(ctx, sl.L.seg.n);
        if (!sl.many && !sl.kind && size_kind(ctx, sl.L.seg.n)) rested(ctx);
    }
    auto cls_of = [](const SrvSlot &sl) { return sl.kind; };
    for (int c = 0; c < NCLS; c++)
        for (int k : act) {
            SrvSlot &sl = S->slots[k];
            if (sl.phase != 0 || cls_of(sl) != CLS[c]) continue;
            for (int t = 0; t < sl.L.ntile; t++) hts[nts++] = Tile{k, t * TILE};
            cls_tiles[c] += sl.L.ntile;
            his[nis++] = k;
            if (CLS[c] == 0) nis_many++;
        }
    int nta_coarse = 0, nia_coarse = 0, nta_whole = 0, nia_whole = 0;
    for (int c = 0; c < 4; c++)        // multi-launch above and up to FINE_MAX, in two launches, one-launch
        for (int k : act) {
            SrvSlot &sl = S->slots[k];
            const int n = sl.L.seg.n, mine = cls_of(sl) != 0 ? 3 : n > FINE_MAX ? 0 : split_iteration(ctx, n) ? 2 : 1;
            if (mine != c) continue;
            for (int t = 0; t < sl.L.ntile; t++) hta[nta++] = Tile{k, t * TILE};
            hia[nia++] = k;
            if (c == 0) {
                nta_coarse = nta;
                nia_coarse = nia;
            }
            if (c <= 1) {
                nta_whole = nta;
                nia_whole = nia;
            }
            if (c <= 2) {
                nta_many = nta;
                nia_many = nia;
            }
        }
    HIPCHK(hipMemcpyAsync(S->dtiles_setup, hts, sizeof(Tile) * std::max(nts, 1), hipMemcpyHostToDevice, st));
    HIPCHK(hipMemcpyAsync(S->dtiles_act, hta, sizeof(Tile) * nta, hipMemcpyHostToDevice, st));
    HIPCHK(hipMemcpyAsync(S->dids_setup, his, sizeof(int) * std::max(nis, 1), hipMemcpyHostToDevice, st));
    HIPCHK(hipMemcpyAsync(S->dids_act, hia, sizeof(int) * nia, hipMemcpyHostToDevice, st));
    const dim3 b(TILE);
    if (nts) {
        const dim3 g(nts), gs(nis);
        const int *sid = S->dids_setup;
        Tile *T = S->dtiles_setup;
        hipLaunchKernelGGL(k_call_init, dim3((nis + 63) / 64), dim3(64), 0, st, sid, S->dsegs, nis, 0);
        hipLaunchKernelGGL(k_check_disp, g, b, 0, st, T, S->dsegs);
        hipLaunchKernelGGL(k_bin_clear, g, b, 0, st, T, S->dsegs);
        hipLaunchKernelGGL(k_bin, g, b, 0, st, T, S->dsegs);
        hipLaunchKernelGGL(k_scan_part, g, b, 0, st, T, S->dsegs);
        hipLaunchKernelGGL(k_scan_mid, gs, b, 0, st, sid, S->dsegs);
        hipLaunchKernelGGL(k_scan_fin, g, b, 0, st, T, S->dsegs);
        hipLaunchKernelGGL(k_scatter, g, b, 0, st, T, S->dsegs);
        hipLaunchKernelGGL(k_cell_sort, g, b, 0, st, T, S->dsegs);
        hipLaunchKernelGGL(k_gather<R>, g, b, 0, st, T, S->dsegs, -1);
        hipLaunchKernelGGL(k_fin_qshift, gs, b, 0, st, sid, S->dsegs);
        hipLaunchKernelGGL(k_qfix, g, b, 0, st, T, S->dsegs);
        const int nto = nts - cls_tiles[NCLS - 1], nio = nis - nis_many;   // of the one-launch solve
        if (nto) {
            launch_build<R>(true, T, nto, S->dsegs, prm, st);
            launch_rev(true, T, nto, S->dsegs, st);
            launch_assemble<R>(true, T, nto, S->dsegs, ctx->pd, st);
        }
        if (nis_many) {
            launch_build<R>(false, T + nto, nts - nto, S->dsegs, prm, st);
            launch_rev(false, T + nto, nts - nto, S->dsegs, st);
            hipLaunchKernelGGL(k_mark_built, dim3((nis_many + 63) / 64), dim3(64), 0, st, sid + nio, S->dsegs,
                               nis_many);
            launch_assemble<R>(false, T + nto, nts - nto, S->dsegs, ctx->pd, st);
        }
        // covalent energy and forces need only the lists: side stream, forked
        // after the assembly so that they run beside the solve
        HIPCHK(hipEventRecord(S->ev_fork, st));
        HIPCHK(hipStreamWaitEvent(S->side, S->ev_fork, 0));
        const bool fine = nts <= FINE_MAX / TILE;
        launch_bond<R>(fine, T, nts, S->dsegs, ctx->pd, S->side);
        launch_force_cov<R>(fine, T, nts, S->dsegs, prm, S->side);
        HIPCHK(hipEventRecord(S->ev_join, S->side));
        if (nto) {
            // (the kinds' launches run one after another)
            int most = 0;
            for (int c = 0; c < NCLS - 1; c++) most = std::max(most, solve_blocks(CLS[c], cls_tiles[c]));
            const int prc = pass.enter(most, ctx->ncu, st);
            if (prc) return prc;
        }
        for (int c = 0, t0 = 0; c < NCLS - 1; t0 += cls_tiles[c++])
            if (cls_tiles[c]) {
                launch_solve_prep<R>(ctx, CLS[c], T + t0, cls_tiles[c], S->dsegs, st);
                launch_solve<R>(CLS[c], ctx->ncu, T + t0, cls_tiles[c], S->dsegs, solve_ctl(ctx, 0), st);
            }
        if (nto) {
            // (where multi-launch iterations follow, others wait for the solves
            // alone; the event's own wait is on the side stream by now)
            const int lrc = pass.launched(nia_many ? S->ev_fork : nullptr);
            if (lrc) return lrc;
        }
        if (nis_many) {
            const dim3 gm(cls_tiles[NCLS - 1]);
            const Tile *Tm = T + nto;
            hipLaunchKernelGGL((k_hslice<R>), gm, b, 0, st, Tm, S->dsegs);
            hipLaunchKernelGGL(k_fin_w0, dim3(nis_many), b, 0, st, sid + (nis - nis_many), S->dsegs);
            hipLaunchKernelGGL((k_cg1_update<true>), gm, b, 0, st, Tm, S->dsegs);
        }
    }
    {
        const dim3 g(nta), gs(nia);
        const int *sid = S->dids_act;
        Tile *T = S->dtiles_act;
        CgCtl ctl{ctx->opts.cg_tol, ctx->opts.cg_maxit};
        // single-reduction solve: a solve of n iterations takes n + 1 rounds
        // (its first finalize counts none)
        poll = poll && nia == nia_many;
        const int limit = nia_many == 0 ? 0 : poll ? ctx->opts.cg_maxit + 2 : cg_iters;
        for (int c = 0; c < limit;) {
            const int first = std::max(ctx->opts.cg_check, std::min(S->iters_hint, ctx->opts.cg_maxit) + 1);
            const int chunk = poll ? std::min(limit - c, c == 0 ? first : ctx->opts.cg_check) : cg_iters;
            for (int k = 0; k < chunk; k++) {
                if (nia_whole) launch_cg1<R>(nullptr, false, T, nta_whole, sid, nia_whole, S->dsegs, ctl, st);
                if (nia_many > nia_whole)
                    launch_cg1<R>(nullptr, true, T + nta_whole, nta_many - nta_whole, sid + nia_whole,
                                  nia_many - nia_whole, S->dsegs, ctl, st);
            }
            c += chunk;
            if (!poll || c >= limit) break;
            hipLaunchKernelGGL(k_collect, dim3((nia_many + 63) / 64), dim3(64), 0, st, sid, S->dsegs, nia_many, S->dflags);
            HIPCHK(hipGetLastError());
            HIPCHK(hipMemcpyAsync(S->hflags, S->dflags, sizeof(int4) * nia_many, hipMemcpyDeviceToHost, st));
            HIPCHK(hipStreamSynchronize(st));
            bool any_done = false;
            for (int a = 0; a < nia_many; a++) any_done = any_done || S->hflags[a].x != 0;
            if (any_done) break;
            if (c >= cg_iters) {
                std::lock_guard<std::mutex> lk(S->mu);
                if (!S->pending.empty()) break;
            }
        }
        if (nts) HIPCHK(hipStreamWaitEvent(st, S->ev_join, 0));
        if (nia_coarse)
            launch_force_coul<R>(false, T, nta_coarse, sid, nia_coarse, S->dsegs, ctx->pd, 1, st);
        if (nia > nia_coarse)
            launch_force_coul<R>(true, T + nta_coarse, nta - nta_coarse, sid + nia_coarse, nia - nia_coarse, S->dsegs,
                                 ctx->pd, 1, st);
        hipLaunchKernelGGL(k_collect, dim3((nia + 63) / 64), dim3(64), 0, st, sid, S->dsegs, nia, S->dflags);
        HIPCHK(hipGetLastError());
        HIPCHK(hipMemcpyAsync(S->hflags, S->dflags, sizeof(int4) * nia, hipMemcpyDeviceToHost, st));
        // results of those finished, for which there is pinned room: handed
        // out to the systems solved in one launch first, the smallest first
        size_t at = 0;
        int most = 1;
        for (int a = nia - 1; a >= 0; a--) {
            const SrvReq &r = S->slots[hia[a]].req;
            const size_t f = r.F_out ? 24 * (size_t)r.n : 0, b = f + (r.q_out ? 8 * (size_t)r.n : 0);
            SrvOut &o = S->hout[a];
            o = SrvOut{nullptr, nullptr, hia[a], r.n};
            if (b == 0 || at + b > S->stage_bytes) continue;
            if (r.F_out) o.F = (double *)(S->stage + at);
            if (r.q_out) o.q = (double *)(S->stage + at + f);
            at += b;
            most = std::max(most, S->slots[hia[a]].L.ntile);
        }
        hipLaunchKernelGGL(k_deliver, dim3(nia, std::min(most, 64)), dim3(TILE), 0, st, S->hout, S->dsegs, S->hE);
        HIPCHK(hipGetLastError());
        HIPCHK(hipStreamSynchronize(st));
    }
    // harvest
    std::vector<int> fin;
    for (int a = 0; a < nia; a++) {
        SrvSlot &sl = S->slots[hia[a]];
        sl.phase = 1;
        if (S->hflags[a].y > 0) {
            fin.push_back(a);
        } else if (cls_of(sl) != 0) {
            // its one-launch solve gave up: set up again, multi-launch
            sl.many = true;
            sl.phase = 0;
            gave_up(ctx, -S->hflags[a].y);
        }
    }
    bool copies = false;
    for (int a : fin) {
        SrvSlot &sl = S->slots[hia[a]];
        const SrvReq &r = sl.req;
        const SrvOut &o = S->hout[a];
        const SrvArrays d = slot_arrays(S, sl);
        const size_t n = (size_t)r.n;
        if (r.F_out && o.F) memcpy(r.F_out, o.F, 24 * n);
        if (r.q_out && o.q) memcpy(r.q_out, o.q, 8 * n);
        if (r.E_out) *r.E_out = S->hE[a];
        if (r.F_out && !o.F) {
            HIPCHK(hipMemcpyAsync(r.F_out, d.F, 24 * n, hipMemcpyDeviceToHost, st));
            copies = true;
        }
        if (r.q_out && !o.q) {
            HIPCHK(hipMemcpyAsync(r.q_out, d.q, 8 * n, hipMemcpyDeviceToHost, st));
            copies = true;
        }
    }
    if (copies) HIPCHK(hipStreamSynchronize(st));
    const double t = now_s();
    std::vector<ctbop_result> res;
    for (int a : fin) {
        SrvSlot &sl = S->slots[hia[a]];
        ctbop_result r;
        r.ticket = sl.req.ticket;
        r.status = map_status(S->hflags[a].z);
        r.cg_iters = S->hflags[a].w;
        if (cls_of(sl) == 0) S->iters_hint = r.cg_iters;
        r.n_atoms = sl.req.n;
        r.t_submit = sl.req.t_submit;
        r.t_admit = sl.req.t_admit;
        r.t_done = t;
        res.push_back(r);
        sl.last_use = t;
        if (sl.sys_id >= 0) {
            sl.state = RETAINED;
        } else {
            range_free(S, sl.off, sl.bytes);
            sl.state = FREE;
        }
        sl.req.pos.clear();
        sl.req.pos.shrink_to_fit();
        sl.req.types.clear();
        sl.req.types.shrink_to_fit();
    }
    {
        std::lock_guard<std::mutex> lk(S->mu);
        for (auto &r : res) S->done.push_back(r);
        S->completed += (long)res.size();
        S->ticks++;
    }
    if (!res.empty()) S->cv.notify_all();
    return CTBOP_OK;
}

// into the queue, for the next tick
int queue_request(ctbop_server *S, SrvReq &r, long *ticket)
{
    r.t_submit = now_s();
    {
        std::lock_guard<std::mutex> lk(S->mu);
        if (S->stop) return fail(S->error ? S->error : CTBOP_E_INVAL, "server stopped: " + S->errmsg);
        if (S->pending.size() >= S->max_pending) return fail(CTBOP_E_BUSY, "pending queue full");
        r.ticket = S->next_ticket++;
        if (ticket) *ticket = r.ticket;
        S->pending.push_back(std::move(r));
    }
    S->cv.notify_all();
    return CTBOP_OK;
}

// the server's stream, events and pinned tables (whichever exist)
void release_handles(ctbop_server *S)
{
    if (S->side) {
        (void)hipStreamSynchronize(S->side);
        (void)hipStreamDestroy(S->side);
    }
    if (S->ev_fork) (void)hipEventDestroy(S->ev_fork);
    if (S->ev_join) (void)hipEventDestroy(S->ev_join);
    leave_turn(S->turn_dev);
    if (S->htiles) (void)hipHostFree(S->htiles);
    if (S->hids) (void)hipHostFree(S->hids);
    if (S->hflags) (void)hipHostFree(S->hflags);
    if (S->stage) (void)hipHostFree(S->stage);
}

void server_loop(ctbop_server *S)
{
    (void)hipSetDevice(S->device);
    for (;;) {
        // solver iterations of this tick: with nobody waiting for admission,
        // iterate until the active systems converge (checked between chunks),
        // so a lone request finishes in one tick (each tick costs table
        // uploads, host round trips and the gated force launches)
        int cg_iters = S->cg_per_tick;
        bool poll = false;
        {
            std::unique_lock<std::mutex> lk(S->mu);
            bool any_active = false;
            for (auto &sl : S->slots)
                if (sl.state == ACTIVE) any_active = true;
            S->cv.wait(lk, [&] { return S->stop || !S->pending.empty() || any_active; });
            if (S->stop) return;
            // admission in arrival order
            while (!S->pending.empty()) {
                bool placed = false;
                int rc = admit_one(S, S->pending.front(), placed);
                if (rc) {
                    S->error = rc;
                    S->errmsg = g_err;
                    ctbop_result r;
                    memset(&r, 0, sizeof r);
                    r.ticket = S->pending.front().ticket;
                    r.status = rc;
                    r.n_atoms = S->pending.front().n;
                    r.t_submit = S->pending.front().t_submit;
                    r.t_admit = r.t_done = now_s();
                    S->done.push_back(r);
                    S->pending.pop_front();
                    continue;
                }
                if (!placed) break;
                S->pending.pop_front();
            }
            if (S->pending.empty()) poll = true;
        }
        const double t0 = now_s();
        int rc = S->ctx->opts.fp64 ? server_tick<double>(S, S->ctx->pd, cg_iters, poll)
                                   : server_tick<float>(S, S->ctx->pf, cg_iters, poll);
        S->busy_s += now_s() - t0;
        if (rc) {
            std::lock_guard<std::mutex> lk(S->mu);
            S->error = rc;
            S->errmsg = g_err;
            S->stop = true;
            S->cv.notify_all();
            return;
        }
    }
}

// A server with `stage` bytes of pinned room for inputs and results (0: each
// is copied by itself).  A request's inputs are under 1/350 of its region at
// the default list sizes, so 1/256 of the arena holds those of a full one.
constexpr size_t STAGE_MAX = (size_t)8 << 20;
int create_server(ctbop_ctx *ctx, void *arena, size_t arena_bytes, int max_slots, int cg_per_tick, void *stream,
                  size_t stage, ctbop_server **out)
{
    if (!ctx || !arena || !out || max_slots <= 0) return fail(CTBOP_E_INVAL, "bad argument");
    if (ctx->opts.fq_kappa > 0.0) return fail(CTBOP_E_INVAL, "server: not available with fq_kappa > 0");
    ctbop_server *S = new ctbop_server();
    S->ctx = ctx;
    S->arena = (char *)arena;
    S->arena_bytes = arena_bytes;
    S->max_slots = max_slots;
    S->cg_per_tick = cg_per_tick > 0 ? cg_per_tick : 8;
    S->stream = (hipStream_t)stream;
    S->max_tiles = 2 * (int)std::min<size_t>(arena_bytes / ((size_t)TILE * 1024) + max_slots, 1 << 22);
    const size_t tb = ctbop_server_table_bytes(max_slots, S->max_tiles);
    S->stage_bytes = stage;
    if (tb + (1 << 20) > arena_bytes) {
        delete S;
        return fail(CTBOP_E_NOMEM, "arena too small for the server tables");
    }
    char *p = S->arena;
    S->dsegs = (Seg *)p;
    p += align_up(sizeof(Seg) * max_slots, 256);
    S->dtiles_setup = (Tile *)p;
    p += align_up(sizeof(Tile) * S->max_tiles, 256);
    S->dtiles_act = (Tile *)p;
    p += align_up(sizeof(Tile) * S->max_tiles, 256);
    S->dids_setup = (int *)p;
    p += align_up(sizeof(int) * max_slots, 256);
    S->dids_act = (int *)p;
    p += align_up(sizeof(int) * max_slots, 256);
    S->dflags = (int4 *)p;
    p += align_up(sizeof(int4) * max_slots, 256);
    S->free_ranges[tb] = arena_bytes - tb;
    S->slots.resize(max_slots);
    const size_t per_slot = sizeof(int4) + sizeof(double) + sizeof(SrvOut) + sizeof(SrvAdmit);
    if (hipGetDevice(&S->device) != hipSuccess ||
        hipStreamCreateWithFlags(&S->side, hipStreamNonBlocking) != hipSuccess ||
        hipEventCreateWithFlags(&S->ev_fork, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&S->ev_join, hipEventDisableTiming) != hipSuccess ||
        join_turn(S->turn_dev) != CTBOP_OK ||
        hipHostMalloc((void **)&S->htiles, sizeof(Tile) * 2 * S->max_tiles, hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc((void **)&S->hids, sizeof(int) * 2 * max_slots, hipHostMallocDefault) != hipSuccess ||
        hipHostMalloc((void **)&S->hflags, per_slot * max_slots, hipHostMallocDefault) != hipSuccess) {
        release_handles(S);
        delete S;
        return fail(CTBOP_E_HIP, "server stream, events or pinned host tables");
    }
    if (stage && hipHostMalloc((void **)&S->stage, stage, hipHostMallocDefault) != hipSuccess) {
        (void)hipGetLastError();
        S->stage = nullptr;
        S->stage_bytes = 0;
    }
    S->hE = (double *)(S->hflags + max_slots);
    S->hout = (SrvOut *)(S->hE + max_slots);
    S->hadm = (SrvAdmit *)(S->hout + max_slots);
    S->th = std::thread(server_loop, S);
    ctx->servers++;
    *out = S;
    return CTBOP_OK;
}

} // namespace

extern "C" {

size_t ctbop_server_table_bytes(int max_slots, int max_tiles)
{
    return align_up(sizeof(Seg) * max_slots, 256) + 2 * align_up(sizeof(Tile) * max_tiles, 256) +
           2 * align_up(sizeof(int) * max_slots, 256) + align_up(sizeof(int4) * max_slots, 256);
}

int ctbop_server_request_bytes(ctbop_ctx *ctx, int n, const double *box, const int *pbc, size_t *bytes)
{
    if (!ctx || !bytes) return fail(CTBOP_E_INVAL, "null argument");
    Layout L;
    int rc = make_layout(ctx, n, box, pbc, nullptr, L);
    if (rc) return rc;
    *bytes = io_bytes(n) + L.bytes;
    return CTBOP_OK;
}

int ctbop_server_create(ctbop_ctx *ctx, void *arena, size_t arena_bytes, int max_slots, int cg_per_tick,
                        void *stream, ctbop_server **out)
{
    return create_server(ctx, arena, arena_bytes, max_slots, cg_per_tick, stream,
                         std::min(STAGE_MAX, align_up(arena_bytes / 256, 4096)), out);
}

int ctbop_server_submit(ctbop_server *S, const ctbop_request *rq, long *ticket)
{
    if (!S || !rq || !rq->pos_host || !rq->types_host || rq->n <= 0) return fail(CTBOP_E_INVAL, "bad request");
    size_t need;
    int rc = ctbop_server_request_bytes(S->ctx, rq->n, rq->box, rq->pbc, &need);
    if (rc) return rc;
    if (need + ctbop_server_table_bytes(S->max_slots, S->max_tiles) > S->arena_bytes)
        return fail(CTBOP_E_NOMEM, "request larger than the serving arena");
    SrvReq r;
    r.n = rq->n;
    r.pos.assign(rq->pos_host, rq->pos_host + 3 * (size_t)rq->n);
    r.types.assign(rq->types_host, rq->types_host + rq->n);
    memcpy(r.box, rq->box, sizeof r.box);
    for (int a = 0; a < 3; a++) r.pbc[a] = rq->pbc[a];
    r.Q = rq->total_charge;
    r.sys_id = rq->system_id;
    if (rq->q0_host) r.q0.assign(rq->q0_host, rq->q0_host + rq->n);
    r.E_out = rq->E_host;
    r.F_out = rq->F_host;
    r.q_out = rq->q_host;
    return queue_request(S, r, ticket);
}

int ctbop_server_poll(ctbop_server *S, ctbop_result *out, int max, double wait_s, int *n_done)
{
    if (!S || !n_done) return fail(CTBOP_E_INVAL, "null argument");
    std::unique_lock<std::mutex> lk(S->mu);
    if (S->done.empty() && wait_s > 0)
        S->cv.wait_for(lk, std::chrono::duration<double>(wait_s), [&] { return !S->done.empty() || S->stop; });
    int k = 0;
    while (k < max && !S->done.empty()) {
        out[k++] = S->done.front();
        S->done.pop_front();
    }
    *n_done = k;
    if (S->stop && S->error) return fail(S->error, "server stopped: " + S->errmsg);
    return CTBOP_OK;
}

int ctbop_server_stats(ctbop_server *S, double *out, int nout)
{
    if (!S || !out) return fail(CTBOP_E_INVAL, "null argument");
    std::lock_guard<std::mutex> lk(S->mu);
    int active = 0, retained = 0;
    for (auto &sl : S->slots) {
        active += sl.state == ACTIVE;
        retained += sl.state == RETAINED;
    }
    double v[9] = {(double)S->ticks, (double)S->admitted, (double)S->completed, (double)S->pending.size(),
                   (double)active, (double)retained, (double)S->used_bytes, (double)S->peak_bytes, S->busy_s};
    for (int k = 0; k < nout && k < 9; k++) out[k] = v[k];
    return CTBOP_OK;
}

int ctbop_server_destroy(ctbop_server *S)
{
    if (!S) return CTBOP_OK;
    {
        std::lock_guard<std::mutex> lk(S->mu);
        S->stop = true;
    }
    S->cv.notify_all();
    if (S->th.joinable()) S->th.join();
    (void)hipStreamSynchronize(S->stream);
    release_handles(S);
    S->ctx->servers--;
    delete S;
    return CTBOP_OK;
}

} // extern "C"
