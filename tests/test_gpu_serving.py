"""Continuous-batching server (ctbop_server_*) on the GPU.

  - every request's E, F, q in a mixed batch of uneven sizes (8 to 3000
    atoms, clusters and periodic cells) is bitwise identical to the same
    request served alone, and to the single-system call;
  - results match the CPU oracle within the mixed-precision tolerances,
    also over the stream's whole size range (requests up to 20000 atoms),
    and to 1e-10 with an FP64 context;
  - with an arena that holds only a couple of requests at a time, admission
    waits for space (peak bytes stay within the arena) and results are
    unchanged;
  - a bad request (two atoms 0.35 A apart) fails alone with E_TOO_CLOSE and
    leaves the other results bitwise unchanged;
  - a retained system (system_id >= 0) reuses its lists and charges: the
    second request for slightly moved atoms converges in fewer iterations
    and matches a cold evaluation.
"""
import numpy as np
import pytest

from ctbop_inputs import generators as G

pytestmark = pytest.mark.gpu


def _requests(count=40, seed=7, nmax=3000):
    reqs = G.serving_requests(count, seed=seed, nmax=nmax)
    return [G.request_structure(r) for r in reqs]


@pytest.fixture(scope="module")
def ct():
    import paper_1802_07871_amd as ct
    return ct


@pytest.fixture(scope="module")
def structs():
    return _requests()


@pytest.fixture(scope="module")
def alone(ct, theta, structs):
    from paper_1802_07871_amd.serving import Server
    print(f"[serving] {len(structs)} requests alone", flush=True)
    srv = Server(ct.Potential(theta), 1 << 30, max_slots=64)
    out = []
    for s in structs:
        t = srv.submit(s.pos, s.types, s.box, s.pbc)
        out.append(srv.wait_all([t])[t])
    srv.close()
    return out


def _same(a, b):
    return a["E"] == b["E"] and np.array_equal(a["F"], b["F"]) and np.array_equal(a["q"], b["q"])


def test_mix_equals_alone_bitwise(ct, theta, structs, alone):
    from paper_1802_07871_amd.serving import Server
    print("[serving] mixed batch", flush=True)
    srv = Server(ct.Potential(theta), 1 << 30, max_slots=64)
    tickets = [srv.submit(s.pos, s.types, s.box, s.pbc) for s in structs]
    got = srv.wait_all(tickets)
    st = srv.stats()
    srv.close()
    assert st["completed"] == len(structs)
    for t, a in zip(tickets, alone):
        assert got[t]["status"] == 0
        assert _same(got[t], a)
    # requests really overlapped on the device: the largest number of them
    # admitted and not yet finished at one time
    ev = sorted([(got[t]["t_admit"], 1) for t in tickets] + [(got[t]["t_done"], -1) for t in tickets])
    cur = best = 0
    for _, d in ev:
        cur += d
        best = max(best, cur)
    assert best >= 8


def test_server_equals_single_system_call(ct, theta, structs, alone):
    pot = ct.Potential(theta)
    for s, a in list(zip(structs, alone))[:12]:
        E, F, q, info = pot.compute(s.pos, s.types, s.box, s.pbc, warm=False)
        assert E == a["E"]
        assert np.array_equal(F.cpu().numpy(), a["F"])
        assert np.array_equal(q.cpu().numpy(), a["q"])


def test_results_match_oracle(orc, theta, structs, alone):
    for s, a in list(zip(structs, alone))[:10]:
        if s.n > 1500:
            continue
        Eo, Fo, qo, _ = orc.evaluate(s.pos, s.types, s.box, s.pbc, theta, tol=1e-13)
        assert abs(a["E"] - Eo) / s.n < 1e-6
        if np.linalg.norm(Fo) > 0:
            assert np.linalg.norm(a["F"] - Fo) / np.linalg.norm(Fo) < 1e-5
        assert np.abs(a["q"] - qo).max() < 1e-6


def test_full_size_range_matches_oracle(ct, orc, theta):
    """Requests over the serving stream's whole size range, up to its largest
    (a 20000-atom cluster and a 20000-atom periodic cell), served in one mixed
    batch: each matches the oracle and, bit for bit, the single-system call."""
    from paper_1802_07871_amd.serving import Server
    reqs = G.serving_requests(12, seed=19, nmax=20000)
    reqs[0].update(n=20000, periodic=False)
    reqs[1].update(n=20000, periodic=True)
    structs = [G.request_structure(r) for r in reqs]
    print(f"[serving] full size range: {[s.n for s in structs]}", flush=True)
    srv = Server(ct.Potential(theta), 4 << 30, max_slots=64)
    tickets = [srv.submit(s.pos, s.types, s.box, s.pbc) for s in structs]
    got = srv.wait_all(tickets)
    srv.close()
    pot = ct.Potential(theta)
    for s, t in zip(structs, tickets):
        a = got[t]
        assert a["status"] == 0
        E, F, q, _ = pot.compute(s.pos, s.types, s.box, s.pbc, warm=False)
        assert E == a["E"] and np.array_equal(F.cpu().numpy(), a["F"]) and np.array_equal(q.cpu().numpy(), a["q"])
        Eo, Fo, qo, _ = orc.evaluate(s.pos, s.types, s.box, s.pbc, theta, tol=1e-13)
        assert abs(a["E"] - Eo) / s.n < 1e-6
        if np.linalg.norm(Fo) > 0:
            assert np.linalg.norm(a["F"] - Fo) / np.linalg.norm(Fo) < 1e-5
        assert np.abs(a["q"] - qo).max() < 1e-6


def test_fp64_server_matches_oracle(ct, orc, theta):
    """The server on an FP64 context (FP64 pair terms, charges solved to
    1e-13): a mixed batch of clusters and periodic cells, each request
    against the oracle to 1e-10 (energy per atom, relative forces,
    charges)."""
    from paper_1802_07871_amd.serving import Server
    reqs = G.serving_requests(8, seed=23, nmax=2500)
    structs = [G.request_structure(r) for r in reqs]
    print(f"[serving] fp64 batch: {[s.n for s in structs]}", flush=True)
    srv = Server(ct.Potential(theta, fp64=True, cg_tol=1e-13), 1 << 30, max_slots=16)
    tickets = [srv.submit(s.pos, s.types, s.box, s.pbc) for s in structs]
    got = srv.wait_all(tickets)
    srv.close()
    for s, t in zip(structs, tickets):
        a = got[t]
        assert a["status"] == 0
        Eo, Fo, qo, _ = orc.evaluate(s.pos, s.types, s.box, s.pbc, theta, tol=1e-13)
        assert abs(a["E"] - Eo) / s.n < 1e-10
        if np.linalg.norm(Fo) > 0:
            assert np.linalg.norm(a["F"] - Fo) / np.linalg.norm(Fo) < 1e-10
        assert np.abs(a["q"] - qo).max() < 1e-10


def test_admission_by_arena_budget(ct, theta, structs, alone):
    from paper_1802_07871_amd.serving import Server
    pot = ct.Potential(theta)
    probe = Server(pot, 1 << 26, max_slots=8)
    sizes = [probe.request_bytes(s.n, s.box, s.pbc) for s in structs]
    probe.close()
    arena = int(2.5 * max(sizes)) + (4 << 20)
    assert sum(sizes) > arena              # the batch cannot be resident at once
    print(f"[serving] tight arena {arena} bytes (largest request {max(sizes)})", flush=True)
    srv = Server(pot, arena, max_slots=8)
    tickets = [srv.submit(s.pos, s.types, s.box, s.pbc) for s in structs]
    got = srv.wait_all(tickets)
    st = srv.stats()
    srv.close()
    assert st["peak_bytes"] <= arena
    assert st["completed"] == len(structs)
    for t, a in zip(tickets, alone):
        assert _same(got[t], a)


def test_bad_request_fails_alone(ct, theta, structs, alone):
    from paper_1802_07871_amd.serving import Server
    bad = G.zincblende(2, sigma=0.0)
    bpos = bad.pos.copy()
    bpos[1] = bpos[0] + 0.2
    srv = Server(ct.Potential(theta), 1 << 30, max_slots=64)
    tickets = [srv.submit(s.pos, s.types, s.box, s.pbc) for s in structs[:10]]
    tb = srv.submit(bpos, bad.types, bad.box, bad.pbc)
    tickets += [srv.submit(s.pos, s.types, s.box, s.pbc) for s in structs[10:20]]
    got = srv.wait_all(tickets + [tb])
    srv.close()
    import paper_1802_07871_amd as ctm
    assert got[tb]["status"] == ctm.E_TOO_CLOSE
    for t, a in zip(tickets, alone[:20]):
        assert got[t]["status"] == 0 and _same(got[t], a)


def test_retained_system_warm_start(ct, orc, theta):
    from paper_1802_07871_amd.serving import Server
    s = G.random_system(1500, 0.7, 2.8, True, seed=71)
    srv = Server(ct.Potential(theta), 1 << 30, max_slots=16)
    t1 = srv.submit(s.pos, s.types, s.box, s.pbc, system_id=3)
    r1 = srv.wait_all([t1])[t1]
    pos2 = s.pos + np.random.Generator(np.random.PCG64(2)).normal(0, 0.005, s.pos.shape)
    t2 = srv.submit(pos2, s.types, s.box, s.pbc, system_id=3)
    r2 = srv.wait_all([t2])[t2]
    st = srv.stats()
    srv.close()
    assert st["retained"] == 1
    assert r2["cg_iters"] < r1["cg_iters"]
    Eo, Fo, qo, _ = orc.evaluate(pos2, s.types, s.box, s.pbc, theta, tol=1e-13)
    assert abs(r2["E"] - Eo) / s.n < 1e-6
    assert np.linalg.norm(r2["F"] - Fo) / np.linalg.norm(Fo) < 1e-5
    assert np.abs(r2["q"] - qo).max() < 1e-6


def test_inputs_past_the_pinned_room(ct, theta):
    """A server has 8 MiB of pinned room for a tick's inputs and results, an
    input of 314,432 atoms takes 8.8 million bytes and is copied by itself;
    beside it requests that go through the room, one with starting charges."""
    from paper_1802_07871_amd.serving import Server
    pot = ct.Potential(theta)
    big, small = G.zincblende(34, sigma=0.02, seed=91), G.zincblende(4, sigma=0.05, seed=92)
    print(f"[serving] inputs past the pinned room n={big.n}", flush=True)
    single = [pot.compute(s.pos, s.types, s.box, s.pbc, warm=False) for s in (small, big)]
    q0 = single[0][2].cpu().numpy()
    srv = Server(pot, 2 * Server(pot, 1 << 26, max_slots=2).request_bytes(big.n, big.box, big.pbc), max_slots=8)
    t = [srv.submit(small.pos, small.types, small.box, small.pbc), srv.submit(big.pos, big.types, big.box, big.pbc),
         srv.submit(small.pos, small.types, small.box, small.pbc, q0=q0)]
    got = srv.wait_all(t)
    srv.close()
    for k, (E, F, q, _) in zip(t, single):
        assert got[k]["status"] == 0 and got[k]["E"] == E
        assert np.array_equal(got[k]["F"], F.cpu().numpy()) and np.array_equal(got[k]["q"], q.cpu().numpy())
    # solved again from its own charges: at once, to the solver's tolerance
    assert got[t[2]]["status"] == 0 and got[t[2]]["cg_iters"] <= 2
    assert np.abs(got[t[2]]["q"] - q0).max() <= 1e-8


@pytest.mark.parametrize("way", [1, 2, 3, 4], ids=["multi", "no wait", "crowded", "late"])
def test_requests_by_the_multi_launch_solve(ct, orc, theta, way):
    """Requests whose one-launch solve gives up are set up again and solved in
    many launches, beside larger ones that always are (57,600 atoms: two
    launches per iteration)."""
    from paper_1802_07871_amd.serving import Server
    pot = ct.Potential(theta)
    structs = _requests(10, seed=9) + [G.random_system(33000, 0.7, 2.4, True, seed=93), G.slab_4h(60, 40, 6, seed=94)]
    assert structs[-1].n == 57600
    print(f"[serving] way {way}: {[s.n for s in structs]}", flush=True)
    ref = [pot.compute(s.pos, s.types, s.box, s.pbc, warm=False) for s in structs]
    pot.debug_solve(way)
    srv = Server(pot, 6 << 30, max_slots=16)
    tickets = [srv.submit(s.pos, s.types, s.box, s.pbc) for s in structs]
    got = srv.wait_all(tickets)
    srv.close()
    # (after a wait that ran out, later requests take the multi-launch solve at once)
    gave_up = pot.debug_solve()
    assert gave_up == (len(structs) - 1 if way == 3 else 0) if way in (1, 3) else 0 < gave_up < len(structs)
    for s, t, (E, F, q, _) in zip(structs, tickets, ref):
        a = got[t]
        F = F.cpu().numpy()
        assert a["status"] == 0
        assert abs(a["E"] - E) / s.n < 1e-6
        if np.linalg.norm(F) > 0:
            assert np.linalg.norm(a["F"] - F) / np.linalg.norm(F) < 1e-5
        assert np.abs(a["q"] - q.cpu().numpy()).max() < 1e-6


@pytest.mark.parametrize("way", [0, 2, 3], ids=["one launch", "no wait", "crowded"])
def test_errors_of_the_lists_are_kept(ct, theta, way):
    """Errors that the lists' build finds (two atoms 0.35 A apart, a Coulomb
    list that overflows) reach a request that is set up a second time too,
    and no other one."""
    from paper_1802_07871_amd.serving import Server
    pot = ct.Potential(theta, long_cap=320)          # (a row of the good crystal holds 274, of the dense cell 376)
    pot.debug_solve(way)
    good = G.zincblende(2, sigma=0.05, seed=95)
    close = good.pos.copy()
    close[1] = close[0] + 0.2
    dense = G.random_system(900, 0.9, 3.2, True, seed=96)
    print(f"[serving] errors of the lists, way {way}", flush=True)
    srv = Server(pot, 1 << 28, max_slots=8)
    t = [srv.submit(good.pos, good.types, good.box, good.pbc), srv.submit(close, good.types, good.box, good.pbc),
         srv.submit(dense.pos, dense.types, dense.box, dense.pbc)]
    got = srv.wait_all(t)
    srv.close()
    gave_up = pot.debug_solve()
    assert gave_up == way if way != 2 else 0 < gave_up <= 3
    assert [got[k]["status"] for k in t] == [0, ct.E_TOO_CLOSE, ct.E_NEIGH_OVERFLOW]


def test_small_requests_do_not_wait_for_a_large_one(ct, theta):
    """Requests solved in one launch beside one that takes many (74,088
    atoms): they are delivered in an earlier tick, with the results of a plain
    call."""
    from paper_1802_07871_amd.serving import Server
    pot = ct.Potential(theta)
    big = G.zincblende(21, sigma=0.05, seed=97)
    small = [G.zincblende(k, sigma=0.05, seed=98 + k) for k in (2, 4)]
    print(f"[serving] small requests beside n={big.n}", flush=True)
    ref = [pot.compute(s.pos, s.types, s.box, s.pbc, warm=False) for s in [big] + small]
    srv = Server(pot, 3 << 30, max_slots=8)
    t = [srv.submit(s.pos, s.types, s.box, s.pbc) for s in [big] + small]
    got = srv.wait_all(t)
    srv.close()
    for k, (E, F, q, _) in zip(t, ref):
        assert got[k]["status"] == 0 and got[k]["E"] == E
        assert np.array_equal(got[k]["F"], F.cpu().numpy()) and np.array_equal(got[k]["q"], q.cpu().numpy())
    assert all(got[k]["t_done"] < got[t[0]]["t_done"] for k in t[1:])


def test_every_form_of_the_solve_in_one_batch(ct, theta):
    """One launch, two and four launches per iteration (a stride of 640 takes
    60,000 atoms past the size for two), and systems above 65,536 atoms: each
    request gets the bits of the plain call."""
    from paper_1802_07871_amd.serving import Server
    pot = ct.Potential(theta, long_cap=640)
    structs = [G.slab_4h(50, 42, 6, seed=101), G.zincblende(21, sigma=0.05, seed=102), G.slab_4h(50, 50, 6, seed=103),
               G.zincblende(5, sigma=0.05, seed=104), G.slab_4h(34, 42, 6, seed=105)]
    assert [s.n for s in structs] == [50400, 74088, 60000, 1000, 34272]
    print("[serving] every form of the solve", flush=True)
    ref = [pot.compute(s.pos, s.types, s.box, s.pbc, warm=False) for s in structs]
    srv = Server(pot, 8 << 30, max_slots=8)
    tickets = [srv.submit(s.pos, s.types, s.box, s.pbc) for s in structs]
    got = srv.wait_all(tickets)
    srv.close()
    for t, (E, F, q, _) in zip(tickets, ref):
        assert got[t]["status"] == 0 and got[t]["E"] == E
        assert np.array_equal(got[t]["F"], F.cpu().numpy()) and np.array_equal(got[t]["q"], q.cpu().numpy())
