"""The ways out of the one-launch charge solve.  A solve whose wait runs out,
whose blocks have too many neighbours, or that only a part of its blocks
finished is done again by the multi-launch solve, whose own path small systems
take on request too.  The library is told which (the kernels end as they
always do), at a size of each kind of the one-launch solve: 8 lanes per row, 4,
and blocks of 256 rows; the results must meet the oracle as the usual path's
do.  Tolerances as in the other parity tests: mixed 1e-5 relative RMS forces,
1e-6 eV/atom, 1e-6 e; FP64 1e-10 (charges solved to 1e-13 there).
"""
import numpy as np
import pytest

from ctbop_inputs import generators as G

pytestmark = pytest.mark.gpu

TOL = {"mixed": dict(F=1e-5, E=1e-6, q=1e-6), "fp64": dict(F=1e-10, E=1e-10, q=1e-10)}
WAYS = {"multi": 1, "no wait": 2, "crowded": 3, "late": 4}

# (atoms, periodic, carbon fraction, density g/cm^3)
CASES = [(40, False, 0.7, 2.6), (900, True, 0.9, 3.2), (17000, True, 0.9, 3.2), (33000, True, 0.7, 2.4)]
FQ_CASES = [(40, False, 0.7, 2.6), (900, True, 0.9, 3.2), (17000, True, 0.9, 3.2)]


@pytest.fixture(scope="module")
def ct():
    import paper_1802_07871_amd as ct
    return ct


@pytest.fixture(scope="module")
def reference(orc, theta):
    done = {}

    def get(case, kappa):
        if (case, kappa) not in done:
            n, periodic, c_frac, density = case
            s = G.random_system(n, c_frac, density, periodic, seed=4000 + n)
            args = s.pos, s.types, s.box, s.pbc, theta
            done[case, kappa] = s, orc.evaluate_fq(*args, kappa, tol=1e-13) if kappa else orc.evaluate(*args, tol=1e-13)
        return done[case, kappa]
    return get


def _check(got, ref, n, prec):
    (E, F, q, info), (Eo, Fo, qo, _), t = got, ref, TOL[prec]
    assert info["status"] == 0
    assert abs(E - Eo) / n <= t["E"]
    assert np.linalg.norm(F.cpu().numpy() - Fo) / np.linalg.norm(Fo) <= t["F"]
    assert np.abs(q.cpu().numpy() - qo).max() <= t["q"]


def _both(ct, theta, s, ref, way, prec, kappa):
    """A cold call, and a second one from its charges."""
    pot = ct.Potential(theta, fp64=(prec == "fp64"), cg_tol=1e-9 if prec == "mixed" else 1e-13, fq_kappa=kappa)
    assert pot.debug_solve(WAYS[way]) == 0
    # (asked again before each call: after a wait that ran out a context rests)
    _check(pot.compute(s.pos, s.types, s.box, s.pbc, warm=False), ref, s.n, prec)
    gave_up = pot.debug_solve(WAYS[way])
    assert gave_up == (0 if way == "multi" else 1)
    _check(pot.compute(s.pos, s.types, s.box, s.pbc, warm=True), ref, s.n, prec)
    assert pot.debug_solve() == 2 * gave_up
    # and the usual path again, on the same buffer
    _check(pot.compute(s.pos, s.types, s.box, s.pbc, warm=False), ref, s.n, prec)
    assert pot.debug_solve() == 2 * gave_up


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("way", ["multi", "no wait", "crowded", "late"])
@pytest.mark.parametrize("case", CASES, ids=[str(c[0]) for c in CASES])
def test_evaluation(ct, theta, reference, case, way, prec):
    s, ref = reference(case, 0.0)
    print(f"[ways out] n={s.n} {way} {prec}", flush=True)
    _both(ct, theta, s, ref, way, prec, 0.0)


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("way", ["multi", "no wait", "crowded", "late"])
@pytest.mark.parametrize("case", FQ_CASES, ids=[str(c[0]) for c in FQ_CASES])
def test_coupling(ct, theta, reference, case, way, prec):
    s, ref = reference(case, 1.0)
    print(f"[ways out, coupling] n={s.n} {way} {prec}", flush=True)
    _both(ct, theta, s, ref, way, prec, 1.0)


def test_bond_past_the_coulomb_cutoff(ct, theta):
    """Bonds longer than the Coulomb cutoff (2.4 A; within the lists' 3.2 A) are
    not among a block's neighbours: the coupling then takes the multi-launch
    solve by itself (the oracle has no pairs past the cutoff)."""
    th = theta.copy()
    th[54] = 2.4
    s = G.random_system(300, 0.4, 2.6, False, seed=4300)
    print("[ways out] bond past the Coulomb cutoff", flush=True)
    pot = ct.Potential(th, fq_kappa=1.0, skin=0.8)
    pot.debug_solve(WAYS["multi"])
    E, F, q, _ = pot.compute(s.pos, s.types, s.box, s.pbc, warm=False)
    assert pot.debug_solve() == 0
    got = pot.compute(s.pos, s.types, s.box, s.pbc, warm=False)
    assert pot.debug_solve() == 1
    _check(got, (E, F.cpu().numpy(), q.cpu().numpy(), None), s.n, "mixed")


@pytest.mark.parametrize("kappa", [0.0, 1.0])
def test_molecular_dynamics(ct, theta, kappa):
    """Steps with extrapolated starting charges: the trajectory of the usual
    path (charges solved to a residual of 1e-11)."""
    s = G.zincblende(4, sigma=0.05, seed=4400)
    vel = G.maxwell_velocities(s.types, 1000.0, seed=4401)
    print(f"[ways out] MD, coupling {kappa}", flush=True)
    out = []
    for way in (0, 1, 2, 3):
        pot = ct.Potential(theta, fp64=True, cg_tol=1e-11, fq_kappa=kappa)
        pot.debug_solve(way)
        x, v, F, q, th, info = pot.md_run(s.pos, vel, s.types, s.box, s.pbc, 0.5, 10, thermo_every=1)
        assert info["status"] == 0
        # (after a wait that ran out the next evaluations take the multi-launch solve)
        assert pot.debug_solve() == (0, 0, 1, 11)[way]
        out.append((th, q.cpu().numpy()))
    for th, q in out[1:]:
        assert np.abs(th - out[0][0]).max() / s.n < 1e-10
        assert np.abs(q - out[0][1]).max() < 1e-8


def test_rest_after_a_wait_that_ran_out(ct, theta):
    """A context whose solve gave up waiting takes the multi-launch solve for
    its next 256 evaluations, then the one-launch solve again."""
    s = G.random_system(300, 0.7, 2.6, True, seed=4500)
    pot = ct.Potential(theta)
    print("[ways out] rest", flush=True)
    usual = pot.compute(s.pos, s.types, s.box, s.pbc, warm=False)[0]
    pot.debug_solve(WAYS["no wait"])
    E = [pot.compute(s.pos, s.types, s.box, s.pbc, warm=False)[0] for _ in range(258)]
    assert pot.debug_solve() == 2
    assert max(abs(e - usual) for e in E) / s.n < 1e-9
    fresh = pot.system(s.n, s.box, s.pbc)
    assert pot.compute(s.pos, s.types, s.box, s.pbc, warm=False, sysbuf=fresh)[0] == usual


def test_callers_on_one_device(ct, theta):
    """Four threads with a stream and a context each, and a server beside them,
    with solves that fit the device one at a time only, one that always fits
    and one with 1024 threads per block: none gives up, and every result is bit
    for bit the lone caller's."""
    import threading

    import torch
    from paper_1802_07871_amd.serving import Server
    systems = [G.random_system(n, 0.7, 2.6, True, seed=4600 + n) for n in (12000, 20000, 600, 33000)]
    requests = [G.random_system(n, 0.7, 2.6, True, seed=4700 + n) for n in (9000, 300, 17000, 2500)]
    pot = ct.Potential(theta)
    alone = [pot.compute(s.pos, s.types, s.box, s.pbc, warm=False) for s in systems + requests]
    torch.cuda.synchronize()
    print("[ways out] callers on one device", flush=True)
    errors = []

    def same(got, ref):
        return got[0] == ref[0] and bool((got[1] == ref[1]).all()) and bool((got[2] == ref[2]).all())

    def caller(k):
        try:
            s = systems[k]
            mine = ct.Potential(theta)
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                buf = mine.system(s.n, s.box, s.pbc).buf
                for _ in range(25):
                    # (a new system each time: its state starts the sums of the next solve)
                    got = mine.compute(s.pos, s.types, s.box, s.pbc, warm=False,
                                       sysbuf=mine.system(s.n, s.box, s.pbc, buf=buf))
                    stream.synchronize()
                    if not same(got, alone[k]):
                        raise AssertionError(f"caller {k}: other bits than alone")
            if mine.debug_solve() != 0:
                raise AssertionError(f"caller {k}: {mine.debug_solve()} solves given up")
        except BaseException as e:
            errors.append(e)

    threads = [threading.Thread(target=caller, args=(k,)) for k in range(len(systems))]
    for t in threads:
        t.start()
    theirs = ct.Potential(theta)
    srv = Server(theirs, 2 << 30, max_slots=8)
    for _ in range(8):
        tickets = [srv.submit(s.pos, s.types, s.box, s.pbc) for s in requests]
        got = srv.wait_all(tickets)
        for t, (E, F, q, _) in zip(tickets, alone[len(systems):]):
            assert got[t]["status"] == 0 and got[t]["E"] == E
            assert np.array_equal(got[t]["F"], F.cpu().numpy()) and np.array_equal(got[t]["q"], q.cpu().numpy())
    srv.close()
    for t in threads:
        t.join()
    assert not errors, errors
    assert theirs.debug_solve() == 0


def test_bad_way_is_refused(ct, theta):
    with pytest.raises(ct.CtbopError) as e:
        ct.Potential(theta).debug_solve(5)
    assert e.value.code == ct.E_INVAL
