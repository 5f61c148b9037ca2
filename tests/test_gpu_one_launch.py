"""The charge solve in one launch (systems of up to 49,152 atoms) against the
oracle, at the sizes where its layout changes: one row block and its
neighbours (64 rows of 8 lanes), the change from 8 to 4 lanes per row (16,384
atoms on 256 CUs), the last size of blocks of 128 rows and the first that takes
the multi-launch solve, and rows longer than the entries a lane keeps in
registers (192: dense carbon has ~340 neighbours inside the cutoff), with
both numbers of lanes; at 4,096 atoms, the last size whose sorted frame is made
by one block; and at 65,536 atoms, the last size whose row kernels
run in blocks of 16 rows.  Tolerances as in the other parity tests: mixed 1e-5
relative RMS forces, 1e-6 eV/atom, 1e-6 e; FP64 1e-10 (charges solved to
1e-13 there).
"""
import numpy as np
import pytest

from ctbop_inputs import generators as G

pytestmark = pytest.mark.gpu

TOL = {"mixed": dict(F=1e-5, E=1e-6, q=1e-6), "fp64": dict(F=1e-10, E=1e-10, q=1e-10)}

# (atoms, periodic, carbon fraction, density g/cm^3)
CASES = [(63, False, 0.7, 2.6), (64, False, 0.7, 2.6), (65, True, 0.7, 2.6), (257, True, 0.6, 3.0),
         (4096, True, 0.7, 2.8), (4097, False, 0.7, 2.8),
         (900, True, 0.9, 3.2), (16384, True, 0.7, 2.8), (16385, False, 0.7, 2.8), (17000, True, 0.9, 3.2),
         (32512, True, 0.7, 2.4), (32513, True, 0.7, 2.4), (65536, True, 0.7, 2.8), (65537, True, 0.7, 2.8)]


@pytest.fixture(scope="module")
def ct():
    import paper_1802_07871_amd as ct
    return ct


@pytest.fixture(scope="module")
def reference(orc, theta):
    done = {}

    def get(case):
        if case not in done:
            n, periodic, c_frac, density = case
            s = G.random_system(n, c_frac, density, periodic, seed=3000 + n)
            done[case] = s, orc.evaluate(s.pos, s.types, s.box, s.pbc, theta, tol=1e-13)
        return done[case]
    return get


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("case", CASES, ids=[str(c[0]) for c in CASES])
def test_matches_oracle(ct, theta, reference, case, prec):
    s, (Eo, Fo, qo, _) = reference(case)
    print(f"[one launch] n={s.n} {prec}", flush=True)
    pot = ct.Potential(theta, fp64=(prec == "fp64"), cg_tol=1e-9 if prec == "mixed" else 1e-13)
    E, F, q, info = pot.compute(s.pos, s.types, s.box, s.pbc, warm=False)
    F, q, t = F.cpu().numpy(), q.cpu().numpy(), TOL[prec]
    assert info["status"] == 0
    assert abs(E - Eo) / s.n <= t["E"]
    assert np.linalg.norm(F - Fo) / np.linalg.norm(Fo) <= t["F"]
    assert np.abs(q - qo).max() <= t["q"]
    again = ct.Potential(theta, fp64=(prec == "fp64"), cg_tol=1e-9 if prec == "mixed" else 1e-13).compute(
        s.pos, s.types, s.box, s.pbc, warm=False)
    assert again[0] == E and np.array_equal(again[1].cpu().numpy(), F) and np.array_equal(again[2].cpu().numpy(), q)


# The charge coupling's solve, at its own edges: a block of 64 rows and one
# more, the change of lanes per row, rows and bonds past what a lane keeps in
# registers, the last size that takes it.  Its tolerances are the same (both
# sides solve the nonlinear charges to the tolerances above).
FQ_CASES = [(64, False, 0.7, 2.6), (65, True, 0.7, 2.6), (900, True, 0.9, 3.2), (16385, False, 0.7, 2.8),
            (32512, True, 0.7, 2.4)]


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("case", FQ_CASES, ids=[str(c[0]) for c in FQ_CASES])
def test_coupling_matches_oracle(ct, orc, theta, case, prec):
    n, periodic, c_frac, density = case
    s = G.random_system(n, c_frac, density, periodic, seed=3000 + n)
    print(f"[one launch, coupling] n={s.n} {prec}", flush=True)
    Eo, Fo, qo, _ = orc.evaluate_fq(s.pos, s.types, s.box, s.pbc, theta, 1.0, tol=1e-13)
    runs = []
    for _ in range(2):
        pot = ct.Potential(theta, fp64=(prec == "fp64"), cg_tol=1e-9 if prec == "mixed" else 1e-13, fq_kappa=1.0)
        E, F, q, info = pot.compute(s.pos, s.types, s.box, s.pbc, warm=False)
        assert info["status"] == 0
        runs.append((E, F.cpu().numpy(), q.cpu().numpy()))
    E, F, q = runs[0]
    t = TOL[prec]
    assert abs(E - Eo) / s.n <= t["E"]
    assert np.linalg.norm(F - Fo) / np.linalg.norm(Fo) <= t["F"]
    assert np.abs(q - qo).max() <= t["q"]
    assert runs[1][0] == E and np.array_equal(runs[1][1], F) and np.array_equal(runs[1][2], q)


# Blocks of 256 rows (32,769 to 49,152 atoms): one row in the last block, every
# row of the last size, rows past what a lane keeps in registers (128 entries),
# and a crystal whose blocks have more neighbours each than any other case.
WIDE_CASES = {"32769": lambda: G.random_system(32769, 0.7, 2.4, True, seed=3101),
              "49152": lambda: G.random_system(49152, 0.7, 2.8, False, seed=3102),
              "dense 33000": lambda: G.random_system(33000, 0.9, 3.2, True, seed=3103),
              "crystal 39304": lambda: G.zincblende(17, sigma=0.05, seed=3104)}


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("name", list(WIDE_CASES))
def test_blocks_of_256_rows(ct, orc, theta, name, prec):
    s = WIDE_CASES[name]()
    print(f"[one launch] {name} n={s.n} {prec}", flush=True)
    Eo, Fo, qo, _ = orc.evaluate(s.pos, s.types, s.box, s.pbc, theta, tol=1e-13)
    pot = ct.Potential(theta, fp64=(prec == "fp64"), cg_tol=1e-9 if prec == "mixed" else 1e-13)
    E, F, q, info = pot.compute(s.pos, s.types, s.box, s.pbc, warm=False)
    F, q, t = F.cpu().numpy(), q.cpu().numpy(), TOL[prec]
    assert info["status"] == 0
    assert abs(E - Eo) / s.n <= t["E"]
    assert np.linalg.norm(F - Fo) / np.linalg.norm(Fo) <= t["F"]
    assert np.abs(q - qo).max() <= t["q"]


# Lanes per row and entries that a lane keeps in registers
SLOT_CASES = [("small", 4, 0.0, 8, 24), ("small, coupling", 4, 1.0, 8, 24), ("middling", 13, 0.0, 4, 48),
              ("middling, coupling", 13, 1.0, 4, 48), ("blocks of 256 rows", 17, 0.0, 4, 32)]


@pytest.mark.parametrize("name,cells,kappa,lanes,regs", SLOT_CASES, ids=[c[0] for c in SLOT_CASES])
def test_slots_of_the_product(ct, theta, name, cells, kappa, lanes, regs):
    """The slots that a product reads, in a perfect crystal, where every row
    has the same length: groups of eight entries per lane up to what the
    registers hold, then single entries; the last wave's rows past the last
    atom are read with it."""
    s = G.zincblende(cells, sigma=0.0)
    print(f"[one launch] slots, {name} n={s.n}", flush=True)
    info = ct.Potential(theta, fq_kappa=kappa).compute(s.pos, s.types, s.box, s.pbc, warm=False)[3]
    row = info["nnz_coul"] // s.n
    assert row * s.n == info["nnz_coul"] and row > 100
    in_regs = min((row + 8 * lanes - 1) // (8 * lanes) * 8, regs) * lanes
    rows = (s.n + 64 // lanes - 1) // (64 // lanes) * (64 // lanes)
    assert info["nnz_coul_slots"] == rows * in_regs + s.n * max(0, row - regs * lanes)
