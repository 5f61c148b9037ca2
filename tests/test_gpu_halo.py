"""The three forms of the charge-solve product's sliced rows, each against the
oracle: 16-bit positions in the tile's halo (the neighbours' p staged in LDS),
16-bit offsets (a tile whose halo is too large to stage) and full 32-bit
entries (rows that reach across the periodic seam of the sorted frame).

Which forms a system uses follows from its geometry, and the statistics of
the evaluation say how many entries took each; every case here asserts that
the form it is meant to cover occurs.  Tolerances as in the other parity
tests: mixed 1e-5 relative RMS forces, 1e-6 eV/atom, 1e-6 e; FP64 1e-10.
"""
import numpy as np
import pytest

from ctbop_inputs import generators as G

pytestmark = pytest.mark.gpu

TOL = {"mixed": dict(F=1e-5, E=1e-6, q=1e-6), "fp64": dict(F=1e-10, E=1e-10, q=1e-10)}


def _slab():
    s = G.slab_4h(40, 40, 8, step=True, deplete=0.3, seed=171)
    rng = np.random.Generator(np.random.PCG64(172))
    s.pos = s.pos + rng.normal(0.0, 0.05, s.pos.shape)
    return s


CASES = {
    # stepped slab of 50240 atoms: most tiles stage their halo; the rows next
    # to the periodic seam of the slowest axis of the sorted frame, whose
    # neighbours across it lie ~48000 rows away, keep full entries
    "stepped slab": (_slab, ("halo", "full")),
    # bulk crystal of 32768 atoms: a tile is a thin column of cells through
    # the whole box, whose neighbours are too many to stage
    "3C-SiC 32768": (lambda: G.zincblende(16, sigma=0.05, seed=173), ("off16",)),
    # small periodic system: every neighbour of a tile fits
    "periodic 1000": (lambda: G.random_system(1000, 0.6, 3.0, True, seed=174), ("halo",)),
}


@pytest.fixture(scope="module")
def ct():
    import paper_1802_07871_amd as ct
    return ct


@pytest.fixture(scope="module")
def systems():
    return {k: f() for k, (f, _) in CASES.items()}


@pytest.fixture(scope="module")
def oracle_results(orc, theta, systems):
    return {k: orc.evaluate(s.pos, s.types, s.box, s.pbc, theta, tol=1e-13) for k, s in systems.items()}


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("name", list(CASES))
def test_forms_match_oracle(ct, theta, systems, oracle_results, name, prec):
    s = systems[name]
    print(f"[halo] {name} n={s.n} {prec}", flush=True)
    pot = ct.Potential(theta, fp64=(prec == "fp64"), cg_tol=1e-9 if prec == "mixed" else 1e-13)
    E, F, q, info = pot.compute(s.pos, s.types, s.box, s.pbc, warm=False)
    Eo, Fo, qo, _ = oracle_results[name]
    nnz, wide, halo = info["nnz_coul"], info["nnz_coul_wide"], info["nnz_coul_halo"]
    forms = {"halo": halo, "full": wide, "off16": nnz - wide - halo}
    print(f"[halo] entries {nnz}: halo {halo}, 16-bit offsets {forms['off16']}, full {wide}", flush=True)
    for f in CASES[name][1]:
        assert forms[f] > 0, (name, f, forms)
    assert min(forms.values()) >= 0
    F = F.cpu().numpy()
    q = q.cpu().numpy()
    t = TOL[prec]
    assert info["status"] == 0
    assert abs(E - Eo) / s.n <= t["E"], (E, Eo)
    assert np.linalg.norm(F - Fo) / np.linalg.norm(Fo) <= t["F"]
    assert np.abs(q - qo).max() <= t["q"]


def test_repeat_is_bitwise(ct, theta, systems):
    """The staged product sums in a fixed order: two cold evaluations of the
    same input give identical bits."""
    s = systems["stepped slab"]
    print("[halo] repeat", flush=True)
    a = ct.Potential(theta).compute(s.pos, s.types, s.box, s.pbc, warm=False)
    b = ct.Potential(theta).compute(s.pos, s.types, s.box, s.pbc, warm=False)
    assert a[0] == b[0]
    assert bool((a[1] == b[1]).all()) and bool((a[2] == b[2]).all())


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
def test_rows_that_fill_their_stride(ct, theta, orc, prec):
    """Halo positions go in groups of eight 12-bit numbers, unless a slice's
    longest row would not fit its stride rounded up to a group: with no skin
    the Coulomb list holds the entries inside rc only, and a stride of the
    longest row, and of the next multiple of eight, takes each form (a system
    too large for the one-launch solve)."""
    s = G.slab_4h(40, 40, 6, seed=175)
    s.pos = s.pos + np.random.Generator(np.random.PCG64(176)).normal(0.0, 0.05, s.pos.shape)
    tol = 1e-9 if prec == "mixed" else 1e-13
    Eo, Fo, qo, _ = orc.evaluate(s.pos, s.types, s.box, s.pbc, theta, tol=1e-13)
    t = TOL[prec]
    cap = 512
    for k in range(3):
        print(f"[halo] stride {cap} n={s.n} {prec}", flush=True)
        pot = ct.Potential(theta, fp64=(prec == "fp64"), cg_tol=tol, skin=0.0, long_cap=cap)
        E, F, q, info = pot.compute(s.pos, s.types, s.box, s.pbc, warm=False)
        assert info["status"] == 0 and info["nnz_coul_halo"] > 0
        assert abs(E - Eo) / s.n <= t["E"]
        assert np.linalg.norm(F.cpu().numpy() - Fo) / np.linalg.norm(Fo) <= t["F"]
        assert np.abs(q.cpu().numpy() - qo).max() <= t["q"]
        longest = info["max_long"]
        cap = longest if k == 0 else (longest + 7) // 8 * 8


# The same forms above 65,536 atoms, where the product has a lane per row (the
# 32,768 and 50,240 atoms above run it with eight waves per row slice), and
# rows that fill their stride on both sides of that size.
LARGE = {
    "stepped slab": (lambda: G.slab_4h(50, 50, 8, step=True, deplete=0.3, seed=177), ("halo", "full")),
    "3C-SiC 74088": (lambda: G.zincblende(21, sigma=0.05, seed=178), ("off16",)),
    "full rows": (lambda: G.slab_4h(54, 54, 6, seed=179), ("halo",)),
    "full rows 60000": (lambda: G.slab_4h(50, 50, 6, seed=181), ("halo",)),
}


@pytest.mark.parametrize("name", list(LARGE))
def test_forms_of_a_large_system(ct, theta, orc, name):
    s = LARGE[name][0]()
    s.pos = s.pos + np.random.Generator(np.random.PCG64(180)).normal(0.0, 0.05, s.pos.shape)
    assert s.n > 65536 or name == "full rows 60000" and 49152 < s.n < 65536
    Eo, Fo, qo, _ = orc.evaluate(s.pos, s.types, s.box, s.pbc, theta, tol=1e-13)
    t, opts = TOL["mixed"], {}
    if name.startswith("full rows"):
        # a stride of the longest row: its slice keeps 16-bit positions
        opts = dict(skin=0.0, long_cap=ct.Potential(theta, skin=0.0).compute(s.pos, s.types, s.box, s.pbc)[3]["max_long"])
    print(f"[halo] {name} n={s.n} {opts}", flush=True)
    E, F, q, info = ct.Potential(theta, **opts).compute(s.pos, s.types, s.box, s.pbc, warm=False)
    nnz, wide, halo = info["nnz_coul"], info["nnz_coul_wide"], info["nnz_coul_halo"]
    forms = {"halo": halo, "full": wide, "off16": nnz - wide - halo}
    assert all(forms[f] > 0 for f in LARGE[name][1]), forms
    assert info["status"] == 0
    assert abs(E - Eo) / s.n <= t["E"]
    assert np.linalg.norm(F.cpu().numpy() - Fo) / np.linalg.norm(Fo) <= t["F"]
    assert np.abs(q.cpu().numpy() - qo).max() <= t["q"]


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
def test_halo_positions_of_a_small_system(ct, theta, systems, oracle_results, prec):
    """The "periodic 1000" system by the multi-launch solve (its own takes one launch,
    which has no slices): halo positions for every entry."""
    s = systems["periodic 1000"]
    print(f"[halo] multi-launch, periodic 1000 {prec}", flush=True)
    pot = ct.Potential(theta, fp64=(prec == "fp64"), cg_tol=1e-9 if prec == "mixed" else 1e-13)
    pot.debug_solve(ct.SOLVE_MULTI)
    E, F, q, info = pot.compute(s.pos, s.types, s.box, s.pbc, warm=False)
    Eo, Fo, qo, _ = oracle_results["periodic 1000"]
    t = TOL[prec]
    assert info["status"] == 0 and info["nnz_coul_halo"] == info["nnz_coul"] <= info["nnz_coul_slots"]
    assert info["nnz_coul_slots"] % 64 == 0
    assert abs(E - Eo) / s.n <= t["E"]
    assert np.linalg.norm(F.cpu().numpy() - Fo) / np.linalg.norm(Fo) <= t["F"]
    assert np.abs(q.cpu().numpy() - qo).max() <= t["q"]


@pytest.mark.parametrize("prec,cap", [("mixed", 752), ("mixed", 768), ("fp64", 656), ("fp64", 672)])
def test_sides_of_the_split_product(ct, theta, systems, oracle_results, prec, cap):
    """50,240 atoms with list strides on both sides of the rule that gives the
    product eight waves per row slice.
    """
    s = systems["stepped slab"]
    print(f"[halo] stride {cap} {prec}", flush=True)
    pot = ct.Potential(theta, fp64=(prec == "fp64"), cg_tol=1e-9 if prec == "mixed" else 1e-13, long_cap=cap)
    E, F, q, info = pot.compute(s.pos, s.types, s.box, s.pbc, warm=False)
    Eo, Fo, qo, _ = oracle_results["stepped slab"]
    t = TOL[prec]
    assert info["status"] == 0
    assert abs(E - Eo) / s.n <= t["E"]
    assert np.linalg.norm(F.cpu().numpy() - Fo) / np.linalg.norm(Fo) <= t["F"]
    assert np.abs(q.cpu().numpy() - qo).max() <= t["q"]
