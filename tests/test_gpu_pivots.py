"""The coarsest factorisation where the rows of an inversion window hold no good pivots: the
pivots of a separator then come from all its rows."""
import numpy as np
import pytest
import scipy.linalg as sl

import synth
from tests.gpu_helpers import oracle_hierarchy, rect_problem, rel

pytestmark = pytest.mark.gpu

from paper_2604_19501_amd import HELM_OP_C, from_problem  # noqa: E402
from paper_2604_19501_amd import _lib as L  # noqa: E402

# both solves are exact up to rounding, and the coarsest operators here have condition numbers of
# at most about 1e5
TOL = {"f64": 1e-10, "f32": 1e-4}


def undamped(n, omega):
    """layered medium without absorbing layers and complex shift: a real symmetric operator"""
    p = rect_problem(n, beta=0.0, alpha2=1.0)
    p.layer, p.sigma_max, p.alpha, p.omega = tuple((0, 0) for _ in n), 0.0, 1.0, omega
    return p


def resonance(n, rows):
    """a frequency at which the coarsest operator's first `rows` rows and columns are singular
    (K - omega^2 M there) and the whole operator is farthest from it"""
    a1, a2 = (oracle_hierarchy(undamped(n, w)).A[2].toarray().real for w in (1.0, 2.0))
    M = (a1 - a2) / 3.0
    K = a1 + M
    part = sl.eigh(K[:rows, :rows], M[:rows, :rows], eigvals_only=True)[3:40]
    whole = sl.eigh(K, M, eigvals_only=True)
    return float(np.sqrt(max(part, key=lambda v: np.min(np.abs(whole - v) / v))))


def check(s, H, p, prec):
    rng = np.random.default_rng(5)
    N3 = s.level_size(3)
    r = rng.standard_normal(N3) + 1j * rng.standard_normal(N3)
    e = rel(s.coarse_solve(r).cpu().numpy(), H.lu3.solve(r))
    print("  %s error %.2e" % (prec, e), flush=True)
    assert e < TOL[prec]
    if p.stack != "compact":
        ec = rel(s.coarse_solve(r, op=HELM_OP_C).cpu().numpy(), np.conj(H.lu3.solve(np.conj(r))))
        assert ec < TOL[prec]


# one front of the whole coarsest grid: 32 x 48, 32 x 34 and 11^3 nodes in two of the default
# windows, 16 x 16 in windows of 16 rows
@pytest.mark.parametrize("n,win,rows", [((124, 188), 1024, 768), ((124, 132), 1024, 544),
                                        ((40, 40, 40), 1024, 672), ((60, 60), 16, 16)])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_window_at_a_resonance(monkeypatch, n, win, rows, prec):
    """A frequency at which the first window's block is singular, the whole separator's far from
    it, reached by a set-up and by a refactorisation from one and back to one where the windows
    serve."""
    monkeypatch.setenv("HELM_ND_LEAF", "4000")
    monkeypatch.setenv("HELM_ND_WIN", str(win))
    w = resonance(n, rows)
    print("resonance", n, win, w, flush=True)
    p = undamped(n, w)
    H = oracle_hierarchy(p)
    s = from_problem(p, cycle_prec=prec)
    check(s, H, p, prec)
    assert s.info()["fronts"] == 1 and s.info()["whole_pivots"]
    low = undamped(n, 0.5)                       # definite: every window serves
    s.refactor(omega=low.omega)
    check(s, oracle_hierarchy(low), low, prec)
    assert not s.info()["whole_pivots"]
    s.refactor(omega=w)
    check(s, H, p, prec)
    assert s.info()["whole_pivots"]
    s.close()


# (problem, environment): separators up to 1331 rows (register panels up to 1152), symmetric
# operators and not
PROBLEMS = {
    "2d": (lambda: synth.config2(128), {"HELM_ND_WIN": "16"}),
    "2d_root_700": (lambda: synth.config2(192), {"HELM_ND_WIN": "48", "HELM_ND_ROOT": "700"}),
    "2d_dense_1088": (lambda: rect_problem((124, 132)), {"HELM_ND_LEAF": "4000"}),
    "2d_dense_1152": (lambda: rect_problem((124, 140)), {"HELM_ND_LEAF": "4000"}),
    "3d": (lambda: synth.config3(64), {"HELM_ND_WIN": "112"}),
    "3d_dense": (lambda: synth.config3(40), {"HELM_ND_ROOT": "1331"}),
    "compact_2d": (lambda: synth.paper_stack((192, 128), "cubic"), {"HELM_ND_WIN": "112", "HELM_ND_ROOT": "300"}),
    "compact_3d_dense": (lambda: synth.paper_3d((48, 40, 32)), {"HELM_ND_LEAF": "4000"}),
}


@pytest.mark.parametrize("name", sorted(PROBLEMS))
@pytest.mark.parametrize("block,block_mb", [(128, 32), (64, 0)])
def test_pivots_from_whole_separators(monkeypatch, name, block, block_mb):
    """Every separator of several windows exchanged again with pivots from all its rows (a limit
    of 0 for the multipliers), below and above the 1024 rows of a register panel."""
    make, env = PROBLEMS[name]
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    monkeypatch.setenv("HELM_ND_GROWTH", "0")
    monkeypatch.setenv("HELM_ND_KB_OUTER", str(block))
    monkeypatch.setenv("HELM_ND_REG_BLOCK_MB", str(block_mb))
    p = make()
    print("whole separators", name, block, block_mb, flush=True)
    H = oracle_hierarchy(p)
    for prec in ("f64", "f32"):
        s = from_problem(p, cycle_prec=prec)
        check(s, H, p, "f64" if p.stack == "compact" else prec)
        assert s.info()["whole_pivots"]
        s.close()


# separators that fill a panel's rows (64, 128, 256, 512, 1024; 1152 after two windows) and 1536
@pytest.mark.parametrize("n", [(28, 28), (28, 60), (60, 60), (60, 124), (124, 124), (124, 140), (124, 188)])
def test_last_row_without_a_pivot_is_singular(monkeypatch, n):
    """a medium that is not a number at the last node reaches only the last entry of the coarsest
    operator's last row, the one that is left for the last column: a zero pivot is reported"""
    monkeypatch.setenv("HELM_ND_LEAF", "4000")
    p = undamped(n, 0.5)
    p.slowness = p.slowness.copy()
    p.slowness.ravel()[-1] = np.nan
    print("no pivot", n, flush=True)
    with pytest.raises(L.HelmError) as e:
        from_problem(p, cycle_prec="f64")
    assert e.value.code == L.HELM_ESINGULAR


# undamped grids with fronts whose interiors are close to a resonance: (n, seed, G, schedule)
RESONANT = [((428, 484), 536, 12.0, ("32", "1100")), ((28, 64, 28), 216, 8.0, ("8", "1")),
            ((44, 48, 80), 135, 8.0, ("8", "1"))]


@pytest.mark.parametrize("n,seed,G,schedule", RESONANT)
def test_fp64_factors_near_interior_resonances(monkeypatch, n, seed, G, schedule):
    """The blocks of a front that is close to singular are far from each other's rounding: left and
    right ones are formed separately in FP64, so that the solve stays within the operator's own
    condition, 100 eps cond_1(A3)."""
    import scipy.sparse.linalg as spla
    monkeypatch.setenv("HELM_ND_LEAF", schedule[0])
    monkeypatch.setenv("HELM_ND_ROOT", schedule[1])
    monkeypatch.setenv("HELM_ND_MERGE", "none")
    h = 1.0 / max(n)
    kap = synth.layered_slowness(n, 4, 2.0, seed)
    p = synth.Problem("resonant", len(n), n, h, kap, synth.omega_for_G(G, h, kap.max()),
                      tuple((0, 0) for _ in n), 0.0, 1.05, 0.0, [tuple(k // 2 for k in n)], G, alpha2=1.0)
    print("interior resonances", n, flush=True)
    H = oracle_hierarchy(p)
    A = H.A[2].tocsc().astype(complex)
    inv = spla.LinearOperator(A.shape, matvec=H.lu3.solve, rmatvec=lambda v: np.conj(H.lu3.solve(np.conj(v), "T")),
                              dtype=complex)
    cond = spla.norm(A, 1) * spla.onenormest(inv)
    s = from_problem(p, cycle_prec="f64")
    rng = np.random.default_rng(seed)
    for op in (0, HELM_OP_C):
        r = rng.standard_normal(A.shape[0]) + 1j * rng.standard_normal(A.shape[0])
        x = H.lu3.solve(r) if op == 0 else np.conj(H.lu3.solve(np.conj(r)))
        e = rel(s.coarse_solve(r, op=op).cpu().numpy(), x)
        print("  error %.2e, eps cond %.2e" % (e, 2.0 ** -53 * cond), flush=True)
        assert e < 100 * 2.0 ** -53 * cond
    s.close()
