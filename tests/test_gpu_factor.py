"""The coarsest level's factorisation at the edges of its panels, blocks and windows, against
the oracle's sparse LU through helm_coarse_solve, and its substitution for several
right-hand sides."""
import numpy as np
import pytest

from tests.gpu_helpers import oracle_hierarchy, rect_problem, rel

pytestmark = pytest.mark.gpu

from paper_2604_19501_amd import HELM_OP_C, from_problem  # noqa: E402
import synth  # noqa: E402

# (problem, root merge limit): separators of a few rows up to 1100, odd counts among them
PROBLEMS = {
    "2d_root_1": (lambda: synth.config2(128), 1),
    "2d_root_700": (lambda: synth.config2(192), 700),
    "2d_dense": (lambda: synth.config2(124), 1100),        # one front: 32 x 32 coarsest nodes
    "3d": (lambda: synth.config3(64), 1),
    "3d_dense": (lambda: synth.config3(40), 1331),         # one front: 11^3 nodes, over one window
    "compact_2d": (lambda: synth.paper_stack((192, 128), "cubic"), 300),
    "compact_3d": (lambda: synth.paper_3d((48, 40, 32)), 1),
}


@pytest.mark.parametrize("name", sorted(PROBLEMS))
@pytest.mark.parametrize("win,block,block_mb", [(1024, 128, 32), (1024, 128, 0), (48, 16, 0), (112, 64, 0), (16, 1, 32)])
def test_factorisation_panels_blocks_windows(monkeypatch, name, win, block, block_mb):
    """A single panel, several panels per block, several blocks per window and several windows
    per separator (win rows each), in every parity of the two copies.  Both solves are exact
    up to rounding: 1e-10 relative in FP64 (condition numbers of at most about 1e5 at these
    sizes) and 1e-4 with FP32 factors."""
    make, root = PROBLEMS[name]
    monkeypatch.setenv("HELM_ND_ROOT", str(root))
    monkeypatch.setenv("HELM_ND_WIN", str(win))
    monkeypatch.setenv("HELM_ND_KB_OUTER", str(block))
    monkeypatch.setenv("HELM_ND_REG_BLOCK_MB", str(block_mb))
    p = make()
    print("factorisation", name, win, block, block_mb, flush=True)
    H = oracle_hierarchy(p)
    rng = np.random.default_rng(5)
    for prec in ("f64", "f32"):
        s = from_problem(p, cycle_prec=prec)
        N3 = s.level_size(3)
        r = rng.standard_normal(N3) + 1j * rng.standard_normal(N3)
        tol = 1e-10 if prec == "f64" or p.stack == "compact" else 1e-4
        e = rel(s.coarse_solve(r).cpu().numpy(), H.lu3.solve(r))
        print("  %s error %.2e" % (prec, e), flush=True)
        assert e < tol, (prec, e)
        if p.stack != "compact":
            ec = rel(s.coarse_solve(r, op=HELM_OP_C).cpu().numpy(), np.conj(H.lu3.solve(np.conj(r))))
            assert ec < tol, (prec, ec)
        s.close()


@pytest.mark.parametrize("n,leaf,merge", [((128, 96), 8, "none"), ((128, 96), 64, "1,2,4,5"), ((192, 192), 32, "1,3,5"),
                                          ((40, 32, 24), 8, "none"), ((48, 48, 40), 64, "1,3")])
@pytest.mark.parametrize("splitk", [0, 1 << 30])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_substitution_shares_entries_over_right_hand_sides(monkeypatch, n, leaf, merge, splitk, prec):
    """1 to 9 right-hand sides in one lock-step group (1, 2, 4 or 8 of them share a launch's
    matrix entries): every solution equals the separate solve's bit for bit, with row-block
    items of 16, 32 and 64 rows, one to several waves, and split-K tiles."""
    import torch
    monkeypatch.setenv("HELM_ND_LEAF", str(leaf))
    monkeypatch.setenv("HELM_ND_MERGE", merge)
    monkeypatch.setenv("HELM_ND_SPLITK_KB", str(splitk))
    p = rect_problem(n)
    print("shared entries", n, leaf, merge, splitk, prec, flush=True)
    rng = np.random.default_rng(8)
    qs = [rng.standard_normal(p.N) + 1j * rng.standard_normal(p.N) for _ in range(9)]
    one = from_problem(p, nu=(1, 1), cycle_prec=prec)
    ref = [one.solve(q, tol=1e-300, max_iter=3, op=HELM_OP_C)[0] for q in qs]
    many = from_problem(p, nu=(1, 1), cycle_prec=prec, max_rhs=9)
    for nr in (1, 2, 3, 5, 9):
        xs, _ = many.solve_many(qs[:nr], tol=1e-300, max_iter=3, op=HELM_OP_C)
        for k in range(nr):
            assert torch.equal(xs[k], ref[k]), (nr, k)
    one.close()
    many.close()


@pytest.mark.parametrize("n", [(1024, 640), (96, 88, 80)])
@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_substitution_shares_entries_on_large_grids(n, prec):
    """launches of enough work-groups that 2, 4 and 8 right-hand sides share one: bit for bit the
    separate solves"""
    import torch
    p = rect_problem(n)
    print("shared entries, large", n, prec, flush=True)
    rng = np.random.default_rng(9)
    qs = [torch.from_numpy(rng.standard_normal(p.N) + 1j * rng.standard_normal(p.N)).cuda() for _ in range(11)]
    one = from_problem(p, nu=(1, 1), cycle_prec=prec)
    ref = [one.solve(q, tol=1e-300, max_iter=2)[0] for q in qs]
    one.close()
    many = from_problem(p, nu=(1, 1), cycle_prec=prec, max_rhs=11)
    for nr in (2, 3, 8, 11):
        xs, _ = many.solve_many(qs[:nr], tol=1e-300, max_iter=2)
        for k in range(nr):
            assert torch.equal(xs[k], ref[k]), (nr, k)
    many.close()
