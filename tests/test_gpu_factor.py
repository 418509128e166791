"""The coarsest level's factorisation at the edges of its panels, blocks and windows, against
the oracle's sparse LU through helm_coarse_solve."""
import numpy as np
import pytest

from tests.gpu_helpers import oracle_hierarchy, rel

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
