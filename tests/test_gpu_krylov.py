"""The FGMRES passes' node layouts (one node per thread up to 65536 nodes, two up to 131072, four
above), at the edges of their blocks and on both sides of those lines."""
import numpy as np
import pytest
import torch

import synth
from oracle import operators as ops
from tests.gpu_helpers import rect_problem

pytestmark = pytest.mark.gpu

from paper_2604_19501_amd import from_problem  # noqa: E402

# 225, 273, 4209, 2457 nodes (blocks of 256 partly filled), 130321 (below the line), 131765
GRIDS = [(8, 24), (12, 20), (60, 68), (8, 12, 20), (360, 360), (364, 360)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n", GRIDS)
def test_estimate_is_the_residual(n, prec):
    """Every Arnoldi column of the last restart cycle enters the residual estimate, which equals
    the residual of the returned solution up to FP64 rounding, about restart * eps * |H||x| / |b|
    < 1e-12 here (whether or not 400 iterations reach the tolerance: on the 360^2 grids of this
    medium they do not); two solves agree bit by bit."""
    p = rect_problem(n)
    q = np.random.default_rng(3).standard_normal((2, p.N))
    q = q[0] + 1j * q[1]
    H = ops.helmholtz(p.n, p.h, p.slowness.ravel() ** 2, p.omega, ops.layer_sigma(p.n, p.layer, p.sigma_max))
    print("krylov", n, prec, p.N, flush=True)
    s = from_problem(p, nu=(1, 1), cycle_prec=prec, restart=20)
    x, info = s.solve(q, tol=1e-8, max_iter=390, history=True)
    x2, info2 = s.solve(q, tol=1e-8, max_iter=390)
    s.close()
    res = np.linalg.norm(q - H @ x.cpu().numpy()) / np.linalg.norm(q)
    assert abs(res - info["true_rel_residual"]) <= 1e-12
    assert abs(res - info["history"][-1]) <= 1e-12
    assert info["status"] != 0 or res <= 1e-8 * (1 + 1e-3)
    assert info["iterations"] == info2["iterations"] and torch.equal(x, x2)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("stack", ["p5", "compact"])
@pytest.mark.parametrize("n", [(252, 256), (256, 256), (360, 360)])
def test_two_nodes_per_thread(n, stack, prec):
    """65021 nodes (one per thread), 66049 and 130321 (two, the last block partly filled), both outer
    operators: the residual estimate is the returned solution's residual, to the bound above, and
    right-hand sides in lock-step take the separate solves' bits"""
    p = synth.paper_stack(n, "cubic") if stack == "compact" else rect_problem(n)
    print("krylov two nodes", n, stack, prec, p.N, flush=True)
    op = ops.helmholtz_compact if stack == "compact" else ops.helmholtz
    H = op(p.n, p.h, p.slowness.ravel() ** 2, p.omega, ops.layer_sigma(p.n, p.layer, p.sigma_max))
    rng = np.random.default_rng(7)
    qs = [rng.standard_normal(p.N) + 1j * rng.standard_normal(p.N) for _ in range(3)]
    s = from_problem(p, nu=(1, 1), cycle_prec=prec, restart=20, max_rhs=3)
    one = [s.solve(q, tol=1e-8, max_iter=70, history=True) for q in qs]
    many, _ = s.solve_many([torch.from_numpy(q).cuda() for q in qs], tol=1e-8, max_iter=70)
    s.close()
    for q, (x, info), y in zip(qs, one, many):
        res = np.linalg.norm(q - H @ x.cpu().numpy()) / np.linalg.norm(q)
        assert abs(res - info["history"][-1]) <= 1e-12
        assert torch.equal(x, y)
