"""When FGMRES iterations are captured as graphs: for calls of a kind (operator, tolerance, right-hand
sides, operators' scalars) that has served before and whose host was the slower side then."""
import numpy as np
import pytest
import torch

from tests.gpu_helpers import rect_problem

pytestmark = pytest.mark.gpu

from paper_2604_19501_amd import HELM_OP_C, from_problem  # noqa: E402


def test_graphs_follow_the_calls_that_repay_them(monkeypatch):
    """with every window of 64 iterations counted as late: no capture in the first solve of a new
    frequency, tolerance, operator or right-hand side count, and the same solution either way"""
    p = rect_problem((64, 48))
    rng = np.random.default_rng(4)
    qs = [torch.from_numpy(rng.standard_normal(p.N) + 1j * rng.standard_normal(p.N)).cuda() for _ in range(2)]
    monkeypatch.setenv("HELM_GRAPHS", "0")
    plain = from_problem(p, nu=(1, 1), cycle_prec="f64", restart=20)
    ref = plain.solve(qs[0], tol=1e-8)[0]
    plain.close()
    monkeypatch.delenv("HELM_GRAPHS")
    monkeypatch.setenv("HELM_GRAPHS_LATE", "0")
    s = from_problem(p, nu=(1, 1), cycle_prec="f64", restart=20, max_rhs=2)

    def repeat(**kw):
        """solves of one kind until their graphs are held; the first one captures none"""
        for k in range(40):
            x, info = s.solve(qs[0], **kw)
            held = s.info()["graphs"]
            print("  solve", k, kw, info["iterations"], "graphs", held, flush=True)
            if k == 0:
                before = held
            if held > before:
                return x
        raise AssertionError("no graphs")

    print("graphs", flush=True)
    assert s.info()["graphs"] == 0
    x = repeat(tol=1e-8)
    assert s.info()["graphs"] == 20 and torch.equal(x, ref)
    # another operator: its own graphs, once its calls repeat
    repeat(tol=1e-8, op=HELM_OP_C)
    assert s.info()["graphs"] == 40
    # another frequency: the graphs go, and the sweep's first solve captures none
    for k in range(1, 5):
        s.refactor(omega=p.omega * (1 + 0.01 * k))
        s.solve(qs[0], tol=1e-8)
        assert s.info()["graphs"] == 0
    repeat(tol=1e-8)
    assert s.info()["graphs"] == 20
    s.refactor(omega=p.omega)
    assert torch.equal(repeat(tol=1e-8), ref)
    # the same frequency: a new medium keeps them
    s.refactor()
    assert s.info()["graphs"] == 20 and torch.equal(s.solve(qs[0], tol=1e-8)[0], ref)
    xs, _ = s.solve_many(qs, tol=1e-8)
    assert torch.equal(xs[0], ref)
    s.close()
