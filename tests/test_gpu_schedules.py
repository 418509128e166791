"""The exact coarsest solve under every parameter of its schedule that is in force: leaf size,
root limit, merged levels, split-K threshold, and the factorisation's windows and blocks."""
import numpy as np
import pytest

import synth
from tests.gpu_helpers import oracle_hierarchy, rect_problem, rel

pytestmark = pytest.mark.gpu

from paper_2604_19501_amd import HELM_OP_C, from_problem  # noqa: E402

VARIABLES = ("HELM_ND_LEAF", "HELM_ND_ROOT", "HELM_ND_MERGE", "HELM_ND_SPLITK_KB")
ODD = ",".join(str(h) for h in range(1, 40, 2))
TWO_OF_THREE = ",".join(str(h) for h in range(1, 40) if h % 3)
# leaf, root limit, merged heights, split-K threshold in KB (None: not set)
SCHEDULES = {
    "plain": (8, 1, "none", 1 << 30),
    "splitk": (8, 1, "none", 0),
    "leaf_64": (64, 1, "none", 1 << 30),
    "root_600": (8, 600, "none", 1 << 30),
    "merge_odd": (8, 1, ODD, 1 << 30),
    "merge_odd_splitk": (8, 1, ODD, 0),
    "merge_two_of_three": (16, 1, TWO_OF_THREE, 1 << 30),
    "merge_two_of_three_root_700": (16, 700, TWO_OF_THREE, 0),
}


def apply(monkeypatch, schedule):
    for name, v in zip(VARIABLES, schedule):
        if v is None:
            monkeypatch.delenv(name, raising=False)
        else:
            monkeypatch.setenv(name, str(v))


def check(p, prec, s, H):
    rng = np.random.default_rng(4)
    N3 = s.level_size(3)
    r = rng.standard_normal(N3) + 1j * rng.standard_normal(N3)
    tol = 1e-10 if prec == "f64" else 1e-4
    assert rel(s.coarse_solve(r).cpu().numpy(), H.lu3.solve(r)) < tol
    assert rel(s.coarse_solve(r, op=HELM_OP_C).cpu().numpy(), np.conj(H.lu3.solve(np.conj(r)))) < tol


@pytest.mark.parametrize("dim,n", [(2, 256), (3, 64)])
def test_every_schedule_is_exact_and_another(monkeypatch, dim, n):
    """each schedule against the oracle's sparse LU, in both precisions; no two of them build the
    same fronts and launches"""
    p = synth.config2(n) if dim == 2 else synth.config3(n)
    H = oracle_hierarchy(p, nu_pre=1, nu_post=1)
    seen = {}
    for name, schedule in SCHEDULES.items():
        apply(monkeypatch, schedule)
        for prec in ("f64", "f32"):
            print("schedule", dim, n, name, prec, flush=True)
            s = from_problem(p, nu=(1, 1), cycle_prec=prec)
            check(p, prec, s, H)
            i = s.info()
            key = (prec, i["fronts"], i["L_entries"], i["fwd_launches"], i["bwd_launches"])
            assert key not in seen, (name, seen[key])
            seen[key] = name
            s.close()


def test_split_k_takes_blocks_of_many_columns(monkeypatch):
    """64 KB per height: heights of many small fronts (at most 256 columns) keep one row-block
    launch each, one front of 1024 rows takes tiles and their sums"""
    p = synth.config2(256)
    H = oracle_hierarchy(p)
    launches = {}
    for kb in (64, 1 << 30):
        apply(monkeypatch, (32, 1, "none", kb))
        s = from_problem(p, cycle_prec="f64")
        check(p, "f64", s, H)
        launches[kb] = (s.info()["fwd_launches"], s.info()["bwd_launches"])
        s.close()
    print("split-K columns", launches, flush=True)
    assert launches[64] == launches[1 << 30]
    apply(monkeypatch, (4000, 1, "none", 64))
    p = rect_problem((124, 124))
    s = from_problem(p, cycle_prec="f64")
    check(p, "f64", s, oracle_hierarchy(p))
    assert s.info()["fwd_launches"] == 2
    s.close()


@pytest.mark.parametrize("n", [(280, 280), (332, 332)])
def test_row_blocks_of_long_vectors(monkeypatch, n):
    """one front of 71 x 71 or 84 x 84 rows in row blocks: its FP64 vector takes 80 or 113 KB of
    LDS, more than the 64 KB that a launch may take unasked"""
    apply(monkeypatch, (8000, 1, "none", 1 << 30))
    p = rect_problem(n)
    H = oracle_hierarchy(p)
    for prec in ("f64", "f32"):
        print("long vectors", prec, flush=True)
        s = from_problem(p, cycle_prec=prec, max_rhs=2)
        assert s.info()["fronts"] == 1
        check(p, prec, s, H)
        s.close()
