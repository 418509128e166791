"""The boxes that variant 0 of the tiled level kernels takes on small grids, against its
default-sized boxes and the oracle's cycle."""
import numpy as np
import pytest

from tests.gpu_helpers import maxabs_rel, oracle_hierarchy, rect_problem

pytestmark = pytest.mark.gpu

from paper_2604_19501_amd import HELM_OP_C, from_problem  # noqa: E402

# Each node's sums are the same in every box; only the contraction of products into FMAs may
# differ, a few units in the last place per application.  About ten applications follow one
# another in a cycle, and the coarsest solve amplifies by up to about 10: 512 eps.
EPS = {"f32": 2.0 ** -24, "f64": 2.0 ** -53}
# against the oracle, as for every other cycle: rounding order in FP64, the coarsest solve's
# FP32 rounding in FP32
TOL = {"f64": 1e-10, "f32": 3e-4}


@pytest.mark.parametrize("nu", [(1, 1), (2, 2)])
@pytest.mark.parametrize("n", [(8, 20), (72, 132), (128, 128), (20, 8, 12), (44, 28, 36), (64, 64, 64)])
def test_small_boxes_match_default_boxes(monkeypatch, n, nu):
    """grids of one box and of partial boxes in every direction, up to one with 459 default
    sweep boxes and 405 restriction boxes (64^3; the small boxes end at 512)"""
    p = rect_problem(n)
    r = np.random.default_rng(11).standard_normal((2, p.N))
    r = r[0] + 1j * r[1]
    ref = oracle_hierarchy(p, cycle=2, nu_pre=nu[0], nu_post=nu[1]).precond(r)
    for prec in ("f64", "f32"):
        out = {}
        for boxes in ("0,0,0,0", "1,1,1,1"):
            monkeypatch.setenv("HELM_BOXES", boxes)
            print("small boxes", n, nu, prec, boxes, flush=True)
            s = from_problem(p, cycle=2, nu=nu, cycle_prec=prec)
            out[boxes] = [s.vcycle(r).cpu().numpy(), s.vcycle(r, op=HELM_OP_C).cpu().numpy()]
            s.close()
        for a, b in zip(out["0,0,0,0"], out["1,1,1,1"]):
            d = np.abs(a - b).max() / np.abs(b).max()
            print("  %s: max difference %.3e of the largest entry" % (prec, d), flush=True)
            assert d < 512 * EPS[prec], (prec, d)
        assert maxabs_rel(out["0,0,0,0"][0], ref) < TOL[prec]
