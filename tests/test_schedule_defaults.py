"""The merged dissection levels that a grid without a tuned schedule takes (host only: they show in
the workspace a grid needs)."""
import pytest

pytest.importorskip("paper_2604_19501_amd._lib")
from paper_2604_19501_amd.solver import workspace_bytes  # noqa: E402

TWO_OF_THREE = ",".join(str(h) for h in range(1, 41) if h % 3)
ODD = ",".join(str(h) for h in range(1, 41, 2))
ODD_TO_9 = "1,3,5,7,9"


def need(n, **kw):
    return workspace_bytes(n, 1.0 / max(n), tuple((8, 8) for _ in n), 2.0, nu=(1, 1), cycle_prec="f32", **kw)


@pytest.mark.parametrize("n,merge,others", [
    ((600, 640), TWO_OF_THREE, (ODD, "none")),
    ((2048, 2040), TWO_OF_THREE, (ODD_TO_9, "none")),
    ((5120, 1024), ODD_TO_9, (TWO_OF_THREE, "none")),      # the fronts near the root stay apart
    ((3072, 3072), ODD_TO_9, (TWO_OF_THREE, ODD)),
    ((76, 52, 44), ODD, (TWO_OF_THREE, "none")),
    ((160, 128, 96), "none", (ODD,)),
])
def test_default_merges(monkeypatch, n, merge, others):
    monkeypatch.setenv("HELM_TUNE_CACHE", "")
    for v in ("HELM_ND_LEAF", "HELM_ND_ROOT", "HELM_ND_MERGE", "HELM_ND_SPLITK_KB"):
        monkeypatch.delenv(v, raising=False)
    default = need(n)
    monkeypatch.setenv("HELM_ND_MERGE", merge)
    assert need(n) == default
    for o in others:
        monkeypatch.setenv("HELM_ND_MERGE", o)
        assert need(n) != default, o
