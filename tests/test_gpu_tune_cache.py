"""The tuning cache keeps the folded and the unfolded dense FP64 solve apart."""
import numpy as np
import pytest

from paper_1806_04593_amd import workloads as W

pytestmark = pytest.mark.gpu


def _grid(yyg, n_theta, n_phi):
    d = W.make_desc("cache", np.linspace(0.0, 1.0, 13), 9.0, 8, 0.9, 0)
    return yyg.Grid(dict(d, n_theta=n_theta, n_phi=n_phi), 0)


def test_folded_and_unfolded_entries(tmp_path, monkeypatch):
    """24 rows and 81 columns: 22 x 100 cells (1.3e7 products) fold into a
    quarter patch of 11 x 50, the size at which 11 x 50 cells (3.2e6) contract
    as they are."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_04593_amd import yyg
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("YYG_TUNE_CACHE", str(cache))
    folded, plain = _grid(yyg, 22, 100), _grid(yyg, 11, 50)
    folded.autotune("fp64")
    first = cache.read_text().splitlines()
    plain.autotune("fp64")
    both = cache.read_text().splitlines()
    assert len(first) == 2 and len(both) == 4, both
    assert folded.plan_info()["folded"] == 1 and plain.plan_info()["folded"] == 0
    keys = [ln.split(" -> ")[0] for ln in both]
    assert len(set(keys)) == 4, keys
    # what a plan finds under its own keys it takes: nothing is timed again
    cache.write_text("".join(f"{k} -> {v} 1\n" for k, v in zip(keys, (3, 4, 5, 6))))
    for g, (va, vs) in ((_grid(yyg, 22, 100), (3, 4)), (_grid(yyg, 11, 50), (5, 6))):
        g.autotune("fp64")
        info = g.plan_info()
        assert (info["var_ana"], info["split_ana"], info["var_syn"]) == (va, 1, vs)
    assert len(cache.read_text().splitlines()) == 4
