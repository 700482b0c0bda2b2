"""Dense FP64 solve folded about both mirror planes, at the sizes where the
fold can go wrong, against the separable solve of the same plan."""
import numpy as np
import pytest

from paper_1806_04593_amd import workloads as W
from paper_1806_04593_amd import yyg

pytestmark = pytest.mark.gpu

# Potentials relative to the largest: both solves sum the same few thousand
# products per value in different orders, some 1e3 eps = 2e-13 at worst.
# Moments of one column relative to the largest of that column's degree: the
# terms cancel to well below the largest, so 1e-10.
TOL_PHI, TOL_MOM = 1e-12, 1e-10

CASES = {
    # both counts even, both odd, mixed; L = 2 has one column in a class
    "even": dict(kind="yinyang", n_theta=32, n_phi=92, n_r=20, lmax=12),
    "odd": dict(kind="yinyang", n_theta=33, n_phi=95, n_r=19, lmax=13),
    "mixed": dict(kind="yinyang", n_theta=32, n_phi=91, n_r=70, lmax=7),
    "low": dict(kind="yinyang", n_theta=47, n_phi=138, n_r=33, lmax=2),
    # rows past the register scan
    "loop_scan": dict(kind="yinyang", n_theta=12, n_phi=32, n_r=1030, lmax=3),
    "polar": dict(kind="polar", n_theta=36, n_phi=72, n_r=37, lmax=9),
    "polar_odd": dict(kind="polar", n_theta=37, n_phi=73, n_r=65, lmax=16),
    # a single row or column of cells meets itself
    "one_row": dict(kind="polar", n_theta=1, n_phi=73, n_r=900, lmax=8),
    "one_column": dict(kind="polar", n_theta=73, n_phi=1, n_r=900, lmax=8),
}


def _grid(c):
    d = (W.make_desc if c["kind"] == "yinyang" else W.make_polar_desc)(
        "fold", np.linspace(0.0, 1.0, c["n_r"] + 1), 3.0, c["lmax"], 0.9, 0)
    return yyg.Grid(dict(d, n_theta=c["n_theta"], n_phi=c["n_phi"]), 0)


def _rho(g):
    import torch
    gen = torch.Generator(device="cpu").manual_seed(5)
    return torch.rand(tuple(g.shape), generator=gen, dtype=torch.float64).to("cuda")


def _solve(g, rho):
    import torch
    phi = torch.full_like(rho, float("nan"))
    g.upload_rho(rho)
    g.solve(phi)
    torch.cuda.synchronize()
    return phi.cpu().numpy()


@pytest.mark.parametrize("name", sorted(CASES))
def test_folded_dense_solve(name):
    g = _grid(CASES[name])
    rho = _rho(g)
    assert np.prod(g.shape) * g.Q * (1 + g.patches) >= 4e6  # the folded path's range
    dense, mom = _solve(g, rho), g.moments()
    again = _solve(g, rho)
    assert np.array_equal(dense, again)
    g.set_method("separable")
    sep, smom = _solve(g, rho), g.moments()
    scale = np.abs(sep).max()
    print(f"{name}: {np.abs(dense - sep).max() / scale:.2e}, moments {np.abs(mom - smom).max() / np.abs(smom).max():.2e}")
    assert np.abs(dense - sep).max() <= TOL_PHI * scale
    assert np.abs(mom - smom).max() <= TOL_MOM * np.abs(smom).max()
    # back to the dense form: the moments are in its order again
    g.set_method("dense")
    assert np.array_equal(_solve(g, rho), dense)
    assert np.array_equal(g.moments(), mom)


@pytest.mark.parametrize("variant", range(14))
@pytest.mark.parametrize("split", [1, 3, 64])
def test_every_tile_and_split_folded(variant, split):
    """Ragged class sizes in every tile shape; 64 splits of a contraction
    over 192 cells leave most of them empty."""
    g = _grid(dict(kind="yinyang", n_theta=23, n_phi=32, n_r=45, lmax=7))
    rho = _rho(g)
    ref = _solve(g, rho)
    g.set_config(variant, split, variant)
    got = _solve(g, rho)
    assert np.abs(got - ref).max() <= TOL_PHI * np.abs(ref).max()
