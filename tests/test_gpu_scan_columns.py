"""Radial scans of one-patch plans with four columns of a degree per block,
at the ends of a lane's chunk instances and where the columns no longer fit:
against the dense solve of the same plan (its own scan)."""
import numpy as np
import pytest

from paper_1806_04593_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = 1e-12    # the FP64 gate of the potential


@pytest.mark.parametrize("n_r, lmax", [
    (1, 29), (63, 29), (64, 30), (448, 31), (449, 32), (1087, 29), (1088, 30), (1089, 29),
    (2559, 29),   # the most that four columns hold
    (2560, 29),   # two
], ids=str)
def test_four_columns_per_block(n_r, lmax):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_04593_amd import yyg
    d = W.make_polar_desc("scan", np.linspace(0.0, 1.0, n_r + 1), 10.0, lmax, 0.9, 0)
    g = yyg.Grid(dict(d, n_theta=12, n_phi=20), 0)
    gen = torch.Generator("cuda").manual_seed(7)
    rho = torch.rand(g.shape, dtype=torch.float64, device="cuda", generator=gen) + 0.1
    dense, phi = torch.full_like(rho, float("nan")), torch.full_like(rho, float("nan"))
    g.upload_rho(rho)
    g.solve(dense)
    g.set_method("separable")
    g.upload_rho(rho)
    g.solve(phi)
    err = float(((phi - dense) / dense).abs().max())
    print(n_r, lmax, f"{err:.1e}")
    assert err <= TOL
