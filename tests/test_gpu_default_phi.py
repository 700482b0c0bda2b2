"""The kernels a separable plan starts from: the 32 x 32 tiles where the
sweeps' waves are few or hold long rows of few columns, against the sweeps."""
import numpy as np
import pytest

from paper_1806_04593_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = 1e-12    # the FP64 gate of the potential
ANA_SWEEP, SYN_SWEEP, THETA_STREAM = 38, 37, 18


def _polar(n_t, n_p, n_r, lmax):
    d = W.make_polar_desc("phi", np.linspace(0.0, 1.0, n_r + 1), 10.0, lmax, 0.9, 0)
    return dict(d, n_theta=n_t, n_phi=n_p)


def _yy(n_t, n_p, n_r, lmax):
    d = W.make_desc("phi", np.geomspace(1.0, 20.0, n_r + 1), 3.0, lmax, 0.9, 0)
    return dict(d, n_theta=n_t, n_phi=n_p)


@pytest.mark.parametrize("d, ana, syn", [
    (_polar(2, 2000, 100, 8), "gemm", "gemm"),      # 14 row tiles of 32 cell tiles
    (_polar(20, 100, 150, 10), "gemm", "quad"),     # 200 of 2
    (_polar(40, 320, 256, 10), "gemm", "quad"),     # 640 of 5
    (_polar(90, 1000, 400, 10), "gemm", "gemm"),    # long rows of few columns
    (_polar(180, 1000, 300, 30), "quad", "gemm"),
    (_polar(90, 1000, 400, 32), "quad", "quad"),    # of more columns
    (_polar(180, 1600, 48, 10), "gemm", "quad"),    # longer still
    (_yy(150, 450, 100, 10), "gemm", "gemm"),       # without partners
    (_yy(150, 450, 100, 16), "gemm", "quad"),
    (_yy(40, 116, 200, 0), None, "gemm"),           # one column
    (_yy(40, 116, 200, 1), None, "quad"),
], ids=lambda v: f"{v['kind']}-{v['n_theta']}x{v['n_phi']}-{v['lmax']}" if isinstance(v, dict) else None)
def test_default_form(d, ana, syn):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_04593_amd import yyg
    g = yyg.Grid(d, 0)
    g.set_method("separable")
    names = g.sep_kernel(0), g.sep_kernel(4)
    print(names, flush=True)
    assert (ana is None or ana in names[0]) and syn in names[1], names
    _against(torch, g, (0, ANA_SWEEP), (4, SYN_SWEEP))


@pytest.mark.parametrize("d, tile", [
    (_yy(47, 137, 50, 25), True),      # 51 columns of 7 row tiles
    (_yy(25, 71, 100, 28), True),      # 57 of 13, 25 colatitudes
    (_yy(24, 68, 100, 28), False),
    (_yy(47, 137, 200, 15), False),    # 31 of 25
], ids=["few", "25", "24", "more"])
def test_default_theta_synthesis(d, tile):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_04593_amd import yyg
    g = yyg.Grid(d, 0)
    g.set_method("separable")
    assert ("stream" in g.sep_kernel(3)) != tile, g.sep_kernel(3)
    _against(torch, g, (3, THETA_STREAM))


def _against(torch, g, *config):
    """The plan as created against its kernels named by phase and variant."""
    rho = torch.rand(g.shape, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(3)) + 0.1
    got, ref = torch.full_like(rho, float("nan")), torch.full_like(rho, float("nan"))
    g.upload_rho(rho)
    g.solve(got)
    for phase, variant in config:
        g.sep_config(phase, variant)
        assert "quad" in g.sep_kernel(phase) or "stream" in g.sep_kernel(phase)
    g.solve(ref)
    assert float(((got - ref) / ref).abs().max()) <= TOL


@pytest.mark.parametrize("d, points", [
    (_polar(20, 180, 3, 4), 45),       # a quarter of the row
    (_polar(20, 181, 3, 4), 91),       # odd rows: no partners
    (W.make_desc("half", np.linspace(0.0, 1.0, 3), 2.0, 4, 0.9, 0), 46),   # 137 cells of 2 degrees
    (_yy(30, 91, 3, 4), 46),           # no partners: half the row
])
def test_reported_fold(d, points):
    """The share of a row that the twice-folded kernels contract over, for
    whoever counts their work: cells k and cc - k of the front half pair up."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_04593_amd import yyg
    g = yyg.Grid(d, 0)
    assert g.phi_points() == 0
    g.set_method("separable")
    assert g.phi_points() == points
    assert len(g.sep_info()) == 5
