"""GPU tests of the theta transforms folded about the equator and the moment
rotation by parity class (variants V + 4 and V + 5 of phases 1-3): against
the oracle at the edges of their tiles, and against the tiles where a wave
walks many row tiles."""

import numpy as np
import pytest

import oracle as O
from paper_1806_04593_amd import workloads as W

pytestmark = pytest.mark.gpu

STREAM, TILE = (18, 19), 10
TOL = 1e-12    # the FP64 gate of the potential


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _yy(res, n_r, lmax):
    return W.make_desc("theta", np.geomspace(1.0, 20.0, n_r + 1), res, lmax, 0.9, 0)


def _polar(n_t, n_p, n_r, lmax):
    d = W.make_polar_desc("theta", np.linspace(0.0, 1.0, n_r + 1), 10.0, lmax, 0.9, 0)
    return dict(d, n_theta=n_t, n_phi=n_p)


def _phases(d):
    return (1, 2, 3) if d["kind"] == "yinyang" else (1, 3)


@pytest.mark.parametrize("d", [
    _yy(30.0, 1, 0),         # one degree, one shell, five colatitudes
    _yy(10.0, 17, 1),        # a shell past a row tile; eleven colatitudes (a middle row)
    _yy(9.0, 16, 16),        # nine members in the largest class
    _yy(7.0, 5, 33),         # 17 even degrees: a second tile
    _yy(6.0, 3, 65),         # 33 members: a third tile, nine steps
    _yy(6.0, 2, 80),         # the widest the oracle reaches
    _polar(1, 9, 3, 2),
    _polar(33, 24, 19, 31),
], ids=lambda d: f"{d['kind']}-{d['n_theta']}-{d['lmax']}")
def test_against_oracle(d):
    torch = _torch()
    from paper_1806_04593_amd import yyg
    g = yyg.Grid(d, 0)
    g.set_method("separable")
    rho = np.random.default_rng(11).uniform(0.1, 1.0, g.shape)
    if d["kind"] == "polar":
        ref = O.solve_polar(d["r_edges"], d["n_theta"], d["n_phi"], d["lmax"], d["G"], rho)
    else:
        ref = O.solve(d["r_edges"], d["n_theta"], d["n_phi"], d["delta_theta"], d["delta_phi"], d["lmax"], d["G"], rho)
    phi = torch.empty(g.shape, dtype=torch.float64, device="cuda")
    d_rho = torch.from_numpy(rho).to("cuda")
    for v in STREAM:
        for phase in _phases(d):
            g.sep_config(phase, v)
            assert "stream" in g.sep_kernel(phase)
        phi.fill_(float("nan"))
        g.upload_rho(d_rho)
        g.solve(phi)
        err = float(np.max(np.abs(phi.cpu().numpy().reshape(ref.shape) - ref) / np.abs(ref)))
        print(d["lmax"], [g.sep_kernel(p) for p in _phases(d)], f"{err:.2e}", flush=True)
        assert err <= TOL, v


@pytest.mark.parametrize("d, streams", [
    (_yy(3.0, 601, 20), True),       # 76 row tiles per column, 38 per patch
    (_polar(90, 40, 1003, 94), True),
    (_polar(90, 40, 40, 95), False),   # past the kernels' degrees: the tiles of that number
    (_yy(9.0, 30, 128), False),
], ids=["3deg", "polar94", "polar95", "lmax128"])
def test_many_row_tiles_against_tiles(d, streams):
    torch = _torch()
    from paper_1806_04593_amd import yyg
    g = yyg.Grid(d, 0)
    g.set_method("separable")
    rho = torch.rand(g.shape, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(5)) + 0.1
    ref, phi = torch.empty_like(rho), torch.empty_like(rho)
    g.upload_rho(rho)
    for phase in _phases(d):
        g.sep_config(phase, TILE)
    g.solve(ref)
    for v in STREAM:
        for phase in _phases(d):
            g.sep_config(phase, v)
            assert ("stream" in g.sep_kernel(phase)) == streams
        phi.fill_(float("nan"))
        g.upload_rho(rho)
        g.solve(phi)
        assert float(((phi - ref) / ref).abs().max()) <= TOL, v
