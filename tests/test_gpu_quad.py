"""GPU tests of the phi transforms folded about two meridians (variants
2V + 6 .. 2V + 13 of phases 0 and 4): every variant against the oracle on
grids at the edges of the fold, and against the once-folded tiles where a
block walks many row tiles."""

import math

import numpy as np
import pytest

import oracle as O
from paper_1806_04593_amd import workloads as W

pytestmark = pytest.mark.gpu

BASE, COUNT, TILE = 2 * 14 + 6, 8, 10
TOL = 1e-12    # the FP64 gate of the potential


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _desc(kind, r, n_t, n_p, d_t, d_p, lmax):
    return dict(name="quad", kind=kind, r_edges=np.asarray(r), n_theta=n_t, n_phi=n_p, delta_theta=d_t, delta_phi=d_p,
                lmax=lmax, G=0.9)


def _yy(res, n_r, lmax):
    n_t, n_p, d_t, d_p = W.grid_from_resolution(res)
    return _desc("yinyang", np.geomspace(1.0, 20.0, n_r + 1), n_t, n_p, d_t, d_p, lmax)


def _polar(n_t, n_p, n_r, lmax):
    return _desc("polar", np.linspace(0.0, 1.0, n_r + 1), n_t, n_p, 0.0, 0.0, lmax)


CASES = {
    "lmax0_pairs": _yy(9.0, 3, 0),                 # one even cosine, no sines
    "self_partner": _yy(10.0, 11, 7),              # 29 cells: a centre at 90 degrees and one at 0
    "odd_pairs": _yy(4.0, 9, 12),                  # odd number of pairs: a padding point in front
    "one_more_cosine": _yy(6.0, 5, 32),            # 17 even cosines, 16 of the others
    "no_pairs": _yy(7.0, 9, 13),                   # 180 / 7 is no whole number
    "buffers": _desc("yinyang", [0.5, 0.7, 1.3], 23, 71, math.radians(2.3), math.radians(1.9), 17),
    "one_row": _desc("yinyang", [0.0, 1.0], 3, 2, 0.0, 0.0, 1),
    "short_rows": _desc("yinyang", [0.0, 0.5, 1.0], 4, 5, 0.0, 0.0, 2),
    "six_rows": _desc("yinyang", [0.0, 0.5, 1.0], 4, 6, 0.0, 0.0, 3),
    "polar": _polar(18, 36, 17, 9),
    "polar_odd": _polar(11, 25, 7, 8),
    "polar_two": _polar(5, 2, 3, 1),
    "polar_lmax64": _polar(24, 48, 3, 64),         # 33 even cosines, 32 of the others
    "polar_lmax80": _polar(20, 40, 2, 80),
}


@pytest.mark.parametrize("name", list(CASES))
def test_every_variant_against_oracle(name):
    torch = _torch()
    from paper_1806_04593_amd import yyg
    d = CASES[name]
    g = yyg.Grid(d, 0)
    g.set_method("separable")
    rho = np.random.default_rng(3).uniform(0.1, 1.0, g.shape)
    if d["kind"] == "polar":
        ref = O.solve_polar(d["r_edges"], d["n_theta"], d["n_phi"], d["lmax"], d["G"], rho)
    else:
        ref = O.solve(d["r_edges"], d["n_theta"], d["n_phi"], d["delta_theta"], d["delta_phi"], d["lmax"], d["G"], rho)
    d_rho = torch.from_numpy(rho).to("cuda")
    phi = torch.empty(g.shape, dtype=torch.float64, device="cuda")
    for v in range(COUNT):
        for phase in (0, 4):
            g.sep_config(phase, BASE + v)
        print(name, g.sep_kernel(0), g.sep_kernel(4), flush=True)
        phi.fill_(float("nan"))
        g.upload_rho(d_rho)
        g.solve(phi)
        err = float(np.max(np.abs(phi.cpu().numpy().reshape(ref.shape) - ref) / np.abs(ref)))
        assert err <= TOL, (name, v, err)


@pytest.mark.parametrize("d", [
    _yy(2.0, 203, 8),                                        # 47 x 26 row tiles, the last partial
    _yy(1.0, 131, 40),                                       # six cell tiles, two row tiles side by side
    _yy(0.5, 40, 64),                                        # twelve stages, an extra column
    _polar(60, 120, 300, 33),
    _polar(36, 72, 70, 128),                                 # the widest basis
    _desc("yinyang", np.linspace(0.0, 1.0, 91), 61, 187, 0.04, 0.03, 23),
], ids=["2deg", "1deg", "0.5deg", "polar", "polar128", "no_pairs"])
def test_many_row_tiles_against_single_fold(d):
    """Against the once-folded 32 x 32 tiles on the same density: both round
    sums of at most n_theta n_phi products of one sign pattern, far below the
    gate; a row tile read or written in the wrong place is off by O(1)."""
    torch = _torch()
    from paper_1806_04593_amd import yyg
    g = yyg.Grid(d, 0)
    g.set_method("separable")
    rho = torch.rand(g.shape, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(5)) + 0.1
    ref, phi = torch.empty_like(rho), torch.empty_like(rho)
    g.upload_rho(rho)
    for phase in (0, 4):
        g.sep_config(phase, TILE)
    g.solve(ref)
    for v in range(COUNT):
        for phase in (0, 4):
            g.sep_config(phase, BASE + v)
        print(g.sep_kernel(0), g.sep_kernel(4), flush=True)
        phi.fill_(float("nan"))
        g.upload_rho(rho)
        g.solve(phi)
        assert float(((phi - ref) / ref).abs().max()) <= TOL, v
