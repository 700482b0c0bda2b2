"""Batched separable solves through the sweeps of the single-plan kernels:
mixed shapes in one launch, and the batches they do not cover, against the
same plans solved one by one."""
import numpy as np
import pytest

from paper_1806_04593_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = 1e-12    # the FP64 gate of the potential
SWEEPS = 5


def _yy(res, n_r, lmax):
    return W.make_desc("sweeps", np.geomspace(1.0, 20.0, n_r + 1), res, lmax, 0.9, 0)


def _polar(n_t, n_p, n_r, lmax):
    d = W.make_polar_desc("sweeps", np.linspace(0.0, 1.0, n_r + 1), 10.0, lmax, 0.9, 0)
    return dict(d, n_theta=n_t, n_phi=n_p)


@pytest.mark.parametrize("descs, phi_ana, phi_syn, theta", [
    # one degree, one shell, tile edges, the extra output (32), odd counts
    ([_yy(30.0, 1, 0), _yy(10.0, 17, 1), _yy(9.0, 16, 31), _polar(33, 24, 19, 32), _yy(7.0, 130, 16)], 5, 5, 5),
    # two tiles of outputs, up to nine steps; shells past a lane's 11
    ([_yy(5.0, 40, 33), _polar(20, 50, 705, 12), _yy(6.0, 23, 64), _polar(11, 37, 7, 47)], 5, 5, 5),
    # past the phi analysis (65), and past the synthesis (72): tiles there
    ([_yy(6.0, 10, 65), _yy(9.0, 33, 8)], None, 5, 5),
    ([_yy(6.0, 10, 72), _yy(9.0, 33, 8)], None, None, 5),
    # past the theta kernels, one-patch plans only, one column per scan block
    ([_polar(12, 40, 853, 95), _polar(9, 16, 5, 4)], None, None, None),
], ids=["small", "two-tiles", "lmax65", "lmax72", "polar95"])
def test_against_single_plans(descs, phi_ana, phi_syn, theta):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_04593_amd import yyg
    grids = [yyg.Grid(d, 0) for d in descs]
    rng = np.random.default_rng(3)
    rhos = [torch.from_numpy(rng.uniform(0.1, 1.0, g.shape)).to("cuda") for g in grids]
    refs, phis = [], [torch.full_like(r, float("nan")) for r in rhos]
    for g, r in zip(grids, rhos):
        g.set_method("separable")
        ref = torch.empty_like(r)
        g.upload_rho(r)
        g.solve(ref)
        refs.append(ref)
    b = yyg.Batch(grids, "fp64")
    info = b.info()
    for got, want in ((info["var_ana"], phi_ana), (info["var_syn"], phi_syn), (info["var_theta_ana"], theta)):
        assert (got == SWEEPS) == (want == SWEEPS), info
    for tag in ("first", "replay", "tuned"):
        if tag == "tuned":
            b.autotune()
        for p in phis:
            p.fill_(float("nan"))
        b.solve(rhos, phis)
        torch.cuda.synchronize()
        worst = max(float(((p - r) / r).abs().max()) for p, r in zip(phis, refs))
        print(tag, b.info(), f"{worst:.1e}", flush=True)
        assert worst <= TOL, tag
