"""The folded dense solve's buffers: which plans hold them, and what becomes of
them where memory is short."""
import gc
import threading

import numpy as np
import pytest

from paper_1806_04593_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = 1e-12    # the FP64 gate of the potential: folded and unfolded sums
MIB = 1 << 20


def _env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1806_04593_amd import yyg
    gc.collect()   # plans that only a collection would release
    return torch, yyg


def _plan(yyg, n_r=200, lmax=8):
    """47 x 137 cells: a fold of 21 MB (a density) and 3 MB of bases."""
    d = W.make_desc("mem", np.linspace(0.0, 1.0, n_r + 1), 2.0, lmax, 0.9, 0)
    return yyg.Grid(d, 0)


def _rho(torch, g, seed=4):
    gen = torch.Generator("cuda").manual_seed(seed)
    return torch.rand(g.shape, dtype=torch.float64, device="cuda", generator=gen) + 0.1


def _solve(torch, g, rho):
    phi = torch.full_like(rho, float("nan"))
    g.upload_rho(rho)
    g.solve(phi)
    torch.cuda.synchronize()
    return phi


def _close(a, b):
    return float((a - b).abs().max()) <= TOL * float(b.abs().max())


def _free(torch):
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_held_by_dense_plans_only():
    torch, yyg = _env()
    base, fold = yyg.device_bytes(), 20 * MIB   # one density, the most of it
    g = _plan(yyg)
    created = yyg.device_bytes()
    rho = _rho(torch, g)
    phi = torch.empty_like(rho)
    g.set_method("separable")
    sep = _solve(torch, g, rho)
    separable = yyg.device_bytes()
    assert g.plan_info()["folded"] == 0
    g.close()
    # a plan that solved dense first is back at the same figure
    at = _free(torch)
    g = _plan(yyg)
    assert yyg.device_bytes() == created
    plan = at - _free(torch)
    assert plan < (created - base) + fold   # no fold yet
    g.upload_rho(rho)
    assert g.plan_info()["folded"] == 1 and yyg.device_bytes() == created
    assert at - _free(torch) - plan >= fold
    g.solve(phi)
    dense, mom = phi.clone(), g.moments()
    before = _free(torch)
    g.set_method("separable")
    assert g.plan_info()["folded"] == 0 and yyg.device_bytes() == separable
    assert _free(torch) - before >= fold - (separable - created)
    assert np.array_equal(g.moments(), mom)   # of the last solve, whose buffers are gone
    assert torch.equal(_solve(torch, g, rho), sep)
    # and from then on keeps both forms, the same results
    g.set_method("dense")
    assert g.plan_info()["folded"] == 1
    assert torch.equal(_solve(torch, g, rho), dense)
    g.set_method("separable")
    assert g.plan_info()["folded"] == 1
    assert _close(sep, dense)
    g.close()
    assert yyg.device_bytes() == base


def _call(yyg, call, g, rho, keep):
    if call == "separable":
        g.set_method("separable")
    elif call == "fp32":
        g.prepare("fp32")
    elif call == "host_rho":
        g.upload_rho(rho.cpu().numpy())
    elif call == "plan":
        keep.append(_plan(yyg))
    elif call == "autotune":
        g.autotune("fp64")
    else:
        g.set_config(10, 64, 10)


@pytest.mark.parametrize("call", ["separable", "fp32", "host_rho", "plan", "autotune", "config"])
def test_given_back_under_the_cap(call, monkeypatch):
    """What fits beside a plan that has not solved fits beside one that has."""
    torch, yyg = _env()
    keep = []
    g = _plan(yyg)
    rho = _rho(torch, g)
    held = yyg.device_bytes()
    if call == "autotune":   # 32 splits of the moments, a potential
        need = 32 * 400 * 81 * 8 + rho.numel() * 8
    elif call == "config":     # 64 splits, the former ones beside them
        need = 64 * 400 * 81 * 8
    else:
        monkeypatch.setenv("YYG_MAX_DEVICE_BYTES", str(held))   # no fold
        g.upload_rho(rho)
        monkeypatch.delenv("YYG_MAX_DEVICE_BYTES")
        _call(yyg, call, g, rho, keep)
        assert g.plan_info()["folded"] == 0
        need = yyg.device_bytes() - held
    for x in keep + [g]:
        x.close()
    keep.clear()
    g = _plan(yyg)
    folded = _solve(torch, g, rho)
    assert g.plan_info()["folded"] == 1
    mom = g.moments()
    monkeypatch.setenv("YYG_MAX_DEVICE_BYTES", str(held + need + 2 * MIB))
    _call(yyg, call, g, rho, keep)
    assert yyg.device_bytes() <= held + need
    assert g.plan_info()["folded"] == 0
    assert np.array_equal(g.moments(), mom)   # of the folded solve
    g.set_method("dense")
    assert _close(_solve(torch, g, rho), folded)
    assert _close(torch.from_numpy(g.moments()), torch.from_numpy(mom))
    # asked for, with memory to be had: folded again
    monkeypatch.delenv("YYG_MAX_DEVICE_BYTES")
    g.prepare("fp64")
    assert g.plan_info()["folded"] == 1
    assert _close(_solve(torch, g, rho), folded)
    for o in keep:
        assert _close(_solve(torch, o, rho), folded)
        o.close()
    g.close()


def test_not_taken_at_others_expense(monkeypatch):
    """A fold is not built by giving up another plan's."""
    torch, yyg = _env()
    g, h = _plan(yyg), _plan(yyg)
    rho = _rho(torch, g)
    folded = _solve(torch, g, rho)
    monkeypatch.setenv("YYG_MAX_DEVICE_BYTES", str(yyg.device_bytes() + 30 * MIB))   # one fold
    other = _solve(torch, h, rho)
    assert g.plan_info()["folded"] == 1 and h.plan_info()["folded"] == 0
    assert _close(other, folded)
    g.close()
    h.close()


def test_recorded_solves_keep_their_buffers(monkeypatch):
    torch, yyg = _env()
    g = _plan(yyg)
    rho = _rho(torch, g)
    folded = _solve(torch, g, rho)
    phi = torch.empty_like(rho)
    g.upload_rho(rho)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.solve(phi)
    monkeypatch.setenv("YYG_MAX_DEVICE_BYTES", str(yyg.device_bytes() + 21 * MIB))
    with pytest.raises(yyg.YygError) as e:
        g.upload_rho(rho.cpu().numpy())   # 20 MiB, fits without the fold
    assert e.value.status == yyg.ERR_OUT_OF_MEMORY
    monkeypatch.delenv("YYG_MAX_DEVICE_BYTES")
    g.set_method("separable")
    assert g.plan_info()["folded"] == 1
    for _ in range(3):
        phi.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(phi, folded)
    del graph
    g.close()


def test_first_upload_inside_a_capture():
    """Nothing can be allocated there: the recorded solve is the unfolded one."""
    torch, yyg = _env()
    g = _plan(yyg)
    rho = _rho(torch, g)
    phi = torch.empty_like(rho)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        g.upload_rho(rho)
        g.solve(phi)
    assert g.plan_info()["folded"] == 0
    graph.replay()
    torch.cuda.synchronize()
    first = phi.clone()
    folded = _solve(torch, g, rho)
    assert g.plan_info()["folded"] == 1
    for _ in range(2):
        phi.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(phi, first)
    assert _close(first, folded)
    del graph
    g.close()


def test_given_back_while_other_plans_solve(monkeypatch):
    """One thread solves folded, another makes plans that need its memory."""
    torch, yyg = _env()
    g = _plan(yyg)
    rho = _rho(torch, g)
    folded = _solve(torch, g, rho)
    h = _plan(yyg)
    room = yyg.device_bytes() + 2 * MIB   # two plans without a fold
    h.close()
    monkeypatch.setenv("YYG_MAX_DEVICE_BYTES", str(room))
    bad, stop = [], threading.Event()

    def solver():
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            phi = torch.empty_like(rho)
            for _ in range(200):
                g.upload_rho(rho, stream)
                g.solve(phi, stream=stream)
                stream.synchronize()
                if not _close(phi, folded):
                    bad.append("solve")
                g.prepare("fp64")   # folded again where it fits
                if stop.is_set():
                    break

    t = threading.Thread(target=solver)
    t.start()
    made = 0
    for _ in range(12):
        try:
            h = _plan(yyg)
            made += 1
            h.close()
        except yyg.YygError as e:   # the solver's call held the fold at that moment
            if e.status != yyg.ERR_OUT_OF_MEMORY:
                bad.append(str(e))
    stop.set()
    t.join()
    assert not bad and made > 0, (bad, made)
    g.close()
