"""The marching stencils on lattices whose brick slices are no whole number of
64-site tiles: parts that start anywhere in a tile, shorter last parts, idle
lanes.  The forced bricks give slices of 36, 63, 65, 180 and 540 sites (and half
slices of 18 to 270); the unforced ones the default bricks of such extents.
Bars as for the other lattices: per site 1e-13 / 1e-5 / 5e-3 against the oracle,
solutions against the oracle's CG iterate after the same steps.
"""
import numpy as np
import pytest

import synth
from oracle import cg, evenodd, wilson
from gpu_util import assert_same_count_parity, gauge, rel, site_rel_err

pytestmark = pytest.mark.gpu

BAR = {"f64": 1e-13, "f32": 1e-5, "f16": 5e-3}
CASES = [((6, 10, 14, 4), None), ((10, 10, 10, 6), None), ((18, 2, 6, 4), "18,2,1"),
         ((14, 18, 2, 4), "14,9,1"), ((10, 26, 2, 4), "10,13,1"), ((30, 6, 6, 4), "30,6,1"),
         ((30, 6, 6, 4), "30,6,3")]


@pytest.fixture(scope="module")
def env():
    import torch

    import paper_1810_04201_amd as wd
    assert torch.cuda.is_available()
    return torch, torch.device("cuda:0"), wd


def _lattice(env, monkeypatch, dims, brick, seed):
    torch, dev, wd = env
    if brick:
        monkeypatch.setenv("WD_BRICK", brick)
    lat = wd.Lattice(dims)
    U = gauge(dims, seed)
    lat.set_gauge(torch.from_numpy(U).to(dev))
    return lat, U


@pytest.mark.parametrize("dims,brick", CASES)
@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
def test_stencil_and_schur(env, monkeypatch, dims, brick, prec):
    torch, dev, wd = env
    print(f"ragged dims={dims} brick={brick} prec={prec}", flush=True)
    lat, U = _lattice(env, monkeypatch, dims, brick, 61)
    src = synth.gaussian_sources(dims, [70, 71, 72])
    b = torch.from_numpy(src).to(dev)
    out = torch.full_like(b, float("nan"))
    fi, fo = wd.Field(lat, prec, 3), wd.Field(lat, prec, 3)
    for dagger in (0, 1):
        f = wilson.apply_Ddag if dagger else wilson.apply_D
        want = np.stack([f(U, s, dims, 0.124) for s in src])
        fi.load(b)
        wd.wd_dslash(lat, 0.124, dagger, fi, fo)
        fo.store(out)
        torch.cuda.synchronize()
        assert site_rel_err(out.cpu().numpy(), want) < BAR[prec]
        lat.apply(0.124, b, out, prec=prec, dagger=dagger, nrhs=3)
        torch.cuda.synchronize()
        assert site_rel_err(out.cpu().numpy(), want) < BAR[prec]
        lat.apply_schur(0.124, b, out, prec=prec, dagger=dagger, nrhs=3)
        torch.cuda.synchronize()
        want = np.stack([evenodd.apply_M(U, s, dims, 0.124, bool(dagger)) for s in src])
        par = evenodd.parity(dims)
        got = out.cpu().numpy()
        assert np.all(got[:, par == 1] == 0.0)
        assert site_rel_err(got[:, par == 0], want[:, par == 0]) < BAR[prec]
    fi.close()
    fo.close()
    lat.close()


@pytest.mark.parametrize("dims,brick", CASES)
@pytest.mark.parametrize("even_odd", [False, True])
def test_solve(env, monkeypatch, dims, brick, even_odd):
    torch, dev, wd = env
    print(f"ragged solve dims={dims} brick={brick} even_odd={even_odd}", flush=True)
    lat, U = _lattice(env, monkeypatch, dims, brick, 62)
    src = synth.gaussian_sources(dims, [80, 81])
    b = torch.from_numpy(src).to(dev)
    x = torch.zeros_like(b)
    rc, info = lat.solve(b, x, 0.12, nrhs=2, even_odd=even_odd)
    assert rc == wd.WD_OK, info
    n = info[1]["iters"]
    if even_odd:
        want, _, _ = evenodd.solve(U, src[1], dims, 0.12, tol=1e-300, max_iter=n)
    else:
        want, _, _ = cg.cgnr(lambda v: wilson.apply_D(U, v, dims, 0.12),
                             lambda v: wilson.apply_Ddag(U, v, dims, 0.12), src[1], tol=1e-300,
                             max_iter=n)
    assert_same_count_parity(x[1].cpu().numpy(), want)
    # a batched solve is the single solve, and mixed precision its solution
    one = torch.zeros_like(b[1])
    lat.solve(b[1].contiguous(), one, 0.12, even_odd=even_odd)
    assert torch.equal(one, x[1])
    for prec in ("f32", "f16"):
        lo = torch.zeros_like(b)
        rc, info = lat.solve(b, lo, 0.12, prec=prec, nrhs=2, even_odd=even_odd)
        assert rc == wd.WD_OK and max(i["true_rel_resid"] for i in info) <= 1e-10
        assert rel(lo.cpu().numpy(), x.cpu().numpy()) < 1e-8
    lat.close()
