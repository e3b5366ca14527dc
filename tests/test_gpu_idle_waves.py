"""Marching stencils whose last part leaves a whole wave of its workgroup without
a site (tests/part_lane_check.cpp counts them): 34^2 x 4 x 4 with its default brick
in float32 (578 sites), slices of 386 sites in float64, half slices of 257.  Such a
wave works on the part's last site too, which another wave's tile holds.
Bars as for the other lattices: per site 1e-13 / 1e-5 against the oracle, the float64
iterate after 16 steps 1e-11 against the oracle's, mixed solutions 1e-8 against the
float64 one.
"""
import numpy as np
import pytest

import synth
from oracle import cg, evenodd, wilson
from gpu_util import gauge, rel, site_rel_err

pytestmark = pytest.mark.gpu

BAR = {"f64": 1e-13, "f32": 1e-5, "f16": 5e-3}
CASES = [((34, 34, 4, 4), None), ((386, 2, 2, 4), "386,1,1"), ((514, 2, 2, 12), "514,1,1")]


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


# (a plain float32 application marches from 196608 sites)
@pytest.mark.parametrize("dims,brick", CASES + [((34, 34, 34, 6), None)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
def test_operators(env, monkeypatch, dims, brick, prec):
    torch, dev, wd = env
    print(f"idle waves dims={dims} brick={brick} prec={prec}", flush=True)
    lat, U = _lattice(env, monkeypatch, dims, brick, 63)
    n = -(-65536 // lat.volume)  # (the operator on canonical spinors marches then)
    src = synth.gaussian_sources(dims, list(range(90, 90 + n)))
    b = torch.from_numpy(src).to(dev)
    out = torch.full_like(b, float("nan"))
    fi, fo = wd.Field(lat, prec, n), wd.Field(lat, prec, n)
    for dagger in (0, 1):
        f = wilson.apply_Ddag if dagger else wilson.apply_D
        want = np.stack([f(U, s, dims, 0.124) for s in src])
        fi.load(b)
        wd.wd_dslash(lat, 0.124, dagger, fi, fo)
        fo.store(out)
        torch.cuda.synchronize()
        assert site_rel_err(out.cpu().numpy(), want) < BAR[prec]
        lat.apply(0.124, b, out, prec=prec, dagger=dagger, nrhs=n)
        torch.cuda.synchronize()
        assert site_rel_err(out.cpu().numpy(), want) < BAR[prec]
        lat.apply_schur(0.124, b, out, prec=prec, dagger=dagger, nrhs=n)
        torch.cuda.synchronize()
        want = np.stack([evenodd.apply_M(U, s, dims, 0.124, bool(dagger)) for s in src])
        par = evenodd.parity(dims)
        got = out.cpu().numpy()
        assert np.all(got[:, par == 1] == 0.0)
        assert site_rel_err(got[:, par == 0], want[:, par == 0]) < BAR[prec]
    fi.close()
    fo.close()
    lat.close()


# (the full slice of 514 sites leaves no wave idle)
@pytest.mark.parametrize("dims,brick,even_odd", [CASES[0] + (False,), CASES[0] + (True,),
                                                 CASES[1] + (False,), CASES[2] + (True,)])
def test_solve(env, monkeypatch, dims, brick, even_odd):
    torch, dev, wd = env
    print(f"idle waves solve dims={dims} brick={brick} even_odd={even_odd}", flush=True)
    lat, U = _lattice(env, monkeypatch, dims, brick, 64)
    src = synth.gaussian_spinor(dims, 95)
    b = torch.from_numpy(src).to(dev)
    x = torch.zeros_like(b)
    n = 16
    rc, info = lat.solve(b, x, 0.12, tol=1e-14, max_iter=n, even_odd=even_odd)
    assert rc == wd.WD_ERR_NOCONV and info[0]["iters"] == n
    if even_odd:
        want, _, _ = evenodd.solve(U, src, dims, 0.12, tol=1e-300, max_iter=n)
    else:
        want, _, _ = cg.cgnr(lambda v: wilson.apply_D(U, v, dims, 0.12),
                             lambda v: wilson.apply_Ddag(U, v, dims, 0.12), src, tol=1e-300,
                             max_iter=n)
    assert rel(x.cpu().numpy(), want) <= 1e-11
    rc, info = lat.solve(b, x, 0.12, even_odd=even_odd)
    assert rc == wd.WD_OK, info
    for prec in ("f32", "f16"):
        lo = torch.zeros_like(b)
        rc, info = lat.solve(b, lo, 0.12, prec=prec, even_odd=even_odd)
        assert rc == wd.WD_OK and info[0]["true_rel_resid"] <= 1e-10
        assert rel(lo.cpu().numpy(), x.cpu().numpy()) < 1e-8
    lat.close()
