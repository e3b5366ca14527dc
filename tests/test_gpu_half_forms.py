"""The float64 even-odd operator on half slices that are no whole tiles, marching and
one lane per site (WD_EO_SITE=1): the same bits, and the oracle's result; solves in
the marching form against the oracle's iterate, batched against single.  Such lattices
march from 12 time slices on, below 32768 sites or from 200000."""
import numpy as np
import pytest
import torch

import synth
from oracle import evenodd
from gpu_util import assert_same_count_parity, gauge, site_rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(10, 10, 10, 12), (6, 6, 6, 20), (30, 6, 2, 14),
                                  (26, 26, 26, 12)])
@pytest.mark.parametrize("group", [True, False])
def test_operator_forms_agree(monkeypatch, dims, group):
    import paper_1810_04201_amd as wd
    print(f"half forms dims={dims} group={group}", flush=True)
    lat = wd.Lattice(dims)
    U = gauge(dims, 71) * (1.0 if group else 1.0 + 1e-9)
    lat.set_gauge(torch.from_numpy(U).cuda())
    src = synth.gaussian_sources(dims, [80, 81])
    b = torch.from_numpy(src).cuda()
    for dagger in (0, 1):
        out = []
        for site in ("0", "1"):
            monkeypatch.setenv("WD_EO_SITE", site)
            out.append(torch.full_like(b, float("nan")))
            lat.apply_schur(0.124, b, out[-1], dagger=dagger, nrhs=2)
            torch.cuda.synchronize()
        assert torch.equal(out[0], out[1])
        if lat.volume < 32768:
            want = evenodd.apply_M(U, src[1], dims, 0.124, bool(dagger))
            even = evenodd.parity(dims) == 0
            assert site_rel_err(out[0][1].cpu().numpy()[even], want[even]) < 1e-13
    lat.close()


@pytest.mark.parametrize("dims", [(6, 6, 6, 20), (30, 6, 2, 14)])
def test_solves(dims):
    import paper_1810_04201_amd as wd
    print(f"half forms solve dims={dims}", flush=True)
    lat = wd.Lattice(dims)
    U = gauge(dims, 72)
    lat.set_gauge(torch.from_numpy(U).cuda())
    src = synth.gaussian_sources(dims, [82, 83, 84])
    b = torch.from_numpy(src).cuda()
    x = torch.zeros_like(b)
    rc, info = lat.solve(b, x, 0.12, nrhs=3, even_odd=True)
    assert rc == wd.WD_OK
    want, _, _ = evenodd.solve(U, src[2], dims, 0.12, tol=1e-300, max_iter=info[2]["iters"])
    assert_same_count_parity(x[2].cpu().numpy(), want)
    one = torch.zeros_like(b[2])
    rc, _ = lat.solve(b[2].contiguous(), one, 0.12, even_odd=True)
    assert rc == wd.WD_OK and torch.equal(one, x[2])
    lat.close()
