"""Solves whose caller asks for reliable updates more often than the gated ones
are launched by default (reliable_max_iter 1 to 3, a delta near 1): the solution of
the float64 solve, and an update after every reliable_max_iter iterations.  The last
case is a large one (2^20 sites over its rhs)."""
import pytest
import torch

from gpu_util import gauge, rel
import synth

pytestmark = pytest.mark.gpu

CASES = [((4, 4, 4, 4), 1, False), ((4, 4, 4, 4), 2, True), ((6, 10, 14, 4), 1, False),
         ((16, 16, 16, 32), 8, True)]


@pytest.mark.parametrize("dims,nrhs,even_odd", CASES)
@pytest.mark.parametrize("prec", ["f32", "f16"])
def test_frequent_updates(dims, nrhs, even_odd, prec):
    import paper_1810_04201_amd as wd
    print(f"updates dims={dims} nrhs={nrhs} even_odd={even_odd} prec={prec}", flush=True)
    lat = wd.Lattice(dims)
    lat.set_gauge(torch.from_numpy(gauge(dims, 68)).cuda())
    b = torch.from_numpy(synth.gaussian_sources(dims, list(range(50, 50 + nrhs)))).cuda()
    want = torch.zeros_like(b)
    rc, _ = lat.solve(b, want, 0.12, tol=1e-11, nrhs=nrhs, even_odd=even_odd)
    assert rc == wd.WD_OK
    for kw in (dict(reliable_max_iter=1), dict(reliable_max_iter=3), dict(reliable_delta=0.9)):
        x = torch.zeros_like(b)
        rc, info = lat.solve(b, x, 0.12, prec=prec, nrhs=nrhs, even_odd=even_odd, **kw)
        assert rc == wd.WD_OK
        every = kw.get("reliable_max_iter", 50)
        for i in info:
            assert i["true_rel_resid"] <= 1e-10
            assert i["reliable_updates"] >= 1 + i["iters"] / every
        # 1e-10 of the normal equations' residual each: 1e-8 of the solution, as
        # for the other mixed solves
        assert rel(x.cpu().numpy(), want.cpu().numpy()) < 1e-8
    lat.close()
