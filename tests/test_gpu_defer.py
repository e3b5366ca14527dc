"""CG iterations whose reductions the next kernels finish (small lattices),
against the oracle and against themselves.

The sums are taken by the r update and by the x and p update themselves when a
reduction has at most four partials per thread of the smaller workgroup; the
lattices lie on both sides of that line and at its edges (one partial; one
more than a wave's share).  Frozen, failed and converged sources of a batch must
not disturb the others, whenever their workgroups start: the batches repeat on
busy streams and must be the single solves bit for bit.
"""
import numpy as np
import pytest

import synth
from oracle import cg, evenodd, wilson
from gpu_util import assert_same_count_parity, gauge

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch

    import paper_1810_04201_amd as wd
    assert torch.cuda.is_available()
    return torch, torch.device("cuda:0"), wd


def _lat(env, dims, seed):
    torch, dev, wd = env
    lat = wd.Lattice(dims)
    U = gauge(dims, seed)
    lat.set_gauge(torch.from_numpy(U).to(dev))
    return lat, U


# partials of a float64 reduction: 4, 16, 18 (ragged), 260 (64-lane groups: one
# more than they take), 96
@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (4, 4, 4, 16), (6, 6, 6, 18), (4, 4, 4, 260),
                                  (8, 8, 12, 8)])
@pytest.mark.parametrize("even_odd", [False, True])
def test_iterate_matches_oracle(env, dims, even_odd):
    torch, dev, wd = env
    print(f"defer dims={dims} even_odd={even_odd}", flush=True)
    lat, U = _lat(env, dims, 91)
    b = synth.gaussian_spinor(dims, 92)
    bd = torch.from_numpy(b).to(dev)
    for n in (1, 7):
        x = torch.zeros_like(bd)
        rc, info = lat.solve(bd, x, 0.12, tol=1e-14, max_iter=n, even_odd=even_odd)
        assert rc == wd.WD_ERR_NOCONV and info[0]["iters"] == n
        if even_odd:
            want, _, _ = evenodd.solve(U, b, dims, 0.12, tol=1e-300, max_iter=n)
        else:
            want, _, _ = cg.cgnr(lambda v: wilson.apply_D(U, v, dims, 0.12),
                                 lambda v: wilson.apply_Ddag(U, v, dims, 0.12), b, tol=1e-300,
                                 max_iter=n)
        assert_same_count_parity(x.cpu().numpy(), want, 1e-11)
    lat.close()


@pytest.mark.parametrize("prec,even_odd", [("f64", False), ("f32", False), ("f16", False),
                                           ("f64", True), ("f32", True), ("f16", True)])
def test_batch_equals_singles_on_busy_streams(env, prec, even_odd):
    """Sources that converge at different iterations, a zero one and one with a
    NaN, batched on several streams at once."""
    torch, dev, wd = env
    dims = (12, 12, 12, 12)
    print(f"defer batch prec={prec} even_odd={even_odd}", flush=True)
    lat, _ = _lat(env, dims, 93)
    V = 12 ** 4
    src = synth.gaussian_sources(dims, [1, 2, 3, 4, 5])
    src[1] = synth.point_source(dims, 2, 1, 77)
    src[2] = 0.0
    b = torch.from_numpy(src).to(dev)
    bad = b.clone()
    bad[3, 0, 0, 0, 0] = float("nan")
    ones = []
    for k in range(5):
        x = torch.zeros_like(b[k])
        rc, _ = lat.solve(b[k].contiguous(), x, 0.123, prec=prec, even_odd=even_odd)
        assert rc == wd.WD_OK
        ones.append(x)
    srv = wd.Server(hbm_budget_bytes=16 << 30, max_active=6)
    for rep in range(3):
        xs = [torch.full_like(b, float("nan")) for _ in range(6)]
        tick = [srv.submit(lat, bad if k % 2 else b, xs[k], 0.123, prec=prec, nrhs=5,
                           even_odd=even_odd) for k in range(6)]
        infos = []
        for t in tick:
            rc, info = srv.poll(t)
            while rc == wd.WD_PENDING:
                rc, info = srv.poll(t)
            infos.append((rc, info))
        torch.cuda.synchronize()
        for k, (rc, info) in enumerate(infos):
            for r in range(5):
                if k % 2 and r == 3:
                    assert info[r]["status"] == wd.WD_ERR_NUMERIC
                else:
                    assert info[r]["status"] == wd.WD_OK
                    assert torch.equal(xs[k][r], ones[r]), (rep, k, r)
    srv.close()
    assert V * 24 == b[0].numel()
    lat.close()
