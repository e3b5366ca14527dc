"""Binary16 operators and solves of a batch are the single ones bit for bit where
the chunk lengths could differ between them: the roundings of the first slice of a
chunk are not those of the others.  12^3 x 24, 16^4 and 24^3 x 16 take chunks of one
slice, which do not all fit the chip at once in a batch; 18^3 x 10 has bricks of part
tiles, whose chunks would be longer in a batch."""
import pytest
import torch

from gpu_util import gauge
import synth

pytestmark = pytest.mark.gpu

CASES = [((12, 12, 12, 24), 12), ((16, 16, 16, 16), 12), ((18, 18, 18, 10), 12),
         ((24, 24, 24, 16), 3)]


@pytest.mark.parametrize("dims,nrhs", CASES)
def test_batch_is_its_singles(dims, nrhs):
    import paper_1810_04201_amd as wd
    print(f"f16 batch dims={dims} nrhs={nrhs}", flush=True)
    lat = wd.Lattice(dims)
    lat.set_gauge(torch.from_numpy(gauge(dims, 66)).cuda())
    b = torch.from_numpy(synth.gaussian_sources(dims, list(range(30, 30 + nrhs)))).cuda()
    out, x = torch.empty_like(b), torch.zeros_like(b)
    lat.apply(0.12, b, out, prec="f16", nrhs=nrhs)
    rc, info = lat.solve(b, x, 0.12, prec="f16", nrhs=nrhs)
    assert rc == wd.WD_OK
    for k in (0, nrhs - 1):
        one, y = torch.empty_like(b[k]), torch.zeros_like(b[k])
        lat.apply(0.12, b[k].contiguous(), one, prec="f16")
        rc, single = lat.solve(b[k].contiguous(), y, 0.12, prec="f16")
        torch.cuda.synchronize()
        assert rc == wd.WD_OK and single[0]["iters"] == info[k]["iters"]
        assert torch.equal(out[k], one) and torch.equal(x[k], y)
    lat.close()
