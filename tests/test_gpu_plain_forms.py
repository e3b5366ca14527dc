"""Plain applications on bricks of part tiles, one lane per site and marching: the
same bits.  A batch and its single calls lie on different sides of each line between
the two forms (ragged_marches in csrc/march.hpp)."""
import pytest
import torch

from gpu_util import gauge
import synth

pytestmark = pytest.mark.gpu

# float64 3360 sites march, 12 x 3360 do not; 38416 do not, 2 x 38416 do; 10000 march,
# 12 x 10000 do not; float32 104976 do not, 12 x 104976 do; 209952 do
CASES = [("f64", (6, 10, 14, 4), 12), ("f64", (14, 14, 14, 14), 2), ("f64", (10, 10, 10, 10), 12),
         ("f32", (18, 18, 18, 18), 12), ("f32", (18, 18, 18, 36), 2)]


@pytest.mark.parametrize("prec,dims,nrhs", CASES)
def test_forms_agree(prec, dims, nrhs):
    import paper_1810_04201_amd as wd
    print(f"plain forms prec={prec} dims={dims} nrhs={nrhs}", flush=True)
    lat = wd.Lattice(dims)
    lat.set_gauge(torch.from_numpy(gauge(dims, 69)).cuda())
    b = torch.from_numpy(synth.gaussian_sources(dims, list(range(70, 70 + nrhs)))).cuda()

    def dslash(src, n, dagger):
        fi, fo = wd.Field(lat, prec, n), wd.Field(lat, prec, n)
        fi.load(src)
        wd.wd_dslash(lat, 0.124, dagger, fi, fo)
        out = torch.full_like(src, float("nan"))
        fo.store(out)
        torch.cuda.synchronize()
        fi.close()
        fo.close()
        return out

    for dagger in (0, 1):
        batch = dslash(b, nrhs, dagger)
        direct = torch.full_like(b, float("nan"))
        lat.apply(0.124, b, direct, prec=prec, dagger=dagger, nrhs=nrhs)
        assert torch.equal(direct, batch)
        for k in (0, nrhs - 1):
            assert torch.equal(dslash(b[k].contiguous(), 1, dagger), batch[k])
    lat.close()
