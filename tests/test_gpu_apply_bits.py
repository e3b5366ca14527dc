"""The operator on canonical spinors gives the bits of an import, wd_dslash and an
export, and a batch those of its single calls: on both sides of the size at which
the float64 form marches and float32 imports (65536 sites over all rhs), over whole
and part tiles, with links of 12 and of 18 reals.
"""
import pytest
import torch

from gpu_util import gauge
import synth

pytestmark = pytest.mark.gpu

# (dims, nrhs): below the line; across it (single below, batch above); above
CASES = [((2, 2, 2, 2), 12), ((8, 8, 8, 8), 3), ((16, 16, 16, 8), 2), ((14, 18, 14, 4), 5),
         ((10, 10, 10, 10), 12), ((18, 18, 18, 12), 2)]


@pytest.mark.parametrize("dims,nrhs", CASES)
@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
@pytest.mark.parametrize("group", [True, False])
def test_apply_bits(dims, nrhs, prec, group):
    import paper_1810_04201_amd as wd
    print(f"apply bits dims={dims} nrhs={nrhs} prec={prec} group={group}", flush=True)
    lat = wd.Lattice(dims)
    U = torch.from_numpy(gauge(dims, 67)).cuda()
    lat.set_gauge(U if group else U * (1.0 + 1e-9))
    assert lat.links_info()[0] == (12 if group else 18)
    b = torch.from_numpy(synth.gaussian_sources(dims, list(range(20, 20 + nrhs)))).cuda()
    fi, fo = wd.Field(lat, prec, nrhs), wd.Field(lat, prec, nrhs)
    fi.load(b)
    for dagger in (0, 1):
        want, got = torch.empty_like(b), torch.full_like(b, float("nan"))
        wd.wd_dslash(lat, 0.124, dagger, fi, fo)
        fo.store(want)
        lat.apply(0.124, b, got, prec=prec, dagger=dagger, nrhs=nrhs)
        assert torch.equal(got, want)
        for k in (0, nrhs - 1):
            one = torch.full_like(b[k], float("nan"))
            lat.apply(0.124, b[k].contiguous(), one, prec=prec, dagger=dagger)
            assert torch.equal(got[k], one)
    fi.close()
    fo.close()
    lat.close()
