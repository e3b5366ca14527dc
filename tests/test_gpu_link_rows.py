"""Float64 operators on lattices whose bricks are no whole 64-site tiles read all
18 reals of the caller's links, also where the links pass the check for 12: with
row 2 longer by 9e-15 (the limit is 1e-14), rebuilding it from rows 0 and 1 moves D
by over 3e-15 per site.

The bar: a site is a sum of eight hops of about seven roundings each; 15 roundings
in a row at half a unit are 1.7e-15 in the worst case, and both sides stay below
half of that.
"""
import numpy as np
import pytest

import synth
from oracle import wilson
from gpu_util import gauge, site_rel_err

pytestmark = pytest.mark.gpu

BAR = 1.5e-15


@pytest.mark.parametrize("dims", [(6, 10, 14, 4), (2, 2, 2, 2), (18, 18, 6, 4), (10, 10, 10, 10)])
def test_row_2_is_the_callers(dims):
    import torch

    import paper_1810_04201_amd as wd
    print(f"row 2 dims={dims}", flush=True)
    U = gauge(dims, 31)
    short = U.copy()
    U.reshape(-1, 3, 3, 2)[:, 2] *= 1.0 + 9e-15
    src = synth.gaussian_sources(dims, list(range(5, 12)))
    want = np.stack([wilson.apply_D(U, s, dims, 0.124) for s in src])
    rebuilt = np.stack([wilson.apply_D(short, s, dims, 0.124) for s in src])
    assert site_rel_err(rebuilt, want) > 2 * BAR
    lat = wd.Lattice(dims)
    lat.set_gauge(torch.from_numpy(U).cuda())
    b = torch.from_numpy(src).cuda()
    n = len(src)
    fi, fo = wd.Field(lat, "f64", n), wd.Field(lat, "f64", n)
    fi.load(b)
    wd.wd_dslash(lat, 0.124, 0, fi, fo)
    fields, direct = torch.empty_like(b), torch.empty_like(b)
    fo.store(fields)
    lat.apply(0.124, b, direct, nrhs=n)
    torch.cuda.synchronize()
    for got in (fields, direct):
        assert site_rel_err(got.cpu().numpy(), want) < BAR
    fi.close()
    fo.close()
    lat.close()
