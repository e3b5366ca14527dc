"""The stencil on canonical spinors (wd_apply in float64 and float32) against
the same operator on resident fields (import, wd_dslash, export) and the
oracle.

Sizes sit at the edges of the kernel's shapes: bricks of one part and of
several, a last part with fewer sites, parts that are no multiple of 64 sites,
one site more or less than a wave, lattices below and above the size where the
marching form starts, one and several right-hand sides.  The arithmetic is the
fields' own, so the outputs agree to a rounding of the output: 4 units of the
compute type on each site's norm.
"""
import numpy as np
import pytest

import synth
from oracle import wilson
from gpu_util import gauge, site_rel_err

pytestmark = pytest.mark.gpu

ULP = {"f64": 2.0 ** -52, "f32": 2.0 ** -23}


@pytest.fixture(scope="module")
def env():
    import torch

    import paper_1810_04201_amd as wd
    assert torch.cuda.is_available()
    return torch, torch.device("cuda:0"), wd


def _field_path(wd, torch, lat, kappa, b, prec, dagger, nrhs):
    fi, fo = wd.Field(lat, prec, nrhs), wd.Field(lat, prec, nrhs)
    fi.load(b)
    wd.wd_dslash(lat, kappa, dagger, fi, fo)
    out = torch.empty_like(b)
    fo.store(out)
    torch.cuda.synchronize()
    fi.close()
    fo.close()
    return out


# (dims, brick or None, nrhs): 8^4 and 6x10x14x4 lie below the marching size;
# 18^3x12 and 22^3x8 march over bricks that are no multiple of 64; the forced
# bricks give parts of 192 + 192 + 156, 65, 63 and 36 sites
CASES = [((8, 8, 8, 8), None, 1), ((6, 10, 14, 4), None, 3), ((2, 2, 2, 2), None, 2),
         ((18, 18, 18, 12), None, 1), ((22, 22, 22, 8), None, 1), ((30, 6, 18, 24), "30,6,3", 1),
         ((10, 26, 10, 26), "10,13,1", 2), ((14, 18, 14, 20), "14,9,1", 1),
         ((18, 16, 18, 14), "18,2,1", 1), ((16, 16, 16, 18), None, 12)]


@pytest.mark.parametrize("dims,brick,nrhs", CASES)
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_apply_equals_field_path(env, monkeypatch, dims, brick, nrhs, prec):
    torch, dev, wd = env
    print(f"apply dims={dims} brick={brick} nrhs={nrhs} prec={prec}", flush=True)
    if brick:
        monkeypatch.setenv("WD_BRICK", brick)
    V = int(np.prod(dims))
    lat = wd.Lattice(dims)
    U = gauge(dims, 31)
    lat.set_gauge(torch.from_numpy(U).to(dev))
    src = synth.gaussian_sources(dims, [40 + k for k in range(nrhs)])
    b = torch.from_numpy(src).to(dev)
    for dagger in (0, 1):
        want = _field_path(wd, torch, lat, 0.124, b, prec, dagger, nrhs)
        got = torch.full_like(b, float("nan"))
        lat.apply(0.124, b, got, prec=prec, dagger=dagger, nrhs=nrhs)
        torch.cuda.synchronize()
        assert site_rel_err(got.cpu().numpy(), want.cpu().numpy()) <= 4 * ULP[prec]
        if V <= 40000:
            ref = (wilson.apply_Ddag if dagger else wilson.apply_D)(U, src[-1], dims, 0.124)
            tol = 1e-13 if prec == "f64" else 1e-5
            assert site_rel_err(got[-1].cpu().numpy(), ref) < tol
    lat.close()


@pytest.mark.parametrize("antiperiodic", [True, False])
def test_apply_boundary_and_18_real_links(env, antiperiodic):
    """Links off SU(3) keep 18 reals; both t boundaries; marching size."""
    torch, dev, wd = env
    dims = (18, 18, 18, 12)
    lat = wd.Lattice(dims, antiperiodic)
    U = gauge(dims, 32) * (1.0 + 1e-9)
    lat.set_gauge(torch.from_numpy(U).to(dev))
    assert lat.links_info()[0] == 18
    src = synth.gaussian_spinor(dims, 50)
    b = torch.from_numpy(src).to(dev)
    got = torch.full_like(b, float("nan"))
    lat.apply(0.12, b, got)
    torch.cuda.synchronize()
    assert torch.equal(got, _field_path(wd, torch, lat, 0.12, b, "f64", 0, 1)) or \
        site_rel_err(got.cpu().numpy(),
                     _field_path(wd, torch, lat, 0.12, b, "f64", 0, 1).cpu().numpy()) <= 2.0 ** -50
    ref = wilson.apply_D(U, src, dims, 0.12, antiperiodic_t=antiperiodic)
    assert site_rel_err(got.cpu().numpy(), ref) < 1e-13
    lat.close()


def test_apply_tensors_off_16_bytes(env):
    """Buffers aligned to a double only take the general path."""
    torch, dev, wd = env
    dims = (8, 8, 8, 8)
    n = 8 ** 4 * 24
    lat = wd.Lattice(dims)
    U = gauge(dims, 33)
    lat.set_gauge(torch.from_numpy(U).to(dev))
    src = synth.gaussian_spinor(dims, 51)
    buf = torch.zeros(n + 1, dtype=torch.float64, device=dev)
    buf[1:] = torch.from_numpy(src).to(dev).reshape(-1)
    obuf = torch.full((n + 1,), float("nan"), dtype=torch.float64, device=dev)
    lat.apply(0.12, buf[1:], obuf[1:])
    torch.cuda.synchronize()
    ref = wilson.apply_D(U, src, dims, 0.12)
    assert site_rel_err(obuf[1:].cpu().numpy(), ref) < 1e-13
    lat.close()


@pytest.mark.parametrize("dims,nrhs", [((8, 8, 8, 8), 1), ((4, 6, 8, 10), 3), ((2, 4, 2, 6), 2),
                                       ((6, 10, 14, 4), 1), ((18, 6, 6, 10), 2)])
@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
def test_schur_output_forms_agree(env, dims, nrhs, prec):
    """The even-odd operator with its result written canonically by the second
    launch (odd sites zero) and through separate exports (a buffer aligned to a
    double only): the same bits; brick slices of whole tiles and not, one lane
    per site and marching."""
    torch, dev, wd = env
    print(f"schur dims={dims} nrhs={nrhs} prec={prec}", flush=True)
    V = int(np.prod(dims))
    lat = wd.Lattice(dims)
    lat.set_gauge(torch.from_numpy(gauge(dims, 35)).to(dev))
    b = torch.from_numpy(synth.gaussian_sources(dims, [60 + k for k in range(nrhs)])).to(dev)
    off = torch.zeros(b.numel() + 1, dtype=torch.float64, device=dev)
    off[1:] = b.reshape(-1)
    for dagger in (0, 1):
        got = torch.full_like(b, float("nan"))
        lat.apply_schur(0.12, b, got, prec=prec, dagger=dagger, nrhs=nrhs)
        obuf = torch.full((b.numel() + 1,), float("nan"), dtype=torch.float64, device=dev)
        lat.apply_schur(0.12, off[1:], obuf[1:], prec=prec, dagger=dagger, nrhs=nrhs)
        torch.cuda.synchronize()
        assert torch.equal(got.reshape(-1), obuf[1:])
        par = np.indices(dims[::-1]).sum(axis=0).reshape(-1) % 2
        out = got.cpu().numpy().reshape(nrhs, V, 24)
        assert np.all(out[:, par == 1] == 0.0) and np.all(np.any(out[:, par == 0] != 0.0, axis=2))
    lat.close()


@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
@pytest.mark.parametrize("dims,nrhs", [((2, 2, 2, 2), 1), ((4, 4, 4, 4), 5), ((6, 2, 2, 4), 3),
                                       ((14, 10, 6, 8), 2)])
def test_export_forms_agree(env, dims, nrhs, prec):
    """A field's export through LDS (fields of part of a tile, of whole ones, of
    ragged ones) writes what the per-lane one writes to a buffer aligned to a
    double only, and nothing around it; the conversions there and back are exact in
    float64 and one rounding in float32."""
    torch, dev, wd = env
    print(f"export dims={dims} nrhs={nrhs} prec={prec}", flush=True)
    lat = wd.Lattice(dims)
    n = nrhs * int(np.prod(dims)) * 24
    src = torch.from_numpy(np.random.default_rng(11).standard_normal(n)).to(dev)
    f = wd.Field(lat, prec, nrhs)
    f.load(src)
    even = torch.full((n + 64,), -7.0, dtype=torch.float64, device=dev)
    odd = torch.full((n + 64,), -7.0, dtype=torch.float64, device=dev)
    f.store(even[32:32 + n])
    f.store(odd[33:33 + n])
    torch.cuda.synchronize()
    assert torch.equal(even[32:32 + n], odd[33:33 + n])
    for buf, k in ((even, 32), (odd, 33)):
        assert bool((buf[:k] == -7.0).all()) and bool((buf[k + n:] == -7.0).all())
    if prec == "f64":
        assert torch.equal(even[32:32 + n], src)
    elif prec == "f32":
        assert torch.equal(even[32:32 + n], src.float().double())
    f.close()
    lat.close()


@pytest.mark.parametrize("dims", [(4, 4, 4, 4), (16, 16, 16, 16)])
def test_apply_overlapping_fields(env, dims):
    """Fields that share memory (two rhs against their neighbours' places): the
    same result as with separate ones, one lane per site and marching."""
    torch, dev, wd = env
    print(f"overlap dims={dims}", flush=True)
    V = int(np.prod(dims))
    lat = wd.Lattice(dims)
    lat.set_gauge(torch.from_numpy(gauge(dims, 36)).to(dev))
    src = torch.from_numpy(synth.gaussian_sources(dims, [71, 72])).to(dev).reshape(-1)
    ref = torch.empty_like(src)
    lat.apply(0.12, src, ref, nrhs=2)
    buf = torch.zeros(3 * V * 24, dtype=torch.float64, device=dev)
    buf[:2 * V * 24] = src
    lat.apply(0.12, buf[:2 * V * 24], buf[V * 24:], nrhs=2)
    torch.cuda.synchronize()
    err = (buf[V * 24:] - ref).norm() / ref.norm()
    assert float(err) < 1e-15
    lat.close()
