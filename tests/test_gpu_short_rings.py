"""Ring FFTs of wide batches at small nside: the classes of up to 60 and of 64 pixels leave
the shared launch from 4096 workgroups on, and a grid of one class never takes it.  The same
maps in chunks of 32 run the shared launch; odd batches end in half a map pair."""
import pytest

from .gpu_util import note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-12), ("fp32", 4e-6)])
@pytest.mark.parametrize("nside,lmax,spin,n", [
    (1, 3, 2, 4097), (8, 23, 2, 41), (8, 23, 0, 1501), (12, 35, 2, 1001), (14, 20, 0, 4001), (16, 47, 2, 1401), (16, 47, 0, 4201)])
def test_wide_batch_equals_narrow_chunks(nside, lmax, spin, n, prec, tol):
    import torch
    from paper_2208_10154_amd import sht
    note(f"short rings nside={nside} lmax={lmax} spin={spin} nmaps={n} {prec}")
    g = torch.Generator(device="cuda")
    g.manual_seed(nside + n)
    wide = sht.Plan(nside, lmax, spin, n, chunk=n, precision=prec)
    narrow = sht.Plan(nside, lmax, spin, n, chunk=32, precision=prec)
    maps = torch.randn(wide.map_shape(), generator=g, dtype=torch.float64, device="cuda")
    got = torch.full(wide.alm_shape(), torch.nan, dtype=torch.float64, device="cuda")
    want = torch.empty_like(got)
    wide.map2alm(maps, got)
    narrow.map2alm(maps, want)
    assert ((got - want).norm(dim=-1) <= tol * want.norm(dim=-1)).all()
    back = torch.empty_like(maps)
    narrow.alm2map(want, back)
    maps.fill_(torch.nan)
    wide.alm2map(want, maps)
    assert ((maps - back).norm(dim=-1) <= tol * back.norm(dim=-1)).all()
    wide.close()
    narrow.close()
