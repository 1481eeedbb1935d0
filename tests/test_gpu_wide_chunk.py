"""One chunk of more map sets than fit a single pass: with the ring classes in one launch
its grid would pass 2^32 threads, and an m's rows 4 GiB."""
import pytest

from .gpu_util import note

pytestmark = pytest.mark.gpu


def test_chunk_wider_than_one_pass():
    """6.3 million T maps at nside 11, lmax 0 (two ring classes, 43 rings: 2^23 workgroups
    of 16 map pairs at 6.24 million).  A constant map's a_00 is its value times sqrt(4 pi)."""
    import math

    import torch
    from paper_2208_10154_amd import sht
    n, nside = 6_300_000, 11
    npix = 12 * nside * nside
    if torch.cuda.mem_get_info()[0] < 1.3 * 8 * n * npix:
        pytest.skip("needs 95 GB of device memory")
    note("6.3 million maps in one chunk")
    p = sht.Plan(nside, 0, 0, n, chunk=n)
    want = torch.arange(n, dtype=torch.float64, device="cuda") + 1.0
    maps = want.view(n, 1, 1).expand(n, 1, npix).contiguous()
    alm = torch.full((n, 1, 1), math.nan, dtype=torch.float64, device="cuda")
    p.map2alm(maps, alm)
    p.sync()
    assert ((alm.view(n) / (want * math.sqrt(4 * math.pi)) - 1).abs() < 1e-13).all()
    maps.fill_(math.nan)
    p.alm2map(alm, maps)
    p.sync()
    p.close()
    low, high = torch.aminmax(maps.view(n, npix), dim=1)
    assert ((low / want - 1).abs() < 1e-13).all() and ((high / want - 1).abs() < 1e-13).all()
    del maps, alm, want, low, high
    torch.cuda.empty_cache()
