"""FP64 map2alm of part plans over several l tiles and deals of orders: values against the
whole plan's, and a part's time against its share of the whole plan's."""
import numpy as np
import pytest

from .gpu_util import from_dev, note, rel_rms


@pytest.mark.parametrize("nparts", [2, 3, 4, 5, 8, 16])
def test_owned_orders_grow_by_the_number_of_parts(nparts):
    """the i-th order of a part is at least nparts (i - 1): the bound the kernels size their
    grid by"""
    from paper_2208_10154_amd import sht
    for lmax in range(3, 130):
        for part in range(nparts):
            own = sht.part_orders(lmax, part, nparts)
            assert all(m >= nparts * (i - 1) for i, m in enumerate(own))


@pytest.fixture(scope="module")
def sht():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2208_10154_amd import sht as mod
    mod.lib()
    return mod


# lists of fewer and of more than 128 orders, one to six l tiles, every tile of the dispatch
@pytest.mark.gpu
@pytest.mark.parametrize("spin,nside,lmax,nmaps,nparts,precision", [
    (2, 96, 383, 1, 2, "fp64"), (2, 96, 300, 2, 3, "fp64"), (0, 256, 767, 3, 4, "fp64"), (2, 128, 511, 9, 3, "fp64"),
    (0, 128, 383, 40, 2, "fp64"), (0, 64, 255, 7, 16, "fp64"), (2, 256, 700, 17, 5, "fp64"), (2, 256, 767, 70, 2, "fp32")])
def test_part_map2alm_equals_the_whole(sht, spin, nside, lmax, nmaps, nparts, precision):
    import torch
    note(f"part map2alm spin={spin} nside={nside} lmax={lmax} nmaps={nmaps} nparts={nparts} {precision}")
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    p = sht.Plan(nside, lmax, spin, nmaps, precision=precision)
    maps = torch.randn(p.map_shape(), generator=g, dtype=torch.float64, device="cuda")
    whole = torch.full(p.alm_shape(), np.nan, dtype=torch.float64, device="cuda")
    p.map2alm(maps, whole)
    p.sync()
    p.close()
    alm = torch.full(whole.shape, np.nan, dtype=torch.float64, device="cuda")
    for k in range(nparts):
        p = sht.Plan(nside, lmax, spin, nmaps, precision=precision, part=k, nparts=nparts)
        p.map2alm(maps, alm)
        p.sync()
        p.close()
    assert rel_rms(from_dev(alm), from_dev(whole)).max() < 1e-12


@pytest.mark.gpu
@pytest.mark.parametrize("part", [0, 3])
def test_part_map2alm_takes_its_share_of_the_time(sht, part):
    """One of eight parts at nside 512, two IQU sets: an eighth of the whole plan's Legendre
    time when its work is spread over the chip, several eighths when it runs on the XCDs
    that its orders' residues name.  The line lies at three eighths."""
    import torch
    note(f"time of part {part} of 8")

    def legendre_ms(**kw):
        p = sht.Plan(512, 1535, 2, 2, **kw)
        maps = torch.ones(p.map_shape(), dtype=torch.float64, device="cuda")
        alm = torch.zeros(p.alm_shape(), dtype=torch.float64, device="cuda")
        p.map2alm(maps, alm)
        p.set_profiling(True)
        best = np.inf
        for _ in range(5):
            p.profile(reset=True)
            p.map2alm(maps, alm)
            t = p.profile(reset=True)
            best = min(best, t["m2a_spin0"][0] + t["m2a_spin2"][0])
        p.close()
        return best

    assert legendre_ms(part=part, nparts=8) < 3 / 8 * legendre_ms()
