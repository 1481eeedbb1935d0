"""FP64 map2alm of few, short chains: rings split over a block's waves, or the LDS kernels'
wider column tiles.  Values on both sides of each line against chunks of 4 map sets (which
split), of whole and part plans; and more maps never take less time than fewer."""
import time

import pytest

from .gpu_util import note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spin,nside,lmax,n,nparts", [
    (0, 20, 79, 48, 1), (0, 20, 79, 56, 1),     # 6 and 7 column tiles: the line of 550 blocks
    (0, 16, 60, 120, 1), (0, 16, 60, 128, 1),   # 15 and 16: 950 blocks, 256-column tiles
    (2, 9, 32, 168, 1), (2, 9, 32, 176, 1),     # 42 and 44: 1400 blocks
    (2, 16, 60, 100, 1), (2, 18, 70, 64, 1),    # spin 0 alone splits; spin 2 takes it along
    (2, 64, 150, 20, 1), (2, 64, 150, 48, 1),   # past the line, by the work that padding adds
    (0, 20, 79, 56, 3), (2, 16, 60, 100, 2)])
def test_both_sides_of_the_line(spin, nside, lmax, n, nparts):
    import torch
    from paper_2208_10154_amd import sht
    note(f"m2a split spin={spin} nside={nside} lmax={lmax} nmaps={n} parts={nparts}")
    g = torch.Generator(device="cuda")
    g.manual_seed(nside + n)
    p = sht.Plan(nside, lmax, spin, n, chunk=4)
    maps = torch.randn(p.map_shape(), generator=g, dtype=torch.float64, device="cuda")
    want = torch.empty(p.alm_shape(), dtype=torch.float64, device="cuda")
    p.map2alm(maps, want)
    p.sync()
    p.close()
    got = torch.full_like(want, torch.nan)
    for k in range(nparts):
        p = sht.Plan(nside, lmax, spin, n, **({} if nparts == 1 else dict(part=k, nparts=nparts)))
        p.map2alm(maps, got)
        p.sync()
        p.close()
    assert ((got - want).norm(dim=-1) <= 1e-12 * want.norm(dim=-1)).all()


def test_fewer_maps_take_no_longer():
    """Splitting 400 T maps at nside 16, lmax 47 took 55 us where 512, not split, took 41."""
    import torch
    from paper_2208_10154_amd import sht
    note("m2a time of 400 and 512 maps")
    plans = [sht.Plan(16, 47, 0, n) for n in (400, 512)]
    bufs = [(torch.zeros(p.map_shape(), dtype=torch.float64, device="cuda"),
             torch.zeros(p.alm_shape(), dtype=torch.float64, device="cuda")) for p in plans]
    best = [float("inf")] * 2
    for _ in range(10):
        for i, (p, b) in enumerate(zip(plans, bufs)):
            p.map2alm(*b)
            p.sync()
            t = time.perf_counter()
            for _ in range(10):
                p.map2alm(*b)
            p.sync()
            best[i] = min(best[i], time.perf_counter() - t)
    for p in plans:
        p.close()
    assert best[0] <= 1.1 * best[1], best


@pytest.mark.parametrize("spin,nside,lmax,n", [(0, 8, 23, 3000), (2, 16, 47, 601)])
def test_wide_immediate_levels(spin, nside, lmax, n):
    """the levels of a wide immediate iteration (few orders, many columns) against chunks of 32"""
    import torch
    from paper_2208_10154_amd import sht
    note(f"immediate spin={spin} nside={nside} lmax={lmax} nmaps={n}")
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    out = []
    for chunk in (n, 32):
        p = sht.Plan(nside, lmax, spin, n, chunk=chunk)
        if not out:
            maps = torch.randn(p.map_shape(), generator=g, dtype=torch.float64, device="cuda")
        out.append(torch.full(p.alm_shape(), torch.nan, dtype=torch.float64, device="cuda"))
        p.map2alm_immediate(maps, out[-1], 2)
        p.sync()
        p.close()
    assert ((out[0] - out[1]).norm(dim=-1) <= 1e-12 * out[1].norm(dim=-1)).all()
