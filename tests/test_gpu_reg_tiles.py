"""Register-operand Legendre kernels (k_leg_reg.hip) at the edges of their tiles: map
counts around the 4- and 8-map column tiles, l ranges around the 8-row segments, ring
counts below one 16-ring tile, E or B alone; and the routes of the dispatch against
each other (the same maps in a wide batch and in small ones)."""
import numpy as np
import pytest

import oracle
from paper_2208_10154_amd import synth

from .gpu_util import alm_inputs, from_dev, note, rel_rms, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sht():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2208_10154_amd import sht as mod
    mod.lib()
    return mod


@pytest.mark.parametrize("spin,nside,lmax,nmaps", [
    (2, 1, 2, 1), (2, 2, 7, 4), (2, 5, 9, 5), (2, 24, 71, 2), (2, 7, 20, 3), (0, 24, 71, 3), (0, 13, 38, 4), (2, 8, 31, 8), (2, 12, 25, 13), (2, 24, 71, 33),
    (0, 1, 0, 1), (0, 3, 8, 9), (0, 9, 16, 17), (0, 24, 71, 40)])
def test_tile_edges_against_the_oracle(sht, spin, nside, lmax, nmaps):
    import torch
    note(f"tile edges spin={spin} nside={nside} lmax={lmax} nmaps={nmaps}")
    pol = spin == 2
    a, c = alm_inputs(lmax, nmaps, pol, workload=91)
    maps = synth.white_maps(12 * nside * nside, nmaps, 3 if pol else 1, workload=91)
    ref_m = oracle.alm2map_iqu(nside, lmax, a) if pol else oracle.alm2map(nside, lmax, a[:, 0])[:, None]
    ref_a = oracle.to_compact(oracle.map2alm_iqu(nside, lmax, maps) if pol
                              else oracle.map2alm(nside, lmax, maps[:, 0])[:, None])
    p = sht.Plan(nside, lmax, spin, nmaps)
    m = torch.full(p.map_shape(), np.nan, dtype=torch.float64, device="cuda")
    alm = torch.full(p.alm_shape(), np.nan, dtype=torch.float64, device="cuda")
    p.alm2map(to_dev(c), m)
    p.map2alm(to_dev(maps), alm)
    p.sync()
    assert rel_rms(from_dev(m), ref_m).max() < 1e-10
    assert rel_rms(from_dev(alm), ref_a).max() < 1e-10
    if pol and lmax > 2:
        e = torch.full(p.map_shape(), np.nan, dtype=torch.float64, device="cuda")
        b = torch.full(p.map_shape(), np.nan, dtype=torch.float64, device="cuda")
        p.alm2map_sel("TE", to_dev(c), e)
        p.alm2map_sel("B", to_dev(c), b)
        p.sync()
        # linear: the two parts add up to the whole, on the scale of the whole
        assert rel_rms(from_dev(e) + from_dev(b), ref_m).max() < 1e-10
    p.close()


@pytest.mark.parametrize("spin,nside,lmax,nmaps,part,precision", [
    (0, 64, 255, 33, 3, "fp64"), (2, 64, 150, 40, 5, "fp32"), (0, 64, 191, 192, 8, "fp64"), (2, 256, 700, 3, 1, "fp64"), (0, 200, 599, 9, 2, "fp64"), (2, 48, 143, 70, 5, "fp64"), (2, 128, 383, 21, 7, "fp32"),
    (0, 128, 383, 96, 8, "fp32"), (2, 24, 71, 13, 6, "fp32"), (2, 24, 71, 70, 16, "bf16x3"), (2, 40, 100, 17, 9, "bf16x3"),
    (0, 24, 71, 67, 16, "bf16x3")])
def test_wide_and_small_batches_agree(sht, spin, nside, lmax, nmaps, part, precision):
    """A map's result does not depend on the kernel its batch's width picks: 1e-12, far
    above FP64 rounding; FP32 and BF16x3 rows are summed in one order on any route."""
    import torch
    note(f"routes spin={spin} nside={nside} lmax={lmax} nmaps={nmaps} {precision}")
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    p = sht.Plan(nside, lmax, spin, nmaps, precision=precision)
    maps = torch.randn(p.map_shape(), generator=g, dtype=torch.float64, device="cuda")
    alm = torch.empty(p.alm_shape(), dtype=torch.float64, device="cuda")
    back = torch.empty_like(maps)
    p.map2alm(maps, alm)
    p.alm2map(alm, back)
    p.sync()
    p.close()
    q = sht.Plan(nside, lmax, spin, part, precision=precision)
    for k in range(0, nmaps, part):
        n = min(part, nmaps - k)
        q.set_nmaps(n)
        alm1 = torch.empty(q.alm_shape(), dtype=torch.float64, device="cuda")
        back1 = torch.empty(q.map_shape(), dtype=torch.float64, device="cuda")
        q.map2alm(maps[k:k + n].contiguous(), alm1)
        q.alm2map(alm[k:k + n].contiguous(), back1)
        q.sync()
        assert rel_rms(from_dev(alm1), from_dev(alm[k:k + n])).max() < 1e-12
        assert rel_rms(from_dev(back1), from_dev(back[k:k + n])).max() < 1e-12
    q.close()
