"""Stage times of small IQU calls, whose two spins share a Legendre launch: each spin keeps
a time of its own, and the results are those of the call without the profiler."""
import pytest

from .gpu_util import from_dev, note, rel_rms

pytestmark = pytest.mark.gpu

LEGENDRE = ("m2a_spin0", "m2a_spin2", "a2m_spin0", "a2m_spin2")


@pytest.mark.parametrize("precision", ["fp64", "fp32", "bf16x3"])
@pytest.mark.parametrize("nmaps", [1, 3, 12, 20])
def test_each_spin_has_its_stage_time(precision, nmaps):
    import torch
    from paper_2208_10154_amd import sht
    note(f"stage times nside 32 x{nmaps} {precision}")
    p = sht.Plan(32, 95, 2, nmaps, precision=precision)
    g = torch.Generator(device="cuda")
    g.manual_seed(nmaps)
    maps = torch.randn(p.map_shape(), generator=g, dtype=torch.float64, device="cuda")
    alm = torch.empty(p.alm_shape(), dtype=torch.float64, device="cuda")
    back = torch.empty_like(maps)
    alm1, back1 = torch.empty_like(alm), torch.empty_like(maps)
    p.map2alm(maps, alm)
    p.alm2map(alm, back)
    p.set_profiling(True)
    p.profile(reset=True)
    p.map2alm(maps, alm1)
    p.alm2map(alm, back1)
    prof = p.profile(reset=True)
    for s in LEGENDRE:
        assert prof[s][1] == 1 and prof[s][0] > 0, (s, prof)
    assert torch.equal(alm, alm1)
    assert rel_rms(from_dev(back1), from_dev(back)).max() < 1e-13  # folds with atomics near the poles
    if nmaps == 1:
        p.map2alm_immediate(maps, alm1, 1)
        prof = p.profile(reset=True)
        p.set_profiling(False)
        p.map2alm_immediate(maps, alm, 1)
        assert prof["m2a_spin0"][1] == prof["m2a_spin2"][1] > 1
        assert prof["a2m_spin0"][1] == prof["a2m_spin2"][1] > 1
        assert rel_rms(from_dev(alm1), from_dev(alm)).max() < (1e-13 if precision == "fp64" else 1e-5)
    p.close()
