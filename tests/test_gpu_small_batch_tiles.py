"""Register-operand Legendre kernels in the tile forms that only larger grids pick: one and
two 4-column tiles in one launch per spin with one, two or four ring tiles a wave, runs of 8
and of 16 rows, and 16 columns split and not; E and B together without T (spin 2 in a launch
of its own).  Each against the same maps inside a batch of 33, which runs 16-column tiles."""
import pytest

from .gpu_util import note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("spin,nside,lmax,parts", [
    (2, 16, 47, (1, 2)), (2, 96, 383, (1, 2, 3, 9)), (2, 150, 599, (1, 2, 3, 5)), (2, 200, 599, (1, 2, 4)),
    (2, 192, 767, (1, 2)), (2, 256, 511, (1, 2)), (2, 256, 767, (1, 2)), (0, 48, 191, (1, 2, 3)), (0, 128, 511, (1, 3, 4)),
    (0, 192, 767, (2, 3, 4)), (0, 200, 599, (1, 3, 4)), (0, 256, 767, (1, 3, 4, 5))])
def test_small_batches_equal_a_wide_one(spin, nside, lmax, parts):
    import torch
    from paper_2208_10154_amd import sht
    g = torch.Generator(device="cuda")
    g.manual_seed(nside + lmax)
    p = sht.Plan(nside, lmax, spin, 33)
    maps = torch.randn(p.map_shape(), generator=g, dtype=torch.float64, device="cuda")
    alm = torch.empty(p.alm_shape(), dtype=torch.float64, device="cuda")
    back = torch.empty_like(maps)
    p.map2alm(maps, alm)
    p.alm2map(alm, back)
    p.sync()
    p.close()

    def check(got, want):
        assert ((got - want).norm(dim=-1) <= 1e-12 * want.norm(dim=-1)).all()

    for n in parts:
        note(f"small batch spin={spin} nside={nside} lmax={lmax} nmaps={n}")
        q = sht.Plan(nside, lmax, spin, n)
        a, m = torch.full_like(alm[:n], torch.nan), torch.full_like(maps[:n], torch.nan)
        q.map2alm(maps[:n], a)
        q.alm2map(alm[:n], m)
        check(a, alm[:n])
        check(m, back[:n])
        if spin == 2:
            q.map2alm_sel("EB", maps[:n], a)
            q.alm2map_sel("EB", alm[:n], m)
            check(a[:, 1:], alm[:n, 1:])
            check(m[:, 1:], back[:n, 1:])
            assert (a[:, 0] == 0).all() and (m[:, 0] == 0).all()
        q.close()
