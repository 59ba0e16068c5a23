"""Starts of boxes whose rows are longer than one piece of the staggered sums'
work split: a cell more or less than whole pieces, few rows and many."""
import pytest

from test_gpu_start import test_staggered_momentum_of_a_start as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 4, 1025), (4, 5, 2047), (5, 4, 3072), (4, 4, 20000), (17, 30, 1500)])
def test_long_rows(shape):
    check(shape)


def test_a_long_box_starts_as_fast_as_a_wide_one():
    """20000 x 4 x 4 cells have no more work than 80 x 50 x 80, which has 250
    times the rows: within a factor of four (it had been nine)."""
    import torch
    from paper_1710_04751_amd import solver as S
    if not torch.cuda.is_available():
        pytest.skip("no GPU")

    def time_of(nx, ny, nz):
        p = S.make_params(64, 1e4, u0=0.02)
        p.nx, p.ny, p.nz = nx, ny, nz
        p.lattice_units, p.nu, p.alpha, p.gbeta = 1, 0.02, 0.02, 1e-6
        cav = S.Cavity(p)
        f = [0.01 * torch.rand(nz, ny, nx, device="cuda") for _ in range(4)]
        best = 1e9
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(5):
                cav.init_macros(*f)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        cav.close()
        return best

    assert time_of(20000, 4, 4) < 4 * time_of(80, 50, 80)
