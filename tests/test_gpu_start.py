"""Starts from given fields (lbm_init_macros) at the edges of the staggered
sums' work split: rows shorter and longer than a wave, one row more or less
than the waves of a block, fewer rows than one block, and many blocks."""
import numpy as np
import pytest

from gpu_helpers import log, to_np

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SHAPES = [(4, 4, 4), (5, 4, 63), (4, 5, 65), (7, 5, 128), (97, 93, 8), (31, 300, 130)]


@pytest.mark.parametrize("shape", SHAPES)
def test_staggered_momentum_of_a_start(shape):
    """Velocities of the start against float64 NumPy: u less its staggered
    sums, w with the staggered sum S/2 (lbm.h).  The sums run in another
    order than NumPy's: their error is below 1e-16 times the sum of the
    magnitudes (at most 1 per cell), divided by the cell count."""
    from paper_1710_04751_amd import solver as S
    nz, ny, nx = shape
    log("case: start", shape)
    rng = np.random.default_rng(nx * 1000 + ny)
    f = [(0.02 * rng.standard_normal(shape) + 0.01).astype(np.float32) for _ in range(3)]
    f.append(rng.uniform(-0.5, 0.5, shape).astype(np.float32))
    cav = S.Cavity(S.make_params(nx=nx, ny=ny, nz=nz, Ra=1e3, precision="fp64"))
    cav.init_macros(*[torch.from_numpy(v) for v in f])
    F, G = cav.populations()
    m = {k: to_np(v) for k, v in cav.macros(fp64=True).items()}
    cav.init_macros(*[torch.from_numpy(v) for v in f])
    F2, G2 = cav.populations()
    gb = cav.lattice.gbeta
    cav.close()
    assert torch.equal(F, F2) and torch.equal(G, G2)  # a fixed order of summation
    sx = ((-1.0) ** np.arange(nx))[None, None, :]
    sy = ((-1.0) ** np.arange(ny))[None, :, None]
    sz = ((-1.0) ** np.arange(nz))[:, None, None]
    u = [v.astype(np.float64) for v in f]
    n = nx * ny * nz
    want = {"ux": u[0] - sx * np.sum(sx * u[0]) / n, "uy": u[1] - sy * np.sum(sy * u[1]) / n,
            "uz": u[2] - sz * (np.sum(sz * u[2]) - 0.5 * gb * np.sum(sz * u[3])) / n}
    want["uz"] = want["uz"] - 0.5 * gb * u[3]  # lbm_macros takes off half the force
    for k, v in want.items():
        assert np.max(np.abs(m[k] - v)) < 1e-15, k
    assert np.max(np.abs(m["T"] - u[3])) < 1e-15
