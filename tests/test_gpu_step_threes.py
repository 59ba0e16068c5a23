"""Small boxes take three steps a launch: bit for bit the state that single
steps reach, for every storage type, scalar lattice, wall rule and collision
path, on boxes that end inside a block's tile or are thinner than one."""
import pytest

from gpu_helpers import log

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BOXES = [(16, 16, 16), (4, 4, 4), (13, 9, 21), (61, 6, 4), (5, 30, 7)]
KINDS = [dict(precision="fp64"), dict(precision="fp32"), dict(precision="fp16"),
         dict(precision="fp16", round_stochastic=1), dict(precision="fp64", thermal_q=15),
         dict(precision="fp32", thermal_q=15, scalar_specular=1), dict(precision="fp32", R=1e-4),
         dict(precision="fp16", thermal_q=15, round_stochastic=1, scalar_specular=1)]


@pytest.mark.parametrize("kind", KINDS, ids=lambda k: "-".join(str(v) for v in k.values()))
@pytest.mark.parametrize("box", BOXES, ids=str)
def test_three_steps_a_launch_equal_single_steps(box, kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_04751_amd import solver as S
    log("case: steps in threes", box, kind)
    nx, ny, nz = box
    a, b = (S.Cavity(S.make_params(nx, 3e3, nx=nx, ny=ny, nz=nz, u0=0.05, **kind)) for _ in range(2))
    g = torch.Generator(device="cuda").manual_seed(nx)
    f = [s * torch.randn(nz, ny, nx, generator=g, device="cuda") for s in (0.01, 0.01, 0.01, 0.2)]
    for c in (a, b):
        c.init_macros(*f)
    for n in (10, 4, 3, 5):  # from either state, with one or two single steps behind
        a.step(n)
        for _ in range(n):
            b.step(1)
        assert a.steps_done() == b.steps_done()
        for p, q in zip(a.populations(), b.populations()):
            assert torch.isfinite(p).all()
            assert torch.equal(p, q), n
    a.close()
    b.close()
