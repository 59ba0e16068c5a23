"""The block shape a caller sets governs every step's launch, and the kernel's
name is the one that takes the steps; results do not depend on either."""
import ctypes

import pytest

from gpu_helpers import log

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def solver():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_04751_amd import solver as S
    return S


def launches(cav, stream, steps):
    """Kernel launches of `steps` steps, counted in a capture that is not run."""
    from paper_1710_04751_amd import capi
    hip = capi.lib()  # (its lookups reach the HIP runtime it links)
    graph, count = ctypes.c_void_p(), ctypes.c_size_t()
    torch.cuda.synchronize()
    s = ctypes.c_void_p(stream.cuda_stream)
    assert hip.hipStreamBeginCapture(s, 1) == 0
    capi.lbm_step(cav.h, steps)
    assert hip.hipStreamEndCapture(s, ctypes.byref(graph)) == 0
    assert hip.hipGraphGetNodes(graph, None, ctypes.byref(count)) == 0
    assert hip.hipGraphDestroy(graph) == 0
    return count.value


@pytest.mark.parametrize("precision", ["fp64", "fp32", "fp16"])
def test_a_set_shape_governs_small_boxes(solver, precision):
    log("case: set shape on a small box", precision)
    stream = torch.cuda.Stream()
    a = solver.Cavity(solver.make_params(16, 3e3, precision=precision), stream=stream)
    p = solver.make_params(16, 3e3, precision=precision)
    p.block_x, p.block_y = 64, 1
    b = solver.Cavity(p, stream=stream)
    assert a.kernel_name().startswith("lbm::kern::k_step3<") and launches(a, stream, 6) == 2
    assert b.kernel_name().startswith("lbm::kern::k_step<") and launches(b, stream, 6) == 6
    a.autotune(steps_per_trial=2)
    assert a.kernel_name().startswith("lbm::kern::k_step3<") and launches(a, stream, 6) == 2
    a.set_block(32, 4)
    assert a.kernel_name() == b.kernel_name() and launches(a, stream, 6) == 6
    a.close()
    b.close()


@pytest.mark.parametrize("box,kind", [
    ((128, 37, 9), dict(precision="fp32")),
    ((128, 37, 9), dict(precision="fp64", thermal_q=15, R=1e-5)),
    ((128, 37, 9), dict(precision="fp16", round_stochastic=1)),
    ((192, 150, 100), dict(precision="fp32", thermal_q=15)),
    ((256, 190, 90), dict(precision="fp64"))], ids=str)
def test_every_shape_gives_the_default_shapes_result(solver, box, kind):
    """Tiles of several rows (the second number above 1 and the first a divisor
    of nx, with a last tile past ny), blocks of consecutive cells of every
    size; boxes whose blocks all keep, and some that mix the cache policies."""
    log("case: block shapes", box, kind)
    nx, ny, nz = box
    g = torch.Generator(device="cuda").manual_seed(ny)
    f = [s * torch.randn(nz, ny, nx, generator=g, device="cuda") for s in (0.01, 0.01, 0.01, 0.2)]

    def run(shape):
        c = solver.Cavity(solver.make_params(nx, 3e3, nx=nx, ny=ny, nz=nz, u0=0.05, **kind))
        if shape:
            c.set_block(*shape)
        c.init_macros(*f)
        c.step(4)
        out = [p.clone() for p in c.populations()]
        c.close()
        return out

    want = run(None)
    for shape in [(64, 2), (64, 4), (32, 2), (64, 1), (128, 1), (256, 1), (1024, 1), (128, 8)]:
        for p, q in zip(run(shape), want):
            assert torch.equal(p, q), shape
