"""The brick convolutions' split over blocks (how many bricks a block walks,
bricks of 8 or 4 rows, one or three output groups, a last range that is not
full) follows the batch: at 64^3 it must not change a result."""
import pytest

from gpu_helpers import log

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

GRID = 64
LRA = [3.2, 4.7, 3.9, 5.1, 4.2]


@pytest.fixture(scope="module")
def net():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_04751_amd import network
    n = network.WarmStartNet(GRID, 5, target_scale=(40.0, 300.0, 40.0, 1.5))
    n.set_params(torch.from_numpy(network.init_params(5)))
    yield n
    n.close()


@pytest.fixture(scope="module")
def targets():
    g = torch.Generator(device="cuda").manual_seed(4)
    return 0.02 * torch.randn(5, 4, GRID, GRID, GRID, generator=g, device="cuda")


@pytest.mark.parametrize("n", [2, 3, 5])
def test_forward_of_a_batch_equals_its_samples(net, n):
    """Every layer at this grid adds the same products in the same order
    whatever the split: bit for bit."""
    log("case: conv split forward", n)
    out = net.forward(LRA[:n])
    acts = [net.activation(l, n) for l in (0, 1, 3, 5, 9, 11, 13, 14)]
    for i in range(n):
        one = net.forward(LRA[i:i + 1])
        assert torch.equal(out[i], one[0]), i
        for a, l in zip(acts, (0, 1, 3, 5, 9, 11, 13, 14)):
            assert torch.equal(a[i], net.activation(l, 1)[0]), (i, l)


@pytest.mark.parametrize("n", [2, 4])
def test_gradient_of_a_batch_is_the_mean_of_its_samples(net, targets, n):
    """n a power of two: the output gradient of a batch is 1/n times the
    single sample's exactly, and so are the BF16 gradients of every layer, so
    only the FP32 sums over the voxels differ in their grouping.  A sum over m
    terms in blocked FP32 order is off by a few units of 2^-24 of its
    magnitude sum; the bound allows 1e-5 of the gradient's norm."""
    log("case: conv split gradient", n)
    loss, grad = net.gradient(LRA[:n], targets, list(range(n)))
    mean = torch.zeros_like(grad, dtype=torch.float64)
    total = 0.0
    for i in range(n):
        l, g = net.gradient(LRA[i:i + 1], targets, [i])
        mean += g.double() / n
        total += l / n
    err = float((grad.double() - mean).norm() / mean.norm())
    log("relative difference", err)
    assert err < 1e-5
    assert abs(loss - total) < 1e-12 * abs(total) + 1e-15
