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


@pytest.mark.parametrize("n", [9, 40, 64])
def test_tiled_kernel_groups_on_small_grids(n):
    """Grids of 8 cells and less (the tiled kernel: one, two or four output
    groups a wave, the k range over 4, 2 or 1 waves, by the number of tiles):
    each sample of a batch against its own single call, whose path the oracle
    checks.  Where the k range is split differently, FP32 sums differ in their
    last bits and a BF16 result in its last place now and then: 2^-8 of a value,
    through 15 layers below 2e-2 of the output's norm."""
    from paper_1710_04751_amd import network
    log("case: tiled kernel groups", n)
    lra = [3.0 + 3.0 * i / n for i in range(n)]
    a = network.WarmStartNet(8, n)
    b = network.WarmStartNet(8, 1)
    theta = torch.from_numpy(network.init_params(11))
    a.set_params(theta)
    b.set_params(theta)
    out = a.forward(lra)
    for i in (0, n // 2, n - 1):
        one = b.forward([lra[i]])[0]
        err = float((out[i] - one).norm() / one.norm())
        assert err < 2e-2, (i, err)
    a.close()
    b.close()


@pytest.mark.parametrize("grid,n", [(64, 1), (32, 8), (32, 2), (16, 4)])
def test_pooled_results_are_the_averages(grid, n):
    """The convolutions before a pooling write its averages themselves (on
    grids of 16 cells and more).  A network whose layers after the pooling
    copy their input (centre weight 1 on the diagonal, no bias) shows
    the pooled values as the next layer's results, which must be the averages
    of eight BF16 values added in FP32 in (z, y, x) order, rounded once."""
    import numpy as np
    from paper_1710_04751_amd import network
    log("case: pooled results", grid, n)
    theta = torch.from_numpy(network.init_params(3)).clone()
    at = 0
    for name, (cin, cout, edge) in zip(network.LAYER_NAMES, network.LAYER_SHAPES):
        taps = edge ** 3
        size = cout * taps * cin
        if name in ("enc2a", "enc3a", "bota"):
            w = torch.zeros(cout, taps, cin)
            for c in range(cin):
                w[c, 13, c] = 1.0
            theta[at:at + size] = w.reshape(-1)
            theta[at + size:at + size + cout] = 0.0
        at += size + cout
    assert at == theta.numel()
    net = network.WarmStartNet(grid, n)
    net.set_params(theta)
    net.forward([3.0 + 0.4 * i for i in range(n)])
    for before, after, c in ((1, 2, 16), (3, 4, 32), (5, 6, 64)):
        a = net.activation(before, n).cpu()
        g = a.shape[1]
        a = a.reshape(n, g // 2, 2, g // 2, 2, g // 2, 2, c)
        acc = torch.zeros(n, g // 2, g // 2, g // 2, c)
        for z in range(2):
            for y in range(2):
                for x in range(2):
                    acc = acc + a[:, :, z, :, y, :, x]
        want = (acc * 0.125).to(torch.bfloat16).float()
        got = net.activation(after, n).cpu()[..., :c]
        assert np.array_equal(got.numpy(), want.numpy()), (before, grid)
    net.close()
