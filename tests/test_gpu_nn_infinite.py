"""An infinite weight meets only the voxels its tap reads: the tiled
convolution's k range is padded to whole rounds of steps, which must add
nothing.  At tap 26 (one on in x, y and z) and the last input channel, the last k
of the range, the voxels of the grid's far faces, whose tap lies outside, take
0 times infinity, not a number, in any order; every other voxel is infinite where
its neighbour's value is positive."""
import pytest

from gpu_helpers import log

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("grid,n", [(32, 1), (32, 8), (32, 40), (16, 2), (16, 30)])
@pytest.mark.parametrize("layer", ["enc3a", "enc3b", "bota", "botb", "dec3b"])
def test_an_infinite_weight_stays_in_its_tap(grid, n, layer):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_04751_amd import network
    l = network.LAYER_NAMES.index(layer)
    g = grid >> network.LAYER_OUTPUTS[l][0]
    log("case: infinite weight", grid, n, layer, g)
    theta = torch.from_numpy(network.init_params(7)).clone()
    at = 0
    for name, (cin, cout, edge) in zip(network.LAYER_NAMES, network.LAYER_SHAPES):
        taps = edge ** 3
        if name == layer:
            theta[at + (3 * taps + 26) * cin + cin - 1] = float("inf")  # output channel 3
        at += cout * (taps * cin + 1)
    net = network.WarmStartNet(grid, n)
    net.set_params(theta)
    net.forward([3.0 + 2.0 * i / n for i in range(n)])
    got = net.activation(l, n)
    x = net.activation(l - 1, n)[..., -1]
    if layer in ("enc3a", "bota"):  # (the pooled input: the average of eight values)
        x = x.reshape(n, g, 2, g, 2, g, 2).mean(dim=(2, 4, 6))
    inside = (slice(None),) + (slice(0, g - 1),) * 3
    neighbour = x[:, 1:, 1:, 1:]
    if g > 1:
        want = torch.where(neighbour > 0, float("inf"), float("nan"))
        assert torch.equal(torch.isinf(got[inside][..., 3]), torch.isinf(want))
    others = torch.cat([got[..., :3], got[..., 4:]], -1)
    assert torch.isfinite(others).all()
    net.close()
