"""Gradient calls of fewer samples than the network has room for: on grids of
8 and 16 cells they have more partial sums than a full batch.  They must stay
inside the workspace and give what a network of just that size gives."""
import pytest

from gpu_helpers import log

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

GUARD = 16 << 20


@pytest.mark.parametrize("grid,batch,n", [(8, 12, 11), (8, 12, 7), (8, 25, 24), (16, 5, 3), (16, 17, 16)])
def test_smaller_call_stays_in_the_workspace(grid, batch, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1710_04751_amd import capi, network
    log("case: smaller call", grid, batch, n)
    cfg = capi.nn_config(grid, batch)
    bytes_ = capi.lbm_nn_workspace_bytes(cfg)
    raw = torch.full((256 + bytes_ + GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
    start = -raw.data_ptr() % 256
    torch.cuda.synchronize()
    h = capi.lbm_nn_create(cfg, raw.data_ptr() + start, bytes_, None)
    theta = torch.from_numpy(network.init_params(grid)).cuda()
    capi.lbm_nn_set_params(h, theta.data_ptr())
    g = torch.Generator(device="cuda").manual_seed(n)
    targets = 0.02 * torch.randn(n, 4, grid, grid, grid, generator=g, device="cuda")
    grad = torch.empty(capi.lbm_nn_param_count(), device="cuda")
    lra = [3.0 + 2.0 * i / n for i in range(n)]
    torch.cuda.synchronize()
    loss = capi.lbm_nn_gradient(h, lra, targets.data_ptr(), n, list(range(n)), 4 * grid ** 3,
                                grad.data_ptr())
    torch.cuda.synchronize()
    assert bool((raw[:start] == 0xA5).all()) and bool((raw[start + bytes_:] == 0xA5).all())
    capi.lbm_nn_destroy(h)
    own = network.WarmStartNet(grid, n)
    own.set_params(theta)
    want_loss, want = own.gradient(lra, targets, list(range(n)))
    assert loss == want_loss and torch.equal(grad, want)
    own.close()
