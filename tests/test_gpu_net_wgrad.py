"""Weight and bias gradients of the convolutions at the edges of their split:
bricks cut by the grid (levels down to 2 voxels), a single brick, blocks of
several bricks with a shorter last one, and padded input channels, against
FP64 sums over the GPU's own stored BF16 activations and gradients."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from tests.gpu_util import dev  # noqa: E402
from tests.test_gpu_net import M, gpu_params, net_inputs, unflat  # noqa: E402

# layers whose input and output gradient the GPU still holds after the pass
LAYERS = {"e1a": ("x", "g16b"), "e1b": ("a1", "g16a"), "e2a": ("p1", "g32b"), "e2b": ("a2", "g32a"),
          "b3a": ("p2", "g64b"), "b3b": ("a3", "g64a")}


@pytest.mark.parametrize("n,batch", [(8, 1), (8, 3), (16, 5), (32, 3), (64, 5)])
def test_weight_gradients_at_the_edges_of_the_split(n, batch):
    rng = np.random.default_rng(n + batch)
    v32, _ = gpu_params(3)
    net = M.Net(n, batch)
    M.pm_net_set_params(net, v32)
    for b in range(batch):
        M.pm_net_set_input(net, b, dev(net_inputs(rng, n)))
        M.pm_net_set_target(net, b, dev((0.5 * rng.standard_normal((3, n, n, n))).astype(np.float32)))
    M.pm_net_backward(net, batch)
    g = unflat(M.pm_net_get_grads(net).astype(np.float64))
    for name, (src, dst) in LAYERS.items():
        gw, gb, aw, ab = 0.0, 0.0, 0.0, 0.0
        for b in range(batch):
            a = M.pm_net_get_tensor(net, src, b).double()
            z = M.pm_net_get_tensor(net, dst, b).double()
            zf = z.reshape(z.shape[0], -1)
            taps = [torch.roll(a, (-dz, -dy, -dx), (1, 2, 3)).reshape(a.shape[0], -1)
                    for dz in (-1, 0, 1) for dy in (-1, 0, 1) for dx in (-1, 0, 1)]
            gw = gw + torch.stack([t @ zf.T for t in taps])
            aw = aw + torch.stack([t.abs() @ zf.abs().T for t in taps])
            gb, ab = gb + zf.sum(1), ab + zf.abs().sum(1)
        # A sum of products exact in FP32 over a chain of c additions is off
        # by at most c 2^-23 times the sum of magnitudes (truncation allowed):
        # c = 256 voxels of a brick times the bricks of a block, the groups of
        # a wave (64) and 16 waves.
        bricks = batch * max(1, z.shape[1] // 16) * max(1, z.shape[2] // 4) * max(1, z.shape[3] // 4)
        c = 256 * -(-bricks // (1024 // max(1, a.shape[0] // 16))) + 80
        gw, aw, gb, ab = (t.cpu().numpy() for t in (gw, aw, gb, ab))
        ew = np.abs(g[name + ".w"] - gw)
        print(n, batch, name, float((ew / (aw + 1e-300)).max()), c * 2.0 ** -23)
        assert np.all(ew <= c * 2.0 ** -23 * aw), name
        assert np.all(np.abs(g[name + ".b"] - gb) <= c * 2.0 ** -23 * ab), name
    net.close()
