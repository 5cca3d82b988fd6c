"""Convolutions with output tiles on blocks of their own (few bricks) give the
bits of those with all tiles on one block (many bricks): a region alone and the
same region as the last of a batch, every level on either side of the rule."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

from tests.gpu_util import dev  # noqa: E402
from tests.test_gpu_net import M, gpu_params, net_inputs  # noqa: E402


@pytest.mark.parametrize("n,batch", [(8, 64), (32, 32), (64, 2), (64, 16)])
def test_a_region_alone_equals_the_same_region_in_a_batch(n, batch):
    rng = np.random.default_rng(n)
    v32, _ = gpu_params(4)
    x, t = net_inputs(rng, n), (0.5 * rng.standard_normal((3, n, n, n))).astype(np.float32)
    out = []
    for k in (1, batch):
        net = M.Net(n, k)
        M.pm_net_set_params(net, v32)
        for b in range(k):
            M.pm_net_set_input(net, b, dev(x))
            M.pm_net_set_target(net, b, dev(t))
        M.pm_net_backward(net, k)
        # the gradient of the mean over the batch: 1 / batch, a power of two
        out.append({name: M.pm_net_get_tensor(net, name, k - 1) * (k if name[0] == "g" else 1)
                    for name in M.NET_TENSORS})
        net.close()
    for name in M.NET_TENSORS:
        assert torch.equal(out[0][name], out[1][name]), name
