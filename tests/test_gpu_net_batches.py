"""The network's kernels over batch sizes: every image's output has the same
bits whatever batch it comes in (three images and more run the walks over rows,
whose length depends on the batch and the dilation), and stays within the
forward pass's bound of the oracle; gradients of batches whose walks differ
against the oracle."""
import numpy as np
import pytest
import torch

from oracle import net as ON

pytestmark = pytest.mark.gpu

cc = pytest.importorskip("paper_1306_6883_amd")
from paper_1306_6883_amd import learned as L  # noqa: E402


def images(nb, seed):
    g = np.random.default_rng(seed)
    return torch.as_tensor(g.standard_normal((nb, cc.NET_G, cc.NET_G)).astype(np.float32), device="cuda")


def make(batch, seed=3):
    net = cc.Net(batch=batch, n_max=128)
    p = L.init_params(seed)
    cc.ccmg_net_set_params(net, p)
    return net, p


@pytest.mark.parametrize("nb", [3, 5, 8, 17, 40])
def test_outputs_do_not_depend_on_the_batch(nb):
    print(f"net batch {nb}", flush=True)
    net, p = make(48)
    x = images(48, 7)
    whole = cc.ccmg_net_forward(net, x)
    part = cc.ccmg_net_forward(net, x[:nb].contiguous())
    assert torch.equal(part, whole[:nb])


@pytest.mark.parametrize("nb", [1, 3, 9])
def test_gradients_match_oracle(nb):
    """Per layer within 1e-3 of the oracle with the same rounding points: both
    sum the same products, in FP32 and FP64, and a back-propagated value within
    about sqrt(288) 2^-24 of a bfloat16 midpoint rounds the other way (2^-8 of
    it, about 1e-3 of the values per layer, five rounded stages)."""
    print(f"net gradients, batch {nb}", flush=True)
    net, p = make(nb, seed=4)
    x, t = images(nb, 8), images(nb, 9) * 0.1
    loss, g = cc.ccmg_net_loss_grad(net, x, t)
    lo, go = ON.loss_grad(p.cpu().numpy().astype(np.float64), x.cpu().numpy().astype(np.float64),
                          t.cpu().numpy().astype(np.float64), bf=True)
    assert abs(loss - lo) <= 1e-3 * lo
    g, o = g.cpu().numpy().astype(np.float64), 0
    for l, sz in enumerate(ON.SIZES):
        e = np.linalg.norm(g[o:o + sz] - go[o:o + sz]) / np.linalg.norm(go[o:o + sz])
        print(f"layer {l + 1}: {e:.2e}")
        assert e < 1e-3, l
        o += sz


@pytest.mark.parametrize("nb", [3, 8])
def test_last_layer_in_halves(nb):
    """The last layer in two workgroups a class (up to 8 images) and in one
    (from 9): the same sums in the same order."""
    print(f"last layer, batch {nb}", flush=True)
    net, p = make(9, seed=5)
    x = images(9, 11)
    assert torch.equal(cc.ccmg_net_forward(net, x[:nb].contiguous()), cc.ccmg_net_forward(net, x)[:nb])
