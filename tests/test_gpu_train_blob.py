"""A training step's forward pass reads the weights of the blob it is given: after
the blob alone was rewritten (packed without the training workspace, or copied from
another network) the loss is that network's, bit for bit, in a step, in the loss
alone and in a call of several batches."""
import numpy as np
import pytest

import paper_1203_2394_amd as dpf
from test_gpu_learned import _params

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _net(seed, B):
    return dpf.MLP(dpf.flatten_params(_params(seed)), np.zeros(26), np.ones(26), batch=B)


@pytest.mark.parametrize("B", [32, 544])
@pytest.mark.parametrize("how", ["pack", "copy"])
def test_loss_of_a_rewritten_blob(B, how):
    g = np.random.default_rng(B)
    X = torch.from_numpy(g.normal(size=(B, 32)).astype(np.float32)).cuda()
    xt = torch.from_numpy(g.normal(size=(B, 2)).astype(np.float32)).cuda()
    a, b = _net(21, B), _net(22, B)
    a.train_step(X, xt)  # (the workspace's copies are those of the trained network)
    want = b.loss_and_grad(X, xt)[0]
    assert not torch.equal(a.loss_and_grad(X, xt)[0], want)
    if how == "pack":
        dpf._check(dpf.lib().dpf_mlp_pack(dpf._ptr(b.state[0]), dpf._ptr(a.fmean), dpf._ptr(a.fstd), dpf._ptr(a.blob),
                                          None, 0, a._stream()))
    else:
        a.blob.copy_(b.blob)
    assert torch.equal(a.loss_and_grad(X, xt)[0], want)
    loss = torch.empty(2, device="cuda")
    a.train_batches(X, xt, torch.arange(B, dtype=torch.int32, device="cuda").repeat(2), loss=loss)
    assert torch.equal(loss[:1], want)


def test_loss_under_another_workspace():
    """Validation with a workspace of its own, between training steps."""
    B = 64
    g = np.random.default_rng(5)
    X = torch.from_numpy(g.normal(size=(B, 32)).astype(np.float32)).cuda()
    xt = torch.from_numpy(g.normal(size=(B, 2)).astype(np.float32)).cuda()
    a, val = _net(23, B), _net(23, B)
    for _ in range(3):
        a.train_step(X, xt)
    want = a.loss_and_grad(X, xt)[0]
    loss = torch.empty(1, device="cuda")
    dpf._check(dpf.lib().dpf_mlp_train_step(dpf._ptr(a.state), dpf._ptr(a.blob), dpf._ptr(X), dpf._ptr(xt), B, 0.0, 0,
                                            dpf._ptr(val._ws), val._ws.numel(), dpf._ptr(loss), None, a._stream()))
    assert torch.equal(loss, want)
