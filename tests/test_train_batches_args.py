"""MLP.train_batches hands the library only what the library reads: float32 sets
of the stated shapes, int32 indices that fill whole batches and a loss array that
holds every batch's value; other whole-number indices are converted, anything
else is refused before the call."""
import ctypes

import numpy as np
import pytest

import paper_1203_2394_amd as dpf

torch = pytest.importorskip("torch")

B, N = 32, 50


class _Lib:
    """Reads the call's arrays as the library would."""

    def dpf_mlp_train_batches(self, state, blob, X, xt, n, idx, k, batch, lr, t0, ws, ws_bytes, loss, stream):
        f = lambda p, m, ty: np.ctypeslib.as_array((ty * m).from_address(p.value)).copy() if m else np.zeros(0)  # noqa: E731
        self.X = f(X, n * 32, ctypes.c_float).reshape(n, 32)
        self.xt = f(xt, n * 2, ctypes.c_float).reshape(n, 2)
        self.idx = f(idx, k * batch, ctypes.c_int32)
        self.loss, self.k = loss, k
        return 0


@pytest.fixture
def net(monkeypatch):
    L = _Lib()
    monkeypatch.setattr(dpf, "lib", lambda: L)
    monkeypatch.setattr(dpf, "_stream_ptr", lambda device: None)
    m = dpf.MLP.__new__(dpf.MLP)
    m.device, m.batch, m.adam_t = torch.device("cpu"), B, 0
    m.state = torch.zeros(3, 8)
    m.blob = torch.zeros(8, dtype=torch.uint8)
    m._ws = torch.zeros(8, dtype=torch.uint8)
    return m, L


def _set():
    g = torch.Generator().manual_seed(3)
    return torch.randn(N, 32, generator=g), torch.randn(N, 2, generator=g)


@pytest.mark.parametrize("kind", ["int32", "int64", "int16", "numpy64", "strided", "two_d"])
def test_indices_arrive_as_int32(net, kind):
    m, L = net
    X, xt = _set()
    want = np.random.default_rng(1).integers(0, N, size=2 * B)
    idx = torch.from_numpy(want)
    idx = {"int32": idx.int(), "int64": idx, "int16": idx.short(), "numpy64": want,
           "strided": torch.stack([idx, idx + 1], dim=1)[:, 0], "two_d": idx.reshape(2, B)}[kind]
    m.train_batches(X, xt, idx)
    assert L.k == 2 and m.adam_t == 2
    assert np.array_equal(L.idx, want)


def test_indices_beyond_32_bits_stay_outside_the_set(net):
    m, L = net
    X, xt = _set()
    idx = torch.zeros(B, dtype=torch.int64)
    idx[:4] = torch.tensor([1 << 32, -(1 << 40), (1 << 32) + 3, -1])
    m.train_batches(X, xt, idx)
    assert ((L.idx[:4] < 0) | (L.idx[:4] >= N)).all() and (L.idx[4:] == 0).all()


@pytest.mark.parametrize("kind", ["float64", "strided", "numpy"])
def test_sets_arrive_as_contiguous_float32(net, kind):
    m, L = net
    X, xt = _set()
    a, b = {"float64": (X.double(), xt.double()), "numpy": (X.numpy(), xt.numpy()),
            "strided": (torch.cat([X, X], dim=1)[:, :32], torch.cat([xt, xt], dim=1)[:, :2])}[kind]
    m.train_batches(a, b, torch.arange(B, dtype=torch.int32))
    assert np.array_equal(L.X, X.numpy()) and np.array_equal(L.xt, xt.numpy())


def test_targets_beyond_the_set_are_left_alone(net):
    m, L = net
    X, xt = _set()
    m.train_batches(X[:N - 9], xt, torch.arange(B, dtype=torch.int32))
    assert np.array_equal(L.xt, xt[:N - 9].numpy())


@pytest.mark.parametrize("bad", ["cols", "flat", "targets", "target_cols", "remainder", "float_idx", "bool_idx",
                                 "short_loss", "loss64", "strided_loss"])
def test_what_the_library_would_misread_is_refused(net, bad):
    m, L = net
    X, xt = _set()
    idx, loss = torch.arange(B, dtype=torch.int32).repeat(2), torch.zeros(2)
    if bad == "cols":
        X = X[:, :26]
    if bad == "flat":
        X = X.reshape(-1)
    if bad == "targets":
        xt = xt[:-1]
    if bad == "target_cols":
        xt = xt[:, :1]
    if bad == "remainder":
        idx = idx[:-1]
    if bad == "float_idx":
        idx = idx.float()
    if bad == "bool_idx":
        idx = idx > 3
    if bad == "short_loss":
        loss = loss[:1]
    if bad == "loss64":
        loss = loss.double()
    if bad == "strided_loss":
        loss = torch.zeros(4)[::2]
    with pytest.raises(dpf.DPFError):
        m.train_batches(X, xt, idx, loss=loss)
    assert not hasattr(L, "k") and m.adam_t == 0


def test_no_batches_is_no_step(net):
    m, L = net
    X, xt = _set()
    m.train_batches(X, xt, torch.zeros(0, dtype=torch.int32), loss=torch.zeros(0))
    assert m.adam_t == 0
