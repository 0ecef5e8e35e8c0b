"""dpf_copy_buffer gives the weights of each filter's own last step: after runs
that filters leave early or take no part in, and after a run, a step or an import
that follows, the look-ahead and outer weights are the bits that step calls with
the same activity leave."""
import numpy as np
import pytest

import dpf_synth as S
import paper_1203_2394_amd as dpf

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SPECS = {"lingauss": S.lingauss_c1(True), "nonlin": S.nonlin_c2(1), "fourdim": S.fourdim_table1(),
         "highdim": S.highdim_c4(1)}


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _weights_equal(a, b):
    for which in (dpf.BUF_ELL, dpf.BUF_LOGW):
        u, v = a.copy_buffer(which), b.copy_buffer(which)
        assert torch.equal(u, v), which
        assert torch.equal(b.copy_buffer(which), v), which  # a second look sees the same


@pytest.mark.parametrize("algo,K", [("plain", 0), ("lookahead", 0), ("lookahead", 2)])
@pytest.mark.parametrize("name,N,M", [("lingauss", [1, 256, 257, 700, 90], [5, 40, 200, 33, 300]),
                                      ("fourdim", [100, 7, 250], [20, 64, 3]),
                                      ("nonlin", [300, 20, 513], [50, 130, 256]),
                                      ("highdim", [9, 20], [30, 70])])
@pytest.mark.parametrize("split,use_graph", [([5], True), ([4, 3], False)])
def test_weights_after_uneven_runs(algo, K, name, N, M, split, use_graph):
    spec, F, T = SPECS[name], len(N), sum(split)
    Y = np.stack([S.simulate(spec, T + 1, 30 + q % 4)[2] for q in range(F)], axis=1).astype(np.float32)
    # every parity of the last step, one filter that takes one step only
    Tf = np.array([1] + [T - q % 4 for q in range(F - 1)], dtype=np.int32)
    mk = lambda: dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, N, M, seed=8, algo=algo)  # noqa: E731
    a, b = mk(), mk()
    if K:
        a.set_companions(K)
        b.set_companions(K)
    step = lambda f, t, on: (f.step if algo == "plain" else f.lookahead_step)(torch.from_numpy(Y[t]), active=on)  # noqa: E731
    at = 0
    for n in split:
        for t in range(at, at + n):
            step(a, t, torch.from_numpy((Tf > t).astype(np.uint8)))
        at += n
        b.run(torch.from_numpy(Y[:at]), Tf=torch.from_numpy(np.minimum(Tf, at)), use_graph=use_graph)
        _weights_equal(a, b)
    b.run(torch.from_numpy(Y[:2]), use_graph=use_graph)  # every filter but the first is past these
    step(a, 1, torch.from_numpy((np.arange(F) == 0).astype(np.uint8)))
    _weights_equal(a, b)
    for f in (a, b):
        f.import_state(a.export_state())
    _weights_equal(a, b)
    on = torch.from_numpy((np.arange(F) % 2).astype(np.uint8))
    for f in (a, b):
        step(f, T, on)
    _weights_equal(a, b)
    if algo == "lookahead":
        for f in (a, b):
            f.reset()
        _weights_equal(a, b)
