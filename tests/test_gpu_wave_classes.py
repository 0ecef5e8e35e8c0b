"""Classes of one wave per particle stand in for the default ones of two and
four in large handles: every bit of a filter's particles, weights, ancestors,
evidence and ESS is that of the default class, by step, run and graph, with
companions and the predicted observation."""
import numpy as np
import pytest

import dpf_synth as S
import paper_1203_2394_amd as dpf
from test_gpu_narrow import _pair, _same

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# edges of 64 x 2 (the nonlinear model), 64 x 6 and 64 x 8, and the sizes beyond
MS = [65, 66, 127, 128, 257, 300, 320, 321, 384, 385, 448, 500, 512, 513, 64]
SPECS = {"lingauss": S.lingauss_c1(True), "nonlin": S.nonlin_c2(1), "nonlin_b": S.nonlin_c2(2, bmode=1),
         "twodim": S.twodim_table1(), "twodimz": S.twodim_table1(zfirst=True), "fourdim": S.fourdim_table1()}


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("algo", ["lookahead", "plain"])
@pytest.mark.parametrize("model", sorted(SPECS))
def test_wave_classes_give_the_default_classes_bits(model, algo):
    spec, T = SPECS[model], 3
    Ns = [100 + 13 * q for q in range(len(MS))]
    Y = torch.from_numpy(np.stack([S.simulate(spec, T, 40 + q % 4)[2] for q in range(len(MS))], axis=1).astype(np.float32))
    a, b = _pair(spec, Ns, MS, algo)
    predict = algo == "lookahead" and spec.dy == 1
    traces = [f.set_prediction(True, trace_T=T) for f in (a, b)] if predict else []
    for f in (a, b):
        f.run(Y)
    _same(a, b, spec)
    if predict:  # (the sums are the default class's, in its order)
        assert torch.equal(traces[0], traces[1])
    for f in (a, b):
        (f.lookahead_step if algo == "lookahead" else f.step)(Y[T - 1])
    _same(a, b, spec)


@pytest.mark.parametrize("model", ["nonlin", "twodim", "fourdim"])
def test_wave_classes_with_companions(model):
    spec, T = SPECS[model], 2
    Ms = [65, 128, 260, 384, 400, 512]
    Ns = [300] * len(Ms)
    Y = torch.from_numpy(np.stack([S.simulate(spec, T, 40 + q % 4)[2] for q in range(len(Ms))], axis=1).astype(np.float32))
    a, b = _pair(spec, Ns, Ms, "lookahead")
    # on, off and on again
    for K in (3, 0, 2):
        for f in (a, b):
            f.set_companions(K)
            f.reset()
            f.run(Y)
        _same(a, b, spec)


def test_learned_steps_after_wave_classes():
    """A proposal brings a handle back to the default classes."""
    import test_gpu_learned as L

    spec = S.nonlin_c2(1)
    Ns, Ms = [700, 900], [100, 300]
    Y = torch.from_numpy(np.stack([S.simulate(spec, 4, 40 + q)[2] for q in range(2)], axis=1).astype(np.float32))
    a, b = _pair(spec, Ns, Ms, "lookahead")
    for f in (a, b):
        f.run(Y[:2])
        f.set_proposal(L._mlp(L._params(15)), ess_frac=0.1)
        f.learned_step(Y[2])
        f.lookahead_step(Y[3])
        f.learned_step(Y[3])
    assert torch.equal(a.export_state(), b.export_state())
    assert torch.equal(a.copy_buffer(dpf.BUF_MDN), b.copy_buffer(dpf.BUF_MDN))
