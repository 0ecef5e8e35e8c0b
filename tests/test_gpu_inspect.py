"""A look at a large handle's features leaves its steps as they were: the narrow
tile classes stay, so estimates, state and evidence are the bits of a handle that
was not looked at, also for steps that the caller captured before the look."""
import numpy as np
import pytest

import dpf_synth as S
import paper_1203_2394_amd as dpf

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# 2125 waves of eight particles; 2600 of one (the nonlinear model)
CASES = [(S.fourdim_table1(), [9000, 8000], [20, 20]), (S.nonlin_c2(1), [2000, 600], [90, 128])]


def _y(spec, T):
    return [torch.tensor(np.stack([v, v]), dtype=torch.float32, device="cuda") for v in S.simulate(spec, T, 8)[2]]


def _same(a, b):
    assert torch.equal(a.export_state(), b.export_state())
    ea, eb = a.estimate(), b.estimate()
    for k in ea:
        assert torch.equal(ea[k], eb[k]), k


@pytest.mark.parametrize("spec,Ns,Ms", CASES)
def test_features_change_no_step(spec, Ns, Ms):
    y = _y(spec, 6)
    mk = lambda: dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, Ns, Ms, seed=4)  # noqa: E731
    a, b = mk(), mk()
    for t in range(3):
        fa = a.features(y[t]) if t != 1 else None
        a.lookahead_step(y[t])
        b.lookahead_step(y[t])
        _same(a, b)
    Y = torch.stack(y)
    a.run(Y)
    b.run(Y)
    _same(a, b)
    assert torch.equal(a.features(y[0]), b.features(y[0])) and bool(torch.isfinite(fa).all())


@pytest.mark.parametrize("spec,Ns,Ms", CASES)
def test_captured_step_after_a_look_at_the_features(spec, Ns, Ms):
    y = _y(spec, 5)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        a = dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, Ns, Ms, seed=4)
        a.lookahead_step(y[0])
        yb = y[1].clone()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        a.lookahead_step(yb)
    b = dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, Ns, Ms, seed=4)
    b.lookahead_step(y[0])
    for t in range(1, 5):
        with torch.cuda.stream(s):
            yb.copy_(y[t])
            g.replay()
            a.features(y[t])
        torch.cuda.synchronize()
        b.lookahead_step(y[t])
        _same(a, b)
        torch.cuda.synchronize()


def test_default_classes_serve_the_proposal():
    """With a proposal the steps keep its moments up to date: learned and
    look-ahead steps in turn are those of a handle whose classes were asked for."""
    spec = S.nonlin_c2(1)
    Ns, Ms = [2000, 600], [90, 128]
    y = _y(spec, 4)
    m = dpf.MLP(dpf.init_params(3, 26), np.zeros(26), np.full(26, 5.0), batch=32)
    a, b = (dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, Ns, Ms, seed=4) for _ in range(2))
    b.set_tiling([2, 2])
    for f in (a, b):
        f.lookahead_step(y[0])
        f.set_proposal(m, ess_frac=0.0)
        f.learned_step(y[1])
        f.lookahead_step(y[2])
        f.learned_step(y[3])
    _same(a, b)
    assert torch.equal(a.copy_buffer(dpf.BUF_MDN), b.copy_buffer(dpf.BUF_MDN))
