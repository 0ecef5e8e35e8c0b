"""A nested run of filters of one resampling group leaves each step's estimates
to the next launch: its traces, predicted observations and state are the bits
of step calls, with filters that stop early, in one run or several."""
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


@pytest.mark.parametrize("F", [3, 70])  # below and above the many-groups line
@pytest.mark.parametrize("use_graph", [True, False])
@pytest.mark.parametrize("split", [[6], [3, 3], [1, 5]])
def test_nested_run_pipeline(F, use_graph, split):
    spec = S.twodim_table1()
    N = [1 + (37 * q) % 256 for q in range(F)]
    N[0] = 256
    M = [20 if q % 3 else 9 for q in range(F)]
    T = sum(split)
    Y = np.stack([S.simulate(spec, T, 80 + q % 4)[2] for q in range(F)], axis=1).astype(np.float32)
    Tf = np.array([max(1, T - q % 4) for q in range(F)], dtype=np.int32)
    mk = lambda: dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, N, M, seed=5)  # noqa: E731
    a, b = mk(), mk()
    for f in (a, b):
        f.set_companions(3)
    a.set_prediction(True)
    want = {"x": [], "z": [], "y": []}
    for t in range(T):
        on = (Tf > t).astype(np.uint8)
        a.lookahead_step(torch.from_numpy(Y[t]), active=torch.from_numpy(on))
        e = a.estimate()
        want["x"].append((on, e["xhat"].cpu().numpy()))
        want["z"].append((on, e["zhat"].cpu().numpy()))
        want["y"].append((on, a.predicted_observation().cpu().numpy().reshape(F, 1)))
    at = 0
    for n in split:
        yt = b.set_prediction(True, trace_T=T)  # rows by the filter's own time
        xt, zt = b.run(torch.from_numpy(Y[:at + n] if at == 0 else Y[:at + n]), Tf=torch.from_numpy(np.minimum(Tf, at + n)),
                       use_graph=use_graph)
        for t in range(at, at + n):
            for got, key in ((xt, "x"), (zt, "z"), (yt, "y")):
                on, ref = want[key][t]
                g = got[t].cpu().numpy().reshape(F, -1)
                assert np.array_equal(g[on == 1], ref[on == 1]), (key, t)
        at += n
    assert torch.equal(a.export_state(), b.export_state())
    ea, eb = a.estimate(), b.estimate()
    for k in ea:
        assert torch.equal(ea[k], eb[k]), k
