"""Steps of small handles end in their new-cloud launch: over many steps, with
filters that sit some out, on their own and between runs, the state, estimates
and predicted observations are the bits of a run, which forms them elsewhere."""
import numpy as np
import pytest

import dpf_synth as S
import paper_1203_2394_amd as dpf

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SPECS = {"lingauss": S.lingauss_c1(True), "nonlin": S.nonlin_c2(1), "twodim": S.twodim_table1(),
         "fourdim": S.fourdim_table1()}


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# 24 and 32 workgroups (the line), several classes in a handle, one workgroup
@pytest.mark.parametrize("N,M", [([100], [50]), ([64, 1, 37], [20, 33, 7]), ([1], [1]), ([128], [64]),
                                 ([20, 8, 3], [20, 200, 300])])
@pytest.mark.parametrize("algo", ["lookahead", "plain"])
@pytest.mark.parametrize("model", sorted(SPECS))
def test_small_handles_steps_equal_a_run(model, algo, N, M):
    spec, F, T = SPECS[model], len(N), 40
    Y = np.stack([S.simulate(spec, T + 2, 50 + q)[2] for q in range(F)], axis=1).astype(np.float32)
    mk = lambda: dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, N, M, seed=8, algo=algo)  # noqa: E731
    a, b = mk(), mk()
    step = lambda f: f.lookahead_step if algo == "lookahead" else f.step  # noqa: E731
    predict = algo == "lookahead" and spec.dy == 1
    yt = None
    if predict:
        a.set_prediction(True)
        yt = b.set_prediction(True, trace_T=T)
    xt, zt = b.run(torch.from_numpy(Y[:T]))
    for t in range(T):
        step(a)(torch.from_numpy(Y[t]))
        e = a.estimate()
        assert torch.equal(e["xhat"], xt[t]) and torch.equal(e["zhat"], zt[t]), t
        if predict:
            assert torch.equal(a.predicted_observation().reshape(-1), yt[t].reshape(-1)), t

    def same():
        sa, sb = a.unpack_state(a.export_state()), b.unpack_state(b.export_state())
        for k in ("t", "x", "z") + (("lam",) if algo == "lookahead" else ()):
            for u, v in zip(sa[k], sb[k]):
                assert np.array_equal(u, v), k
        ea, eb = a.estimate(), b.estimate()
        for k in ea:
            assert torch.equal(ea[k], eb[k]), k

    same()
    # filters that sit a step out keep their state and estimates; then all again, and a run after steps
    on = torch.tensor([q % 2 for q in range(F)], dtype=torch.uint8)
    for f in (a, b):
        step(f)(torch.from_numpy(Y[T]), active=on)
        step(f)(torch.from_numpy(Y[T + 1]))
        f.run(torch.from_numpy(Y), use_graph=False)
    same()
