"""Narrow tile classes stand in for the default ones in large handles: a
filter's particles, weights, ancestors, evidence and ESS are the same bits as
in the default class (which a small handle, or dpf_set_tiling, runs)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import dpf_synth as S  # noqa: E402
import paper_1203_2394_amd as dpf  # noqa: E402

# inner sizes at the edges of every narrow class (8, 16, 24, 32 lanes-items; 48, 64; 80, 96, 112, 128)
MS = [1, 7, 8, 9, 16, 17, 20, 24, 25, 32, 33, 48, 49, 64, 65, 80, 81, 96, 97, 112, 113, 128]


def _default_class(M):
    return next(k for k, (seg, jpt) in enumerate(dpf.tile_classes()[:6]) if M <= seg * jpt)


def _pair(spec, Ns, Ms, algo, seed=11):
    mk = lambda: dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, Ns, Ms, seed=seed, algo=algo)  # noqa: E731
    a, b = mk(), mk()
    b.set_tiling([_default_class(m) for m in Ms])  # asked for: no stand-in
    return a, b


def _same(a, b, spec):
    # what the step ends in: every bit of the state, the resampling and the evidence
    # (the plain filter's state is the proposals; its lam block is unused)
    sa, sb = a.unpack_state(a.export_state()), b.unpack_state(b.export_state())
    for k in ("t", "x", "z") + (("lam",) if a.algo == dpf.ALGO_LOOKAHEAD else ()):
        for u, v in zip(sa[k], sb[k]):
            assert u.tobytes() == v.tobytes(), k
    for which in (dpf.BUF_ELL, dpf.BUF_LOGW, dpf.BUF_ANC, dpf.BUF_SEL):
        assert torch.equal(a.copy_buffer(which), b.copy_buffer(which)), which
    ea, eb = a.estimate(), b.estimate()
    for k in ("ess", "loglik", "flags"):
        assert torch.equal(ea[k], eb[k]), k
    # the estimates' inner sums take another order: FP32 sums of up to 128 terms, then FP64
    for k in ("xhat", "zhat"):
        ref = eb[k].double().cpu().numpy()
        scale = max(1.0, float(np.abs(ref).max()))
        assert np.allclose(ea[k].double().cpu().numpy(), ref, rtol=0, atol=128 * 2.0 ** -24 * 4 * scale), k


@pytest.mark.parametrize("algo", ["lookahead", "plain"])
@pytest.mark.parametrize("model", ["lingauss", "twodim", "twodimz", "fourdim"])
def test_narrow_classes_give_the_default_classes_bits(model, algo):
    spec = {"lingauss": S.lingauss_c1(True), "twodim": S.twodim_table1(), "twodimz": S.twodim_table1(zfirst=True),
            "fourdim": S.fourdim_table1()}[model]
    # every inner size, outer sizes of one group, several, ragged ends of a tile; enough particles for the narrow classes
    Ms = MS * 2
    Ns = [600 + 7 * q for q in range(len(MS))] + [200 + 5 * q for q in range(len(MS))]
    T = 4
    Y = torch.from_numpy(np.stack([S.simulate(spec, T, 40 + q % 4)[2] for q in range(len(Ms))], axis=1).astype(np.float32))
    a, b = _pair(spec, Ns, Ms, algo)
    for f in (a, b):
        f.run(Y, use_graph=False)
    _same(a, b, spec)
    for f in (a, b):
        (f.lookahead_step if algo == "lookahead" else f.step)(Y[T - 1])
    _same(a, b, spec)


@pytest.mark.parametrize("K,predict", [(0, True), (1, False), (4, True)])
def test_narrow_nested_and_prediction(K, predict):
    spec = S.twodim_table1()
    Ms = [10, 20, 24, 31, 50, 64, 100]
    Ns, T = [2100] * 7, 3
    Y = torch.from_numpy(np.stack([S.simulate(spec, T, 60 + q)[2] for q in range(7)], axis=1).astype(np.float32))
    a, b = _pair(spec, Ns, Ms, "lookahead")
    out = []
    for f in (a, b):
        f.set_companions(K)
        if predict:
            f.set_prediction(True)
        f.run(Y)
        out.append(f.predicted_observation().cpu().numpy() if predict else None)
    _same(a, b, spec)
    if predict:
        assert np.allclose(out[0], out[1], rtol=0, atol=2e-5 * max(1.0, np.abs(out[1]).max()))


def test_learned_passes_leave_the_narrow_classes():
    """Cloud moments run in the public classes: a handle that asks for them
    goes over to those, and its steps stay the same bits."""
    spec = S.fourdim_table1()
    Ns, Ms = [4000, 3000], [20, 30]
    _, _, ys = S.simulate(spec, 3, 8)
    y = [torch.tensor(np.stack([v, v]), dtype=torch.float32) for v in ys]
    a, b = _pair(spec, Ns, Ms, "lookahead")
    for f in (a, b):
        f.lookahead_step(y[0])
        f.features(y[1])
        f.lookahead_step(y[1])
    assert torch.equal(a.export_state(), b.export_state())
