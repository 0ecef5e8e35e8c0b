"""A plain run forms each step's weights in the previous step's new-cloud
launch and its estimates in the next one's: state, weights, ancestors,
estimates and traces are the bits of step calls, for filters of one group and
of several, that stop early, over odd and even numbers of steps, in one run or
several, and from steps to a run and back."""
import numpy as np
import pytest

import dpf_synth as S
import paper_1203_2394_amd as dpf

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SPECS = {
    "lingauss": S.lingauss_c1(True),
    "nonlin": S.nonlin_c2(1),
    "twodim": S.twodim_table1(),
    "twodimz": S.twodim_table1(zfirst=True),
    "fourdim": S.fourdim_table1(),
}


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _same_state(a, b):
    # (the plain filter's state is the proposals; its lam block is unused)
    sa, sb = a.unpack_state(a.export_state()), b.unpack_state(b.export_state())
    assert np.array_equal(sa["t"], sb["t"])
    for k in ("x", "z"):
        for u, v in zip(sa[k], sb[k]):
            assert u.tobytes() == v.tobytes(), k


def _check(name, N, M, split, use_graph):
    spec, F, T = SPECS[name], len(N), sum(split)
    Y = np.stack([S.simulate(spec, T + 1, 90 + q % 4)[2] for q in range(F)], axis=1).astype(np.float32)
    Tf = np.array([max(1, T - q % 3) for q in range(F)], dtype=np.int32)
    mk = lambda: dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, N, M, seed=6, algo="plain")  # noqa: E731
    a, b = mk(), mk()
    want = []
    for t in range(T):
        on = (Tf > t).astype(np.uint8)
        a.step(torch.from_numpy(Y[t]), active=torch.from_numpy(on))
        e = a.estimate()
        want.append((on == 1, e["xhat"].cpu().numpy(), e["zhat"].cpu().numpy()))
    at = 0
    for n in split:
        xt, zt = b.run(torch.from_numpy(Y[:at + n]), Tf=torch.from_numpy(np.minimum(Tf, at + n)), use_graph=use_graph)
        for t in range(at, at + n):
            on, x, z = want[t]
            assert np.array_equal(xt[t].cpu().numpy()[on], x[on]), t
            assert np.array_equal(zt[t].cpu().numpy()[on], z[on]), t
        at += n

    def same(last):
        _same_state(a, b)
        ea, eb = a.estimate(), b.estimate()
        for k in ea:
            assert torch.equal(ea[k], eb[k]), k
        if not last:
            return
        for which in (dpf.BUF_ELL, dpf.BUF_LOGW, dpf.BUF_ANC, dpf.BUF_SEL):
            assert torch.equal(a.copy_buffer(which), b.copy_buffer(which)), which

    same(False)  # (the weights of a filter that stopped early lie in either buffer)
    for f in (a, b):
        f.step(torch.from_numpy(Y[T]))
    same(True)


@pytest.mark.parametrize("name", sorted(SPECS))
@pytest.mark.parametrize("split,use_graph", [([5], True), ([4], False), ([1, 4], True), ([3, 2], False)])
def test_plain_run_equals_steps(name, split, use_graph):
    # one group, several; inner sizes of several classes
    _check(name, [1, 256, 257, 700, 90], [5, 40, 200, 33, 300], split, use_graph)


@pytest.mark.parametrize("name", ["lingauss", "fourdim"])
def test_plain_run_equals_steps_one_group(name):
    _check(name, [1, 256, 100], [7, 30, 70], [4], True)


@pytest.mark.parametrize("name", ["twodim", "fourdim"])
def test_plain_run_equals_steps_many_filters(name):
    """Narrow tile classes, many groups."""
    _check(name, [150 + 9 * q for q in range(60)], [20, 50, 100] * 20, [6], True)


def test_plain_run_equals_steps_large_filter():
    """More particles than the estimates' virtual threads, more than 64 groups."""
    _check("lingauss", [17000, 3], [8, 8], [3], True)


def test_plain_run_with_degenerate_weights():
    """Observations so far off that every weight underflows or is not finite."""
    spec = S.nonlin_c2(1)
    N, M = [300, 40], [64, 20]
    Y = np.stack([S.simulate(spec, 4, 3)[2]] * 2, axis=1).astype(np.float32)
    Y[1] = 1e25
    Y[2, 0] = np.nan
    mk = lambda: dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, N, M, seed=6, algo="plain")  # noqa: E731
    a, b = mk(), mk()
    for t in range(4):
        a.step(torch.from_numpy(Y[t]))
    b.run(torch.from_numpy(Y))
    eq = lambda p, q: torch.equal(p.cpu().contiguous().view(torch.uint8), q.cpu().contiguous().view(torch.uint8))  # noqa: E731
    _same_state(a, b)
    ea, eb = a.estimate(), b.estimate()
    for k in ea:
        assert eq(ea[k], eb[k]), k
