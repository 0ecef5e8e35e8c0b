"""Nothing a handle gives back depends on what its workspace held before: states,
estimates and weights are the same bits over workspaces filled with different
bytes, and the block that a plain filter's state does not use is zero."""
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


@pytest.mark.parametrize("algo", ["plain", "lookahead"])
@pytest.mark.parametrize("spec,N,M", [(S.lingauss_c1(True), [1, 256, 300], [5, 40, 200]),
                                      (S.nonlin_c2(1), [300, 20], [50, 256]), (S.highdim_c4(1), [9, 20], [30, 70])])
def test_results_over_any_workspace(monkeypatch, algo, spec, N, M):
    F, T = len(N), 5
    Y = torch.from_numpy(np.stack([S.simulate(spec, T, 30 + q)[2] for q in range(F)], axis=1).astype(np.float32))
    empty, got = torch.empty, []
    for fill in (0x00, 0x7F, 0xFF):
        with monkeypatch.context() as m:
            m.setattr(torch, "empty", lambda *a, **k: empty(*a, **k).fill_(fill)
                      if k.get("dtype") == torch.uint8 else empty(*a, **k))
            f = dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, N, M, seed=8, algo=algo)
        out = [f.export_state()]
        (f.step if algo == "plain" else f.lookahead_step)(Y[0])
        out.append(f.export_state())
        f.run(Y, Tf=torch.tensor([2, T, 3][:F], dtype=torch.int32))
        out += [f.export_state()] + [f.copy_buffer(w) for w in (dpf.BUF_ELL, dpf.BUF_LOGW, dpf.BUF_ANC, dpf.BUF_SEL)]
        out += list(f.estimate().values())
        got.append([v.cpu().contiguous().view(torch.uint8) for v in out])
        if algo == "plain":
            n = 4 * f.NMT
            assert all(not bool(b[-n:].any()) for b in got[-1][:3])
    for other in got[1:]:
        for u, v in zip(got[0], other):
            assert torch.equal(u, v)
