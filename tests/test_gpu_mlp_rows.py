"""The network on the state of a large handle takes one, two or four 16-row
tiles per workgroup: at the edges of those ranges, with filters whose rows
share a tile and one that sits the step out, its outputs are those of the
forward pass on the same features.  The sums are the same products in the
same order; the bound leaves 1e-6 for the standardisation's rounding, as the
small handles' test does."""
import numpy as np
import pytest

import dpf_synth as S
import paper_1203_2394_amd as dpf
from test_gpu_learned import _mlp, _params, _rel_l2, _spec

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("rows", [8191, 8192, 8193, 16383, 16384, 16385, 16449, 33000])
def test_state_network_row_tiles(rows):
    spec = _spec()
    Ns = [37, rows - 37 - 901, 1, 900]
    Ms = [8, 4, 16, 8]
    f = dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, Ns, Ms, seed=31)
    Y = torch.tensor(np.stack([S.simulate(spec, 1, 60 + q)[2][0] for q in range(4)]), dtype=torch.float32)
    fmean = np.r_[np.zeros(2), np.zeros(8), np.zeros(8), np.full(8, 0.1)].astype(np.float32)
    fstd = np.r_[np.full(2, 5.0), np.full(8, 3.0), np.full(8, 3.0), np.full(8, 0.5)].astype(np.float32)
    m = _mlp(_params(15), fmean, fstd)
    f.set_proposal(m, ess_frac=0.0)
    feat = f.features(Y)
    X = torch.zeros(rows, 32, device=feat.device)
    X[:, :26] = (feat[:, :26] - m.fmean[:26]) / m.fstd[:26]
    ref = m.forward(X).cpu().numpy()
    f.learned_step(Y, active=torch.tensor([1, 1, 0, 1], dtype=torch.int32))
    got = f.copy_buffer(dpf.BUF_MDN).cpu().numpy().reshape(rows, 32)
    on = np.ones(rows, dtype=bool)
    on[Ns[0] + Ns[1]] = False
    assert np.isfinite(got[on]).all()
    assert _rel_l2(got[on], ref[on]) < 1e-6
    assert np.abs(got[on] - ref[on]).max() <= 1e-5 * np.abs(ref).max()


@pytest.mark.parametrize("ess_frac", [0.0, 1.0])
def test_fallback_decision_over_many_groups(ess_frac):
    """Filters decided by a wave each (up to 64 groups of 256) and by a whole
    workgroup (more): none of them falls back at a threshold of 0, all at 1
    (no filter of several particles has an ESS of exactly N)."""
    spec = _spec()
    Ns, Ms = [40, 17000, 300, 16384, 16385, 2], [8, 4, 16, 4, 8, 8]
    f = dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, Ns, Ms, seed=31)
    Y = torch.tensor(np.stack([S.simulate(spec, 1, 60 + q)[2][0] for q in range(len(Ns))]), dtype=torch.float32)
    m = _mlp(_params(15), np.zeros(26, dtype=np.float32), np.full(26, 5.0, dtype=np.float32))
    f.set_proposal(m, ess_frac=ess_frac)
    f.learned_step(Y)
    fell = (f.estimate()["flags"].cpu().numpy() & dpf.FLAG_FALLBACK) != 0
    assert fell.all() if ess_frac else not fell.any(), fell
    assert np.isfinite(f.copy_buffer(dpf.BUF_LOGW).cpu().numpy()).all()
