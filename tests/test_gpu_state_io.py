"""State export and import move every byte, for sizes that fill no group or
vector and for external buffers at any 4-byte alignment."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import dpf_synth as S  # noqa: E402
import paper_1203_2394_amd as dpf  # noqa: E402

CASES = [(S.lingauss_c1(), "lookahead", [1], [1]), (S.lingauss_c1(), "plain", [257, 3], [3, 50]),
         (S.fourdim_table1(), "lookahead", [255, 256, 513, 1], [7, 64, 33, 1]),
         (S.nonlin_c2(1), "lookahead", [100, 37, 300], [9, 256, 100]), (S.twodim_table1(), "lookahead", [20] * 9, [10] * 9),
         (S.highdim_c4(1), "lookahead", [5], [40])]


@pytest.mark.parametrize("spec,algo,N,M", CASES)
@pytest.mark.parametrize("shift", [0, 4])
def test_import_then_export_is_the_identity(spec, algo, N, M, shift):
    f = dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, N, M, seed=3, algo=algo)
    nb = f.state_bytes()
    head = (4 * f.F + 15) & ~15
    g = np.random.default_rng(nb)
    blob = np.zeros(nb, dtype=np.uint8)
    blob[:4 * f.F] = g.integers(0, 50, size=f.F).astype(np.int32).view(np.uint8)
    blob[head:] = g.normal(size=(nb - head) // 4).astype(np.float32).view(np.uint8)
    raw = torch.zeros(nb + 64, dtype=torch.uint8, device="cuda")
    raw[shift:shift + nb] = torch.from_numpy(blob).cuda()
    f.import_state(raw[shift:shift + nb])
    out = torch.full((nb + 64,), 0xAB, dtype=torch.uint8, device="cuda")
    dpf._check(dpf.lib().dpf_export_state(f._h, dpf._ptr(out[shift:]), nb))
    o = out.cpu().numpy()
    assert np.array_equal(o[shift:shift + nb], blob)
    assert (o[:shift] == 0xAB).all() and (o[shift + nb:] == 0xAB).all()  # nothing beyond the state


def test_export_after_steps_reads_the_current_copy():
    """A stepped state exported, imported elsewhere and stepped on gives the
    same bits as the filter that went on."""
    spec = S.fourdim_table1()
    _, _, ys = S.simulate(spec, 4, 5)
    a = dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, [300, 41], [21, 100], seed=9)
    y = [torch.tensor(np.stack([v, v]), dtype=torch.float32) for v in ys]
    for t in range(3):
        a.lookahead_step(y[t])
    b = dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, [300, 41], [21, 100], seed=9)
    b.import_state(a.export_state())
    assert torch.equal(a.export_state(), b.export_state())
    a.lookahead_step(y[3])
    b.lookahead_step(y[3])
    assert torch.equal(a.export_state(), b.export_state())
