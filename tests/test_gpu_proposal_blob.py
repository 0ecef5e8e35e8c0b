"""dpf_set_proposal takes the blob wherever the runtime can copy it from: device
memory at any byte, pinned or ordinary host memory give the network of the plain
device blob, and the caller's memory may go once the stream has passed the call."""
import ctypes

import numpy as np
import pytest

import dpf_synth as S
import paper_1203_2394_amd as dpf
from test_gpu_learned import _mlp, _params, _spec

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("where", ["byte_1", "byte_2", "pinned", "pageable"])
def test_blob_from_any_memory(where):
    spec = _spec()
    y = torch.tensor(S.simulate(spec, 1, 7)[2][:1], dtype=torch.float32)
    m = _mlp(_params(19))
    mk = lambda: dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, [70], [20], seed=5)  # noqa: E731
    a, b = mk(), mk()
    a.set_proposal(m, ess_frac=0.0)
    n = m.blob.numel()
    host = m.blob.cpu()
    if where.startswith("byte"):
        s = int(where[-1])
        raw = torch.zeros(n + 16, dtype=torch.uint8, device="cuda")
        raw[s:s + n] = m.blob
        ptr = raw.data_ptr() + s
    else:
        raw = host.pin_memory() if where == "pinned" else host.numpy().copy()
        ptr = raw.data_ptr() if where == "pinned" else raw.ctypes.data
    print(where, flush=True)
    dpf._check(dpf.lib().dpf_set_proposal(b._h, ctypes.c_void_p(ptr), n, 0.0))
    torch.cuda.synchronize()
    if where == "pageable":
        raw[:] = 0
    else:
        raw.zero_()
    for f in (a, b):
        f.learned_step(y)
    assert torch.equal(a.copy_buffer(dpf.BUF_MDN), b.copy_buffer(dpf.BUF_MDN))
    assert bool((a.copy_buffer(dpf.BUF_MDN) != 0).any())
    assert torch.equal(a.export_state(), b.export_state())
