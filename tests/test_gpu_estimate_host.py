"""dpf_estimate into ordinary host memory, alone or beside device arrays, goes
through the runtime's copies: the same bits, and nothing around them."""
import ctypes

import numpy as np
import pytest

import dpf_synth as S
import paper_1203_2394_amd as dpf

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

KEYS = ("xhat", "zhat", "ess", "loglik", "flags")


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("F", [1, 300])
@pytest.mark.parametrize("host", [KEYS, ("loglik",), ("xhat", "flags")])
def test_estimate_into_pageable_memory(F, host):
    spec = S.nonlin_c2(1)
    f = dpf.Filter(spec.kind, spec.dx, spec.dz, spec.dy, spec.blob, [20] * F, [8] * F, seed=3)
    f.lookahead_step(torch.tensor(np.repeat(S.simulate(spec, 1, 3)[2][:1], F, axis=0), dtype=torch.float32))
    full = {k: v.cpu().numpy().reshape(-1) for k, v in f.estimate().items()}
    bufs, ptrs = {}, []
    for k in KEYS:
        n = full[k].size
        if k in host:
            bufs[k] = np.full(n + 6, 77, dtype=full[k].dtype)
            ptrs.append(ctypes.c_void_p(bufs[k].ctypes.data + 3 * bufs[k].itemsize))
        else:
            bufs[k] = torch.full((n + 6,), 77, dtype=torch.from_numpy(full[k]).dtype, device="cuda")
            ptrs.append(ctypes.c_void_p(bufs[k].data_ptr() + 3 * bufs[k].element_size()))
    print(F, host, flush=True)
    assert dpf.lib().dpf_estimate(f._h, *ptrs) == 0
    torch.cuda.synchronize()
    for k, b in bufs.items():
        got, n = (b if k in host else b.cpu().numpy()), full[k].size
        assert got[3:3 + n].tobytes() == full[k].tobytes(), k
        assert (got[:3] == 77).all() and (got[3 + n:] == 77).all(), k
