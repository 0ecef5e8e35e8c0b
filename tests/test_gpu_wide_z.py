"""The wide-z model at the inner sizes where its new-cloud and look-ahead
passes change shape: one wave per particle or several, one item per lane or
several, a last wave that is nearly empty, and (from 64 lanes on) the shared
part of the transition held one component per lane.  Bounds as for every
step's parity: FP32 values within TOL, index flips only at near ties."""
import pytest

import test_gpu_parity as parity
from parity_util import assert_clean

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# class edges: 32 | 64 | 128 | 256 | 256 x 4 | 256 x 16 lanes x items
SIZES = [(5, 1), (7, 33), (5, 64), (6, 65), (4, 129), (3, 257), (2, 1025)]


@pytest.mark.parametrize("name", ["highdim", "highdim_gauss"])
@pytest.mark.parametrize("N,M", SIZES)
def test_wide_z_lookahead_step(name, N, M):
    for r, info, est, gs, logw in parity._la_case(name, N, M, 1, 1):
        assert_clean(r, n=N, max_flip_frac=0.5)
        parity._check_evidence(est, info, logw, name)
        parity._check_self_estimates(est, gs, logw)


@pytest.mark.parametrize("N,M", SIZES)
def test_wide_z_plain_step(N, M):
    for r, info, est, logw in parity._plain_case("highdim", N, M, 1, 1):
        assert_clean(r, n=N, max_flip_frac=0.5)
        parity._check_evidence(est, info, logw, "highdim")
