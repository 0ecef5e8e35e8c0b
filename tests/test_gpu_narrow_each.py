"""Each narrow and wave class by itself, in a handle large enough for it (1600
waves; 1024 for a wave per particle): the bits of the default class, at the
smallest, a middle and the largest inner size of the class, with uneven outer
sizes; and beside a default class that has too few waves for its stand-in."""
import numpy as np
import pytest

import dpf_synth as S
import paper_1203_2394_amd as dpf
from test_gpu_narrow import _pair, _same

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

SPECS = {"lingauss": S.lingauss_c1(True), "twodim": S.twodim_table1(), "twodimz": S.twodim_table1(zfirst=True),
         "fourdim": S.fourdim_table1(), "nonlin": S.nonlin_c2(1)}
# (lanes, smallest and largest inner size)
SMALL = [(8, 1, 8), (8, 9, 16), (8, 17, 24), (8, 25, 32), (16, 33, 48), (16, 49, 64), (16, 65, 80), (16, 81, 96),
         (16, 97, 112), (16, 113, 128)]
WAVE = [(64, 257, 384), (64, 385, 512)]
CASES = [(m, c) for m in ("lingauss", "twodim", "twodimz", "fourdim") for c in SMALL + WAVE]
CASES += [("nonlin", c) for c in [(64, 65, 128)] + WAVE]


@pytest.fixture(autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _handle(cls):
    lanes, lo, hi = cls
    Ms = [lo, (lo + hi) // 2, hi] * 3
    need = (1024 if lanes == 64 else 1600) * (64 // lanes) // len(Ms)
    return [need + 40 + 7 * q for q in range(len(Ms))], Ms


def _steps(a, b, spec, algo, F, T=2):
    Y = torch.from_numpy(np.stack([S.simulate(spec, T, 40 + q % 4)[2] for q in range(F)], axis=1).astype(np.float32))
    for f in (a, b):
        f.run(Y)
    _same(a, b, spec)
    for f in (a, b):
        (f.lookahead_step if algo == "lookahead" else f.step)(Y[T - 1])
    _same(a, b, spec)


@pytest.mark.parametrize("algo", ["lookahead", "plain"])
@pytest.mark.parametrize("model,cls", CASES)
def test_each_class_gives_the_default_classes_bits(model, cls, algo):
    spec = SPECS[model]
    Ns, Ms = _handle(cls)
    a, b = _pair(spec, Ns, Ms, algo)
    _steps(a, b, spec, algo, len(Ns))


@pytest.mark.parametrize("model", ["twodim", "fourdim", "nonlin"])
def test_companions_beside_and_without_wave_classes(model):
    """On, off and on again, with a class large enough for its stand-in and one that is not."""
    spec = SPECS[model]
    Ns, Ms = _handle((64, 65, 128) if model == "nonlin" else (16, 33, 48))
    Ns, Ms = Ns + [300] * 4 + [50, 60], Ms + [260, 300, 384, 512] + [8, 20]
    a, b = _pair(spec, Ns, Ms, "lookahead")
    Y = torch.from_numpy(np.stack([S.simulate(spec, 2, 40 + q % 4)[2] for q in range(len(Ns))], axis=1).astype(np.float32))
    for K in (2, 0, 3):
        for f in (a, b):
            f.set_companions(K)
            f.reset()
            f.run(Y)
        _same(a, b, spec)


@pytest.mark.parametrize("K", [1, 3, 5, 8])
@pytest.mark.parametrize("model,cls", CASES)
def test_companions_in_each_class(model, cls, K):
    spec = SPECS[model]
    Ns, Ms = _handle(cls)
    a, b = _pair(spec, Ns, Ms, "lookahead")
    for f in (a, b):
        f.set_companions(K)
    _steps(a, b, spec, "lookahead", len(Ns))
