"""The 32-bit integer decoder (csrc/vit_decoder_int.h) against the CPU oracle's
exact integer decoder, bit for bit, where its survivor tags can go wrong: every
constraint length, windows around whole periods and whole survivor words
(entry at every kind of offset), ties on every stage (hard decisions, zeros)
and metrics at their largest (runs of -128 and 127)."""
import numpy as np
import pytest

from test_gpu_int16 import _oracle, _gpu, _same, dev  # noqa: F401
from test_gpu_parity import CODES

pytestmark = pytest.mark.gpu


def _inputs(kind, size, rng):
    if kind == "ties":
        return rng.integers(-1, 2, size=size).astype(np.int8)
    if kind == "hard":
        return rng.integers(0, 2, size=size).astype(np.uint8)
    return np.where(rng.random(size) < 0.5, -128, 127).astype(np.int8)


@pytest.mark.parametrize("kind", ["ties", "hard", "extreme"])
@pytest.mark.parametrize("name", sorted(CODES))
def test_integer_decode_at_word_edges(dev, name, kind):  # noqa: F811
    k, gens = CODES[name]
    p = k - 1
    body = p * (32 // p)
    rng = np.random.default_rng([k, len(kind)])
    for terminated in (True, False):
        for n in (1, p, p + 1, body - 1, body, body + 1, 2 * body + 3, 8 * body + 5):
            llr = _inputs(kind, (n + (p if terminated else 0)) * len(gens), rng)
            hard = 1 - 2 * (llr != 0).astype(np.int8) if kind == "hard" else llr
            for L, v in ((0, 0), (8, 2 * p), (64, 5 * k + 1)):
                want = _oracle(k, gens, hard, n, L, v, None, terminated)
                _same(_gpu(dev, k, gens, llr, n, L, v, None, terminated, 32), want, n, f"{name} {kind} n={n} L={L}")
