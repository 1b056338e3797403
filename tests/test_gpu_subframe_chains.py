"""The parallel traceback's two forms, a chain by stages and by periods of k-1
stages (csrc/vit_decoder.h chooses by the longest chain against the block's
survivor words): around the line between them and far on either side,
against the oracle, bit for bit."""
import numpy as np
import pytest

from test_gpu_subframes import _check, dev  # noqa: F401

pytestmark = pytest.mark.gpu

CODES = {"k4r14": (4, (0o13, 0o15, 0o17, 0o11)), "k5r12": (5, (0o23, 0o35)), "k6r12": (6, (0o53, 0o75)),
         "k7r13": (7, (0o133, 0o171, 0o165)), "k8r12": (8, (0o247, 0o371)),
         "k9r12": (9, (0o561, 0o753)), "k9r14": (9, (0o463, 0o535, 0o733, 0o745))}


@pytest.mark.parametrize("dtype", ["float32", "int8"])
@pytest.mark.parametrize("rule", [0, 1])
@pytest.mark.parametrize("name", sorted(CODES))
def test_both_sides(dev, name, rule, dtype):  # noqa: F811
    k, gens = CODES[name]
    body, regs = 32 // (k - 1) * (k - 1), max(1, 2 ** (k - 1) // 64)
    rng = np.random.default_rng([k, len(gens), rule])
    for L, f0, v in ((1024, 32, 40), (256, 24, 64), (64, 64, 30)):
        words = -(-(L + v - v // 2) // body) * regs
        line = (7 if k >= 8 else 8 if k >= 6 else 4) * words // 4 - f0  # inner overlap at which the chain is as dear as the words
        for w in sorted({0, max(0, line - regs), max(0, line), max(0, line + regs), 3 * words}):
            n = 5 * L - 3
            llr = rng.integers(-8, 9, size=(n + k - 1) * len(gens)).astype(dtype)
            _check(dev, k, gens, llr, n, L, v, f0, w, rule=rule, seed=7)
