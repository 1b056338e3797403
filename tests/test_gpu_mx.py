"""The matrix-core integer decoder (csrc/vit_decoder_mx.h) against the CPU
oracle's exact integer decoder, bit for bit.  It runs where there are blocks
for every SIMD, so the cases have about ten thousand (fewer for k = 8, 9):
every constraint length and rate it takes, windows shorter than a survivor word
and longer than the registers hold words for, blocks of different lengths in a
wave (the first and last of a stream, frames of mixed lengths), ties on every
stage, metrics at their largest, and the last partial wave."""
import numpy as np
import pytest

import synth
from oracle import vref
from test_gpu_int16 import NCPU, _oracle, _same, dev  # noqa: F401

pytestmark = pytest.mark.gpu

CODES = {
    "k5r12": (5, (0o23, 0o35)), "k5r12x": (5, (0o22, 0o35)), "k5r13x": (5, (0o25, 0o33, 0o16)),
    "k5r14": (5, (0o25, 0o27, 0o33, 0o37)), "k6r12": (6, (0o53, 0o75)), "k6r13": (6, (0o47, 0o53, 0o75)),
    "k6r14": (6, (0o53, 0o67, 0o71, 0o75)), "k7r12": (7, (0o171, 0o133)), "k7r13": (7, (0o133, 0o171, 0o165)),
    "k7r14": (7, (0o133, 0o171, 0o165, 0o117)), "k8r12": (8, (0o247, 0o371)), "k8r13": (8, (0o225, 0o331, 0o367)),
    "k8r14": (8, (0o235, 0o275, 0o313, 0o357)), "k9r12": (9, (0o561, 0o753)), "k9r13": (9, (0o557, 0o663, 0o711)),
    "k9r14": (9, (0o463, 0o535, 0o733, 0o745)),
}


def _blocks(k):
    return 10007 if k <= 7 else 5003 if k == 8 else 3001


def _values(kind, k, gens, n, terminated, rng):
    size = (n + (k - 1 if terminated else 0)) * len(gens)
    if kind == "ties":
        return rng.integers(-1, 2, size=size).astype(np.int8)
    if kind == "extreme":
        return np.where(rng.random(size) < 0.5, -128, 127).astype(np.int8)
    if kind == "hard":
        return rng.integers(0, 2, size=size).astype(np.uint8)
    coded = synth.encode(k, gens, synth.info_bits(n, rng), terminated)
    return np.clip(np.rint(9 * (1.0 - 2.0 * coded) + 9 * rng.standard_normal(size)), -127, 127).astype(np.int8)


def _decode(dev, k, gens, llr, n, L, v, v1, terminated):  # noqa: F811
    torch, vit = dev
    print(f"[gpu] mx k={k} gens={[oct(g) for g in gens]} n={n} L={L} v={v} v1={v1} term={terminated}", flush=True)
    nb = (n + 7) // 8
    buf = torch.full((nb + 64,), 0xAB, dtype=torch.uint8, device="cuda")
    vit.decode(vit.make_code(k, gens), torch.from_numpy(llr).cuda(), n, L, v, v1=v1, terminated=terminated, out=buf)
    torch.cuda.synchronize()
    got = buf.cpu().numpy()
    assert (got[nb:] == 0xAB).all(), "the decode wrote past ceil(n/8) bytes"
    return got[:nb]


def _check(dev, k, gens, llr, n, L, v, v1, terminated, what):  # noqa: F811
    exact = 1 - 2 * (llr != 0).astype(np.int8) if llr.dtype == np.uint8 else llr
    want = _oracle(k, gens, exact, n, L, v, v1, terminated)
    _same(_decode(dev, k, gens, llr, n, L, v, v1, terminated), want, n, what)


@pytest.mark.parametrize("kind", ["awgn", "ties", "extreme", "hard"])
@pytest.mark.parametrize("name", sorted(CODES))
def test_short_blocks(dev, name, kind):  # noqa: F811
    # windows of a few stages to a few survivor words; overlaps that clip
    # several blocks at either end of the stream; a last block of one bit
    k, gens = CODES[name]
    rng = np.random.default_rng([k, len(gens), len(kind)])
    for L, v, v1, terminated, extra in ((8, 0, 0, True, 1), (8, 5 * k, None, False, 0), (16, 3 * k, 3 * k, True, -7),
                                        (64, 8 * k, 0, False, 13)):
        n = L * _blocks(k) + extra
        llr = _values(kind, k, gens, n, terminated, rng)
        _check(dev, k, gens, llr, n, L, v, v1, terminated, f"{name} {kind} L={L} v={v}")


@pytest.mark.parametrize("kind", ["awgn", "extreme"])
@pytest.mark.parametrize("name", ["k5r12", "k6r13", "k7r12", "k7r14", "k8r12", "k8r14", "k9r12", "k9r14"])
@pytest.mark.parametrize("L,v", [(200, 35), (256, 64), (520, 70)])
def test_long_blocks(dev, name, kind, L, v):  # noqa: F811
    # survivors in registers and LDS, at their border and beyond; with extreme
    # values the fp32 sums of k = 8, 9 are taken back many times
    k, gens = CODES[name]
    rng = np.random.default_rng([k, L])
    n = L * _blocks(k) * (2 if L > 512 else 1) + 5
    _check(dev, k, gens, _values(kind, k, gens, n, True, rng), n, L, v, None, True, f"{name} {kind} L={L}")


@pytest.mark.parametrize("one_open_bit", [False, True])
@pytest.mark.parametrize("name", ["k5r13x", "k6r12", "k7r12", "k7r13", "k8r12", "k9r12"])
def test_batch_of_mixed_lengths(dev, name, one_open_bit):  # noqa: F811
    # frames of 1 to 700 bits, so that waves hold blocks of many lengths, known
    # and unknown starts, open and terminated ends; with an open frame of one
    # bit (less than a dword of LLRs) the run takes the one-block kernel
    torch, vit = dev
    k, gens = CODES[name]
    rng = np.random.default_rng([k, len(gens)])
    count = 9001 if k <= 7 else 4501 if k == 8 else 2501
    frames, chunks, off, out_off = [], [], 0, 0
    for f in range(count):
        n = int(rng.integers(1, 701))
        term = int(rng.random() < 0.6) if n > 1 else 1
        if one_open_bit and f == 7:
            n, term = 1, 0
        size = (n + (k - 1) * term) * len(gens)
        chunks.append(rng.integers(-20, 21, size=size).astype(np.int8))
        frames.append((0, term, n, off, out_off))
        off += size
        out_off += (n + 7) // 8
    llr = np.concatenate(chunks)
    L, v = 96, 6 * k
    out = torch.full((out_off,), 0xAB, dtype=torch.uint8, device="cuda")
    print(f"[gpu] mx batch {name}: {count} frames, {llr.size} LLRs", flush=True)
    b = vit.Batch()
    b.decode([vit.make_code(k, gens)], frames, torch.from_numpy(llr).cuda(), out, tune=[(L, v, -1, 1)])
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    b.close()
    code = vref.make_code(k, list(gens))
    for _, term, n, lo, oo in frames:
        sub = llr[lo:lo + (n + (k - 1) * term) * len(gens)]
        want = synth.pack_bits(vref.decode_blocked(code, sub, n, L, v // 2, v - v // 2, bool(term)))
        np.testing.assert_array_equal(got[oo:oo + want.size], want, err_msg=f"frame of {n} bits at {lo}")
