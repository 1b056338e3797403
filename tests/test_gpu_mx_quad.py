"""The two layouts of the matrix-core integer decoder (csrc/vit_decoder_mx.h)
where the choice between them changes: the smallest codes (4 registers only),
the 16-register layout of k = 6, 7 (from some ten thousand blocks on), windows
that begin within a dword of LLRs, and survivors at the border of what registers
and LDS hold.  Against the CPU oracle's exact integer decoder, bit for bit."""
import numpy as np
import pytest

import synth
from oracle import vref
from test_gpu_int16 import dev  # noqa: F401
from test_gpu_mx import _check, _values

pytestmark = pytest.mark.gpu

SMALL = {
    "k3r12": (3, (0o7, 0o5)), "k3r13": (3, (0o7, 0o5, 0o7)), "k3r14x": (3, (0o7, 0o5, 0o6, 0o3)),
    "k4r12": (4, (0o17, 0o13)), "k4r13x": (4, (0o15, 0o16, 0o17)), "k4r14": (4, (0o13, 0o15, 0o17, 0o11)),
}
WIDE = {"k6r12": (6, (0o53, 0o75), 80007), "k6r13": (6, (0o47, 0o53, 0o75), 80007),
        "k7r12": (7, (0o171, 0o133), 40007), "k7r14": (7, (0o133, 0o171, 0o165, 0o117), 40007)}


@pytest.mark.parametrize("kind", ["awgn", "ties", "extreme", "hard"])
@pytest.mark.parametrize("name", sorted(SMALL))
def test_smallest_codes(dev, name, kind):  # noqa: F811
    # odd overlaps, so that windows begin within a dword at beta = 2; one bit and
    # seven short of a block at the end; 16 and 17 kept bodies, and many more
    k, gens = SMALL[name]
    rng = np.random.default_rng([k, len(gens), len(kind)])
    body = 32 // (k - 1) * (k - 1)
    for L, v, v1, terminated, extra in ((8, 0, 0, True, 1), (8, 5, 5, False, 0), (24, 3 * k, None, True, -7),
                                        (16 * body // 8 * 8, 3, 3, False, 1), (16 * body // 8 * 8, 40, 7, True, 9),
                                        (1200, 13, 13, True, 3)):
        n = L * (6007 if L < 1000 else 3007) + extra
        _check(dev, k, gens, _values(kind, k, gens, n, terminated, rng), n, L, v, v1, terminated, f"{name} {kind} L={L} v={v}")


@pytest.mark.parametrize("kind", ["ties", "extreme", "hard"])
@pytest.mark.parametrize("name", sorted(WIDE))
def test_sixteen_registers(dev, name, kind):  # noqa: F811
    k, gens, blocks = WIDE[name]
    rng = np.random.default_rng([k, len(gens), len(kind)])
    for L, v, v1, terminated, extra in ((8, 0, 0, True, 1), (16, 3 * k, 3 * k, True, -7), (40, 5 * k, 11, False, 13)):
        n = L * blocks + extra
        _check(dev, k, gens, _values(kind, k, gens, n, terminated, rng), n, L, v, v1, terminated, f"{name} {kind} L={L} v={v}")


@pytest.mark.parametrize("name", ["k3r12", "k3r14x", "k4r13x", "k4r14"])
def test_batch_of_the_smallest_codes(dev, name):  # noqa: F811
    torch, vit = dev
    k, gens = SMALL[name]
    rng = np.random.default_rng([k, len(gens)])
    frames, chunks, off, out_off = [], [], 0, 0
    for _ in range(9001):
        n = int(rng.integers(1, 400))
        term = int(rng.random() < 0.5) if n > 1 else 1
        size = (n + (k - 1) * term) * len(gens)
        chunks.append(rng.integers(-20, 21, size=size).astype(np.int8))
        frames.append((0, term, n, off, out_off))
        off += size
        out_off += (n + 7) // 8
    llr = np.concatenate(chunks)
    L, v = 96, 6 * k
    out = torch.full((out_off,), 0xAB, dtype=torch.uint8, device="cuda")
    print(f"[gpu] quad batch {name}: {len(frames)} frames, {llr.size} LLRs", flush=True)
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
