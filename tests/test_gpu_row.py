"""The FP32 decoder of four blocks a wave (csrc/vit_decoder_row.h), which runs
where there are several blocks for every SIMD: against the CPU oracle, bit for
bit (ties on every stage, values from denormal to near overflow, the first and
last blocks of a stream, partial waves, bodies around those that are traced),
and in batches against the same frames in small batches, which the one-block
kernel decodes (infinities and NaN included)."""
import numpy as np
import pytest

import synth
from oracle import vref
from test_gpu_int16 import NCPU, _same, dev  # noqa: F401

pytestmark = pytest.mark.gpu

CODES = {"k3r12": (3, (0o7, 0o5)), "k3r13": (3, (0o7, 0o5, 0o7)), "k4r12": (4, (0o17, 0o13)),
         "k4r13": (4, (0o13, 0o15, 0o17)), "k5r12": (5, (0o23, 0o35)), "k5r13": (5, (0o25, 0o33, 0o37)),
         "k6r12": (6, (0o53, 0o75)), "k6r13": (6, (0o47, 0o53, 0o75))}


def _values(kind, size, rng):
    if kind == "ties":
        return rng.integers(-1, 2, size).astype(np.float32)
    if kind == "scales":
        return (rng.standard_normal(size) * 10.0 ** rng.integers(-44, 30, size)).astype(np.float32)
    x = rng.standard_normal(size).astype(np.float32)
    if kind == "special":
        x[rng.random(size) < 0.01] = np.inf
        x[rng.random(size) < 0.01] = -np.inf
        x[rng.random(size) < 0.002] = np.nan
    return x


@pytest.mark.parametrize("kind", ["normal", "ties", "scales"])
@pytest.mark.parametrize("name", sorted(CODES))
def test_streams(dev, name, kind):  # noqa: F811
    torch, vit = dev
    k, gens = CODES[name]
    rng = np.random.default_rng([k, len(gens), len(kind)])
    body = 32 // (k - 1) * (k - 1)
    for L, v, v1, terminated, extra in ((8, 0, 0, True, 1), (16, 5 * k, None, False, -7), (96, 3 * k, 3 * k, True, 9),
                                        (8 * body, 40, 7, True, 5)):
        n = L * 9001 + extra
        llr = _values(kind, (n + (k - 1) * terminated) * len(gens), rng)
        print(f"[gpu] row {name} {kind} n={n} L={L} v={v}", flush=True)
        left = v // 2 if v1 is None else v1
        want = synth.pack_bits(vref.decode_blocked(vref.make_code(k, list(gens)), llr, n, L, left, v - left, terminated,
                                                   nthreads=NCPU))
        buf = torch.full(((n + 7) // 8 + 64,), 0xAB, dtype=torch.uint8, device="cuda")
        vit.decode(vit.make_code(k, gens), torch.from_numpy(llr).cuda(), n, L, v, v1=left, terminated=terminated, out=buf)
        torch.cuda.synchronize()
        got = buf.cpu().numpy()
        assert (got[want.size:] == 0xAB).all()
        _same(got[:want.size], want, n, f"{name} {kind} L={L} v={v}")


@pytest.mark.parametrize("kind", ["normal", "special"])
@pytest.mark.parametrize("name", ["k3r13", "k4r12", "k5r12", "k6r13"])
def test_batches(dev, name, kind):  # noqa: F811
    torch, vit = dev
    k, gens = CODES[name]
    rng = np.random.default_rng([k, len(gens), len(kind)])
    n = rng.integers(1, 301, 8001)
    term = (rng.random(n.size) < 0.5).astype(int)
    sizes = (n + (k - 1) * term) * len(gens)
    off, out_off = np.cumsum(sizes) - sizes, np.cumsum((n + 7) // 8) - (n + 7) // 8
    llr = torch.from_numpy(_values(kind, int(sizes.sum()), rng)).cuda()
    frames = [(0, int(t), int(m), int(o), int(p)) for t, m, o, p in zip(term, n, off, out_off)]
    code, tune = [vit.make_code(k, gens)], [(96, 6 * k, -1, 1)]
    outs = [torch.zeros(int(out_off[-1] + (n[-1] + 7) // 8), dtype=torch.uint8, device="cuda") for _ in range(2)]
    print(f"[gpu] row batch {name} {kind}: {n.size} frames", flush=True)
    b = vit.Batch()
    b.decode(code, frames, llr, outs[0], tune=tune)
    for i in range(0, n.size, 200):
        b.decode(code, frames[i:i + 200], llr, outs[1], tune=tune)
    torch.cuda.synchronize()
    b.close()
    np.testing.assert_array_equal(outs[0].cpu().numpy(), outs[1].cpu().numpy())


def test_refused_block_length(dev):  # noqa: F811
    # a block that one wave cannot hold is refused, though four of K=3's would fit beside each other
    torch, vit = dev
    L, blocks = 24000, 5300
    llr = torch.empty(2 * (L * blocks + 2), dtype=torch.float32, device="cuda")
    with pytest.raises(Exception, match="survivor storage"):
        vit.decode(vit.make_code(3, (0o7, 0o5)), llr, L * blocks, L, 15)
