"""Every kernel of the choice in csrc/vit_launch.hip, at block counts for which the
library says that this kernel runs: the 16-register matrix-core kernel of k = 8 at
all its rates and inputs, that of k = 6, 7 with survivors in LDS, the 4-register
one with many more bodies than registers hold, and the fp32 sums of k = 9 where
blocks begin within a period. Against the CPU oracle, bit for bit."""
import numpy as np
import pytest

import synth
from oracle import vref
from test_gpu_int16 import dev  # noqa: F401
from test_gpu_mx import CODES, _check, _values
from test_gpu_mx_quad import SMALL
from test_kernel_choice import HARD, I8, MX16, MX4, choice

pytestmark = pytest.mark.gpu

COUNTS = (2003, 3001, 4507, 6007, 8009, 12007, 20011, 30011, 50021, 70001, 100003)
CODES8 = {name: CODES[name] for name in ("k8r12", "k8r13", "k8r14")}
CODES8.update({"k8r12x": (8, (0o246, 0o371)), "k8r13y": (8, (0o147, 0o331, 0o367))})  # not all taps at both ends


def _blocks(dev, want, k, gens, llr_type, L, v, v1):  # noqa: F811
    props = dev[0].cuda.get_device_properties(0)
    for count in COUNTS:  # (one more: the last block may be of a few bits)
        if all(choice(k, gens, llr_type, c, L, v, v1, props.multi_processor_count) == want for c in (count, count + 1)):
            return count
    raise AssertionError(f"no count up to {COUNTS[-1]} reaches kernel {want}: k={k} L={L} v={v}")


def _run(dev, want, k, gens, kind, L, v, v1, terminated, extra, what):  # noqa: F811
    rng = np.random.default_rng([k, len(gens), len(kind), L])
    n = L * _blocks(dev, want, k, gens, HARD if kind == "hard" else I8, L, v, v1) + extra
    if kind in ("low", "high"):
        llr = np.full((n + (k - 1 if terminated else 0)) * len(gens), -128 if kind == "low" else 127, dtype=np.int8)
    else:
        llr = _values(kind, k, gens, n, terminated, rng)
    _check(dev, k, gens, llr, n, L, v, v1, terminated, f"{what} {kind} L={L} v={v} v1={v1}")


@pytest.mark.parametrize("kind", ["awgn", "ties", "extreme", "hard"])
@pytest.mark.parametrize("name", sorted(CODES8))
def test_k8_sixteen_registers(dev, name, kind):  # noqa: F811
    # windows of less than a body to beyond the eight bodies that registers hold
    k, gens = CODES8[name]
    for L, v, v1, terminated, extra in ((8, 0, 0, True, 1), (8, 40, None, False, 0), (16, 24, 24, True, -7),
                                        (64, 64, 0, False, 13), (200, 56, None, True, 5), (256, 64, 11, False, -1),
                                        (400, 56, None, True, 3)):
        _run(dev, MX16, k, gens, kind, L, v, v1, terminated, extra, name)


@pytest.mark.parametrize("kind", ["ties", "extreme", "hard"])
@pytest.mark.parametrize("name", ["k6r12", "k6r13", "k6r14", "k7r12", "k7r13", "k7r14"])
def test_sixteen_registers_with_survivors_in_lds(dev, name, kind):  # noqa: F811
    # 8, 9, 10 and 12 traced bodies of 30 stages
    k, gens = CODES[name]
    for L, v, v1, terminated, extra in ((200, 40, 0, True, 1), (240, 17, 10, False, -3), (256, 5 * k, None, True, 9),
                                        (320, 40, 11, True, 0)):
        _run(dev, MX16, k, gens, kind, L, v, v1, terminated, extra, name)


@pytest.mark.parametrize("kind", ["ties", "extreme", "hard"])
@pytest.mark.parametrize("name", ["k3r12", "k3r14x", "k4r13x", "k4r14", "k5r12", "k5r13x", "k6r12", "k7r14"])
def test_four_registers_with_many_bodies(dev, name, kind):  # noqa: F811
    k, gens = {**CODES, **SMALL}[name]
    for L, v, v1, terminated, extra in ((720, 4 * k, None, False, 1), (1200, 13, 13, True, 3)):
        _run(dev, MX4, k, gens, kind, L, v, v1, terminated, extra, name)


@pytest.mark.parametrize("kind", ["extreme", "low", "high", "ties"])
@pytest.mark.parametrize("name", ["k8r14", "k9r12", "k9r13", "k9r14"])
def test_starts_within_a_period(dev, name, kind):  # noqa: F811
    # the first block is shorter than its neighbours by v1, so that it starts (in
    # state 0, the others far below) at every offset from a period's end and from
    # the stages at which the fp32 sums are taken back
    k, gens = CODES[name]
    for v1 in range(1, 34, 3 if kind == "ties" else 1):
        _run(dev, MX16, k, gens, kind, 40, v1 + 9, v1, True, 5, name)


@pytest.mark.parametrize("hard", [False, True])
@pytest.mark.parametrize("name", ["k8r13", "k8r14"])
def test_batch_of_k8(dev, name, hard):  # noqa: F811
    torch, vit = dev
    k, gens = CODES[name]
    rng = np.random.default_rng([k, len(gens), hard])
    L, v, frames, off, out_off, items = 96, 56, [], 0, 0, 0
    for _ in range(5001):
        n = int(rng.integers(1, 701))
        term = int(rng.random() < 0.6) if n > 1 else 1
        frames.append((0, term, n, off, out_off))
        off += (n + (k - 1) * term) * len(gens)
        out_off += (n + 7) // 8
        items += -(-n // L)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert choice(k, gens, HARD if hard else I8, items, L, v, None, cus) == MX16
    llr = rng.integers(0, 2, off).astype(np.uint8) if hard else rng.integers(-128, 128, off).astype(np.int8)
    out = torch.full((out_off,), 0xAB, dtype=torch.uint8, device="cuda")
    print(f"[gpu] mx batch {name} hard={hard}: {items} items", flush=True)
    b = vit.Batch()
    b.decode([vit.make_code(k, gens)], frames, torch.from_numpy(llr).cuda(), out, tune=[(L, v, -1, 1)])
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    b.close()
    code = vref.make_code(k, list(gens))
    exact = 1 - 2 * llr.astype(np.int8) if hard else llr
    for _, term, n, lo, oo in frames:
        sub = exact[lo:lo + (n + (k - 1) * term) * len(gens)]
        want = synth.pack_bits(vref.decode_blocked(code, sub, n, L, v // 2, v - v // 2, bool(term)))
        np.testing.assert_array_equal(got[oo:oo + want.size], want, err_msg=f"frame of {n} bits at {lo}")
