"""The serving loop's copy of frames from pinned host memory: every alignment of
a frame's first LLR and lengths around the 16-byte words, the 63 words a wave
stores at a time and the rounds of a workgroup.  Bit for bit against the CPU
oracle's exact integer decoder; the LLRs around each frame are other frames'."""
import numpy as np
import pytest

import synth
from oracle import vref
from test_gpu_int16 import dev  # noqa: F401

pytestmark = pytest.mark.gpu

K, GENS = 3, (0o7, 0o5)
# LLR bytes of a frame (2 a bit, open end)
BYTES = [2, 4, 14, 16, 18, 30, 32, 34, 62, 64, 1006, 1008, 1010, 1022, 1024, 1026, 4030, 4032, 4034, 4046, 4048, 4096,
         16126, 16128, 16130, 20000]


@pytest.mark.parametrize("step", [0, 1, 5])
def test_every_alignment(dev, step):  # noqa: F811
    torch, vit = dev
    rng = np.random.default_rng(step)
    sizes = [b for b in BYTES for _ in range(16)]
    starts, at = [], 64
    for i, b in enumerate(sizes):
        at += (i % 16 + (16 - at % 16)) % 16 if step == 0 else step  # step 0: each length at each offset within a word
        starts.append(at)
        at += b
    total = (at + 63) // 64 * 64
    n = np.array(sizes) // 2
    out_off = total + np.cumsum((n + 15) // 8) - (n + 15) // 8
    host = torch.zeros(int(out_off[-1] + n[-1] // 8 + 64), dtype=torch.uint8, pin_memory=True)
    llr = rng.integers(-30, 31, size=total).astype(np.int8)
    host[:total] = torch.from_numpy(llr.view(np.uint8))
    print(f"[gpu] serving {n.size} frames, step {step}", flush=True)
    server = vit.Server([vit.make_code(K, GENS)], host, tune=[(64, 16, -1, 1)], llr_type=vit.VIT_LLR_I8,
                        arena_bytes=8 << 20, max_frames=1024, max_items=65536)
    req = server.requests(n.size)
    req["code_id"], req["terminated"], req["n"] = 0, 0, n
    req["llr"], req["out"], req["tag"] = host.data_ptr() + np.array(starts), host.data_ptr() + out_off, np.arange(n.size)
    sent = 0
    while sent < n.size:
        sent += server.submit(req[sent:])[1]
    server.drain()
    done = server.poll()
    server.close()
    assert len(done) == n.size and (done["status"] == vit.VIT_OK).all()
    got, code = host.numpy(), vref.make_code(K, list(GENS))
    for i in range(n.size):
        sub = llr[starts[i]:starts[i] + sizes[i]]
        want = synth.pack_bits(vref.decode_blocked(code, sub, int(n[i]), 64, 8, 8, False))
        np.testing.assert_array_equal(got[out_off[i]:out_off[i] + want.size], want, err_msg=f"{sizes[i]} bytes at {starts[i]}")
