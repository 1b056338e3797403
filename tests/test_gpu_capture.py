"""Calls on a stream that is being captured: a batch is refused (its work list
comes from staging that later calls rewrite) and leaves plan and capture as they
were; a stream decode is captured and replays as it ran."""
import numpy as np
import pytest

import synth
from test_gpu_int16 import dev  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("used_before", [False, True])
def test_batch_is_refused(dev, used_before):  # noqa: F811
    torch, vit = dev
    k, gens = synth.CODES["k7r12"]
    code, n = [vit.make_code(k, gens)], 777
    llr = torch.randint(-20, 21, ((n + k - 1) * 2,), dtype=torch.int8, device="cuda")
    want = vit.decode(code[0], llr, n, 256, 35).cpu().numpy()
    out = torch.zeros((n + 7) // 8, dtype=torch.uint8, device="cuda")
    mark = torch.zeros(1, device="cuda")
    b = vit.Batch()
    if used_before:
        b.decode(code, [(0, 1, n, 0, 0)], llr, out, tune=[(256, 35, -1, 1)])
    b._workspace(vit.codes_array(code), vit.frames_array([(0, 1, n, 0, 0)]), None)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        mark += 1
        with pytest.raises(vit.VitError, match="captured") as e:
            b.decode(code, [(0, 1, n, 0, 0)], llr, out, tune=[(256, 35, -1, 1)])
        assert e.value.status == vit.VIT_EUNSUPPORTED
    for turn in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert int(mark.item()) == turn + 1 and not out.any()
        b.decode(code, [(0, 1, n, 0, 0)], llr, out, tune=[(256, 35, -1, 1)])
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy(), want)
    b.close()


@pytest.mark.parametrize("name,n", [("k7r12", 777), ("k7r12", 1 << 21), ("k9r12", 1 << 20)])
@pytest.mark.parametrize("dtype", ["float32", "int8"])
def test_stream_decode_replays(dev, name, n, dtype):  # noqa: F811
    torch, vit = dev
    k, gens = synth.CODES[name]
    code = vit.make_code(k, gens)
    rng = np.random.default_rng(n)
    inputs = [torch.from_numpy(rng.integers(-20, 21, (n + k - 1) * 2).astype(dtype)).cuda() for _ in range(3)]
    eager = [vit.decode(code, x, n, 256, 64).cpu().numpy() for x in inputs]
    llr, out = inputs[0].clone(), torch.zeros((n + 7) // 8, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        vit.decode(code, llr, n, 256, 64, out=out)
    for x, want in zip(inputs, eager):
        llr.copy_(x)
        g.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy(), want)
        vit.decode(code, inputs[1], n, 256, 64)  # the program's own work between the replays
        torch.cuda.synchronize()
