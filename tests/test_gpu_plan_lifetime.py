"""What outlives a call of `Batch.decode`: a plan that is closed or dropped has
waited for its decodes, on every stream they were queued on, so that nothing
reads its workspace any more; a workspace that a larger one replaces is not
handed out again while a decode on another stream still reads it."""
import numpy as np
import pytest

from test_gpu_int16 import dev  # noqa: F401

pytestmark = pytest.mark.gpu


def _batch(dev, frames=4000, n=4096):  # noqa: F811
    # K=9, some half a millisecond of decode kernels behind the work list's
    torch, vit = dev
    code = vit.make_code(9, (0o561, 0o753))
    llr = torch.randint(-20, 21, (frames * (n + 8) * 2,), dtype=torch.int8, device="cuda")
    recs = [(0, 1, n, f * (n + 8) * 2, f * (n // 8)) for f in range(frames)]
    return [code], vit._lib.frames_array(recs), llr, (256, 64, -1, 1), frames * (n // 8)


@pytest.mark.parametrize("drop", ["close", "del"])
def test_a_closed_plan_has_no_work_left(dev, drop):  # noqa: F811
    torch, vit = dev
    codes, frames, llr, tune, nbytes = _batch(dev)
    want = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    keep = vit.Batch()
    keep.decode(codes, frames, llr, want, tune=[tune])
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    out = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    b = vit.Batch()
    b.decode(codes, frames, llr, out, tune=[tune], stream=side)
    if drop == "close":
        b.close()
    else:
        del b
    assert side.query()
    np.testing.assert_array_equal(out.cpu().numpy(), want.cpu().numpy())


def test_a_closed_plan_has_no_work_left_on_an_earlier_stream(dev):  # noqa: F811
    # the third call takes the first one's staging and event again, on another stream
    torch, vit = dev
    codes, frames, llr, tune, nbytes = _batch(dev)
    first, second = torch.cuda.Stream(), torch.cuda.Stream()
    out = [torch.zeros(nbytes, dtype=torch.uint8, device="cuda") for _ in range(2)]
    torch.cuda.synchronize()
    b = vit.Batch()
    b.decode(codes, frames, llr, out[0], tune=[tune], stream=first)
    kept = []
    for _ in range(2):  # workspaces of their own: calls that overlap may not share one
        kept.append(b.ws)
        b.ws = None
        b.decode(codes, frames[:1], llr, out[1], tune=[tune], stream=second)
    b.close()
    assert first.query() and second.query()
    n = 4096 // 8
    np.testing.assert_array_equal(out[0].cpu().numpy()[:n], out[1].cpu().numpy()[:n])


def test_a_replaced_workspace_is_held(dev):  # noqa: F811
    torch, vit = dev
    codes, frames, llr, tune, nbytes = _batch(dev)
    side = torch.cuda.Stream()
    out = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    b = vit.Batch()
    b.decode(codes, frames[:8], llr, out, tune=[tune], stream=side)
    old, size = b.ws.data_ptr(), b.ws.numel()
    b.decode(codes, frames, llr, out, tune=[tune], stream=side)
    assert b.ws.numel() >= 2 * size
    others = [torch.empty(size, dtype=torch.uint8, device="cuda") for _ in range(4)]
    held = all(old != x.data_ptr() for x in others)
    b.close()
    assert held and side.query()
