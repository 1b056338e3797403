"""A batch's work list as the device writes it from the frames' records, where
a block could be lost or written twice: frames of 1, 2 and 3 blocks and of as
many as a record holds, one fewer, one more and several records' worth; cores
that end on a block edge and one bit to either side; overlaps longer than a
block, so that several blocks of a frame are clipped at either end; a code with
no frames; two calls in a row that leave the plan's staging slots in turn."""
import numpy as np
import pytest

from test_gpu_batch import CODES, check_frames, dev, run_batch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("int8", [True, False])
@pytest.mark.parametrize("v", [0, 12, 45])
def test_records_cover_every_block_once(dev, int8, v):  # noqa: F811
    _, vit = dev
    tune = [(8, v, -1, 1), (16, v, v, 2), (8, v, 0, 1), (24, v, -1, 1), (8, v, -1, 3)]
    rng = np.random.default_rng(v + int8)
    b = vit.Batch()
    for call in range(3):
        frames, llr_off, out_off = [], 3, 1
        for nb in (1, 2, 3, 255, 256, 257, 512, 770):
            for cid in (0, 1, 3, 4):  # code 2 has no frames
                n = max(1, nb * tune[cid][0] - int(rng.integers(0, 2)) * int(rng.integers(0, tune[cid][0])))
                term = int(rng.integers(0, 2))
                k, gens = CODES[cid]
                frames.append((cid, term, n, llr_off, out_off))
                llr_off += (n + (k - 1) * term) * len(gens) + int(rng.integers(0, 3))
                out_off += (n + 7) // 8 + int(rng.integers(0, 2))
        order = rng.permutation(len(frames))
        frames = [frames[i] for i in order]
        llr = rng.integers(-128, 128, size=llr_off).astype(np.int8)
        llr = llr if int8 else llr.astype(np.float32)
        got = run_batch(dev, b, frames, llr, out_off, None, tune)
        check_frames(got, frames, llr, tune)
    b.close()
