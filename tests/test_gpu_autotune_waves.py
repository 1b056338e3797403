"""Autotuned shapes: two waves per workgroup are a choice only where the kernel
that runs the shape has such workgroups."""
import numpy as np
import pytest

import synth
from test_gpu_int16 import dev  # noqa: F401
from test_kernel_choice import F32, I8, ONE, choice

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,dtype", [("k7r12", "int8"), ("k9r12", "int8"), ("k5r12", "float32")])
def test_waves_of_the_kernels_of_many_blocks(dev, name, dtype):  # noqa: F811
    torch, vit = dev
    k, gens = synth.CODES.get(name, (5, (0o23, 0o35)))
    rng = np.random.default_rng(k)
    n, count = 2048, 4000
    size = (n + k - 1) * 2
    coded = synth.encode(k, gens, synth.info_bits(n, rng), True)
    one = 8 * (1.0 - 2.0 * coded) + 3 * rng.standard_normal(size)
    llr = np.tile((np.rint(one) if dtype == "int8" else one).astype(dtype), count)
    frames = [(0, 1, n, f * size, f * (n // 8)) for f in range(count)]
    out = torch.zeros(count * (n // 8), dtype=torch.uint8, device="cuda")
    print(f"[gpu] autotune {name} {dtype}: {count} frames", flush=True)
    b = vit.Batch()
    L, v, v1, waves = b.autotune([vit.make_code(k, gens)], frames, torch.from_numpy(llr).cuda(), out)[0]
    b.close()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    ran = choice(k, gens, I8 if dtype == "int8" else F32, count * -(-n // L), L, v, v1, cus)
    assert ran != ONE and waves == 1, (L, v, v1, waves, ran)
