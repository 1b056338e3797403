"""The choice between the decode kernels (csrc/vit_launch.hip), asked through
vit_debug_kernel on the host: what it may choose, over every code size, rate,
type, block length and device size; what it chooses at shapes whose times are
known; and that the GPU tests of each kernel still reach it."""
import ctypes as C
import itertools

import pytest

ONE, MX16, MX4, ROW = range(4)
F32, I8, HARD = range(3)
GENS = {3: (0o7, 0o5, 0o7, 0o5), 4: (0o17, 0o13, 0o15, 0o11), 5: (0o23, 0o35, 0o33, 0o37), 6: (0o53, 0o75, 0o47, 0o71),
        7: (0o171, 0o133, 0o165, 0o117), 8: (0o247, 0o371, 0o331, 0o357), 9: (0o561, 0o753, 0o711, 0o745)}
CUS, LDS = 256, 160 * 1024


def choice(k, gens, llr_type, blocks, L, v, v1=None, cus=CUS, lds=LDS):
    """The kernel, or the status where none takes the blocks."""
    import paper_2011_09337_amd as vit
    code, got = vit.make_code(k, gens), C.c_int32(-1)
    st = vit._lib.lib.vit_debug_kernel(C.byref(code), llr_type, blocks, L, v, -1 if v1 is None else v1, cus, lds,
                                       C.byref(got))
    return got.value if st == 0 else st


@pytest.mark.parametrize("cus,lds", [(CUS, LDS), (32, LDS), (304, 64 * 1024)])
def test_what_may_be_chosen(cus, lds):
    import paper_2011_09337_amd as vit
    seen = set()
    for k, beta, llr_type in itertools.product(range(3, 10), (2, 3, 4), (F32, I8, HARD)):
        gens = GENS[k][:beta]
        body = 32 // (k - 1) * (k - 1)
        for L, v, blocks in itertools.product((8, 64, 256, 520, 2048, 8192, 20480, 65536), (0, 35, 64, 700),
                                              (1, 2, 1000, 5000, 20000, 100000, 1 << 24)):
            got = choice(k, gens, llr_type, blocks, L, v, cus=cus, lds=lds)
            survivors = -(-(L + v) // body) * max(1, 2 ** (k - 1) // 64) * 256  # one block a wave
            exact = llr_type == F32 or (L + v) * 128 * beta < 2 ** 24
            assert (got == vit.VIT_EUNSUPPORTED) == (survivors > lds or not exact), (k, beta, llr_type, L, v)
            if got < 0:
                continue
            allowed = {ONE} if blocks == 1 else {ONE} | (
                ({ROW} if k <= 6 and beta <= 3 else set()) if llr_type == F32 else
                ({MX16} if k >= 6 else set()) | ({MX4} if k <= 7 else set()))
            assert got in allowed, (k, beta, llr_type, L, v, blocks, got)
            seen.add((got, k))
    if cus <= CUS:
        assert {(MX16, k) for k in range(6, 10)} | {(MX4, k) for k in range(3, 8)} | {(ROW, k) for k in range(3, 7)} <= seen
    # a generator without one of the register's ends: the FP32 kernel of four blocks does not take it
    assert choice(5, (0o22, 0o35), F32, 1 << 16, 256, 25) == ONE and choice(5, (0o03, 0o35), F32, 1 << 16, 256, 25) == ONE


def test_at_measured_shapes():
    # 2^24 or 2^22 bits of int8 LLRs, an FP32 stream, a lone frame, sizes either side of a line
    for want, k, llr_type, blocks, L, v in (
            (MX4, 7, I8, 32768, 512, 35), (MX16, 7, I8, 65536, 256, 35), (MX16, 9, I8, 16384, 256, 64),
            (ONE, 9, I8, 1024, 256, 64), (MX4, 5, HARD, 3907, 256, 25), (ONE, 7, I8, 1024, 256, 35),
            (ONE, 7, I8, 1, 1006, 0), (ONE, 8, I8, 4096, 256, 56), (MX16, 8, I8, 16384, 256, 56),
            (ROW, 5, F32, 65536, 256, 25), (ONE, 5, F32, 1024, 256, 25), (ONE, 7, F32, 32768, 512, 35)):
        assert choice(k, GENS[k][:2], llr_type, blocks, L, v) == want, (k, llr_type, blocks, L, v)


def test_the_kernels_own_tests_reach_them():
    import test_gpu_mx as mx
    import test_gpu_mx_quad as quad
    import test_gpu_row as row
    for k, gens in mx.CODES.values():
        if k == 8:  # (in the counts of test_gpu_kernel_reach.py)
            continue
        for L, v, v1 in ((8, 0, 0), (8, 5 * k, None), (16, 3 * k, 3 * k), (64, 8 * k, 0)):
            assert choice(k, gens, I8, mx._blocks(k), L, v, v1) == (MX16 if k > 7 else MX4)
    for k, gens in quad.SMALL.values():
        for L, v, v1 in ((8, 0, 0), (24, 3 * k, None), (480, 40, 7)):
            assert choice(k, gens, I8, 6007, L, v, v1) == MX4
    for k, gens, blocks in quad.WIDE.values():
        for L, v, v1 in ((8, 0, 0), (16, 3 * k, 3 * k), (40, 5 * k, 11)):
            assert choice(k, gens, I8, blocks, L, v, v1) == MX16
    for k, gens in row.CODES.values():
        for L, v, v1 in ((8, 0, 0), (16, 5 * k, None), (96, 3 * k, 3 * k), (240, 40, 7)):
            assert choice(k, gens, F32, 9001, L, v, v1) == ROW


def test_bad_arguments():
    import paper_2011_09337_amd as vit
    for bad in (dict(blocks=0), dict(L=0), dict(v=-1), dict(v1=36), dict(cus=0), dict(lds=0), dict(llr_type=3)):
        args = dict(k=7, gens=GENS[7][:2], llr_type=I8, blocks=5, L=256, v=35)
        args.update(bad)
        assert choice(**args) == vit.VIT_EINVAL, bad
    assert choice(7, (0,), I8, 5, 256, 35) == vit.VIT_EINVAL
