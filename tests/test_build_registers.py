"""The build's check of the registers that the matrix-core kernels name
(paper_2011_09337_amd/build.py): an instruction of the compiler's own on one of
them, alone, in a range, or on an AGPR, stops the build; those inside asm, below
the first named one, or in other kernels do not."""
import importlib.util
import os

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
KERNEL = "_ZN3vit4devm%sILi7ELi2ELi1EEEvNS_10DecodeArgsE:\n"


@pytest.fixture(scope="module")
def check():
    spec = importlib.util.spec_from_file_location("vit_build", os.path.join(ROOT, "paper_2011_09337_amd", "build.py"))
    build = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(build)
    return build.check_named_registers


@pytest.mark.parametrize("kind,first", [("21vit_blocked_mx_kernel", 128), ("20vit_batch_quad_kernel", 64)])
def test_own_use_is_found(check, tmp_path, kind, first):
    asm = tmp_path / "k.s"
    fine = KERNEL % kind + f"\tv_mov_b32_e32 v{first - 1}, s2 ; v{first}\n\t;;#ASMSTART\n\tv_mov_b32 v{first}, v1\n\t;;#ASMEND\n"
    asm.write_text(fine)
    check(str(asm))
    for bad in (f"\tv_add_u32_e32 v3, v{first}, v2\n", f"\tds_read_b64 v[{first - 1}:{first}], v0\n",
                "\tv_accvgpr_write_b32 a3, v2\n", "\tv_mov_b32_e32 v255, 0\n"):
        asm.write_text(fine + bad)
        with pytest.raises(RuntimeError, match="register that the kernel names"):
            check(str(asm))
    asm.write_text("\tv_mov_b32_e32 v255, 0\n")
    with pytest.raises(RuntimeError, match="no matrix-core kernel"):
        check(str(asm))
