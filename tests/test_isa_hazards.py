"""The built gfx950 code keeps the distances that inline assembly takes out of the compiler's hands."""
import glob
import os
import re

import pytest

import paper_2507_16099_amd as fp8
from tests.isa_hazards import check_kernel, disassemble

MFMA = "v_mfma_f32_16x16x128_f8f6f4 a[0:3], v[0:7], v[8:15], a[0:3]"


@pytest.mark.parametrize("bad,text", [
    (True, ["v_accvgpr_write_b32 a3, v20", MFMA]),
    (True, ["v_mov_b32_e32 v9, 0", "s_nop 0", MFMA]),
    (False, ["v_accvgpr_write_b32 a3, v20", "s_nop 1", MFMA, MFMA]),
    (True, [MFMA, "s_nop 10", "v_accvgpr_read_b32 v0, a0"]),
    (False, [MFMA, "s_nop 11", "v_accvgpr_read_b32 v0, a0"]),
    (True, ["global_load_dword v1, v[2:3], off", "buffer_load_dwordx4 v4, s[0:3], 0 offen lds", "s_waitcnt vmcnt(2)", "v_mov_b32_e32 v1, 0"]),
    (False, ["global_load_dword v1, v[2:3], off", "buffer_load_dwordx4 v4, s[0:3], 0 offen lds", "s_waitcnt vmcnt(1)", "v_mov_b32_e32 v1, 0"]),
    (True, ["global_store_dwordx4 v[2:3], v[4:7], off sc0 sc1", "s_nop 0", "v_mov_b32_e32 v6, 0"]),
    (False, ["global_store_dwordx4 v[2:3], v[4:7], off sc0 sc1", "s_nop 1", "v_mov_b32_e32 v6, 0"]),
    (False, ["global_store_dwordx4 v[2:3], v[4:7], off sc0 sc1", "v_mov_b32_e32 v2, 0"]),          # the address
    (True, ["buffer_store_dwordx4 v[4:7], v2, s[0:3], 0 offen", "v_mov_b32_e32 v4, 0"]),
    (False, ["buffer_store_dwordx4 v[4:7], v2, s[0:3], s5 offen", "v_mov_b32_e32 v4, 0"]),
    (True, ["global_load_dword v1, v[2:3], off", "s_cbranch_scc1 1", "s_waitcnt vmcnt(0)", "v_mov_b32_e32 v1, 0"]),    # one path waits
])
def test_the_check_itself(bad, text):
    code = [(4 * n, *line.split(" ", 1)) for n, line in enumerate([*text, "s_endpgm "])]
    assert bool(check_kernel(code)) == bad


def test_no_instruction_comes_too_early():
    kernels = disassemble(fp8.library_path())
    assert any("gemm_fp8_ring" in name for name in kernels) and any("gemm_fp8_stream" in name for name in kernels)
    found = {name: bad for name, code in kernels.items() if (bad := check_kernel(code))}
    assert not found, {name: bad[:3] for name, bad in found.items()}


def test_assembly_loads_write_no_register():
    """A register that an assembly load will write counts as written for the compiler from the load on.  Loads in assembly
    therefore write LDS; the one exception holds its registers as operands of the wait that follows."""
    csrc = os.path.join(os.path.dirname(fp8.library_path()), "csrc")
    found, read = [], set()
    for path in sorted(glob.glob(os.path.join(csrc, "*.h*"))):      # (kernels lie in headers too)
        for m in re.finditer(r"asm volatile\((.*?)\);", open(path).read(), re.S):
            if "_load_" in m[1]:
                read.add(os.path.basename(path))
                if '"=' in m[1]:
                    found.append(os.path.basename(path))
    assert found == ["gemm_fp8_skinny_fused.hip"]
    assert read >= {"gemm_fp8_ring.hpp", "gemm_fp8_stream.hpp", "gemm_fp8_few_stream.hip", "gemm_fp8_skinny.hip", "gemm_fp8_snake.hip", "gemm_mxfp8_snake.hip",
                    "gemm_bf16_at_b_snake.hip"}, read      # no file is left out unseen


def test_codes_are_stored_through_the_l2_or_past_it():
    """Plain stores of codes leave dirty lines that the end of a quantization kernel waits for (3-18 % of its time).  Only the
    rowwise kernel's form for few tokens (last template argument) stores plainly."""
    plain = {}
    for name, code in disassemble(fp8.library_path()).items():
        if re.search(r"\d(quant_row_kernel|cast_kernel|cast_transpose_kernel|mx_quant\w*_kernel|block_quant\w*_kernel)I", name):
            stores = [args for _, op, args in code if op in ("global_store_dwordx2", "global_store_dwordx4")]
            assert stores, name
            few = re.search(r"quant_row_kernelI(Li\d+E)+Lb1E", name)
            if not few and (bad := [args for args in stores if not re.search(r"\bsc0 sc1\b|\bnt\b", args)]):
                plain[name] = bad[0]
    assert not plain


def test_assembly_stores_carry_their_wait_states():
    """The compiler does not see a 128-bit store in assembly, so the two wait states before its data may be written are part of
    the assembly, whatever happens to follow in today's code."""
    followers = {(code[k + 1][1], code[k + 1][2]) for code in disassemble(fp8.library_path()).values()
                 for k, (_, op, args) in enumerate(code) if op == "global_store_dwordx4" and "sc0 sc1" in args}
    assert followers == {("s_nop", "1")}
