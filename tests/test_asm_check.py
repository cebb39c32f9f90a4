"""The build's checks of compiled code: mistakes planted in text are found, and the assembly that the compiler makes of the attention kernels and of a
store at a scalar offset today has none."""
import re
import shutil

import pytest

from paper_2602_00608_amd import asm_check, build

CHAIN = ["v_mfma_f32_32x32x16_f16 v[0:15], v[20:23], v[30:33], 0", "v_mfma_f32_32x32x16_f16 v[0:15], v[24:27], v[34:37], v[0:15]"]
SETTLE = ["s_nop 15", "s_nop 7"]


@pytest.mark.parametrize("lines,faults", [
    (CHAIN + SETTLE + ["v_max3_f32 v40, v0, v1, v2"], 0),
    (CHAIN + ["s_nop 10", "v_max3_f32 v40, v0, v1, v2"], 1),                                      # one state short
    (CHAIN + ["v_add_f32 v50, v51, v52"] * 12 + ["v_max3_f32 v40, v0, v1, v2"], 0),               # other work is a wait too
    (CHAIN[:1] + ["v_mov_b32 v41, v15"] + CHAIN[1:] + SETTLE, 1),                                 # a copy between two of a chain
    (CHAIN[:1] + ["scratch_store_dword off, v3, off"] + SETTLE, 1),                               # a spill
    (CHAIN[:1] + ["v_mfma_f32_32x32x16_f16 a[0:15], v[0:3], v[30:33], a[0:15]"] + SETTLE, 1),     # a result as another's operand
    (["v_mov_b32 v24, v60"] + CHAIN + SETTLE, 1),                                                 # operand one instruction before its use
    (["v_mov_b32 v24, v60", "s_nop 0"] + CHAIN + SETTLE, 0),
    (["v_accvgpr_read_b32 v20, a3"] + CHAIN + SETTLE, 1),
    (["v_permlane32_swap_b32 v60, v20"] + CHAIN + SETTLE, 1),                                     # writes both of its registers
    ([".LBB0_1:", "v_mov_b32 v60, v0", "s_nop 1"] + CHAIN + ["s_cbranch_scc1 .LBB0_1"] + SETTLE, 1),   # round the loop
    (CHAIN + ["s_cbranch_scc1 .LBB0_2"] + SETTLE + [".LBB0_2:", "ds_write_b32 v70, v9"], 1),      # past a branch
    (CHAIN + ["s_cbranch_scc1 2f", "1:", ".subsection 1", "2:", "v_mul_f32 v0, v0, v1", ".subsection 0"] + SETTLE, 0),
])
def test_planted_mistakes_are_found(lines, faults):
    assert len(asm_check.check_code(lines)) == faults


LATE = "buffer_store_dwordx4 v[4:7], v2, s[8:11], s3 offen"


@pytest.mark.parametrize("lines,faults", [
    ([LATE, "s_nop 1", "v_mov_b32_e32 v4, v9"], 0),
    ([LATE, "s_nop 0", "v_mov_b32_e32 v7, v9"], 1),                                      # one state short
    ([LATE, "v_add_f32_e32 v8, v9, v10", "v_mul_f32_e32 v5, v8, v9"], 1),
    ([LATE, "v_add_f32_e32 v8, v4, v10", "s_mov_b32 s0, 1", "v_mul_f32_e32 v5, v8, v9"], 0),   # reading it is no fault
    ([LATE, "v_permlane16_swap_b32_e32 v20, v6"], 1),                                    # writes both of its registers
    ([LATE, "v_mfma_f32_16x16x32_f16 v[6:9], v[20:23], v[30:33], 0"], 1),
    ([LATE, "s_cbranch_scc1 .LBB0_2", "s_nop 1", ".LBB0_2:", "v_mov_b32_e32 v5, 0"], 1),       # past a branch
    (["buffer_store_dwordx4 a[4:7], v2, s[8:11], s3 offen", "v_accvgpr_write_b32 a5, v0"], 1),
    (["buffer_store_dwordx4 a[4:7], v2, s[8:11], s3 offen", "v_mov_b32_e32 v5, v0"], 0),
    (["buffer_store_dwordx4 v[4:7], v2, s[8:11], 0 offen", "v_mov_b32_e32 v5, v0"], 0),  # the compiler waits for these itself
    (["buffer_store_dwordx2 v[4:5], v2, s[8:11], s3 offen", "v_mov_b32_e32 v5, v0"], 0),
])
def test_overwritten_store_data_is_found(lines, faults):
    text = "\n".join(["_Z6kernel:"] + ["\t" + l for l in lines] + ["\ts_endpgm", ".Lfunc_end0:"])
    assert len(asm_check.check_source(text)) == faults


def test_store_at_a_scalar_offset_as_compiled(tmp_path):
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not on PATH")
    src = tmp_path / "store.hip"
    src.write_text("""#include "%s/conv_device.hpp"
using namespace wmdec;
__global__ void store_kernel(float* y, const u32x4* x, int bytes, int rows, int stride) {
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(y, 0, bytes, 0x00020000);
  u32x4 v = x[threadIdx.x];
  for (int r = 0; r < rows; ++r) {
    store_vector(rsrc, v, threadIdx.x * 16, r * stride);
    for (int k = 0; k < 4; ++k) v[k] = v[k] * 3u + r;
  }
}
""" % build.CSRC)
    text = build.device_assembly(str(src))
    stores = [l.strip() for _, lines in asm_check.functions(text) for l in lines if "buffer_store_dwordx4" in l]
    assert stores and asm_check.check_source(text, spills="store_kernel") == []
    data = re.search(r"v\[(\d+):", stores[0]).group(1)
    planted = text.replace(stores[0], stores[0] + "\n\tv_mov_b32_e32 v%s, 0" % data, 1)
    assert len(asm_check.check_source(planted)) == 1
    spilled = re.sub(r"(\.vgpr_spill_count: +)0", r"\g<1>3", text)
    assert any("vgpr_spill_count is 3" in f for f in asm_check.check_source(spilled, spills="store_kernel"))


def test_attention_core_as_compiled():
    if shutil.which("hipcc") is None:
        pytest.skip("hipcc not on PATH")
    text = build.device_assembly("kernels_attn.hip")
    assert asm_check.check(text, "flash_attn_kernel") == []
    assert asm_check.check(text, "no_such_kernel") == ["no instance of no_such_kernel"]
    # the same code with a copy of a result in flight behind its last matrix instruction, and with a spill on record
    score = list(re.finditer(r"\tv_mfma\S+ v\[(\d+):\d+\].*\n", text))[-1]
    copied = text[:score.end()] + "\tv_mov_b32 v1, v%s\n" % score.group(1) + text[score.end():]
    assert any("touched early" in f for f in asm_check.check(copied, "flash_attn_kernel"))
    spilled = re.sub(r"(\.vgpr_spill_count: +)0", r"\g<1>3", text)
    assert any("vgpr_spill_count is 3" in f for f in asm_check.check(spilled, "flash_attn_kernel"))
