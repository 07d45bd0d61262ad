"""The build's check of the wait states around products that are written out as inline assembly, on small pieces of assembly
with and without mistakes.  No GPU needed."""
import pytest

from paper_2511_21317_amd import build
from paper_2511_21317_amd.isa_check import hazards

PRODUCT = "\t;;#ASMSTART\n\tv_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]\n\t;;#ASMEND"
OTHER = PRODUCT.replace("a[0:3]", "a[4:7]")


def kernel(*lines):
    body = "\n".join(line if line.startswith((".", "\t")) else "\t" + line for line in lines)
    return f"kernel: ; @kernel\n; %bb.0:\n{body}\n\ts_endpgm\n\t.end_amdhsa_kernel kernel\n"


@pytest.mark.parametrize("lines,n", [
    ((PRODUCT,), 1),
    (("v_mov_b32_e32 v4, v0", "s_nop 1", PRODUCT), 1),                               # two states
    (("v_mov_b32_e32 v4, v0", "s_nop 0", "v_mov_b32_e32 v20, v0", PRODUCT), 1),
    (("v_mov_b32_e32 v12, v4", PRODUCT, OTHER, PRODUCT, OTHER), 4),                  # reads, other results, sums in a chain
    ((PRODUCT, "s_nop 15", "s_nop 2", "v_accvgpr_read_b32 v0, a3"), 1),
    (("v_accvgpr_write_b32 a3, 0", "s_nop 1", PRODUCT), 1),
    (("v_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], 0", "v_accvgpr_read_b32 v0, a3"), 0),     # the compiler's own
    (("ds_read_b128 v[4:7], v0", "s_waitcnt lgkmcnt(0)", PRODUCT), 1),
])
def test_what_keeps_its_distance_passes(lines, n):
    assert hazards(kernel(*lines)) == (n, [])


@pytest.mark.parametrize("lines", [
    ("v_mov_b32_e32 v4, v0", PRODUCT),
    ("v_mov_b32_e32 v11, v0", "s_nop 0", PRODUCT),
    ("v_cvt_pk_bf16_f32 v9, v0, v1", "s_mov_b32 s0, 0", PRODUCT),
    ("v_permlane16_swap_b32_e32 v0, v8", PRODUCT),                                    # writes both
    ("v_accvgpr_write_b32 a3, 0", PRODUCT),
    ("v_cmpx_gt_i32_e32 v0, v1", "s_nop 2", PRODUCT),
    (PRODUCT, "v_accvgpr_read_b32 v0, a3"),
    (PRODUCT, "s_nop 15", "s_nop 1", "v_accvgpr_read_b32 v0, a0"),
    (PRODUCT, "v_accvgpr_write_b32 a2, 0"),
    (PRODUCT, "v_mfma_f32_16x16x32_bf16 v[0:3], v[4:7], a[0:3], 0"),
    (PRODUCT, PRODUCT.replace("v[4:7]", "a[0:3]")),                                   # as an operand, not as the sum
    (PRODUCT, PRODUCT.replace("a[0:3]", "a[2:5]")),                                   # overlapping sums
    ("v_mfma_f32_16x16x32_bf16 v[4:7], v[20:23], v[24:27], 0", "s_nop 7", PRODUCT),
    (PRODUCT, "s_nop 15", "s_nop 15", "scratch_store_dword off, v0, off"),
], ids=range(14))
def test_what_does_not_is_found(lines):
    assert hazards(kernel(*lines))[1]


def test_every_path_is_followed():
    loop = (".LBB0_1:", PRODUCT, "s_nop 7", "v_mov_b32_e32 v5, v0", "s_cbranch_scc1 .LBB0_1", "s_nop 15", "s_nop 15")
    assert len(hazards(kernel(*loop))[1]) == 1                                        # around the loop, one state away
    assert not hazards(kernel(*loop[:4], "s_nop 0", *loop[4:]))[1]
    skip = (PRODUCT, "s_branch .LBB0_2", ".LBB0_1:", "s_nop 15", "s_nop 15", ".LBB0_2:", "v_accvgpr_read_b32 v0, a0")
    assert hazards(kernel(*skip))[1]
    far = (PRODUCT, "s_getpc_b64 s[0:1]", "s_add_u32 s0, s0, (.LBB0_2-.Lpost_getpc0)&4294967295", "s_addc_u32 s1, s1, (.LBB0_2-.Lpost_getpc0)>>32",
           "s_setpc_b64 s[0:1]", *skip[2:])
    assert hazards(kernel(*far))[1]


def test_every_function_is_looked_at():
    bad, good = kernel("v_mov_b32_e32 v4, v0", PRODUCT), kernel(PRODUCT)
    function = bad.replace("kernel", "function").replace("\ts_endpgm\n\t.end_amdhsa_kernel function\n", "\ts_setpc_b64 s[30:31]\n")
    for asm in (bad + good, good + bad, function + good, good + function):
        n, found = hazards(asm)
        assert n == 2 and len(found) == 1


def test_a_build_with_them_is_refused(tmp_path):
    path = tmp_path / "attention-hip-amdgcn-amd-amdhsa-gfx950.s"
    path.write_text(kernel(PRODUCT))
    build._check_products([str(path)])
    path.write_text(kernel("v_mov_b32_e32 v4, v0", PRODUCT))
    with pytest.raises(RuntimeError, match="wait states"):
        build._check_products([str(path)])
    path.write_text(kernel("s_nop 0"))
    with pytest.raises(RuntimeError, match="none were checked"):
        build._check_products([str(path)])
