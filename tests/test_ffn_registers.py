"""The bf16 expert products name their accumulation registers in asm statements.  That holds as long as the compiler itself uses
none of them and the wait states of the matrix instructions are kept; the build reads both off the assembly of the object that
it links (paper_2503_05066_amd/accumulators.py)."""
import os
import subprocess

import pytest

from paper_2503_05066_amd import accumulators, build

HEAD = """
kernel:
\tds_read_b128 v[8:11], v1
\tds_read_b128 v[12:15], v1 offset:64
\ts_waitcnt lgkmcnt(0)
\ts_nop 1
"""
MATRIX = "\t;;#ASMSTART\n\tv_mfma_f32_16x16x32_bf16 a[4:7], v[8:11], v[12:15], a[4:7]\n\t;;#ASMEND\n"


@pytest.fixture
def hipcc():
    try:
        return build._hipcc()
    except RuntimeError:
        pytest.skip("no hipcc")


def test_accumulators_belong_to_the_asm_statements(hipcc, tmp_path):
    out = tmp_path / "ffn.s"
    subprocess.run([hipcc, *build.COMMON, "--cuda-device-only", "-S", os.path.join(build.CSRC, "ffn.hip"), "-o", str(out)],
                   check=True, capture_output=True, timeout=600)
    # every height of a tile, twice (how its weights are fetched), in three kernels
    assert accumulators.check(out.read_text()) > 5000
    # FLAT accesses wait for every request in flight; LDS and global memory are told apart everywhere
    assert not [line for line in out.read_text().splitlines() if line.strip().startswith("flat_")]


def test_the_build_refuses_accumulators_that_the_compiler_uses(hipcc, tmp_path):
    source, obj = tmp_path / "named.hip", tmp_path / "named.o"
    source.write_text('#include <hip/hip_runtime.h>\n__global__ void k(float* p) { float c = *p; asm volatile("; %0" :: "a"(c)); }\n')
    with pytest.raises(accumulators.AccumulatorError):
        build.compile_source(str(source), str(obj), named_accumulators=True)
    assert not obj.exists()
    assert "ffn.hip" in build.NAMED_ACCUMULATORS  # the only source with such statements
    for name in build.SOURCES:
        with open(os.path.join(build.CSRC, name)) as f:
            assert ("a[%0" in f.read()) == (name in build.NAMED_ACCUMULATORS), name


@pytest.mark.parametrize("rest,reason", [
    ("\tv_accvgpr_write_b32 a9, v1\n" + MATRIX, "the compiler uses"),                       # a spill or copy of its own
    ("\tbuffer_store_dword a200, v1, s[0:3], 0 offen\n", "the compiler uses"),
    ("\tv_mov_b32_e32 v9, 0\n" + MATRIX, "too close ahead"),                                # no wait state
    ("\tv_mov_b32_e32 v9, 0\n\ts_nop 0\n" + MATRIX, "too close ahead"),                     # one of two
    ("\tv_permlane16_swap_b32_e32 v3, v15\n" + MATRIX, "too close ahead"),                  # its second operand is written too
    (".LBB0_1:\n" + MATRIX + "\tv_add_u32_e32 v12, 1, v12\n\ts_cbranch_scc1 .LBB0_1\n", "too close ahead"),  # around a loop
    ("\tv_mov_b32_e32 v12, 0\n\ts_branch .LBB0_2\n\ts_nop 7\n.LBB0_2:\n" + MATRIX, "too close ahead"),         # over a jump
    (MATRIX + "\t;;#ASMSTART\n\tv_accvgpr_read_b32 v0, a5\n\t;;#ASMEND\n", "too close behind"),
    (MATRIX + "\ts_nop 15\n\ts_nop 1\n\t;;#ASMSTART\n\tv_accvgpr_write_b32 a4, 0\n\t;;#ASMEND\n", "too close behind"),
    (".LBB0_1:\n\t;;#ASMSTART\n\tv_accvgpr_read_b32 v0, a5\n\t;;#ASMEND\n\ts_nop 7\n" + MATRIX + "\ts_cbranch_scc1 .LBB0_1\n",
     "too close behind"),
])
def test_planted_mistakes_are_found(rest, reason):
    with pytest.raises(accumulators.AccumulatorError, match=reason):
        accumulators.check(HEAD + rest + "\ts_endpgm\n")


@pytest.mark.parametrize("rest", [
    MATRIX + MATRIX,
    "\tv_mov_b32_e32 v9, 0\n\ts_nop 1\n" + MATRIX,
    "\tv_mov_b32_e32 v7, 0\n" + MATRIX,
    "\tv_mov_b32_e32 v9, 0\n\ts_branch .LBB0_2\n" + MATRIX + ".LBB0_2:\n\ts_nop 0\n" + MATRIX,
    MATRIX + "\ts_nop 15\n\ts_nop 2\n\t;;#ASMSTART\n\tv_accvgpr_read_b32 v0, a5\n\t;;#ASMEND\n",
    MATRIX + "\t;;#ASMSTART\n\tv_accvgpr_read_b32 v0, a8\n\t;;#ASMEND\n",
])
def test_what_keeps_to_the_rules_passes(rest):
    assert accumulators.check(HEAD + rest + "\ts_endpgm\n") == rest.count("v_mfma")
