"""What the build checks in its own device assembly, on text with and without the fault."""
import glob
import os
import re

import pytest

from paper_2506_13472_amd import build as BU


def _loop(head, middle, tail, wait):
    piece = "\t;;#ASMSTART\n\ts_mov_b32 m0, s1\n\tglobal_load_lds_dwordx4 v1, s[2:3] offset:0\n\t;;#ASMEND\n"
    wait_for = "\t;;#ASMSTART\n\ts_waitcnt vmcnt({})\n\t;;#ASMEND\n".format
    load = "\tglobal_load_dwordx4 v[0:3], v4, s[2:3]\n\ts_waitcnt vmcnt(3)\n"
    return (wait_for(0) + load * head + wait_for(wait) + 4 * piece + load * middle + wait_for(wait) + 4 * piece +
            load * tail + wait_for(0))


def test_counted_waits_need_the_loads_they_count():
    assert BU.check_counted_waits(_loop(4, 4, 0, 12) + _loop(6, 8, 2, 20)) == 2
    assert BU.check_counted_waits(_loop(5, 4, 0, 12)) == 1           # more loads only wait longer
    for head, middle, tail, wait in ((3, 4, 0, 12), (4, 3, 0, 12), (6, 8, 1, 20)):
        with pytest.raises(RuntimeError):
            BU.check_counted_waits(_loop(head, middle, tail, wait))


def test_m0_belongs_to_the_hand_written_loads():
    text = _loop(4, 4, 0, 12)
    assert BU.check_counted_waits("\ts_nop 0 ; m0\n" + text) == 1
    for op in ("s_mov_b32 m0, s4", "v_movrels_b32_e32 v1, v2 m0"):
        with pytest.raises(RuntimeError):
            BU.check_counted_waits(text + "\t" + op + "\n")


def test_counted_waits_of_the_built_kernel():
    kept = glob.glob(os.path.join(BU.OBJ, "rosaq_wide-hip-amdgcn*.s"))
    if not kept:
        pytest.skip("no assembly kept from the build")
    with open(kept[0]) as f:
        assert BU.check_counted_waits(f.read()) == 3


_MFMA = "\tv_mfma_f32_16x16x32_f16 v[0:3], v[4:7], v[8:11], v[{}]\n".format


def _states(n):
    return f"\ts_nop {n - 1}\n" if n else ""


@pytest.mark.parametrize("touch,need", [("v_add_f32_e32 v20, v3, v21", 8), ("v_mov_b32_e32 v0, 0", 8), ("v_cvt_f16_f32_e32 v9, v1", 8),
                                        ("global_store_dwordx4 v30, v[0:3], s[0:1]", 8), ("ds_write_b64 v30, v[2:3]", 8),
                                        ("v_mfma_f32_16x16x32_f16 v[12:15], v[0:3], v[8:11], 0", 8),
                                        (";;#ASMSTART\n\tv_and_or_b32 v2, v20, s3, v21\n\t;;#ASMEND", 8),
                                        ("v_mov_b32_e32 v17, 0", 3), ("v_swap_b32 v20, v17", 3)])
def test_mfma_distance_in_straight_code(touch, need):
    end = "\n\ts_endpgm\n"
    assert BU.check_mfma_distance(_MFMA("16:19") + _states(need) + "\t" + touch + end) >= 1
    with pytest.raises(RuntimeError):
        BU.check_mfma_distance(_MFMA("16:19") + _states(need - 1) + "\t" + touch + end)


def test_mfma_distance_ignores_what_may_follow_at_once():
    for op in ("v_mov_b32_e32 v4, 0", "v_add_f32_e32 v20, v17, v21", "v_mfma_f32_16x16x32_f16 v[0:3], v[4:7], v[8:11], v[0:3]",
               "s_mov_b32 s2, s3", "v_add_f32_e32 v12, a0, a1"):
        assert BU.check_mfma_distance(_MFMA("16:19") + "\t" + op + "\n\ts_endpgm\n") >= 1


def test_mfma_distance_along_every_way():
    """The shorter of two ways to a join counts, and the way round a loop."""
    def join(states):
        return (_MFMA("0:3") + "\ts_cbranch_scc1 .LBB0_2\n" + _states(states) + ".LBB0_1:\n" + "\tv_add_f32_e32 v20, v0, v0\n\ts_endpgm\n"
                ".LBB0_2:\n\ts_nop 7\n\ts_nop 7\n\ts_branch .LBB0_1\n")
    assert BU.check_mfma_distance(join(7)) == 1                   # the branch itself is one
    with pytest.raises(RuntimeError):
        BU.check_mfma_distance(join(6))
    loop = ".LBB1_0:\n\tv_cvt_f16_f32_e32 v20, v0\n\ts_nop 7\n{}" + _MFMA("0:3") + "{}\ts_cbranch_scc0 .LBB1_0\n\ts_endpgm\n"
    assert BU.check_mfma_distance(loop.format("", _states(7))) == 1
    with pytest.raises(RuntimeError):
        BU.check_mfma_distance(loop.format(_states(8), _states(6)))


def test_mfma_distance_takes_no_way_or_instruction_on_trust():
    for text in (_MFMA("0:3") + "\ts_setpc_b64 s[30:31]\n", "\tv_mfma_f32_32x32x16_f16 v[0:15], v[16:19], v[20:23], v[0:15]\n\ts_endpgm\n"):
        with pytest.raises(RuntimeError):
            BU.check_mfma_distance(text)
    f64 = "\tv_mfma_f64_16x16x4_f64 a[0:7], v[4:5], v[8:9], a[0:7]\n{}\tv_accvgpr_read_b32 v1, a7\n\ts_endpgm\n"
    assert BU.check_mfma_distance(f64.format(_states(19))) == 1
    with pytest.raises(RuntimeError):
        BU.check_mfma_distance(f64.format(_states(18)))


@pytest.mark.parametrize("source,least", [("rosaq_kernels", 1000), ("rosaq_wide", 100), ("rosaq_rotate", 100), ("rosaq_pca", 10),
                                          ("rosaq_quant", 10)])
def test_mfma_distance_of_the_built_kernels(source, least):
    kept = glob.glob(os.path.join(BU.OBJ, source + "-hip-amdgcn*.s"))
    if not kept:
        pytest.skip("no assembly kept from the build")
    with open(kept[0], errors="replace") as f:
        assert BU.check_mfma_distance(f.read()) >= least


def _built(source):
    kept = glob.glob(os.path.join(BU.OBJ, source + "-hip-amdgcn*.s"))
    if not kept:
        pytest.skip("no assembly kept from the build")
    with open(kept[0], errors="replace") as f:
        return f.read()


def test_gemm_kernel_loads_no_argument_but_its_own():
    """The grid's size, for one, is an argument behind the kernel's own, and a wait of its own in front of the first unit."""
    text = _built("rosaq_kernels")
    kernels = re.findall(r"\.args:\n(.*?)\.symbol:\s+(_ZN5rosaq11gemm_kernel\S+)", text, re.S)
    assert len(kernels) > 100
    for args, name in kernels:
        args = args.rsplit("    .args:", 1)[-1]
        assert "by_value" in args and "hidden_" not in args, name


@pytest.mark.parametrize("rows,channels,depth", [(2, 2, 3), (2, 3, 2), (2, 4, 2), (4, 2, 2), (4, 3, 1), (4, 4, 1), (4, 5, 1)])
def test_all_fp16_units_are_fetched_without_waits(rows, channels, depth):
    """The shapes that the rule takes: nothing in front of the first product waits for all loads under way."""
    text = _built("rosaq_kernels")
    name = f"_ZN5rosaq11gemm_kernelILi16ELi{rows}ELi{channels}ELi8ELi{depth}EEEvNS_7GemmDevE:"
    start = text.index("\n" + name)
    head = text[start:text.index("v_mfma", start)]
    assert head.count("global_load_dwordx4") >= 4 * (rows + channels) * depth
    assert 0 not in [int(n) for n in re.findall(r"vmcnt\((\d+)\)", head)]
