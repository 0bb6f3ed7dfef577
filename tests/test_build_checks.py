"""What the build checks in its own device assembly, on text with and without the fault."""
import glob
import os

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
