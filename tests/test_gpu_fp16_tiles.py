"""All-fp16 launches as 64 x 80 tiles (the dense rotation of a few hundred rows, and layers of K = D): at widths that five
channel tiles divide and do not, at row counts around the 64-row blocks, and where the rule takes them by itself; and
gated pairs of such layers where an odd number of tiles per workgroup would be the plain launch's choice."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import rosaq_oracle as O
from paper_2506_13472_amd import binding as B, synth
from test_gpu_parity import check_output, make_case, run_gpu
from test_gpu_swiglu import check_swiglu, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,D", [(33, 640), (64, 384), (65, 640), (130, 384), (49, 128)])
def test_dense_rotation_as_80_channel_tiles(M, D):
    print(f"case rotation 64 x 80 M={M} D={D}", flush=True)
    lay, Q, lam = make_case(71, M, D, 100, 300, O.MODE_FULL)
    ref = O.pack(lay["W"], Q, lam, 128, 4, O.MODE_FULL)
    p = B.rosaq_pack_weights(lay["W"], Q, lam, 128, 4, B.Q_FULL)
    B.rosaq_tune("rot_mt", 4); B.rosaq_tune("rot_nt", 5); B.rosaq_tune("wide", 1)
    try:
        y = run_gpu(p, lay["x"])
        again = run_gpu(p, lay["x"])
    finally:
        B.rosaq_tune("rot_mt", 0); B.rosaq_tune("rot_nt", 0); B.rosaq_tune("wide", 0)
    check_output(y, lay["x"], Q, ref)
    assert np.array_equal(y.view(np.uint16), again.view(np.uint16))
    p.free()


@pytest.mark.parametrize("M,N", [(256, 5120), (250, 5111), (129, 6400), (512, 2560)])
def test_all_fp16_layer_in_one_round_of_80_channel_tiles(M, N):
    print(f"case K = D, 64 x 80 by the rule M={M} N={N}", flush=True)
    assert B.rosaq_launch_shape(M, -(-N // 16) * 16, 256, 16)[:2] == (4, 5)
    lay, _, lam = make_case(72, M, 256, N, 300, O.MODE_NONE)
    ref = O.pack(lay["W"], None, lam, 256, 4, O.MODE_NONE)
    p = B.rosaq_pack_weights(lay["W"], None, lam, 256, 4, B.Q_NONE)
    B.rosaq_tune("wide", 1)                    # not the kernel for many rows
    try:
        check_output(run_gpu(p, lay["x"]), lay["x"], None, ref)
    finally:
        B.rosaq_tune("wide", 0)
    p.free()


@pytest.mark.parametrize("M", [64, 40, 256])
def test_gated_pair_of_all_fp16_layers(M):
    """2 x 320 channel tiles: the plain launch would take 48 (up to 64 rows) or 80 channels, odd numbers of tiles."""
    print(f"case gated K = D M={M}", flush=True)
    D, N = 128, 5120
    lay, _, lam = make_case(73, M, D, N, 200, O.MODE_NONE)
    W2 = synth.make_weight(74, N, D)
    refs = [O.pack(W, None, lam, D, 4, O.MODE_NONE) for W in (lay["W"], W2)]
    gate, up = [B.rosaq_pack_weights(W, None, lam, D, 4, B.Q_NONE) for W in (lay["W"], W2)]
    B.rosaq_tune("wide", 1)
    try:
        check_swiglu(run(gate, up, lay["x"]), lay["x"], None, refs[0], refs[1])
    finally:
        B.rosaq_tune("wide", 0)
        gate.free(); up.free()
