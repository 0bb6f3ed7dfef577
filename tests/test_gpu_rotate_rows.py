"""The head-wise rotation of many rows (tiles turned in LDS, stored as 16-byte pieces), forced with the tuning key "wide": the
product equals that of rotate_headwise_kernel's activations bit for bit, at row counts around the 64-row blocks and
with selections that leave all, some or few neighbouring storage positions to one head."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import rosaq_oracle as O
from paper_2506_13472_amd import binding as B
from paper_2506_13472_amd import torch_glue as T
from test_gpu_parity import check_output, make_case, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rule", [B.SELECT_TOP, B.SELECT_TOP_PER_HEAD])
@pytest.mark.parametrize("M,D,K", [(65, 128, 0), (65, 128, 128), (127, 256, 128), (128, 1024, 128), (129, 640, 640),
                                   (449, 512, 256)])
def test_rotate_rows(M, D, K, rule):
    print(f"case rotate rows M={M} D={D} K={K} rule={rule}", flush=True)
    lay, Q, lam = make_case(700 + M, M, D, 80, 300, O.MODE_HEADWISE)
    p = B.rosaq_pack_weights(lay["W"], Q, lam, K, 4, B.Q_HEADWISE, select_rule=rule)
    x = torch.from_numpy(lay["x"]).cuda()
    y = torch.empty((M, 80), dtype=torch.float16, device="cuda")
    ws = T.alloc_workspace(p, M)
    ws.fill_(255)
    try:
        for stage, wide in ((1, 2), (2, 1)):          # the rotation alone, then the main GEMM on what it left
            B.rosaq_tune("stages", stage)
            B.rosaq_tune("wide", wide)
            T.linear(p, x, y, ws)
        B.rosaq_tune("stages", 3)
        want = run_gpu(p, lay["x"])
    finally:
        B.rosaq_tune("stages", 3)
        B.rosaq_tune("wide", 0)
    got = y.cpu().numpy()
    assert np.array_equal(got.view(np.uint16), want.view(np.uint16))
    if rule == B.SELECT_TOP:
        check_output(got, lay["x"], Q, O.pack(lay["W"], Q, lam, K, 4, O.MODE_HEADWISE))
    p.free()


def test_rotate_rows_is_the_default_where_it_fills_the_chip():
    """10 heads x 17 blocks: the rule takes the kernel for many rows by itself (and at 10 x 16 does not); against
    rotate_headwise_kernel, with a padded row stride."""
    print("case rotate rows default", flush=True)
    assert [B.rosaq_launch_many_rows(M, 48, 1280, 128, 3, B.Q_HEADWISE)[1] for M in (1024, 1030)] == [False, True]
    lay, Q, lam = make_case(710, 64, 1280, 48, 300, O.MODE_HEADWISE)
    p = B.rosaq_pack_weights(lay["W"], Q, lam, 128, 3, B.Q_HEADWISE)
    x = torch.full((1030, 1288), 7.0, dtype=torch.float16, device="cuda")[:, :1280]
    x.copy_(torch.from_numpy(np.tile(lay["x"], (17, 1))[:1030]))
    got = T.linear(p, x)
    try:
        B.rosaq_tune("wide", 1)
        want = T.linear(p, x)
    finally:
        B.rosaq_tune("wide", 0)
    assert torch.equal(got.view(torch.int16), want.view(torch.int16))
    p.free()
