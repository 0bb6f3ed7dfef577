"""Split launches on workspaces that hold anything: whatever runs in front of one clears its tickets, all of them."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import rosaq_oracle as O
from paper_2506_13472_amd import binding as B
from paper_2506_13472_amd import torch_glue as T
from test_gpu_parity import check_output, make_case

pytestmark = pytest.mark.gpu

DIRTY = 0x01          # as 32-bit words no number of tickets a tile can reach: a tile whose ticket was not cleared is not stored


def _reset():
    for k in ("mt", "nt", "wpb", "depth", "splits", "rot_splits"):
        B.rosaq_tune(k, 0)


def _split_on_dirty_workspace(mode, M, D, N, nt, splits, rot_splits=0):
    lay, Q, lam = make_case(810, M, D, N, 300, mode)
    ref = O.pack(lay["W"], Q, lam, 128, 4, mode)
    p = B.rosaq_pack_weights(lay["W"], Q, lam, 128, 4, mode)
    try:
        for k, v in (("nt", nt), ("splits", splits), ("rot_splits", rot_splits)):
            B.rosaq_tune(k, v)
        assert B.rosaq_launch_shape(M, -(-N // 16) * 16, D, 4)[4] == splits
        ws = T.alloc_workspace(p, M)
        ws.fill_(DIRTY)
        y = torch.full((M, N), 3.0, dtype=torch.float16, device="cuda")
        T.linear(p, torch.from_numpy(lay["x"]).cuda(), y, ws)
        torch.cuda.synchronize()
        check_output(y.cpu().numpy(), lay["x"], Q, ref)
    finally:
        _reset()
        p.free()


@pytest.mark.parametrize("M,D,N,nt", [(33, 256, 232, 4), (48, 512, 232, 2), (40, 640, 100, 4), (33, 896, 5200, 1),
                                      (7, 1152, 1100, 1), (16, 1408, 1100, 1), (20, 1280, 1600, 1), (64, 384, 300, 1)])
def test_headwise_rotation_clears_every_ticket(M, D, N, nt):
    """Heads that do not fill the eight XCDs: the launch has workgroups without a head."""
    print(f"case tickets head-wise M={M} D={D} N={N} nt={nt}", flush=True)
    _split_on_dirty_workspace(O.MODE_HEADWISE, M, D, N, nt, 2)


@pytest.mark.parametrize("mode,M,rot_splits", [(O.MODE_NONE, 5, 0), (O.MODE_NONE, 48, 0), (O.MODE_FULL, 16, 0), (O.MODE_FULL, 33, 0),
                                               (O.MODE_FULL, 33, 2)])
def test_other_prologues_clear_every_ticket(mode, M, rot_splits):
    print(f"case tickets mode={mode} M={M} rot_splits={rot_splits}", flush=True)
    _split_on_dirty_workspace(mode, M, 256, 5200, 1, 2, rot_splits)


@pytest.mark.parametrize("mode,first", [(O.MODE_HEADWISE, 3), (O.MODE_NONE, 1), (O.MODE_FULL, 3)])
def test_main_gemm_alone_splits_on_what_an_unsplit_call_left(mode, first):
    """Tuning key "stages" = 2 takes the activations from the workspace, and nothing else."""
    print(f"case tickets stages=2 mode={mode} first={first}", flush=True)
    M, D, N = 40, 512, 200
    lay, Q, lam = make_case(811, M, D, N, 300, mode)
    ref = O.pack(lay["W"], Q, lam, 128, 4, mode)
    p = B.rosaq_pack_weights(lay["W"], Q, lam, 128, 4, mode)
    x = torch.from_numpy(lay["x"]).cuda()
    y = torch.full((M, N), 3.0, dtype=torch.float16, device="cuda")
    ws = T.alloc_workspace(p, M)
    ws.fill_(DIRTY)
    try:
        B.rosaq_tune("stages", first)
        B.rosaq_tune("splits", 1)
        T.linear(p, x, y, ws)
        y.fill_(3.0)
        B.rosaq_tune("stages", 2)
        B.rosaq_tune("splits", 3)
        for _ in range(2):
            T.linear(p, x, y, ws)
        torch.cuda.synchronize()
    finally:
        B.rosaq_tune("stages", 3)
        _reset()
    check_output(y.cpu().numpy(), lay["x"], Q, ref)
    p.free()
