"""Rows and row tiles past M are not written into the workspace's activations: whatever stands there, NaN patterns
included, must not reach an output."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import rosaq_oracle as O
from paper_2506_13472_amd import binding as B
from paper_2506_13472_amd import torch_glue as T
from test_gpu_parity import check_output, make_case
from test_gpu_swiglu import synth_down

pytestmark = pytest.mark.gpu

ROWS = (1, 4, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 100)


@pytest.mark.parametrize("mode,D,K,bits", [(O.MODE_NONE, 384, 128, 4), (O.MODE_HEADWISE, 640, 128, 3), (O.MODE_FULL, 512, 128, 4),
                                           (O.MODE_NONE, 256, 256, 4)])
def test_linear_on_a_workspace_of_nan(mode, D, K, bits):
    print(f"case dirty workspace mode={mode} D={D} K={K}", flush=True)
    N = 200
    lay, Q, lam = make_case(830, max(ROWS), D, N, 300, mode)
    ref = O.pack(lay["W"], Q, lam, K, bits, mode)
    p = B.rosaq_pack_weights(lay["W"], Q, lam, K, bits, mode)
    try:
        for M in ROWS:
            x16 = lay["x"][:M].copy()
            x = torch.from_numpy(x16).cuda()
            for splits, rot_splits, wide in ((0, 0, 0), (2, 2, 0), (0, 0, 2)):
                if (wide and M <= 64) or (splits and M > 64):
                    continue
                for k, v in (("splits", splits), ("rot_splits", rot_splits), ("wide", wide)):
                    B.rosaq_tune(k, v)
                ys = []
                for fill in (255, 0):
                    ws = T.alloc_workspace(p, M)
                    ws.fill_(fill)
                    y = torch.full((M, N), 3.0, dtype=torch.float16, device="cuda")
                    ys.append(T.linear(p, x, y, ws).cpu().numpy())
                assert np.array_equal(ys[0].view(np.uint16), ys[1].view(np.uint16)), (M, splits, wide)
                check_output(ys[0], x16, Q, ref)
    finally:
        for k in ("splits", "rot_splits", "wide"):
            B.rosaq_tune(k, 0)
        p.free()


@pytest.mark.parametrize("mode", [O.MODE_NONE, O.MODE_HEADWISE, O.MODE_FULL])
def test_mlp_block_on_a_workspace_of_nan(mode):
    """The gated product's rows past M in the down projection's input too, and its tickets."""
    print(f"case dirty workspace, MLP block mode={mode}", flush=True)
    D, F, N = 256, 640, 130
    lay, Q, lam = make_case(831, max(ROWS), D, F, 300, mode)
    Wu = (lay["W"][::-1] * np.float16(1.5)).astype(np.float16)
    pg, pu = (B.rosaq_pack_weights(W, Q, lam, 128, 4, mode) for W in (lay["W"], Wu))
    pd = B.rosaq_pack_weights(synth_down(832, N, F), None, np.arange(F, 0, -1.0), 128, 4, B.Q_NONE)
    try:
        for M in ROWS:
            x = torch.from_numpy(lay["x"][:M].copy()).cuda()
            for splits in (0, 3):
                B.rosaq_tune("splits", splits)
                ys = []
                for fill in (255, 0):
                    ws = torch.full((B.rosaq_workspace_bytes_mlp(pg, pu, pd, M),), fill, dtype=torch.uint8, device="cuda")
                    y = torch.full((M, N), 3.0, dtype=torch.float16, device="cuda")
                    B.rosaq_mlp_swiglu(pg, pu, pd, x.data_ptr(), M, x.stride(0), y.data_ptr(), y.stride(0), ws.data_ptr(),
                                       ws.numel(), T.current_stream_ptr())
                    ys.append(y.cpu().numpy())
                assert np.all(np.isfinite(ys[0])) and np.any(ys[0] != 3.0)
                assert np.array_equal(ys[0].view(np.uint16), ys[1].view(np.uint16)), (M, splits)
    finally:
        B.rosaq_tune("splits", 0)
        for p in (pg, pu, pd):
            p.free()


@pytest.mark.parametrize("rot_mt", [0, 2, 4])
def test_rotation_in_place_with_more_rows_a_workgroup_than_the_call_has(rot_mt):
    """x is read in place up to 16 rows: rows past M of the workgroup's tiles stay inside x, which ends with its last row."""
    print(f"case rotation in place rot_mt={rot_mt}", flush=True)
    D, N = 512, 130
    lay, Q, lam = make_case(833, 16, D, N, 300, O.MODE_FULL)
    ref = O.pack(lay["W"], Q, lam, 128, 4, O.MODE_FULL)
    p = B.rosaq_pack_weights(lay["W"], Q, lam, 128, 4, B.Q_FULL)
    try:
        B.rosaq_tune("rot_mt", rot_mt)
        for M, pad in ((1, 0), (3, 8), (15, 0), (16, 264)):
            x = torch.full((M, D + pad), float("nan"), dtype=torch.float16, device="cuda")[:, :D]
            x.copy_(torch.from_numpy(lay["x"][:M]))
            ws = T.alloc_workspace(p, M)
            ws.fill_(255)
            check_output(T.linear(p, x, None, ws).cpu().numpy(), lay["x"][:M], Q, ref)
    finally:
        B.rosaq_tune("rot_mt", 0)
        p.free()
