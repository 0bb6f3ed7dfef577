"""Low-bit launches as 64 x 80 tiles, where the rule takes them by itself: rows and channels that fill no tile, more than four row
groups, up to 64 rows, one group, groups that the waves share unevenly, a batch whose layers meet inside a tile; and the
one-deep tiles, whose loop fetches ahead, over numbers of groups around the waves' turns."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import rosaq_oracle as O
from paper_2506_13472_amd import binding as B, synth, torch_glue as T
from test_gpu_parity import check_output, make_case, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,D,K,bits", [(256, 5120, 256, 128, 4), (250, 5111, 1152, 128, 3), (512, 5120, 1280, 128, 4), (310, 5105, 2304, 256, 3),
                                          (64, 20480, 256, 128, 4), (49, 20470, 384, 128, 3)])
def test_80_channel_tiles_by_the_rule(M, N, D, K, bits):
    print(f"case 64 x 80 M={M} N={N} D={D} K={K} bits={bits}", flush=True)
    assert B.rosaq_launch_shape(M, -(-N // 16) * 16, D, bits) == (4, 5, 8, 1, 1)
    assert not B.rosaq_launch_many_rows(M, -(-N // 16) * 16, D, K, bits, B.Q_NONE)[0]
    lam = synth.descending_spectrum(60, D)
    W, x = synth.make_weight(61, N, D), synth.make_activations(62, M, D)
    ref = O.pack(W, None, lam, K, bits, O.MODE_NONE)
    p = B.rosaq_pack_weights(W, None, lam, K, bits, B.Q_NONE)
    y = run_gpu(p, x)
    check_output(y, x, None, ref)
    assert np.array_equal(y.view(np.uint16), run_gpu(p, x).view(np.uint16))
    p.free()


def test_80_channel_tiles_of_a_batch():
    D, M, widths = 256, 256, (1700, 1690, 1700)           # 107 + 106 + 107 tiles: 64 of 80 channels, two across a border
    print("case 64 x 80 batch", flush=True)
    lam = synth.descending_spectrum(63, D)
    Ws = [synth.make_weight(64 + i, n, D) for i, n in enumerate(widths)]
    x16 = synth.make_activations(68, M, D)
    ps = [B.rosaq_pack_weights(W, None, lam, 128, 4, B.Q_NONE) for W in Ws]
    x = torch.from_numpy(x16).cuda()
    ws = torch.empty(B.rosaq_workspace_bytes_batch(ps, M), dtype=torch.uint8, device="cuda")
    ys = [torch.full((M, n), 3.0, dtype=torch.float16, device="cuda") for n in widths]
    B.rosaq_linear_batch(B.BatchArgs(ps, [y.data_ptr() for y in ys], list(widths)), x.data_ptr(), M, D, ws.data_ptr(), ws.numel(),
                         T.current_stream_ptr())
    for p, W, y in zip(ps, Ws, ys):
        check_output(y.cpu().numpy(), x16, None, O.pack(W, None, lam, 128, 4, O.MODE_NONE))
        p.free()


@pytest.mark.parametrize("bits", [4, 3])
@pytest.mark.parametrize("mt,nt", [(4, 3), (2, 2), (2, 6), (4, 1)])
def test_one_deep_tiles_over_turns_of_the_waves(mt, nt, bits):
    M, N = 61, 200
    for groups, K in ((1, 128), (7, 128), (8, 256), (9, 128), (16, 128), (17, 384), (25, 128)):
        print(f"case refill mt={mt} nt={nt} bits={bits} groups={groups}", flush=True)
        D = 128 * groups + K
        lam = synth.descending_spectrum(70, D)
        W, x = synth.make_weight(71, N, D), synth.make_activations(72, M, D)
        p = B.rosaq_pack_weights(W, None, lam, K, bits, B.Q_NONE)
        B.rosaq_tune("mt", mt); B.rosaq_tune("nt", nt); B.rosaq_tune("depth", 1)
        try:
            assert B.rosaq_launch_shape(M, -(-N // 16) * 16, D, bits)[:4] == (mt, nt, 8, 1)
            y = run_gpu(p, x)
        finally:
            B.rosaq_tune("mt", 0); B.rosaq_tune("nt", 0); B.rosaq_tune("depth", 0)
        check_output(y, x, None, O.pack(W, None, lam, K, bits, O.MODE_NONE))
        p.free()
