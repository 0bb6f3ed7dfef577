"""Small head-wise layers whose rotation runs inside the GEMM's launch: the same bits as two launches give, over heads, rows,
salient channels (more fp16 k-steps than waves among them), output tiles and their remainders, layers of a batch; outputs
that lie in x; and captured calls.  One launch leaves the workspace as it was, two do not: that tells which ran."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import rosaq_oracle as O
from paper_2506_13472_amd import binding as B, synth, torch_glue as T
from test_gpu_parity import check_output

pytestmark = pytest.mark.gpu


def _layer(D, N, K, bits, seed):
    Q, lam = synth.random_orthogonal_blocks(seed, D // 128), synth.descending_spectrum(seed + 1, D, D // 128)
    W = synth.make_weight(seed + 2, N, D)
    return Q, O.pack(W, Q, lam, K, bits, O.MODE_HEADWISE), B.rosaq_pack_weights(W, Q, lam, K, bits, B.Q_HEADWISE)


def _untouched(ws):
    return bool(torch.all(ws == 255))


def _two_launches(call):
    B.rosaq_tune("wide", 1)                      # at up to 64 rows: nothing but the separate rotation
    try:
        return call()
    finally:
        B.rosaq_tune("wide", 0)


@pytest.mark.parametrize("D,N,K,bits,fused", [(256, 16, 128, 4, True), (256, 4096, 128, 3, True), (512, 1003, 384, 4, True), (640, 200, 128, 3, True),
                                              (768, 4096, 128, 3, True), (896, 1024, 256, 4, True), (1024, 1024, 128, 4, True), (1024, 999, 896, 3, True),
                                              (256, 4097, 128, 4, False), (896, 1025, 128, 4, False), (1024, 1040, 128, 4, False), (1152, 64, 128, 4, False)])
def test_fused_rotation_gives_the_same_bits(D, N, K, bits, fused):
    Q, ref, p = _layer(D, N, K, bits, 80)
    for M in (1, 2, 15, 16):
        print(f"case fused rotation D={D} N={N} K={K} bits={bits} M={M}", flush=True)
        x16 = synth.make_activations(81 + M, M, D)
        stride = D + 8
        buf = torch.full((M * stride + 64,), float("nan"), dtype=torch.float16, device="cuda")
        x = torch.as_strided(buf, (M, D), (stride, 1))
        x.copy_(torch.from_numpy(x16))
        ws = T.alloc_workspace(p, M)

        def call():
            ws.fill_(255)
            y = torch.full((M + 1, N), 3.0, dtype=torch.float16, device="cuda")
            T.linear(p, x, y[:M], ws)
            assert torch.all(y[M] == 3.0)
            return y[:M].cpu().numpy()
        one = call()
        assert _untouched(ws) == fused
        check_output(one, x16, Q, ref)
        assert np.array_equal(one.view(np.uint16), _two_launches(call).view(np.uint16))
        assert not _untouched(ws)
    p.free()


def test_outputs_that_lie_in_x():
    D, M = 256, 16
    print("case fused rotation in place", flush=True)
    Q, ref, p = _layer(D, D, 128, 4, 90)
    x16 = synth.make_activations(91, M, D)
    ws = T.alloc_workspace(p, M)
    for shift in (0, 1):                          # y = x, and y one row further
        buf = torch.empty((M + 1, D), dtype=torch.float16, device="cuda")
        buf[:M] = torch.from_numpy(x16)
        y = buf[shift:shift + M]
        ws.fill_(255)
        T.linear(p, buf[:M], y, ws)
        assert not _untouched(ws)
        check_output(y.cpu().numpy(), x16, Q, ref)
    p.free()


@pytest.mark.parametrize("D", [512, 1024])               # captured, the larger one takes two launches
def test_fused_rotation_of_a_batch_and_under_capture(D):
    M = 5
    print(f"case fused rotation batch, capture D={D}", flush=True)
    Q, lam = synth.random_orthogonal_blocks(95, D // 128), synth.descending_spectrum(96, D, D // 128)
    ps = [B.rosaq_pack_weights(synth.make_weight(97 + i, n, D), Q, lam, 128, 4, B.Q_HEADWISE) for i, n in enumerate((100, 512, 33))]
    x = torch.from_numpy(synth.make_activations(99, M, D)).cuda()
    ws = torch.empty(B.rosaq_workspace_bytes_batch(ps, M), dtype=torch.uint8, device="cuda")
    ys = [torch.zeros((M, p.N), dtype=torch.float16, device="cuda") for p in ps]
    args = B.BatchArgs(ps, [y.data_ptr() for y in ys], [y.stride(0) for y in ys])

    ws.fill_(255)

    def call():
        B.rosaq_linear_batch(args, x.data_ptr(), M, x.stride(0), ws.data_ptr(), ws.numel(), T.current_stream_ptr())

    def result():
        torch.cuda.synchronize()
        out = [y.clone() for y in ys]
        for y in ys:
            y.zero_()
        return out
    call()
    one = result()
    assert _untouched(ws)
    _two_launches(call)
    assert all(torch.equal(a, b) for a, b in zip(one, result()))
    assert not _untouched(ws)
    ws.fill_(255)
    torch.cuda.synchronize()
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        call()
    for _ in range(3):
        graph.replay()
        assert all(torch.equal(a, b) for a, b in zip(one, result()))
        assert _untouched(ws) == (D == 512)
    for p in ps:
        p.free()
