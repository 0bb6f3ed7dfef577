"""Tiles whose conversion runs close behind their MFMAs: what they give is the oracle's, and the same in every call."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import rosaq_oracle as O
from paper_2506_13472_amd import binding as B
from paper_2506_13472_amd import torch_glue as T
from test_gpu_parity import check_output, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits,M,tune", [(3, 64, dict(mt=4, nt=3)), (3, 64, dict(mt=2, nt=3)), (4, 64, dict(mt=4, nt=3)),
                                         (3, 130, dict(wide=2)), (4, 130, dict(wide=2))])
def test_repeated_calls_are_bit_identical(bits, M, tune):
    print(f"case repeat bits={bits} M={M} {tune}", flush=True)
    D, N = 2048, 3000
    lay, _, lam = make_case(901, M, D, N, 300, O.MODE_NONE)
    ref = O.pack(lay["W"], None, lam, 256, bits, O.MODE_NONE)
    p = B.rosaq_pack_weights(lay["W"], None, lam, 256, bits, B.Q_NONE)
    x = torch.from_numpy(lay["x"]).cuda()
    ws = T.alloc_workspace(p, M)
    try:
        for k, v in tune.items():
            B.rosaq_tune(k, v)
        ys = [T.linear(p, x, torch.empty((M, N), dtype=torch.float16, device="cuda"), ws) for _ in range(20)]
        torch.cuda.synchronize()
    finally:
        for k in tune:
            B.rosaq_tune(k, 0)
    ys = [y.cpu().numpy() for y in ys]
    check_output(ys[0], lay["x"], None, ref)
    for y in ys[1:]:
        assert np.array_equal(y.view(np.uint16), ys[0].view(np.uint16))
    p.free()
