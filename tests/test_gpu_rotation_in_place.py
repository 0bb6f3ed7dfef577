"""The dense rotation around the row counts up to which it reads x in place: x with a padded stride that ends with its last row,
in front of a page of NaN, at the tile edges and on both sides of the rule."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import rosaq_oracle as O
from paper_2506_13472_amd import binding as B, synth, torch_glue as T
from test_gpu_parity import check_output

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,rows", [(128, (17, 33, 64, 65)), (2048, (17, 48, 49, 64, 65)), (2176, (32, 47, 48, 49)), (2560, (48, 49)), (2688, (31, 32, 33, 48)), (4096, (32, 33)), (4224, (16, 17, 64))])
def test_dense_rotation_of_few_rows(D, rows):
    rng = np.random.default_rng(D)
    Q, lam = synth.random_orthogonal_dense(76, D), synth.descending_spectrum(77, D)
    N = 100
    W = synth.make_weight(75, N, D)
    ref = O.pack(W, Q, lam, 128, 4, O.MODE_FULL)
    p = B.rosaq_pack_weights(W, Q, lam, 128, 4, B.Q_FULL)
    for M in rows:
        print(f"case rotation in place D={D} M={M}", flush=True)
        x16 = (rng.standard_normal((M, D)) * np.exp(rng.standard_normal(D))).astype(np.float16)
        stride = D + 24
        buf = torch.full((M * stride + 4096,), float("nan"), dtype=torch.float16, device="cuda")
        x = torch.as_strided(buf, (M, D), (stride, 1))
        x.copy_(torch.from_numpy(x16))
        ws = T.alloc_workspace(p, M)
        ws.fill_(255)
        y = torch.empty((M, N), dtype=torch.float16, device="cuda")
        check_output(T.linear(p, x, y, ws).cpu().numpy(), x16, Q, ref)
    p.free()
