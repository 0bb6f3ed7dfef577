"""Calibration at the edges of its block layout: fewer rows than a 64-row step, a row more and a row less than one, fewer
rows than channels (rank-deficient), a single problem of four blocks, a number of blocks that is no power of two."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2506_13472_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("D,n_cal", [(128, 1), (128, 63), (128, 65), (128, 300), (384, 64), (384, 129), (640, 700)])
def test_pca_block_edges(D, n_cal, full):
    print(f"case pca blocks D={D} n_cal={n_cal} full={full}", flush=True)
    rng = np.random.default_rng(1000 + D + n_cal)
    X = (rng.standard_normal((n_cal, D)) * np.exp(rng.standard_normal(D))).astype(np.float16)
    xd = torch.full((n_cal, D + 8), 3.0, dtype=torch.float16, device="cuda")     # a padded row stride
    xd[:, :D] = torch.from_numpy(X).cuda()
    if full:
        Q, lam = B.rosaq_pca_full(xd.data_ptr(), n_cal, D, xd.stride(0))
        Q, lam, width = Q[None], lam[None], D
    else:
        Q, lam = B.rosaq_pca_headwise(xd.data_ptr(), n_cal, D, xd.stride(0))
        lam, width = lam.reshape(-1, 128), 128
    for h in range(D // width):
        x = X[:, h * width:(h + 1) * width].astype(np.float64)
        C = x.T @ x / n_cal
        want = np.linalg.eigvalsh(C)[::-1]
        q = Q[h].astype(np.float64)
        assert np.all(np.diff(lam[h]) <= 0) and np.all(lam[h] >= 0)
        assert np.max(np.abs(lam[h] - want)) <= 1e-10 * want[0]
        # Q is fp32: 2^-24 relative per entry, summed over at most 640 entries of unit columns
        assert np.max(np.abs(q.T @ q - np.eye(width))) <= 2e-6
        assert np.all(q[np.argmax(np.abs(q), axis=0), np.arange(width)] > 0)
        assert np.linalg.norm(q @ np.diag(lam[h]) @ q.T - C) <= 1e-5 * np.linalg.norm(C)


def test_pca_of_more_rows_than_a_grid_dimension_holds():
    """4194305 rows: more than 65536 steps of 64 rows, the limit of a grid's second dimension."""
    n, D = 64 * 65536 + 1, 128
    print(f"case pca rows D={D} n_cal={n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(1001)
    X = torch.empty((n, D), dtype=torch.float16, device="cuda")
    C = torch.zeros((D, D), dtype=torch.float64, device="cuda")
    scale = torch.exp(torch.randn(D, generator=g, device="cuda"))
    for lo in range(0, n, 1 << 18):
        x = (torch.randn((min(n - lo, 1 << 18), D), generator=g, device="cuda") * scale).to(torch.float16)
        X[lo:lo + x.shape[0]] = x
        x = x.double()
        C += x.t().contiguous() @ x
    X[-1] *= 64                                    # the last row alone changes the result
    C += 4095 * torch.outer(X[-1].double(), X[-1].double()) / 4096
    C = (C / n).cpu().numpy()
    Q, lam = B.rosaq_pca_full(X.data_ptr(), n, D, D)
    want = np.linalg.eigvalsh(C)[::-1]
    assert np.max(np.abs(lam - want)) <= 1e-10 * want[0]
    q = Q.astype(np.float64)
    assert np.linalg.norm(q @ np.diag(lam) @ q.T - C) <= 1e-5 * np.linalg.norm(C)
