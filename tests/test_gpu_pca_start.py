"""Calibration sets on which the search for a starting rotation in fp32 ends differently: full rank with channels mixed or not,
eigenvalues that are equal or nearly so, ranks that are missing, channels that are zero, and a NaN."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2506_13472_amd import binding as B

pytestmark = pytest.mark.gpu


def _set(kind, n, D, rng):
    X = rng.standard_normal((n, D)) * np.exp(rng.standard_normal(D))
    if kind == "mixed":
        X = X @ np.linalg.qr(rng.standard_normal((D, D)))[0]
    elif kind == "equal":                               # one channel, copied
        X = np.repeat(X[:, :1], D, axis=1)
    elif kind == "close":                               # unit channels: eigenvalues in a narrow band
        X = np.sign(X)
    elif kind == "rank":
        X = X @ rng.standard_normal((D, D // 2)) @ rng.standard_normal((D // 2, D)) / D
    elif kind == "zeros":
        X[:, ::3] = 0.0
    elif kind == "wide":                                # channels from 6e-5 to 6e4
        X = rng.standard_normal((n, D)) * np.logspace(-4, 4, D)
    return X.astype(np.float16)


@pytest.mark.parametrize("kind", ["plain", "mixed", "equal", "close", "rank", "zeros", "wide"])
@pytest.mark.parametrize("D,n,full", [(256, 300, False), (256, 257, True), (384, 900, True)])
def test_pca_of_sets_that_start_differently(kind, D, n, full):
    print(f"case pca start {kind} D={D} n_cal={n} full={full}", flush=True)
    X = _set(kind, n, D, np.random.default_rng(77 + D + n))
    xd = torch.from_numpy(X).cuda()
    Q, lam = (B.rosaq_pca_full if full else B.rosaq_pca_headwise)(xd.data_ptr(), n, D, D)
    width = D if full else 128
    Q, lam = np.asarray(Q).reshape(-1, width, width).astype(np.float64), np.asarray(lam).reshape(-1, width)
    for h in range(D // width):
        x = X[:, h * width:(h + 1) * width].astype(np.float64)
        want = np.linalg.svd(x, compute_uv=False) ** 2 / n
        # LAPACK's singular values and these are good to width * 2^-53 of the largest each
        assert np.max(np.abs(lam[h] - want)) <= 4 * width * 2.0 ** -53 * want[0]
        q = Q[h]
        assert np.max(np.abs(q.T @ q - np.eye(width))) <= 2e-6           # the rounding of Q to fp32
        y = x @ q                                                        # columns orthogonal up to that rounding
        c = y.T @ y / n
        assert np.max(np.abs(c - np.diag(np.diag(c)))) <= 2.0 ** -24 * 8 * want[0]
        if kind in ("plain", "mixed", "close"):                          # full rank: relative accuracy of every eigenvalue
            cond = np.sqrt(want[0] / want[-1])
            assert np.max(np.abs(lam[h] / want - 1)) <= 4 * width * 2.0 ** -53 * cond


def test_pca_refuses_a_set_that_is_not_a_number():
    print("case pca nan", flush=True)
    x = torch.randn((200, 256), device="cuda", dtype=torch.float16)
    x[17, 200] = float("nan")
    for call in (B.rosaq_pca_full, B.rosaq_pca_headwise):
        with pytest.raises(Exception):
            call(x.data_ptr(), 200, 256, 256)
