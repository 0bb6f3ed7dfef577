"""Calibration sets on which the search for a starting rotation in fp32 ends differently: full rank with channels mixed or not,
eigenvalues that are equal or nearly so, ranks that are missing, fewer rows than channels, channels that are zero or short; and sets that are refused: NaN and infinities."""
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
    elif kind == "repeated":                            # a few rows, again and again: rank n / 8
        X = X[np.arange(n) % (n // 8)]
    elif kind == "few long":                            # rank 8 and what rounding to fp16 adds
        X = X[:, :8] @ rng.standard_normal((8, D))
    elif kind == "one long":                            # short columns of full rank, not along the channels, beside a long one
        X = X @ np.linalg.qr(rng.standard_normal((D, D)))[0] * 2e-5
        X[:, 5] = 100.0 * rng.standard_normal(n)
    elif kind == "wide":                                # channels from 6e-5 to 6e4
        X = rng.standard_normal((n, D)) * np.logspace(-4, 4, D)
    return X.astype(np.float16)


@pytest.mark.parametrize("kind", ["plain", "mixed", "equal", "close", "rank", "zeros", "wide", "repeated", "few long", "one long"])
@pytest.mark.parametrize("D,n,full", [(256, 300, False), (256, 257, True), (384, 900, True), (256, 50, False), (384, 100, True), (512, 500, True)])
def test_pca_of_sets_that_start_differently(kind, D, n, full):
    print(f"case pca start {kind} D={D} n_cal={n} full={full}", flush=True)
    _check(kind, D, n, full)


@pytest.mark.parametrize("kind", ["plain", "mixed", "rank", "one long"])
@pytest.mark.parametrize("D,n,full", [(256, 300, False), (384, 900, True), (384, 100, True)])
def test_pca_by_sweeps_alone(kind, D, n, full):
    print(f"case pca sweeps alone {kind} D={D} n_cal={n} full={full}", flush=True)
    B.rosaq_tune("pca_sweeps", 1)                       # as without memory for the search
    try:
        # up to 20 sweeps pass every column through width / 32 - 1 products of 64 terms, each good to 8 (the root of 64) 2^-53
        # of the column's length, and an eigenvalue is its square
        _check(kind, D, n, full, 2 * 20 * ((D if full else 128) // 32 - 1) * 8 * 2.0 ** -53)
    finally:
        B.rosaq_tune("pca_sweeps", 0)


def _check(kind, D, n, full, good_to=None):
    X = _set(kind, n, D, np.random.default_rng(77 + D + n))
    xd = torch.from_numpy(X).cuda()
    Q, lam = (B.rosaq_pca_full if full else B.rosaq_pca_headwise)(xd.data_ptr(), n, D, D)
    width = D if full else 128
    good_to = good_to or 4 * width * 2.0 ** -53      # LAPACK's singular values and these are good to width * 2^-53 of the largest each
    Q, lam = np.asarray(Q).reshape(-1, width, width).astype(np.float64), np.asarray(lam).reshape(-1, width)
    for h in range(D // width):
        x = X[:, h * width:(h + 1) * width].astype(np.float64)
        want = np.zeros(width)
        want[:min(n, width)] = np.linalg.svd(x, compute_uv=False) ** 2 / n
        assert np.max(np.abs(lam[h] - want)) <= good_to * want[0]
        q = Q[h]
        assert np.max(np.abs(q.T @ q - np.eye(width))) <= 2e-6           # the rounding of Q to fp32
        y = x @ q                                                        # columns orthogonal up to that rounding
        c = y.T @ y / n
        assert np.max(np.abs(c - np.diag(np.diag(c)))) <= 2.0 ** -24 * 8 * want[0]
        if n >= width and kind in ("plain", "mixed", "close"):                          # full rank: relative accuracy of every eigenvalue
            cond = np.sqrt(want[0] / want[-1])
            assert np.max(np.abs(lam[h] / want - 1)) <= good_to * cond


def _spoil(x, kind):
    """What keeps a set from being numbers; where every inner product of a problem is lost, no angle is left to find that."""
    nan, inf = float("nan"), float("inf")
    if kind == "element":
        x[17, 200] = nan
    elif kind == "row":
        x[17] = nan
    elif kind == "head":                       # the channels of one head, in every row
        x[:, 128:] = nan
    elif kind == "all":
        x[:] = nan
    elif kind == "channel among zeros":
        x[:] = 0.0
        x[:, 200] = nan
    elif kind == "infinity":
        x[17, 200] = inf
    elif kind == "infinity among zeros":
        x[:] = 0.0
        x[17, 200] = -inf
    else:                                      # a row of infinities
        x[17] = inf


@pytest.mark.parametrize("n", [100, 300])
@pytest.mark.parametrize("kind", ["element", "row", "head", "all", "channel among zeros", "infinity", "infinity among zeros", "row of infinities"])
def test_pca_refuses_a_set_that_is_not_numbers(kind, n):
    x = torch.randn((n, 256), device="cuda", generator=torch.Generator("cuda").manual_seed(5)).half()
    _spoil(x, kind)
    for call in (B.rosaq_pca_full, B.rosaq_pca_headwise):
        for sweeps in (0, 1):
            print(f"case pca not numbers {kind} n_cal={n} {call.__name__} sweeps alone {sweeps}", flush=True)
            B.rosaq_tune("pca_sweeps", sweeps)
            try:
                with pytest.raises(B.RosaqError) as error:
                    call(x.data_ptr(), n, 256, 256)
            finally:
                B.rosaq_tune("pca_sweeps", 0)
            assert error.value.code == -8          # ROSAQ_ERR_HIP
