"""The offline step on the GPU at the edges of its row chunks and of the 128 x 128 tiles of the rotation: against the host
path, which shares no arithmetic code with it, bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2506_13472_amd import binding as B
from paper_2506_13472_amd import synth

pytestmark = pytest.mark.gpu


# 8 MiB of W or more to a chunk: D = 1024 -> 8192 rows with a dense rotation (64 row tiles x 8), 4096 without
@pytest.mark.parametrize("mode,bits,D,N", [(B.Q_HEADWISE, 4, 128, 1), (B.Q_FULL, 3, 256, 127), (B.Q_FULL, 4, 384, 129),
                                           (B.Q_FULL, 3, 1024, 8193), (B.Q_HEADWISE, 4, 1024, 4097), (B.Q_NONE, 3, 1024, 8320)])
def test_chunks_equal_the_host_path(mode, bits, D, N):
    print(f"case pack chunks mode={mode} bits={bits} D={D} N={N}", flush=True)
    W = synth.make_weight(700 + N, N, D)
    Q = {B.Q_NONE: lambda: None, B.Q_FULL: lambda: synth.random_orthogonal_dense(701, D),
         B.Q_HEADWISE: lambda: synth.random_orthogonal_blocks(702, D // 128)}[mode]()
    lam = synth.descending_spectrum(703, D, D // 128 if mode == B.Q_HEADWISE else 1)
    a = B.rosaq_pack_weights(W, Q, lam, 0 if D == 128 else 128, bits, mode)
    b = B.rosaq_pack_weights(W, Q, lam, 0 if D == 128 else 128, bits, mode, host_only=True)
    ea, eb = B.rosaq_packed_export(a), B.rosaq_packed_export(b)
    for k in ea:
        assert np.array_equal(ea[k].view(np.uint8), eb[k].view(np.uint8)), k
    for which in (0, 1):
        assert np.array_equal(B.rosaq_packed_image(a, which + 2), B.rosaq_packed_image(b, which)), which
    a.free(); b.free()


def test_chunks_of_a_pitched_weight_equal_the_host_path():
    """Three chunks of a weight whose rows are further apart than its columns (NaN between them)."""
    D, N, ldw = 1024, 8300, 1032
    print(f"case pack pitched N={N}", flush=True)
    wide = np.full((N, ldw), np.nan, np.float16)
    wide[:, :D] = synth.make_weight(705, N, D)
    Q, lam = synth.random_orthogonal_blocks(706, D // 128), synth.descending_spectrum(707, D, D // 128)
    a, b = (B.rosaq_pack_weights(wide, Q, lam, 128, 3, B.Q_HEADWISE, ldw=ldw, out_features=N, in_features=D, host_only=h)
            for h in (False, True))
    ea, eb = B.rosaq_packed_export(a), B.rosaq_packed_export(b)
    for k in ea:
        assert np.array_equal(ea[k].view(np.uint8), eb[k].view(np.uint8)), k
    for which in (0, 1):
        assert np.array_equal(B.rosaq_packed_image(a, which + 2), B.rosaq_packed_image(b, which)), which
    a.free(); b.free()


# the last row of two or three chunks (and Q's last entry), a sum that overflows in the last chunk
@pytest.mark.parametrize("where,mode,N", [("W", B.Q_NONE, 4097)] + [(w, m, n) for w in ("W", "Q", "rotated weight")
                                                                    for m, n in ((B.Q_FULL, 8193), (B.Q_HEADWISE, 8300))])
def test_non_finite_input_is_found_in_the_last_chunk(where, mode, N):
    print(f"case pack non-finite {where} mode={mode} N={N}", flush=True)
    D = 1024
    W = np.full((N, D), 2.0 ** -5, np.float16)
    Q = None if mode == B.Q_NONE else np.full((D, D) if mode == B.Q_FULL else (D // 128, 128, 128), 0.25, np.float32)
    if where == "rotated weight":
        W[-1] = 60000.0                              # 128 or 1024 quarters of it
    else:
        (W if where == "W" else Q).reshape(-1)[-1] = np.inf
    with pytest.raises(B.RosaqError) as e:
        B.rosaq_pack_weights(W, Q, synth.descending_spectrum(712, D, 1), 128, 4, mode)
    assert B.ERR_NAMES[e.value.code] == "NONFINITE" and where + (" overflows" if " " in where else " contains") in str(e.value)


@pytest.mark.parametrize("mode", [B.Q_FULL, B.Q_HEADWISE])
def test_rotation_adds_the_channels_in_order(mode):
    """The host adds the products one channel after the other in fp64.  Every sum here depends on that order: among each
    four channels, the share of one matrix instruction, two products of 2^57 cancel, and what is added between them is
    rounded to a multiple of 16 or 32, so that another order, or a wider intermediate, gives other whole numbers."""
    print(f"case pack order mode={mode}", flush=True)
    D, N = 256, 130
    rng = np.random.default_rng(720)
    blocks, width = (1, D) if mode == B.Q_FULL else (D // 128, 128)
    small = rng.integers(-31, 32, (blocks, width // 4, 2, width)).astype(np.float64)
    big = 2.0 ** 57 * rng.choice([-1.0, 1.0], (blocks, width // 4, 1, width))
    four = rng.permuted(np.concatenate([small, big, -big], axis=2), axis=2)
    Q = four.reshape(blocks, width, width).astype(np.float32)
    W = rng.choice([-1.0, 1.0], N).astype(np.float16)[:, None] * np.ones((1, D), np.float16)
    want, back = np.zeros((blocks, width)), np.zeros((blocks, width))
    for k in range(width):                           # numpy's adds round as the host's do
        want += Q[:, k]
        back += Q[:, width - 1 - k]
    assert np.mean(want != back) > 0.9 and np.max(np.abs(want)) <= 2048        # whole numbers that fp16 holds
    lam = synth.descending_spectrum(721, D, 1)
    a = B.rosaq_pack_weights(W, Q[0] if mode == B.Q_FULL else Q, lam, D, 4, mode)       # all channels stay fp16
    b = B.rosaq_pack_weights(W, Q[0] if mode == B.Q_FULL else Q, lam, D, 4, mode, host_only=True)
    ea, eb = B.rosaq_packed_export(a), B.rosaq_packed_export(b)
    assert np.array_equal(eb["W_S"], (W[:, :1].astype(np.float64) * want.reshape(1, D)).astype(np.float16))
    assert np.array_equal(ea["W_S"], eb["W_S"])
    a.free(); b.free()
