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


@pytest.mark.parametrize("where", ["W", "Q"])
def test_non_finite_input_is_found_in_the_last_chunk(where):
    D, N = 256, 300
    W = synth.make_weight(710, N, D)
    Q = synth.random_orthogonal_dense(711, D)
    (W if where == "W" else Q)[-1, -1] = np.inf
    with pytest.raises(B.RosaqError) as e:
        B.rosaq_pack_weights(W, Q, synth.descending_spectrum(712, D, 1), 128, 4, B.Q_FULL)
    assert B.ERR_NAMES[e.value.code] == "NONFINITE" and where + " contains" in str(e.value)
