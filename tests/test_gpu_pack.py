"""Packing of float assignments into variable bits, exactly: word counts
around a wave's run of words, ragged last words, thresholds and NaN."""
import numpy as np
import pytest

from paper_2511_07737_amd import gen, tsat

from parity_util import solver_or_skip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,N", [(3, 1), (7, 64), (8, 63), (33, 65), (301, 100), (129, 200), (5, 1000), (4099, 24)])
def test_pack_equals_host(V, N):
    torch = pytest.importorskip("torch")
    s = solver_or_skip()
    if not torch.cuda.is_available():
        pytest.skip("torch sees no GPU")
    s.load(gen.planted_ksat(V, V, 3 if V > 3 else 2, seed=1))
    rng = np.random.default_rng(V * 1000 + N)
    a = rng.choice(np.array([0, 1, 0.5, np.nextafter(np.float32(0.5), np.float32(1)), -3, np.nan, np.inf, -np.inf],
                            dtype=np.float32), size=(V, N))
    t = torch.from_numpy(a).cuda()
    W = (N + 63) // 64
    out = torch.full((V * W + 8,), -1, dtype=torch.int64, device="cuda")
    s.pack_dev(t.data_ptr(), N, out.data_ptr(), torch.cuda.current_stream().cuda_stream)
    got = out.cpu().numpy()
    s.close()
    assert (got[V * W:] == -1).all()
    with np.errstate(invalid="ignore"):
        want = tsat.pack_bits((a > 0.5).astype(np.uint8))
    assert np.array_equal(got[:V * W].view(np.uint64).reshape(V, W), want.reshape(V, W))
