"""The allocation-free forward on a store whose unit tables fill its fixed
array at the launch shape's clauses per thread: coarser units, same results."""
import numpy as np
import pytest

from parity_util import solver_or_skip

pytestmark = pytest.mark.gpu


def test_unit_table_fits_by_coarser_units():
    torch = pytest.importorskip("torch")
    s = solver_or_skip()
    V, C, N = 100000, 5_800_000, 1024
    rng = np.random.default_rng(1)
    stream = np.zeros((C, 2), dtype=np.int32)
    stream[:, 0] = (rng.integers(1, V + 1, C) * rng.choice([-1, 1], C)).astype(np.int32)
    s.load_cnf(V, stream.ravel())
    s.set_launch_config(fwd_target_blocks=1 << 20)
    bits = torch.randint(-2**62, 2**62, (V, N // 64), device="cuda", dtype=torch.int64)
    st = torch.cuda.current_stream().cuda_stream
    out = [(torch.empty(N, device="cuda"), torch.empty((N, 2), dtype=torch.int32, device="cuda")) for _ in range(2)]
    s.fwd_dev(bits.data_ptr(), N, 1.0, out[0][0].data_ptr(), out[0][1].data_ptr(), st)
    s.fwd_dev_noalloc(bits.data_ptr(), N, 1.0, out[1][0].data_ptr(), out[1][1].data_ptr(), st)
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    assert int(out[1][1][0].sum()) == C
    s.close()
