"""Forward histograms of candidate counts around the tiles of a block (33 to 63
dwords go in two tiles), one width and several, against the oracle, exactly."""
import numpy as np
import pytest

import oracle as orc
from paper_2511_07737_amd import gen, tsat

from parity_util import solver_or_skip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [1000, 1024, 1025, 1056, 1057, 1088, 1089, 1500, 2015, 2016, 2017, 2047, 2048, 2049, 3000])
@pytest.mark.parametrize("case", ["3sat", "mixed"])
def test_histogram_vs_oracle(case, N):
    torch = pytest.importorskip("torch")
    s = solver_or_skip()
    rng = np.random.default_rng(N)
    if case == "3sat":
        cnf = gen.planted_ksat(60, 500, 3, seed=1)
    else:
        widths = [1] * 5 + [2] * 200 + [3] * 300 + [4] * 90 + [6] * 20
        cnf = gen.CNF.from_clauses(60, [[int(x) for x in (rng.choice(60, size=k, replace=False) + 1) *
                                         rng.choice([-1, 1], size=k)] for k in widths])
    s.load(cnf)
    b = (rng.random((60, N)) < 0.5).astype(np.uint8)
    bits = torch.tensor(tsat.pack_bits(b).view(np.int64), device="cuda")
    S = torch.empty(N, device="cuda")
    H = torch.empty((N, s.max_width + 1), dtype=torch.int32, device="cuda")
    s.fwd_dev(bits.data_ptr(), N, 1.0, S.data_ptr(), H.data_ptr(), torch.cuda.current_stream().cuda_stream)
    assert np.array_equal(H.cpu().numpy().astype(np.int64), orc.histogram(orc.Cnf.from_gen(cnf), b))
    s.close()
