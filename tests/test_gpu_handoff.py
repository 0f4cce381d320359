"""The hand-off selection against a host ranking of the library's own
gradient: candidates by satisfied clauses, then the k smallest |g| of the
variables that occur (ties: lower index), exactly.  More candidates than one
tile of slots, several variable chunks, k past the eligible variables, keys
that tie in long runs (an underflowing temperature), every gather that stores
the selected columns."""
import numpy as np
import pytest

from paper_2511_07737_amd import gen, tsat

from parity_util import solver_or_skip

pytestmark = pytest.mark.gpu


def unused_tail(cnf, extra):
    return gen.CNF.from_clauses(cnf.num_vars + extra, [list(cnf.clause(c)) for c in range(cnf.num_clauses)])


@pytest.mark.parametrize("V,C,k_sat,N,cands,k,tau,mode", [
    (40, 150, 3, 8, 8, 64, 1.0, tsat.MODE_MEAN),       # k past the eligible variables
    (700, 2800, 3, 32, 5, 20, 1.0, tsat.MODE_MEAN),    # two variables per wave
    (3001, 12000, 3, 100, 100, 33, 2.0, tsat.MODE_NONE),  # several tiles of slots and chunks
    (900, 3600, 2, 300, 33, 20, 1.0, tsat.MODE_MEAN),  # a team of waves per row
    (2000, 8000, 3, 64, 7, 300, 900.0, tsat.MODE_NONE),   # most gradients underflow to 0
    (1500, 6000, 0, 70, 40, 25, 1.0, tsat.MODE_NONE),  # mixed widths
    (600, 2400, 4, 20, 3, 4, 1.0, tsat.MODE_MEAN),
])
def test_selection_equals_host_ranking(V, C, k_sat, N, cands, k, tau, mode):
    solver_or_skip().close()
    cnf = unused_tail(gen.planted_ksat(V, C, k_sat, seed=3) if k_sat else gen.structured(V, C, seed=3), 5)
    s = tsat.Solver(params=tsat.default_params(norm_mode=mode, tau=tau))
    s.load(cnf)
    s.init_batch(N, seed=17)
    _, g = s.get_grad()
    sat, _ = s.check()
    bits = tsat.unpack_bits(s.get_bits(), N)
    for call in range(2):  # the second one on scratch the first has used
        ids, lits, counts = s.extract_partial(cands, k)
        order = np.lexsort((np.arange(N), -sat))[:cands]
        assert np.array_equal(ids, order) and np.array_equal(counts, sat[order])
        occurs = np.zeros(cnf.num_vars, bool)
        occurs[np.abs(cnf.lits) - 1] = True
        el = np.nonzero(occurs)[0]
        for a, i in enumerate(order):
            pick = el[np.lexsort((el, np.abs(g[el, i])))][:k]
            want = np.zeros(k, np.int32)
            want[:pick.size] = np.where(bits[pick, i] == 1, pick + 1, -(pick + 1))
            assert np.array_equal(lits[a], want), (call, a)
    s.close()
