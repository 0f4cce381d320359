"""Features of uniform stores of every width that has header-less records, with
degrees around the record batch (0, 1, 3, 4, 5, 8, 9 records of a variable),
tautologies among them, against the FP64 oracle: FP32 sums of O(degree) terms
per round, 2e-5 of the largest magnitude of a column."""
import numpy as np
import pytest

import oracle as orc
from paper_2511_07737_amd import gen

from parity_util import solver_or_skip

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [2, 3, 4])
def test_degrees_around_the_batch(k):
    rng = np.random.default_rng(k)
    V, clauses = 60, []
    for v, deg in enumerate([0, 1, 3, 4, 5, 8, 9, 12, 13]):
        for _ in range(deg):
            others = rng.choice(np.arange(10, V + 1), size=k - 1, replace=False)
            sg = rng.choice([-1, 1], size=k)
            clauses.append([int((v + 1) * sg[0]), *(int(x) for x in others * sg[1:])])
    if k > 2:
        clauses += [[20, -20, *range(30, 28 + k)], [40, 21, -40, 50][:k]]
    else:
        clauses += [[20, -20], [40, -40]]
    cnf = gen.CNF.from_clauses(V, clauses)
    assert (np.diff(cnf.offsets) == k).all()
    s = solver_or_skip()
    s.load(cnf)
    X = s.get_features()
    s.close()
    ref = orc.features(orc.Cnf.from_gen(cnf))
    assert (np.abs(X - ref) <= 2e-5 * np.abs(ref).max(axis=0) + 1e-12).all()
