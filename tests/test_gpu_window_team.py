"""Window gather of rows of more than 256 candidates (a team of waves per
block) against the record gather of the same rows, bit for bit, and one
iteration against the FP64 oracle: candidate counts around the team's edges
(257, whole and partial words and waves, 1024), widths 2 and 3, records over
several windows, variables without occurrences, instance boundaries and
frozen instances inside a team's variables, mixing, and the adjoint."""
import numpy as np
import pytest

import oracle as orc
from paper_2511_07737_amd import gen, tsat

from parity_util import TOL_GRAD, abs_adjoint, grad_bound, make_state, solver_or_skip
from test_gpu_window_gather import assert_same, hub_cnf, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,N", [(3, 257), (3, 320), (2, 512), (3, 513), (3, 700), (2, 1000), (3, 1024)])
def test_team_equals_record_gather(k, N):
    V = 301
    cnf = gen.planted_ksat(V, int((4.0 if k == 3 else 1.5) * V), k, seed=80 + k)
    print(f"[team] k={k} N={N}", flush=True)
    for mode in (tsat.MODE_MEAN, tsat.MODE_NONE):
        p = tsat.default_params(norm_mode=mode, tau=2.0 if mode == tsat.MODE_NONE else 1.0)
        assert_same(run([cnf], N, 1, 9, params=p), run([cnf], N, 0, 9, params=p))


def test_team_long_records_and_unused_variables():
    hub = hub_cnf()
    cnf = gen.CNF.from_clauses(hub.num_vars + 3, [list(hub.clause(c)) for c in range(hub.num_clauses)])
    p = tsat.default_params()
    assert_same(run([cnf], 600, 1, 5, params=p), run([cnf], 600, 0, 5, params=p))


def test_team_batch_with_frozen_instances():
    sizes = [(201, 560), (333, 1365), (99, 260), (150, 615), (77, 200)]
    cnfs = [gen.planted_ksat(V, C, 3, seed=60 + j) for j, (V, C) in enumerate(sizes)]
    p = tsat.default_params(norm_mode=tsat.MODE_NONE, tau=2.0)
    a = run(cnfs, 300, 1, 120, params=p, stop=True, seed=8)
    assert any(x["frozen"] for x in a["status"]) and not all(x["frozen"] for x in a["status"])
    assert_same(a, run(cnfs, 300, 0, 120, params=p, stop=True, seed=8))


def test_team_mixing():
    cnf = gen.planted_ksat(150, 620, 3, seed=5)
    p = tsat.default_params(mix=1, restart_every=6)
    assert_same(run([cnf], 400, 1, 15, params=p), run([cnf], 400, 0, 15, params=p))


@pytest.mark.parametrize("N", [257, 1000])
def test_team_gradient_vs_oracle(N):
    cnf = gen.planted_ksat(200, 820, 3, seed=21)
    th, _, _ = make_state(200, N, 900 + N, t_moments=False, min_abs_mu=1e-2)
    s = solver_or_skip()
    s.load(cnf)
    s.init_batch(N, init_logits=th)
    U, g = s.get_grad()
    hist, _, _ = s.eval()
    s.close()
    oc = orc.Cnf.from_gen(cnf)
    ref = orc.step(oc, th.astype(np.float64), np.zeros((200, N)), np.zeros((200, N)), 0)
    assert np.array_equal(hist.astype(np.int64), ref["H"])
    b, mu = orc.binarize(th.astype(np.float64), orc.MODE_MEAN)
    _, table, _ = orc.smoothmin(orc.histogram(oc, b), 1.0)
    aU = abs_adjoint(oc, b, table)
    assert (np.abs(U - orc.adjoint(oc, b, table)) <= TOL_GRAD * aU + 1e-30).all()
    assert (np.abs(g - ref["g"]) <= TOL_GRAD * grad_bound(aU, th, mu, ref["g"]) + 1e-30).all()


@pytest.mark.parametrize("V", [2048, 2049, 8193])
def test_variables_per_wave(V):
    """One, two and four variables per wave by the store's size (the last item
    cut short)."""
    cnf = gen.planted_ksat(V, 4 * V, 3, seed=V)
    p = tsat.default_params()
    assert_same(run([cnf], 65, 1, 3, params=p), run([cnf], 65, 0, 3, params=p))
