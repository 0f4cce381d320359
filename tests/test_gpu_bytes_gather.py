"""Generic records over the forward's bytes of R (clauses wider than 15, or
mixed widths and N > 256) against the row gather (clause planes off): both add
the same table entries in FP64 in the same order, so step, gradient and
adjoint agree bit for bit; and one iteration's histogram and adjoint against
the FP64 oracle.  Clauses up to 32 wide, candidate counts around words and
dwords, heavy variables (chunked records), batches with frozen members,
mixing, one and several narrow widths."""
import numpy as np
import pytest

import oracle as orc
from paper_2511_07737_amd import gen, tsat

from parity_util import TOL_GRAD, abs_adjoint, make_state, solver_or_skip
from test_gpu_window_gather import assert_same

pytestmark = pytest.mark.gpu


def random_cnf(V, counts, seed, hubs=0):
    """counts: {width: clauses}; with hubs, every other clause holds one of the
    first `hubs` variables."""
    rng = np.random.default_rng(seed)
    clauses = []
    for k, n in counts.items():
        for c in range(n):
            vs = rng.choice(np.arange(hubs, V), size=k, replace=False) + 1
            if hubs and c % 2:
                vs[0] = 1 + c % hubs
            clauses.append([int(x) for x in vs * rng.choice([-1, 1], size=k)])
    return gen.CNF.from_clauses(V, clauses)


CNFS = {
    "wide": lambda: random_cnf(400, {1: 3, 2: 300, 3: 500, 4: 100, 5: 60, 9: 40, 16: 30, 17: 20, 32: 10}, 1),
    "only_wide": lambda: random_cnf(300, {20: 200, 31: 50}, 2),
    "one_narrow": lambda: random_cnf(300, {3: 600, 18: 60}, 3),
    "mixed15": lambda: random_cnf(300, {2: 300, 3: 300, 7: 100, 15: 40}, 4),
    "hubs": lambda: random_cnf(260, {3: 1500, 6: 600, 20: 200}, 5, hubs=3),
}


def run(cnfs, N, planes, steps, params, stop=False, seed=5):
    s = solver_or_skip()
    s.load_batch(cnfs)
    s.set_launch_config(clause_planes=planes)
    s.init_batch(N, seed=seed)
    rep = s.step(steps, params=params, stop_on_sat=stop)
    th, m, v, t = s.get_state()
    out = dict(theta=th, m=m, v=v, t=t, bits=s.get_bits(), steps=rep.steps_done)
    out["U"], out["g"] = s.get_grad(params)
    out["status"] = s.instance_status()
    out["witness"] = [s.get_witness_instance(j, c.num_vars) if x["first_sat_step"] >= 0 else None
                      for j, (x, c) in enumerate(zip(out["status"], cnfs))]
    s.close()
    return out


@pytest.mark.parametrize("name,N", [("wide", 1), ("wide", 20), ("wide", 64), ("wide", 100), ("wide", 200), ("wide", 390),
                                    ("only_wide", 33), ("one_narrow", 130), ("mixed15", 257), ("mixed15", 1000),
                                    ("hubs", 70), ("hubs", 300)])
def test_bytes_equal_row_gather(name, N):
    cnf = CNFS[name]()
    print(f"[bytes] {name} N={N}", flush=True)
    for mode in (tsat.MODE_MEAN, tsat.MODE_NONE):
        p = tsat.default_params(norm_mode=mode, tau=2.0 if mode == tsat.MODE_NONE else 1.0)
        assert_same(run([cnf], N, 1, 6, p), run([cnf], N, 0, 6, p))


def test_bytes_batch_frozen_and_mixing():
    cnfs = [random_cnf(V, {2: V // 2, 3: 2 * V, 16: 5}, V) for V in (50, 81, 200)] + [CNFS["hubs"]()]
    p = tsat.default_params(norm_mode=tsat.MODE_NONE, tau=2.0)
    a = run(cnfs, 40, 1, 200, p, stop=True)
    assert any(x["frozen"] for x in a["status"]) and not all(x["frozen"] for x in a["status"])
    assert_same(a, run(cnfs, 40, 0, 200, p, stop=True))
    p = tsat.default_params(mix=1, restart_every=5)
    assert_same(run(cnfs, 40, 1, 12, p), run(cnfs, 40, 0, 12, p))


@pytest.mark.parametrize("name,N", [("wide", 100), ("mixed15", 300)])
def test_bytes_adjoint_vs_oracle(name, N):
    cnf = CNFS[name]()
    th, _, _ = make_state(cnf.num_vars, N, 70 + N, t_moments=False)
    s = tsat.Solver(params=tsat.default_params(norm_mode=tsat.MODE_NONE))
    s.load(cnf)
    s.init_batch(N, init_logits=th)
    U, _ = s.get_grad()
    hist, _, _ = s.eval()
    s.close()
    oc = orc.Cnf.from_gen(cnf)
    b = (th > 0).astype(np.uint8)
    H = orc.histogram(oc, b)
    assert np.array_equal(hist.astype(np.int64), H)
    _, table, _ = orc.smoothmin(H, 1.0)
    assert (np.abs(U - orc.adjoint(oc, b, table)) <= TOL_GRAD * abs_adjoint(oc, b, table) + 1e-30).all()
