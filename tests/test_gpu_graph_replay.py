"""Graph replay of runs around the long graph's length (16 iterations), run
lengths that leave short graphs and an eager iteration, batches re-started in
the same buffers (the graph is kept) and in others, and stops between two
looks at the stop flag: everything as in the eager run, bit for bit."""
import numpy as np
import pytest

from paper_2511_07737_amd import gen, tsat

from parity_util import solver_or_skip

pytestmark = pytest.mark.gpu

KEYS = ("first_sat_step", "first_converged_step", "frozen", "best_sat_count", "best_candidate", "loss")


def outcome(s, rep):
    return (rep.steps_done, rep.next_step, s.get_logits(), s.get_bits(),
            [[x[k] for k in KEYS] for x in s.instance_status()])


def same(a, b):
    assert a[0] == b[0] and a[1] == b[1]
    assert np.array_equal(a[2], b[2]) and np.array_equal(a[3], b[3]) and a[4] == b[4]


def test_run_lengths_and_restarts():
    cnf = gen.planted_ksat(120, 500, 3, seed=2)
    eager, graph = solver_or_skip(), tsat.Solver()
    eager.load(cnf)
    graph.load(cnf)
    graph.set_graph(True)
    for N, lengths in ((40, (1, 2, 15, 16, 17, 18, 33, 50)), (100, (49, 16)), (40, (48, 3))):
        for s in (eager, graph):
            s.init_batch(N, seed=N)
        for n in lengths:
            outs = []
            for s in (eager, graph):
                rep = s.step(n)
                outs.append(outcome(s, rep))
                s.eval()  # eager work between replays
            same(*outs)
    eager.close()
    graph.close()


@pytest.mark.parametrize("stop", [1, 2])
def test_stops(stop):
    p = tsat.default_params(norm_mode=tsat.MODE_NONE, tau=2.0)
    cnfs = [gen.planted_ksat(V, 3 * V, 3, seed=V) for V in (60, 90, 130)]
    for cap in (500, 37):
        outs = []
        for graph in (False, True):
            s = tsat.Solver(params=p)
            s.load_batch(cnfs)
            s.set_graph(graph)
            for _ in range(2):  # the second start replays the first one's graph
                s.init_batch(64, seed=3)
                rep = s.step(cap, stop_on_sat=stop)
            outs.append(outcome(s, rep))
            s.close()
        if cap == 500:
            assert all(r[2] for r in outs[0][4]), "every instance stops"
        same(*outs)
