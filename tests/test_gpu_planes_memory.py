"""Where the memory for R past 256 candidates, or in bytes, does not fit: the
call runs on the row gather with the same results.  Each program runs in a
child process with allocations over a size refused."""
import os
import subprocess
import sys

import pytest

from parity_util import solver_or_skip

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# V = 200, C = 20000: the planes of N = 300 take 2.6 MB (bytes of R at N = 100
# the same, at N = 300 6.4 MB), every other buffer less than 1.3 MB
SETUP = """
import sys, hashlib; sys.path.insert(0, '.'); sys.path.insert(0, 'tests')
import numpy as np, torch
from paper_2511_07737_amd import gen, tsat
s = tsat.Solver()
uniform = gen.planted_ksat(200, 20000, 3, seed=1)
rng = np.random.default_rng(2)
wide = gen.CNF.from_clauses(200, [[int(x) for x in (rng.choice(200, size=k, replace=False) + 1) * rng.choice([-1, 1], size=k)]
                                  for k in [3] * 19900 + [18] * 100])
def digest(*arrays):
    return hashlib.sha256(b''.join(np.ascontiguousarray(a).tobytes() for a in arrays)).hexdigest()
def solve(N):
    s.init_batch(N, seed=3)
    s.step(4)
    return digest(*s.get_state()[:3], s.get_bits(), *s.get_grad())
def backward(N):
    b = torch.randint(-2**62, 2**62, (200, (N + 63) // 64), device='cuda', generator=torch.Generator('cuda').manual_seed(N))
    dS, U = torch.linspace(-1, 1, N, device='cuda'), torch.empty((200, N), device='cuda')
    s.bwd_dev(b.data_ptr(), N, 1.0, dS.data_ptr(), U.data_ptr(), torch.cuda.current_stream().cuda_stream)
    return digest(U.cpu().numpy())
"""


def run(body, over):
    env = dict(os.environ)
    if over:
        env["TSAT_FAIL_ALLOC_OVER"] = str(over)
    r = subprocess.run([sys.executable, "-c", SETUP + body], cwd=ROOT, env=env, capture_output=True, text=True,
                       timeout=100)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


@pytest.fixture(scope="module", autouse=True)
def gpu():
    solver_or_skip().close()


@pytest.mark.parametrize("cnf,N", [("uniform", 300), ("uniform", 1000), ("wide", 100), ("wide", 300)])
def test_row_gather_without_the_memory(cnf, N):
    body = f"s.load({cnf}); print(solve({N}), backward({N}), solve({N}))"
    assert run(body, 2_000_000) == run(body, 0)


def test_switched_on_later():
    body = "s.load(uniform); s.set_launch_config(clause_planes=0); s.init_batch(300, seed=1); " \
           "s.set_launch_config(clause_planes=1); s.step(3); print(digest(*s.get_state()[:3]))"
    assert run(body, 2_000_000) == run(body, 0)


def test_one_buffer_does_not_speak_for_the_others():
    """The scratch of a larger evaluation does not fit: the step, and forwards
    saved in the caller's memory, keep the bytes of R."""
    body = "s.load(wide); s.init_batch(100, seed=1); a = s.saved_bytes(100); backward(300); " \
           "print(a == s.saved_bytes(100), solve(100))"
    out = run(body, 4_000_000)
    assert out.startswith("True") and out == run(body, 0)
