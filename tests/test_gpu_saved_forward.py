"""Backward from a saved forward against the plain calls, bit for bit: every
row form (packed planes, windows, teams of waves, mixed widths, literal rows
for clauses past the planes), both normalizations, several backwards from one
forward, and a key that no longer matches (launch shapes changed, another CNF
loaded), where the plain call runs."""
import numpy as np
import pytest

from paper_2511_07737_amd import gen, tsat

from parity_util import solver_or_skip

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    s = solver_or_skip()
    if not torch.cuda.is_available():
        pytest.skip("torch sees no GPU")
    from paper_2511_07737_amd import autograd

    yield torch, s, autograd
    s.close()


def plain_loss_grad(torch, s, T, tau, mode, scale):
    V, N = T.shape
    st = torch.cuda.current_stream().cuda_stream
    loss, g = torch.empty((), device="cuda"), torch.empty_like(T)
    d = torch.full((), scale, device="cuda")
    s.loss_dev(T.data_ptr(), N, tau, mode, loss.data_ptr(), None, None, st)
    s.loss_backward_dev(T.data_ptr(), N, tau, mode, d.data_ptr(), g.data_ptr(), None, st)
    return loss, g


CNFS = {
    "3sat": lambda: gen.planted_ksat(501, 2000, 3, seed=4),
    "4sat": lambda: gen.planted_ksat(301, 1500, 4, seed=4),
    "mixed": lambda: gen.structured(640, 3000, seed=4),
    "wide": lambda: gen.structured(640, 3000, seed=4, kmax=24, communities=3),
}


@pytest.mark.parametrize("name,N", [("3sat", 1), ("3sat", 32), ("3sat", 200), ("3sat", 300), ("4sat", 70),
                                    ("mixed", 100), ("wide", 100), ("wide", 256)])
def test_saved_equals_plain(env, name, N):
    torch, s, ag = env
    cnf = CNFS[name]()
    s.load(cnf)
    T = torch.tensor(gen.normal_logits(cnf.num_vars, N, 60 + N), device="cuda", requires_grad=True)
    for normalize in (True, False):
        mode = tsat.MODE_MEAN if normalize else tsat.MODE_NONE
        loss = ag.loss_of(T, s, 1.5, normalize=normalize)
        (g,) = torch.autograd.grad(2.5 * loss, T, retain_graph=True)
        (g2,) = torch.autograd.grad(2.5 * loss, T)
        want_l, want_g = plain_loss_grad(torch, s, T.detach(), 1.5, mode, 2.5)
        assert torch.equal(loss.detach(), want_l) and torch.equal(g, want_g) and torch.equal(g2, want_g)
        with torch.no_grad():
            assert torch.equal(ag.loss_of(T, s, 1.5, normalize=normalize), want_l)
    # the layer
    A = (T.detach() > 0).float().requires_grad_()
    S = ag.smoothmin_sat(A, s, 1.0)
    dS = torch.linspace(-1, 2, N, device="cuda")
    (U,) = torch.autograd.grad(S, A, dS)
    bits = torch.empty((cnf.num_vars, (N + 63) // 64), dtype=torch.int64, device="cuda")
    st = torch.cuda.current_stream().cuda_stream
    s.pack_dev(A.data_ptr(), N, bits.data_ptr(), st)
    want_S, want_U = torch.empty(N, device="cuda"), torch.empty_like(A)
    s.fwd_dev(bits.data_ptr(), N, 1.0, want_S.data_ptr(), None, st)
    s.bwd_dev(bits.data_ptr(), N, 1.0, dS.data_ptr(), want_U.data_ptr(), st)
    assert torch.equal(S.detach(), want_S) and torch.equal(U, want_U)


def test_key_that_no_longer_matches(env):
    torch, s, ag = env
    cnf = CNFS["3sat"]()
    T = torch.tensor(gen.normal_logits(cnf.num_vars, 30, 7), device="cuda", requires_grad=True)
    s.load(cnf)
    want_l, want_g = plain_loss_grad(torch, s, T.detach(), 1.0, tsat.MODE_MEAN, 1.0)
    loss = ag.loss_of(T, s, 1.0)
    for cfg in (dict(window_gather=0), dict(clause_planes=0), dict(window_gather=1, clause_planes=1)):
        s.set_launch_config(**cfg)
        (g,) = torch.autograd.grad(loss, T, retain_graph=True)
        assert torch.equal(g, want_g), cfg
    other = gen.planted_ksat(cnf.num_vars, 1000, 3, seed=9)
    s.load(other)
    (g,) = torch.autograd.grad(loss, T)
    assert torch.equal(g, plain_loss_grad(torch, s, T.detach(), 1.0, tsat.MODE_MEAN, 1.0)[1])


def test_saved_buffer_is_checked(env):
    torch, s, _ = env
    s.load(CNFS["3sat"]())
    T = torch.zeros((501, 64), device="cuda")
    loss = torch.empty((), device="cuda")
    need = s.saved_bytes(64)
    buf = torch.empty(need, dtype=torch.uint8, device="cuda")
    for ptr, n in ((buf.data_ptr(), need - 1), (buf.data_ptr() + 16, need)):
        with pytest.raises(tsat.TsatError) as e:
            s.loss_save_dev(T.data_ptr(), 64, 1.0, tsat.MODE_MEAN, loss.data_ptr(), ptr, n)
        assert e.value.code == tsat.E_ARG
