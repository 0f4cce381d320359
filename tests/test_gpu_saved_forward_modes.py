"""When a forward is saved for its backward, and what happens to the saved
memory in between: nothing is saved without autograd."""
import pytest

from paper_2511_07737_amd import gen, tsat

from test_gpu_saved_forward import CNFS, env  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def inputs(torch, cnf, N, seed):
    T = torch.tensor(gen.normal_logits(cnf.num_vars, N, seed), device="cuda", requires_grad=True)
    return T, (T.detach() > 0).float().requires_grad_()


@pytest.mark.parametrize("guard", ["no_grad", "inference_mode", "set_grad_enabled"])
def test_nothing_saved_without_autograd(env, monkeypatch, guard):
    torch, s, ag = env
    cnf = CNFS["3sat"]()
    s.load(cnf)
    T, A = inputs(torch, cnf, 40, 3)
    want = ag.loss_of(T, s).detach(), ag.smoothmin_sat(A, s).detach()

    def refuse(*a, **k):
        raise AssertionError("a forward was saved")

    for name in ("saved_bytes", "loss_save_dev", "fwd_save_dev"):
        monkeypatch.setattr(tsat.Solver, name, refuse)
    with torch.set_grad_enabled(False) if guard == "set_grad_enabled" else getattr(torch, guard)():
        got = ag.loss_of(T, s), ag.smoothmin_sat(A, s)
    assert all(torch.equal(x, y) for x, y in zip(got, want))
    with pytest.raises(AssertionError):
        ag.loss_of(T, s)
