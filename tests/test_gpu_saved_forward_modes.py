"""When a forward is saved for its backward, and what happens to the saved
memory in between: nothing is saved without autograd, and a saved-tensor hook
may hand the memory back at any offset."""
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


def test_hooks_may_move_the_saved_state(env):
    torch, s, ag = env
    cnf = CNFS["3sat"]()
    s.load(cnf)
    T, A = inputs(torch, cnf, 40, 4)
    dS = torch.linspace(-1, 2, 40, device="cuda")

    def grads():
        return torch.autograd.grad(ag.loss_of(T, s), T) + torch.autograd.grad(ag.smoothmin_sat(A, s), A, dS)

    want = grads()
    spaced = lambda t: torch.stack([t, t], -1)[..., 0] if t.dtype == torch.uint8 else t  # noqa: E731
    for off in (1, 8, 64):
        def pack(t):
            # one arena for all tensors, offsets as they come (each type's own alignment kept)
            arena = torch.empty(off + 256 + t.numel() * t.element_size(), dtype=torch.uint8, device="cuda")
            at = off if t.dtype == torch.uint8 else 8
            part = arena[at:at + t.numel() * t.element_size()]
            part.copy_(t.reshape(-1).view(torch.uint8))
            return part, t.dtype, t.shape

        with torch.autograd.graph.saved_tensors_hooks(pack, lambda p: p[0].view(p[1]).view(p[2])):
            got = grads()
        assert all(torch.equal(x, y) for x, y in zip(got, want)), off
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t, spaced):
        assert all(torch.equal(x, y) for x, y in zip(grads(), want))
