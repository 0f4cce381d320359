"""When a forward is saved for its backward, and what happens to the saved
memory in between: nothing is saved without autograd, and a saved-tensor hook
may hand the memory back at any offset; several forwards before their
backwards."""
import pytest

from paper_2511_07737_amd import gen, tsat

from test_gpu_saved_forward import CNFS, env, plain_loss_grad  # noqa: F401  (env: fixture)

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


@pytest.mark.parametrize("name,N,cfg", [
    ("3sat", 20, {}), ("3sat", 20, dict(window_gather=0)), ("3sat", 130, {}), ("3sat", 130, dict(window_gather=0)),
    ("3sat", 300, {}), ("3sat", 300, dict(clause_planes=0)), ("4sat", 300, {}), ("4sat", 70, {}), ("mixed", 130, {}),
    ("mixed", 130, dict(window_gather=0)), ("mixed", 300, {}), ("wide", 100, {}), ("wide", 100, dict(clause_planes=0)),
])
def test_several_forwards_before_their_backwards(env, name, N, cfg):
    """Packed planes, windows, record by record, teams, levels, bytes and rows:
    by the first backward the solver's scratch is the last forward's."""
    torch, s, ag = env
    cnf = CNFS[name]()
    s.load(cnf)
    s.set_launch_config(**cfg)
    try:
        T1, _ = inputs(torch, cnf, N, 5)
        T2, A = inputs(torch, cnf, N, 6)
        dS = torch.linspace(-1, 2, N, device="cuda")
        l1, S, l2 = ag.loss_of(T1, s, 1.0), ag.smoothmin_sat(A, s, 1.5), ag.loss_of(T2, s, 2.0, normalize=False)
        got = [torch.autograd.grad(l1, T1)[0], torch.autograd.grad(S, A, dS)[0], torch.autograd.grad(l2, T2)[0]]
        bits = torch.empty((cnf.num_vars, (N + 63) // 64), dtype=torch.int64, device="cuda")
        st, U = torch.cuda.current_stream().cuda_stream, torch.empty_like(A)
        s.pack_dev(A.data_ptr(), N, bits.data_ptr(), st)
        s.bwd_dev(bits.data_ptr(), N, 1.5, dS.data_ptr(), U.data_ptr(), st)
        want = [plain_loss_grad(torch, s, T1.detach(), 1.0, tsat.MODE_MEAN, 1.0)[1], U,
                plain_loss_grad(torch, s, T2.detach(), 2.0, tsat.MODE_NONE, 1.0)[1]]
        assert all(torch.equal(x, y) for x, y in zip(got, want))
    finally:
        s.set_launch_config(clause_planes=1, window_gather=1)
