"""torch.autograd.Functions over the gfx950 kernels of the differentiable path.

The paper's graph (Sec. III-B, Fig. 3): logits theta [V][N] -> per-variable
normalization (Eq. 5) -> binarization B (Eq. 2, straight-through estimator
backward) -> R = P A (Eq. 1) -> SmoothMin per candidate (Eq. 4) -> loss
(Eq. 3).  Every step, forward and backward, runs in the HIP library through
its device-pointer entry points; this module only allocates the tensors,
passes their pointers and torch's current stream, and wires the backward.

* ``smoothmin_sat(assign)``: binary assignment A [V][N] (0/1 floats) -> S [N];
  backward dS -> dA through the transpose product (+1 for x_v, -1 for not x_v).
* ``binarize(theta, mode)``: Eq. 5 then Eq. 2 -> A (0/1 floats); backward is
  the Eq. 5 backward of the gradient the STE passes through Eq. 2.
* ``loss_of(theta)``: the whole chain to the scalar loss in one call, its
  backward in one fused pass (adjoint, Eq. 5 backward).

The layer and the loss keep the forward's histogram, row means and clause
planes (or bytes of R, or literal rows) in a saved tensor, so that the backward
does not form the forward again.  Each node holds its own until it is freed:
two to four bits per clause and candidate, or a byte where clauses pass 15
literals and for mixed widths past 256 candidates (up to 8 GiB).  Without a
gradient to compute nothing is kept: inside ``forward`` autograd is off and
``needs_input_grad`` only says that the input asks for a gradient, so the
wrappers pass on whether autograd was recording.
"""
from __future__ import annotations

import torch

from . import tsat


def _stream(t: torch.Tensor) -> int:
    return torch.cuda.current_stream(t.device).cuda_stream


def _logits(theta: torch.Tensor, solver: tsat.Solver) -> torch.Tensor:
    if not theta.is_cuda or theta.dtype != torch.float32 or theta.dim() != 2:
        raise ValueError("logits must be a 2-D float32 CUDA tensor [V][N]")
    if theta.shape[0] != solver.V:
        raise ValueError(f"logits have {theta.shape[0]} rows, the loaded CNF has {solver.V} variables")
    return theta.contiguous()


def _saved_buffer(solver: tsat.Solver, n: int, device) -> torch.Tensor | None:
    """Memory for a forward's saved state, or None where it does not fit or the
    candidates are too many for a backward (which then says so)."""
    if n > tsat.MAX_STEP_N:
        return None
    try:
        return torch.empty(solver.saved_bytes(n), dtype=torch.uint8, device=device)
    except torch.cuda.OutOfMemoryError:
        return None


def _readable(saved: list) -> bool:
    """Whether a backward has a saved state it can read: saved-tensor hooks may
    hand back a copy at any offset or stride (the plain call then runs)."""
    return bool(saved) and saved[0].is_cuda and saved[0].is_contiguous() and saved[0].data_ptr() % 256 == 0


def _upstream(t: torch.Tensor) -> torch.Tensor:
    if t.dtype != torch.float32:
        raise ValueError(f"upstream gradient must be float32 (got {t.dtype})")
    return t.contiguous()


class SmoothMinSat(torch.autograd.Function):
    @staticmethod
    def forward(ctx, assign: torch.Tensor, solver: tsat.Solver, tau: float, grad: bool = True):
        assign = _logits(assign, solver)
        V, N = assign.shape
        W = (N + 63) // 64
        stream = _stream(assign)
        bits = torch.empty((V, W), dtype=torch.int64, device=assign.device)
        solver.pack_dev(assign.data_ptr(), N, bits.data_ptr(), stream)
        S = torch.empty(N, dtype=torch.float32, device=assign.device)
        saved = _saved_buffer(solver, N, assign.device) if grad and ctx.needs_input_grad[0] else None
        if saved is None:
            solver.fwd_dev(bits.data_ptr(), N, tau, S.data_ptr(), None, stream)
            ctx.save_for_backward(bits)
        else:
            ctx.key = solver.fwd_save_dev(bits.data_ptr(), N, tau, S.data_ptr(), saved.data_ptr(), saved.numel(),
                                          stream)
            ctx.save_for_backward(bits, saved)
        ctx.solver = solver
        ctx.tau = tau
        ctx.shape = (V, N)
        return S

    @staticmethod
    def backward(ctx, dS: torch.Tensor):
        bits, *saved = ctx.saved_tensors
        V, N = ctx.shape
        dS = _upstream(dS)
        U = torch.empty((V, N), dtype=torch.float32, device=bits.device)
        if _readable(saved):
            ctx.solver.bwd_saved_dev(bits.data_ptr(), N, ctx.tau, dS.data_ptr(), U.data_ptr(), saved[0].data_ptr(),
                                     saved[0].numel(), ctx.key, _stream(bits))
        else:
            ctx.solver.bwd_dev(bits.data_ptr(), N, ctx.tau, dS.data_ptr(), U.data_ptr(), _stream(bits))
        return U, None, None, None


def smoothmin_sat(assign: torch.Tensor, solver: tsat.Solver, tau: float = 1.0) -> torch.Tensor:
    """S[N] of the binary assignment ``assign`` [V][N] (differentiable via the STE adjoint).
    With a gradient to compute, the node keeps ``solver.saved_bytes(N)`` bytes of GPU memory."""
    return SmoothMinSat.apply(assign, solver, float(tau), torch.is_grad_enabled())


class Binarize(torch.autograd.Function):
    @staticmethod
    def forward(ctx, theta: torch.Tensor, solver: tsat.Solver, mode: int):
        theta = _logits(theta, solver)
        assign = torch.empty_like(theta)
        solver.binarize_dev(theta.data_ptr(), theta.shape[1], mode, None, assign.data_ptr(), None, _stream(theta))
        ctx.save_for_backward(theta)
        ctx.solver = solver
        ctx.mode = mode
        return assign

    @staticmethod
    def backward(ctx, dA: torch.Tensor):
        (theta,) = ctx.saved_tensors
        dA = _upstream(dA)
        g = torch.empty_like(theta)
        ctx.solver.norm_backward_dev(theta.data_ptr(), dA.data_ptr(), theta.shape[1], ctx.mode, g.data_ptr(),
                                     _stream(theta))
        return g, None, None


def binarize(theta: torch.Tensor, solver: tsat.Solver, mode: int = tsat.MODE_MEAN) -> torch.Tensor:
    """A = B(theta / mean_row(theta)) (Eq. 5, Eq. 2; mode ``tsat.MODE_NONE``: B(theta))
    as 0/1 floats, with the straight-through estimator and the Eq. 5 backward."""
    return Binarize.apply(theta, solver, int(mode))


class LogitLoss(torch.autograd.Function):
    @staticmethod
    def forward(ctx, theta: torch.Tensor, solver: tsat.Solver, tau: float, mode: int, grad: bool = True):
        theta = _logits(theta, solver)
        loss = torch.empty((), dtype=torch.float32, device=theta.device)
        N, stream = theta.shape[1], _stream(theta)
        saved = _saved_buffer(solver, N, theta.device) if grad and ctx.needs_input_grad[0] else None
        if saved is None:
            solver.loss_dev(theta.data_ptr(), N, tau, mode, loss.data_ptr(), None, None, stream)
            ctx.save_for_backward(theta)
        else:
            ctx.key = solver.loss_save_dev(theta.data_ptr(), N, tau, mode, loss.data_ptr(), saved.data_ptr(),
                                           saved.numel(), stream)
            ctx.save_for_backward(theta, saved)
        ctx.solver = solver
        ctx.tau = tau
        ctx.mode = mode
        return loss

    @staticmethod
    def backward(ctx, dloss: torch.Tensor):
        theta, *saved = ctx.saved_tensors
        dloss = _upstream(dloss)
        g = torch.empty_like(theta)
        args = (theta.data_ptr(), theta.shape[1], ctx.tau, ctx.mode, dloss.data_ptr(), g.data_ptr(), None)
        if _readable(saved):
            ctx.solver.loss_backward_saved_dev(*args, saved[0].data_ptr(), saved[0].numel(), ctx.key, _stream(theta))
        else:
            ctx.solver.loss_backward_dev(*args, _stream(theta))
        return g, None, None, None, None


def loss_of(theta: torch.Tensor, solver: tsat.Solver, tau: float = 1.0, normalize: bool = True) -> torch.Tensor:
    """L = -sum_i S_i (Eq. 3) of the logits theta [V][N], as a 0-d tensor.
    With a gradient to compute, the node keeps ``solver.saved_bytes(N)`` bytes of GPU memory."""
    mode = tsat.MODE_MEAN if normalize else tsat.MODE_NONE
    return LogitLoss.apply(theta, solver, float(tau), mode, torch.is_grad_enabled())
