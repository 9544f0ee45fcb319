"""torch.autograd.Function over the C ABI: nsteps semi-implicit steps as a
differentiable map (T0, chi) -> T_N.  The forward runs
asd_adjoint_forward_states (the steps, storing a checkpoint every ckpt_every
steps, or every state when there are at most two segments); the backward is
the hand-written adjoint asd_adjoint_step_states, which recomputes each
segment that was not stored from its checkpoint.  A forward that no gradient
can follow stores the checkpoints alone."""
import torch

from . import binding


class SemiImplicitSteps(torch.autograd.Function):
    """T_N = SemiImplicitSteps.apply(T0, chi, grid, dt, nsteps, ckpt_every)

    grid: a binding.Grid built with per_cell_chi=True and b already set.
    T0, chi: contiguous CUDA tensors of the grid's shape and dtype.
    Gradients flow to T0 and chi.
    """

    @staticmethod
    def forward(ctx, T0, chi, grid, dt, nsteps, ckpt_every):
        cur = torch.cuda.current_stream()
        grid.stream.wait_stream(cur)
        with torch.cuda.stream(grid.stream):
            chi_c = chi.detach().contiguous()
            grid.set_field("chi", chi_c)
            T = T0.detach().clone()
            grid.set_field("T", T)
            ws = grid.adjoint_forward(dt, nsteps, ckpt_every, states=any(ctx.needs_input_grad[:2]))
        cur.wait_stream(grid.stream)
        ctx.save_for_backward(chi_c)
        ctx.ws = ws  # the checkpoints (states at steps 0, k, 2k, ...), or all states
        ctx.grid, ctx.dt, ctx.nsteps, ctx.k = grid, dt, nsteps, ckpt_every
        return T

    @staticmethod
    def backward(ctx, gT):
        (chi,) = ctx.saved_tensors
        grid = ctx.grid
        cur = torch.cuda.current_stream()
        grid.stream.wait_stream(cur)
        with torch.cuda.stream(grid.stream):
            grid.set_field("chi", chi)
            gT0, gchi = grid.adjoint_stored(ctx.dt, ctx.nsteps, ctx.k, ctx.ws, gT.contiguous(), grad_chi=True,
                                            states=True)
        cur.wait_stream(grid.stream)
        ctx.ws = None
        return gT0, gchi, None, None, None, None


def semi_implicit_steps(T0, chi, grid, dt, nsteps, ckpt_every=10):
    if not torch.is_grad_enabled():  # needs_input_grad is of the tensors, not of the mode
        T0, chi = T0.detach(), chi.detach()
    return SemiImplicitSteps.apply(T0, chi, grid, dt, nsteps, ckpt_every)
