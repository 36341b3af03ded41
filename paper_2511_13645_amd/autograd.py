"""torch.autograd wrapper around the C-ABI operator (Sec. 3.3 of arXiv 2511.13645:
``save_indices`` records the sampled IDs in forward and replays them in backward, so that
gradients reach the same sampled neighborhoods).

Only glue: forward calls ``fsa_sample_mean_fwd``, backward calls ``fsa_mean_bwd_dense`` where that pays, else
``fsa_mean_bwd`` (fp32) or ``fsa_mean_bwd_lp`` (16-bit tables or gradients), on the IDs saved by that forward.  IDs are
emitted only when the feature table needs a gradient (or the caller asks for them), as in the
paper's optional flag.

A bf16 / fp16 table gets its gradient in its own type, or --
when the caller passes ``master_grad``, an fp32 [N,D] tensor -- the backward accumulates into
that master gradient instead and leaves ``x.grad`` unset.  A master gradient is added to with
atomics, so backward passes on several streams may share one.  ``workspace`` (any contiguous GPU
tensor, optional) goes to ``fsa_mean_bwd_ws``: wide-row 2-hop backward passes over an fp32 table
then update every destination row once instead of once per sampled leaf.
"""
from __future__ import annotations

from typing import Optional, Sequence, Tuple

import torch

from . import binding


class _FusedSampleMean(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, indptr, indices, seeds, fanouts, seed, want_h1, save_indices, master_grad, workspace):
        fan = [int(k) for k in fanouts]
        need_ids = bool(save_indices or x.requires_grad)
        out, h1, ids1, ids2 = binding.fsa_sample_mean_fwd(indptr, indices, x, seeds, fan, seed,
                                                          emit_h1=bool(want_h1) and len(fan) == 2,
                                                          emit_ids=need_ids)
        ctx.shape = tuple(x.shape)
        ctx.x_dtype = x.dtype
        ctx.hops = len(fan)
        ctx.master_grad = master_grad
        ctx.workspace = workspace
        # gradients of outputs that the loss does not use stay None: the IDs' (and an unused out_h1's) would
        # each be an allocation and a fill launch
        ctx.set_materialize_grads(False)
        ids = tuple(t for t in (ids1, ids2) if t is not None)
        ctx.save_for_backward(*ids)
        ctx.mark_non_differentiable(*ids)
        return out, h1, ids1, ids2

    @staticmethod
    def backward(ctx, g_out, g_h1, _g_ids1, _g_ids2):
        saved = ctx.saved_tensors
        if not saved:
            raise RuntimeError("backward needs the sampled IDs: call with save_indices=True or a table that requires grad")
        ids1 = saved[0]
        ids2 = saved[1] if ctx.hops == 2 else None
        gh = None
        if ctx.hops == 2 and g_h1 is not None and g_h1.numel() > 0:
            gh = g_h1.contiguous()
        if g_out is None:                       # only out_h1 was used
            g_out = ids1.new_zeros((ids1.shape[0], ctx.shape[1]), dtype=ctx.x_dtype)
        g_out = g_out.contiguous()
        if ctx.master_grad is not None:
            binding.fsa_mean_bwd_lp(g_out, ids1, ids2, gh, grad_x=ctx.master_grad)
            return (None,) * 10
        n, d = ctx.shape
        # x.grad is a tensor of its own: written row by row where that is faster than clearing it and adding, unless
        # a caller's workspace buys sums whose order does not vary; 16-bit rows of odd length are summed in fp32 to the end
        if ctx.x_dtype == torch.float32:
            owned = (ctx.workspace is not None and ids2 is not None and
                     binding.fsa_mean_bwd_workspace_bytes(ids1.shape[0], ids1.shape[1], ids2.shape[2], d) > 0)
        else:
            owned = d % 2 != 0
        if not owned:
            if ctx.workspace is not None and ctx.x_dtype == torch.float32:
                binding.check_workspace(ctx.workspace, g_out)       # unused here, and refused all the same if it is no workspace
            if g_out.dtype is not ctx.x_dtype:
                g_out = g_out.to(ctx.x_dtype)
            if gh is not None and gh.dtype is not ctx.x_dtype:
                gh = gh.to(ctx.x_dtype)
            grad_x = binding.grad_dense(g_out, ids1, ids2, gh, n)
            if grad_x is not None:
                return (grad_x,) + (None,) * 9
        if ctx.x_dtype == torch.float32:
            grad_x = torch.zeros(ctx.shape, dtype=torch.float32, device=g_out.device)
            binding.fsa_mean_bwd_ws(g_out.float(), ids1, ids2, None if gh is None else gh.float(), grad_x=grad_x,
                                    workspace=ctx.workspace)
        elif ctx.shape[1] % 2 == 0:
            grad_x = torch.zeros(ctx.shape, dtype=ctx.x_dtype, device=g_out.device)
            binding.fsa_mean_bwd_lp(g_out, ids1, ids2, gh, grad_x=grad_x)
        else:                                   # packed atomics take element pairs: odd D goes through fp32
            master = torch.zeros(ctx.shape, dtype=torch.float32, device=g_out.device)
            binding.fsa_mean_bwd_lp(g_out, ids1, ids2, gh, grad_x=master)
            grad_x = master.to(ctx.x_dtype)
        return (grad_x,) + (None,) * 9


def fused_sample_mean(x: torch.Tensor, indptr: torch.Tensor, indices: torch.Tensor, seeds: torch.Tensor,
                      fanouts: Sequence[int], seed: int, *, want_h1: bool = False, save_indices: bool = False,
                      master_grad: Optional[torch.Tensor] = None, workspace: Optional[torch.Tensor] = None
                      ) -> Tuple[torch.Tensor, Optional[torch.Tensor], Optional[torch.Tensor], Optional[torch.Tensor]]:
    """Differentiable fused sample + mean.  Returns (out, out_h1 | None, ids1 | None, ids2 | None).
    `master_grad` (fp32 [N,D], optional): backward accumulates the table's gradient into it.
    `workspace` (optional, see binding.fsa_mean_bwd_workspace_bytes): lets the fp32 backward own its rows."""
    if master_grad is not None and (master_grad.dtype != torch.float32 or tuple(master_grad.shape) != tuple(x.shape)):
        raise ValueError("master_grad must be an fp32 tensor of the table's shape")
    out, h1, ids1, ids2 = _FusedSampleMean.apply(x, indptr, indices, seeds, tuple(fanouts), int(seed),
                                                 bool(want_h1), bool(save_indices), master_grad, workspace)
    return (out, h1, ids1 if ids1 is not None and ids1.numel() else None, ids2 if ids2 is not None and ids2.numel() else None)
