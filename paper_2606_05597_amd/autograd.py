"""torch.autograd wrappers of the loss entry points, for training loops that call ``loss.backward()``.

Each forward runs one library call that produces the loss and its gradients together (the GRPO loss of Eq. 1,
dual clip of Eq. 2), saves the gradients, and returns the loss as a 0-dim fp64 tensor; backward hands the saved
gradients back.  Behaviour and advantages are constants (no gradient), as in the paper's objective.

Neither direction synchronises with the host.  How backward treats the incoming gradient g of the loss is the
``upstream`` option:
  "scale" (default)  the saved gradients times g, on the device (an elementwise pass over them; exact when g is
                     1 or a power of two);
  "unit"             the saved gradients as the library wrote them: the caller guarantees g = 1 (``loss.backward()``
                     on this loss, or on a sum it enters with weight 1) and folds any known factor into the forward's
                     ``grad_scale``.  No extra pass: the right mode for the logits path, whose gradient is as large
                     as the logits.
"""
from __future__ import annotations

import torch

from . import _check, _lib, _ptr, _stream, fused_lmhead_grpo, fused_lmhead_grpo_blocked, grpo_loss_fwd_bwd

_UPSTREAM = ("scale", "unit")


def _upstream(opts):
    mode = opts.pop("upstream", "scale")
    if mode not in _UPSTREAM:
        raise ValueError(f"upstream must be one of {_UPSTREAM}, got {mode!r}")
    return mode


def _apply_upstream(mode, grads, grad_output):
    if mode == "unit":
        return grads
    return tuple(None if t is None else torch.mul(t, grad_output.to(t.dtype)) for t in grads)


def _plain(t):
    """A tensor whose memory a kernel may be handed: no subclass, not batched or otherwise wrapped by a transform, its
    values as they lie in memory (a zero tensor has none)."""
    return (type(t) is torch.Tensor and not torch._C._functorch.is_functorch_wrapped_tensor(t) and t.is_cuda
            and not t.is_neg() and not t._is_zerotensor())


def _watched():
    """Whether something follows the torch operations made now: a graph, forward-mode derivatives, a dispatch mode
    (fake tensors, a tracer, a flop counter), a function mode, a trace or the compiler."""
    return (torch.is_grad_enabled() or torch.autograd.forward_ad._current_level >= 0
            or torch._C._len_torch_dispatch_stack() > 0 or torch._C._len_torch_function_stack() > 0
            or torch._C._get_tracing_state() is not None
            or torch.compiler.is_compiling())


# Elements of dW from which its scale and its rounding are one pass: 8 bytes less to move per element, 6 us at 5.3 TB/s
# here, what a call of the library costs the autograd engine's thread more than the two torch operations do.  A backward
# of 64 x 512 weights took 85 us of host time with the one pass and 80 with the two operations.
_ONE_PASS_MIN = 1 << 22


def _scaled_to_bf16(t, grad_output):
    """(t * grad_output in fp32) rounded to bf16, in one pass over t where nothing has to see the two operations
    (_watched, _plain), a contiguous t as the library wrote it."""
    if (_watched() or not (_plain(t) and _plain(grad_output))
            or t.dtype != torch.float32 or not t.is_contiguous() or t.data_ptr() % 16 or grad_output.numel() != 1
            or grad_output.device != t.device):
        return torch.mul(t, grad_output.to(t.dtype)).to(torch.bfloat16)
    out = torch.empty_like(t, dtype=torch.bfloat16)
    g = grad_output.to(torch.float32)
    _check(_lib.load().grpo_binding_scale_to_bf16(_ptr(t), _ptr(g), _ptr(out), t.numel(), _stream(None)),
           "grpo_binding_scale_to_bf16")
    return out


class GrpoLoss(torch.autograd.Function):
    """``loss = GrpoLoss.apply(logits, actions, behave_logp, adv, step_tok_off, traj_step_off, group_size, opts)``

    logits [T, V] (bf16 or fp32, on the GPU); ``opts`` is a dict of the keyword options of ``grpo_loss_fwd_bwd``
    (prox_logp, norm, k, eps_low, eps_high, dual_clip_c, grad_scale, n_groups_total, aux, stream) plus
    ``upstream`` (above).  dlogits are formed in the same pass over the logits as the loss when ``logits``
    requires grad.
    """

    @staticmethod
    def forward(ctx, logits, actions, behave_logp, adv, step_tok_off, traj_step_off, group_size, opts=None):
        opts = dict(opts or {})
        ctx.upstream = _upstream(opts)
        want = bool(ctx.needs_input_grad[0])
        loss, dlogits = grpo_loss_fwd_bwd(logits.detach(), actions, behave_logp, adv, step_tok_off, traj_step_off,
                                          group_size, dlogits=want, **opts)
        ctx.save_for_backward(dlogits if want else None)
        return loss.view(())

    @staticmethod
    def backward(ctx, grad_output):
        (dlogits,) = ctx.saved_tensors
        (dlogits,) = _apply_upstream(ctx.upstream, (dlogits,), grad_output)
        return dlogits, None, None, None, None, None, None, None


class FusedLmHeadGrpoLoss(torch.autograd.Function):
    """``loss = FusedLmHeadGrpoLoss.apply(hidden, w_lm, actions, behave_logp, adv, step_tok_off, traj_step_off,
    group_size, opts)``

    hidden [T, H] and w_lm [H, V], bf16 on the GPU.  ``opts``: the keyword options of ``fused_lmhead_grpo_blocked``
    (token_block, aux_stream, ...), or with ``schedule="chunked"`` those of ``fused_lmhead_grpo`` (vocab_chunk, ...),
    plus ``upstream`` (above).  dhidden and dW come from the same call as the loss.  The library's dW is fp32;
    autograd needs the gradient in w_lm's dtype, so it is rounded to bf16 here (call the entry point directly to
    keep the fp32 dW).
    """

    @staticmethod
    def forward(ctx, hidden, w_lm, actions, behave_logp, adv, step_tok_off, traj_step_off, group_size, opts=None):
        opts = dict(opts or {})
        ctx.upstream = _upstream(opts)
        entry = fused_lmhead_grpo if opts.pop("schedule", "blocked") == "chunked" else fused_lmhead_grpo_blocked
        loss, dhidden, dw = entry(hidden.detach(), w_lm.detach(), actions, behave_logp, adv, step_tok_off,
                                  traj_step_off, group_size, **opts)
        ctx.save_for_backward(dhidden, dw)
        return loss.view(())

    @staticmethod
    def backward(ctx, grad_output):
        dhidden, dw = ctx.saved_tensors
        dh = dW = None
        if ctx.needs_input_grad[0]:
            (dh,) = _apply_upstream(ctx.upstream, (dhidden,), grad_output)
        if ctx.needs_input_grad[1]:  # w_lm is bf16 (the entry points take nothing else)
            if ctx.upstream == "scale" and dw.numel() >= _ONE_PASS_MIN:
                dW = _scaled_to_bf16(dw, grad_output)
            else:
                dW = _apply_upstream(ctx.upstream, (dw,), grad_output)[0].to(torch.bfloat16)
        return dh, dW, None, None, None, None, None, None, None
