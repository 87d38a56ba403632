"""torch.autograd entry points over the binding, so that the fused objective (Sec. 3.2.2) can sit in
a training script where a log-softmax / gather / clipped-ratio chain would otherwise be:

    loss = ulorl.autograd.token_loss(logits, token_ids, cu_seqlens, advantages, old_logp, params)
    loss.backward()                     # logits.grad holds dlogits

Every function forwards tensors to the library calls and hands their results to autograd (the two-call nodes are
native, in ``csrc/torch_marshal.cpp``: backward runs on autograd's device thread, where Python cost 50 us a
call); the one thing computed there is the product of the saved coefficients and the upstream gradient.
There is no CPU path.

Two ways to run the logits path:
  * ``fused=False`` (default): ``ulorl_token_loss_fwd`` in forward, ``ulorl_token_loss_bwd`` in
    backward with the upstream gradient as ``grad_out``.  Any upstream scale is honoured.
  * ``fused=True``: ``ulorl_token_loss_fwd_bwd`` in forward (the logits are read once and the
    gradient of an upstream 1 is written in the same pass); backward hands that gradient out and
    refuses any other upstream gradient.  ``in_place=True`` lets the gradient overwrite ``logits``.

The upstream gradient is a 0-dim device tensor, and ``grad_out`` a host scalar of the C ABI.  The two-call
paths multiply it into the saved coefficients on the device (one small launch, the same fp32 product the
kernels form) instead of reading it back, which left the GPU idle for about 50 us per backward; only
``fused=True`` reads it (``float()``), to refuse anything but 1.
"""
from typing import Optional

import torch

from . import binding
from .binding import FwdResult, Launch, Params


class _FusedTokenLoss(torch.autograd.Function):
    @staticmethod
    def forward(ctx, logits, token_ids, cu_seqlens, advantages, old_logp, params, segment_ids, in_place, launch, sink):
        res, ctx.dlogits = binding.token_loss_fwd_bwd(logits, token_ids, cu_seqlens, advantages, old_logp, params,
                                                      segment_ids=segment_ids, grad_out=1.0, inplace=bool(in_place),
                                                      launch=launch)
        if sink is not None:
            sink.append(res)
        return res.loss.reshape(())

    @staticmethod
    def backward(ctx, grad_loss):
        g = float(grad_loss)
        if g != 1.0:
            raise RuntimeError("token_loss(fused=True) computed the gradient of an upstream 1 in its forward pass; "
                               "got an upstream gradient of %r: scale through Params.denominator or use fused=False" % g)
        d = ctx.dlogits
        ctx.dlogits = None
        return (d,) + (None,) * 9


def token_loss(logits: torch.Tensor, token_ids, cu_seqlens, advantages, old_logp=None, params: Optional[Params] = None,
               segment_ids=None, fused: bool = False, in_place: bool = False, launch: Optional[Launch] = None,
               results: Optional[list] = None) -> torch.Tensor:
    """The masked, clipped policy-gradient loss of Sec. 3.2.2 as a differentiable 0-dim tensor (gradient
    to ``logits`` only).  ``results``: a list that receives the call's ``FwdResult`` (per-token
    log-probs, entropies, mask, ratio, counters)."""
    if fused:
        return _FusedTokenLoss.apply(logits, token_ids, cu_seqlens, advantages, old_logp, params, segment_ids, in_place, launch,
                                     results)
    if in_place:
        raise ValueError("in_place needs fused=True (the two-call path reads the logits again in backward)")
    with_params, with_launch = binding._structs(params, launch)
    loss, fields = binding.native().autograd_token_loss(logits, token_ids, cu_seqlens, advantages, old_logp, segment_ids,
                                                        binding._addr(with_params), binding._addr(with_launch), results is not None)
    if results is not None:
        results.append(FwdResult(*fields))
    return loss


def lmhead_token_loss(hidden: torch.Tensor, weight: torch.Tensor, token_ids, cu_seqlens, advantages, old_logp=None,
                      params: Optional[Params] = None, segment_ids=None, vocab_chunk: int = 8192,
                      launch: Optional[Launch] = None, results: Optional[list] = None) -> torch.Tensor:
    """The same loss from the last hidden states and the lm_head weight [hidden, vocabulary], the
    logits never materialised; gradients to ``hidden`` and ``weight`` (both computed, bf16)."""
    with_params, with_launch = binding._structs(params, launch)
    loss, fields = binding.native().autograd_lmhead(hidden, weight, token_ids, cu_seqlens, advantages, old_logp, segment_ids,
                                                    binding._addr(with_params), binding._addr(with_launch), vocab_chunk,
                                                    results is not None)
    if results is not None:
        results.append(FwdResult(*fields))
    return loss


__all__ = ["token_loss", "lmhead_token_loss", "FwdResult"]
