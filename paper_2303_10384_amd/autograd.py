"""torch.autograd wrapper: the forward call computes the losses and the row records of the
gradient, backward streams the gradient once with the upstream gradient as a factor.

The forward call used to write the gradient and backward to scale it: up to three more
passes over a tensor of the logits' size (bf16 logits, B=32, T=250, U=80, V=1025, forward
and backward: 2.73 ms so, 0.51 ms now).  The logits are saved for backward, so, as with any
operation that saves its input, changing them in place between the two is an error.
"""
import torch

from .binding import rnnt_loss, step_forward, step_gradient


class _RNNTLossFunction(torch.autograd.Function):
    @staticmethod
    def forward(ctx, logits, labels, logit_lens, label_lens, blank, variant, reduction):
        ctx.reduction = reduction
        ctx.blank = blank
        if logits.requires_grad:
            loss, rows = step_forward(logits, labels, logit_lens, label_lens, blank, variant)
            ctx.save_for_backward(logits, rows)
        else:
            loss, _ = rnnt_loss(logits, labels, logit_lens, label_lens, blank=blank, variant=variant, need_grad=False)
        ctx.batch = loss.shape[0]
        if reduction == "sum":
            return loss.sum()
        if reduction == "mean":
            return loss.mean()
        return loss

    @staticmethod
    def backward(ctx, grad_loss):
        logits, rows = ctx.saved_tensors
        scale = grad_loss.to(torch.float32)
        if torch.is_grad_enabled():  # create_graph: the product with the upstream gradient is recorded
            g = step_gradient(logits.detach(), rows, ctx.blank)
            if ctx.reduction == "none":
                scale = scale.view(-1, 1, 1, 1)
            elif ctx.reduction == "mean":
                scale = scale / ctx.batch
            g = (g.to(torch.float32) * scale).to(g.dtype)
        else:
            g = step_gradient(logits, rows, ctx.blank, scale.contiguous(),
                              ctx.batch if ctx.reduction == "mean" else 1)
        return g, None, None, None, None, None, None


def rnnt_loss_autograd(logits, labels, logit_lens, label_lens, blank=0, variant="rnnt", reduction="mean"):
    """Differentiable RNN-T / W-RNNT loss; reduction in {"none", "sum", "mean"}."""
    if reduction not in ("none", "sum", "mean"):
        raise ValueError("reduction must be none, sum or mean")
    return _RNNTLossFunction.apply(logits, labels, logit_lens, label_lens, blank, variant, reduction)


class RNNTLoss(torch.nn.Module):
    def __init__(self, blank=0, variant="rnnt", reduction="mean"):
        super().__init__()
        self.blank, self.variant, self.reduction = blank, variant, reduction

    def forward(self, logits, labels, logit_lens, label_lens):
        return rnnt_loss_autograd(logits, labels, logit_lens, label_lens, self.blank, self.variant, self.reduction)
