"""torch.autograd glue: `rnn_apply` runs pararnn_forward and registers pararnn_backward as its gradient, so
the library can sit inside a PyTorch training step.  The graph nodes are native (csrc/host_binding.cpp); no
arithmetic happens there: both directions run in the HIP kernels, on the current stream."""
from . import binding
from .binding import _host


def input_projection_apply(x, Wx, bias=None, n_heads: int = 1):
    """u = B x + b for all gates (multi-head input matrices), differentiable with respect to x, Wx
    and bias: pararnn_input_projection with pararnn_input_projection_backward as its gradient."""
    return _host.input_projection_apply(x, Wx, bias, n_heads)


def rnn_layer(cell, x, Wx, bias, params, h0=None, n_heads: int = 1, tol: float = 1e-6, max_iter: int = 64):
    """The paper's cell applied to a sequence: the input projection followed by the Newton solve of
    the recurrence, differentiable end to end (one node).  Returns (h, iters)."""
    return _host.rnn_layer(binding._api(cell).host, x, Wx, bias, params, h0, n_heads, tol, max_iter)


def rnn_apply(cell: str, params, u, h0=None, tol: float = 1e-6, max_iter: int = 64):
    """h = RNN(u) by the Newton solve, differentiable with respect to params, u
    and h0 (Eq. (6)).  Returns (h, iters); iters is the device int32[2] tensor
    {iterations, status} of pararnn_forward."""
    return _host.rnn_apply(binding._api(cell).host, params, u, h0, tol, max_iter)
