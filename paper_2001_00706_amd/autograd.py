"""`signature` and `logsignature` as differentiable PyTorch operations (paper section 5.3): the forward passes
are `sig_signature`, `sig_log` and `sig_lyndon_gather`, the backward passes `sig_lyndon_scatter`,
`sig_log_backward` and `sig_backward` (`sig_backward_chunked` for few long paths); all run in the HIP library.  Glue only.

Plain calls go through the same glue in C++ (`torch_node/sig_torch.cpp`), where the host is not what a small call waits for (forward
and gradient, queued: 128 x 128 points, d = 4, N = 5, fp64: 65 or 103 us a pass through the functions below, by where the autograd
engine's thread runs); it hands back what it does not take, and what the library refuses, and the functions below serve that."""
from __future__ import annotations

import warnings

import torch

from . import binding

try:
    from ._sig_torch import built_with, interval as _interval, transform as _transform
    if built_with != torch.__version__:   # the node reaches into torch's own structures
        raise ImportError(f"built against torch {built_with}, this is {torch.__version__}")
except ImportError as e:
    warnings.warn(f"_sig_torch.so does not load ({e}); calls go through slower Python functions.  Build it with "
                  "`python -c 'import __graft_entry__ as g; g.build()'`", RuntimeWarning)

    def _transform(*args):
        return NotImplemented

    _interval = _transform


def _plain_signature(path, basepoint_value, depth, stream, basepoint):
    """The signature itself; `path` contiguous."""
    bp = basepoint_value.contiguous() if basepoint_value is not None else bool(basepoint)
    B, L, d = path.shape
    chunks = 1 if stream else binding.sig_forward_chunks_hint(B, L, d, depth, bool(basepoint), binding._dtype_of(path))
    if chunks > 1:   # few long paths: the scan as a reduction over the length (section 5.1)
        return binding.sig_forward_chunked(path, depth, chunks, basepoint=bp)
    return binding.sig_signature(path, depth, stream=stream, basepoint=bp)


def _signature_gradients(path, plain, basepoint_value, grad_out, args):
    """Gradients with respect to the path and the basepoint, from that with respect to the operation's output."""
    depth, stream, basepoint, inverse, d = args
    grad_out = grad_out.contiguous()
    if inverse:
        # the inverse is a signed permutation that is its own transpose
        grad_out = binding.sig_invert(grad_out, d, depth)
    bp = basepoint_value.contiguous() if basepoint_value is not None else bool(basepoint)
    grad_bp = (torch.empty_like(basepoint_value, memory_format=torch.contiguous_format) if basepoint_value is not None
               else None)   # not with the strides of a basepoint that is a transposed view
    B, L, _ = path.shape
    chunks = 1 if stream else binding.sig_backward_chunks_fastest(B, L, d, depth, bool(basepoint), binding._dtype_of(path))
    grad_path = None
    while chunks > 1 and grad_path is None:   # few long paths: the walk back along the path cut into stretches
        try:
            grad_path = binding.sig_backward_chunked(path, grad_out, depth, chunks, basepoint=bp, grad_basepoint=grad_bp)
        except torch.OutOfMemoryError:   # every stretch takes memory: with fewer it may do
            fewer = binding.sig_backward_chunks_hint(B, L, d, depth, bool(basepoint), binding._dtype_of(path))
            chunks = fewer if fewer < chunks else 1
    if grad_path is None:
        scanned = stream or binding.sig_forward_chunks_hint(B, L, d, depth, bool(basepoint), binding._dtype_of(path)) <= 1   # by _plain_signature
        grad_path = binding.sig_backward(path, plain, grad_out, depth, stream=stream, basepoint=bp,
                                         grad_basepoint=grad_bp, scanned=scanned)
    return grad_path, grad_bp


def _log_of(sig, channels, depth, mode):
    return binding.sig_log(sig, channels, depth) if mode == "expand" else binding.sig_log_words(sig, channels, depth)


def _log_gradient(sig, grad_out, channels, depth, mode):
    grad_out = grad_out.contiguous()
    grad_log = grad_out if mode == "expand" else binding.sig_lyndon_scatter(grad_out, channels, depth)
    return binding.sig_log_backward(sig, grad_log, channels, depth)


class _Signature(torch.autograd.Function):
    @staticmethod
    def forward(ctx, path, basepoint_value, depth, stream, basepoint, inverse):
        path = path.contiguous()
        plain = _plain_signature(path, basepoint_value, depth, stream, basepoint)
        d = path.shape[2]
        out = binding.sig_invert(plain, d, depth) if inverse else plain
        ctx.save_for_backward(path, plain, basepoint_value)
        ctx.args = (depth, stream, basepoint, inverse, d)
        return out

    @staticmethod
    def backward(ctx, grad_out):
        path, plain, basepoint_value = ctx.saved_tensors
        return (*_signature_gradients(path, plain, basepoint_value, grad_out, ctx.args), None, None, None, None)


class _Logsignature(torch.autograd.Function):
    """`_Signature` and `_SignatureToLogsignature` as one node: every node costs the autograd engine 10 to 20 us a pass."""

    @staticmethod
    def forward(ctx, path, basepoint_value, depth, stream, basepoint, inverse, mode):
        path = path.contiguous()
        plain = _plain_signature(path, basepoint_value, depth, stream, basepoint)
        d = path.shape[2]
        sig = binding.sig_invert(plain, d, depth) if inverse else None   # None: the plain one
        ctx.save_for_backward(path, plain, basepoint_value, sig)
        ctx.args = (depth, stream, basepoint, inverse, d)
        ctx.mode = mode
        return _log_of(plain if sig is None else sig, d, depth, mode)

    @staticmethod
    def backward(ctx, grad_out):
        path, plain, basepoint_value, sig = ctx.saved_tensors
        depth, _, _, _, d = ctx.args
        grad_sig = _log_gradient(plain if sig is None else sig, grad_out, d, depth, ctx.mode)
        return (*_signature_gradients(path, plain, basepoint_value, grad_sig, ctx.args), None, None, None, None, None)


class _Combine(torch.autograd.Function):
    @staticmethod
    def forward(ctx, a, b, channels, depth):
        a, b = a.contiguous(), b.contiguous()
        ctx.save_for_backward(a, b)
        ctx.args = (channels, depth)
        return binding.sig_combine(a, b, channels, depth)

    @staticmethod
    def backward(ctx, grad_out):
        a, b = ctx.saved_tensors
        channels, depth = ctx.args
        grad_a, grad_b = binding.sig_combine_backward(a, b, grad_out.contiguous(), channels, depth)
        return grad_a, grad_b, None, None


class _CombineGrouped(torch.autograd.Function):
    @staticmethod
    def forward(ctx, a, sigs, channels, depth):
        a, sigs = a.contiguous(), sigs.contiguous()
        ctx.save_for_backward(a, sigs)
        ctx.args = (channels, depth)
        return binding.sig_combine_grouped(a, sigs, channels, depth)

    @staticmethod
    def backward(ctx, grad_out):
        a, sigs = ctx.saved_tensors
        channels, depth = ctx.args
        grad_a, grad_sigs = binding.sig_combine_grouped_backward(a, sigs, grad_out.contiguous(), channels, depth)
        return grad_a, grad_sigs, None, None


def signature_combine(sig1, sig2, channels: int, depth: int):
    """Group product `sig1 [x] sig2` of two batches of signatures `[B, S]` (section 5.5, "combining adjacent
    intervals"), differentiable in both."""
    return _Combine.apply(sig1, sig2, int(channels), int(depth))


def multi_signature_combine(sigs, channels: int, depth: int):
    """Ordered product of a list of batches of signatures `[B, S]`, differentiable in each: neighbours are joined
    pairwise, in ceil(log2 n) rounds of products (the product is associative)."""
    sigs = list(sigs)
    if not sigs:
        raise ValueError("at least one signature is needed")
    while len(sigs) > 1:
        joined = [signature_combine(sigs[i], sigs[i + 1], channels, depth) for i in range(0, len(sigs) - 1, 2)]
        if len(sigs) % 2:
            joined.append(sigs[-1])
        sigs = joined
    return sigs[0]


def signature(path, depth: int, stream: bool = False, basepoint=False, inverse: bool = False, initial=None):
    """Depth-`depth` signature of a batch of paths `[B, L, d]` on the GPU, differentiable in `path`,
    in `basepoint` when that is a `[B, d]` tensor, and in `initial` (argument names as in section 5.5).

    `initial` `[B, S]` is the signature of the data that came before; the result is `initial [x] Sig(path)`, in
    stream mode for every prefix (inverted as a whole if `inverse`).

    The gradient of few long paths is computed in stretches and takes up to 2 GiB besides its result while it runs, less
    where that much cannot be had (`sig_backward_chunks_fastest`, then `sig_backward_chunks_hint`, then none)."""
    if initial is None and not torch.compiler.is_compiling():
        out = _transform(path, depth, stream, basepoint, inverse, 0, None)
        if out is not NotImplemented:
            return out
    value = basepoint if isinstance(basepoint, torch.Tensor) else None
    flag = value is not None or bool(basepoint)
    if initial is None:
        return _Signature.apply(path, value, int(depth), bool(stream), flag, bool(inverse))
    d = path.shape[2]
    needs_grad = torch.is_grad_enabled() and any(t is not None and t.requires_grad for t in (path, value, initial))
    if not needs_grad:   # one call, `initial` applied in place behind the scan
        bp = value.contiguous() if value is not None else flag
        return binding.sig_signature(path.contiguous(), int(depth), stream=bool(stream), basepoint=bp, inverse=bool(inverse),
                                     initial=initial.contiguous())
    plain = _Signature.apply(path, value, int(depth), bool(stream), flag, False)
    if stream:
        joined = _CombineGrouped.apply(initial, plain, d, int(depth))
    else:
        joined = signature_combine(initial, plain, d, depth)
    return _Invert.apply(joined, d, int(depth)) if inverse else joined


class _Invert(torch.autograd.Function):
    @staticmethod
    def forward(ctx, sig, channels, depth):
        ctx.args = (channels, depth)
        return binding.sig_invert(sig.contiguous(), channels, depth)

    @staticmethod
    def backward(ctx, grad_out):
        # only used on signatures (group-like elements), where the inverse is a signed permutation of the scalars
        # (section 5.4) and therefore its own transpose
        channels, depth = ctx.args
        return binding.sig_invert(grad_out.contiguous(), channels, depth), None, None


class _SignatureToLogsignature(torch.autograd.Function):
    @staticmethod
    def forward(ctx, sig, channels, depth, mode):
        sig = sig.contiguous()
        ctx.save_for_backward(sig)
        ctx.args = (channels, depth, mode)
        return _log_of(sig, channels, depth, mode)

    @staticmethod
    def backward(ctx, grad_out):
        (sig,) = ctx.saved_tensors
        return _log_gradient(sig, grad_out, *ctx.args), None, None, None


def signature_to_logsignature(sig, channels: int, depth: int, mode: str = "words"):
    """Logsignature from signatures `[..., S]` (sections 2.3, 4.3), differentiable in `sig`: the logarithm, then for
    mode "words" the coefficients of the Lyndon words (appendix A.2.4); mode "expand" keeps every word."""
    if mode not in ("words", "expand"):
        raise ValueError('mode must be "words" or "expand"')
    return _SignatureToLogsignature.apply(sig, int(channels), int(depth), mode)


def logsignature(path, depth: int, stream: bool = False, basepoint=False, inverse: bool = False, mode: str = "words"):
    """Depth-`depth` logsignature of a batch of paths `[B, L, d]` on the GPU, differentiable in `path` (and in a
    tensor `basepoint`)."""
    if mode not in ("words", "expand"):
        raise ValueError('mode must be "words" or "expand"')
    if type(depth) is int and isinstance(path, torch.Tensor) and path.dim() == 3 and not torch.compiler.is_compiling():
        # kept since the first call; beyond the depths of sig_log_words, which the node would find out behind the scan, not asked for
        words = mode == "words" and depth <= binding._LOG_WORDS_MAX_DEPTH
        table = binding._lyndon_tables.get((path.shape[2], depth, path.device)) if words else None
        if mode == "expand" or table is not None:
            out = _transform(path, depth, stream, basepoint, inverse, 1 if mode == "expand" else 2, table)
            if out is not NotImplemented:
                return out
    value = basepoint if isinstance(basepoint, torch.Tensor) else None
    return _Logsignature.apply(path, value, int(depth), bool(stream), value is not None or bool(basepoint), bool(inverse), mode)
