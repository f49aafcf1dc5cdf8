"""Drop-in PyTorch layers over the C ABI (the way the paper ships its kernels: App. F).

Only what is stashed for backward differs from the stock layers:
  InplaceGELU        keeps the output (which the next Linear keeps anyway) and a 1-bit mask
  InplaceSiLU        the same for SiLU (Sec. 5.1)
  InplaceLayerNorm   keeps the output and one float per row
  TempoAttentionCore softmax -> dropout -> (. @ V) keeping the softmax output P and a 1-bit
                     mask; the dropout output is a transient in forward and is recomputed by
                     the backward kernel for the gradient of V (Sec. 3.3).
  TempoEncoderLayer  an encoder layer of the three: in float32 one native call each way on HIP
                     kernels alone where nothing else can see its parts, else those parts
Every arithmetic step of the three layers runs in the HIP kernels; the matrix products around
them, where the layer is made of its parts, are ordinary library GEMMs (torch.matmul, nn.Linear).
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F
from torch import nn
from torch.autograd import forward_ad
from torch.nn.modules import linear, module

from . import binding as B


def _words(n: int, device) -> torch.Tensor:
    return torch.empty(B.mask_words(n), dtype=torch.int32, device=device)


# `made`, in the three functions below: what the forward has already made, which is then not run (x and scores give only their
# place in the graph).

class _InplaceGELUFn(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, kind, made):
        if made is None:
            x = x.contiguous()
            y = torch.empty_like(x)
            mask = _words(x.numel(), x.device)
            if kind == "silu":
                B.tempo_silu_fwd(x, y, mask)
            else:
                B.tempo_gelu_fwd(x, y, mask, kind)
        else:
            y, mask = made[0].detach(), made[1]
        ctx.kind = kind
        ctx.save_for_backward(y, mask)
        return y

    @staticmethod
    def backward(ctx, dy):
        y, mask = ctx.saved_tensors
        dy = dy.contiguous()
        dx = torch.empty_like(dy)
        if ctx.kind == "silu":
            B.tempo_silu_bwd(dy, y, mask, dx)
        else:
            B.tempo_gelu_bwd(dy, y, mask, dx, ctx.kind)
        return dx, None, None


class InplaceGELU(nn.Module):
    """GELU whose backward needs the output and one bit per element (Sec. 3.1)."""

    def __init__(self, approximate: str = "none"):
        super().__init__()
        self.kind = {"none": "erf", "tanh": "tanh"}[approximate]

    def forward(self, x):
        return _InplaceGELUFn.apply(x, self.kind, None)


class InplaceSiLU(nn.Module):
    """SiLU with the same stash as InplaceGELU: the in-place recipe for elementwise layers
    (Sec. 5.1) on another activation with a single minimum."""

    def forward(self, x):
        return _InplaceGELUFn.apply(x, "silu", None)


class _InplaceLayerNormFn(torch.autograd.Function):
    @staticmethod
    def forward(ctx, x, gamma, beta, eps, made):
        if made is None:
            x = x.contiguous()
            M = x.shape[-1]
            N = x.numel() // M
            y = torch.empty_like(x)
            rstd = torch.empty(N, dtype=torch.float32, device=x.device)
            B.tempo_layernorm_fwd(x, gamma, beta, y, rstd, None, eps)
        else:
            y, rstd = made[0].detach(), made[1]
        ctx.save_for_backward(y, gamma, beta, rstd)
        return y

    @staticmethod
    def backward(ctx, dy):
        y, gamma, beta, rstd = ctx.saved_tensors
        dy = dy.contiguous()
        M = y.shape[-1]
        N = y.numel() // M
        dx = torch.empty_like(dy)
        dgamma = torch.empty_like(gamma)
        dbeta = torch.empty_like(beta)
        ws = torch.empty(B.tempo_layernorm_bwd_workspace_bytes(N, M), dtype=torch.uint8,
                         device=y.device)
        B.tempo_layernorm_bwd(dy, y, gamma, beta, rstd, dx, dgamma, dbeta, ws)
        return dx, dgamma, dbeta, None, None


class InplaceLayerNorm(nn.Module):
    """LayerNorm over the last dimension whose backward needs the output and rstd (Sec. 3.2).
    Parameters are float32 whatever the activation dtype; gamma must stay non-zero."""

    def __init__(self, hidden: int, eps: float = 1e-5):
        super().__init__()
        self.weight = nn.Parameter(torch.ones(hidden, dtype=torch.float32))
        self.bias = nn.Parameter(torch.zeros(hidden, dtype=torch.float32))
        self.eps = eps

    def _apply(self, fn, recurse=True):
        # .bfloat16() / .half() / .to(dtype) on a model must not narrow gamma and beta: the
        # kernels read them as float32.  Follow the device of the cast, keep the values.
        def keep_float32(t):
            out = fn(t)
            if t.dtype == torch.float32 and out.dtype != torch.float32:
                out = t.to(device=out.device)
            return out
        return super()._apply(keep_float32, recurse)

    def forward(self, x):
        w, b = self.weight, self.bias
        if w.dtype != torch.float32 or b.dtype != torch.float32:   # parameters replaced by hand
            w, b = w.float(), b.float()
        return _InplaceLayerNormFn.apply(x, w, b, self.eps, None)


class _AttentionCoreFn(torch.autograd.Function):
    @staticmethod
    def forward(ctx, scores, v, key_len, causal, p, seed, offset, store_mask, made):
        if made is None:
            scores = scores.contiguous()
            probs = torch.empty_like(scores)
            out = torch.empty_like(scores)      # transient: freed when forward returns
            keep = _words(scores.numel(), scores.device)
            B.tempo_attn_softmax_dropout_fwd(scores, key_len, causal, probs, out, keep, p, seed, offset)
        else:
            probs, keep = made[:2]
        ctx.rng = (p, seed, offset)
        ctx.store_mask = store_mask
        if store_mask:
            ctx.save_for_backward(probs, v, keep)
        else:                                   # the mask is a transient too: drawn again later
            ctx.save_for_backward(probs, v)
        return torch.matmul(out, v) if made is None else made[2].detach()

    @staticmethod
    def backward(ctx, dctx):
        probs, v = ctx.saved_tensors[:2]
        dout = torch.matmul(dctx, v.transpose(-1, -2)).contiguous()
        out_re = torch.empty_like(probs)
        dscores = torch.empty_like(probs)
        p, seed, offset = ctx.rng
        if ctx.store_mask:
            B.tempo_attn_softmax_dropout_bwd(dout, probs, ctx.saved_tensors[2], dscores, out_re, p)
        else:
            B.tempo_attn_softmax_dropout_bwd_regen(dout, probs, dscores, out_re, p, seed, offset)
        dv = torch.matmul(out_re.transpose(-1, -2), dctx)
        return (dscores, dv) + (None,) * 7


class TempoAttentionCore(nn.Module):
    """context = dropout(softmax(mask(scores))) @ V for scores [B, A, Sq, Sk] already scaled by
    1/sqrt(d).  Each forward in training mode draws a fresh mask: the counter offset advances.
    store_mask=False keeps no mask for backward, which then draws the same bits again."""

    def __init__(self, p: float = 0.1, seed: int = 0x5EED, store_mask: bool = True):
        super().__init__()
        self.p, self.seed, self.offset, self.store_mask = p, seed, 0, store_mask

    def forward(self, scores, v, key_len=None, causal=False):
        p = self.p if self.training else 0.0
        self.offset += 1
        return _AttentionCoreFn.apply(scores, v, key_len, causal, p, self.seed, self.offset,
                                      self.store_mask, None)


class _EncoderLayerFn(torch.autograd.Function):
    """The whole layer, whose forward has been made (_native.tempo_encoder_fwd): keeps what the layer's parts keep for the
    inputs that require a gradient.  The backward is one native call too."""

    @staticmethod
    def forward(ctx, made, setting, store_mask, x, *params):
        qkv, probs, keep, ctxt, y1, rstd1, h, side, y2, rstd2, place = made
        wqkv, bqkv, wproj, bproj, w1, b1, w2, b2, gamma1, beta1, gamma2, beta2 = params
        # where _grads_of_parts() finds the inputs' graphs: not kept for their values, which may change
        ctx.places = place, wqkv, bqkv, wproj, bproj, w1, b1, w2, b2
        ctx.setting, ctx.store_mask = setting, store_mask
        of = ctx.needs_input_grad[3:]
        inner = of[0] or of[1] or of[2]                                        # the gradient goes on to qkv,
        first = inner or of[3] or of[4] or of[9] or of[10]                     # to the first LayerNorm,
        second = first or of[5] or of[6]                                       # to GELU
        ctx.save_for_backward(
            x if of[1] else None, wqkv if of[0] else None, wproj if inner else None, w1 if first else None,
            w2 if second else None, gamma1 if first else None, beta1 if first else None, gamma2, beta2,
            qkv if inner else None, probs if inner else None, keep if inner and store_mask else None, ctxt if of[3] else None,
            y1 if first or of[5] else None, rstd1 if first else None, h if second or of[7] else None,
            side if second else None, y2, rstd2)
        return y2

    @staticmethod
    def backward(ctx, dy):
        needed = ctx.needs_input_grad[3:]
        grads = None
        if not torch.is_grad_enabled():
            wanted = sum(1 << i for i, n in enumerate(needed) if n)
            grads = B.encoder_bwd(dy.contiguous(), wanted, *ctx.setting, *ctx.saved_tensors)
        if grads is None:     # create_graph, or a tensor that is no plain one any more: the gradients of the parts
            grads = _grads_of_parts(ctx, dy, needed)
        return (None,) * 3 + grads


class _PlaceFn(torch.autograd.Function):
    """x's place in its graph, without its values; nothing looks at those it has."""

    @staticmethod
    def forward(ctx, x):
        return x.new_empty(()).expand(x.shape)

    @staticmethod
    def backward(ctx, dx):
        return dx


class _MadeLinearFn(torch.autograd.Function):
    """y = x w^T + b, already made."""

    @staticmethod
    def forward(ctx, y, x, w, b):
        ctx.save_for_backward(x, w)
        return y.detach()

    @staticmethod
    def backward(ctx, dy):
        x, w = ctx.saved_tensors
        rows = dy.reshape(-1, dy.shape[-1])
        dx = torch.matmul(dy, w) if ctx.needs_input_grad[1] else None
        dw = torch.matmul(rows.t(), x.reshape(-1, x.shape[-1])) if ctx.needs_input_grad[2] else None
        return None, dx, dw, rows.sum(0) if ctx.needs_input_grad[3] else None


class _MadeScoresFn(torch.autograd.Function):
    """scale q k^T of every head, already made; only its place in the graph is needed."""

    @staticmethod
    def forward(ctx, scores, q, k, scale):
        ctx.scale = scale
        ctx.save_for_backward(q, k)
        return scores.detach()

    @staticmethod
    def backward(ctx, ds):
        q, k = ctx.saved_tensors
        ds = ds * ctx.scale
        return None, torch.matmul(ds, k), torch.matmul(ds.transpose(-1, -2), q), None


def _grads_of_parts(ctx, dy, needed):
    """The gradients as the layer made of its parts gives them, connected to its inputs under create_graph.  The graph of the
    parts is laid over what the forward made: nothing of the forward runs again, and only what was kept is looked at."""
    heads, ffn, p, seed, offset, kind = ctx.setting
    x, wqkv, wproj, w1, w2, g1, be1, g2, be2, qkv, probs, keep, ctxt, y1, rstd1, h, side, y2, rstd2 = ctx.saved_tensors
    Bn, S, H = dy.shape
    d = H // heads

    def value(t, *shape):     # t in that shape; zeros without memory in the place of what nothing looks at
        return dy.new_zeros(()).expand(shape) if t is None else t.reshape(shape)
    with torch.enable_grad():
        # Aliases, which are inputs of this graph alone: x may depend on these parameters, and two of them may be the same
        # tensor, whose gradients the caller's backward adds up.
        kept, places = (x, wqkv, None, wproj, None, w1, None, w2, None), ctx.places
        inputs = [t.view_as(t) if t is not None else None
                  for t in (*(p if k is None else k for k, p in zip(kept, places)), g1, be1, g2, be2)]
        x, wqkv, bqkv, wproj, bproj, w1, b1, w2, b2, g1, be1, g2, be2 = inputs

        def core(q, k, v):
            scores = _MadeScoresFn.apply(value(None, Bn, heads, S, S), q, k, 1.0 / math.sqrt(d))
            made = (probs, keep, value(ctxt, Bn, S, heads, d).permute(0, 2, 1, 3))
            return _AttentionCoreFn.apply(scores, v, None, False, p, seed, offset, ctx.store_mask, made)

        rows = value(None, Bn, S, H)
        x, g1, be1 = (value(t, *shape) for t, shape in ((x, (Bn, S, H)), (g1, (H,)), (be1, (H,))))
        a = _attention(_MadeLinearFn.apply(value(qkv, Bn, S, 3 * H), x, wqkv, bqkv), dy.shape, heads, core)
        y1 = _InplaceLayerNormFn.apply(x + _MadeLinearFn.apply(rows, a, wproj, bproj), g1, be1, None,
                                       (value(y1, Bn, S, H), rstd1))
        h = _InplaceGELUFn.apply(_MadeLinearFn.apply(value(None, Bn, S, ffn), y1, w1, b1), kind, (value(h, Bn, S, ffn), side))
        out = _InplaceLayerNormFn.apply(y1 + _MadeLinearFn.apply(rows, h, w2, b2), g2, be2, None, (y2, rstd2))
    grads = iter(torch.autograd.grad(out, [t for t, n in zip(inputs, needed) if n], dy, create_graph=torch.is_grad_enabled()))
    return tuple(next(grads) if n else None for n in needed)


def _attention(qkv, shape, heads, core):
    Bn, S, H = shape
    q, k, v = qkv.view(Bn, S, 3, heads, H // heads).permute(2, 0, 3, 1, 4)
    return core(q, k, v.contiguous()).permute(0, 2, 1, 3).reshape(Bn, S, H)


class TempoEncoderLayer(nn.Module):
    """A post-LN BERT encoder layer built from the three memory-reduced layers (Fig. 1 of the
    paper); hidden-state dropouts are left out (they are not part of the method)."""

    def __init__(self, hidden: int, heads: int, ffn: int, p_attn: float = 0.1, eps: float = 1e-12,
                 dtype=torch.float32):
        super().__init__()
        self.heads = heads
        self.qkv = nn.Linear(hidden, 3 * hidden, dtype=dtype)
        self.proj = nn.Linear(hidden, hidden, dtype=dtype)
        self.fc1 = nn.Linear(hidden, ffn, dtype=dtype)
        self.fc2 = nn.Linear(ffn, hidden, dtype=dtype)
        self.ln1 = InplaceLayerNorm(hidden, eps)
        self.ln2 = InplaceLayerNorm(hidden, eps)
        self.act = InplaceGELU()
        self.core = TempoAttentionCore(p_attn)

    def forward(self, x, key_len=None):
        out = self._as_one(x, key_len)
        if out is not None:
            return out

        def core(q, k, v):
            scores = torch.matmul(q, k.transpose(-1, -2)) * (1.0 / math.sqrt(q.shape[-1]))
            return self.core(scores, v, key_len)
        Bn, S, H = x.shape
        ctxt = _attention(self.qkv(x), (Bn, S, H), self.heads, core)
        x = self.ln1(x + self.proj(ctxt))
        return self.ln2(x + self.fc2(self.act(self.fc1(x))))

    def _as_one(self, x, key_len):
        """The layer as one native call each way, or None where something may see or change its parts: hooks, other
        modules in their places, a forward, a call or a product replaced, autocast, function transforms, tracing, dispatch
        and function modes, forward-mode AD, tensor subclasses, other types and layouts."""
        if torch.compiler.is_compiling():
            return None
        if not _plain(x):
            return None
        if (torch.is_autocast_enabled() or torch._C._len_torch_dispatch_stack() or torch._C._len_torch_function_stack()
                or torch._C._functorch.peek_interpreter_stack() is not None or forward_ad._current_level >= 0
                or torch.jit.is_tracing() or module._has_any_global_hook() or _calls() != _CALLS):
            return None
        parts = self._modules
        for name, kind in _PARTS:
            m = parts.get(name)
            if (type(m) is not kind or m._forward_hooks or m._forward_pre_hooks or m._backward_hooks
                    or m._backward_pre_hooks or "forward" in m.__dict__ or m._compiled_call_impl is not None):
                return None
        qkv, proj, fc1, fc2, ln1, ln2, core = (parts[n] for n in ("qkv", "proj", "fc1", "fc2", "ln1", "ln2", "core"))
        params = (qkv.weight, qkv.bias, proj.weight, proj.bias, fc1.weight, fc1.bias, fc2.weight, fc2.bias,
                  ln1.weight, ln1.bias, ln2.weight, ln2.bias)
        p, kind = core.p if core.training else 0.0, parts["act"].kind
        made = B.encoder_fwd(x, key_len, core.__dict__, self.heads, ln1.eps, ln2.eps, p, core.seed, kind, *params)
        if made is None:
            return None
        offset, *made = made
        if not torch.is_grad_enabled():
            return made[8]
        setting = (self.heads, fc1.weight.shape[0], p, core.seed, offset, kind)
        made.append(_PlaceFn.apply(x) if x.requires_grad and not qkv.weight.requires_grad else None)    # else x itself is kept
        return _EncoderLayerFn.apply(made, setting, core.store_mask, x, *params)


def _plain(x):
    if type(x) not in (torch.Tensor, nn.Parameter) or x.dtype != torch.float32 or not x.is_cuda:
        return False
    B.load()
    return B._native is not None


_PARTS = (("qkv", nn.Linear), ("proj", nn.Linear), ("fc1", nn.Linear), ("fc2", nn.Linear), ("ln1", InplaceLayerNorm),
          ("ln2", InplaceLayerNorm), ("act", InplaceGELU), ("core", TempoAttentionCore))


def _calls():
    """What a layer made of its parts goes through."""
    return (nn.Linear.forward, InplaceLayerNorm.forward, InplaceGELU.forward, TempoAttentionCore.forward, nn.Linear.__call__,
            InplaceLayerNorm.__call__, InplaceGELU.__call__, TempoAttentionCore.__call__, F.linear, torch.matmul)


_CALLS = _calls()                                # what the native call stands for
if _CALLS[0].__globals__ is not vars(linear) or _CALLS[4] is not nn.Module._wrapped_call_impl or F.linear is not torch._C._nn.linear:
    _CALLS = None                                # replaced before this module was loaded
