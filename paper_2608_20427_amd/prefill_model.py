"""Whole-model prefill of the paper's timing study (§4.3, §5.3) on one GPU.

A decoder stack of the evaluated geometry (Qwen3-0.6B: 28 layers, 16 query
heads, 8 kv-heads, head dimension 128, §4.1) whose attention layers run this
library's kernels: bf1_attn_fwd on the BF1 route for the chosen layers, the
in-house dense causal kernel (bf1_dense_causal_fwd) for the others.  The
projections around them are library GEMMs; the norms with their residual adds,
the per-head norm with the rotary embedding and the SwiGLU product between
them are one HIP kernel each (plain PyTorch operators with the same rounding
where those kernels do not apply).  The study measures the time to first token (the
last position's logits) with no, the middle eight, or all layers on the BF1
route.  The trained weights are not available: callers pass seeded random
weights of the published shapes (timing does not depend on their values).
"""

import contextlib

import torch
from torch.autograd import forward_ad
from torch.utils._device import DeviceContext

from . import _check, _ptr, _stream, attn_fwd, dense_causal_fwd, load

__all__ = ["middle_layers", "PrefillStack"]


def middle_layers(cfg, count=8):
    """Indices of the `count` central layers of the stack (the paper converts
    eight middle layers of 28, §4.4; here layers 10..17)."""
    start = (cfg.layers - count) // 2
    return set(range(start, start + count))


def _operators_followed():
    """Whether something follows the operators of a call themselves (tracing,
    compilation, function transforms, forward-mode derivatives, torch's operator
    modes), to which a kernel launched by pointers would be invisible."""
    return (torch.compiler.is_compiling() or torch._C._get_tracing_state() is not None
            or torch._C._functorch.peek_interpreter_stack() is not None or forward_ad._current_level >= 0
            or torch._C._len_torch_dispatch_stack() > 0 or torch._ops._len_torch_dispatch_stack_pre_dispatch() > 0
            or (torch._C._len_torch_function_stack() > 0 and any(
                not isinstance(m, DeviceContext) for m in torch.overrides._get_current_function_mode_stack())))


class PrefillStack:
    """cfg: a synth.ModelConfig; weights: the generator's bf16 tensors
    (projections stored [in, out]); B, L: block width and local width of the
    BF1 layers.

    ``w`` holds the weights as they were given where they are contiguous tensors
    of ``device`` already (an update in place is seen by the next call), copies
    of them otherwise.  (Projections kept joined and transposed would make the
    GEMMs of 8192 tokens, hidden 1024, 218 us per layer instead of 284, but as a
    second copy of every projection, which no longer follows the caller's.)"""

    def __init__(self, cfg, weights, device="cuda", B=64, L=2):
        self.cfg, self.B, self.L = cfg, B, L
        self.w = {k: v.to(device).contiguous() for k, v in weights.items()}
        self.device = device
        self._rope_n = -1

    def _rope_tables(self, n):
        if n != self._rope_n:
            d = self.cfg.head_dim
            inv = self.cfg.rope_theta ** (-torch.arange(0, d, 2, dtype=torch.float64, device=self.device) / d)
            ang = torch.arange(n, dtype=torch.float64, device=self.device)[:, None] * inv[None, :]
            self._cos = torch.cat([ang.cos(), ang.cos()], dim=-1).float()[:, None, :]
            self._sin = torch.cat([ang.sin(), ang.sin()], dim=-1).float()[:, None, :]
            self._rope_n = n
        return self._cos, self._sin

    def _rms(self, x, w):
        xf = x.float()
        y = xf * torch.rsqrt(xf.pow(2).mean(-1, keepdim=True) + self.cfg.eps)
        return (y * w.float()).to(torch.bfloat16)

    def _rope(self, x, cos, sin):
        xf = x.float()
        half = xf.shape[-1] // 2
        rot = torch.cat([-xf[..., half:], xf[..., :half]], dim=-1)
        return (xf * cos + rot * sin).to(torch.bfloat16)

    # ---- one layer ------------------------------------------------------------

    def _attention(self, l, Q, K, V, bf1_layers, dense_attention):
        if l in bf1_layers:
            return attn_fwd(Q, K, V, self.B, self.L, want_lse=False)[0]
        if dense_attention is not None:
            return dense_attention(Q, K, V)
        return dense_causal_fwd(Q, K, V, want_lse=False)[0]

    def _layer_plain(self, l, h, cos, sin, bf1_layers, dense_attention):
        """One layer, operator by operator: any device, type and shape."""
        cfg, w, p = self.cfg, self.w, f"{l}."
        n, H, Hkv, d = h.shape[0], cfg.heads, cfg.kv_heads, cfg.head_dim
        a = self._rms(h, w[p + "in_norm"])
        q = self._rms((a @ w[p + "wq"]).view(n, H, d), w[p + "q_norm"])
        k = self._rms((a @ w[p + "wk"]).view(n, Hkv, d), w[p + "k_norm"])
        v = (a @ w[p + "wv"]).view(n, Hkv, d)
        q, k = self._rope(q, cos, sin), self._rope(k, cos, sin)
        Q = q.transpose(0, 1).contiguous().unsqueeze(0)
        K = k.transpose(0, 1).contiguous().unsqueeze(0)
        V = v.transpose(0, 1).contiguous().unsqueeze(0)
        O = self._attention(l, Q, K, V, bf1_layers, dense_attention)
        return self._tail_plain(l, h, O[0].transpose(0, 1).reshape(n, H * d))

    def _tail_plain(self, l, h, O):
        """A layer after its attention output O [n, heads * d]."""
        w, p = self.w, f"{l}."
        h = h + O @ w[p + "wo"]
        a = self._rms(h, w[p + "post_norm"])
        return h + (torch.nn.functional.silu(a @ w[p + "wg"]) * (a @ w[p + "wu"])) @ w[p + "wd"]

    def _fused(self, l, h, cos):
        """Whether layer l can run on the row kernels: bf16 weights of matching
        shapes on h's GPU, the kernels' head sizes and widths, GEMMs that give bf16,
        no autograd graph wanted through the layer and nothing else that follows
        its operators."""
        cfg, w, p = self.cfg, self.w, f"{l}."
        if type(h) is not torch.Tensor or not h.is_cuda or h.dtype != torch.bfloat16 or h.dim() != 2 \
                or cos.device != h.device:
            return False
        if torch.is_autocast_enabled("cuda") and torch.get_autocast_dtype("cuda") != torch.bfloat16:
            return False  # the GEMMs' results would not be bf16
        if _operators_followed():
            return False
        n, hidden = h.shape
        H, Hkv, d = cfg.heads, cfg.kv_heads, cfg.head_dim
        if n == 0 or d not in (64, 128) or hidden % 8 or hidden > 4096 or max(H, Hkv) > 4096:
            return False
        inter = w[p + "wg"].shape[-1]
        # the kernels' launches: a wave per row, d / 16 lanes per head, a lane per 8 of inter
        if inter % 8 or n * max(64, (H + 2 * Hkv) * (d // 16), inter // 8) >= 1 << 32:
            return False
        grad = torch.is_grad_enabled()
        if grad and h.requires_grad:
            return False
        for name, shape in (("in_norm", (hidden,)), ("q_norm", (d,)), ("k_norm", (d,)), ("post_norm", (hidden,)),
                            ("wq", (hidden, H * d)), ("wk", (hidden, Hkv * d)), ("wv", (hidden, Hkv * d)),
                            ("wo", (H * d, hidden)), ("wg", (hidden, inter)), ("wu", (hidden, inter)),
                            ("wd", (inter, hidden))):
            t = w[p + name]
            if not self._weight(t, shape, h.device, grad):
                return False
        return True

    def _weight(self, t, shape, device, grad):
        """Whether t is a plain bf16 weight of `shape` on `device` that wants no
        gradient, and if it is a norm gain one that can be read by its pointer."""
        return (type(t) is torch.Tensor or type(t) is torch.nn.Parameter) and t.shape == shape \
            and t.dtype is torch.bfloat16 and t.device == device and not (grad and t.requires_grad) \
            and (len(shape) > 1 or (t.is_contiguous() and t.data_ptr() % 16 == 0 and not t.is_neg()))

    def _rms_fused(self, h, r, gain):
        """h <- h + r in place (if r is given), then RMSNorm(h) * gain."""
        out = torch.empty_like(h)
        _check(load().bf1_stack_rms(_ptr(h), _ptr(r), _ptr(gain), _ptr(out), h.shape[0], h.shape[1], self.cfg.eps,
                                    _stream(None, h.device)), "bf1_stack_rms")
        return out

    # Three GEMMs of one input cost 18 us of host time each, which bounds prefills
    # below some 2K tokens; putting small matrices side by side first costs one
    # launch and a copy.  Per layer, hidden 1024 (4.2M and 6.3M entries), us,
    # separate / side by side: 128 to 2048 tokens 187 / 159, 8192 tokens 428 / 409,
    # 16384 724 / 729; hidden 4096 (16.8M and 100M entries) 128 tokens 309 / 421, 8192
    # tokens 2458 / 2605.
    def _project(self, a, keys):
        """a @ w[k] for each key: one GEMM on the matrices side by side while they
        are small."""
        ts = [self.w[k] for k in keys]
        if sum(t.numel() for t in ts) > 8 << 20:
            return [a @ t for t in ts]
        return (a @ torch.cat(ts, 1)).split([t.shape[1] for t in ts], dim=1)

    def _layer_fused(self, l, h, r, cos, sin, bf1_layers, dense_attention):
        """One layer between library GEMMs on the row kernels; h is updated in
        place.  r is the previous layer's MLP output (None before the first),
        not yet added to h; returns h and this layer's r.  An attention callable
        may return what the kernels must not take by its pointer, such as a tensor
        with a gradient: the layer then ends operator by operator."""
        cfg, w, p, lib = self.cfg, self.w, f"{l}.", load()
        n, H, Hkv, d = h.shape[0], cfg.heads, cfg.kv_heads, cfg.head_dim
        a = self._rms_fused(h, r, w[p + "in_norm"])
        q, k, v = self._project(a, (p + "wq", p + "wk", p + "wv"))
        Q, K, V = (torch.empty((1, x, n, d), dtype=h.dtype, device=h.device) for x in (H, Hkv, Hkv))
        _check(lib.bf1_stack_heads(_ptr(q), _ptr(k), _ptr(v), q.stride(0), k.stride(0), v.stride(0),
                                   _ptr(w[p + "q_norm"]), _ptr(w[p + "k_norm"]), _ptr(cos), _ptr(sin), _ptr(Q),
                                   _ptr(K), _ptr(V), n, H, Hkv, d, cfg.eps, _stream(None, h.device)), "bf1_stack_heads")
        if l not in bf1_layers and dense_attention is not None:
            O = dense_attention(Q, K, V)[0].transpose(0, 1).reshape(n, H * d)
            if type(O) is not torch.Tensor or O.dtype != torch.bfloat16 or O.device != h.device \
                    or (O.requires_grad and torch.is_grad_enabled()):
                return self._tail_plain(l, h, O), None
        else:
            O = torch.empty((n, H * d), dtype=h.dtype, device=h.device)
            _check(lib.bf1_attn_fwd_token_major(_ptr(Q), _ptr(K), _ptr(V), _ptr(O), 1, n, H, Hkv, d, int(self.B),
                                                int(self.L), int(l not in bf1_layers), _stream(None, h.device)),
                   "bf1_attn_fwd_token_major")
        a = self._rms_fused(h, O @ w[p + "wo"], w[p + "post_norm"])
        g, u = self._project(a, (p + "wg", p + "wu"))
        s = torch.empty(g.shape, dtype=g.dtype, device=g.device)
        _check(lib.bf1_stack_swiglu(_ptr(g), _ptr(u), g.stride(0), u.stride(0), _ptr(s), n, g.shape[1],
                                    _stream(None, h.device)), "bf1_stack_swiglu")
        return h, s @ w[p + "wd"]

    def last_logits(self, ids, bf1_layers, dense_attention=None):
        """Logits (float32, [vocab]) of the last position after the prefill of
        token ids (int64 device tensor [n]).  dense_attention, if given,
        replaces the in-house dense kernel for the non-BF1 layers: a callable
        (Q, K, V) -> O on [1, heads, n, d] bf16 tensors (a comparator)."""
        cfg, w = self.cfg, self.w
        cos, sin = self._rope_tables(ids.shape[0])
        h = w["embed"][ids]
        r = None  # MLP output of the layer before, not yet added to h
        with torch.cuda.device(h.device) if h.is_cuda else contextlib.nullcontext():
            for l in range(cfg.layers):
                if self._fused(l, h, cos):
                    h, r = self._layer_fused(l, h, r, cos, sin, bf1_layers, dense_attention)
                    continue
                h, r = h if r is None else h + r, None
                h = self._layer_plain(l, h, cos, sin, bf1_layers, dense_attention)
            last = h[-1:]
            gain = w["final_norm"]
            if r is not None and self._weight(gain, h.shape[1:], h.device, torch.is_grad_enabled()):
                last = self._rms_fused(last, r[-1:], gain)  # h's last row is not read again
            else:
                last = self._rms(last if r is None else last + r[-1:], gain)
        return (last @ w["embed"].t()).float()[0]
