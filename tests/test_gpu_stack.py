"""GPU checks of the prefill stack's row kernels: RMSNorm with the residual
add, head split with per-head norm and rotary embedding, SwiGLU, and the
token-major attention output.

Bars, from the arithmetic: every kernel computes in fp32 (a handful of
roundings of 2^-24 each, the mean over up to 4096 terms another 2^-20) and
rounds to bf16 (8 significant bits: at most half an ulp, 2^-8 relative) where
the operator sequence rounds.  One rounding: |err| <= (2^-8 + 2^-16) |y|.  Two
roundings, the first scaled by the second factor (norm then rotation, silu then
product): 2^-7 plus
the same slack, of the magnitudes that are added.
"""

import ctypes

import pytest
import torch

import paper_2608_20427_amd as bf1
from paper_2608_20427_amd import synth
from paper_2608_20427_amd.prefill_model import PrefillStack

pytestmark = pytest.mark.gpu
EPS = 1e-6


def _n(g, *shape, mul=1.0):
    return (mul * torch.randn(shape, generator=g, device="cuda")).to(torch.bfloat16)


def _g(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _call(name, *args):
    conv = [ctypes.c_void_p(a.data_ptr()) if isinstance(a, torch.Tensor) else a for a in args]
    st = getattr(bf1.load(), name)(*conv, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    return st


@pytest.mark.parametrize("residual", [False, True])
@pytest.mark.parametrize("rows,cols", [(1, 8), (3, 504), (4, 512), (5, 1024), (6, 1032), (9, 2048), (2, 2056),
                                       (7, 4096)])
def test_rms(rows, cols, residual):
    print("rms", rows, cols, residual, flush=True)
    g = _g(rows * 10000 + cols)
    h, r, w = _n(g, rows, cols, mul=3), _n(g, rows, cols), _n(g, cols)
    want_h = (h + r) if residual else h.clone()
    x = want_h.double()
    ref = x * torch.rsqrt(x.pow(2).mean(-1, keepdim=True) + EPS) * w.double()
    out = torch.empty_like(h)
    assert _call("bf1_stack_rms", h, r if residual else None, w, out, rows, cols, EPS) == bf1.BF1_OK
    assert torch.equal(h, want_h)
    assert ((out.double() - ref).abs() <= (2.0 ** -8 + 2.0 ** -16) * ref.abs()).all()


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n,H,Hkv,pad", [(1, 1, 1, 0), (7, 4, 2, 0), (129, 3, 1, 8), (64, 16, 8, 0)])
def test_heads(d, n, H, Hkv, pad):
    print("heads", d, n, H, Hkv, pad, flush=True)
    g = _g(d + n + H)
    q, k, v = (_n(g, n, x * d + pad, mul=2) for x in (H, Hkv, Hkv))
    wq, wk = _n(g, d), _n(g, d)
    ang = torch.arange(n, dtype=torch.float64, device="cuda")[:, None] * \
        1e6 ** (-torch.arange(0, d, 2, dtype=torch.float64, device="cuda") / d)[None]
    cos, sin = (torch.cat([f, f], -1).float().contiguous() for f in (ang.cos(), ang.sin()))
    Q, K, V = (torch.empty((x, n, d), dtype=torch.bfloat16, device="cuda") for x in (H, Hkv, Hkv))
    assert _call("bf1_stack_heads", q, k, v, q.stride(0), k.stride(0), v.stride(0), wq, wk, cos, sin, Q, K, V, n, H,
                 Hkv, d, EPS) == bf1.BF1_OK
    assert torch.equal(V, v[:, :Hkv * d].view(n, Hkv, d).transpose(0, 1))
    for got, src, w, heads in ((Q, q, wq, H), (K, k, wk, Hkv)):
        x = src[:, :heads * d].reshape(n, heads, d).double()
        x = x * torch.rsqrt(x.pow(2).mean(-1, keepdim=True) + EPS) * w.double()
        a, b = x[..., :d // 2], x[..., d // 2:]
        c, s = cos.double()[:, None, :d // 2], sin.double()[:, None, :d // 2]
        ref = torch.cat([a * c - b * s, b * c + a * s], -1).transpose(0, 1)
        mag = torch.cat([(a * c).abs() + (b * s).abs(), (b * c).abs() + (a * s).abs()], -1).transpose(0, 1)
        assert ((got.double() - ref).abs() <= (2.0 ** -7 + 2.0 ** -14) * mag).all()


@pytest.mark.parametrize("rows,cols,pad", [(1, 8, 0), (3, 40, 8), (257, 3072, 0)])
def test_swiglu(rows, cols, pad):
    print("swiglu", rows, cols, pad, flush=True)
    g = _g(rows + cols)
    a, u = _n(g, rows, cols + pad, mul=8), _n(g, rows, cols + pad)
    a[0, 0], a[0, 1] = -100.0, 100.0      # exp overflows to infinity and to zero
    out = torch.empty((rows, cols), dtype=torch.bfloat16, device="cuda")
    assert _call("bf1_stack_swiglu", a, u, a.stride(0), u.stride(0), out, rows, cols) == bf1.BF1_OK
    x = a[:, :cols].double()
    ref = x * torch.sigmoid(x) * u[:, :cols].double()
    # results below fp32's smallest normal number may be flushed
    assert ((out.double() - ref).abs() <= (2.0 ** -7 + 2.0 ** -14) * ref.abs() + 1e-36).all()


@pytest.mark.parametrize("cfg", [(1, 64, 2, 1, 64, 64), (2, 129, 4, 2, 128, 64), (1, 700, 8, 1, 64, 128),
                                 (2, 300, 2, 2, 128, 128)])
@pytest.mark.parametrize("dense", [0, 1])
@pytest.mark.parametrize("split", [1, 2])
def test_token_major_output_is_bitwise_the_forward(cfg, dense, split):
    batch, n, Hq, Hkv, d, B = cfg
    print("token major", cfg, dense, split, flush=True)
    g = _g(n)
    q, k, v = _n(g, batch, Hq, n, d), _n(g, batch, Hkv, n, d), _n(g, batch, Hkv, n, d)
    out = torch.full((batch, n, Hq, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    bf1.set_forward_key_split(split)
    try:
        ref, _ = bf1.dense_causal_fwd(q, k, v) if dense else bf1.attn_fwd(q, k, v, B, 2)
        assert _call("bf1_attn_fwd_token_major", q, k, v, out, batch, n, Hq, Hkv, d, B, 2, dense) == bf1.BF1_OK
    finally:
        bf1.set_forward_key_split(0)
    assert torch.equal(out.transpose(1, 2), ref)


def test_arguments_rejected():
    t = torch.zeros(8192, dtype=torch.bfloat16, device="cuda")
    f = torch.zeros(128, device="cuda")
    odd = ctypes.c_void_p(t.data_ptr() + 2)
    assert _call("bf1_stack_rms", t, None, t, t, 1, 12, EPS) == bf1.BF1_ERR_UNSUPPORTED
    assert _call("bf1_stack_rms", t, None, t, t, 1, 4104, EPS) == bf1.BF1_ERR_UNSUPPORTED
    assert _call("bf1_stack_rms", odd, None, t, t, 1, 8, EPS) == bf1.BF1_ERR_INVALID_ARG
    assert _call("bf1_stack_swiglu", t, t, 4, 8, t, 1, 8) == bf1.BF1_ERR_INVALID_ARG
    assert _call("bf1_stack_swiglu", t, t, 12, 12, t, 1, 12) == bf1.BF1_ERR_UNSUPPORTED
    assert _call("bf1_stack_heads", t, t, t, 96, 96, 96, t, t, f, f, t, t, t, 1, 1, 1, 96, EPS) == \
        bf1.BF1_ERR_UNSUPPORTED
    assert _call("bf1_attn_fwd_token_major", t, t, t, t, 1, 8, 1, 1, 64, 96, 2, 0) == bf1.BF1_ERR_UNSUPPORTED
    assert _call("bf1_attn_fwd_token_major", t, t, t, t, 1, 8, 1, 1, 64, 64, 2, 2) == bf1.BF1_ERR_INVALID_ARG


CFG = synth.ModelConfig(layers=3, hidden=256, heads=4, kv_heads=2, head_dim=64, intermediate=512, vocab=1000)


def _stack(cfg=CFG, **replace):
    st = PrefillStack(cfg, synth.make_model_weights(cfg, 11), device="cuda")
    st.w.update({k: f(st.w[k]) for k, f in replace.items()})
    return st


def test_fused_stack_matches_the_operators_and_mixes_with_them():
    # the two forms round at the same places, so a few bf16 ulps of the largest
    # logit separate them; a layer the kernels do not take (a float32 norm gain
    # here) runs operator by operator between fused ones
    ids = torch.from_numpy(synth.make_tokens(CFG, 333, 4)).cuda()
    st = _stack()
    plain = _stack()
    plain._fused = lambda *a: False
    mixed = _stack(**{"1.in_norm": lambda t: t.float()})
    cos, _ = mixed._rope_tables(333)
    h = mixed.w["embed"][ids]
    assert [mixed._fused(l, h, cos) for l in range(3)] == [True, False, True]
    for layers in (set(), {0, 2}, {0, 1, 2}):
        a, b, c = (s.last_logits(ids, layers) for s in (st, plain, mixed))
        top = b.abs().max()
        assert (a - b).abs().max() <= 2e-2 * top and (c - b).abs().max() <= 2e-2 * top


def test_autograd_keeps_the_operators():
    st = _stack(**{"2.wd": lambda t: t.clone().requires_grad_()})
    ids = torch.from_numpy(synth.make_tokens(CFG, 70, 4)).cuda()
    st.last_logits(ids, {0}).sum().backward()
    assert st.w["2.wd"].grad is not None and torch.isfinite(st.w["2.wd"].grad).all()


def _soft(Q, K, V):
    # dense causal attention by plain operators, in fp32, for a callable
    G, n = int(Q.shape[1]) // int(K.shape[1]), int(Q.shape[2])
    Q, K, V = Q.float(), K.float().repeat_interleave(G, 1), V.float().repeat_interleave(G, 1)
    s = Q @ K.transpose(2, 3).contiguous() / Q.shape[-1] ** 0.5
    s = s.masked_fill(torch.ones(n, n, device=Q.device).triu(1).bool(), float("-inf"))
    return (s.softmax(-1) @ V).to(torch.bfloat16)


@pytest.mark.parametrize("leaf", ["scale", "scale and final_norm"])
def test_gradients_through_the_attention_callable(leaf):
    # a callable with a parameter of its own: the logits carry its gradient as
    # they do operator by operator, whatever else wants one.  bf16 gradients of
    # three layers, a few roundings (2^-8) each, summed over a thousand entries of
    # both signs.
    ids = torch.from_numpy(synth.make_tokens(CFG, 70, 4)).cuda()
    grads = []
    for plain in (False, True):
        st = _stack()
        if leaf != "scale":
            st.w["final_norm"].requires_grad_()
        if plain:
            st._fused = lambda *a: False
        scale = torch.ones(64, device="cuda", requires_grad=True)
        out = st.last_logits(ids, {0}, lambda Q, K, V: (_soft(Q, K, V) * scale).to(torch.bfloat16))
        out.square().sum().backward()
        grads.append(scale.grad)
    assert (grads[0] - grads[1]).abs().max() <= 5e-2 * grads[1].abs().max() and grads[1].abs().max() > 0


def test_autocast_to_another_type_keeps_the_operators():
    # projections under fp16 autocast are fp16: the attention entry refuses such
    # V, a callable gets them; under bf16 autocast nothing changes
    st = _stack()
    ids = torch.from_numpy(synth.make_tokens(CFG, 70, 4)).cuda()
    base, seen = st.last_logits(ids, {0}), []
    with torch.autocast("cuda", dtype=torch.float16):
        with pytest.raises(ValueError, match="dtype"):
            st.last_logits(ids, {0, 1, 2})

        def dense(Q, K, V):
            seen.append(V.dtype)
            return bf1.dense_causal_fwd(Q, K, V.to(torch.bfloat16), want_lse=False)[0]
        a = st.last_logits(ids, set(), dense)
    assert seen == [torch.float16] * 3
    assert (a - st.last_logits(ids, set())).abs().max() <= 2e-2 * base.abs().max()
    with torch.autocast("cuda", dtype=torch.bfloat16):
        assert torch.equal(st.last_logits(ids, {0}), base)


def _follow_vmap(st, ids, run):
    return torch.vmap(run)(torch.stack([ids, ids.flip(0)]))[1]


def _follow_jvp(st, ids, run):
    # tangent of every V projection its own value: the derivative along a scaling
    keys = [f"{l}.wv" for l in range(CFG.layers)]
    kept = [st.w[k] for k in keys]

    def f(*ts):
        st.w.update(zip(keys, ts))
        return run(ids)
    out = torch.func.jvp(f, tuple(kept), tuple(kept))[1]
    st.w.update(zip(keys, kept))
    return out


def _follow_dual(st, ids, run):
    kept = st.w["0.in_norm"]
    with torch.autograd.forward_ad.dual_level():
        st.w["0.in_norm"] = torch.autograd.forward_ad.make_dual(kept, kept.clone())
        out = torch.autograd.forward_ad.unpack_dual(run(ids)).tangent
    st.w["0.in_norm"] = kept
    return torch.zeros_like(run(ids)) if out is None else out


def _follow_trace(st, ids, run):
    from torch.fx.experimental.proxy_tensor import make_fx
    return make_fx(run)(ids)(ids.flip(0))


def _follow_jit(st, ids, run):
    return torch.jit.trace(run, ids, check_trace=False)(ids.flip(0))


def _follow_compile(st, ids, run):
    return torch.compile(run, backend="eager")(ids)


def _follow_mode(st, ids, run):
    class Count(torch.utils._python_dispatch.TorchDispatchMode):
        seen = 0

        def __torch_dispatch__(self, f, types, args=(), kwargs=None):
            Count.seen += f is torch.ops.aten.silu.default
            return f(*args, **(kwargs or {}))
    with Count():
        run(ids)
    return torch.tensor([float(Count.seen)])


@pytest.mark.parametrize("follow", [_follow_vmap, _follow_jvp, _follow_dual, _follow_trace, _follow_jit,
                                    _follow_compile, _follow_mode], ids=lambda f: f.__name__[8:])
@pytest.mark.filterwarnings("ignore")
def test_what_follows_the_operators_sees_them(follow):
    # transforms, traces and modes over a stack of plain operators (a callable for
    # every layer) give what they give with the row kernels switched off
    ids = torch.from_numpy(synth.make_tokens(CFG, 70, 4)).cuda()
    got = []
    for plain in (True, False):
        st = _stack()
        if plain:
            st._fused = lambda *a: False
        with torch.no_grad():
            st._rope_tables(70)
            got.append(follow(st, ids, lambda x: st.last_logits(x, set(), _soft)))
    assert got[0].abs().max() > 0
    assert (got[0] - got[1]).abs().max() <= 2e-2 * got[0].abs().max()


def test_sizes_past_a_launch_run_on_operators():
    # rows that share their memory stand for a prompt of that length
    st = _stack()
    row = st.w["embed"][:1]
    cos, _ = st._rope_tables(1)
    assert st._fused(0, row.expand((1 << 26) - 1, -1), cos)
    assert not st._fused(0, row.expand(1 << 26, -1), cos)


def test_default_device_keeps_the_kernels():
    st = _stack()
    h = st.w["embed"][:4].clone()
    with torch.device("cuda"):
        assert st._fused(0, h, st._rope_tables(4)[0])


def test_dense_attention_callable_sees_contiguous_heads():
    st = _stack()
    ids = torch.from_numpy(synth.make_tokens(CFG, 200, 4)).cuda()
    seen = []

    def dense(Q, K, V):
        seen.append((tuple(Q.shape), tuple(K.shape), Q.is_contiguous() and K.is_contiguous() and V.is_contiguous()))
        return bf1.dense_causal_fwd(Q, K, V, want_lse=False)[0]
    a = st.last_logits(ids, {1}, dense)
    assert seen == [((1, 4, 200, 64), (1, 2, 200, 64), True)] * 2
    assert torch.equal(a, st.last_logits(ids, {1}))


@pytest.mark.parametrize("hidden,inter,joined", [(256, 512, True), (1024, 4096, True), (1024, 4104, False)])
def test_projections_side_by_side(hidden, inter, joined):
    # up to 2^23 entries one GEMM (rows of all matrices), above one each; a product
    # of bf16 with fp32 sums of 1024 terms, rounded once (2^-8, and 2^-16 of the
    # terms' magnitudes for the sums)
    g = _g(hidden + inter)
    st = _stack()
    st.w["0.wg"], st.w["0.wu"] = _n(g, hidden, inter), _n(g, hidden, inter)
    a = _n(g, 33, hidden)
    got = st._project(a, ("0.wg", "0.wu"))
    assert [t.stride() for t in got] == [(2 * inter if joined else inter, 1)] * 2
    for t, k in zip(got, ("0.wg", "0.wu")):
        ref, mag = a.double() @ st.w[k].double(), a.double().abs() @ st.w[k].double().abs()
        assert ((t.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 2.0 ** -16 * mag).all()


def test_weights_are_the_callers():
    # contiguous weights on the device are shared, not copied: an update in place
    # of what the caller passed reaches the next call (bitwise a stack built from
    # the changed values), two layers may be one tensor, and a replaced entry is
    # used.  The updates change the result visibly: a norm follows Q and K, so V,
    # gate and up are the projections changed.
    ids = torch.from_numpy(synth.make_tokens(CFG, 90, 4)).cuda()
    given = {k: v.cuda() for k, v in synth.make_model_weights(CFG, 11).items()}
    for x in ("wq", "wk", "wv", "wo", "wg", "wu", "wd"):
        given[f"2.{x}"] = given[f"1.{x}"]
    before = torch.cuda.memory_allocated()
    st = PrefillStack(CFG, given, device="cuda")
    assert torch.cuda.memory_allocated() == before
    assert all(st.w[k].data_ptr() == given[k].data_ptr() and st.w[k].is_contiguous() for k in given)
    base = st.last_logits(ids, {0})
    top = base.abs().max()
    for change in ("1.wv", "0.wg", "0.wu"):
        last = st.last_logits(ids, {0})
        given[change].neg_()
        now = st.last_logits(ids, {0})
        assert (now - last).abs().max() > 0.1 * top
        assert torch.equal(now, PrefillStack(CFG, {k: v.clone() for k, v in given.items()}).last_logits(ids, {0}))
    last = st.last_logits(ids, {0})
    st.w["0.wv"] = -st.w["0.wv"]
    assert (st.last_logits(ids, {0}) - last).abs().max() > 0.1 * top
    # host weights are copied, on the device and contiguous as well
    host = PrefillStack(CFG, synth.make_model_weights(CFG, 11), device="cuda")
    assert all(t.is_cuda and t.is_contiguous() for t in host.w.values())
