"""The workloads this library is timed on, through its public entry points.

Three kinds of call stand for what a user of the library has it do: prefill
attention (forward, dense comparator and backward, in the Qwen3-0.6B layer
geometry of the paper's study and in the smaller geometries of the tests),
one-token decode over a paged cache, and the whole-model prefill stack.  Every
listed size is one of the repository's own workloads or sweep points;
``draw`` spreads over the ranges between and around them.

All inputs are drawn on the GPU from the seed: standard normal Q, K, V, dO
(optionally with 5% of the key positions scaled by three, which gives peaked
softmax rows), random page orders, and seeded random weights and tokens.
"""

import math

import numpy as np
import torch

import paper_2608_20427_amd as bf1
from paper_2608_20427_amd import synth
from paper_2608_20427_amd.prefill_model import PrefillStack


def _attn(name, entry, n, batch=1, Hq=16, Hkv=8, d=128, B=64, L=2, peaked=False):
    return {"name": name, "kind": "attn", "entry": entry, "n": n, "batch": batch, "Hq": Hq, "Hkv": Hkv, "d": d,
            "B": B, "L": L, "peaked": peaked}


def _decode(name, batch, ctx, ragged, Hq=16, Hkv=8, d=128, B=64, L=2, dense=False, replan=False):
    return {"name": name, "kind": "decode", "batch": batch, "ctx": ctx, "ragged": ragged, "Hq": Hq, "Hkv": Hkv,
            "d": d, "B": B, "L": L, "dense": dense, "replan": replan}


def _model(name, n, layers, bf1_layers):
    return {"name": name, "kind": "model", "n": n, "layers": layers, "bf1_layers": bf1_layers}


def listed():
    return [
        # a short prompt: one layer's attention, where launches and latency count
        _attn("prefill_1k", "fwd", 1024),
        # the headline step: route planner and attention kernel, one 32K prompt
        _attn("prefill_32k", "plan_csr", 32768),
        # two long prompts of an odd length with peaked rows (30001 = 468 * 64 + 49)
        _attn("prefill_ragged_b2", "fwd", 30001, batch=2, peaked=True),
        # the longest point of the length sweep, wide blocks, no device allocation
        # (the form for graph capture and serving loops)
        _attn("prefill_64k_wide", "noalloc", 65536, B=128),
        # a dense layer of a mixed stack (the 20 of 28 that stay dense in the study)
        _attn("dense_8k", "dense", 8192),
        # the training direction at a short context and at the headline one
        _attn("backward_4k", "bwd", 4096),
        _attn("backward_32k", "bwd", 32768),
        # the small head dimension, odd length, two sequences, wider group
        _attn("backward_small", "bwd", 1500, batch=2, Hq=8, Hkv=2, d=64),
        # a serving step: one sequence (latency), and a full batch of mixed lengths
        _decode("decode_32k_b1", 1, 32768, False),
        _decode("decode_64k_b32", 32, 65536, True),
        # blocks of the model: four layers on the BF1 route at a short prompt
        _model("stack4_2k", 2048, 4, "all"),
        # time to first token of a stack that mixes BF1 and dense layers, at the
        # shortest context of the whole-model study; ten layers deep, because the
        # bf16 rounding of 28 would put two correct implementations 3% apart
        _model("stack10_8k", 8192, 10, "half"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    u = rng.random()
    if u < 0.60:
        entry = rng.choice(["fwd", "fwd", "plan_csr", "noalloc", "sliding", "dense", "bwd", "bwd", "bwd"])
        Hq, Hkv = rng.choice([(16, 8), (16, 8), (16, 8), (8, 8), (8, 2), (16, 2), (2, 1)])
        d = rng.choice([128, 128, 64])
        B = rng.choice([64, 64, 128])
        L = rng.choice([2, 2, 1, 3])
        batch = rng.choice([1, 1, 2, 4])
        top = {"dense": 16384, "bwd": 32768}.get(entry, 65536) // batch
        n = _log_int(rng, 300, top)
        if rng.random() < 0.3:
            n = max(64, n // 64 * 64)
        if entry == "bwd" and Hq // Hkv * B < 128:
            B = 128  # the backward needs 128 stacked rows per block
        c = _attn("", entry, n, batch, Hq, Hkv, d, B, L, rng.random() < 0.3)
    elif u < 0.85:
        Hq, Hkv = rng.choice([(16, 8), (16, 8), (8, 8), (8, 2), (16, 2)])
        dense = rng.random() < 0.15
        batch = _log_int(rng, 1, 48)
        c = _decode("", batch, _log_int(rng, 500, 65536), rng.random() < 0.6, Hq, Hkv, rng.choice([128, 128, 64]),
                    rng.choice([64, 64, 128]), rng.choice([2, 2, 1, 3]), dense, rng.random() < 0.25)
    else:
        layers = rng.randint(1, 6)
        c = _model("", _log_int(rng, 200, 8192), layers, rng.choice(["all", "none", "half"]))
    del c["name"]
    return c


# ---- inputs -------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _normal(g, *shape):
    return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(torch.bfloat16)


def _qkv(c, g):
    q = _normal(g, c["batch"], c["Hq"], c["n"], c["d"])
    k = _normal(g, c["batch"], c["Hkv"], c["n"], c["d"])
    v = _normal(g, c["batch"], c["Hkv"], c["n"], c["d"])
    if c["peaked"]:
        at = torch.rand((c["batch"], 1, c["n"], 1), generator=g, device="cuda") < 0.05
        k = torch.where(at, k * 3, k)
    return q, k, v


def _cfg(c):
    q = synth.QWEN3_06B
    return synth.ModelConfig(layers=c["layers"], hidden=q.hidden, heads=q.heads, kv_heads=q.kv_heads,
                             head_dim=q.head_dim, intermediate=q.intermediate, vocab=q.vocab,
                             rope_theta=q.rope_theta, eps=q.eps)


def _bf1_layers(c):
    return {"all": set(range(c["layers"])), "none": set(), "half": set(range(0, c["layers"], 2))}[c["bf1_layers"]]


def _seq_lens(c, seed):
    if not c["ragged"]:
        return np.full(c["batch"], c["ctx"], dtype=np.int32)
    rng = np.random.Generator(np.random.PCG64([seed, 1]))
    lens = rng.integers(max(1, c["ctx"] // 2), c["ctx"] + 1, size=c["batch"]).astype(np.int32)
    lens[0] = c["ctx"]
    return lens


def prepare(case, seed):
    c = case
    if c["kind"] == "attn":
        g = _gen(seed)
        q, k, v = _qkv(c, g)
        s = {"case": c, "q": q, "k": k, "v": v}
        if c["entry"] == "bwd":
            s["do"] = _normal(g, *q.shape)
            s["o"], s["lse"] = bf1.attn_fwd(q, k, v, c["B"], c["L"])
            need = bf1.bwd_workspace_size(c["batch"], c["n"], c["Hq"], c["Hkv"], c["d"], c["B"], c["L"])
            s["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
        elif c["entry"] == "noalloc":
            s["o"] = torch.empty_like(q)
            s["lse"] = torch.empty(q.shape[:3], dtype=torch.float32, device="cuda")
        elif c["entry"] == "plan_csr":
            nb, nnz, _ = bf1.plan_size(c["n"], c["B"], c["L"])
            s["rp"] = torch.empty(nb + 1, dtype=torch.int32, device="cuda")
            s["ci"] = torch.empty(nnz, dtype=torch.int32, device="cuda")
            s["o"] = torch.empty_like(q)
            s["lse"] = torch.empty(q.shape[:3], dtype=torch.float32, device="cuda")
        elif c["entry"] == "sliding":
            rp, ci = bf1.plan_variant("sliding", c["n"], c["B"], c["L"])
            s["rp"], s["ci"] = torch.from_numpy(rp).cuda(), torch.from_numpy(ci).cuda()
        return s
    if c["kind"] == "decode":
        lens = _seq_lens(c, seed)
        g = _gen(seed)
        owned = -(-lens.astype(np.int64) // c["B"])
        pages = int(owned.sum())
        q = _normal(g, c["batch"], c["Hq"], c["d"])
        shape = (pages, c["Hkv"], c["B"], c["d"])
        kp = torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)
        vp = torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)
        order = torch.randperm(pages, generator=g, device="cuda").to(torch.int32)
        table = torch.full((c["batch"], int(owned.max())), -1, dtype=torch.int32, device="cuda")
        at = 0
        for b, m in enumerate(owned.tolist()):
            table[b, :m] = order[at:at + m]
            at += m
        sl = torch.from_numpy(lens).cuda()
        stride = bf1.decode_plan_stride(c["ctx"], c["B"], c["L"], c["dense"])
        need = bf1.decode_workspace_size(c["batch"], c["Hq"], c["Hkv"], c["d"], stride)
        return {"case": c, "q": q, "kp": kp, "vp": vp, "sl": sl, "table": table, "pages": pages, "stride": stride,
                "plan": bf1.decode_plan(sl, table, pages, stride, c["B"], c["L"], c["dense"]),
                "o": torch.empty_like(q), "lse": torch.empty(q.shape[:2], dtype=torch.float32, device="cuda"),
                "ws": torch.empty(max(16, need), dtype=torch.uint8, device="cuda")}
    cfg = _cfg(c)
    stack = PrefillStack(cfg, synth.make_model_weights(cfg, seed, device="cuda"))
    ids = torch.from_numpy(synth.make_tokens(cfg, c["n"], seed)).cuda()
    return {"case": c, "stack": stack, "ids": ids, "layers": _bf1_layers(c)}


# ---- one pass -----------------------------------------------------------------

def run(state):
    s, c = state, state["case"]
    if c["kind"] == "attn":
        q, k, v, B, L = s["q"], s["k"], s["v"], c["B"], c["L"]
        if c["entry"] == "fwd":
            return bf1.attn_fwd(q, k, v, B, L)
        if c["entry"] == "plan_csr":
            bf1.plan(c["n"], B, L, s["rp"], s["ci"])
            return bf1.attn_fwd_csr(q, k, v, B, s["rp"], s["ci"], out=s["o"], lse=s["lse"])
        if c["entry"] == "noalloc":
            return bf1.attn_fwd_noalloc(q, k, v, s["o"], s["lse"], B, L)
        if c["entry"] == "sliding":
            return bf1.attn_fwd_csr(q, k, v, B, s["rp"], s["ci"])
        if c["entry"] == "dense":
            return bf1.dense_causal_fwd(q, k, v)
        return bf1.attn_bwd(q, k, v, s["o"], s["do"], s["lse"], B, L, workspace=s["ws"])
    if c["kind"] == "decode":
        if c["replan"]:  # the first token of a block: its pages are listed anew
            bf1.decode_plan(s["sl"], s["table"], s["pages"], s["stride"], c["B"], c["L"], c["dense"], plan=s["plan"])
        return bf1.attn_decode(s["q"], s["kp"], s["vp"], s["sl"], s["plan"], c["B"], out=s["o"], lse=s["lse"],
                               workspace=s["ws"])
    return s["stack"].last_logits(s["ids"], s["layers"])


# ---- the route, written out plainly --------------------------------------------

def _row(j, L):
    """Blocks query block j attends to, ascending, itself last (Eq. 1)."""
    s = {j, 0} | {j - t for t in range(1, L + 1)} | {j - (1 << r) for r in range(2, 40)}
    return sorted(i for i in s if 0 <= i <= j)


def _rows(c, n):
    nb = -(-n // c["B"])
    if c.get("entry") == "dense":
        return [range(j + 1) for j in range(nb)]
    rows = [_row(j, c["L"]) for j in range(nb)]
    if c.get("entry") == "sliding":
        rows = [range(j - len(r) + 1, j + 1) for j, r in enumerate(rows)]
    return rows


def _pairs(c, n):
    """Selected (query, key) pairs per (sequence, q-head)."""
    if c.get("entry") == "dense":
        return n * (n + 1) // 2
    B, total = c["B"], 0
    for j in range(-(-n // B)):
        m = min(B, n - j * B)
        total += m * (len(_row(j, c["L"])) - 1) * B + m * (m + 1) // 2
    return total


def _decode_keys(c, lens):
    """Keys each sequence's newest token attends to."""
    out = []
    for n in lens.tolist():
        j = (n - 1) // c["B"]
        out.append(n if c["dense"] else (len(_row(j, c["L"])) - 1) * c["B"] + (n - 1) % c["B"] + 1)
    return out


def work(case):
    c = case
    if c["kind"] == "attn":
        rows = c["batch"] * c["n"]
        qo, kv = rows * c["Hq"] * c["d"], rows * c["Hkv"] * c["d"]
        pairs = _pairs(c, c["n"]) * c["batch"] * c["Hq"]
        if c["entry"] == "bwd":  # Q, O, dO, K, V and LSE in, fp32 dQ, dK, dV out; five products
            return {"bytes": 2 * (3 * qo + 2 * kv) + 4 * rows * c["Hq"] + 4 * (qo + 2 * kv),
                    "flops": 10 * c["d"] * pairs}
        return {"bytes": 2 * (2 * qo + 2 * kv) + 4 * rows * c["Hq"], "flops": 4 * c["d"] * pairs}
    if c["kind"] == "decode":
        # ragged lengths are drawn from the seed: counted at their mean, 3/4 of the context
        lens = np.full(c["batch"], c["ctx"] * 3 // 4 if c["ragged"] else c["ctx"])
        keys = sum(_decode_keys(c, np.maximum(lens, 1)))
        io = c["batch"] * c["Hq"] * (4 * c["d"] + 4)
        return {"bytes": 4 * keys * c["Hkv"] * c["d"] + io, "flops": 4 * keys * c["Hq"] * c["d"]}
    cfg, n = _cfg(c), c["n"]
    per = sum(int(np.prod(s)) for s in [
        (cfg.hidden, (cfg.heads + 2 * cfg.kv_heads) * cfg.head_dim), (cfg.heads * cfg.head_dim, cfg.hidden),
        (3 * cfg.hidden, cfg.intermediate)])
    nbf1 = len(_bf1_layers(c))
    pairs = nbf1 * _pairs({"B": 64, "L": 2}, n) + (cfg.layers - nbf1) * (n * (n + 1) // 2)
    return {"bytes": 2 * (cfg.layers * per + cfg.vocab * cfg.hidden) + 8 * n + 4 * cfg.vocab,
            "flops": 2 * n * per * cfg.layers + 4 * cfg.head_dim * cfg.heads * pairs + 2 * cfg.vocab * cfg.hidden}


# Two paths of the library that differ only in the order of their fp32 sums
# (the forward's one- and two-key-group forms) are 0.0013-0.0024 (rel) and
# 0.011-0.025 (max) apart in O, and a stack built on them 0.004 sqrt(layers)
# (0.0081 at four layers, 0.025 at 28) and at most five times that (max).
# The backward's gradients are 0.0017 off float64, decode's outputs 0.0017
# (their own bf16 rounding).
def tolerance(case):
    c = case
    if c["kind"] == "model":
        rel = min(0.03, 0.012 * math.sqrt(c["layers"]))
        return {"rel": rel, "max": 6 * rel}
    if c["kind"] == "decode":
        return {"rel": 4e-3, "max": 2e-2}
    if c["entry"] == "bwd":
        return {"rel": 8e-3, "max": 0.1}
    return {"rel": 1e-2, "max": 0.1}


# ---- the same results in 64 bits, in plain torch --------------------------------

def _attn_exact(q, k, v, c, do=None):
    """O and LSE (and dQ, dK, dV for an upstream gradient) in float64."""
    batch, Hq, n, d = q.shape
    Hkv, B = k.shape[1], c["B"]
    G = Hq // Hkv
    scale = 1.0 / math.sqrt(d)
    q = q.double().view(batch, Hkv, G, n, d)
    k, v = k.double(), v.double()
    O = torch.empty_like(q)
    LSE = torch.empty(q.shape[:4], dtype=torch.float64, device=q.device)
    if do is not None:
        do = do.double().view_as(q)
        dq, dk, dv = torch.empty_like(q), torch.zeros_like(k), torch.zeros_like(v)
    for j, row in enumerate(_rows(c, n)):
        t0, t1 = j * B, min(n, (j + 1) * B)
        m = t1 - t0
        if isinstance(row, range):
            idx = torch.arange(row[0] * B, t1, device=q.device)
        else:
            idx = torch.cat([torch.arange(i * B, min(n, (i + 1) * B), device=q.device) for i in row])
        kk, vv = k[:, :, idx], v[:, :, idx]
        qj = q[:, :, :, t0:t1].reshape(batch, Hkv, G * m, d)
        s = torch.matmul(qj, kk.transpose(2, 3).contiguous()) * scale
        pos = torch.arange(t0, t1, device=q.device).repeat(G)
        s.masked_fill_(idx[None, :] > pos[:, None], -math.inf)
        l = torch.logsumexp(s, dim=-1, keepdim=True)
        p = torch.exp(s - l)
        o = torch.matmul(p, vv)
        O[:, :, :, t0:t1] = o.view(batch, Hkv, G, m, d)
        LSE[:, :, :, t0:t1] = l.view(batch, Hkv, G, m)
        if do is not None:
            g = do[:, :, :, t0:t1].reshape(batch, Hkv, G * m, d)
            ds = p * (torch.matmul(g, vv.transpose(2, 3).contiguous()) - (g * o).sum(-1, keepdim=True))
            dq[:, :, :, t0:t1] = (torch.matmul(ds, kk) * scale).view(batch, Hkv, G, m, d)
            dk.index_add_(2, idx, torch.matmul(ds.transpose(2, 3).contiguous(), qj) * scale)
            dv.index_add_(2, idx, torch.matmul(p.transpose(2, 3).contiguous(), g))
    if do is not None:
        return dq.view(batch, Hq, n, d), dk, dv
    return O.view(batch, Hq, n, d), LSE.view(batch, Hq, n)


def _decode_exact(s, c):
    lens = s["sl"].tolist()
    Hkv, G = c["Hkv"], c["Hq"] // c["Hkv"]
    out, lse = [], []
    for b, n in enumerate(lens):
        j = (n - 1) // c["B"]
        row = range(j + 1) if c["dense"] else _row(j, c["L"])
        pages = s["table"][b, torch.tensor(list(row), device="cuda")].long()
        keys = (len(row) - 1) * c["B"] + (n - 1) % c["B"] + 1
        kk = s["kp"][pages].double().transpose(0, 1).reshape(Hkv, -1, c["d"])[:, :keys]
        vv = s["vp"][pages].double().transpose(0, 1).reshape(Hkv, -1, c["d"])[:, :keys]
        q = s["q"][b].double().view(Hkv, G, c["d"])
        sc = torch.matmul(q, kk.transpose(1, 2).contiguous()) / math.sqrt(c["d"])
        l = torch.logsumexp(sc, dim=-1)
        out.append(torch.matmul(torch.exp(sc - l[..., None]), vv).reshape(c["Hq"], c["d"]))
        lse.append(l.reshape(c["Hq"]))
    return torch.stack(out), torch.stack(lse)


def _model_exact(c, seed):
    cfg, n = _cfg(c), c["n"]
    w = synth.make_model_weights(cfg, seed, device="cuda")
    ids = torch.from_numpy(synth.make_tokens(cfg, n, seed)).cuda()
    H, Hkv, d = cfg.heads, cfg.kv_heads, cfg.head_dim
    inv = cfg.rope_theta ** (-torch.arange(0, d, 2, dtype=torch.float64, device="cuda") / d)
    ang = torch.arange(n, dtype=torch.float64, device="cuda")[:, None] * inv
    cos, sin = ang.cos()[:, None, :], ang.sin()[:, None, :]

    def norm(x, g):
        return x * torch.rsqrt(x.pow(2).mean(-1, keepdim=True) + cfg.eps) * g.double()

    def turn(x):
        a, b = x[..., :d // 2], x[..., d // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], dim=-1)

    h = w["embed"][ids].double()
    for l in range(cfg.layers):
        p = {k[len(f"{l}."):]: v for k, v in w.items() if k.startswith(f"{l}.")}
        a = norm(h, p["in_norm"])
        q = turn(norm((a @ p["wq"].double()).view(n, H, d), p["q_norm"])).transpose(0, 1)
        k = turn(norm((a @ p["wk"].double()).view(n, Hkv, d), p["k_norm"])).transpose(0, 1)
        v = (a @ p["wv"].double()).view(n, Hkv, d).transpose(0, 1)
        if l in _bf1_layers(c):
            o = _attn_exact(q[None], k[None].contiguous(), v[None].contiguous(), {"B": 64, "L": 2})[0][0]
        else:
            o = _attn_exact(q[None], k[None].contiguous(), v[None].contiguous(), {"B": 512, "entry": "dense"})[0][0]
        h = h + o.transpose(0, 1).reshape(n, H * d) @ p["wo"].double()
        a = norm(h, p["post_norm"])
        g = a @ p["wg"].double()
        h = h + (g * torch.sigmoid(g) * (a @ p["wu"].double())) @ p["wd"].double()
    return (norm(h[-1:], w["final_norm"]) @ w["embed"].double().t())[0]


def exact(case, seed):
    c = case
    if c["kind"] == "attn":
        g = _gen(seed)
        q, k, v = _qkv(c, g)
        do = _normal(g, *q.shape) if c["entry"] == "bwd" else None
        return _attn_exact(q, k, v, c, do)
    if c["kind"] == "decode":
        return _decode_exact(prepare(c, seed), c)
    return _model_exact(c, seed)
