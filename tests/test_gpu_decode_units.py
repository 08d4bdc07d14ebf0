"""GPU checks of the decode kernel's 16-key matrix units and of the split rule:
lengths at the edges of units, pages and tiles, every column-group count (one,
two, four and eight q-heads per kv-head), and (sequence, kv-head) counts on both
sides of each line of the rule, against the float64 oracle.  The unused tail of
a page and the pages nobody owns hold NaN.

Bar, from the arithmetic: weights enter the value product as three bf16 parts
(2^-24 relative), everything else is fp32, so O is within half a bf16 ulp (2^-8
relative) plus some 2^-16 of the largest value; the LSE within 1e-5."""

import numpy as np
import pytest
import torch

import paper_2608_20427_amd as bf1
from oracle import bf1_oracle as orc
from paper_2608_20427_amd import synth

pytestmark = pytest.mark.gpu

EDGES = [1, 15, 16, 17, 48, 49, 63, 64, 65, 80, 127, 128, 129, 200]


def _check(lens, Hq, Hkv, d, B, L, dense, seed, row=0):
    lens = np.asarray(lens, dtype=np.int32)
    w = synth.DecodeWorkload("units", len(lens), int(lens.max()), Hq, Hkv, d, B, L, seed=seed)
    q, k, v, sl = synth.make_decode_host(w, lens)
    q = q * 3                                   # peaked rows as well as flat ones
    kp, vp, table, pages = synth.page_cache(k, v, sl, B, seed)
    dev = torch.from_numpy(sl).cuda()
    stride = bf1.decode_plan_stride(max(row, int(lens.max())), B, L, dense)
    plan = bf1.decode_plan(dev, table.cuda(), pages, stride, B, L, dense)
    need = bf1.decode_workspace_size(len(lens), Hq, Hkv, d, stride)
    ws = torch.full((max(16, need),), 255, dtype=torch.uint8, device="cuda")
    o, lse = bf1.attn_decode(q.cuda(), kp.cuda(), vp.cuda(), dev, plan, B, workspace=ws)
    torch.cuda.synchronize()
    # dense: every earlier block, which is the route with every block local
    ref, lref = orc.attn_decode_fp64(synth.to_f64(q), synth.to_f64(k), synth.to_f64(v), sl, B,
                                     int(lens.max()) if dense else L)
    o, lse = o.cpu().double().numpy(), lse.cpu().double().numpy()
    assert np.isfinite(o).all() and np.isfinite(lse).all()
    assert (np.abs(o - ref) <= 2.0 ** -8 * np.abs(ref) + 2.0 ** -16 * 5).all()
    assert np.abs(lse - lref).max() <= 1e-5 * max(1.0, np.abs(lref).max())


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("d,B", [(64, 64), (128, 64), (64, 128), (128, 128)])
def test_unit_edges(G, d, B):
    print("units", G, d, B, flush=True)
    _check(EDGES, 2 * G, 2, d, B, 2, False, 40 + G + d + B)


# units of work below, at and above 64, 192 and 256 (the whole list in one split)
@pytest.mark.parametrize("batch,Hkv", [(1, 1), (16, 4), (13, 5), (95, 2), (24, 8), (65, 4)])
@pytest.mark.parametrize("dense", [False, True])
def test_split_rule_edges(batch, Hkv, dense):
    print("splits", batch, Hkv, dense, flush=True)
    rng = np.random.default_rng(batch)
    _check(rng.integers(1, 1500, size=batch), 2 * Hkv, Hkv, 64, 64, 2, dense, 90 + batch)


# lists over 32 pages with few kv-heads: several rounds of the merge, and lists of
# several lengths (one page, one round and both sides of it) in rows of one length,
# also rows that could hold far more (131072 tokens: 2048 pages)
@pytest.mark.parametrize("lens", [[4500], [70, 1, 64 * 16, 64 * 17, 64 * 64, 64 * 65 + 1]])
@pytest.mark.parametrize("G,d", [(1, 64), (2, 128), (8, 128)])
@pytest.mark.parametrize("row", [0, 131072])
def test_long_lists(lens, G, d, row):
    print("long lists", lens, G, d, row, flush=True)
    _check(lens, G, 1, d, 64, 2, True, 120 + len(lens), row)


@pytest.mark.parametrize("G", [1, 2, 4, 8])
@pytest.mark.parametrize("d,B,batch", [(64, 64, 1), (128, 64, 1), (128, 128, 1), (128, 64, 100)])
def test_infinite_values(G, d, B, batch):
    # A visible value row with an infinity gives that infinity in its dim (its
    # weight is positive whatever it rounds to), both signs or a NaN give NaN,
    # and the other dims stay what they are.  With 100 sequences the lists are
    # not cut; with one they are, and the merge sees the infinities as well.
    # Bar of the finite entries as above.
    print("infinite values", G, d, B, batch, flush=True)
    Hkv, inf = 2, float("inf")
    lens = np.full(batch, 5 * B + 21, dtype=np.int32)
    lens[0] = 5 * B + 1
    w = synth.DecodeWorkload("inf", batch, int(lens.max()), Hkv * G, Hkv, d, B, 2, seed=70 + G)
    q, k, v, sl = synth.make_decode_host(w, lens)
    # newest token in block 5: blocks 0, 1, 3, 4 and 5 are selected
    for b in range(batch):
        n = int(lens[b])
        v[b, :, 3, 0] = inf                                  # first unit of the first page
        v[b, :, B + 20, 1] = -inf                            # another wave
        v[b, :, n - 1, 2] = inf                              # the newest key
        v[b, :, 5, 3], v[b, :, 4 * B + 40, 3] = inf, -inf    # NaN
        v[b, :, 3 * B + B - 1, 4] = float("nan")
        v[b, :, 2 * B:3 * B, 5] = inf                        # not selected
        v[b, 0, :n, d - 1] = inf                             # every key, one kv-head
    kp, vp, table, pages = synth.page_cache(k, v, sl, B, 70)
    dev = torch.from_numpy(sl).cuda()
    stride = bf1.decode_plan_stride(int(lens.max()), B, 2)
    plan = bf1.decode_plan(dev, table.cuda(), pages, stride, B, 2)
    o, lse = bf1.attn_decode(q.cuda(), kp.cuda(), vp.cuda(), dev, plan, B)
    torch.cuda.synchronize()
    assert list(orc.route(5, 2)) == [0, 1, 3, 4, 5]
    with np.errstate(invalid="ignore"):
        ref, lref = orc.attn_decode_fp64(synth.to_f64(q), synth.to_f64(k), synth.to_f64(v), sl, B, 2)
    o, lse = o.cpu().double().numpy(), lse.cpu().double().numpy()
    assert np.isinf(ref[:, :, :3]).all() and np.isnan(ref[:, :, 3:5]).all() and np.isfinite(ref[:, :, 5]).all()
    assert np.array_equal(np.isnan(o), np.isnan(ref))
    assert np.array_equal(np.where(np.isinf(o), o, 0), np.where(np.isinf(ref), ref, 0))
    fin = np.isfinite(ref)
    assert (np.abs(o[fin] - ref[fin]) <= 2.0 ** -8 * np.abs(ref[fin]) + 2.0 ** -16 * 5).all()
    assert np.abs(lse - lref).max() <= 1e-5 * max(1.0, np.abs(lref).max())


@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_infinite_value_at_a_tiny_weight(G):
    # The key with the infinity scores 20 to 150 powers of two below the others.
    # A fp32 weight is positive down to 2^-149 (times V: infinite), zero below.
    print("tiny weights", G, flush=True)
    d, B, n = 64, 64, 130
    for at in (-20.0, -40.0, -43.0, -45.0, -47.0, -50.0, -52.0):
        q, kp, vp = torch.zeros(1, G, d), torch.zeros(3, 1, B, d), torch.ones(3, 1, B, d)
        q[..., 0], kp[0, 0, 7, 0], vp[0, 0, 7, 0] = 16.0, at, float("inf")
        q, kp, vp = (t.to(torch.bfloat16).cuda() for t in (q, kp, vp))
        sl = torch.tensor([n], dtype=torch.int32, device="cuda")
        table = torch.tensor([[0, 1, 2]], dtype=torch.int32, device="cuda")
        plan = bf1.decode_plan(sl, table, 3, bf1.decode_plan_stride(n, B, 2), B, 2)
        o, lse = bf1.attn_decode(q, kp, vp, sl, plan, B)
        o, lse = o.float().cpu(), lse.cpu()
        power = 16 * at / d ** 0.5 / np.log(2)            # log2 of the weight
        assert (torch.isinf(o[..., 0]) & (o[..., 0] > 0)).all() if power > -149 else torch.isnan(o[..., 0]).all()
        assert (o[..., 1:] == 1).all() and (lse - np.log(n - 1)).abs().max() <= 1e-5 * np.log(n)
