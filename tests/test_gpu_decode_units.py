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


def _check(lens, Hq, Hkv, d, B, L, dense, seed):
    lens = np.asarray(lens, dtype=np.int32)
    w = synth.DecodeWorkload("units", len(lens), int(lens.max()), Hq, Hkv, d, B, L, seed=seed)
    q, k, v, sl = synth.make_decode_host(w, lens)
    q = q * 3                                   # peaked rows as well as flat ones
    kp, vp, table, pages = synth.page_cache(k, v, sl, B, seed)
    dev = torch.from_numpy(sl).cuda()
    stride = bf1.decode_plan_stride(int(lens.max()), B, L, dense)
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


# units of work below, at and above 64 and 192 (the whole list in one split)
@pytest.mark.parametrize("batch,Hkv", [(1, 1), (16, 4), (13, 5), (95, 2), (24, 8), (65, 4)])
@pytest.mark.parametrize("dense", [False, True])
def test_split_rule_edges(batch, Hkv, dense):
    print("splits", batch, Hkv, dense, flush=True)
    rng = np.random.default_rng(batch)
    _check(rng.integers(1, 1500, size=batch), 2 * Hkv, Hkv, 64, 64, 2, dense, 90 + batch)
