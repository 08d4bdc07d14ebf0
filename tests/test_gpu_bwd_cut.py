"""GPU checks of how the backward cuts the transposed route: the segment length
follows the work of the call (sequence, batch, heads), and partial tiles lie
in dQ for the short ones.  The cut changes only the order of fp32 sums, so the
gradients of one sequence agree, whatever batch it is in.

Bar: dS, and so dQ, is the same bits.  dK and dV are fp32 sums of the same
terms in another order; with at most some 10^3 partial sums of 64 terms the
difference stays below 2^-24 times a few tens of the largest sum of
magnitudes, allowed here as 1e-5 of the largest gradient.
"""

import pytest
import torch

import paper_2608_20427_amd as bf1

pytestmark = pytest.mark.gpu


def _inputs(batch, n, Hq, Hkv, d, B, L, seed=3):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    q, k, v, do = (torch.randn((batch, h, n, d), generator=g, device="cuda").to(torch.bfloat16)
                   for h in (Hq, Hkv, Hkv, Hq))
    o, lse = bf1.attn_fwd(q, k, v, B, L)
    return q, k, v, o, do, lse


def _bwd(args, B, L):
    q, k = args[0], args[1]
    need = bf1.bwd_workspace_size(q.shape[0], q.shape[2], q.shape[1], k.shape[1], q.shape[3], B, L)
    nan = float("nan")
    return bf1.attn_bwd(*args, B, L, dq=torch.full(q.shape, nan, device="cuda"),
                        dk=torch.full(k.shape, nan, device="cuda"), dv=torch.full(k.shape, nan, device="cuda"),
                        workspace=torch.full((need,), 255, dtype=torch.uint8, device="cuda"))


# sequences of one to some 130 blocks, partial last blocks and sub-tiles, both
# widths and head sizes, every group size
@pytest.mark.parametrize("n,Hq,Hkv,d,B,L", [(1, 2, 1, 64, 64, 2), (64, 2, 1, 128, 64, 2), (65, 2, 1, 64, 64, 0),
                                            (300, 8, 1, 64, 64, 1), (1500, 8, 2, 64, 64, 2), (1030, 4, 2, 128, 64, 2),
                                            (1000, 2, 2, 128, 128, 2), (1473, 4, 1, 64, 128, 3),
                                            (8200, 2, 1, 64, 64, 2)])
def test_cut_follows_the_batch_and_not_the_result(n, Hq, Hkv, d, B, L):
    print("cut", n, Hq, Hkv, d, B, L, flush=True)
    args = _inputs(8, n, Hq, Hkv, d, B, L)
    dq, dk, dv = _bwd(args, B, L)
    for b in (0, 7):
        one = _bwd(tuple(t[b:b + 1].contiguous() for t in args), B, L)
        assert torch.equal(one[0], dq[b:b + 1])
        for a, ref in ((one[1], dk[b:b + 1]), (one[2], dv[b:b + 1])):
            assert torch.isfinite(a).all()
            assert (a - ref).abs().max() <= 1e-5 * ref.abs().max()


def test_every_cut_exists_after_the_first_call():
    # a plan made for one sequence serves a captured call on more of them
    n, B, L = 1337, 64, 2
    one = _inputs(1, n, 4, 2, 64, B, L)
    _bwd(one, B, L)
    many = _inputs(6, n, 4, 2, 64, B, L, seed=4)
    out = [torch.empty(t.shape, device="cuda") for t in (many[0], many[1], many[1])]
    ws = torch.empty(bf1.bwd_workspace_size(6, n, 4, 2, 64, B, L), dtype=torch.uint8, device="cuda")
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        bf1.attn_bwd(*many, B, L, dq=out[0], dk=out[1], dv=out[2], workspace=ws)
    ref = _bwd(many, B, L)
    for _ in range(3):
        for t in out:
            t.fill_(float("nan"))
        ws.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, ref))
