"""The prefill stack on the CPU: without BF1 layers and with a caller's dense
attention it runs operator by operator on any device."""

import torch

from oracle import model_oracle as mo
from paper_2608_20427_amd import synth
from paper_2608_20427_amd.prefill_model import PrefillStack


def test_stack_runs_on_the_cpu_with_a_dense_callable():
    cfg = synth.ModelConfig(layers=2, hidden=96, heads=4, kv_heads=2, head_dim=32, intermediate=160, vocab=300)
    w = synth.make_model_weights(cfg, 3)
    ids = synth.make_tokens(cfg, 50, 9)

    def dense(Q, K, V):
        Q, K, V = Q.float(), K.float().repeat_interleave(2, 1), V.float().repeat_interleave(2, 1)
        s = Q @ K.transpose(2, 3) / Q.shape[-1] ** 0.5
        s = s.masked_fill(torch.ones(50, 50).triu(1).bool(), float("-inf"))
        return (s.softmax(-1) @ V).to(torch.bfloat16)
    got = PrefillStack(cfg, w, device="cpu").last_logits(torch.from_numpy(ids), set(), dense).double().numpy()
    ref = mo.prefill_last_logits_fp64(ids, {k: v.double().numpy() for k, v in w.items()}, cfg, set())
    # bf16 activations rounded after every operator (2^-8 each, two layers)
    assert abs(got - ref).max() <= 5e-2 * abs(ref).max()
