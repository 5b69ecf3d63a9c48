"""The attention's work list and split sequences: partition lengths from the
shortest on, sequences that end at a partition boundary or one token past it,
several planning workgroups, lone waves and shared items. Each case states the
cut it is for. Compared with the oracle as the other attention cases are."""

import numpy as np
import pytest
import torch

import synth
from gpu_helpers import assert_bf16_within_ulp, kernels_of
from test_gpu_kernels import _attn_oracle, _attn_run, _attn_setup

pytestmark = pytest.mark.gpu


def _mixed(n, hi, seed):
    return np.random.default_rng(seed).integers(1, hi + 1, n).tolist()


WHOLE = 1 << 20


# part, waves, combine: the cut that the case is meant to exercise (sidp_attention_plan)
@pytest.mark.parametrize("hq,hkv,d,seqs,part,waves,combine", [
    (4, 2, 64, [2000], 256, 0, 1),                                      # shortest partitions, seven and a rest
    (8, 1, 128, [768, 769, 1024, 1025, 256, 257, 1, 255], 256, 0, 1),   # ends at and past partition boundaries
    (8, 1, 128, [511, 512, 513, 767], WHOLE, 0, 0),                     # tables short enough for one launch
    (16, 1, 128, [5000, 17, 3000], 256, 0, 1),                          # the largest group
    (64, 8, 128, [4096, 8192, 4097, 5000, 6143], 1024, 0, 1),
    (4, 2, 64, _mixed(65, 1500, 1), WHOLE, 0, 0),                       # two planning workgroups, the second with one sequence
    (4, 2, 64, _mixed(300, 2500, 2), 3072, 0, 1),                       # five, per-thread runs of two sequences; no record
    (4, 2, 64, [1] * 70 + [9000] + [2] * 70, 256, 0, 1),                # one long sequence among short ones
    (2, 1, 64, _mixed(700, 900, 3), WHOLE, 0, 0),                       # many whole sequences
    (64, 8, 128, _mixed(130, 300, 4), WHOLE, 1, 0),                     # a wave an item, uneven waves
    (16, 1, 128, _mixed(600, 290, 5), WHOLE, 1, 0),                     # a wave an item, the largest group
    (16, 1, 128, _mixed(600, 700, 5), WHOLE, 0, 0),                     # too long for that
    (8, 2, 64, _mixed(400, 1000, 6) + [1, 15, 16, 17, 31, 32, 33, 5000], 2048, 0, 1),  # mostly whole, some partitions
    (16, 8, 64, [64] * 200 + [8192, 8191, 769, 768, 767], 1024, 0, 1),  # partitions a little too long for lone waves
    (16, 8, 64, [64] * 200 + [8192, 769, 768, 767], 768, 1, 1),         # a wave an item, some of them partitions
    (64, 8, 128, _mixed(255, 64, 7) + [8192], WHOLE, 0, 0),             # whole sequences, one long among 255 short
    (16, 8, 64, [40] * 255 + [1024], WHOLE, 1, 0),                      # the longest sequence that a lone wave takes there
    (16, 8, 64, [40] * 255 + [1025], WHOLE, 0, 0),                      # and one token more
    (16, 8, 64, [3000, 2999, 3072], 384, 0, 1),                         # the next length over the mean's
    (16, 8, 64, _mixed(20, 2000, 8) + [2048], WHOLE, 0, 0),             # whole sequences on fewer items than workgroups
])
def test_split_attention_parity(lib, hq, hkv, d, seqs, part, waves, combine):
    cfg = synth.get_config("tiny_layer", num_q_heads=hq, num_kv_heads=hkv, head_dim=d)
    ctx, tables, nblk, k, v, q, maxb = _attn_setup(lib, cfg, seqs)
    plan = lib.sidp_attention_plan(ctx, maxb, hkv, torch.cuda.get_device_properties(0).multi_processor_count)
    assert (plan["part_tokens"], plan["wave_items"], plan["combine"]) == (part, waves, combine)
    got = _attn_run(lib, cfg, ctx, tables, nblk, k, v, q, maxb)
    want = _attn_oracle(cfg, ctx, tables, k, v, q)
    pv = _attn_oracle(cfg, ctx, tables, k, v, q, absv=True)
    assert_bf16_within_ulp(got, want, what=f"split attention {hq}/{hkv} x {d}", abs_tol=2.0 ** -12 * pv)


@pytest.mark.parametrize("batch,tokens,split", [(24, 1500, 0), (12, 1024, 0), (11, 1024, 1), (20, 2049, 1)])
def test_combine_is_launched_only_for_split_sequences(lib, batch, tokens, split):
    cfg = synth.get_config("tiny_layer", num_q_heads=8, num_kv_heads=8, head_dim=64)
    maxb = -(-tokens // 16)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert lib.sidp_attention_plan([tokens - 1] * batch, maxb, 8, cus)["combine"] == split
    nblk = batch * maxb
    h = lib.sidp_create(lib.make_config(dict(cfg, num_layers=1), batch, maxb * 16))
    try:
        kc = torch.zeros(nblk, 8, 8, 16, 8, dtype=torch.bfloat16, device="cuda")
        vc = torch.zeros(nblk, 8, 64, 16, dtype=torch.bfloat16, device="cuda")
        lib.sidp_kv_attach(h, kc, vc, nblk, 1)
        bt = torch.arange(nblk, dtype=torch.int32, device="cuda").view(batch, maxb)
        pos = torch.full((batch,), tokens - 1, dtype=torch.int32, device="cuda")
        q = torch.ones(batch, 8, 64, dtype=torch.bfloat16, device="cuda")
        out = torch.empty_like(q)
        ran = kernels_of(lambda: lib.sidp_attention(h, q, 0, pos, bt, maxb, batch, out))
        assert sum("k_attn" in name for name in ran) == 2 + split, ran  # plan, attention, combine
        assert any("k_attn_combine" in name for name in ran) == bool(split), ran
        lib.sidp_sync(h)
    finally:
        lib.sidp_destroy(h)
