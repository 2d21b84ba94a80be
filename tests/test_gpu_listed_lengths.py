"""Sequences with lengths of their own whose waves are dealt out by the device (rules: tests/test_routes.py): one sequence over many
blocks, several to a block, whole blocks and single waves to a slot, sequences of one token, the fewest slots a call may have."""
import pytest
import torch

import paper_2604_16957_amd as tq
import tq_workloads as wl
from gpu_common import counter_sets_left, errors, gpu_cache_from, listed_slots, make, oracle_cache_from, shared_workspace
from test_gpu_uneven_lengths import _reference, _uneven, check

pytestmark = pytest.mark.gpu


# one sequence; lengths around a tile, a sequence of nothing but its new token among them; two that take whole blocks
@pytest.mark.parametrize("Hq,Hkv,d,group", [(16, 2, 128, 32), (8, 8, 128, 32), (64, 8, 128, 128), (32, 16, 256, 32), (8, 4, 256, 64)])
@pytest.mark.parametrize("lens", [[4097], [1, 2, 31, 32, 33, 34, 64, 65, 1, 96], [2049, 2049], [700, 3, 1500, 40, 1]])
def test_few_sequences(Hq, Hkv, d, group, lens):
    S = max(lens) + 1
    assert listed_slots(len(lens), Hq, Hkv, d, S, group) == 2048 // Hkv
    check(len(lens), Hq, Hkv, d, lens, S, group=group, route="waves dealt")
    check(len(lens), Hq, Hkv, d, lens, S, group=group, page=64, route="waves dealt")


# many sequences to a block, waves of their own; 48 on 32 KV heads: four slots to three of them
@pytest.mark.parametrize("B,Hq,Hkv,d,longest,group,page", [
    (24, 64, 8, 128, 2500, 32, 256), (63, 16, 8, 128, 900, 64, 0), (80, 32, 8, 128, 1100, 32, 0), (48, 32, 32, 128, 2049, 32, 0),
    (40, 32, 16, 256, 900, 32, 0), (40, 16, 16, 256, 900, 128, 32), (256, 8, 1, 128, 1000, 32, 0)])
def test_many_sequences(B, Hq, Hkv, d, longest, group, page):
    assert listed_slots(B, Hq, Hkv, d, longest, group) == 2048 // Hkv
    check(B, Hq, Hkv, d, _uneven(B, longest, 5 + B), longest, group=group, page=page, route="waves dealt")


# max_seq_len only bounds the lengths: the waves are dealt by the lengths alone, so a program that passes its cache's capacity gets
# the same shares, and the same bits, as one that passes the longest length.
@pytest.mark.parametrize("Hq,Hkv,d,lens", [(64, 8, 128, [4000]), (16, 2, 128, [1000, 4000, 2077, 33]), (16, 8, 256, [300, 2999, 1410])])
def test_a_bound_far_above_the_lengths(Hq, Hkv, d, lens):
    B, S, page = len(lens), max(lens), 64
    w = wl.custom(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, seq_len=S, seed=300 + S, outlier_channels=4)
    q, k, v = make(w)
    blocks = -(-S // page)
    cache = tq.KVCache(B * blocks, Hkv, d, page)
    near = torch.randperm(B * blocks, generator=torch.Generator().manual_seed(S)).to(torch.int32).reshape(B, blocks).cuda()
    far = torch.cat([near, torch.zeros(B, 2048 - blocks, dtype=torch.int32, device="cuda")], 1).contiguous()
    tq.tq_quantize_kv_paged(cache, near, k.cuda(), v.cuda(), torch.zeros(B, dtype=torch.int32, device="cuda"))
    lens_dev = torch.tensor(lens, dtype=torch.int32).cuda()
    outs = []
    for table, bound in ((near, S), (far, 131072)):
        assert listed_slots(B, Hq, Hkv, d, bound) == 2048 // Hkv
        outs.append(tq.tq_sdpa_int4_decode_paged(cache, table, q.cuda(), lens_dev, bound, w.attn_scale, workspace=shared_workspace(B, Hq, d)))
    torch.cuda.synchronize()
    assert errors(outs[0], _reference(q, oracle_cache_from(k, v), lens, w.attn_scale, 0))[1] <= 1e-3
    assert torch.equal(outs[0], outs[1])


# Sequences of one or two waves' shares have fewer references of the exponentials than when eight waves shared each, and with one fp16
# operand per weight 12 % more error than then (2.60e-4 for 2.33e-4 on 64 sequences of 128 .. 4096 tokens); their weights go in two parts.  The output's own rounding
# is 2.07e-4, the long sequences' single operand at most 2.56e-4, and the mix of both below 2.33e-4: a bound between that and one operand for all.
def test_short_sequences_weights_in_two_parts():
    B, Hq, Hkv, S = 40, 32, 4, 2000
    w = wl.custom(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, seq_len=S, seed=77, outlier_channels=4)
    q, k, v = make(w)
    lens = [int(round(60 * (S / 60) ** (i / (B - 1)))) for i in range(B)]
    ref = _reference(q, oracle_cache_from(k, v), lens, w.attn_scale, 0)
    cache = gpu_cache_from(k, v)
    out = tq.tq_sdpa_int4_decode_varlen(cache, q.cuda(), torch.tensor(lens, dtype=torch.int32).cuda(), S, w.attn_scale)
    torch.cuda.synchronize()
    assert listed_slots(B, Hq, Hkv, 128, S) == 512
    assert errors(out, ref)[1] <= 2.35e-4


# Sequences of three to seven waves keep one operand, and the error they had with eight waves (grouped by the number of waves 2.46e-4 .. 2.65e-4 either
# way).  The output's rounding, 2.07e-4, and that of the weights (2^-12 at most, evenly spread: 1.4e-4 .. 1.6e-4) make 2.6e-4; an eighth of that for one sequence's spread.
def test_each_sequence_of_three_to_seven_waves():
    B, Hq, Hkv, S = 48, 64, 8, 2500
    w = wl.custom(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, seq_len=S, seed=78, outlier_channels=4)
    q, k, v = make(w)
    lens = [1100 + (S - 1100) * i // (B - 1) for i in range(B)]             # 256 slots for 86 000 tokens: twelve tiles a wave
    ref = _reference(q, oracle_cache_from(k, v), lens, w.attn_scale, 0)
    cache = gpu_cache_from(k, v)
    assert listed_slots(B, Hq, Hkv, 128, S) == 256 and counter_sets_left() > 0
    out = tq.tq_sdpa_int4_decode_varlen(cache, q.cuda(), torch.tensor(lens, dtype=torch.int32).cuda(), S, w.attn_scale,
                                        workspace=shared_workspace(B, Hq, 128))
    torch.cuda.synchronize()
    worst = max(errors(out[b:b + 1], ref[b:b + 1])[1] for b in range(B))
    assert worst <= 2.9e-4, worst
