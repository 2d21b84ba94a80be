"""The matrix-core kernel for many query rows per KV head: where its rounds, tiles and references can go wrong."""
import pytest
import torch

import paper_2604_16957_amd as tq
import tq_workloads as wl
from gpu_common import assert_close, gpu_cache_from, make, oracle_attend, oracle_cache_from

pytestmark = pytest.mark.gpu

# a wave scores 16 tokens of a round of 128; a supertile of 32 is the unit of P V
LENGTHS = {512: (15, 16, 17, 31, 48, 65, 112, 127, 128, 129, 144, 145, 255, 257, 300)}


def _poisoned(k, v, S):
    """The cache of S tokens in a larger one, NaN in every scale and zero-point behind them."""
    cache = gpu_cache_from(k, v, capacity=S + 40)
    for t in cache.tensors():
        if t.dtype == torch.float16:
            t[:, :, S:] = float("nan")
    return cache


@pytest.mark.parametrize("heads", [(1, 1), (17, 1), (34, 2), (20, 1)])
@pytest.mark.parametrize("head_dim", [512])
def test_rounds_and_their_remainders(head_dim, heads):
    """Every remainder of a round, in one chunk and in two: waves without tokens, half supertiles, rows of a last tile
    that has few; nothing behind the sequence's end is used."""
    for S in LENGTHS[head_dim]:
        w = wl.custom(n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=head_dim, seq_len=S, attn_scale=1.0, qk_std=0.1,
                      v_std=0.5, seed=2100 + S)
        q, k, v = make(w)
        cache, ocache = _poisoned(k, v, S), oracle_cache_from(k, v)
        ref = oracle_attend(q, ocache, S, w.attn_scale)
        for n_splits in (0, 1, 2):
            out = tq.tq_sdpa_int4_decode(cache, q.cuda(), S, w.attn_scale, n_splits=n_splits)
            torch.cuda.synchronize()
            assert_close(out, ref, f"d={head_dim} {heads} S={S} n_splits={n_splits}")


@pytest.mark.parametrize("head_dim", [512])
def test_references_that_move_in_every_round(head_dim):
    """Scores that grow along the sequence: the rows' references move round after round, by another wave each time."""
    S = 1000
    w = wl.custom(n_q_heads=20, n_kv_heads=1, head_dim=head_dim, seq_len=S, attn_scale=1.0, qk_std=0.1, seed=2200)
    q, k, v = make(w)
    ramp = torch.linspace(0.2, 6.0, S).reshape(1, 1, S, 1)
    k = (k.float() * ramp).half()
    ocache = oracle_cache_from(k, v)
    cache = gpu_cache_from(k, v)
    for n_splits in (1, 3):
        out = tq.tq_sdpa_int4_decode(cache, q.cuda(), S, w.attn_scale, n_splits=n_splits)
        torch.cuda.synchronize()
        assert_close(out, oracle_attend(q, ocache, S, w.attn_scale), f"d={head_dim} n_splits={n_splits}")


@pytest.mark.parametrize("scale", [-0.7, 0.0, 1.0e-6])
def test_any_finite_scale_at_512(scale):
    S = 333
    w = wl.custom(n_q_heads=8, n_kv_heads=1, head_dim=512, seq_len=S, attn_scale=1.0, qk_std=0.1, seed=2300)
    q, k, v = make(w)
    out = tq.tq_sdpa_int4_decode(gpu_cache_from(k, v), q.cuda(), S, scale)
    torch.cuda.synchronize()
    assert_close(out, oracle_attend(q, oracle_cache_from(k, v), S, scale), f"scale={scale}")
