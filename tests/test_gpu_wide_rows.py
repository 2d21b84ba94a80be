"""The matrix-core kernel for many query rows per KV head: where its rounds, tiles and references can go wrong."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_16957_amd as tq
import tq_workloads as wl
from gpu_common import (assert_cache_bit_exact, assert_close, assert_close_elementwise, gpu_cache_from, kernel_of, make, np16, oracle_attend, oracle_cache_from)

pytestmark = pytest.mark.gpu

# a wave scores 16 tokens of a round of 128 (head_dim 256 and 128: 32 of 256); a supertile of 32 is the unit of P V
LENGTHS = {512: (15, 16, 17, 31, 48, 65, 112, 127, 128, 129, 144, 145, 255, 257, 300),
           128: (2, 31, 33, 65, 97, 161, 225, 255, 256, 257, 300, 513),
           256: (2, 31, 32, 33, 65, 96, 224, 225, 255, 256, 257, 289, 511, 513, 600)}


# At head_dim 256 the kernel takes small calls with several query tokens only (at 128: also with nine rows and more).
QUERIES = {512: 1, 256: 2, 128: 2}


def _poisoned(k, v, S):
    """The cache of S tokens in a larger one, NaN in every scale and zero-point behind them."""
    cache = gpu_cache_from(k, v, capacity=S + 40)
    for t in cache.tensors():
        if t.dtype == torch.float16:
            t[:, :, S:] = float("nan")
    return cache


def _queries(w, nq):
    gen = torch.Generator().manual_seed(w.seed + 1)
    q = (torch.randn(w.batch, nq, w.n_q_heads, w.head_dim, generator=gen) * 0.1).half()
    return q if nq > 1 else q[:, 0].contiguous()


def _reference(q, ocache, S, alpha):
    if q.dim() == 3:
        return oracle_attend(q, ocache, S, alpha)
    nq = q.shape[1]
    return np.stack([oracle.attend_packed(np16(q[:, t]), *ocache, seq_len=S - (nq - 1 - t), alpha=alpha) for t in range(nq)], axis=1)


@pytest.mark.parametrize("heads", [(5, 1), (17, 1), (34, 2), (20, 1)])
@pytest.mark.parametrize("head_dim", [128, 256, 512])
def test_rounds_and_their_remainders(head_dim, heads):
    """Every remainder of a round, in one chunk and in two: waves without tokens, half supertiles, rows of a last tile
    that has few; nothing behind the sequence's end is used."""
    nq = QUERIES[head_dim]
    for S in LENGTHS[head_dim]:
        w = wl.custom(n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=head_dim, seq_len=S, attn_scale=1.0, qk_std=0.1,
                      v_std=0.5, seed=2100 + S)
        _, k, v = make(w)
        q = _queries(w, nq)
        cache, ocache = _poisoned(k, v, S), oracle_cache_from(k, v)
        ref = _reference(q, ocache, S, w.attn_scale)
        assert kernel_of(1, *heads, head_dim, S, n_queries=nq) == "wide rows"
        for n_splits in (0, 1, 2):
            out = tq.tq_sdpa_int4_decode(cache, q.cuda(), S, w.attn_scale, n_splits=n_splits)
            torch.cuda.synchronize()
            assert_close(out, ref, f"d={head_dim} {heads} S={S} n_splits={n_splits}")


@pytest.mark.parametrize("head_dim", [128, 256, 512])
def test_references_that_move_in_every_round(head_dim):
    """Scores that grow along the sequence: the rows' references move round after round, by another wave each time."""
    S = 1000
    w = wl.custom(n_q_heads=20, n_kv_heads=1, head_dim=head_dim, seq_len=S, attn_scale=1.0, qk_std=0.1, seed=2200)
    _, k, v = make(w)
    q = _queries(w, QUERIES[head_dim])
    k = (k.float() * torch.linspace(0.2, 6.0, S).reshape(1, 1, S, 1)).half()
    ocache = oracle_cache_from(k, v)
    cache = gpu_cache_from(k, v)
    for n_splits in (1, 3):
        out = tq.tq_sdpa_int4_decode(cache, q.cuda(), S, w.attn_scale, n_splits=n_splits)
        torch.cuda.synchronize()
        assert_close(out, _reference(q, ocache, S, w.attn_scale), f"d={head_dim} n_splits={n_splits}")


@pytest.mark.parametrize("kind", ["fixed", "lengths", "paged"])
def test_eight_rows_at_256_with_one_query_token(kind):
    """The smallest calls with one query token that take this kernel at head_dim 256, next to ones that do not: same result."""
    for S, B in ((3072, 1), (3071, 1), (1100, 3)):
        w = wl.custom(batch=B, n_q_heads=32, n_kv_heads=4, head_dim=256, seq_len=S, attn_scale=1.0, qk_std=0.1, seed=2500 + S)
        q, k, v = make(w)
        ocache = oracle_cache_from(k, v)
        lens = [S - 37 * b for b in range(B)]
        ref = np.concatenate([oracle.attend_packed(np16(q[b:b + 1]), *[np.ascontiguousarray(a[b:b + 1]) for a in ocache],
                                                   seq_len=n if kind != "fixed" else S, alpha=1.0) for b, n in enumerate(lens)])
        lens = torch.tensor(lens, dtype=torch.int32).cuda()
        if kind == "paged":
            pages = -(-S // 64)
            pool = tq.KVCache(B * pages, 4, 256, 64)
            table = torch.randperm(B * pages, generator=torch.Generator().manual_seed(S)).to(torch.int32).reshape(B, pages).cuda()
            tq.tq_quantize_kv_paged(pool, table, k.cuda(), v.cuda(), torch.zeros(B, dtype=torch.int32).cuda())
            out = tq.tq_sdpa_int4_decode_paged(pool, table, q.cuda(), lens, S, 1.0)
        else:
            cache = gpu_cache_from(k, v)
            out = (tq.tq_sdpa_int4_decode(cache, q.cuda(), S, 1.0) if kind == "fixed" else
                   tq.tq_sdpa_int4_decode_varlen(cache, q.cuda(), lens, S, 1.0))
        torch.cuda.synchronize()
        assert_close(out, ref, f"{kind} S={S} B={B}")


@pytest.mark.parametrize("scale", [-0.7, 0.0, 1.0e-6])
def test_any_finite_scale_at_512(scale):
    S = 333
    w = wl.custom(n_q_heads=8, n_kv_heads=1, head_dim=512, seq_len=S, attn_scale=1.0, qk_std=0.1, seed=2300)
    q, k, v = make(w)
    out = tq.tq_sdpa_int4_decode(gpu_cache_from(k, v), q.cuda(), S, scale)
    torch.cuda.synchronize()
    assert_close(out, oracle_attend(q, oracle_cache_from(k, v), S, scale), f"scale={scale}")


@pytest.mark.parametrize("head_dim,scales", [(128, (1e-38, 1e-44)), (256, (1e-38, 1e-44)), (512, (1e-38, 1e-44, -1e-38, -1e-44))])
def test_scales_of_the_smallest_size(head_dim, scales):
    """Scales down to fp32's subnormals: every token weighs the same (on whichever kernel the call takes)."""
    S = 333
    for heads, nq in (((8, 1), 1), ((2, 1), 1), ((9, 1), 2)):
        w = wl.custom(n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=head_dim, seq_len=S, attn_scale=1.0, seed=2350)
        _, k, v = make(w)
        q, ocache, cache = _queries(w, nq), oracle_cache_from(k, v), gpu_cache_from(k, v)
        for scale in scales:
            out = tq.tq_sdpa_int4_decode(cache, q.cuda(), S, scale)
            torch.cuda.synchronize()
            assert_close(out, _reference(q, ocache, S, scale), f"d={head_dim} {heads} nq={nq} scale={scale}")


@pytest.mark.parametrize("head_dim,nq", [(128, 1), (128, 2), (128, 3), (128, 8), (256, 2), (256, 5), (256, 8), (512, 1), (512, 2), (512, 8)])
def test_new_tokens_across_tiles_and_chunks(head_dim, nq):
    """A step's new tokens at every place of a supertile, across two of them and across two chunks: stored bit for bit, attended,
    and nothing that the cache held in their place (NaN here) is used."""
    for S in (nq, nq + 1, 17, 31 + nq // 2, 32, 64 + nq - 1, 65, 96 + nq // 2, 130, 257, 260):
        if S < nq:
            continue
        for n_splits in (0, 3):
            w = wl.custom(batch=2, n_q_heads=18, n_kv_heads=2, head_dim=head_dim, seq_len=S, attn_scale=1.0, qk_std=0.1,
                          v_std=0.5, seed=2400 + S)
            _, k, v = make(w)
            gen = torch.Generator().manual_seed(S)
            q = (torch.randn(2, nq, 18, head_dim, generator=gen) * 0.1).half()
            ocache = oracle_cache_from(k, v)
            cache = tq.KVCache(2, 2, head_dim, S + 40)
            for t in cache.tensors():
                t.fill_(float("nan")) if t.dtype == torch.float16 else t.fill_(0xEE)
            if S > nq:
                tq.tq_quantize_kv(cache, k[:, :, :S - nq].contiguous().cuda(), v[:, :, :S - nq].contiguous().cuda(), 0)
            kn, vn = k[:, :, S - nq:].contiguous().cuda(), v[:, :, S - nq:].contiguous().cuda()
            qd = q.cuda() if nq > 1 else q[:, 0].contiguous().cuda()
            out = tq.tq_sdpa_int4_append_decode(cache, kn, vn, qd, S, w.attn_scale, n_splits=n_splits)
            torch.cuda.synchronize()
            assert_cache_bit_exact(cache, ocache, S)
            for t in cache.tensors():
                rest = t[:, :, S:]
                assert bool(torch.isnan(rest).all() if t.dtype == torch.float16 else (rest == 0xEE).all())
            rows = [oracle.attend_packed(np16(q[:, t]), *ocache, seq_len=S - (nq - 1 - t), alpha=1.0) for t in range(nq)]
            ref = np.stack(rows, axis=1) if nq > 1 else rows[0]
            assert_close(out, ref, f"d={head_dim} nq={nq} S={S} n_splits={n_splits}")


# heads, query tokens, the last length of one sequence whose step (decode) is on this kernel
@pytest.mark.parametrize("heads,nq,last,of", [((4, 4), 2, 32063, "step"), ((12, 4), 2, 61503, "step"), ((8, 2), 2, 123007, "step"),
                                              ((24, 3), 3, 106751, "step"), ((24, 3), 3, 51285, "decode"), ((32, 4), 2, 115263, "step"),
                                              ((32, 4), 2, 76863, "decode"), ((64, 4), 1, 70463, "step"), ((64, 4), 1, 57663, "decode")])
def test_steps_and_decodes_around_the_line_at_128(heads, nq, last, of):
    """Two to 24 rows per KV head: the last length that the kernel is chosen for by its load, and the next: step and decode agree with the
    oracle, on whichever kernel each is."""
    for S in (last, last + 1):
        assert (kernel_of(1, *heads, 128, S, of, n_queries=nq) == "wide rows") == (S == last)
        w = wl.custom(n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=128, seq_len=S, seed=2600 + nq)
        _, k, v = make(w)
        q = torch.randn(1, nq, heads[0], 128, generator=torch.Generator().manual_seed(S)).half()
        q = q if nq > 1 else q[:, 0].contiguous()
        ocache = oracle_cache_from(k, v)
        cache = gpu_cache_from(k[:, :, :S - nq].contiguous(), v[:, :, :S - nq].contiguous(), capacity=S + 1)
        out = tq.tq_sdpa_int4_append_decode(cache, k[:, :, S - nq:].contiguous().cuda(), v[:, :, S - nq:].contiguous().cuda(), q.cuda(),
                                            S, w.attn_scale)
        torch.cuda.synchronize()
        assert_cache_bit_exact(cache, ocache, S)
        again = tq.tq_sdpa_int4_decode(cache, q.cuda(), S, w.attn_scale)
        torch.cuda.synchronize()
        ref = _reference(q, ocache, S, w.attn_scale)
        assert_close_elementwise(out, ref, f"step {heads} nq={nq} S={S}")
        assert_close_elementwise(again, ref, f"decode {heads} nq={nq} S={S}")


@pytest.mark.parametrize("heads,nq", [((4, 4), 2), ((12, 4), 2), ((8, 2), 2), ((24, 3), 3)])
def test_steps_of_several_query_tokens_at_128(heads, nq):
    """Two to 24 rows per KV head, steps on this kernel (their decodes with up to eight rows on the other): both agree with the oracle,
    under a window too."""
    for S, window in ((nq, 0), (70, 0), (1500, 0), (1500, 100), (66000 // heads[1], 0)):
        assert kernel_of(1, *heads, 128, S, "step", n_queries=nq, window=window) == "wide rows"
        w = wl.custom(n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=128, seq_len=S, seed=2600 + S)
        _, k, v = make(w)
        q = (torch.randn(1, nq, heads[0], 128, generator=torch.Generator().manual_seed(S))).half()
        ocache = oracle_cache_from(k, v)
        cache = gpu_cache_from(k[:, :, :max(1, S - nq)].contiguous(), v[:, :, :max(1, S - nq)].contiguous(), capacity=S + 1)
        out = tq.tq_sdpa_int4_append_decode(cache, k[:, :, S - nq:].contiguous().cuda(), v[:, :, S - nq:].contiguous().cuda(), q.cuda(),
                                            S, w.attn_scale, window=window)
        torch.cuda.synchronize()
        assert_cache_bit_exact(cache, ocache, S)
        again = tq.tq_sdpa_int4_decode(cache, q.cuda(), S, w.attn_scale, window=window)
        torch.cuda.synchronize()
        rows = []
        for t in range(nq):
            n = S - (nq - 1 - t)
            lo = max(0, n - window) if window else 0
            part = [np.ascontiguousarray(a[:, :, lo:n]) for a in ocache]
            rows.append(oracle.attend_packed(np16(q[:, t]), *part, seq_len=n - lo, alpha=w.attn_scale))
        ref = np.stack(rows, axis=1)
        assert_close_elementwise(out, ref, f"step {heads} nq={nq} S={S} window={window}")
        assert_close_elementwise(again, ref, f"decode {heads} nq={nq} S={S} window={window}")


def _spread_inputs(head_dim, heads, S, nq, sigma, v_std, seed):
    """Scores of a Gaussian spread of sigma (attention scale 1), V of spread v_std (a number, or one per element of the head)."""
    gen = torch.Generator().manual_seed(seed)
    shape = (1, heads[1], S, head_dim)
    k = torch.randn(shape, generator=gen).half()
    v = (torch.randn(shape, generator=gen) * torch.as_tensor(v_std)).half()
    q = (torch.randn(1, nq, heads[0], head_dim, generator=gen) * (sigma / head_dim ** 0.5)).half()
    return (q if nq > 1 else q[:, 0].contiguous()), k, v


def _assert_weights_whole(out, ref, dims, what):
    """The relative error (2-norm) over `dims` of the head: the output's own fp16 rounding, as it falls on this reference, and one fp16
    rounding of every weight, 2^-10 / sqrt(12) of a weight's power of two, sqrt(1/2) of that relative to a weight on average, independent from
    token to token like V; a quarter on top of both for the fp32 arithmetic and for chance."""
    ref = ref[..., dims]
    err = np.linalg.norm(np16(out).astype(np.float64)[..., dims] - ref) / np.linalg.norm(ref)
    own = np.linalg.norm(ref.astype(np.float16).astype(np.float64) - ref) / np.linalg.norm(ref)
    bar = 1.25 * np.hypot(own, 2.0 ** -10 / 24 ** 0.5)
    assert err <= bar, f"{what}: {err:.2e} over {bar:.2e} (the output's rounding {own:.2e})"


@pytest.mark.parametrize("v_std", [30.0, 1.0, 1e-2, 1e-3, 1e-4])
@pytest.mark.parametrize("head_dim", [128, 256, 512])
def test_weights_keep_their_bits_whatever_the_size_of_v(head_dim, v_std):
    """P V takes fp16 operands p s_v: they stay in fp16's normal range for large scales of V and for small ones, flat softmax or sharp."""
    nq = QUERIES[head_dim]
    for heads, S, n_splits, sigma in (((2, 1), 300, 0, 2.0), ((16, 1), 2000, 0, 0.3), ((32, 2), 2000, 1, 2.0), ((9, 1), 5000, 4, 2.0)):
        if head_dim == 128 and heads == (2, 1):
            heads = (9, 1)                          # (up to eight rows the kernel takes steps only)
        assert kernel_of(1, *heads, head_dim, S, n_queries=nq) == "wide rows"
        q, k, v = _spread_inputs(head_dim, heads, S, nq, sigma, v_std, 2700 + S)
        out = tq.tq_sdpa_int4_decode(_poisoned(k, v, S), q.cuda(), S, 1.0, n_splits=n_splits)
        torch.cuda.synchronize()
        _assert_weights_whole(out, _reference(q, oracle_cache_from(k, v), S, 1.0), slice(None), f"d={head_dim} {heads} S={S} v_std={v_std}")


@pytest.mark.parametrize("head_dim", [128, 256, 512])
def test_the_longest_chunk_a_plan_makes(head_dim):
    """16384 tokens in one chunk: what the accumulators pick up over its 512 (256, 128) tiles does not show."""
    S, heads = 16384, (16, 1)
    for sigma in (0.16, 1.0):
        q, k, v = _spread_inputs(head_dim, heads, S, QUERIES[head_dim], sigma, 1.0, 2900)
        out = tq.tq_sdpa_int4_decode(gpu_cache_from(k, v), q.cuda(), S, 1.0, n_splits=1)
        torch.cuda.synchronize()
        _assert_weights_whole(out, _reference(q, oracle_cache_from(k, v), S, 1.0), slice(None), f"d={head_dim} sigma={sigma}")


@pytest.mark.parametrize("head_dim", [128, 256, 512])
def test_scales_of_v_that_grow_differ_and_turn_negative(head_dim):
    """Large scales first met rounds into the chunk, next to groups whose scales stay small, and scales of either sign."""
    nq, S, heads = QUERIES[head_dim], 3000, (10, 1)
    v_std = torch.full((head_dim,), 0.03)
    large = torch.arange(head_dim) // 32 % 3 == 1  # every third group
    v_std[large] = 3.0
    for case in ("late", "negative"):
        q, k, v = _spread_inputs(head_dim, heads, S, nq, 1.0, v_std, 2800)
        if case == "late":
            v = (v.float() * torch.where(large, torch.linspace(-2.0, 5.0, S)[:, None].exp2(), torch.ones(1))).half()
        cache, arrays = gpu_cache_from(k, v), list(oracle_cache_from(k, v))
        if case == "negative":
            flip = torch.rand(arrays[4].shape, generator=torch.Generator().manual_seed(1)) < 0.3
            arrays[4] = np.where(flip.numpy(), -arrays[4], arrays[4])
            cache.v_scale.copy_(torch.from_numpy(arrays[4]))
        ref = _reference(q, arrays, S, 1.0)
        for n_splits in (1, 3):
            out = tq.tq_sdpa_int4_decode(cache, q.cuda(), S, 1.0, n_splits=n_splits)
            torch.cuda.synchronize()
            for dims in (large.numpy(), ~large.numpy()):
                _assert_weights_whole(out, ref, dims, f"d={head_dim} {case} n_splits={n_splits} {int(dims.sum())} dims")
