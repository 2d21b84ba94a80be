"""Query rows of nine and more per KV head (head_dim 256: three and more, with several query tokens) on the kernels with few rows to a
block: calls that the kernel for wide rows does not take, each asserted to be one."""
import numpy as np
import pytest
import torch

import oracle
import paper_2604_16957_amd as tq
import tq_workloads as wl
from gpu_common import (assert_cache_bit_exact, assert_close_elementwise, gpu_cache_from, kernel_of, make, np16, oracle_cache_from)

pytestmark = pytest.mark.gpu


def _reference(q, ocache, lens, alpha, window=0):
    """Query token t of sequence b attends the first lens[b] - (nq - 1 - t) tokens, under a window the last `window` of those."""
    q4 = q if q.dim() == 4 else q[:, None]
    nq, out = q4.shape[1], np.empty(tuple(q4.shape), dtype=np.float64)
    together = [(slice(None), lens[0])] if len(set(lens)) == 1 else [(slice(b, b + 1), n) for b, n in enumerate(lens)]
    for b, n in together:
        for t in range(nq):
            hi = n - (nq - 1 - t)
            lo = max(0, hi - window) if window else 0
            part = [np.ascontiguousarray(a[b, :, lo:hi]) for a in ocache]
            out[b, t] = oracle.attend_packed(np16(q4[b, t]), *part, seq_len=hi - lo, alpha=alpha)
    return out if q.dim() == 4 else out[:, 0]


def _check_every_entry(w, kernel, nq=1, window=0, n_splits=0, page=64):
    """Decode, step, both with per-sequence lengths, and over a paged pool, each on `kernel`."""
    B, Hq, Hkv, d, S, scale = w.batch, w.n_q_heads, w.n_kv_heads, w.head_dim, w.seq_len, w.attn_scale
    what = f"{Hq}/{Hkv} d={d} S={S} nq={nq} window={window} n_splits={n_splits}"
    for call in ("decode", "step", "lengths"):
        assert kernel_of(B, Hq, Hkv, d, S, call, scale, n_queries=nq, window=window, n_splits=n_splits) == kernel, f"{what} {call}"
    q, k, v = make(w)
    if nq > 1:
        q = torch.stack([q.roll(t, 0) for t in range(nq)], dim=1).contiguous()
    ocache = oracle_cache_from(k, v)
    ref = _reference(q, ocache, [S] * B, scale, window)
    cache = gpu_cache_from(k, v, capacity=S + 3)
    kw = dict(window=window, n_splits=n_splits)
    out = tq.tq_sdpa_int4_decode(cache, q.cuda(), S, scale, **kw)
    torch.cuda.synchronize()
    assert_close_elementwise(out, ref, f"decode {what}")
    if S > nq:
        for t in cache.tensors():                   # the new tokens' rows are wiped, and have to come back bit for bit
            t[:, :, S - nq:S].view(torch.uint8).fill_(0xEE)
        kn, vn = k[:, :, S - nq:].contiguous().cuda(), v[:, :, S - nq:].contiguous().cuda()
        out = tq.tq_sdpa_int4_append_decode(cache, kn, vn, q.cuda(), S, scale, **kw)
        torch.cuda.synchronize()
        assert_cache_bit_exact(cache, ocache, S)
        assert_close_elementwise(out, ref, f"step {what}")
    lens = [max(nq, S - 7 * (b % 5)) for b in range(B)]
    lens_dev = torch.tensor(lens, dtype=torch.int32).cuda()
    ref = _reference(q, ocache, lens, scale, window)
    out = tq.tq_sdpa_int4_decode_varlen(cache, q.cuda(), lens_dev, S, scale, **kw)
    torch.cuda.synchronize()
    assert_close_elementwise(out, ref, f"lengths {what}")
    pages = -(-S // page)
    pool = tq.KVCache(B * pages, Hkv, d, page)
    for t in pool.tensors():
        t.view(torch.uint8).fill_(0xEE)
    table = torch.randperm(B * pages, generator=torch.Generator().manual_seed(S)).to(torch.int32).reshape(B, pages).cuda()
    tq.tq_quantize_kv_paged(pool, table, k.cuda(), v.cuda(), torch.zeros(B, dtype=torch.int32).cuda())
    out = tq.tq_sdpa_int4_decode_paged(pool, table, q.cuda(), lens_dev, S, scale, **kw)
    torch.cuda.synchronize()
    assert_close_elementwise(out, ref, f"pages {what}")
    last = [torch.stack([a[b, :, n - nq:n] for b, n in enumerate(lens)]).contiguous().cuda() for a in (k, v)]
    out = tq.tq_sdpa_int4_append_decode_varlen(cache, *last, q.cuda(), lens_dev, S, scale, **kw)
    torch.cuda.synchronize()
    assert_cache_bit_exact(cache, ocache, S)
    assert_close_elementwise(out, ref, f"step with lengths {what}")
    out = tq.tq_sdpa_int4_append_decode_paged(pool, table, *last, q.cuda(), lens_dev, S, scale, **kw)
    torch.cuda.synchronize()
    assert_close_elementwise(out, ref, f"step over pages {what}")


@pytest.mark.parametrize("gqa", [9, 10, 16, 24, 40])
def test_sixteen_row_tiles_of_many_sequences(gqa):
    """132 (sequence, KV head) rows: the 16-row tile, partly filled, full, and several per KV head (24 = 2 x 12, 40 = 4 x 10), at ragged
    lengths around the 32-token supertile, with forced chunks, a window, and a sharp softmax where every row moves its own reference."""
    for S, window, n_splits, sharp in ((1, 0, 0, False), (31, 0, 0, False), (32, 0, 0, False), (33, 0, 0, False), (321, 0, 0, False),
                                       (300, 0, 7, False), (500, 130, 0, False), (400, 0, 0, True), (290, 77, 3, False)):
        kw = dict(attn_scale=1.0, v_std=0.5) if sharp else {}
        _check_every_entry(wl.custom(batch=33, n_q_heads=4 * gqa, n_kv_heads=4, head_dim=128, seq_len=S, seed=3000 + gqa + S, outlier_channels=4, **kw),
                           "16 rows", window=window, n_splits=n_splits)


@pytest.mark.parametrize("gqa,nq", [(8, 2), (8, 3), (3, 4), (8, 8), (5, 6), (16, 2)])
def test_sixteen_row_tiles_of_several_query_tokens(gqa, nq):
    """The same tile with rows of several query tokens, causal among themselves, whose masked tokens fall into one supertile, two, or a
    chunk of their own; windows down to one token."""
    for S, window, n_splits in ((nq, 0, 0), (31, 0, 0), (33, 0, 0), (64 + nq // 2, 0, 0), (65, 5, 0), (300, 0, 4), (300, 1, 0), (310, 40, 0),
                                (333, 100, 3)):
        _check_every_entry(wl.custom(batch=33, n_q_heads=4 * gqa, n_kv_heads=4, head_dim=128, seq_len=S, seed=3100 + gqa + S), "16 rows", nq=nq,
                           window=window, n_splits=n_splits)


@pytest.mark.parametrize("gqa,nq", [(2, 2), (2, 8), (1, 3), (4, 5)])
def test_several_query_tokens_at_256_of_many_sequences(gqa, nq):
    """head_dim 256 past 128 (sequence, KV head) rows and below 512 tokens: the tile of two rows, several blocks to a KV head."""
    for S, window, n_splits in ((nq, 0, 0), (31, 0, 0), (33, 0, 0), (64 + nq // 2, 0, 0), (65, 5, 0), (300, 0, 4), (300, 1, 0), (511, 40, 0)):
        _check_every_entry(wl.custom(batch=17, n_q_heads=8 * gqa, n_kv_heads=8, head_dim=256, seq_len=S, seed=3200 + gqa + S, attn_scale=1.0,
                                     qk_std=0.1), "8 rows", nq=nq, window=window, n_splits=n_splits)


@pytest.mark.parametrize("heads,kv,d,nq,S", [(64, 8, 128, 4, 40032), (64, 8, 128, 5, 20032), (128, 8, 128, 1, 35232), (16, 8, 128, 2, 16032)])
def test_one_long_sequence_past_the_line(heads, kv, d, nq, S):
    """The shortest lengths of one sequence at which a step is on these kernels, and its decode too."""
    w = wl.custom(n_q_heads=heads, n_kv_heads=kv, head_dim=d, seq_len=S, seed=3300 + nq, outlier_channels=4)
    kernel = "8 rows" if heads // kv * nq <= 8 else "16 rows"
    assert all(kernel_of(1, heads, kv, d, S, call, n_queries=nq) == kernel for call in ("decode", "step"))
    q, k, v = make(w)
    if nq > 1:
        q = torch.randn(1, nq, heads, d, generator=torch.Generator().manual_seed(S)).half()
    ocache = oracle_cache_from(k, v)
    cache = gpu_cache_from(k[:, :, :S - nq].contiguous(), v[:, :, :S - nq].contiguous(), capacity=S)
    kn, vn = k[:, :, S - nq:].contiguous().cuda(), v[:, :, S - nq:].contiguous().cuda()
    step = tq.tq_sdpa_int4_append_decode(cache, kn, vn, q.cuda(), S, w.attn_scale)
    again = tq.tq_sdpa_int4_decode(cache, q.cuda(), S, w.attn_scale)
    torch.cuda.synchronize()
    assert_cache_bit_exact(cache, ocache, S)
    ref = _reference(q, ocache, [S], w.attn_scale)
    assert_close_elementwise(step, ref, f"step {heads}/{kv} nq={nq} S={S}")
    assert_close_elementwise(again, ref, f"decode {heads}/{kv} nq={nq} S={S}")
