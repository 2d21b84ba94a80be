"""Many sequences with lengths of their own: the launches in which every (sequence, KV head) row is one chunk of a block
of its own, longest row first, and where they give way to the device-planned chunk list or to waves dealt to the sequences.  Every
row against the oracle; and, for the mixes that an ordering or a bound exists for, that it does what it is there for."""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_2604_16957_amd as tq
import tq_workloads as wl
from gpu_common import assert_close_elementwise, counter_sets_left, gpu_cache_from, lengths_route, make, np16, oracle_cache_from, shared_workspace

pytestmark = pytest.mark.gpu


def _uneven(batch, longest, seed):
    """Mostly short lengths with many ties, a few long ones (the longest among them), in no order."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(2, 97, batch)
    lens[: batch // 4] = rng.choice([32, 33, 64, 65, 96], batch // 4)
    lens[: max(1, batch // 32)] = rng.integers(longest // 2, longest + 1, max(1, batch // 32))
    lens[0] = longest
    return [int(n) for n in rng.permutation(lens)]


def _reference(q, ocache, lens, alpha, window):
    rows = []
    for b, n in enumerate(lens):
        lo = max(0, n - window) if window else 0
        one = [np.ascontiguousarray(a[b:b + 1, :, lo:n]) for a in ocache]
        rows.append(oracle.attend_packed(np16(q[b:b + 1]), *one, seq_len=n - lo, alpha=alpha))
    return np.concatenate(rows, axis=0)


def check(B, Hq, Hkv, d, lens, S, group=32, page=0, window=0, route=None, workspace=None):
    """A decode, twice (bit for bit alike), and a step that brings every sequence's last token, against the oracle, in a workspace of NaNs
    (the shared one, or `workspace`).  route: how the call has to spread its sequences (see lengths_route)."""
    if route is not None:
        assert lengths_route(B, Hq, Hkv, d, S, group, window) == route
        assert route != "waves dealt" or counter_sets_left() > 0
    w = wl.custom(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, seq_len=max(lens), seed=9000 + B + Hkv + S + group)
    q, k, v = make(w)
    ocache = oracle_cache_from(k, v, group=group)
    ref = _reference(q, ocache, lens, w.attn_scale, window)
    lens_dev = torch.tensor(lens, dtype=torch.int32).cuda()
    k_new = torch.stack([k[b, :, n - 1:n] for b, n in enumerate(lens)]).contiguous().cuda()
    v_new = torch.stack([v[b, :, n - 1:n] for b, n in enumerate(lens)]).contiguous().cuda()
    more = lambda: dict(window=window, workspace=shared_workspace(B, Hq, d) if workspace is None else workspace.fill_(0xFF))
    if page:
        blocks = -(-S // page)
        cache = tq.KVCache(B * blocks, Hkv, d, page, group_size=group)
        table = torch.randperm(B * blocks, generator=torch.Generator().manual_seed(B + S)).to(torch.int32).reshape(B, blocks).cuda()
        tq.tq_quantize_kv_paged(cache, table, k.cuda(), v.cuda(), torch.zeros(B, dtype=torch.int32, device="cuda"))
        decode = lambda: tq.tq_sdpa_int4_decode_paged(cache, table, q.cuda(), lens_dev, S, w.attn_scale, **more())
        step = lambda: tq.tq_sdpa_int4_append_decode_paged(cache, table, k_new, v_new, q.cuda(), lens_dev, S, w.attn_scale, **more())
    else:
        cache = gpu_cache_from(k, v, capacity=S + (S & 1), group=group)
        decode = lambda: tq.tq_sdpa_int4_decode_varlen(cache, q.cuda(), lens_dev, S, w.attn_scale, **more())
        step = lambda: tq.tq_sdpa_int4_append_decode_varlen(cache, k_new, v_new, q.cuda(), lens_dev, S, w.attn_scale, **more())
    what = f"{B} sequences, {Hq}/{Hkv} heads, d={d}, bound {S}, g={group}, page={page}, window={window}"
    out = decode()
    again = decode()
    torch.cuda.synchronize()
    assert_close_elementwise(out, ref, "decode: " + what)
    assert torch.equal(out, again), what
    # the step: the last tokens' rows are wiped first, and have to come back bit for bit
    before = [t.clone() for t in cache.tensors()]
    for b, n in enumerate(lens):
        for t in cache.tensors():
            row = t[int(table[b, (n - 1) // page]), :, (n - 1) % page] if page else t[b, :, n - 1]
            row.view(torch.uint8).fill_(0xEE)
    out = step()
    torch.cuda.synchronize()
    assert_close_elementwise(out, ref, "step: " + what)
    for t, old in zip(cache.tensors(), before):
        assert torch.equal(t.view(torch.uint8), old.view(torch.uint8)), "step: " + what


# more than 256 sequences: the order comes from eight registers of lanes instead of four; above 512 it is the given one
@pytest.mark.parametrize("B,Hkv,longest", [(257, 2, 1500), (300, 4, 1300), (512, 1, 1500), (512, 8, 600), (513, 1, 900)])
def test_hundreds_of_sequences_each_row_once(B, Hkv, longest):
    check(B, 2 * Hkv, Hkv, 128, _uneven(B, longest, 31 + B), longest)


# How the sequences are spread follows from their number, the heads, the bound and the window alone: (sequences, query heads, KV heads, d, longest,
# bound, window, how); "even": all lengths within two tiles of each other.  A window next to the bound (everything is attended) is one of the
# ways to the chunk list.
ROUTES = {
    "one round of 4 waves a row": (64, 16, 8, 128, 1100, 2048, 0, "4 waves a row"),
    "8 waves a row": (64, 16, 8, 128, 2300, 3072, 0, "8 waves a row"),
    "8 waves a row, two rounds and a bit": (88, 64, 8, 128, 700, 4096, 0, "8 waves a row"),
    "4 waves a row": (97, 16, 8, 128, 1100, 3072, 0, "4 waves a row"),
    "4 waves a row, past two rounds": (129, 16, 8, 128, 700, 2048, 0, "4 waves a row"),
    "2 waves a row": (161, 16, 8, 128, 900, 1024, 0, "2 waves a row"),
    "1 wave a row": (261, 16, 8, 128, 600, 1024, 0, "1 waves a row"),
    "sixteen rows to a tile, 4 waves": (64, 96, 8, 128, 400, 1024, 0, "4 waves a row"),
    "sixteen rows to a tile, 8 waves": (64, 128, 8, 128, 300, 4000, 0, "8 waves a row"),
    "sixteen rows to a tile, two tiles to a KV head": (64, 96, 4, 128, 400, 1024, 0, "4 waves a row"),
    "d = 256, 4 waves": (32, 32, 16, 256, 600, 1024, 0, "4 waves a row"),
    "d = 256, 8 waves": (32, 32, 16, 256, 1500, 2048, 0, "8 waves a row"),
    "d = 256, 2 waves": (80, 32, 16, 256, 300, 1000, 0, "2 waves a row"),
    "d = 256, 1 wave": (130, 16, 16, 256, 200, 500, 0, "1 waves a row"),
    "chunk list, 8 waves a slot": (12, 16, 8, 128, 1500, 6000, 5999, "8 waves a slot"),
    "chunk list, 4 waves a slot": (30, 16, 8, 128, 900, 6000, 5999, "4 waves a slot"),
    "chunk list, 2 waves a slot": (61, 16, 8, 128, 700, 3000, 2999, "2 waves a slot"),
    "chunk list, 1 wave a slot": (97, 16, 8, 128, 900, 6000, 0, "1 waves a slot"),
    "chunk list, 1 wave a slot, d = 256": (115, 16, 16, 256, 400, 2500, 0, "1 waves a slot"),
    "waves dealt, 256 slots for 12": (12, 16, 8, 128, 1500, 6000, 0, "waves dealt"),
    "waves dealt, 256 slots for 61": (61, 16, 8, 128, 700, 3000, 0, "waves dealt"),
    "waves dealt, past 512 rows": (65, 16, 8, 128, 900, 6000, 0, "waves dealt"),
    "waves dealt, d = 256": (33, 32, 16, 256, 500, 2500, 0, "waves dealt"),
}


@pytest.mark.parametrize("mix", ["uneven", "even"])
@pytest.mark.parametrize("route", ROUTES)
def test_every_kind_of_block(route, mix):
    B, Hq, Hkv, d, longest, S, window, how = ROUTES[route]
    lens = _uneven(B, longest, 77 + B)
    if mix == "even":
        lens = [int(n) for n in np.random.default_rng(B).integers(130, 194, B)]
    check(B, Hq, Hkv, d, lens, S, window=window, route=how)


@pytest.mark.parametrize("group", [64, 128])
@pytest.mark.parametrize("route", ["one round of 4 waves a row", "2 waves a row", "sixteen rows to a tile, 4 waves", "d = 256, 4 waves",
                                   "d = 256, 2 waves", "chunk list, 1 wave a slot", "chunk list, 1 wave a slot, d = 256", "waves dealt, past 512 rows"])
def test_larger_groups_in_every_kind_of_block(route, group):
    B, Hq, Hkv, d, longest, S, window, how = ROUTES[route]
    check(B, Hq, Hkv, d, _uneven(B, min(longest, 400), 78 + B), S, group=group, window=window, route=how)


@pytest.mark.parametrize("window", [0, 77])
@pytest.mark.parametrize("page", [32, 64])
@pytest.mark.parametrize("route", ["one round of 4 waves a row", "4 waves a row", "2 waves a row", "1 wave a row",
                                   "sixteen rows to a tile, 4 waves", "d = 256, 4 waves", "chunk list, 1 wave a slot", "chunk list, 4 waves a slot",
                                   "waves dealt, past 512 rows"])
def test_pages_and_windows_in_every_kind_of_block(route, page, window):
    """(Under a window the bound is the window: the same rows, then, are ranked with the fewest tokens to a wave.)"""
    B, Hq, Hkv, d, longest, S, own_window, how = ROUTES[route]
    check(B, Hq, Hkv, d, _uneven(B, min(longest, 500), 79 + B), S, page=page, window=window or own_window, route=None if window else how)


# chunks of more than 64 pages: the kernel keeps 64 page numbers at hand and fetches on as it goes.  (B, query heads, KV
# heads, d, lengths, bound): one whole block to a chunk, half and a quarter of one, a row of its own, eight query rows.
@pytest.mark.parametrize("window", [0, 4500])
@pytest.mark.parametrize("B,Hq,Hkv,d,lens,S", [
    (1, 64, 64, 128, [14000], 14000), (1, 64, 64, 256, [12031], 12031), (2, 128, 128, 128, [5003, 4100], 5003),
    (9, 32, 32, 128, [4700 + 3 * i for i in range(9)], 4800), (64, 16, 8, 128, [4090] + [50 + i for i in range(63)], 4090),
    (1, 256, 32, 128, [20001], 20001)])
def test_chunks_of_more_than_64_pages(B, Hq, Hkv, d, lens, S, window):
    check(B, Hq, Hkv, d, lens, S, page=32, window=window)


def _time_us(hq, hkv, lens, S, page=0):
    """us per decode, from a graph of 20 calls, the median of several replays (caches of random codes)."""
    B, d = len(lens), 128
    if page:
        blocks = -(-S // page)
        cache = tq.KVCache(B * blocks, hkv, d, page)
        table = torch.arange(B * blocks, dtype=torch.int32, device="cuda").reshape(B, blocks)
    else:
        cache = tq.KVCache(B, hkv, d, S)
    for t in cache.tensors():
        t.zero_() if t.dtype != torch.uint8 else t.random_(0, 255)
    cache.k_scale.fill_(0.05), cache.v_scale.fill_(0.2)
    q = torch.randn(B, hq, d, device="cuda").half()
    n = torch.tensor(lens, dtype=torch.int32, device="cuda")
    ws = torch.empty(tq.tq_workspace_bytes(B, hq, d), dtype=torch.uint8, device="cuda")
    out = torch.empty_like(q)

    def call():
        if page:
            tq.tq_sdpa_int4_decode_paged(cache, table, q, n, S, 0.09, out=out, workspace=ws)
        else:
            tq.tq_sdpa_int4_decode_varlen(cache, q, n, S, 0.09, out=out, workspace=ws)

    for _ in range(20):
        call()
    torch.cuda.synchronize()
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.stream(side):
        call()
        with torch.cuda.graph(graph, stream=side):
            for _ in range(20):
                call()
    times = []
    for _ in range(9):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        graph.replay()
        a.record()
        for _ in range(10):
            graph.replay()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3 / 200)
    return sorted(times)[4]


def _spread_over_the_logarithm(n, lo, hi):
    lens = [int(round(lo * (hi / lo) ** (i / (n - 1)))) for i in range(n)]
    return [lens[i] for i in torch.randperm(n, generator=torch.Generator().manual_seed(5)).tolist()]


def test_the_order_of_lengths_is_kept_past_256_sequences():
    """300 sequences against 256 of the same mix: 1.17 times the rows.  In the given order, two rows to a block
    whatever their lengths, they took 2.5 times as long; ordered, 1.25 times (the bar lies in the middle)."""
    few = _time_us(32, 4, _spread_over_the_logarithm(256, 64, 2048), 2048)
    many = _time_us(32, 4, _spread_over_the_logarithm(300, 64, 2048), 2048)
    assert many < 1.75 * few, f"256 sequences {few:.1f} us, 300 {many:.1f} us"


@pytest.mark.parametrize("page", [0, 64])
def test_one_long_sequence_does_not_hold_up_many_short_ones(page):
    """64 sequences of 128 tokens, 8 KV heads, a bound of 8192: with one of them at the bound the plan cuts it up, and
    the launch takes about as long as the sum of the lengths; as one chunk of one block it took 4 times as long as the
    short ones alone."""
    short = _time_us(64, 8, [128] * 64, 8192, page)
    long = _time_us(64, 8, [128] * 40 + [8192] + [128] * 23, 8192, page)
    assert long < 1.8 * short, f"64 of 128 tokens {short:.1f} us, one of 8192 among them {long:.1f} us"
