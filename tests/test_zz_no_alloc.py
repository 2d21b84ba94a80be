"""The allocation-free entry point, tq_sdpa_int4_decode_static, against tq_sdpa_int4_decode (and the oracle):
several calls in a row on the same static scratch array, each with a smaller input than the one before, so that
every later call finds the earlier one's partial results lying in the array."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2604_16957_amd as tq
import tq_workloads as wl
from paper_2604_16957_amd import binding as B

from gpu_common import (MAX_ABS, REL_L2, assert_cache_bit_exact, assert_close, counter_sets_left, gpu_cache_from, lengths_waves, make, np16, oracle_attend,
                        oracle_cache_from)
from test_gpu_uneven_lengths import _uneven, check

pytestmark = pytest.mark.gpu


def _case(batch, hq, hkv, d, S, seed):
    w = wl.custom(batch=batch, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, seq_len=S, seed=seed, outlier_channels=4)
    q, k, v = make(w)
    return w, q, gpu_cache_from(k, v), oracle_cache_from(k, v)


def test_static_scratch_decode_matches_the_workspace_call_on_calls_in_a_row():
    torch.cuda.set_device(0)
    # 84 MB of cache (two launches: partial kernel + merge kernel), then a sequence short enough for the
    # one-launch route with its in-kernel chunk merge, then a single chunk
    shapes = [(2, 64, 8, 128, 32768, 71), (1, 64, 8, 128, 6000, 72), (1, 16, 2, 128, 700, 73)]
    launches = []
    for batch, hq, hkv, d, S, seed in shapes:
        w, q, cache, ocache = _case(batch, hq, hkv, d, S, seed)
        assert tq.tq_workspace_bytes(batch, hq, d) <= B.TQ_STATIC_SCRATCH_BYTES
        launches.append(tq.tq_decode_launches(cache, hq, S, w.attn_scale))
        qg = q.cuda()
        want = tq.tq_sdpa_int4_decode(cache, qg, S, w.attn_scale)
        got = torch.full_like(want, float("nan"))
        tq.tq_sdpa_int4_decode_static(cache, qg, S, w.attn_scale, got)
        torch.cuda.synchronize()
        diff = (got.double() - want.double()).cpu().numpy()
        ref = np16(want).astype(np.float64)
        assert np.isfinite(diff).all(), f"S={S}: non-finite output"
        assert np.abs(diff).max() <= MAX_ABS and np.linalg.norm(diff) <= REL_L2 * np.linalg.norm(ref), \
            f"S={S}: static-scratch call differs from the workspace call by {np.abs(diff).max():.3e}"
        assert_close(got, oracle_attend(q, ocache, S, w.attn_scale), f"static scratch, S={S}")
    assert launches[0] == 2 and launches[1] == 1 and launches[2] == 1


def test_static_scratch_decode_rejects_what_does_not_fit():
    torch.cuda.set_device(0)
    w, q, cache, _ = _case(1, 16, 2, 128, 64, 74)
    big = B.TqKvCacheStruct.from_buffer_copy(cache.struct)
    big.batch = 64                                   # 64 x 16 heads x 128 chunks x 130 floats: 68 MB of partials
    assert tq.tq_workspace_bytes(64, 16, 128) > B.TQ_STATIC_SCRATCH_BYTES
    out = torch.empty((64, 16, 128), dtype=torch.float16, device="cuda")
    q64 = torch.zeros((64, 16, 128), dtype=torch.float16, device="cuda")
    rc = B.raw().tq_sdpa_int4_decode_static(ctypes.byref(big), q64.data_ptr(), 16, 64, 0.1, out.data_ptr(), None, None)
    assert rc == B.TQ_ERR_WORKSPACE
    rc = B.raw().tq_sdpa_int4_decode_static(ctypes.byref(cache.struct), None, 16, 64, 0.1, out.data_ptr(), None, None)
    assert rc == B.TQ_ERR_NULL


def test_more_workspaces_than_counter_sets_take_the_merge_kernel():
    """(Kept at the very end of the GPU suite: it uses up the library's sets of arrival counters for the rest of the
    process.)  The one-launch decode route gives every workspace a set of arrival counters of its own for the life
    of the process; a workspace that finds them all taken gets the merge kernel (two launches) instead, never a set
    shared with another workspace.  300 distinct workspaces (more than there are sets), in flight 8 at a time: all
    results right."""
    torch.cuda.set_device(0)
    w, q, cache, ocache = _case(2, 24, 3, 128, 5000, 75)
    qg = q.cuda()
    assert tq.tq_decode_launches(cache, 24, 5000, w.attn_scale) == 1
    ref = oracle_attend(q, ocache, 5000, w.attn_scale)
    nbytes = tq.tq_workspace_bytes(2, 24, 128)
    ws = [torch.empty(nbytes, dtype=torch.uint8, device="cuda") for _ in range(300)]
    streams = [torch.cuda.Stream() for _ in range(8)]
    outs = [torch.zeros_like(qg) for _ in ws]
    torch.cuda.synchronize()
    for i, (wsp, o) in enumerate(zip(ws, outs)):
        with torch.cuda.stream(streams[i % len(streams)]):
            tq.tq_sdpa_int4_decode(cache, qg, 5000, w.attn_scale, out=o, workspace=wsp)
    torch.cuda.synchronize()
    for i, o in enumerate(outs):
        assert_close(o, ref, f"workspace {i}")


def _without_counters(batch, hq, d):
    """A workspace that finds every set of arrival counters taken (any that are left are taken here first), and those that took them."""
    w, q, cache, _ = _case(1, 8, 1, 128, 1000, 76)
    nbytes, taken = max(tq.tq_workspace_bytes(1, 8, 128), 1 << 20), []
    while counter_sets_left() > 0:
        taken.append(torch.empty(nbytes, dtype=torch.uint8, device="cuda"))
        tq.tq_sdpa_int4_decode(cache, q.cuda(), 1000, w.attn_scale, workspace=taken[-1])
    torch.cuda.synchronize()
    # (an odd 256 bytes into an allocation of its own: an address that no workspace has had)
    return torch.empty(tq.tq_workspace_bytes(batch, hq, d) + 768, dtype=torch.uint8, device="cuda")[768:], taken


# (sequences, query heads, KV heads, d, longest, bound, group, page, waves of a slot): calls that deal their waves to the sequences, without counters
@pytest.mark.parametrize("B,Hq,Hkv,d,longest,S,group,page,waves", [
    (12, 16, 8, 128, 1500, 6000, 32, 0, 8), (30, 16, 8, 128, 900, 6000, 32, 64, 4), (61, 16, 8, 128, 700, 3000, 32, 0, 2),
    (65, 16, 8, 128, 500, 6000, 64, 0, 1), (33, 32, 16, 256, 500, 2500, 32, 32, 1)])
def test_lengths_without_counters_take_the_chunk_list(B, Hq, Hkv, d, longest, S, group, page, waves):
    workspace, _taken = _without_counters(B, Hq, d)
    assert counter_sets_left() == 0 and lengths_waves(B, Hq, Hkv, d, S, group) == -waves
    check(B, Hq, Hkv, d, _uneven(B, longest, 77 + B), S, group=group, page=page, workspace=workspace)
    assert counter_sets_left() == 0


# one chunk that would be cut with counters; several chunks (the merge kernel)
@pytest.mark.parametrize("hq,hkv,d,S", [(64, 8, 128, 480), (32, 16, 256, 300), (32, 8, 128, 2000)])
def test_short_sequences_without_counters(hq, hkv, d, S):
    w, q, cache, ocache = _case(1, hq, hkv, d, S, 78)
    workspace, _taken = _without_counters(1, hq, d)
    workspace.fill_(0xFF)
    assert counter_sets_left() == 0
    out = tq.tq_sdpa_int4_decode(cache, q.cuda(), S, w.attn_scale, workspace=workspace)
    assert_close(out, oracle_attend(q, ocache, S, w.attn_scale), "decode")
    k, v = make(w)[1:]
    for t in cache.tensors():
        t[:, :, S - 1].view(torch.uint8).fill_(0xEE)
    out = tq.tq_sdpa_int4_append_decode(cache, k[:, :, S - 1:].contiguous().cuda(), v[:, :, S - 1:].contiguous().cuda(), q.cuda(), S, w.attn_scale,
                                        workspace=workspace)
    torch.cuda.synchronize()
    assert_close(out, oracle_attend(q, ocache, S, w.attn_scale), "step")
    assert_cache_bit_exact(cache, ocache, S)
