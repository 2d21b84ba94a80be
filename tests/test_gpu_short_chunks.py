"""Short sequences, cut into chunks of two to eight 32-token tiles that the decode kernel merges in place: at the edges where
the number of tiles to a chunk changes, with waves that have no tile, and with the step's new token on either kind of wave."""
import numpy as np
import pytest
import torch

import paper_2604_16957_amd as tq
import tq_workloads as wl
from gpu_common import assert_cache_bit_exact, assert_close, gpu_cache_from, make, oracle_attend, oracle_cache_from

pytestmark = pytest.mark.gpu

# tiles: 8 | 9 .. 15 (one chunk, or two tiles each; 13: the first that every instance cuts) | 16, 32 | 33, 48 (three) | 49, 128 (four) |
# 129 (five, where 32 chunks fit)
LENGTHS = [256, 257, 289, 384, 385, 480, 481, 512, 1024, 1025, 1536, 1537, 4096, 4097]
SHAPES = [(1, 8, 1, 128, 32), (1, 8, 8, 128, 32), (3, 40, 5, 128, 32), (1, 16, 2, 128, 128), (1, 4, 2, 256, 32), (2, 16, 8, 256, 64)]


@pytest.mark.parametrize("B,Hq,Hkv,d,group", SHAPES)
def test_short_sequences_in_fine_chunks(B, Hq, Hkv, d, group):
    w = wl.custom(batch=B, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, seq_len=max(LENGTHS), seed=77 + Hq + d + group)
    q, k, v = make(w)
    whole = oracle_cache_from(k, v, group=group)
    workspace = torch.empty(tq.tq_workspace_bytes(B, Hq, d), dtype=torch.uint8, device="cuda")
    for n in LENGTHS:
        ocache = [np.ascontiguousarray(a[:, :, :n]) for a in whole]
        ref = oracle_attend(q, ocache, n, w.attn_scale)
        cache = gpu_cache_from(k[:, :, :n].contiguous(), v[:, :, :n].contiguous(), capacity=n + n % 2, group=group)
        workspace.fill_(0xFF)                           # (NaNs: nothing that is not written may be read)
        out = tq.tq_sdpa_int4_decode(cache, q.cuda(), n, w.attn_scale, workspace=workspace)
        again = tq.tq_sdpa_int4_decode(cache, q.cuda(), n, w.attn_scale, workspace=workspace)
        torch.cuda.synchronize()
        assert_close(out, ref, f"decode of {n}")
        assert torch.equal(out, again), n
        for t in cache.tensors():
            t[:, :, n - 1].view(torch.uint8).fill_(0xEE)
        workspace.fill_(0xFF)
        out = tq.tq_sdpa_int4_append_decode(cache, k[:, :, n - 1:n].contiguous().cuda(), v[:, :, n - 1:n].contiguous().cuda(), q.cuda(),
                                            n, w.attn_scale, workspace=workspace)
        torch.cuda.synchronize()
        assert_close(out, ref, f"step of {n}")
        assert_cache_bit_exact(cache, ocache, n)
