"""Helpers for the GPU parity tests: the HIP path on one side, the CPU oracle on the other,
fed the same seeded fp16 bits.  Nothing computed by the HIP path is ever given to the oracle."""
from __future__ import annotations

import ctypes

import numpy as np
import torch

import oracle
import paper_2604_16957_amd as tq
import tq_workloads as wl
from paper_2604_16957_amd import binding

MAX_ABS = 2e-3      # attention output: max |gpu - oracle|
REL_L2 = 1e-3       # attention output: |gpu - oracle|_2 / |oracle|_2
# Outputs of magnitude above 1 (sharp softmaxes reproduce single value vectors): the fp16 output's own rounding is
# up to 2^-11 of the value, which the absolute bar cannot absorb beyond |value| = 4; the per-element bar there is
# MAX_ABS + 2^-11 |oracle value| (no slack beyond that representability term), the relative-L2 bar is unchanged.
FP16_HALF_ULP = 2.0 ** -11


def np16(t: torch.Tensor) -> np.ndarray:
    return t.detach().cpu().contiguous().numpy()


def gpu_cache_from(k: torch.Tensor, v: torch.Tensor, capacity=None, pos=0, fill=0xEE, group=32):
    """Quantise fp16 CPU tensors k, v [B,Hkv,S,d] into a fresh device cache with the HIP kernel."""
    B, Hkv, S, d = k.shape
    cache = tq.KVCache(B, Hkv, d, capacity or (pos + S), group_size=group)
    for t in cache.tensors():
        t.view(torch.uint8).fill_(fill)
    tq.tq_quantize_kv(cache, k.cuda(), v.cuda(), pos)
    return cache


def oracle_cache_from(k: torch.Tensor, v: torch.Tensor, group=32):
    kc, ks, kz = oracle.quantize(np16(k), group=group)
    vc, vs, vz = oracle.quantize(np16(v), group=group)
    return kc, ks, kz, vc, vs, vz


def assert_cache_bit_exact(cache, ocache, S, pos=0):
    names = ("k_codes", "k_scale", "k_zero", "v_codes", "v_scale", "v_zero")
    for name, g, o in zip(names, cache.tensors(), ocache):
        g = np16(g)[:, :, pos:pos + S]
        if g.dtype == np.float16:
            g, o = g.view(np.uint16), o.view(np.uint16)
        bad = int((g != o).sum())
        assert bad == 0, f"{name}: {bad} of {g.size} entries differ from the oracle"


def errors(out_gpu: torch.Tensor, ref: np.ndarray):
    got = np16(out_gpu).astype(np.float64)
    assert np.isfinite(got).all(), "non-finite output"
    diff = got - ref
    return float(np.abs(diff).max()), float(np.linalg.norm(diff) / np.linalg.norm(ref))


def assert_close(out_gpu, ref, what=""):
    max_abs, rel = errors(out_gpu, ref)
    assert max_abs <= MAX_ABS and rel <= REL_L2, f"{what}: max-abs {max_abs:.3e}, rel-L2 {rel:.3e}"
    return max_abs, rel


def assert_close_elementwise(out_gpu, ref, what=""):
    """Every element within MAX_ABS + 2^-11 |ref| (the fp16 output's own rounding), and the relative-L2 bar."""
    got = np16(out_gpu).astype(np.float64)
    assert np.isfinite(got).all(), f"{what}: non-finite output"
    diff = np.abs(got - ref)
    over = diff - (MAX_ABS + FP16_HALF_ULP * np.abs(ref))
    rel = float(np.linalg.norm(got - ref) / np.linalg.norm(ref))
    assert over.max() <= 0.0 and rel <= REL_L2, \
        f"{what}: {int((over > 0).sum())} elements over the bar (worst by {over.max():.2e}, max-abs {diff.max():.2e}), rel-L2 {rel:.3e}"
    return float(diff.max()), rel


def oracle_attend_dense_fp16(q: torch.Tensor, ocache, seq_len: int, alpha: float) -> np.ndarray:
    """What the unfused comparator computes by definition: attention (fp64) over K^ and V^ rounded to dense fp16."""
    kd = oracle.dequantize_f16(*[a[:, :, :seq_len] for a in ocache[:3]]).astype(np.float64)
    vd = oracle.dequantize_f16(*[a[:, :, :seq_len] for a in ocache[3:]]).astype(np.float64)
    return oracle.attend_dense(np16(q), kd, vd, alpha)


def assert_comparator_close(out_gpu, q, ocache, seq_len, alpha, what=""):
    """The unfused comparator materialises K^ and V^ as dense fp16 (Sec. 3.1's baseline): that rounding is part of
    what it computes, and it moves the result away from attention over the exact dequantised cache by more than
    the kernels' own error (up to 1.0e-3 relative-L2 on the shapes with outlier key channels, by the oracle's own
    evaluation of both definitions).  It is therefore held, at the same bars as the fused path, to ITS definition:
    the oracle's attention over the oracle's fp16-rounded dense tensors."""
    return assert_close(out_gpu, oracle_attend_dense_fp16(q, ocache, seq_len, alpha), what)


def oracle_attend(q: torch.Tensor, ocache, seq_len: int, alpha: float) -> np.ndarray:
    return oracle.attend_packed(np16(q), *ocache, seq_len=seq_len, alpha=alpha)


def make(w: wl.Workload):
    q, k, v = wl.make_inputs(w, device="cpu")
    return q, k, v


KERNELS = ("refused", "generic", "8 rows", "16 rows", "wide rows")   # matrix-core tiles of up to 8 (d = 256: 2) and of 16 rows


def kernel_of(batch, n_q_heads, n_kv_heads, head_dim, seq_len, call="decode", scale=1.0, group=32, n_queries=1, window=0,
              variant=0, n_splits=0):
    """Which kernel the library takes for such a call ("decode", "step", or "lengths" for per-sequence lengths of at most seq_len and for
    pages); asked on the host, nothing is launched."""
    fake = 0x10000
    struct = binding.TqKvCacheStruct(fake, fake, fake, fake, fake, fake, batch, n_kv_heads, head_dim, group, seq_len + seq_len % 2, 0)
    opts = binding.TqDecodeOptsStruct(n_splits, variant, window, n_queries)
    ask = binding.raw().tq_internal_decode_kernel
    ask.restype = ctypes.c_int32
    ask.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_int32, ctypes.c_float, ctypes.c_void_p, ctypes.c_int32]
    return KERNELS[ask(ctypes.byref(struct), n_q_heads, seq_len, scale, ctypes.byref(opts), ("decode", "step", "lengths").index(call))]


def listed_slots(batch, n_q_heads, n_kv_heads, head_dim, max_seq_len, group=32, n_queries=1, window=0, n_splits=0, variant=0):
    """Waves to a KV head that a call with per-sequence lengths deals to its sequences, 0 where it goes another way; asked on the host."""
    fake = 0x10000
    struct = binding.TqKvCacheStruct(fake, fake, fake, fake, fake, fake, batch, n_kv_heads, head_dim, group, max_seq_len + max_seq_len % 2, 0)
    opts = binding.TqDecodeOptsStruct(n_splits, variant, window, n_queries)
    ask = binding.raw().tq_internal_listed_slots
    ask.restype = ctypes.c_int32
    ask.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_int32, ctypes.c_float, ctypes.c_void_p]
    return ask(ctypes.byref(struct), n_q_heads, max_seq_len, 1.0, ctypes.byref(opts))


def lengths_waves(batch, n_q_heads, n_kv_heads, head_dim, max_seq_len, group=32, window=0):
    """Where a call with per-sequence lengths does not deal its waves out (see listed_slots): waves of a block that a row has to itself, or, negative,
    of a slot of the chunk list; asked on the host."""
    fake = 0x10000
    struct = binding.TqKvCacheStruct(fake, fake, fake, fake, fake, fake, batch, n_kv_heads, head_dim, group, max_seq_len + max_seq_len % 2, 0)
    opts = binding.TqDecodeOptsStruct(0, 0, window, 1)
    ask = binding.raw().tq_internal_lengths_waves
    ask.restype = ctypes.c_int32
    ask.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_int32, ctypes.c_float, ctypes.c_void_p]
    return ask(ctypes.byref(struct), n_q_heads, max_seq_len, 1.0, ctypes.byref(opts))


def counter_sets_left():
    """Sets of arrival counters that no workspace has taken: with none left, calls merge in a launch of their own."""
    return binding.raw().tq_internal_counter_sets_left()


def fine_chunks(batch, n_q_heads, n_kv_heads, head_dim, tokens, group=32, n_queries=1):
    """Chunks that a short sequence is cut into where the decode kernel merges them itself (1: no finer than otherwise); asked on the host."""
    fake = 0x10000
    struct = binding.TqKvCacheStruct(fake, fake, fake, fake, fake, fake, batch, n_kv_heads, head_dim, group, tokens + tokens % 2, 0)
    opts = binding.TqDecodeOptsStruct(0, 0, 0, n_queries)
    ask = binding.raw().tq_internal_fine_chunks
    ask.restype = ctypes.c_int32
    ask.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_int32, ctypes.c_void_p]
    return ask(ctypes.byref(struct), n_q_heads, tokens, ctypes.byref(opts))


def lengths_route(batch, n_q_heads, n_kv_heads, head_dim, max_seq_len, group=32, window=0):
    """How a call with per-sequence lengths (one query token, a workspace with arrival counters) spreads its sequences, in words; asked on the host."""
    if listed_slots(batch, n_q_heads, n_kv_heads, head_dim, max_seq_len, group, window=window):
        return "waves dealt"
    waves = lengths_waves(batch, n_q_heads, n_kv_heads, head_dim, max_seq_len, group, window)
    return f"{waves} waves a row" if waves > 0 else f"{-waves} waves a slot" if waves < 0 else "another kernel"


_workspace = None


def shared_workspace(batch, n_q_heads, head_dim):
    """The same workspace for every test that asks for one, filled with NaNs (nothing that the call has not written may count): the library has
    a limited number of sets of arrival counters, one for each workspace it ever sees, and a call without one merges in a launch of its own."""
    global _workspace
    need = tq.tq_workspace_bytes(batch, n_q_heads, head_dim)
    if _workspace is None or _workspace.numel() < need:
        _workspace = torch.empty(max(need, 1 << 30), dtype=torch.uint8, device="cuda")
    _workspace[:need].fill_(0xFF)
    return _workspace[:need]
