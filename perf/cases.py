"""The work this library is measured on: one layer's share of a decode step, or of a prompt, over the sizes it serves.

A case is one call of the public entry points as a serving program makes it: the cache, the workspace and the output
buffer are kept from call to call, the step's query and new token are on the GPU.  The shapes are the ones the
benchmark, the tests and the design document use (the 70B attention shape, the local, global and grouped-query shapes of the
kernel configuration table), with ragged lengths among them.  Every decode step appends its token(s) and attends.

`exact` evaluates the same definition with plain torch in 64 bits from the same seeded inputs: the quantiser's
stored values (whose fp32 steps are reproduced bit for bit), then softmax attention over the dequantised cache.
"""
import math

import torch

import paper_2604_16957_amd as tq

PIECE = 1 << 24                     # elements of K drawn at a time


def _case(name, kind, batch, n_q_heads, n_kv_heads, head_dim, seq_len, **more):
    c = {"name": name, "kind": kind, "batch": batch, "n_q_heads": n_q_heads, "n_kv_heads": n_kv_heads,
         "head_dim": head_dim, "seq_len": seq_len, "min_len": seq_len, "group": 32, "window": 0, "n_queries": 1,
         "page": 0}
    c.update(more)
    return c


def listed():
    return [
        # the smallest call: one short sequence of a model with one KV head; launches and latencies
        _case("tiny_step", "step", 1, 8, 1, 128, 1024),
        # a chat-length sequence of the 70B attention shape
        _case("llama8k_step", "step", 1, 64, 8, 128, 8191),
        # the headline: one 128K sequence of the 70B attention shape
        _case("llama128k_step", "step", 1, 64, 8, 128, 131072),
        # the largest: one layer of the batch-4 sweep at 128K
        _case("llama128k_b4_step", "step", 4, 64, 8, 128, 131072),
        # head dimension 256 with two query heads per KV head, whole sequence
        _case("gemma32k_step", "step", 1, 32, 16, 256, 32768),
        # the same model's local layers, which are most of its layers: a sliding window of 1024 tokens
        _case("gemma_local_step", "step", 1, 32, 16, 256, 20011, window=1024),
        # the global layers of the configuration table: head dimension 512, 32 query heads on one KV head
        _case("global512_32k_step", "step", 1, 32, 1, 512, 32768),
        # speculative verification: four query tokens a step
        _case("llama_verify4", "step", 1, 64, 8, 128, 32763, n_queries=4),
        # continuous batching over a contiguous cache: every sequence at a length of its own
        _case("llama_varlen64", "varlen", 64, 64, 8, 128, 4096, min_len=128),
        # continuous batching over a pool of 256-token pages
        _case("llama_paged24", "paged", 24, 64, 8, 128, 16384, min_len=1000, page=256),
        # the 4.5-bit format (groups of 64) at head dimension 256
        _case("gemma32k_g64_step", "step", 1, 32, 16, 256, 32768, group=64),
        # a prompt quantised in one call
        _case("prefill32k", "prefill", 1, 64, 8, 128, 32749),
    ]


HEADS = {128: [(8, 1), (32, 8), (64, 8), (64, 8), (128, 8), (32, 32)], 256: [(16, 8), (32, 16), (32, 4)],
         512: [(32, 1), (16, 2)]}


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: kinds, shapes, formats and lengths of the listed ones, at most as large as the largest."""
    kind = rng.choice(["step", "step", "step", "step", "local", "verify", "varlen", "varlen", "paged", "prefill"])
    dim = rng.choice({"local": [256], "verify": [128, 128, 256], "varlen": [128, 128, 256],
                      "paged": [128, 128, 256]}.get(kind, [128, 128, 128, 256, 256, 512]))
    n_q, n_kv = rng.choice(HEADS[dim])
    group = 32
    if dim != 512 and kind in ("step", "prefill", "varlen"):
        group = rng.choice([32, 32, 32, 32, 64, 128])
    per_token = 2 * n_kv * (dim // 2 + 4 * (dim // group))
    # bytes of packed cache a call may attend (a shape with many query heads per byte works longer on each)
    most = {512: 40e6}.get(dim, 600e6 if n_q <= 8 * n_kv else 200e6)
    if group != 32 and dim == 256:
        most = 150e6
    if kind == "verify":
        most = 80e6 if n_q <= 8 * n_kv else 40e6
    if kind in ("varlen", "paged"):
        batch = _log(rng, 4, 128)
        top = int(min(32768, max(256, most / per_token / batch)))
        hi = _log(rng, 200, top)
        return _case_of(kind, batch, n_q, n_kv, dim, hi, group, min_len=max(2, _log(rng, max(2, hi // 64), hi)),
                        page=rng.choice([64, 256]) if kind == "paged" else 0)
    if kind == "prefill":
        batch = rng.choice([1, 1, 1, 2, 4])
        per_token += 2 * n_kv * dim * 2                          # (the fp16 source counts as well)
        return _case_of(kind, batch, n_q, n_kv, dim, _log(rng, 64, min(131072, most / per_token / batch)), group)
    batch = rng.choice([1, 1, 1, 2, 4, 8, 32])
    hi = max(600, min(131072, most / per_token / batch))
    if kind == "local":
        return _case_of("step", batch, n_q, n_kv, dim, _log(rng, 600, min(hi, 32768)), group, window=rng.choice([512, 1024]))
    if kind == "verify":
        return _case_of("step", min(batch, 4), n_q, n_kv, dim, _log(rng, 512, hi), group, n_queries=rng.randint(2, 8))
    return _case_of("step", batch, n_q, n_kv, dim, _log(rng, 512, hi), group)


def _case_of(kind, batch, n_q, n_kv, dim, seq_len, group, **more):
    c = _case("", kind, batch, n_q, n_kv, dim, seq_len, group=group, **more)
    del c["name"]
    return c


# ---- inputs, from the seed alone -----------------------------------------------------------------------------

def _device():
    return torch.device("cuda")


def _lengths(case, seed):
    """Every sequence's length: spread evenly over the logarithm of the range (so that a case is the same amount of
    work for every seed), in an order of the seed's."""
    n, lo, hi = case["batch"], case["min_len"], case["seq_len"]
    lens = [int(round(lo * (hi / lo) ** (i / max(1, n - 1)))) for i in range(n)]
    order = torch.randperm(n, generator=torch.Generator().manual_seed(seed)).tolist()
    return [lens[i] for i in order]


def _attn(case):
    """(attention scale, spread of q and K): d = 128 as the llama shapes, the others as the gemma shapes."""
    return (1.0 / math.sqrt(case["head_dim"]), 1.0) if case["head_dim"] == 128 else (1.0, 0.1)


class _Draws:
    """The case's tensors in a fixed order: queries, new tokens, then the cached tokens piece by piece."""

    def __init__(self, case, seed):
        self.case, dev = case, _device()
        self.gen = torch.Generator(device=dev).manual_seed(seed)
        self.std = _attn(case)[1]
        b, hq, hkv, d, nq = (case[k] for k in ("batch", "n_q_heads", "n_kv_heads", "head_dim", "n_queries"))
        # outlier key channels, four per KV head, eight times the others (d = 128 shapes)
        gain = torch.ones(hkv, d)
        if d == 128:
            host = torch.Generator().manual_seed(seed + 17)
            for h in range(hkv):
                gain[h, torch.randperm(d, generator=host)[:4]] = 8.0
        self.gain = gain.to(dev).reshape(1, hkv, 1, d)
        self.q = self.randn((b, nq, hq, d) if nq > 1 else (b, hq, d), self.std)
        self.k_new, self.v_new = self.kv(nq)

    def randn(self, shape, std):
        return (torch.randn(shape, generator=self.gen, device=_device()) * std).to(torch.float16)

    def kv(self, n):
        c = self.case
        shape = (c["batch"], c["n_kv_heads"], n, c["head_dim"])
        k = (torch.randn(shape, generator=self.gen, device=_device()) * (self.gain * self.std)).to(torch.float16)
        return k, self.randn(shape, 1.0)

    def pieces(self):
        c = self.case
        per = c["batch"] * c["n_kv_heads"] * c["head_dim"]
        step = max(32, PIECE // per // 32 * 32)
        for at in range(0, c["seq_len"], step):
            k, v = self.kv(min(step, c["seq_len"] - at))
            yield at, k, v


def prepare(case, seed):
    draws = _Draws(case, seed)
    b, hq, hkv, d, s = (case[k] for k in ("batch", "n_q_heads", "n_kv_heads", "head_dim", "seq_len"))
    st = {"case": case, "scale": _attn(case)[0]}
    if case["page"]:
        blocks = -(-s // case["page"])
        cache = tq.KVCache(b * blocks, hkv, d, case["page"], group_size=case["group"])
        order = torch.randperm(b * blocks, generator=torch.Generator().manual_seed(seed + 5))
        st["table"] = order.to(torch.int32).reshape(b, blocks).to(_device())
    else:
        cache = tq.KVCache(b, hkv, d, s, group_size=case["group"])
    for t in cache.tensors():
        t.zero_()
    st["cache"] = cache
    if case["kind"] == "prefill":
        pieces = list(draws.pieces())
        st["k"] = torch.cat([k for _, k, _ in pieces], dim=2).contiguous()
        st["v"] = torch.cat([v for _, _, v in pieces], dim=2).contiguous()
        return st
    for at, k, v in draws.pieces():
        if case["page"]:
            tq.tq_quantize_kv_paged(cache, st["table"], k, v, torch.full((b,), at, dtype=torch.int32, device=_device()))
        else:
            tq.tq_quantize_kv(cache, k, v, at)
    st["q"], st["k_new"], st["v_new"] = draws.q, draws.k_new, draws.v_new
    if case["kind"] in ("varlen", "paged"):
        st["lens"] = torch.tensor(_lengths(case, seed), dtype=torch.int32, device=_device())
    st["out"] = torch.zeros_like(draws.q)
    st["workspace"] = torch.empty(tq.tq_workspace_bytes(b * case["n_queries"], hq, d), dtype=torch.uint8, device=_device())
    return st


def run(st):
    """One call: the output (and the cache it wrote into)."""
    case, cache = st["case"], st["cache"]
    if case["kind"] == "prefill":
        tq.tq_quantize_kv(cache, st["k"], st["v"], 0)
        return cache.tensors()
    if case["kind"] == "varlen":
        tq.tq_sdpa_int4_append_decode_varlen(cache, st["k_new"], st["v_new"], st["q"], st["lens"], case["seq_len"],
                                             st["scale"], out=st["out"], workspace=st["workspace"])
    elif case["kind"] == "paged":
        tq.tq_sdpa_int4_append_decode_paged(cache, st["table"], st["k_new"], st["v_new"], st["q"], st["lens"],
                                            case["seq_len"], st["scale"], out=st["out"], workspace=st["workspace"])
    else:
        tq.tq_sdpa_int4_append_decode(cache, st["k_new"], st["v_new"], st["q"], case["seq_len"], st["scale"],
                                      out=st["out"], workspace=st["workspace"], window=case["window"])
    return (st["out"],) + cache.tensors()


def work(case):
    b, hq, hkv, d, nq = (case[k] for k in ("batch", "n_q_heads", "n_kv_heads", "head_dim", "n_queries"))
    row = 2 * hkv * (d // 2 + 4 * (d // case["group"]))          # packed bytes of one token, K and V
    if case["kind"] == "prefill":
        tokens = b * case["seq_len"]
        return {"bytes": tokens * (row + 2 * hkv * d * 2), "flops": 0}
    if case["kind"] in ("varlen", "paged"):
        tokens = sum(_lengths(case, 0))
    else:
        tokens = b * (min(case["seq_len"], case["window"] + nq - 1) if case["window"] else case["seq_len"])
    vectors = b * nq * d * 2 * (2 * hq + 2 * hkv)                # q in, out out, new tokens in
    return {"bytes": tokens * row + vectors, "flops": 4 * tokens * nq * hq * d}


def tolerance(case):
    # Stored codes, scales and zero-points are the same bits.  The attention output is rounded to fp16, and one
    # operand of each matrix product is (the weights, and the dequantised V at d = 512).  Measured against `exact`
    # over the listed cases and thirty drawn ones: relative error 1.9e-4 to 3.6e-4, the largest single one 1.8e-3
    # of the output's size; four times that.
    if case["kind"] == "prefill":
        return "exact"
    return {"rel": 1.4e-3, "max": 7.2e-3, "differ": 0.0}


# ---- the definition in 64 bits --------------------------------------------------------------------------------

def _quantize(x, group):
    """The stored format, from fp16 values [..., d]: scales, zero-points (fp16) and codes, with the fp32 steps of the
    definition (a 64-bit quotient rounded to fp32 is the correctly rounded fp32 quotient)."""
    g = x.float().reshape(x.shape[:-1] + (-1, group))
    mn, mx = g.amin(-1, keepdim=True), g.amax(-1, keepdim=True)
    s = ((mx - mn).double() / 15.0).float().half()
    s = torch.where(s == 0, torch.ones_like(s), s)
    z = ((-mn).double() / s.double()).float().half().clamp(-65504, 65504) + 0.0
    code = ((g.double() / s.double()).float() + z.float()).round().clamp(0, 15)
    return s, z, code


def _dequantized(x, group):
    s, z, code = _quantize(x, group)
    return ((code.double() - z.double()) * s.double()).reshape(x.shape)


def exact(case, seed):
    draws = _Draws(case, seed)
    b, hq, hkv, d, nq, group = (case[k] for k in ("batch", "n_q_heads", "n_kv_heads", "head_dim", "n_queries", "group"))
    if case["kind"] == "prefill":
        outs = []
        for i in (1, 2):                                         # scale = range / 15; zero-point from the stored scale
            x = torch.cat([p[i] for p in _Draws(case, seed).pieces()], dim=2)
            g = x.double().reshape(x.shape[:-1] + (-1, group))
            s, _, _ = _quantize(x, group)
            outs.append(((g.amax(-1) - g.amin(-1)) / 15.0, -g.amin(-1) / s.double().squeeze(-1)))
        return (None, outs[0][0], outs[0][1], None, outs[1][0], outs[1][1])
    lens = _lengths(case, seed) if case["kind"] in ("varlen", "paged") else [case["seq_len"]] * b
    scale, gqa = _attn(case)[0], hq // hkv
    rows = nq * gqa                                              # query rows per KV head: (query token, head)
    q = draws.q.double().reshape(b, nq, hkv, gqa, d).permute(0, 2, 1, 3, 4).reshape(b, hkv, rows, d)
    q = (q * scale).transpose(2, 3).contiguous()                 # [b, kv head, d, rows]
    dev = q.device
    own = torch.arange(nq, device=dev).repeat_interleave(gqa)    # a row's query token
    m = torch.full((b, hkv, rows), -math.inf, dtype=torch.float64, device=dev)
    l = torch.zeros_like(m)
    o = torch.zeros((b, hkv, rows, d), dtype=torch.float64, device=dev)

    def take(i, h, at, k, v):
        """Tokens at, at + 1, ... of sequence i (dequantised, one KV head) into the running softmax."""
        x = k @ q[i, h]                                          # [tokens, rows]
        tok = torch.arange(at, at + k.shape[0], device=dev).unsqueeze(1)
        end = lens[i] - (nq - 1 - own).unsqueeze(0)              # first token a row must not see
        seen = tok < end
        if case["window"]:
            seen &= tok >= end - case["window"]
        x = torch.where(seen, x, torch.full_like(x, -math.inf))
        top = torch.maximum(m[i, h], x.amax(0))
        ref = torch.where(torch.isinf(top), torch.zeros_like(top), top)
        keep, p = torch.exp(m[i, h] - ref), torch.exp(x - ref)
        l[i, h] = l[i, h] * keep + p.sum(0)
        o[i, h] = o[i, h] * keep.unsqueeze(1) + p.t().contiguous() @ v
        m[i, h] = top

    for at, k, v in draws.pieces():
        for i in range(b):
            n = min(k.shape[2], lens[i] - nq - at)               # (the step's own tokens replace what lies there)
            lo = max(0, lens[i] - nq - case["window"] - at) if case["window"] else 0
            if n <= lo:
                continue
            kd, vd = _dequantized(k[i, :, lo:n], group), _dequantized(v[i, :, lo:n], group)
            for h in range(hkv):
                take(i, h, at + lo, kd[h], vd[h])
    kd, vd = _dequantized(draws.k_new, group), _dequantized(draws.v_new, group)
    for i in range(b):
        for h in range(hkv):
            take(i, h, lens[i] - nq, kd[i, h], vd[i, h])
    out = (o / l.unsqueeze(-1)).reshape(b, hkv, nq, gqa, d).permute(0, 2, 1, 3, 4)
    out = out.reshape(b, nq, hq, d) if nq > 1 else out.reshape(b, hq, d)
    return (out,) + (None,) * 6
