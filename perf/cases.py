"""The work that a user of this library has it do, as cases to be measured: one layer's share of a prefill chunk or of a
decode step, through the entry points of `paper_2508_10395_amd`, on synthetic tensors of the shapes that `xq_inputs`
names (Llama-2-7B- and Llama-3-8B-shaped layers), from the small layer of its first workload to contexts of 32768.

A case is a dict of plain values; `kind` says which calls a pass makes:

  append       quantise a chunk of T new rows per sequence into the X cache (prefill)
  decode       append one token per sequence, attend over the X cache (rope: keys rotated)
  prefill      append T tokens per sequence, causal attention of these T queries
  cl_prefill   cross-layer chunk: load the base layer into the accumulator, quantise the chunk's deltas, merge them
  cl_decode    cross-layer decode step: base layer and deltas into the accumulator, attend from it
  latent       grouped-query latent cache: project and append one token, attend (keys per token or per channel)
  per_channel  attend over a per-channel cache and its residual window (terms recomputed or kept)
  cl_gqa       cross-layer deltas of a grouped-query model: project and append one token's latent delta, merge the
               latent deltas into the accumulator, attend from it

Inputs come from the seed alone.  X ~ N(0, 1) with one channel in a hundred 30 times larger, weights ~ N(0, 1/d),
queries ~ N(0, 1), as in `xq_inputs`.
"""
import math

import torch

import paper_2508_10395_amd as xq

HD = 128
DEV = "cuda"


# ---------------------------------------------------------------------------------------------- the cases

def listed():
    return [
        # the smallest call there is: a short context on a small layer (first workload of xq_inputs); launches and latency
        _case("decode_small", "decode", B=1, L=512, d=256, Hq=2, Hkv=2, bits=4, group=128),
        # decode step of a Llama-2-7B-shaped layer, batch 8, 4096 tokens, 3 bits: the benchmark's own step
        _case("decode_mha", "decode", B=8, L=4096, d=4096, Hq=32, Hkv=32, bits=3, group=128),
        # decode step of a Llama-3-8B-shaped layer, 2 bits in groups of 64, sequences of different lengths
        _case("decode_gqa", "decode", B=16, L=8191, d=4096, Hq=32, Hkv=8, bits=2, group=64, ragged=True),
        # long contexts, 2 bits: the largest case
        _case("decode_long", "decode", B=4, L=32768, d=4096, Hq=32, Hkv=32, bits=2, group=128),
        # decode step of a rotary model from a 4-bit cache, sequences of different lengths, odd batch
        _case("decode_rope", "decode", B=5, L=4001, d=4096, Hq=32, Hkv=8, bits=4, group=128, ragged=True, rope=True),
        # a chunk of a chunked prefill, rotary model, causal
        _case("prefill_chunk", "prefill", B=2, L=4096, T=128, d=4096, Hq=32, Hkv=32, bits=3, group=128, rope=True),
        # prompts go into the cache: bulk quantisation
        _case("append_prompt", "append", B=8, L=4096, T=4096, d=4096, bits=3, group=128),
        # cross-layer prefill of a chunk: base layer, deltas of the chunk, merge
        _case("cl_prefill", "cl_prefill", B=4, L=4000, T=1000, d=4096, bits=2, group=128, base_bits=4),
        # cross-layer decode step, 4-bit base and 2-bit deltas
        _case("cl_decode", "cl_decode", B=4, L=6000, d=4096, Hq=32, Hkv=32, bits=2, group=128, base_bits=4, ragged=True),
        # latent cache of a grouped-query layer
        _case("latent_decode", "latent", B=16, L=8192, d=4096, Hq=32, Hkv=8, bits=2, group=64),
        # per-channel groups with a residual window, block terms kept by the caller
        _case("per_channel", "per_channel", B=8, L=4077, d=4096, Hq=32, Hkv=32, bits=3, group=128, terms=True, ragged=True),
        # cross-layer deltas of a grouped-query layer
        _case("cl_gqa", "cl_gqa", B=4, L=4096, d=4096, Hq=32, Hkv=8, bits=2, group=64, base_bits=4),
    ]


def _case(name, kind, **kw):
    c = {"name": name, "kind": kind, "B": 1, "L": 1, "T": 1, "d": 256, "Hq": 2, "Hkv": 2, "bits": 4, "group": 128,
         "ragged": False, "rope": False, "base_bits": 4, "terms": False, "per_channel_keys": False}
    c.update(kw)
    return c


_KINDS = ["decode", "decode", "decode", "decode", "decode", "prefill", "append", "cl_prefill", "cl_decode", "latent",
          "per_channel", "cl_gqa"]
_MOST_TOKENS_X_D = 4 * 32768 * 4096                       # of the largest listed case


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(_KINDS)
    group = rng.choice([64, 128])
    bits = rng.choice([2, 3, 4, 8]) if kind in ("decode", "prefill", "append") else rng.choice([2, 3, 4])
    if kind in ("latent", "cl_gqa"):
        Hkv = rng.choice([2, 4, 8])
        gq = rng.choice([2, 4, 8])
    else:
        Hkv = rng.choice([2, 4, 8, 32, 40])
        gq = rng.choice([1, 2, 4, 8]) if Hkv <= 8 else 1
    d = rng.choice([256, 512, 1024, 2048, 4096, 5120])
    if kind in ("latent", "cl_gqa"):
        d = max(d, 2 * Hkv * HD)
    T = 1
    if kind == "prefill":
        T = _log_int(rng, 2, 512)
    B = _log_int(rng, 1, 16)
    most_l = 32768 if kind == "decode" else 8192
    cap = _MOST_TOKENS_X_D // 8 if kind in ("prefill", "cl_decode", "cl_gqa", "cl_prefill") else _MOST_TOKENS_X_D // 2
    # (the cost of an attention pass goes with the columns of the weights too: never above that of the largest listed case)
    if kind not in ("append", "cl_prefill"):
        cap = min(cap, int(_MOST_TOKENS_X_D * 4096 / (max(Hkv, 8) * HD) / (1 if kind != "prefill" else 8)))
        if bits == 8:
            cap //= 2
    L = _log_int(rng, max(T, 2), most_l)
    while B > 1 and B * L * d > cap:
        B -= 1
    L = max(T, 2, min(L, cap // (B * d)))
    if kind in ("append", "cl_prefill"):
        T = _log_int(rng, 1, L)
    c = _case("drawn", kind, B=B, L=L, T=T, d=d, Hq=Hkv * gq, Hkv=Hkv, bits=bits, group=group,
              ragged=rng.random() < 0.6 and kind not in ("append", "cl_prefill"), base_bits=rng.choice([3, 4]),
              rope=kind in ("decode", "prefill") and rng.random() < 0.4, terms=rng.random() < 0.5,
              per_channel_keys=kind == "latent" and rng.random() < 0.4)
    del c["name"]
    return c


def _lens(c):
    """Rows attended per sequence (or, for the chunk kinds, rows that hold something), the newest T included."""
    B, L, T = c["B"], c["L"], c["T"]
    if not c["ragged"]:
        return [L] * B
    return [max(T, L - (b * b * 37 + b * 113) % max(1, L // 2)) for b in range(B)]


# ---------------------------------------------------------------------------------------------- inputs

def _gen(seed, tag):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + tag) % (1 << 62))
    return g


def _outlier_scale(c, seed, n):
    """Column factors of X: one channel in a hundred is 30 times larger."""
    g = torch.Generator()
    g.manual_seed(int(seed) + 77)
    col = torch.ones(n)
    col[torch.randperm(n, generator=g)[:max(1, n // 100)]] = 30.0
    return col.to(DEV)


def _rows(seed, tag, B, L, d, col=None):
    x = torch.empty((B, L, d), dtype=torch.bfloat16, device=DEV)
    g = _gen(seed, tag)
    for b in range(B):
        r = torch.randn((L, d), generator=g, device=DEV)
        x[b] = r if col is None else r * col
    return x


def _weights(seed, tag, rows, cols, std):
    return (torch.randn((rows, cols), generator=_gen(seed, tag), device=DEV) * std).to(torch.bfloat16)


def _basis_t(seed, tag, n_lat, d):
    """n_lat orthonormal directions of the hidden space, [n_lat][d] bf16 (what the offline SVD hands over, transposed)."""
    q, _ = torch.linalg.qr(torch.randn((d, n_lat), generator=_gen(seed, tag), device=DEV))
    return q.t().contiguous().to(torch.bfloat16)


def _rope_table(n):
    pos = torch.arange(n, dtype=torch.float64)[:, None]
    ang = pos * (10000.0 ** (-torch.arange(HD // 2, dtype=torch.float64) / (HD // 2)))[None]
    return torch.stack([ang.cos(), ang.sin()], dim=-1).float().to(DEV).contiguous()


def _inputs(c, seed):
    """Every random tensor of the case, from the seed alone."""
    B, L, T, d, Hq, Hkv, kind = c["B"], c["L"], c["T"], c["d"], c["Hq"], c["Hkv"], c["kind"]
    i = {}
    if kind in ("append", "decode", "prefill", "per_channel"):
        i["x"] = _rows(seed, 1, B, L, d, _outlier_scale(c, seed, d))
    if kind in ("cl_prefill", "cl_decode", "cl_gqa"):
        i["x0"] = _rows(seed, 1, B, L, d)                                     # base layer
        g = _gen(seed, 2)
        i["x1"] = torch.empty_like(i["x0"])                                   # next layer: a small step away
        for b in range(B):
            i["x1"][b] = i["x0"][b].float() + math.sqrt(0.1) * torch.randn((L, d), generator=g, device=DEV)
    if kind in ("decode", "prefill", "per_channel", "cl_decode", "cl_gqa"):
        i["wk"] = _weights(seed, 3, d, Hkv * HD, d ** -0.5)
        i["wv"] = _weights(seed, 4, d, Hkv * HD, d ** -0.5)
    if kind == "latent":
        r = Hkv * HD
        col = torch.ones(2 * r, device=DEV)
        col[0] = 25.0                                                         # X Uk collects the outliers in its first channel
        i["lat"] = _rows(seed, 1, B, L, 2 * r, col)
        i["x_new"] = _rows(seed, 5, B, 1, d)
        i["ut"] = _basis_t(seed, 6, 2 * r, d)
        i["wk"] = _weights(seed, 3, r, r, r ** -0.5)
        i["wv"] = _weights(seed, 4, r, r, r ** -0.5)
    if kind == "cl_gqa":
        i["ut"] = _basis_t(seed, 6, 2 * Hkv * HD, d)
    if kind not in ("append", "cl_prefill"):
        shape = (B, T, Hq, HD) if kind == "prefill" else (B, Hq, HD)
        i["q"] = torch.randn(shape, generator=_gen(seed, 7), device=DEV).to(torch.bfloat16)
    if c["rope"]:
        i["rope"] = _rope_table(L + 16)
        i["pos0"] = [b % 16 for b in range(B)]
    return i


def _newest(x, lens, T):
    return torch.stack([x[b, n - T:n] for b, n in enumerate(lens)]).contiguous()


def _attn(c):
    return xq.XQAttn(c["Hq"], c["Hkv"], HD, HD ** -0.5)


def _ws(n):
    return torch.empty(max(n, 16), dtype=torch.uint8, device=DEV)


# ---------------------------------------------------------------------------------------------- one pass

def prepare(c, seed):
    i = _inputs(c, seed)
    B, L, T, d, bits, G, kind = c["B"], c["L"], c["T"], c["d"], c["bits"], c["group"], c["kind"]
    lens = _lens(c)
    s = {"case": c, "lens": lens}
    if kind in ("append", "decode", "prefill"):
        s["cache"] = xq.alloc_cache(B, L, d, G, bits)
        s["start"] = [n - T for n in lens]
        s["x_new"] = _newest(i["x"], lens, T)
        if kind != "append":
            xq.xq_quantize_append(s["cache"], i["x"], [0] * B)               # the rows cached so far
    if kind in ("decode", "prefill"):
        s["attn"] = _attn(c)
        s["wprep"] = xq.xq_prepare_weights(s["attn"], d, G, bits, i["wk"], i["wv"])
        walk = (2 * d, 128) if bits == 8 else (d, G)
        if kind == "decode":
            s["ws"] = _ws(xq.xq_remat_attn_workspace_bytes(s["attn"], B, max(lens), *walk))
        else:
            s["ws"] = _ws(xq.xq_remat_attn_prefill_workspace_bytes(s["attn"], B, T, max(lens), *walk))
        s["out"] = torch.empty(i["q"].shape, dtype=torch.float32, device=DEV)
    if kind == "per_channel":
        s["attn"] = _attn(c)
        nblk = L // G
        s["cache"] = xq.alloc_cache_per_channel(B, max(1, nblk) * G, d, G, bits)
        if nblk:
            xq.xq_quantize_blocks_per_channel(s["cache"], i["x"][:, :nblk * G].contiguous(), [0] * B)
        s["tail"] = _tail(i["x"], lens, G)
        s["wc"] = xq.xq_prepare_weights(s["attn"], d, 128, bits, i["wk"], i["wv"])
        s["wd"] = xq.xq_prepare_weights(s["attn"], d, 0, 16, i["wk"], i["wv"])
        s["ws"] = _ws(xq.xq_remat_attn_per_channel_workspace_bytes(s["attn"], B, max(lens), d, G))
        s["out"] = torch.empty((B, c["Hq"], HD), dtype=torch.float32, device=DEV)
        s["terms"] = xq.alloc_per_channel_terms(s["cache"], c["Hkv"]) if c["terms"] else None
    if kind in ("cl_prefill", "cl_decode", "cl_gqa"):
        s["base"] = xq.alloc_cache(B, L, d, G, c["base_bits"])
        xq.xq_quantize_append(s["base"], i["x0"], [0] * B)
        s["acc"] = torch.zeros((B, L, d), dtype=torch.bfloat16, device=DEV)
        s["start"] = [n - T for n in lens]
        s["x_new"] = _newest(i["x1"], lens, T)
    if kind in ("cl_prefill", "cl_decode"):
        s["delta"] = xq.alloc_cache(B, L, d, G, bits)
        xq.xq_cl_accumulate(s["acc"], s["base"], [L] * B, True)
        xq.xq_cl_delta_quantize(s["delta"], i["x1"], s["acc"], [0] * B)      # the rows cached so far
    if kind == "cl_gqa":
        n_lat = i["ut"].shape[0]
        s["ut"] = i["ut"]
        s["delta"] = xq.alloc_cache(B, L, n_lat, G, bits)
        xq.xq_cl_accumulate(s["acc"], s["base"], [L] * B, True)
        xq.xq_quantize_append(s["delta"], _small_latents(c, seed, n_lat), [0] * B)
        s["uprep"] = xq.xq_prepare_upproject(d, G, bits, i["ut"])
        s["up_ws"] = _ws(xq.xq_cl_accumulate_latent_workspace_bytes(B, max(lens), n_lat, G))
    if kind in ("cl_decode", "cl_gqa"):
        s["attn"] = _attn(c)
        s["wprep"] = xq.xq_prepare_weights(s["attn"], d, 0, 16, i["wk"], i["wv"])
        s["ws"] = _ws(xq.xq_remat_attn_workspace_bytes(s["attn"], B, max(lens), d, 0))
        s["out"] = torch.empty((B, c["Hq"], HD), dtype=torch.float32, device=DEV)
    if kind == "latent":
        s["attn"] = _attn(c)
        r = c["Hkv"] * HD
        s["ut"], s["x_new"], s["start"] = i["ut"], i["x_new"], [n - 1 for n in lens]
        s["out"] = torch.empty((B, c["Hq"], HD), dtype=torch.float32, device=DEV)
        if c["per_channel_keys"]:
            nblk = L // G
            s["kc"] = xq.alloc_cache_per_channel(B, max(1, nblk) * G, r, G, bits)
            if nblk:
                xq.xq_quantize_blocks_per_channel(s["kc"], i["lat"][:, :nblk * G, :r].contiguous(), [0] * B)
            s["ktail"] = _tail(i["lat"][:, :, :r], lens, G)
            s["vc"] = xq.alloc_cache(B, L, r, G, bits)
            xq.xq_quantize_append(s["vc"], i["lat"][:, :, r:].contiguous(), [0] * B)
            s["wkc"] = xq.xq_prepare_weights_pairs(s["attn"], r, 128, bits, i["wk"])
            s["wkd"] = xq.xq_prepare_weights_pairs(s["attn"], r, 0, 16, i["wk"])
            s["wvc"] = xq.xq_prepare_weights_pairs(s["attn"], r, G, bits, i["wv"])
            s["ws"] = _ws(xq.xq_remat_attn_latent_per_channel_workspace_bytes(s["attn"], B, max(lens), r, G, G))
            s["terms"] = xq.alloc_per_channel_terms(s["kc"], c["Hkv"] // 2) if c["terms"] else None
        else:
            s["cache"] = xq.alloc_cache(B, L, 2 * r, G, bits)
            xq.xq_quantize_append(s["cache"], i["lat"], [0] * B)
            s["wprep"] = xq.xq_prepare_weights_latent(s["attn"], r, G, bits, i["wk"], i["wv"])
            s["ws"] = _ws(xq.xq_remat_attn_latent_workspace_bytes(s["attn"], B, max(lens), r, G))
    if "q" in i:
        s["q"] = i["q"]
    if c["rope"]:
        s["rope"], s["pos0"] = i["rope"], i["pos0"]
    if s.get("terms") is not None:                                            # terms as the step after a block's completion leaves them
        _attend(s, valid=False)
    return s


def _tail(x, lens, G):
    t = torch.zeros((x.shape[0], G, x.shape[2]), dtype=torch.bfloat16, device=DEV)
    for b, n in enumerate(lens):
        k = n // G * G
        t[b, :n - k] = x[b, k:n]
    return t


def _small_latents(c, seed, n_lat):
    return (_rows(seed, 8, c["B"], c["L"], n_lat).float() * math.sqrt(0.1)).to(torch.bfloat16)


def _attend(s, valid=True):
    c = s["case"]
    if c["kind"] == "per_channel":
        return xq.xq_remat_attn_decode_per_channel(s["attn"], s["q"], s["cache"], s["tail"], s["lens"], s["wc"], s["wd"], out=s["out"],
                                                   workspace=s["ws"], terms=s["terms"], terms_valid=valid and s["terms"] is not None)
    return xq.xq_remat_attn_decode_latent_per_channel(s["attn"], s["q"], s["kc"], s["ktail"], s["vc"], s["wkc"], s["wkd"], s["wvc"],
                                                      s["lens"], out=s["out"], workspace=s["ws"], terms=s["terms"],
                                                      terms_valid=valid and s["terms"] is not None)


def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind in ("append", "decode", "prefill"):
        k = s["cache"]
        xq.xq_quantize_append(k, s["x_new"], s["start"])
        got = {"codes": k.codes, "scale": k.scale, "zero": k.zero}
        rope = dict(rope_cos_sin=s["rope"], pos0=s["pos0"]) if c["rope"] else {}
        if kind == "decode":
            got["out"] = xq.xq_remat_attn_decode(s["attn"], s["q"], s["wprep"], s["lens"], xcache=k, out=s["out"], workspace=s["ws"], **rope)
        elif kind == "prefill":
            got["out"] = xq.xq_remat_attn_prefill(s["attn"], s["q"], s["wprep"], s["lens"], xcache=k, out=s["out"], workspace=s["ws"], **rope)
        return got
    if kind in ("cl_prefill", "cl_decode"):
        k, acc, lens = s["delta"], s["acc"], s["lens"]
        xq.xq_cl_accumulate(acc, s["base"], lens, True)
        xq.xq_cl_delta_quantize(k, s["x_new"], acc, s["start"])
        xq.xq_cl_accumulate(acc, k, lens, False)
        got = {"acc": acc, "codes": k.codes, "scale": k.scale, "zero": k.zero}
        if kind == "cl_decode":
            got["out"] = xq.xq_remat_attn_decode(s["attn"], s["q"], s["wprep"], lens, acc_bf16=acc, out=s["out"], workspace=s["ws"])
        return got
    if kind == "cl_gqa":
        k, acc, lens = s["delta"], s["acc"], s["lens"]
        xq.xq_cl_accumulate(acc, s["base"], lens, True)
        new = xq.xq_cl_latent_delta_project(s["x_new"], acc, s["ut"], s["start"])
        xq.xq_quantize_append(k, new, s["start"])
        xq.xq_cl_accumulate_latent(acc, k, s["uprep"], lens, workspace=s["up_ws"])
        out = xq.xq_remat_attn_decode(s["attn"], s["q"], s["wprep"], lens, acc_bf16=acc, out=s["out"], workspace=s["ws"])
        return {"acc": acc, "new": new, "out": out}
    if kind == "latent":
        new = xq.xq_latent_project(s["x_new"], s["ut"])
        if c["per_channel_keys"]:                         # (the new token's key latents wait in the window, which the caller keeps)
            r = c["Hkv"] * HD
            xq.xq_quantize_append(s["vc"], new[:, :, r:].contiguous(), s["start"])
            return {"new": new, "codes": s["vc"].codes, "scale": s["vc"].scale, "zero": s["vc"].zero, "out": _attend(s)}
        k = s["cache"]
        xq.xq_quantize_append(k, new, s["start"])
        out = xq.xq_remat_attn_decode_latent(s["attn"], s["q"], s["wprep"], s["lens"], k, out=s["out"], workspace=s["ws"])
        return {"new": new, "codes": k.codes, "scale": k.scale, "zero": k.zero, "out": out}
    return {"out": _attend(s)}


# ---------------------------------------------------------------------------------------------- what a pass cannot do without

def work(c):
    """Bytes: every input read once, every output written once.  Operations: those of the cheapest order in which the
    products can be taken; for one query per sequence that is (q Wk^T) X^T and (p X) Wv."""
    B, T, d, bits, G, Hq, Hkv, kind = c["B"], c["T"], c["d"], c["bits"], c["group"], c["Hq"], c["Hkv"], c["kind"]
    M = sum(_lens(c))
    row = d * bits / 8 + 4 * d / G
    wbytes = 2 * d * Hkv * HD * 2
    io = B * T * Hq * HD * (2 + 4)
    if kind == "append":
        return {"bytes": B * T * (2 * d + row), "flops": 0}
    base_row = d * c["base_bits"] / 8 + 4 * d / G
    if kind == "cl_prefill":
        return {"bytes": B * T * (2 * d + row) + M * (base_row + row + 2 * d), "flops": 2 * M * d}
    rows = T * Hq
    absorbed = 4 * M * d * rows + 4 * B * d * rows * HD
    remat = 4 * M * d * Hkv * HD + 4 * M * rows * HD
    half = remat / 2 + absorbed / 2                                     # rotated keys have to be there one by one
    flops = min(half if c["rope"] else absorbed, remat)
    if kind in ("decode", "prefill"):
        return {"bytes": B * T * 2 * d + M * row + wbytes + io + (M * HD * 4 / B if c["rope"] else 0), "flops": flops}
    if kind == "per_channel":
        return {"bytes": M * row + wbytes + io, "flops": flops}
    if kind == "cl_decode":
        return {"bytes": B * 4 * d + M * (base_row + row + 2 * d) + wbytes + io, "flops": flops + 2 * M * d}
    r = Hkv * HD
    if kind == "latent":
        return {"bytes": M * (2 * r * bits / 8 + 8 * r / G) + 2 * r * d * 2 + 2 * r * r * 2 + B * 2 * d + io,
                "flops": 4 * M * r * Hq + 4 * B * r * Hq * HD + 4 * B * d * r}
    return {"bytes": M * (base_row + 2 * r * bits / 8 + 8 * r / G + 2 * d) + 2 * r * d * 2 * 2 + wbytes + io + B * 2 * d,
            "flops": flops + 4 * M * d * r + 4 * B * d * r}


# relative error of the start's outputs against 64 bits, times four and rounded up: see tolerance()
_REL = {"decode": 3e-5, "prefill": 4e-5, "per_channel": 2e-5, "cl_decode": 4e-6, "latent": 8e-5, "cl_gqa": 1.2e-4}


def tolerance(c):
    """Codes, scales, zero-points and the element-wise accumulator are defined bit for bit.  Attention outputs sum thousands
    of 32-bit products whose order is free; large group offsets cancel in them.  Latent rows are rounded to bf16 after a 32-bit
    sum, so one in a thousand falls to the neighbouring number, and its code with it."""
    kind = c["kind"]
    if kind in ("append", "cl_prefill"):
        return "exact"
    return {"rel": _REL[kind], "max": min(0.9, 40 * _REL[kind])}


# ---------------------------------------------------------------------------------------------- the same in 64 bits

def _bf16(x):
    return x.float().to(torch.bfloat16).double()


def _f32(x):
    return x.float().double()


def _dequantised(x, G, bits):
    """Rows x (64-bit, last axis grouped) through the quantiser that the storage format defines, and back: the definition's
    32-bit roundings where it has them, the rest exact."""
    shape = x.shape
    g = x.reshape(*shape[:-1], shape[-1] // G, G)
    mn, mx = g.amin(-1, keepdim=True), g.amax(-1, keepdim=True)
    zero = _bf16(mn)
    scale = _bf16(_f32(_f32(mx - mn) / ((1 << bits) - 1)))
    safe = torch.where(scale == 0, torch.ones_like(scale), scale)
    code = torch.round(_f32(_f32(g - zero) / safe)).clamp_(0, (1 << bits) - 1)
    return (torch.where(scale == 0, torch.zeros_like(code), code) * scale + zero).reshape(shape)


def _dequantised_blocks(x, G, bits):
    """The same with groups along the token axis, [n G][d]."""
    n = x.shape[0] // G
    t = x.reshape(n, G, -1).transpose(1, 2).contiguous()
    return _dequantised(t, G, bits).transpose(1, 2).reshape(x.shape)


def _attention(c, xk, xv, wk, wv, q, rope=None, pos0=0):
    """q [T][Hq][128] against the rows xk, xv (64-bit); query t sees rows up to len - T + t."""
    n, T, gq = xk.shape[0], q.shape[0], c["Hq"] // c["Hkv"]
    out = torch.empty((T, c["Hq"], HD), dtype=torch.float64, device=DEV)
    seen = torch.arange(n, device=DEV)[None, :] <= (n - T + torch.arange(T, device=DEV))[:, None]
    for h in range(c["Hkv"]):
        k, v = xk @ wk[:, h * HD:(h + 1) * HD], xv @ wv[:, h * HD:(h + 1) * HD]
        if rope is not None:
            cs = rope[pos0:pos0 + n].double()
            a, b = k[:, :64], k[:, 64:]
            k = torch.cat([a * cs[..., 0] - b * cs[..., 1], b * cs[..., 0] + a * cs[..., 1]], dim=1)
        for j in range(h * gq, (h + 1) * gq):
            sc = (q[:, j].double() @ k.t().contiguous()) * HD ** -0.5
            out[:, j] = torch.softmax(sc.masked_fill(~seen, -math.inf), dim=1) @ v
    return out


def exact(c, seed):
    kind, G, bits, B, T, L = c["kind"], c["group"], c["bits"], c["B"], c["T"], c["L"]
    if kind in ("append",):
        return None                                                     # whole numbers and stored bytes only
    i = _inputs(c, seed)
    lens = _lens(c)
    r = c["Hkv"] * HD
    q = i["q"].reshape(B, T, c["Hq"], HD) if "q" in i else None
    wk, wv = (i["wk"].double(), i["wv"].double()) if "wk" in i else (None, None)
    out = []
    if kind in ("decode", "prefill"):
        for b, n in enumerate(lens):
            x = _dequantised(i["x"][b, :n].double(), G, bits)
            out.append(_attention(c, x, x, wk, wv, q[b], i.get("rope"), i["pos0"][b] if c["rope"] else 0))
        return {"codes": None, "scale": None, "zero": None, "out": torch.stack(out).reshape(i["q"].shape)}
    if kind == "per_channel":
        for b, n in enumerate(lens):
            k = n // G * G
            x = i["x"][b, :n].double()
            x = torch.cat([_dequantised_blocks(x[:k], G, bits), x[k:]])
            out.append(_attention(c, x, x, wk, wv, q[b]))
        return {"out": torch.cat(out)}
    if kind in ("cl_prefill", "cl_decode", "cl_gqa"):
        acc = torch.zeros((B, L, c["d"]), dtype=torch.bfloat16, device=DEV)
        new = []
        small = _small_latents(c, seed, 2 * r) if kind == "cl_gqa" else None
        for b, n in enumerate(lens):
            a = _bf16(_dequantised(i["x0"][b].double(), G, c["base_bits"]))
            if kind == "cl_gqa":
                ut = i["ut"].double()
                lat = small[b].double()
                lat[n - 1] = _bf16((i["x1"][b, n - 1].double() - a[n - 1])[None] @ ut.t().contiguous())[0]
                new.append(lat[n - 1:n].clone())
                a = _bf16(a + _dequantised(lat, G, bits) @ ut)
            else:
                # (value and sum of the definition are rounded to 32 bits, then to bf16)
                a = _bf16(_f32(a + _f32(_dequantised(_f32(i["x1"][b].double() - a), G, bits))))
            acc[b, :n] = a[:n].to(torch.bfloat16)
            if n < L:                                                   # rows past the length keep what the set-up left there
                acc[b, n:] = _bf16(_dequantised(i["x0"][b, n:].double(), G, c["base_bits"])).to(torch.bfloat16)
            if q is not None:
                x = a[:n]
                out.append(_attention(c, x, x, wk, wv, q[b]))
        got = {"acc": acc}
        if kind == "cl_gqa":
            got["new"] = torch.stack(new)
        else:
            got.update(codes=None, scale=None, zero=None)
        if q is not None:
            got["out"] = torch.cat(out)
        return got
    new = i["x_new"].double() @ i["ut"].double().t().contiguous()
    for b, n in enumerate(lens):
        lat = i["lat"][b, :n].double()
        xk, xv = lat[:, :r].clone(), lat[:, r:].clone()
        row = _bf16(new[b, 0])
        xv[n - 1] = row[r:]
        if c["per_channel_keys"]:
            k = n // G * G
            xk = torch.cat([_dequantised_blocks(xk[:k], G, bits), xk[k:]])
        else:
            xk[n - 1] = row[:r]
            xk = _dequantised(xk, G, bits)
        out.append(_attention(c, xk, _dequantised(xv, G, bits), wk, wv, q[b]))
    return {"new": _bf16(new), "codes": None, "scale": None, "zero": None, "out": torch.cat(out)}
