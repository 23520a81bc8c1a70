"""GPU parity of the latent (grouped-query) path, Sec. 3.3.1 of arxiv 2508.10395:
xq_latent_project, xq_prepare_weights_latent, xq_remat_attn_decode_latent against the oracle."""
import numpy as np
import pytest
import torch

import xq_inputs as xi
from oracle import xq_oracle as xo
from tests.util import assert_cache_equals, bits_to_torch, oracle_cache, rel_errors, torch_to_bits

pytestmark = pytest.mark.gpu

TOL = 2e-3


@pytest.fixture(scope="module")
def xq():
    import paper_2508_10395_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.load_library()
    return m


def bf(x):
    return xi.from_bf16_bits(x)


def bits(x):
    return xi.to_bf16_bits(np.asarray(x, np.float32))


def _check_projection(got_bits, ref_bits, x_bits, ut_bits):
    """fp32 accumulation against the oracle's double: the same bf16 number or its neighbour, up to
    the fp32 accumulation error itself where the sum cancels to something tiny."""
    g, r = bf(got_bits).astype(np.float64), bf(ref_bits).astype(np.float64)
    ulp = 2.0 ** (np.floor(np.log2(np.maximum(np.abs(r), 1e-30))) - 7)
    absum = np.abs(bf(x_bits)).astype(np.float64) @ np.abs(bf(ut_bits)).astype(np.float64).T
    assert np.all(np.abs(g - r) <= ulp * 1.0001 + absum * 2.0 ** -20)
    assert np.mean(got_bits != ref_bits) < 5e-3


@pytest.mark.parametrize("M,d,n_lat", [(1, 256, 64), (16, 512, 256), (33, 384, 96), (300, 256, 512)])
def test_projection_matches_oracle(xq, M, d, n_lat):
    rng = np.random.default_rng(M + d)
    x = bits(rng.standard_normal((M, d)))
    ut = bits(rng.standard_normal((n_lat, d)) * d ** -0.5)
    out = torch.full((M, n_lat), 9.0, dtype=torch.bfloat16, device="cuda")
    xq.xq_latent_project(bits_to_torch(x), bits_to_torch(ut), out=out)
    torch.cuda.synchronize()
    _check_projection(torch_to_bits(out), xo.project_rows(x, ut), x, ut)


@pytest.mark.parametrize("M,d,n_lat", [(17, 128, 32), (33, 4224, 64), (16, 5120, 96), (256, 1024, 512), (257, 1024, 512)])
def test_projection_tiles(xq, M, d, n_lat):
    """Ragged row tiles, one step per wave, steps in rounds of loads of every size, either side of the larger tiles."""
    test_projection_matches_oracle(xq, M, d, n_lat)


@pytest.mark.parametrize("d,n_lat", [(4096, 512), (3968, 96), (128, 1024)])
def test_a_row_has_the_same_latents_however_many_rows_come_with_it(xq, d, n_lat):
    """One order of the sums for every number of rows: a token's latents have the same bits in a decode step as in a chunk."""
    gen = torch.Generator("cuda").manual_seed(d)
    x = torch.randn((1700, d), generator=gen, device="cuda").bfloat16()
    ut = torch.randn((n_lat, d), generator=gen, device="cuda").mul(d ** -0.5).bfloat16()
    want = xq.xq_latent_project(x, ut)
    for m in (1, 16, 17, 64, 128, 129, 300):
        for r0 in (0, 1700 - m):
            assert torch.equal(xq.xq_latent_project(x[r0:r0 + m].contiguous(), ut), want[r0:r0 + m]), (m, r0)


def test_projection_exact_case_and_noop(xq):
    rng = np.random.default_rng(5)
    x = rng.integers(-1, 2, size=(40, 256)).astype(np.float32)
    u = (rng.integers(0, 2, size=(256, 64)) * 2 - 1).astype(np.float32) / 16.0
    out = xq.xq_latent_project(bits_to_torch(bits(x)), bits_to_torch(bits(u.T)))
    torch.cuda.synchronize()
    assert np.array_equal(bf(torch_to_bits(out)).astype(np.float64), x.astype(np.float64) @ u.astype(np.float64))
    empty = torch.empty((0, 256), dtype=torch.bfloat16, device="cuda")
    assert xq.xq_latent_project(empty, bits_to_torch(bits(u.T))).shape == (0, 64)


def _svd_factors(w, cfg_seed):
    """Offline step: W [d][Hkv*hd] (bf16 bits) -> U^T [r][d] and S B^T [r][Hkv*hd], both rounded to bf16."""
    u, s, bt = np.linalg.svd(bf(w).astype(np.float64), full_matrices=False)
    return bits(u.T), bits(np.diag(s) @ bt)


def _run_latent(xq, w, bits_, G, lens, pairs=None):
    """The latent path twice on the GPU against ONE reference, the oracle's own chain (project, quantise, attend
    with the block-diagonal fused weights), on the sequences that the pairs name.

    End to end: the library keeps its own latent rows, quantises them and attends; nothing of the oracle's
    enters.  Its projection accumulates in fp32, the oracle's in double, so a few elements per thousand come
    out as the neighbouring bf16 number; such an element changes its own dequantised value by at most one
    quantisation step when it sits on a rounding boundary, and the scale or zero-point of its group by one
    bf16 ulp when it is the group's extreme.  The outputs are held to the same 2e-3 as everything else; the
    share of cache bytes that differ is reported.

    Stage by stage: the oracle's latent rows replace the library's on those sequences; now both sides quantise
    the same rows, so the caches must agree byte for byte, and each side attends over its own cache."""
    r = w.Hkv * w.hd
    x = xi.gen_x(w)
    wk, wv = xi.gen_weights(w)
    q = xi.gen_q(w)
    utk, wfk = _svd_factors(wk, 1)
    utv, wfv = _svd_factors(wv, 2)
    ut = np.concatenate([utk, utv], axis=0)                              # [2r][d]
    if pairs is None:
        pairs = [(b, h) for b in range(w.B) for h in range(w.Hq)]
    seqs = sorted({b for b, _ in pairs})
    attn = xq.XQAttn(w.Hq, w.Hkv, w.hd, w.hd ** -0.5)
    wprep = xq.xq_prepare_weights_latent(attn, r, G, bits_, bits_to_torch(wfk), bits_to_torch(wfv))
    lat = xq.xq_latent_project(bits_to_torch(x), bits_to_torch(ut))     # [B][L][2r]
    cache_own = xq.alloc_cache(w.B, w.L, 2 * r, G, bits_)
    xq.xq_quantize_append(cache_own, lat, [0] * w.B)
    out_own = xq.xq_remat_attn_decode_latent(attn, bits_to_torch(q), wprep, lens, cache_own)
    torch.cuda.synchronize()
    got_own = out_own.cpu().numpy()
    # the oracle's chain
    lat_ref = np.zeros((w.B, w.L, 2 * r), np.uint16)
    for b in seqs:
        lat_ref[b] = xo.project_rows(x[b], ut)
        _check_projection(torch_to_bits(lat[b]), lat_ref[b], x[b], ut)
    packed, scale, zero = oracle_cache(lat_ref, G, bits_, seqs=seqs)
    zk, zv = np.zeros_like(wfk), np.zeros_like(wfv)
    ref = xo.remat_attn_pairs(q_bf16=q, Wk=np.concatenate([wfk, zv], axis=0), Wv=np.concatenate([zk, wfv], axis=0),
                              Hq=w.Hq, Hkv=w.Hkv, hd=w.hd, softmax_scale=w.hd ** -0.5, lens=lens, pairs=pairs,
                              packed=packed, scale=scale, zero=zero, G=G, bits=bits_)
    # end to end
    sel = np.array([got_own[b, h] for b, h in pairs])
    normwise, maxwise = rel_errors(sel, ref)
    assert np.all(np.isfinite(sel)) and normwise.max() <= TOL and maxwise <= TOL, ("end to end", float(normwise.max()), float(maxwise))
    own_codes = cache_own.codes.cpu().numpy()
    byte_share = float(np.mean([np.mean(own_codes[b, :lens[b]] != packed[b, :lens[b]]) for b in seqs]))
    assert byte_share < 0.02, byte_share
    e2e = float(normwise.max())
    # stage by stage
    for b in seqs:
        lat[b] = bits_to_torch(lat_ref[b])
    cache = xq.alloc_cache(w.B, w.L, 2 * r, G, bits_)
    xq.xq_quantize_append(cache, lat, [0] * w.B)
    out = xq.xq_remat_attn_decode_latent(attn, bits_to_torch(q), wprep, lens, cache)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert_cache_equals(cache, packed, scale, zero, w.L, seqs=seqs)
    sel = np.array([got[b, h] for b, h in pairs])
    normwise, maxwise = rel_errors(sel, ref)
    assert np.all(np.isfinite(sel)) and normwise.max() <= TOL and maxwise <= TOL, (float(normwise.max()), float(maxwise))
    print(f"latent {w.name} {bits_}-bit G={G}: end to end {e2e:.2e} (cache bytes differing {byte_share:.2e}), "
          f"from shared latent rows {float(normwise.max()):.2e}")
    return float(normwise.max()), e2e


# (3- and 4-bit groups of 64 have no stream of 16-column fragments: their value pass runs on the 32x32x16 kernel)
@pytest.mark.parametrize("bits_,G", [(2, 64), (3, 128), (4, 128), (2, 128), (3, 64), (4, 64)])
def test_latent_pipeline_small(xq, bits_, G):
    w = xi.C4.scaled(B=3, L=420, d=512, Hq=8, Hkv=2, n_outlier=5)      # r = 256, g = 4
    _run_latent(xq, w, bits_, G, lens=[420, 257, 31])


@pytest.mark.parametrize("Hq,Hkv", [(2, 2), (4, 2), (12, 4), (16, 2), (32, 2)])
def test_latent_query_heads_per_kv_head(xq, Hq, Hkv):
    """1, 2, 3, 8 and 16 (the library's maximum) query heads per KV head: the value pass takes its 16 query rows per
    KV head in one group; ragged lengths across a tile boundary."""
    w = xi.C4.scaled(B=2, L=300, d=512, Hq=Hq, Hkv=Hkv, n_outlier=3)
    _run_latent(xq, w, 2, 64, lens=[300, 256])
    _run_latent(xq, w, 3, 128, lens=[1, 289])


def test_latent_close_to_plain_gqa_at_high_precision(xq):
    """4-bit latent cache against the same layer served from the 4-bit naive X cache: two different
    lossy encodings of the same K, V, so the outputs agree only roughly -- a sanity bound."""
    w = xi.C4.scaled(B=1, L=300, d=512, Hq=8, Hkv=2, n_outlier=0)
    r = w.Hkv * w.hd
    x, (wk, wv), q = xi.gen_x(w), xi.gen_weights(w), xi.gen_q(w)
    attn = xq.XQAttn(w.Hq, w.Hkv, w.hd, w.hd ** -0.5)
    cache = xq.alloc_cache(1, w.L, w.d, 128, 4)
    xq.xq_quantize_append(cache, bits_to_torch(x), [0])
    plain = xq.xq_remat_attn_decode(attn, bits_to_torch(q), xq.xq_prepare_weights(attn, w.d, 128, 4, bits_to_torch(wk),
                                    bits_to_torch(wv)), [w.L], xcache=cache).cpu().numpy()
    utk, wfk = _svd_factors(wk, 1)
    utv, wfv = _svd_factors(wv, 2)
    lat = xq.xq_latent_project(bits_to_torch(x), bits_to_torch(np.concatenate([utk, utv], axis=0)))
    lcache = xq.alloc_cache(1, w.L, 2 * r, 128, 4)
    xq.xq_quantize_append(lcache, lat, [0])
    wprep = xq.xq_prepare_weights_latent(attn, r, 128, 4, bits_to_torch(wfk), bits_to_torch(wfv))
    latent = xq.xq_remat_attn_decode_latent(attn, bits_to_torch(q), wprep, [w.L], lcache).cpu().numpy()
    normwise, _ = rel_errors(latent.reshape(-1, w.hd), plain.reshape(-1, w.hd))
    assert normwise.max() < 0.25


def test_full_size_llama3_8b_latent_sampled_pairs(xq):
    """Config 4's shape served from the latent cache (r = 1024, cache width 2048): B=16, L=8192,
    d=4096, 32 query / 8 KV heads, 2-bit, group 64."""
    w = xi.C4
    # the oracle projects every row of the compared sequences (13 s each on 8 cores): the sample keeps
    # to the first and the last sequence, with all four query heads of one KV head among its pairs
    pairs = [p for p in xi.sample_pairs(w, 8) if p[0] in (0, w.B - 1)] + [(w.B - 1, 9), (w.B - 1, 20)]
    worst, e2e = _run_latent(xq, w, w.bits, w.G, [w.L] * w.B, pairs=pairs)
    print(f"c4 latent sampled pairs: worst norm-wise rel err {worst:.2e}, end to end {e2e:.2e}")


@pytest.mark.parametrize("M,d,n_lat", [(1, 256, 256), (300, 256, 512), (777, 512, 256), (5000, 384, 768)])
def test_bulk_projection_matches_oracle(xq, M, d, n_lat):
    """The matrix-core route of the same projection (dense-source contraction kernel, rows stored as bf16)."""
    rng = np.random.default_rng(M + d + 1)
    x = bits(rng.standard_normal((M, d)))
    ut = bits(rng.standard_normal((n_lat, d)) * d ** -0.5)
    proj = xq.xq_prepare_projection(bits_to_torch(ut))
    out = torch.full((M, n_lat), 9.0, dtype=torch.bfloat16, device="cuda")
    xq.xq_latent_project_bulk(bits_to_torch(x), proj, n_lat, out=out)
    torch.cuda.synchronize()
    sample = np.unique(np.concatenate([np.arange(min(M, 40)), np.arange(max(M - 40, 0), M), rng.integers(0, M, 60)]))
    _check_projection(torch_to_bits(out)[sample], xo.project_rows(x[sample], ut), x[sample], ut)
    small = xq.xq_latent_project(bits_to_torch(x[sample]), bits_to_torch(ut))
    assert np.mean(torch_to_bits(small) != torch_to_bits(out)[sample]) < 5e-3      # two accumulation orders of the same sum
    assert xq.xq_latent_project_bulk(torch.empty((0, d), dtype=torch.bfloat16, device="cuda"), proj, n_lat).shape == (0, n_lat)
