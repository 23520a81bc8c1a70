"""GPU parity of the folded decode kernels (the query times Wk, then scores and weighted sums over the codes) against the
CPU oracle, at the sizes where their tiles and splits end: 128-token score tiles, 256-token value tiles, pairs of 128-channel
slabs, 16- and 32-row query blocks, launch groups of a small workspace."""
import numpy as np
import pytest
import torch

import xq_inputs as xi
from oracle import xq_oracle as xo
from tests.test_gpu_per_channel import _attend
from tests.util import bits_to_torch, oracle_cache, oracle_cache_per_channel, rel_errors

pytestmark = pytest.mark.gpu

# The folded operands keep 22 bits and the sums are fp32, so a score of magnitude <= 2^4 is off by at most 2^4 (2^-21 plus a
# random walk of 2^-24 over 2^12 terms) < 2^-15 in log2 units: weights and outputs within 2^-15; 4 times that here.
TOL = 2.0 ** -13


@pytest.fixture(scope="module")
def xq():
    import paper_2508_10395_amd as m
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    m.load_library()
    return m


def _kernels(call):
    """Names of the kernels that a call launches."""
    torch.cuda.synchronize()
    with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    return [e.name for e in p.events()]


def _folds(call):
    names = _kernels(call)
    folded = any("fold_scores" in n for n in names)
    assert folded != any("remat_attn" in n for n in names), names
    return folded


def _step(xq, B, L, d, Hq, Hkv, bits, G=128, per_channel=False, terms=False):
    """One decode step on caches of arbitrary codes, as a call without arguments."""
    gen = torch.Generator("cuda").manual_seed(B * L + d)
    attn = xq.XQAttn(Hq, Hkv, 128, 128 ** -0.5)
    wk, wv = (torch.randn((d, Hkv * 128), generator=gen, device="cuda").mul(d ** -0.5).bfloat16() for _ in range(2))
    q = torch.randn((B, Hq, 128), generator=gen, device="cuda").bfloat16()
    lens = [L - b % 3 for b in range(B)]
    if bits == 16:
        x = torch.randn((B, L, d), generator=gen, device="cuda", dtype=torch.bfloat16)
        wp = xq.xq_prepare_weights(attn, d, 0, 16, wk, wv)
        return lambda: xq.xq_remat_attn_decode(attn, q, wp, lens, acc_bf16=x)
    groups = (L // G, d) if per_channel else (L, d // G)
    codes = torch.randint(0, 256, (B, L // G * G if per_channel else L, d * bits // 8), generator=gen, device="cuda", dtype=torch.uint8)
    scale, zero = (torch.rand((B, *groups), generator=gen, device="cuda").mul(f).sub(1.0 - f).bfloat16().abs() * s for f, s in ((0.5, 1), (0.3, -1)))
    cache = xq.XQCache(codes, scale.contiguous(), zero.contiguous(), B, codes.shape[1], d, G, bits)
    wp = xq.xq_prepare_weights(attn, d, 128 if per_channel else G, bits, wk, wv)
    if not per_channel:
        return lambda: xq.xq_remat_attn_decode(attn, q, wp, lens, xcache=cache)
    wd = xq.xq_prepare_weights(attn, d, 0, 16, wk, wv)
    tail = torch.randn((B, G, d), generator=gen, device="cuda", dtype=torch.bfloat16)
    t = xq.alloc_per_channel_terms(cache, Hkv) if terms else None
    if terms:
        xq.xq_remat_attn_decode_per_channel(attn, q, cache, tail, lens, wp, wd, terms=t, terms_valid=False)
    return lambda: xq.xq_remat_attn_decode_per_channel(attn, q, cache, tail, lens, wp, wd, terms=t, terms_valid=terms)


@pytest.mark.parametrize("folded,step", [
    (False, dict(B=16, L=8192, d=1024, Hq=1, Hkv=1, bits=16)), (False, dict(B=16, L=2048, d=2048, Hq=32, Hkv=2, bits=16)),
    (False, dict(B=16, L=100, d=2048, Hq=128, Hkv=8, bits=3)), (False, dict(B=16, L=8192, d=128, Hq=2, Hkv=2, bits=3, per_channel=True, terms=True)),
    (False, dict(B=1, L=512, d=256, Hq=2, Hkv=2, bits=4)),
    (True, dict(B=4, L=2048, d=1024, Hq=32, Hkv=32, bits=16)), (True, dict(B=2, L=1000, d=4096, Hq=32, Hkv=8, bits=2, G=64)),
    (True, dict(B=2, L=1000, d=2304, Hq=16, Hkv=16, bits=8)), (True, dict(B=4, L=1000, d=4096, Hq=32, Hkv=32, bits=3, per_channel=True, terms=True)),
    (True, dict(B=16, L=7000, d=512, Hq=2, Hkv=2, bits=3, per_channel=True))])
def test_which_order_a_step_takes(xq, folded, step):
    """The order that was measured to be the faster one, on either side of the rule."""
    call = _step(xq, **step)
    call()
    assert _folds(call) == folded


def _run(xq, w, bits, G, lens, x_bits=None, workspaces=(None,), pairs=None, wk=None, scale_sign=None):
    x = xi.gen_x(w) if x_bits is None else x_bits
    wk0, wv = xi.gen_weights(w)
    wk = wk0 if wk is None else wk
    q = xi.gen_q(w)
    attn = xq.XQAttn(w.Hq, w.Hkv, w.hd, w.hd ** -0.5)
    pairs = pairs or [(b, h) for b in range(w.B) for h in sorted({0, 1, w.Hq // 2, w.Hq - 1})]
    kw = dict(q_bf16=q, Wk=wk, Wv=wv, Hq=w.Hq, Hkv=w.Hkv, hd=w.hd, softmax_scale=w.hd ** -0.5, lens=lens, pairs=pairs)
    if bits == 16:
        src = dict(acc_bf16=bits_to_torch(x))
        ref = xo.remat_attn_pairs(acc_bf16=x, **kw)
    else:
        cache = xq.alloc_cache(w.B, w.L + 3, w.d, G, bits)
        cache.codes.fill_(0xFF)                              # rows past the data must not be read
        cache.scale.view(torch.int16).fill_(0x7FC0)
        cache.zero.view(torch.int16).fill_(0x7FC0)
        xq.xq_quantize_append(cache, bits_to_torch(x), [0] * w.B)
        src = dict(xcache=cache)
        packed, scale, zero = oracle_cache(x, G, bits, seqs=[b for b, _ in pairs])
        if scale_sign is not None:                           # rows whose stored scales change their sign
            scale[:, scale_sign] ^= 0x8000
            cache.scale[:, scale_sign] = -cache.scale[:, scale_sign]
        ref = xo.remat_attn_pairs(packed=packed, scale=scale, zero=zero, G=G, bits=bits, **kw)
    wprep = xq.xq_prepare_weights(attn, w.d, G, bits, bits_to_torch(wk), bits_to_torch(wv))
    for n in workspaces:
        ws = None if n is None else torch.full((n,), 0xFF, dtype=torch.uint8, device="cuda")
        call = lambda: xq.xq_remat_attn_decode(attn, bits_to_torch(q), wprep, lens, workspace=ws, **src)
        out = call().cpu().numpy()
        if n is None:
            assert _folds(call)
        assert np.all(np.isfinite(out))
        rows, worst = rel_errors(np.array([out[b, h] for b, h in pairs]), ref)
        assert rows.max() <= TOL and worst <= TOL, (n, float(rows.max()), float(worst))


@pytest.mark.parametrize("bits,G", [(2, 64), (2, 128), (3, 64), (3, 128), (4, 64), (4, 128), (8, 64), (8, 128), (16, 128)])
@pytest.mark.parametrize("Hq,Hkv,d,lens", [(16, 16, 4096, [300, 1, 129]), (32, 8, 4224, [257, 33]), (40, 40, 4096, [511])])
def test_formats_rows_and_tile_edges(xq, bits, G, Hq, Hkv, d, lens):
    w = xi.C2.scaled(B=len(lens), L=max(lens), d=d, Hq=Hq, Hkv=Hkv, n_outlier=d // 100)
    _run(xq, w, bits, G, lens)


@pytest.mark.parametrize("bits,G,d", [(2, 64, 256), (3, 128, 256), (16, 128, 256), (3, 128, 640), (16, 128, 640)])
def test_token_ways_of_a_score_workgroup(xq, bits, G, d):
    """Enough tiles for score workgroups of four waves, two of them without a slab on the narrow layer (one of them, or a wave with
    fewer than the others, on the wider one), and tiles past the length."""
    w = xi.C2.scaled(B=16, L=4000, d=d, Hq=64, Hkv=8, n_outlier=2)
    lens = [4000, 3969, 129, 128, 1, 2049] + [100] * 10
    _run(xq, w, bits, G, lens, pairs=[(0, 0), (0, 63), (1, 17), (2, 5), (3, 40), (4, 33), (5, 62), (15, 8)])


@pytest.mark.parametrize("Hq,Hkv,d,lens,split", [(32, 32, 640, [4096, 3969, 129, 1], True), (32, 32, 640, [4100, 257, 128, 1], False),
                                                 (40, 40, 4096, [511, 33], True), (32, 8, 4224, [700, 33, 1], True), (16, 16, 4096, [300, 1, 129], False)])
def test_row_tiles_of_a_score_workgroup(xq, Hq, Hkv, d, lens, split):
    """Over bf16 rows a workgroup has one row tile of a row block up to 128 tiles, both of them beyond (16 rows have only one): rows of
    padding in the last row block, waves without a slab, tiles past the length."""
    w = xi.C2.scaled(B=len(lens), L=max(lens), d=d, Hq=Hq, Hkv=Hkv, n_outlier=d // 100)
    x = bits_to_torch(xi.gen_x(w))
    wk, wv = xi.gen_weights(w)
    attn = xq.XQAttn(Hq, Hkv, 128, 128 ** -0.5)
    wprep = xq.xq_prepare_weights(attn, d, 128, 16, bits_to_torch(wk), bits_to_torch(wv))
    names = _kernels(lambda: xq.xq_remat_attn_decode(attn, bits_to_torch(xi.gen_q(w)), wprep, lens, acc_bf16=x))
    assert any("fold_scores_dense_kernel<1, 2>" in n for n in names) == split, names
    _run(xq, w, 16, 128, lens, pairs=[(b, h) for b in range(w.B) for h in (0, 15, Hq - 16, Hq - 1)])


@pytest.mark.parametrize("step", [dict(L=2048), dict(L=2048, Hq=48), dict(L=1792, taken=False), dict(L=2304, taken=False), dict(L=2048, bits=3, taken=False),
                                  dict(L=4096, Hq=16, taken=False)])
def test_which_steps_take_queries_in_digits(xq, step):
    step = dict(dict(B=32, d=640, Hq=64, bits=2, taken=True), **step)
    taken = step.pop("taken")
    call = _step(xq, Hkv=step["Hq"], **step)
    call()
    assert any("digits" in n for n in _kernels(call)) == taken


# (groups of 10 bytes a row; a last row block of 16 rows; 52 groups, which come in two runs; whole runs)
@pytest.mark.parametrize("d,G,Hq,Hkv,B", [(640, 128, 64, 64, 32), (384, 64, 48, 48, 32), (3328, 64, 128, 32, 16), (1024, 64, 64, 64, 32)])
@pytest.mark.parametrize("small_rows", [False, True])
def test_queries_in_digits(xq, d, G, Hq, Hkv, B, small_rows):
    """Enough tiles for queries in base-32 digits, with lengths at the edges of tiles and products.  Weight rows 2^-10 of the others
    against channels 2^10 as large take further digits."""
    w = xi.C2.scaled(B=B, L=2048, d=d, Hq=Hq, Hkv=Hkv, n_outlier=d // 100)
    lens = [2048, 2047, 1025, 257, 256, 129, 65, 33, 1] + [40] * (B - 9)
    x, wk = xi.gen_x(w), xi.gen_weights(w)[0]
    if small_rows:
        rows = [3, 70, 71, 200]
        x, wk = xi.from_bf16_bits(x).copy(), xi.from_bf16_bits(wk).copy()
        x[:, :, rows] *= 2.0 ** 10
        wk[rows] *= 2.0 ** -10
        x, wk = xi.to_bf16_bits(x), xi.to_bf16_bits(wk)
    _run(xq, w, 2, G, lens, x_bits=x, wk=wk, pairs=[(b, (11 * b + 5) % Hq) for b in range(10)] + [(0, Hq - 1), (1, 0)])


@pytest.mark.parametrize("bits,G", [(2, 64), (2, 128), (3, 64), (3, 128), (4, 64), (4, 128), (8, 128)])
def test_steps_of_a_value_workgroup(xq, bits, G):
    """Ranges of one to four steps of 128 tokens, with a last step that is full, holds one token, or is missing."""
    w = xi.C2.scaled(B=32, L=1100, d=1024, Hq=32, Hkv=8, n_outlier=10)
    lens = [1100, 1025, 897, 896, 513, 512, 385, 130] + [64] * 24
    _run(xq, w, bits, G, lens, pairs=[(b, (5 * b + 3) % 32) for b in range(9)])


@pytest.mark.parametrize("bits,G", [(2, 64), (3, 128), (8, 128), (16, 128)])
@pytest.mark.parametrize("Hq,Hkv,lens", [(16, 16, [4608, 2300, 300, 1]), (16, 4, [4600] + [260 * b + 7 for b in range(10)])])
def test_sums_over_many_token_splits(xq, bits, G, Hq, Hkv, lens):
    """Columns of up to 18 token splits beside such of one, in output workgroups with a piece per thread and with several."""
    w = xi.C2.scaled(B=len(lens), L=max(lens), d=640, Hq=Hq, Hkv=Hkv, n_outlier=6)
    _run(xq, w, bits, G, lens, pairs=[(b, (3 * b + 1) % Hq) for b in range(len(lens))])


@pytest.mark.parametrize("B", [15, 16, 17, 29])
def test_sequences_dealt_over_the_chip(xq, B):
    """From 16 sequences on they are taken in another order than they come in; lengths of every kind, several the same."""
    w = xi.C2.scaled(B=B, L=700, d=1024, Hq=16, Hkv=16, n_outlier=10)
    lens = [1 + (b * b * 97 + 41 * b) % 700 if b % 3 else 700 - b for b in range(B)]
    _run(xq, w, 3, 128, lens, pairs=[(b, (3 * b + 1) % 16) for b in range(B)])


@pytest.mark.parametrize("B", [16, 29])
@pytest.mark.parametrize("source,G", [("acc", 128), ("per_channel", 64), ("per_channel", 128)])
def test_sequences_of_other_sources_dealt_over_the_chip(xq, source, G, B):
    """The same over bf16 rows, and over blocks with a window, some of them windows alone."""
    w = xi.C2.scaled(B=B, L=700, d=1024, Hq=16, Hkv=16, n_outlier=10)
    lens = [1 + (b * b * 97 + 41 * b) % 700 if b % 3 else 700 - b for b in range(B)]
    pairs = [(b, (3 * b + 1) % 16) for b in range(B)]
    if source == "acc":
        return _run(xq, w, 16, G, lens, pairs=pairs)
    err = []
    assert _folds(lambda: err.append(_attend(xq, w, 3, G, lens, pairs=pairs)))
    assert err[0] <= TOL


@pytest.mark.parametrize("bits", [3, 16])
def test_smaller_workspaces(xq, bits):
    """Between the smallest workspace that is accepted and the one that is asked for, the launch goes in groups of sequences,
    or through the kernels that rematerialise keys and values."""
    B, L, d, Hq = 3, 130, 4096, 32
    w = xi.C2.scaled(B=B, L=L, d=d, Hq=Hq, Hkv=8, n_outlier=20)
    asked = xq.xq_remat_attn_workspace_bytes(xq.XQAttn(Hq, 8, 128, 1.0), B, L, d, 128 if bits < 16 else 0)
    least = B * Hq * 2 * 4 * 130 * 4 + (B * 2 * (d // 128 + 1) * 128 * 2 if bits < 16 else 0)
    assert least < asked
    _run(xq, w, bits, 128, [130, 128, 7], workspaces=(asked, asked // 2 + 16, asked // 3 + 16, least))


def test_scales_of_every_magnitude(xq):
    """Constant groups (scale 0) and groups 1000 times larger than their neighbours, large offsets."""
    w = xi.C2.scaled(B=1, L=300, d=2304, Hq=16, Hkv=16, n_outlier=0)
    x = xi.from_bf16_bits(xi.gen_x(w)).copy()
    x[0, :, 128:256] = 0.5
    x[0, ::2, 256:384] *= 30.0
    x[0, 1::3, 512:640] += 100.0
    x[0, :, 640:768] *= 1e-3
    _run(xq, w, 3, 128, [300], x_bits=xi.to_bf16_bits(x))


CODED = [(2, 64), (2, 128), (3, 64), (3, 128), (4, 64), (4, 128), (8, 64), (8, 128)]


@pytest.mark.parametrize("bits,G", CODED)
@pytest.mark.parametrize("Hq,Hkv", [(16, 16), (32, 8)])
def test_a_few_rows_far_larger_than_the_others(xq, bits, G, Hq, Hkv):
    """Rows 2^28 times larger than their neighbours: heads that attend to them see little else, the others must not lose the
    ordinary rows' digits to them.  They lie in different token ranges of the value kernel, one range has none."""
    w = xi.C2.scaled(B=2, L=900, d=2304, Hq=Hq, Hkv=Hkv, n_outlier=23)
    x = xi.from_bf16_bits(xi.gen_x(w)).copy()
    x[0, [5, 300]] *= 2.0 ** 28
    x[1, 77] *= 2.0 ** 36
    x[1, 79] *= 2.0 ** -40
    _run(xq, w, bits, G, [900, 130], x_bits=xi.to_bf16_bits(x), pairs=[(b, h) for b in range(2) for h in range(Hq)])


def _small_weight_rows(w, k, nats, rows):
    """X and Wk for which `rows` (of sequence 0) score 0 and all others about `nats`, the former holding nothing but channels
    128-255 (which no key sees) 2^k times larger: they count as much as the others where 2^k exp(-nats) is about 1."""
    x = xi.from_bf16_bits(xi.gen_x(w)).copy() * 0.1
    wk = xi.from_bf16_bits(xi.gen_weights(w)[0]).copy()
    q = xi.from_bf16_bits(xi.gen_q(w))[0]
    wk[128:256] = 0.0
    for h in range(w.Hkv):
        v = q[h * (w.Hq // w.Hkv)]
        wk[0, h * w.hd:(h + 1) * w.hd] = v / (v @ v) * w.hd ** 0.5 * nats
    x[0, :, 0] = 1.0
    big = x[0, rows, 128:256] * 10.0 * 2.0 ** k
    x[0, rows] = 0.0
    x[0, rows, 128:256] = big
    return xi.to_bf16_bits(x), xi.to_bf16_bits(wk)


@pytest.mark.parametrize("bits,G", CODED)
@pytest.mark.parametrize("rows", [[77, 690], list(range(256, 512))])
def test_large_rows_of_small_weight(xq, bits, G, rows):
    """The softmax weight of a row may be 2^-40 and the row still count: single rows, and a whole token range of them."""
    w = xi.C2.scaled(B=1, L=700, d=2304, Hq=16, Hkv=16, n_outlier=0)
    x, wk = _small_weight_rows(w, 40, 28.0, rows)
    _run(xq, w, bits, G, [700], x_bits=x, wk=wk, pairs=[(0, h) for h in range(w.Hq)])


@pytest.mark.parametrize("bits,G", CODED)
@pytest.mark.parametrize("rows", [[5, 300], list(range(256, 520)), [899]])
@pytest.mark.parametrize("nats", [3.0, -28.0])
def test_rows_of_zeros(xq, bits, G, rows, nats):
    """Rows of zeros (every scale 0) among rows that score `nats`: with the weights of the others, or with nearly all of it, when
    the output is what the others' small weights leave."""
    w = xi.C2.scaled(B=1, L=900, d=2304, Hq=16, Hkv=16, n_outlier=0)
    x, wk = _small_weight_rows(w, 0, nats, rows)
    x[0, rows] = 0
    _run(xq, w, bits, G, [900], x_bits=x, wk=wk, pairs=[(0, h) for h in (0, 7, 15)])


@pytest.mark.parametrize("bits,G", CODED)
@pytest.mark.parametrize("Hq,Hkv", [(16, 16), (32, 8)])
def test_weights_of_tiles_whose_maxima_nearly_agree(xq, bits, G, Hq, Hkv):
    """Two tokens in different tiles, one 1.5 to 2 times 2^-22 (log2) above the other, hold all the weight and opposite values: the
    output is half the difference of their weights, 4 to 6 times 2^-24.  The weights and their two sums are rounded to 2^-24
    or 2^-25 (and exp2 by one such step): within 0.6 of it.  With the tiles' factor formed from steps of 2^-20 it is 0."""
    d, L = 4096, 256
    x = torch.zeros((1, L, d // G, G))
    x[0, :, :, 3], x[0, :, :, 4] = -1.0, 2.0 ** bits - 2.0                # every group: scale 1, zero-point -1
    x[0, :, 0, 0] = -1.0                                                  # key channels 0 and 2, value channel 1
    x[0, [3, 140], 0, 0] = 0.0
    x[0, 140, 0, 2] = 1.0
    x[0, 140, 0, 1], x[0, 3, 0, 1] = 1.0, -1.0
    wk, wv = torch.zeros((d, Hkv, 128)), torch.zeros((d, Hkv, 128))
    wk[0, :, 0] = wk[2, :, 1] = 1.0
    wv[1] = 1.0
    step = (1.5 + torch.arange(Hq) % 16 / 32) * 2.0 ** -22
    q = torch.zeros((1, Hq, 128))
    q[0, :, 0], q[0, :, 1] = 64.0, step
    gpu = lambda t: t.to("cuda", torch.bfloat16).contiguous()
    attn = xq.XQAttn(Hq, Hkv, 128, float(np.log(2.0)))
    cache = xq.alloc_cache(1, L, d, G, bits)
    xq.xq_quantize_append(cache, gpu(x.reshape(1, L, d)), [0])
    wprep = xq.xq_prepare_weights(attn, d, G, bits, gpu(wk.reshape(d, -1)), gpu(wv.reshape(d, -1)))
    call = lambda: xq.xq_remat_attn_decode(attn, gpu(q), wprep, [L], xcache=cache)
    out = call().cpu().double()[0]
    assert _folds(call)
    ref = torch.tanh(step.double() * np.log(2.0) / 2)[:, None]
    assert float((out / ref - 1).abs().max()) <= 0.6, (out[:, 0] / ref[:, 0]).tolist()


@pytest.mark.parametrize("bits,G", CODED)
def test_scales_of_either_sign(xq, bits, G):
    """x^ = code scale + zero holds for a negative scale too."""
    w = xi.C2.scaled(B=1, L=600, d=2304, Hq=16, Hkv=16, n_outlier=0)
    _run(xq, w, bits, G, [600], scale_sign=[3, 299], pairs=[(0, h) for h in range(w.Hq)])


@pytest.mark.parametrize("bits,G", [(2, 64), (3, 128), (4, 64)])
@pytest.mark.parametrize("small", [False, True])
def test_latent_halves(xq, bits, G, small):
    """Scores from the first r channels of a row, weighted sums from the last r, weights in streams of head pairs; also with
    the smallest workspace that is accepted."""
    r, B, L, lens = 640, 3, 290, [290, 1, 129]
    w = xi.C4.scaled(B=B, L=L, d=2 * r, Hq=12, Hkv=4, n_outlier=12)
    x, q = xi.gen_x(w), xi.gen_q(w)
    wk, wv = xi.gen_weights(w)
    wfk, wfv = np.ascontiguousarray(wk[:r]), np.ascontiguousarray(wv[r:])
    attn = xq.XQAttn(w.Hq, w.Hkv, w.hd, w.hd ** -0.5)
    cache = xq.alloc_cache(B, L, 2 * r, G, bits)
    xq.xq_quantize_append(cache, bits_to_torch(x), [0] * B)
    wprep = xq.xq_prepare_weights_latent(attn, r, G, bits, bits_to_torch(wfk), bits_to_torch(wfv))
    tiles = 2                                               # of 256 tokens; 8 partials, a score and two scales per token each
    least = 4 * B * w.Hq * tiles * (8 * 130 + 256) + 4 * B * tiles * (r // G + 1) * 256
    assert least <= xq.xq_remat_attn_latent_workspace_bytes(attn, B, L, r, G)
    ws = torch.full((least,), 0xFF, dtype=torch.uint8, device="cuda") if small else None
    out = xq.xq_remat_attn_decode_latent(attn, bits_to_torch(q), wprep, lens, cache, workspace=ws).cpu().numpy()
    packed, scale, zero = oracle_cache(x, G, bits)
    wk0, wv0 = wk.copy(), wv.copy()
    wk0[r:], wv0[:r] = 0, 0
    ref = xo.remat_attn_pairs(q_bf16=q, Wk=wk0, Wv=wv0, Hq=w.Hq, Hkv=w.Hkv, hd=w.hd, softmax_scale=w.hd ** -0.5, lens=lens,
                              pairs=[(b, h) for b in range(B) for h in range(w.Hq)], packed=packed, scale=scale, zero=zero, G=G, bits=bits)
    rows, worst = rel_errors(out.reshape(-1, w.hd), ref)
    assert np.all(np.isfinite(out)) and rows.max() <= TOL and worst <= TOL, (float(rows.max()), float(worst))


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("G", [64, 128])
@pytest.mark.parametrize("Hq,Hkv,d,lens", [(16, 16, 4096, [330, 1, 256, 320]), (32, 8, 4224, [257, 63]), (40, 40, 4096, [512]), (16, 16, 4096, [50])])
def test_per_channel_blocks_and_window(xq, bits, G, Hq, Hkv, d, lens):
    """Blocks that end inside a 128- or 256-token tile, no window, a window alone, nothing but windows."""
    err = []
    w = xi.C2.scaled(B=len(lens), L=max(lens), d=d, Hq=Hq, Hkv=Hkv, n_outlier=d // 100)
    assert _folds(lambda: err.append(_attend(xq, w, bits, G, lens, pairs=[(b, h) for b in range(len(lens)) for h in (0, Hq - 1)])))
    assert err[0] <= TOL


def test_per_channel_scales_of_every_magnitude(xq):
    w = xi.C2.scaled(B=1, L=300, d=2304, Hq=16, Hkv=16, n_outlier=0)
    err = []
    assert _folds(lambda: err.append(_attend(xq, w, 3, 128, [300], pairs=[(0, 0), (0, 9)], scale_spread=64.0)))
    assert err[0] <= TOL


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("G", [64, 128])
@pytest.mark.parametrize("Hq,Hkv", [(16, 16), (32, 8)])
def test_per_channel_large_block_of_small_weight(xq, bits, G, Hq, Hkv):
    """A block whose rows are 2^40 larger and whose softmax weights are 2^-40 counts as much as the others: with its neighbour
    in one tile (blocks of 64), in a tile of its own, and as the last block before the window."""
    L = 600
    pairs = [(0, h) for h in (0, 1, Hq - 1)]
    for block in sorted({1, L // G // 2, L // G - 1}):
        w = xi.C2.scaled(B=1, L=L, d=2304, Hq=Hq, Hkv=Hkv, n_outlier=0)
        x, wk = _small_weight_rows(w, 40, 28.0, list(range(block * G, (block + 1) * G)))
        wv, q = xi.gen_weights(w)[1], xi.gen_q(w)
        nblk, rem = divmod(L, G)
        cache = xq.alloc_cache_per_channel(1, nblk * G, w.d, G, bits)
        xt = bits_to_torch(x)
        xq.xq_quantize_blocks_per_channel(cache, xt[:, :nblk * G].contiguous(), [0])
        tail = torch.full((1, G, w.d), float("nan"), dtype=torch.bfloat16, device="cuda")
        tail[:, :rem] = xt[:, nblk * G:]
        attn = xq.XQAttn(Hq, Hkv, w.hd, w.hd ** -0.5)
        wc, wd = (xq.xq_prepare_weights(attn, w.d, g, b, bits_to_torch(wk), bits_to_torch(wv)) for g, b in ((128, bits), (0, 16)))
        out = xq.xq_remat_attn_decode_per_channel(attn, bits_to_torch(q), cache, tail, [L], wc, wd).cpu().numpy()
        packed, scale, zero, tail_o = oracle_cache_per_channel(x, G, bits, [L])
        ref = xo.remat_attn_pairs_per_channel(q_bf16=q, Wk=wk, Wv=wv, Hq=Hq, Hkv=Hkv, hd=w.hd, softmax_scale=w.hd ** -0.5, lens=[L],
                                              pairs=pairs, packed=packed, scale=scale, zero=zero, G=G, bits=bits, tail_bf16=tail_o)
        rows, worst = rel_errors(np.array([out[b, h] for b, h in pairs]), ref)
        assert np.all(np.isfinite(out)) and rows.max() <= TOL and worst <= TOL, (block, float(rows.max()), float(worst))


def test_per_channel_terms_serve_both_orders(xq):
    """Block terms kept by the caller, computed by a step of the folded order, used by one that rematerialises."""
    B, G, d, Hkv = 64, 128, 1792, 2
    x = torch.randn((B, 512, d), device="cuda", generator=torch.Generator("cuda").manual_seed(1)).bfloat16()
    cache = xq.alloc_cache_per_channel(B, 512, d, G, 4)
    xq.xq_quantize_blocks_per_channel(cache, x, [0] * B)
    tail = x[:, :G].contiguous()
    attn = xq.XQAttn(Hkv, Hkv, 128, 128 ** -0.5)
    wk, wv = (torch.randn((d, Hkv * 128), device="cuda").mul(d ** -0.5).bfloat16() for _ in range(2))
    wc, wd = xq.xq_prepare_weights(attn, d, G, 4, wk, wv), xq.xq_prepare_weights(attn, d, 0, 16, wk, wv)
    q = torch.randn((B, Hkv, 128), device="cuda").bfloat16()
    terms = xq.alloc_per_channel_terms(cache, Hkv)
    xq.xq_remat_attn_decode_per_channel(attn, q, cache, tail, [513] * B, wc, wd, terms=terms, terms_valid=False)
    assert _folds(lambda: xq.xq_remat_attn_decode_per_channel(attn, q, cache, tail, [513] * B, wc, wd, terms=terms, terms_valid=True))
    assert not _folds(lambda: xq.xq_remat_attn_decode_per_channel(attn, q, cache, tail, [512] * B, wc, wd, terms=terms, terms_valid=True))
    kept = xq.xq_remat_attn_decode_per_channel(attn, q, cache, tail, [512] * B, wc, wd, terms=terms, terms_valid=True)
    fresh = xq.xq_remat_attn_decode_per_channel(attn, q, cache, tail, [512] * B, wc, wd)
    assert torch.equal(kept, fresh)


def _cases(xq, kind, B=3, L=700, Hq=32, Hkv=8):
    """A large step of every source, as call(q, lens, order, workspace): sequences in the given order (None: as they are)."""
    take = lambda t, order: t if order is None else t[order].contiguous()
    gen = torch.Generator("cuda").manual_seed(11)
    attn = xq.XQAttn(Hq, Hkv, 128, 128 ** -0.5)
    d = 1280 if kind == "latent" else 4096
    rows = torch.randn((B, L, 2 * d if kind == "latent" else d), generator=gen, device="cuda").bfloat16()
    wk, wv = (torch.randn((d, Hkv * 128), generator=gen, device="cuda").mul(d ** -0.5).bfloat16() for _ in range(2))
    q = torch.randn((B, Hq, 128), generator=gen, device="cuda").bfloat16()
    if kind == "acc":
        wp = xq.xq_prepare_weights(attn, d, 0, 16, wk, wv)
        return q, lambda q, lens, order, ws=None: xq.xq_remat_attn_decode(attn, take(q, order), wp, lens if order is None else [lens[i] for i in order],
                                                                          acc_bf16=take(rows, order), workspace=ws), rows
    if kind == "per_channel":
        G, nblk = 64, L // 64
        cache = xq.alloc_cache_per_channel(B, nblk * G, d, G, 3)
        xq.xq_quantize_blocks_per_channel(cache, rows[:, :nblk * G].contiguous(), [0] * B)
        wc, wd = xq.xq_prepare_weights(attn, d, 128, 3, wk, wv), xq.xq_prepare_weights(attn, d, 0, 16, wk, wv)
        tail = rows[:, :G].contiguous()
    elif kind == "latent":
        cache = xq.alloc_cache(B, L, 2 * d, 64, 2)
        xq.xq_quantize_append(cache, rows, [0] * B)
        wp = xq.xq_prepare_weights_latent(attn, d, 64, 2, wk, wv)
    else:
        cache = xq.alloc_cache(B, L, d, 128, 3)
        xq.xq_quantize_append(cache, rows, [0] * B)
        wp = xq.xq_prepare_weights(attn, d, 128, 3, wk, wv)

    def call(q, lens, order, ws=None):
        c = xq.XQCache(*(take(t, order) for t in (cache.codes, cache.scale, cache.zero)), B, cache.cap, cache.d, cache.group, cache.bits)
        qq, ll = take(q, order), lens if order is None else [lens[i] for i in order]
        if kind == "per_channel":
            return xq.xq_remat_attn_decode_per_channel(attn, qq, c, take(tail, order), ll, wc, wd, workspace=ws)
        if kind == "latent":
            return xq.xq_remat_attn_decode_latent(attn, qq, wp, ll, c, workspace=ws)
        return xq.xq_remat_attn_decode(attn, qq, wp, ll, xcache=c, workspace=ws)
    return q, call, cache


KINDS = ["coded", "acc", "latent", "per_channel"]


@pytest.mark.parametrize("kind", KINDS)
def test_same_bits_again_in_any_order_on_any_workspace(xq, kind):
    """A batch's results do not depend on what the workspace held, nor on the order of its sequences."""
    q, call, _ = _cases(xq, kind)
    lens = [700, 130, 515]
    assert _folds(lambda: call(q, lens, [0, 1, 2]))
    want = call(q, lens, [0, 1, 2])
    n = 64 << 20
    for fill in (0x00, 0xFF, 0x7F):
        got = call(q, lens, [0, 1, 2], torch.full((n,), fill, dtype=torch.uint8, device="cuda"))
        assert torch.equal(got, want), fill
    assert torch.equal(call(q, lens, [2, 0, 1]), want[[2, 0, 1]])


@pytest.mark.parametrize("kind", KINDS)
def test_same_bits_in_any_order_of_many_sequences(xq, kind):
    """The same where the launch takes its sequences in an order of its own."""
    q, call, _ = _cases(xq, kind, B=17, L=400)
    lens = [1 + (b * b * 97 + 41 * b) % 399 for b in range(16)] + [400]
    as_they_are = list(range(17))
    assert _folds(lambda: call(q, lens, as_they_are))
    want = call(q, lens, as_they_are)
    for order in (as_they_are[::-1], [(5 * b + 3) % 17 for b in range(17)]):
        assert torch.equal(call(q, lens, order), want[order]), order


@pytest.mark.parametrize("kind", KINDS)
def test_numbers_that_are_not_finite_stay_in_their_sequence(xq, kind):
    """NaN or infinity in a cached row makes that sequence's outputs NaN, in a query only its own head's; all others keep their
    bits."""
    q, call, src = _cases(xq, kind)
    lens, order = [700, 130, 515], None
    want = call(q, lens, order)
    rows, at = (src, 40) if kind == "acc" else (src.scale, 40 if kind == "per_channel" else 3)
    for v in (float("nan"), float("inf")):
        keep = rows[1, 0, at].clone()
        rows[1, 0, at] = v
        got = call(q, lens, order)
        rows[1, 0, at] = keep
        assert bool(got[1].isnan().all()) and torch.equal(got[[0, 2]], want[[0, 2]]), v
    bad = q.clone()
    bad[2, 5, 17] = float("nan")
    got = call(bad, lens, order)
    assert bool(got[2, 5].isnan().all())
    got[2, 5] = want[2, 5]
    assert torch.equal(got, want)


@pytest.mark.parametrize("kind", KINDS)
def test_large_step_replays_from_a_graph(xq, kind):
    """The five kernels in a graph, replayed with eager work between the replays, against the eager result."""
    q, call, _ = _cases(xq, kind)
    lens, order = [700, 130, 515], None
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    static_q = q.clone()
    call(static_q, lens, order, ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = call(static_q, lens, order, ws)
    gen = torch.Generator("cuda").manual_seed(4)
    for _ in range(4):
        static_q.copy_(torch.randn(q.shape, generator=gen, device="cuda").bfloat16())
        graph.replay()
        torch.cuda.synchronize()
        got = out.clone()
        assert torch.equal(got, call(static_q, lens, order))
