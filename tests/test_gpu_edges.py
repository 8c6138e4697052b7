"""Sizes at which a tile, a remainder or a dispatch rule of the kernels can go wrong, against the oracle."""
import numpy as np
import pytest

from oracle import stack as ost
from oracle import tlq_oracle as orc
from paper_2602_07899_amd import tlq

pytestmark = pytest.mark.gpu

BF = lambda a: orc.round_to_bf16(np.asarray(a, np.float64).astype(np.float32))
F16 = lambda a: np.asarray(a, np.float64).astype(np.float16)


def dev(a, gpu, bf16):
    import torch
    t = torch.from_numpy(np.ascontiguousarray(np.asarray(a, np.float32)))
    return t.to(torch.bfloat16 if bf16 else torch.float16).to(gpu)


def host(t):
    return t.detach().float().cpu().numpy().astype(np.float64)


def host64(t):
    return t.detach().double().cpu().numpy()


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("seq,heads,samples", [(31, 9, 1), (33, 1, 9), (63, 3, 3), (64, 2, 1), (65, 1, 1), (96, 1, 2),
                                               (128, 1, 1), (160, 2, 1), (257, 1, 1), (1100, 1, 1), (400, 7, 1),
                                               (300, 2, 3), (140, 4, 2), (513, 1, 9)])
def test_attention_step_and_block_edges(gpu, bf16, seq, heads, samples):
    """32-key steps, 128-query blocks, eight (sample, head) pairs per grid group, or fewer
    whose query blocks are dealt over the chip."""
    import torch
    g = np.random.default_rng([21, seq, heads])
    n, width = seq * samples, heads * 128
    rnd = BF if bf16 else F16
    q, k, v = (np.asarray(rnd(g.standard_normal((n, width)) * 1.5), np.float64) for _ in range(3))
    want = ost.causal_attention(q, k, v, heads, seq)
    mag = ost.causal_attention(q, k, np.abs(v), heads, seq)
    p = tlq.params(x_dtype=tlq.BF16 if bf16 else tlq.F16)
    out = torch.empty((n, width), dtype=torch.bfloat16 if bf16 else torch.float16, device=gpu)
    tlq.causal_attention(dev(q, gpu, bf16), dev(k, gpu, bf16), dev(v, gpu, bf16), heads, seq, p, out)
    eps = 2.0 ** -8 if bf16 else 2.0 ** -11       # one rounding of every probability, one of the output
    assert np.all(np.abs(host(out) - want) <= eps * (mag + np.abs(want)) + 2e-6)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("seq,heads,samples", [(1, 1, 1), (15, 2, 1), (17, 1, 5), (48, 1, 2), (79, 3, 1), (80, 1, 1), (95, 1, 1),
                                               (97, 2, 1), (127, 1, 2), (129, 1, 1), (191, 1, 1), (193, 2, 1), (321, 1, 1),
                                               (257, 43, 2), (271, 86, 1), (273, 29, 3), (304, 86, 1), (321, 43, 2), (335, 29, 3),
                                               (383, 86, 1), (385, 65, 1)])
def test_attention_tile_remainders(gpu, bf16, seq, heads, samples):
    """Sequences that end inside 16, 32, 64 and 128 keys and just behind them, in launches of few blocks and of more than one a
    unit; scores that grow with the key make every step meet new maxima in some queries."""
    import torch
    g = np.random.default_rng([24, seq, heads])
    n, width = seq * samples, heads * 128
    rnd = BF if bf16 else F16
    grow = 1.0 + 2.0 * (np.arange(n) % seq)[:, None] / seq
    q, k, v = (np.asarray(rnd(g.standard_normal((n, width)) * f), np.float64) for f in (1.5, grow, 1.0))
    want, mag = ost.causal_attention(q, k, v, heads, seq), ost.causal_attention(q, k, np.abs(v), heads, seq)
    p = tlq.params(x_dtype=tlq.BF16 if bf16 else tlq.F16)
    out = torch.empty((n, width), dtype=torch.bfloat16 if bf16 else torch.float16, device=gpu)
    tlq.causal_attention(dev(q, gpu, bf16), dev(k, gpu, bf16), dev(v, gpu, bf16), heads, seq, p, out)
    eps = 2.0 ** -8 if bf16 else 2.0 ** -11       # one rounding of every probability, one of the output
    assert np.all(np.abs(host(out) - want) <= eps * (mag + np.abs(want)) + 2e-6)


@pytest.mark.parametrize("seq,heads", [(200, 2), (300, 86)])
@pytest.mark.parametrize("bf16,size", [(False, 8192.0), (False, 65504.0), (True, 2.0 ** 15), (True, 2.0 ** 18), (True, 2.0 ** 40)])
def test_attention_scores_of_any_size(gpu, bf16, size, seq, heads):
    """Scores up to 2^80: a query gives all its weight to its largest key, or shares it evenly among equal ones.  One channel of
    q and k is not zero, so the products are exact in 32 bits, and different ones are at least 1/128 apart, thousands in the exponent."""
    import torch
    g = np.random.default_rng([32, seq, int(np.log2(size))])
    width = heads * 128
    rnd = BF if bf16 else F16
    q, k = np.zeros((seq, width)), np.zeros((seq, width))
    at = np.arange(heads) * 128 + g.integers(0, 128, heads)
    q[:, at] = rnd(g.choice([-1.0, 1.0], (seq, heads)) * size * g.uniform(0.5, 1.0, (seq, heads)))
    k[:, at] = rnd(size * g.integers(-64, 65, (seq, heads)) / 64.0)
    v = np.asarray(rnd(g.standard_normal((seq, width))), np.float64)
    want, mag = ost.causal_attention(q, k, v, heads, seq), ost.causal_attention(q, k, np.abs(v), heads, seq)
    p = tlq.params(x_dtype=tlq.BF16 if bf16 else tlq.F16)
    out = torch.empty((seq, width), dtype=torch.bfloat16 if bf16 else torch.float16, device=gpu)
    tlq.causal_attention(dev(q, gpu, bf16), dev(k, gpu, bf16), dev(v, gpu, bf16), heads, seq, p, out)
    eps = 2.0 ** -8 if bf16 else 2.0 ** -11       # as above
    assert np.all(np.abs(host(out) - want) <= eps * (mag + np.abs(want)) + 2e-6)


@pytest.mark.parametrize("seq,heads", [(200, 2), (300, 86)])
@pytest.mark.parametrize("bf16,gap", [(False, 7.671875), (False, 7.78125), (True, 7.28125), (True, 7.625)])
def test_attention_divides_by_the_sum_in_32_bits(gpu, bf16, gap, seq, heads):
    """The probabilities are rounded to 16 bits for the product with V, not for their sum.  Key 0 has weight 1, all others
    exp(-gap / sqrt(128)), just above 1/2 and nearly half a unit of the last place off its rounding: dividing by the sum of
    the rounded ones would be off by 2^-11 (bf16: 2^-8), almost a unit of an output just below 2."""
    import torch
    g = np.random.default_rng([33, seq, int(gap * 64)])
    width = heads * 128
    rnd = BF if bf16 else F16
    q, k = np.zeros((seq, width)), np.zeros((seq, width))
    q[:, ::128], k[0, ::128] = 1.0, gap
    assert float(rnd(np.array([gap]))[0]) == gap
    v = np.asarray(rnd(np.broadcast_to(g.uniform(1.5, 2.0, width), (seq, width))), np.float64)
    weight = np.exp(-gap / np.sqrt(128.0))
    rounded = float(rnd(np.array([weight]))[0])
    n = np.arange(seq)[:, None]
    want = v * (1.0 + n * rounded) / (1.0 + n * weight)
    p = tlq.params(x_dtype=tlq.BF16 if bf16 else tlq.F16)
    out = torch.empty((seq, width), dtype=torch.bfloat16 if bf16 else torch.float16, device=gpu)
    tlq.causal_attention(dev(q, gpu, bf16), dev(k, gpu, bf16), dev(v, gpu, bf16), heads, seq, p, out)
    half = 2.0 ** (np.floor(np.log2(want)) - (8 if bf16 else 11))      # the output's rounding; sums of up to 300 terms in 32 bits
    assert np.all(np.abs(host(out) - want) <= half + want * (seq + 8) * 2.0 ** -24)


@pytest.mark.parametrize("bf16,seq,heads,samples", [(False, 72, 8, 40), (True, 300, 8, 16), (True, 513, 6, 11)])
def test_attention_of_a_sample_does_not_depend_on_its_neighbours(gpu, bf16, seq, heads, samples):
    """A calibration set may be split into any batches: a sample's outputs have the same bits alone and beside others."""
    import torch
    gen = torch.Generator(device=gpu)
    gen.manual_seed(34 + seq)
    dt, p = (torch.bfloat16, tlq.params(x_dtype=tlq.BF16)) if bf16 else (torch.float16, tlq.params())
    q, k, v = ((torch.randn((seq * samples, heads * 128), generator=gen, device=gpu) * 1.4).to(dt) for _ in range(3))
    out, one = torch.empty_like(q), torch.empty_like(q)
    tlq.causal_attention(q, k, v, heads, seq, p, out)
    for b in range(samples):
        r = slice(b * seq, (b + 1) * seq)
        tlq.causal_attention(q[r], k[r], v[r], heads, seq, p, one[r])
    assert torch.equal(out.view(torch.int16), one.view(torch.int16))


@pytest.mark.parametrize("bf16,seq,heads,samples,far", [(False, 40, 1, 1, "K"), (True, 35, 1, 1, "V"), (True, 33, 25, 3, ""),
                                                        (True, 259, 87, 1, "K"), (False, 257, 87, 1, "V")])
def test_attention_far_rows_and_partial_groups(gpu, bf16, seq, heads, samples, far):
    """Row strides of 2^27 elements and more (beyond 32-bit offsets inside a wave's rows) give the bits of dense rows;
    75 (sample, head) pairs leave the second group of pairs partly filled."""
    import torch
    g = np.random.default_rng([23, seq, heads])
    n, width = seq * samples, heads * 128
    rnd = BF if bf16 else F16
    q, k, v = (np.asarray(rnd(g.standard_normal((n, width)) * 1.5), np.float64) for _ in range(3))
    p = tlq.params(x_dtype=tlq.BF16 if bf16 else tlq.F16)
    t = {"Q": dev(q, gpu, bf16), "K": dev(k, gpu, bf16), "V": dev(v, gpu, bf16)}
    out = torch.empty((n, width), dtype=t["Q"].dtype, device=gpu)
    tlq.causal_attention(t["Q"], t["K"], t["V"], heads, seq, p, out)
    want, mag = ost.causal_attention(q, k, v, heads, seq), ost.causal_attention(q, k, np.abs(v), heads, seq)
    eps = 2.0 ** -8 if bf16 else 2.0 ** -11       # one rounding of every probability, one of the output
    assert np.all(np.abs(host(out) - want) <= eps * (mag + np.abs(want)) + 2e-6)
    if far:
        flat = torch.empty((n - 1) * (1 << 27) + width, dtype=out.dtype, device=gpu)
        t[far] = flat.as_strided((n, width), (1 << 27, 1)).copy_(t[far])
        again = torch.empty_like(out)
        tlq.causal_attention(t["Q"], t["K"], t["V"], heads, seq, p, again)
        assert torch.equal(out.view(torch.int16), again.view(torch.int16))


@pytest.mark.parametrize("seq,heads", [(200, 1), (300, 86)])
def test_attention_infinite_value_stays_behind_its_key(gpu, seq, heads):
    """An infinite V row reaches only the queries of its own 32-query block and later ones."""
    import torch
    g = np.random.default_rng(22)
    q, k, v = (F16(g.standard_normal((seq, heads * 128))).astype(np.float64) for _ in range(3))
    v[170] = np.inf
    out = torch.empty((seq, heads * 128), dtype=torch.float16, device=gpu)
    tlq.causal_attention(dev(q, gpu, False), dev(k, gpu, False), dev(v, gpu, False), heads, seq, tlq.params(), out)
    got = host(out)
    assert np.all(np.isfinite(got[:160])) and np.all(np.isinf(got[170:]))


def test_bf16_results_round_half_to_even(gpu):
    """float -> bf16: every tie, both neighbours, the overflow to infinity, NaN."""
    import torch
    a = np.arange(1 << 16, dtype=np.uint32).astype(np.uint16)
    ta = torch.from_numpy(a.view(np.int16)).view(torch.bfloat16).to(gpu).view(64, 1024)
    # x + x * 2^-8 lands on ties and off them: one float addition, one rounding
    tb = (ta.float() * 2.0 ** -8).to(torch.bfloat16)
    out = torch.empty_like(ta)
    tlq.residual_add(ta, tb, tlq.params(x_dtype=tlq.BF16), out)
    want = (ta.float().cpu() + tb.float().cpu()).numpy()
    want = np.where(np.isnan(want), np.nan, BF(np.nan_to_num(want, nan=0.0, posinf=np.inf, neginf=-np.inf)))
    np.testing.assert_array_equal(out.float().cpu().numpy(), want)


# one size per kernel and remainder: groups of 3, 5, 6 and 7 lanes, a wave of 1 / 2 / 4 chunks, a block of 2 / 4 / 8 chunks, the two-sweep
# kernel beyond 16384 channels, power-of-two groups with and without two rows per wave; odd row counts
@pytest.mark.parametrize("group,ci,co,sym,bits,bf16", [
    (24, 240, 5, 0, 4, False), (24, 24, 3, 1, 4, True), (40, 520, 6, 0, 3, True), (48, 3120, 2051, 1, 4, False),
    (56, 1064, 9, 0, 8, False), (56, 448, 300, 0, 4, True), (320, 640, 7, 1, 3, True), (0, 520, 3, 0, 4, True), (0, 1000, 9, 1, 4, False),
    (0, 1032, 2, 0, 8, False), (1536, 3072, 5, 0, 4, True), (0, 2056, 6, 1, 4, False), (0, 4104, 3, 0, 4, True),
    (0, 8200, 2, 1, 4, False), (0, 16384, 1, 0, 3, False), (0, 16392, 2, 1, 4, True), (8, 520, 3, 0, 4, False),
    (512, 1024, 5, 1, 4, False), (128, 1152, 2051, 0, 4, True)])
def test_quantiser_group_layouts(gpu, group, ci, co, sym, bits, bf16):
    import torch
    g = np.random.default_rng([23, group, ci, co])
    W = g.standard_normal((co, ci)).astype(np.float32) * 0.05
    W[0, :8] = 0.0
    W = BF(W) if bf16 else F16(W)
    s = np.exp(g.standard_normal(ci)).astype(np.float32)
    G = ci // (group or ci)
    code = tlq.BF16 if bf16 else tlq.F16
    p = tlq.params(bits=bits, group=group, symmetric=sym, x_dtype=code, yref_dtype=tlq.F32)
    tW = dev(W, gpu, bf16)
    codes = torch.full((co, ci), 99, dtype=torch.uint8, device=gpu)
    zp, delta = torch.empty((co, G), dtype=torch.uint8, device=gpu), torch.empty((co, G), dtype=torch.float32, device=gpu)
    wdq = torch.empty((co, ci + 8), dtype=tW.dtype, device=gpu)[:, :ci]
    tlq.fake_quant(tW, torch.from_numpy(s).to(gpu), p, codes, zp, delta, wdq)
    rc, rz, rd, rq = orc.fake_quant(W, s, bits, group, symmetric=bool(sym))
    np.testing.assert_array_equal(codes.cpu().numpy(), rc)
    np.testing.assert_array_equal(zp.cpu().numpy(), rz)
    np.testing.assert_array_equal(delta.cpu().numpy().view(np.uint32), rd.view(np.uint32))
    np.testing.assert_array_equal(host(wdq), (BF(rq) if bf16 else F16(rq)).astype(np.float64))
    # the candidates' operands (folded from 65536 outputs on at these bits, else the difference form),
    # stretches of candidates split over the grid
    n, na = (65536 + co - 1) // co if co > 256 and bits < 6 else 19, 7
    X = (BF if bf16 else F16)(g.standard_normal((n, ci)))
    w = np.full(n, 1.0 / n, np.float32)
    Y = orc.ref_output(X, W).astype(np.float32)
    al = (np.arange(na) / na).astype(np.float32)
    best, idx = torch.empty(ci, dtype=torch.float32, device=gpu), torch.empty(1, dtype=torch.int32, device=gpu)
    losses = torch.empty(na, dtype=torch.float32, device=gpu)
    ldy = co + -co % 4
    tY = torch.zeros((n, ldy), dtype=torch.float32, device=gpu)[:, :co]
    tY.copy_(torch.from_numpy(Y))
    tlq.scale_search(dev(X, gpu, bf16), tW, tY, torch.from_numpy(w).to(gpu), torch.from_numpy(al).to(gpu), p, best, idx,
                     losses)
    ref = orc.scale_search(X, W, Y, w, bits, group, al, symmetric=bool(sym))
    np.testing.assert_allclose(losses.cpu().numpy(), ref["losses"], rtol=1e-3)   # the parity bar of the search


@pytest.mark.parametrize("n,ci", [(1, 8), (255, 1024), (256, 1024), (257, 1024), (1030, 264), (4097, 72), (3, 131072), (1025, 512)])
def test_token_preparation_by_one_two_and_three_launches(gpu, n, ci):
    """Tokens up to 512 KB are prepared in one launch, larger ones in two where the call has scratch for the maxima of
    blocks (here with the reciprocals of the scales) and in three elsewhere: the same bits, with the largest
    magnitude in the last token's last channel.  The statistic of up to 1024 rows is one launch too."""
    import torch
    g = np.random.default_rng([26, n, ci])
    co = 40
    X, W = BF(g.standard_normal((n, ci)) * 3.0), BF(g.standard_normal((co, ci)) * 0.05)
    X[n - 1, ci - 1] = BF(np.array([3.0e5]))[0]
    tX, tW = dev(X, gpu, True), dev(W, gpu, True)
    s = torch.from_numpy(np.exp(g.standard_normal(ci)).astype(np.float32)).to(gpu)
    p = tlq.params(bits=4, group=8, x_dtype=tlq.BF16, yref_dtype=tlq.BF16)
    prepared = torch.zeros(tlq.prepared_tokens_bytes(n, ci, p), dtype=torch.uint8, device=gpu)
    tlq.prepare_tokens(tX, p, prepared)
    k = max(0, int(np.floor(np.log2(3.0e5))) + 1 - 15)          # the shift that brings the largest below 2^15
    body = prepared[256:256 + 2 * n * ci].view(torch.float16).view(n, ci)
    np.testing.assert_array_equal(host(body), F16(X * 2.0 ** -k).astype(np.float64))    # (subnormals round to fp16's grid)
    out = [torch.empty((n, co), dtype=torch.bfloat16, device=gpu) for _ in range(2)]
    tlq.apply_best(tX, tW, s, p, out[0])
    tlq.apply_best(tX, tW, s, p, out[1], prepared=prepared)
    assert torch.equal(out[0].view(torch.int16), out[1].view(torch.int16))
    xs = torch.empty(ci, dtype=torch.float32, device=gpu)
    tlq.x_stat(tX, p, xs)
    np.testing.assert_array_equal(host(xs), np.abs(X.astype(np.float64)).mean(0).astype(np.float32).astype(np.float64))


@pytest.mark.parametrize("n,sym", [(19, 0), (64, 0), (64, 1)])
def test_two_rows_of_a_wave_divide_together(gpu, n, sym):
    """Two rows share a wave and one test for quotients near a tie: here every quotient of the even rows lies on one at
    exponent zero, none of the odd rows' does; an odd number of rows, a last block of 128 channels, difference form
    (n = 19) and folded operands.  A tie that is rounded the wrong way moves a whole step: the losses see it."""
    import torch
    g = np.random.default_rng([25, n, sym])
    co, ci, na, bits = 2101, 1152, 4, 4
    W = g.standard_normal((co, ci)) * 0.05
    # steps of 1/16: quotients k + 1/2 between the group's ends, which are whole steps apart
    k = g.integers(-7, 7, (co, ci)) + 0.5
    k[:, 0::128], k[:, 1::128] = (-7.0, 7.0) if sym else (-8.0, 7.0)
    W[0::2] = k[0::2] / 16.0
    W, X = F16(W), F16(g.standard_normal((n, ci)))
    Y = orc.ref_output(X, W).astype(np.float32)
    w, al = np.full(n, 1.0 / n, np.float32), np.array([0.0, 0.25, 0.5, 0.75], np.float32)
    p = tlq.params(bits=bits, group=128, symmetric=sym, x_dtype=tlq.F16, yref_dtype=tlq.F32)
    best, idx = torch.empty(ci, dtype=torch.float32, device=gpu), torch.empty(1, dtype=torch.int32, device=gpu)
    losses = torch.empty(na, dtype=torch.float32, device=gpu)
    tY = torch.zeros((n, co + 3), dtype=torch.float32, device=gpu)[:, :co]
    tY.copy_(torch.from_numpy(Y))
    tlq.scale_search(dev(X, gpu, False), dev(W, gpu, False), tY, torch.from_numpy(w).to(gpu), torch.from_numpy(al).to(gpu), p,
                     best, idx, losses)
    ref = orc.scale_search(X, W, Y, w, bits, 128, al, symmetric=bool(sym))
    np.testing.assert_allclose(losses.cpu().numpy(), ref["losses"], rtol=1e-3)   # the parity bar of the search


@pytest.mark.parametrize("n,ci,co,pad", [(1, 8, 1, 0), (3, 520, 2, 8), (4097, 72, 5, 0), (9, 4104, 3, 16),
                                         (1, 131080, 2, 0), (6, 70000, 1, 8), (130, 1544, 2, 0)])
def test_token_preparation_and_folding_edges(gpu, n, ci, co, pad):
    """bf16 tokens beyond the fp16 range: the exponent shift follows the largest magnitude wherever it is
    (last row, last chunk), for row counts around the grid and widths around one wave and one block, and
    for rows that are split over the chip."""
    import torch
    g = np.random.default_rng([24, n, ci])
    X = BF(g.standard_normal((n, ci)) * 3.0)
    X[n - 1, ci - 1] = BF(np.array([-3.0e5]))[0]
    W = BF(g.standard_normal((co, ci)) * 0.05)
    p = tlq.params(bits=4, group=8, x_dtype=tlq.BF16, yref_dtype=tlq.F32)
    tX = torch.zeros((n, ci + pad), dtype=torch.bfloat16, device=gpu)[:, :ci]
    tX.copy_(dev(X, gpu, True))
    prep = torch.zeros(tlq.prepared_tokens_bytes(n, ci, p), dtype=torch.uint8, device=gpu)
    tlq.prepare_tokens(tX, p, prep)
    bits = int(prep[:4].view(torch.int32).item())
    assert bits == int(dev(np.abs(X).max().reshape(1), gpu, True).view(torch.int16).item())
    shift = max(0, min(24, ((bits >> 7) & 0xff) - 141))
    got = prep[256:256 + 2 * n * ci].view(torch.float16).float().cpu().numpy().reshape(n, ci)
    np.testing.assert_array_equal(got, F16(X.astype(np.float64) * 2.0 ** -shift).astype(np.float32))
    # the folded operand: one output per row, one token per column
    inv = (1.0 / np.exp(g.standard_normal(ci))).astype(np.float32)
    Y = np.zeros((n, co + -co % 4), np.float32)
    w = np.full(n, 1.0 / n, np.float32)
    loss, err = torch.empty(1, dtype=torch.float32, device=gpu), torch.empty(n, dtype=torch.float32, device=gpu)
    tlq.weighted_layer_err(tX, dev(W, gpu, True), torch.from_numpy(inv).to(gpu), torch.from_numpy(Y).to(gpu)[:, :co],
                           torch.from_numpy(w).to(gpu), p, loss, per_token_err=err)
    want = orc.per_token_err(Y[:, :co], orc.quantised_output(X, W, inv_s=inv))
    # the folded weight is rounded once to fp16: every output within 2^-11 sum |x inv w|, its square twice that
    mag = (np.abs(X.astype(np.float64) * inv) @ np.abs(W.astype(np.float64)).T)
    bound = (2.0 ** -10 * mag * mag + 1e-5 * mag * mag).mean(axis=1)
    assert np.all(np.abs(err.cpu().numpy() - want) <= bound)


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("n,c,pad,two,period", [(1, 8, 0, False, 0), (5, 72, 8, True, 3), (3, 1024, 0, False, 0),
                                                (3, 1032, 0, True, 0), (4, 5120, 0, False, 2), (2, 5128, 8, True, 0),
                                                (3, 75, 0, True, 2), (2, 520, 4, False, 0), (5, 64, 0, True, 2),
                                                (5, 72, 0, False, 2)])
def test_rmsnorm_row_widths(gpu, bf16, n, c, pad, two, period):
    """Rows held in registers (2 and 10 stretches), rows read twice, widths and strides that need the
    element-wise kernel; the second factor and the two multipliers."""
    import torch
    g = np.random.default_rng([25, n, c])
    rnd = BF if bf16 else F16
    z, zb = np.asarray(rnd(g.standard_normal((n, c)) * 3), np.float64), np.asarray(rnd(g.standard_normal((n, c))), np.float64)
    ma, mb = (np.float32(g.uniform(0.5, 2.0, c)) for _ in range(2))
    p = tlq.params(x_dtype=tlq.BF16 if bf16 else tlq.F16)
    dt = torch.bfloat16 if bf16 else torch.float16
    wide = lambda a: torch.zeros((n, c + pad), dtype=dt, device=gpu)[:, :c].copy_(dev(a, gpu, bf16))
    out = torch.full((n, c + pad), 7.0, dtype=dt, device=gpu)
    t = lambda a: torch.from_numpy(a).to(gpu)
    tlq.rmsnorm_mul(wide(z), p, out[:, :c], Zb=wide(zb) if two else None, m_a=t(ma), m_b=t(mb), period=period,
                    split=1 if period else 0)
    v = z * zb if two else z
    m = np.where(((np.arange(n) % period) >= 1)[:, None], mb, ma) if period else ma
    want = v / np.sqrt((v * v).mean(axis=1, keepdims=True) + 1e-6) * m
    got = host(out)
    assert np.all(got[:, c:] == 7.0)
    eps = 2.0 ** -8 if bf16 else 2.0 ** -11       # one rounding of the result, float arithmetic before it
    assert np.all(np.abs(got[:, :c] - want) <= eps * np.abs(want) * 1.001 + 1e-6 * np.abs(want) + 6e-8)


@pytest.mark.parametrize("B,N,C,l2", [(1, 1, 8, 0), (17, 65, 72, 1), (3, 64, 520, 0), (33, 1, 75, 1), (2, 129, 1096, 0),
                                       (3, 70, 248, 1), (3, 70, 256, 0),
                                       (7, 257, 8, 0), (8, 300, 8, 1)])
def test_selection_block_edges(gpu, B, N, C, l2):
    """64 positions a block, sixteen stretches of samples and rivals, 16-byte and 2-byte gradient rows; the
    masked maximum with a period that four interleaved rows wrap around, and one that is shorter."""
    import torch
    g = np.random.default_rng([26, B, N, C])
    G = F16(g.standard_normal((B * N, C)))
    p = tlq.params()
    sum_n = torch.empty(N, dtype=torch.float64, device=gpu)
    tlq.token_importance(dev(G, gpu, False), B, p, sum_n, l2=bool(l2))
    want = orc.token_importance(G, B, l2=bool(l2))
    np.testing.assert_allclose(sum_n.cpu().numpy(), want, rtol=1e-13)     # double sums in another order
    vals = np.floor(want * 4)                                             # ties
    mask = torch.empty(N, dtype=torch.uint8, device=gpu)
    k = (N + 1) // 2
    tlq.topk_mask(torch.from_numpy(vals).to(gpu), k, mask)
    rm = orc.top_fraction_mask(vals, k)
    np.testing.assert_array_equal(mask.cpu().numpy().astype(bool), rm)
    if C % 8 == 0:
        X = F16(g.standard_normal((B * N, C)))
        xs = torch.empty(C, dtype=torch.float32, device=gpu)
        tlq.x_stat_masked(dev(X, gpu, False), mask, p, xs)
        np.testing.assert_array_equal(xs.cpu().numpy(), orc.x_stat_topk_max(X, rm))
        tlq.x_stat(dev(X, gpu, False), p, xs)
        np.testing.assert_array_equal(xs.cpu().numpy(), orc.x_stat_mean(X))


# 128- and 256-tiles on both sides of the rule, k-tiles with 8 .. 56 channels in the last one, tokens and
# outputs around the tile edges, token tiles that fill one patch, strided operands
@pytest.mark.parametrize("n,ci,co,pad,bf16", [
    (1, 8, 1, 0, False), (127, 72, 129, 8, True), (128, 64, 128, 0, False), (129, 120, 127, 0, True),
    (257, 136, 255, 8, False), (1030, 184, 1290, 0, True), (1281, 264, 3330, 8, False), (5000, 72, 3400, 0, False)])
def test_products_at_tile_edges(gpu, n, ci, co, pad, bf16):
    import torch
    g = np.random.default_rng([27, n, ci, co])
    rnd = BF if bf16 else F16
    X, W = rnd(g.standard_normal((n, ci))), rnd(g.standard_normal((co, ci)) * 0.05)
    code = tlq.BF16 if bf16 else tlq.F16
    p = tlq.params(bits=4, group=8, x_dtype=code, yref_dtype=tlq.F32)
    wide = lambda a: torch.full((a.shape[0], ci + pad), 9.0, dtype=torch.bfloat16 if bf16 else torch.float16,
                                device=gpu)[:, :ci].copy_(dev(a, gpu, bf16))
    tX, tW = wide(X), wide(W)
    Y = torch.full((n, co + -co % 4 + 4), 7.0, dtype=torch.float32, device=gpu)
    tlq.ref_output(tX, tW, Y[:, :co], p)
    want = orc.ref_output(X, W)
    mag = np.abs(X.astype(np.float64)) @ np.abs(W.astype(np.float64)).T
    got = Y.cpu().numpy()
    assert np.all(got[:, co:] == 7.0)
    # exact products, float accumulation: ci roundings of at most 2^-24 of the magnitude
    assert np.all(np.abs(got[:, :co] - want) <= (ci + 2) * 2.0 ** -24 * mag + 1e-30)
    # the loss of the same product, against a target away from it, with and without per-token errors
    T = (want + g.standard_normal(want.shape)).astype(np.float32)
    Y[:, :co].copy_(torch.from_numpy(T))
    w = np.full(n, 1.0 / n, np.float32)
    ref, e = orc.weighted_layer_err(X, W.astype(np.float64), T, w)
    for per_tok in (False, True):
        loss, err = torch.empty(1, dtype=torch.float32, device=gpu), torch.empty(n, dtype=torch.float32, device=gpu)
        tlq.weighted_layer_err(tX, tW, None, Y[:, :co], torch.from_numpy(w).to(gpu), p, loss,
                               per_token_err=err if per_tok else None)
        np.testing.assert_allclose(float(loss.item()), ref, rtol=2e-5)      # float sums of positive terms
        if per_tok:
            np.testing.assert_allclose(err.cpu().numpy(), e, rtol=2e-5)


@pytest.mark.parametrize("n,co,ydt,bf16", [(300, 520, tlq.F16, False), (257, 264, tlq.BF16, True), (130, 203, tlq.F32, False),
                                           (8000, 3400, tlq.BF16, True)])
def test_difference_target_in_the_product_epilogue(gpu, n, co, ydt, bf16):
    """Eight bits: the target minus the full-precision product is formed where the product is stored - 16-bit
    targets inside the tiles through LDS, at the edges and in float directly, small and big tiles."""
    import torch
    g = np.random.default_rng([28, n, co])
    ci, na = 64, 2
    rnd = BF if bf16 else F16
    X, W = rnd(g.standard_normal((n, ci))), rnd(g.standard_normal((co, ci)) * 0.05)
    Yd = orc.ref_output(X, W) + 0.01 * g.standard_normal((n, co))
    tdt = {tlq.F16: torch.float16, tlq.BF16: torch.bfloat16, tlq.F32: torch.float32}[ydt]
    Y = torch.zeros((n, co + -co % 8 + 8), dtype=tdt, device=gpu)[:, :co]
    Y.copy_(torch.from_numpy(Yd).to(gpu))
    Yv = Y.double().cpu().numpy()
    w = g.uniform(0.1, 1.0, n).astype(np.float32) / n
    al = np.array([0.0, 0.5], np.float32)
    p = tlq.params(bits=8, group=32, x_dtype=tlq.BF16 if bf16 else tlq.F16, yref_dtype=ydt)
    best, idx = torch.empty(ci, dtype=torch.float32, device=gpu), torch.empty(1, dtype=torch.int32, device=gpu)
    losses = torch.empty(na, dtype=torch.float32, device=gpu)
    t = lambda a: torch.from_numpy(a).to(gpu)
    tlq.scale_search(dev(X, gpu, bf16), dev(W, gpu, bf16), Y, t(w), t(al), p, best, idx, losses)
    ref = orc.scale_search(X, W, Yv, w, 8, 32, al)
    np.testing.assert_allclose(losses.cpu().numpy(), ref["losses"], rtol=1e-3)   # the parity bar of the search


@pytest.mark.parametrize("n,ci,co", [(4500, 2304, 40), (9000, 264, 300), (300, 4096, 2100)])
def test_symmetric_products_deal_every_tile(gpu, n, ci, co):
    """9 tile columns (one full block of eight and one over), one column block with a k tail in the loss, eight
    patches per candidate: every element of the matrix and the losses through it."""
    import torch
    g = np.random.default_rng([29, n, ci])
    X, W = F16(g.standard_normal((n, ci))), F16(g.standard_normal((co, ci)) * 0.05)
    w = g.uniform(0.1, 1.0, n).astype(np.float32) / n
    p = tlq.params(bits=3, group=8)
    tX, tw = dev(X, gpu, False), torch.from_numpy(w).to(gpu)
    gram = torch.zeros(tlq.token_gram_bytes(ci), dtype=torch.uint8, device=gpu)
    tlq.token_gram(tX, tw, p, gram)
    f, cs, C = tlq.gram_views(gram, ci)
    G = f.double() * cs.double()[:, None] * cs.double()[None, :] * C.double()
    Xd = tX.double()
    want = Xd.t().contiguous() @ (Xd * tw.double()[:, None])
    scale = want.diagonal().sqrt()
    # tokens times sqrt(w) and the matrix itself are rounded to fp16 once each
    assert (((G - want).abs() / (scale[:, None] * scale[None, :])).max().item()) <= 3 * 2.0 ** -11
    al = np.array([0.0, 0.4, 0.8], np.float32)
    xs = torch.empty(ci, dtype=torch.float32, device=gpu)
    tlq.x_stat(tX, p, xs)
    best, idx = torch.empty(ci, dtype=torch.float32, device=gpu), torch.empty(1, dtype=torch.int32, device=gpu)
    losses, table = torch.empty(3, dtype=torch.float32, device=gpu), torch.empty((3, ci), dtype=torch.float32, device=gpu)
    tlq.scale_search_gram(gram, dev(W, gpu, False), torch.from_numpy(al).to(gpu), p, xs, best, idx, losses, s_table_out=table)
    for k in range(3):
        s = table[k].cpu().numpy()
        deq = torch.from_numpy(orc.fake_quant(W, s, 3, 8)[3].astype(np.float64)).to(gpu)
        d = dev(W, gpu, False).double() - deq / table[k].double()[None, :]
        ref = (((d @ want) * d).sum() / co).item()
        assert abs(losses[k].item() - ref) <= 1e-3 * ref      # the parity bar of the search


@pytest.mark.parametrize("kind", [0, 1])
@pytest.mark.parametrize("n,ci,co,na,bf16", [(1, 8, 1, 1, False), (1024, 72, 3, 20, False), (1025, 72, 3, 20, False),
                                             (130, 520, 2, 17, False), (1, 8, 1, 1, True), (700, 64, 1, 1, True),
                                             (3000, 1032, 5, 33, True), (20000, 136, 4, 2, True)])
def test_table_of_a_search_that_takes_its_own_statistic(gpu, n, ci, co, na, bf16, kind):
    """The statistic inside a search (one launch up to 1024 rows, else chunks; with bf16 tokens their maximum comes from
    the same pass if its words fit into the operands' place) gives the table of the two separate calls and the
    losses of the search that is handed the statistic."""
    import torch
    g = torch.Generator(device=gpu)
    g.manual_seed(41 + n)
    dt, code = (torch.bfloat16, tlq.BF16) if bf16 else (torch.float16, tlq.F16)
    X = torch.randn((n, ci), generator=g, device=gpu)
    X[:, 0] *= 3e5 if bf16 else 30.0             # (the shift of the fp16 re-expression is not zero)
    X, W = X.to(dt), (torch.randn((co, ci), generator=g, device=gpu) * 0.05).to(dt)
    Y = torch.randn((n, co + -co % 8), generator=g, device=gpu).to(dt)[:, :co]
    w, al = torch.rand(n, generator=g, device=gpu) / n, torch.arange(na, device=gpu) / (1.0 * na)
    p = tlq.params(group=8, xstat_kind=kind, x_dtype=code, yref_dtype=code)
    f = lambda *s: torch.empty(s, dtype=torch.float32, device=gpu)
    xs, table, got = f(ci), f(na, ci), f(na * ci + 1)
    tlq.x_stat(X, p, xs)
    tlq.scale_table(xs, al, table)
    res = []
    for stat in (None, xs):
        best, idx, losses = f(ci), torch.empty(1, dtype=torch.int32, device=gpu), f(na)
        tlq.scale_search(X, W, Y, w, al, p, best, idx, losses, x_stat_in=stat, s_table_out=got[1:].view(na, ci))
        if bf16:      # sums of a wide range in another order: the last bit of a double, seldom one of the float
            assert torch.allclose(got[1:].view(na, ci), table, rtol=2.0 ** -22, atol=0.0)
        else:
            assert torch.equal(got[1:].view(na, ci), table)
        res.append((losses, idx, best))
    torch.testing.assert_close(res[0][0], res[1][0], rtol=1e-3 if bf16 else 0.0, atol=0.0)


@pytest.mark.parametrize("n,ci,bf16", [(1, 8, False), (7, 512, True), (8, 520, False), (9, 4096, True), (17, 4104, False),
                                       (10, 8192, True), (3, 9008, False), (70, 1024, True)])
def test_activation_codes_at_strip_and_block_edges(gpu, n, ci, bf16):
    """Blocks of eight rows, strips of 512 channels, eight waves: codes and steps bit for bit, infinities and NaN among
    the tokens, an odd row stride."""
    import torch
    g = np.random.default_rng([45, n, ci])
    X = g.standard_normal((n, ci + 8)).astype(np.float32) * 3.0
    X[0, ci // 2] = 200.0
    if n > 2:
        X[1], X[2, ci - 1] = 0.0, 1e-7
    X = (BF if bf16 else F16)(X)
    inv = (1.0 / g.lognormal(0, 0.6, ci)).astype(np.float32)
    p = tlq.params(group=8, act_bits=6, x_dtype=tlq.BF16 if bf16 else tlq.F16)
    codes, sigma = torch.empty((n, ci), dtype=torch.float16, device=gpu), torch.empty(n, dtype=torch.float32, device=gpu)
    tX = dev(X, gpu, bf16)
    tlq.act_fake_quant(tX[:, :ci], torch.from_numpy(inv).to(gpu), p, codes, sigma)
    rc, rs = orc.act_quant(np.ascontiguousarray(X[:, :ci]), inv, 6)
    assert np.array_equal(sigma.cpu().numpy().view(np.uint32), rs.view(np.uint32))
    assert np.array_equal(codes.cpu().numpy().astype(np.int16), rc)
    if n > 4:        # a NaN takes the lowest code and does not count for the step; an infinity makes the others zero
        tX[3, 0], tX[4, ci - 1] = float("nan"), float("inf")
        tlq.act_fake_quant(tX[:, :ci], torch.from_numpy(inv).to(gpu), p, codes, sigma)
        c = codes.cpu().numpy()
        assert c[3, 0] == -32 and np.array_equal(c[:3].astype(np.int16), rc[:3]) and np.array_equal(c[5:].astype(np.int16), rc[5:])
        assert not c[4, :ci - 1].any() and c[4, ci - 1] == -32 and np.isinf(sigma[4].item())


@pytest.mark.parametrize("n,ci,co,bits,sym,abits,bf16", [
    (1, 72, 1, 4, True, 8, False), (130, 128, 129, 8, True, 8, True), (257, 136, 258, 7, False, 6, False),
    (300, 1000, 70, 3, True, 8, True), (520, 1096, 261, 4, False, 8, False), (40, 4104, 33, 4, True, 2, False),
    (64, 8200, 20, 2, False, 8, True), (9, 16384, 10, 4, True, 8, False), (1000, 136, 2001, 4, True, 8, False)])
def test_integer_contraction_edges(gpu, n, ci, co, bits, sym, abits, bf16):
    """One step per weight row and activation codes: widths that are no multiple of the 128-code k-tile, each width class
    of the quantiser, ragged tiles; the losses of a search and the propagated output."""
    import torch
    g = np.random.default_rng([47, n, ci])
    rnd = BF if bf16 else F16
    X, W = rnd(g.standard_normal((n, ci)) * 2.0), rnd(g.standard_normal((co, ci)) * 0.05)
    code, dt = (tlq.BF16, torch.bfloat16) if bf16 else (tlq.F16, torch.float16)
    Y = torch.zeros((n, co + -co % 8), dtype=torch.float32, device=gpu)[:, :co]
    Y.copy_(torch.from_numpy(orc.ref_output(X, W) + 0.05 * g.standard_normal((n, co))).to(gpu))
    w = g.uniform(0.1, 1.0, n).astype(np.float32) / n
    al = np.array([0.0, 0.4, 0.8], np.float32)
    p = tlq.params(bits=bits, group=0, symmetric=int(sym), act_bits=abits, x_dtype=code, yref_dtype=tlq.F32)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(gpu)
    f = lambda *s: torch.empty(s, dtype=torch.float32, device=gpu)
    best, idx, losses, table = f(ci), torch.empty(1, dtype=torch.int32, device=gpu), f(3), f(3, ci)
    tlq.scale_search(dev(X, gpu, bf16), dev(W, gpu, bf16), Y, t(w), t(al), p, best, idx, losses, s_table_out=table)
    ref = orc.scale_search(X, W, Y.double().cpu().numpy(), w, bits, 0, al, s_table=table.cpu().numpy(), symmetric=sym, act_bits=abits)
    # exact sums of codes; three float roundings of a product, then float sums of squares (n * co / 64 terms a lane at most);
    # a residual is at least a hundredth of the product's size here: 2 * 100 * 4 * 2^-24
    np.testing.assert_allclose(losses.cpu().numpy(), ref["losses"], rtol=5e-5)
    s = table[1].contiguous()
    Z = torch.full((n, co + -co % 8 + 8), 7.0, dtype=dt, device=gpu)
    tlq.apply_best(dev(X, gpu, bf16), dev(W, gpu, bf16), s, p, Z[:, :co])
    want = orc.apply_best(X, W, s.cpu().numpy(), bits, 0, symmetric=sym, act_bits=abits)
    got = host(Z)
    assert np.all(got[:, co:] == 7.0)
    # one rounding of the result to 16 bits, four float roundings before it; the oracle's dequantised weights are floats,
    # each 2^-24 of itself away from code times step, which stays where a sum cancels
    c, sg = orc.act_quant(X, orc.recip_scale(s.cpu().numpy()), abits)
    deq = orc.fake_quant(W, s.cpu().numpy(), bits, 0, symmetric=sym)[3]
    mag = (np.abs(c.astype(np.float64)) * sg.astype(np.float64)[:, None]) @ np.abs(deq.astype(np.float64)).T
    eps = 2.0 ** -8 if bf16 else 2.0 ** -11
    assert np.all(np.abs(got[:, :co] - want) <= (eps + 4 * 2.0 ** -24) * np.abs(want) + 2.0 ** -24 * (mag + 1.0))


# (tokens, outputs): products of codes in tiles of 192, 256 and 320 tokens, more than 256 of 128 x 128 and fewer, each with
# whole tiles and with remainders on both sides
@pytest.mark.parametrize("n,co,bf16", [(2500, 4101, True), (2496, 4096, False), (4000, 4002, False), (4096, 4096, True),
                                       (4700, 4090, True), (4800, 4096, False), (2000, 3001, False), (2048, 3072, True), (1000, 2001, True)])
def test_integer_products_in_every_tile(gpu, n, co, bf16):
    import torch
    g = np.random.default_rng([48, n, co])
    ci, rnd = 136, BF if bf16 else F16
    X, W = rnd(g.standard_normal((n, ci)) * 2.0), rnd(g.standard_normal((co, ci)) * 0.05)
    code, dt = (tlq.BF16, torch.bfloat16) if bf16 else (tlq.F16, torch.float16)
    s = np.exp(g.uniform(-1.0, 1.0, ci)).astype(np.float32)
    p = tlq.params(bits=4, group=0, symmetric=1, act_bits=8, x_dtype=code, yref_dtype=code)
    Z = torch.full((n, co + -co % 8 + 8), 7.0, dtype=dt, device=gpu)
    tlq.apply_best(dev(X, gpu, bf16), dev(W, gpu, bf16), torch.from_numpy(s).to(gpu), p, Z[:, :co])
    assert bool((Z[:, co:] == 7.0).all())
    c, sg = orc.act_quant(X, orc.recip_scale(s), 8)
    deq = orc.fake_quant(W, s, 4, 0, symmetric=True)[3]
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).to(gpu)
    tc, td, ts = t(c), t(deq), t(sg)[:, None]
    want, mag = (tc @ td.t()) * ts, (tc.abs() @ td.abs().t()) * ts
    # the bound of test_integer_contraction_edges
    eps = 2.0 ** -8 if bf16 else 2.0 ** -11
    assert bool(((Z[:, :co].double() - want).abs() <= (eps + 4 * 2.0 ** -24) * want.abs() + 2.0 ** -24 * (mag + 1.0)).all())


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("sym,inf", [(1, np.inf), (1, -np.inf), (0, np.inf), (0, -np.inf)])
def test_integer_products_of_an_infinite_weight(gpu, bf16, sym, inf):
    """The step of its row is infinite and the codes beside it are zero: NaN for every token, like the oracle's dequantised
    weights, and nothing of it in the other rows."""
    import torch
    g = np.random.default_rng(50)
    n, ci, co, rnd = 130, 136, 72, BF if bf16 else F16
    X, W = rnd(g.standard_normal((n, ci)) * 2.0), rnd(g.standard_normal((co, ci)) * 0.05)
    bad = W.copy()
    bad[3, 7] = inf
    with np.errstate(invalid="ignore"):
        assert np.isnan(np.delete(orc.fake_quant(bad[3:4], None, 4, 0, symmetric=bool(sym))[3], 7)).all()
    code, dt = (tlq.BF16, torch.bfloat16) if bf16 else (tlq.F16, torch.float16)
    p = tlq.params(bits=4, group=0, symmetric=sym, act_bits=8, x_dtype=code, yref_dtype=code)
    tX, s = dev(X, gpu, bf16), torch.ones(ci, device=gpu)
    out = [torch.empty((n, co), dtype=dt, device=gpu) for _ in range(2)]
    tlq.apply_best(tX, dev(W, gpu, bf16), s, p, out[0])
    tW = dev(W, gpu, bf16)
    tW[3, 7] = float(inf)
    tlq.apply_best(tX, tW, s, p, out[1])
    rest = [r for r in range(co) if r != 3]
    assert bool(out[1][:, 3].isnan().all()) and torch.equal(out[0][:, rest].view(torch.int16), out[1][:, rest].view(torch.int16))


def test_integer_losses_in_square_tiles(gpu):
    """40 candidates of 250 x 72 x 1000: 160 tiles of 256 x 256, one round; the partial sums of smaller ones would not fit."""
    import torch
    n, ci, co, na = 250, 72, 1000, 40
    g = np.random.default_rng(49)
    X, W = F16(g.standard_normal((n, ci)) * 2.0), F16(g.standard_normal((co, ci)) * 0.05)
    Y = F16(orc.ref_output(X, W) + 0.05 * g.standard_normal((n, co)))
    w, al = g.uniform(0.1, 1.0, n).astype(np.float32) / n, (np.arange(na) / na).astype(np.float32)
    p = tlq.params(bits=4, group=0, symmetric=1, act_bits=8)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(gpu)
    f = lambda *s: torch.empty(s, dtype=torch.float32, device=gpu)
    best, idx, losses, table = f(ci), torch.empty(1, dtype=torch.int32, device=gpu), f(na), f(na, ci)
    tlq.scale_search(t(X), t(W), t(Y), t(w), t(al), p, best, idx, losses, s_table_out=table)
    ref = orc.scale_search(X, W, Y, w, 4, 0, al, s_table=table.cpu().numpy(), symmetric=True, act_bits=8)
    np.testing.assert_allclose(losses.cpu().numpy(), ref["losses"], rtol=5e-5)      # the bound of test_integer_contraction_edges


def test_search_over_more_candidates_than_a_block_takes(gpu):
    """40 candidates with activation codes (a block's maxima hold 32), few rows and many."""
    import torch
    for n in (9, 3000):
        g = np.random.default_rng([46, n])
        X, W = F16(g.standard_normal((n, 128))), F16(g.standard_normal((24, 128)) * 0.05)
        Y, w, al = F16(orc.ref_output(X, W)), np.full(n, 1.0 / n, np.float32), (np.arange(40) / 40).astype(np.float32)
        p = tlq.params(group=0, symmetric=1, act_bits=6)
        t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(gpu)
        best, idx = torch.empty(128, device=gpu), torch.empty(1, dtype=torch.int32, device=gpu)
        losses = torch.empty(40, device=gpu)
        tlq.scale_search(t(X), t(W), t(Y), t(w), t(al), p, best, idx, losses)
        ref = orc.scale_search(X, W, Y, w, 4, 0, al, symmetric=True, act_bits=6)
        np.testing.assert_allclose(losses.cpu().numpy(), ref["losses"], rtol=1e-3)     # the parity bar of the search


# What is read of more than 320 MB, and outputs of more than 230 MB, go past the caches by other instructions: the same
# bits as in pieces that do not.
def pieces(n, k):
    return [slice(i * n // k, (i + 1) * n // k) for i in range(k)]


@pytest.mark.parametrize("mb", [170, 240])             # of one matrix: loads past the caches, and stores too
@pytest.mark.parametrize("c", [1000, 4096, 5128])      # rows held in 2 and 10 registers quads, and read twice
def test_long_streams_of_the_glue(gpu, c, mb):
    import torch
    n = int(mb * 1e6) // (2 * c)
    g = torch.Generator(device=gpu)
    g.manual_seed(51)
    A, B = (torch.randn((n, c), generator=g, device=gpu, dtype=torch.bfloat16) for _ in range(2))
    m, p = torch.rand(c, generator=g, device=gpu), tlq.params(x_dtype=tlq.BF16)
    for call in (lambda r, o: tlq.rmsnorm_mul(A[r], p, o, m_a=m), lambda r, o: tlq.rmsnorm_mul(A[r], p, o, Zb=B[r]),
                 lambda r, o: tlq.silu_mul(A[r], B[r], p, o), lambda r, o: tlq.residual_add(A[r], B[r], p, o)):
        whole, parts = torch.empty_like(A), torch.empty_like(A)
        call(slice(0, n), whole)
        for r in pieces(n, 3):
            call(r, parts[r])
        assert torch.equal(whole.view(torch.int16), parts.view(torch.int16))
    # the tokens in fp16, behind 256 bytes that hold the maximum: the same one in every piece
    for r in pieces(n, 3):
        A[r.start] = 9.0
    ready = lambda r: tlq.prepare_tokens(A[r], p, torch.zeros(tlq.prepared_tokens_bytes(r.stop - r.start, c, p),
                                                              dtype=torch.uint8, device=gpu))
    p = tlq.params(group=8, x_dtype=tlq.BF16)
    whole = ready(slice(0, n))[256:256 + 2 * n * c].view(torch.int16)
    parts = [ready(r)[256:256 + 2 * (r.stop - r.start) * c].view(torch.int16) for r in pieces(n, 3)]
    assert torch.equal(whole, torch.cat(parts)) and int(whole.abs().max()) > 0


def test_long_streams_of_statistics_and_codes(gpu):
    import torch
    n, c = 42000, 4096
    g = torch.Generator(device=gpu)
    g.manual_seed(52)
    X = torch.randn((n, c), generator=g, device=gpu, dtype=torch.float16)
    p, f = tlq.params(act_bits=8), lambda *s: torch.empty(s, dtype=torch.float32, device=gpu)
    norms = [torch.empty(n, dtype=torch.float64, device=gpu) for _ in range(2)]
    tlq.token_importance(X, 1, p, norms[0])
    xs, mask = f(c), (torch.rand(700, generator=g, device=gpu) < 0.9).to(torch.uint8)
    tlq.x_stat(X, p, xs)
    assert torch.equal(xs, (X.abs().sum(0, dtype=torch.float64) / n).float())       # sums of fp16 are exact in double
    tlq.x_stat_masked(X, mask, p, xs)
    assert torch.equal(xs, X.view(-1, 700, c)[:, mask.bool()].abs().amax((0, 1)).float())
    codes, sg = [torch.empty((n, c), dtype=torch.float16, device=gpu) for _ in range(2)], [f(n), f(n)]
    tlq.act_fake_quant(X, None, p, codes[0], sg[0])
    for r in pieces(n, 3):
        tlq.token_importance(X[r], 1, p, norms[1][r])
        tlq.act_fake_quant(X[r], None, p, codes[1][r], sg[1][r])
    for a, b in (norms, codes, sg):
        assert torch.equal(a, b)
    # operands of 18 candidates: 755 MB (fp16) or, with one step per row, 377 MB (int8) together
    W, n = X[:5120], 64
    Y, w = torch.randn((n, 5120), generator=g, device=gpu, dtype=torch.float16), torch.rand(n, generator=g, device=gpu) / n
    al = torch.arange(18, device=gpu) / 20.0
    for q in (tlq.params(), tlq.params(group=0, symmetric=1, act_bits=8)):
        best, idx, many, one = f(c), torch.empty(1, dtype=torch.int32, device=gpu), f(18), f(18)
        tlq.scale_search(X[6000:6000 + n], W, Y, w, al, q, best, idx, many)
        for k in range(18):
            tlq.scale_search(X[6000:6000 + n], W, Y, w, al[k:k + 1], q, best, idx, one[k:k + 1])
        torch.testing.assert_close(many, one, rtol=1e-5, atol=0.0)         # (tiles of another size: sums in another order)


# Row strides of 2^21 elements and more leave the pipelined kernel's 32-bit offsets: the register-staged kernel
# serves them.  257 or 300 rows (two tiles, the second ragged) of a matrix that is never allocated densely.
WIDE = 1 << 21


def wide_rows(a, gpu, bf16):
    import torch
    n, c = a.shape
    dt = torch.bfloat16 if bf16 else torch.float16
    flat = torch.empty((n - 1) * WIDE + c, dtype=dt, device=gpu)
    return flat.as_strided((n, c), (WIDE, 1)).copy_(dev(a, gpu, bf16))


@pytest.mark.parametrize("n,ci,co,side,bf16", [(300, 136, 300, "X", False), (257, 64, 520, "X", True),
                                               (130, 200, 257, "W", True), (513, 72, 129, "W", False)])
def test_products_with_very_wide_rows(gpu, n, ci, co, side, bf16):
    """Full-precision product (float and 16-bit output) and the loss with and without per-token errors."""
    import torch
    g = np.random.default_rng([31, n, ci, co])
    rnd = BF if bf16 else F16
    X, W = rnd(g.standard_normal((n, ci))), rnd(g.standard_normal((co, ci)) * 0.05)
    tX = wide_rows(X, gpu, bf16) if side == "X" else dev(X, gpu, bf16)
    tW = wide_rows(W, gpu, bf16) if side == "W" else dev(W, gpu, bf16)
    want = orc.ref_output(X, W)
    mag = np.abs(X.astype(np.float64)) @ np.abs(W.astype(np.float64)).T
    code = tlq.BF16 if bf16 else tlq.F16
    p = tlq.params(group=8, x_dtype=code, yref_dtype=tlq.F32)
    Y = torch.full((n, co + -co % 4 + 4), 7.0, dtype=torch.float32, device=gpu)
    tlq.ref_output(tX, tW, Y[:, :co], p)
    got = Y.cpu().numpy()
    assert np.all(got[:, co:] == 7.0)
    # exact products, float accumulation: ci roundings of at most 2^-24 of the magnitude
    assert np.all(np.abs(got[:, :co] - want) <= (ci + 2) * 2.0 ** -24 * mag + 1e-30)
    H = torch.full((n, co + -co % 8 + 8), 7.0, dtype=tX.dtype, device=gpu)
    tlq.ref_output(tX, tW, H[:, :co], tlq.params(group=8, x_dtype=code, yref_dtype=code))
    # ... and one rounding of the result (and at most one float rounding apart from the float output's)
    eps = 2.0 ** -8 if bf16 else 2.0 ** -11
    assert np.all(host(H)[:, co:] == 7.0)
    assert np.all(np.abs(host(H)[:, :co] - want) <= eps * np.abs(want) * 1.01 + (ci + 2) * 2.0 ** -23 * mag + 2.0 ** -24)
    T = (want + g.standard_normal(want.shape)).astype(np.float32)
    Y[:, :co].copy_(torch.from_numpy(T))
    w = np.full(n, 1.0 / n, np.float32)
    ref, e = orc.weighted_layer_err(X, W.astype(np.float64), T, w)
    for per_tok in (False, True):
        loss, err = torch.empty(1, dtype=torch.float32, device=gpu), torch.empty(n, dtype=torch.float32, device=gpu)
        tlq.weighted_layer_err(tX, tW, None, Y[:, :co], torch.from_numpy(w).to(gpu), p, loss,
                               per_token_err=err if per_tok else None)
        np.testing.assert_allclose(float(loss.item()), ref, rtol=2e-5)      # float sums of positive terms
        if per_tok:
            np.testing.assert_allclose(err.cpu().numpy(), e, rtol=2e-5)


@pytest.mark.parametrize("bits,act,ydt,bf16", [(4, 0, tlq.F16, False), (8, 0, tlq.F16, False), (8, 0, tlq.BF16, True),
                                               (8, 0, tlq.F32, False), (4, 8, tlq.F16, False)])
def test_search_and_propagation_with_very_wide_token_rows(gpu, bits, act, ydt, bf16):
    """Folded and difference form (the target is subtracted where that kernel stores), several candidates,
    activation quantisation (whose codes are dense again); then the propagated output."""
    import torch
    n, ci, co, na = 300, 136, 300, 3
    g = np.random.default_rng([32, bits, act])
    rnd = BF if bf16 else F16
    X, W = rnd(g.standard_normal((n, ci))), rnd(g.standard_normal((co, ci)) * 0.05)
    tdt = {tlq.F16: torch.float16, tlq.BF16: torch.bfloat16, tlq.F32: torch.float32}[ydt]
    Y = torch.zeros((n, co + -co % 8), dtype=tdt, device=gpu)[:, :co]
    Y.copy_(torch.from_numpy(orc.ref_output(X, W) + 0.01 * g.standard_normal((n, co))).to(gpu))
    w = g.uniform(0.1, 1.0, n).astype(np.float32) / n
    al = np.array([0.0, 0.4, 0.8], np.float32)
    code = tlq.BF16 if bf16 else tlq.F16
    p = tlq.params(bits=bits, group=8, act_bits=act, x_dtype=code, yref_dtype=ydt)
    tX, tW = wide_rows(X, gpu, bf16), dev(W, gpu, bf16)
    f = lambda *s: torch.empty(s, dtype=torch.float32, device=gpu)
    best, idx, losses = f(ci), torch.empty(1, dtype=torch.int32, device=gpu), f(na)
    t = lambda a: torch.from_numpy(a).to(gpu)
    tlq.scale_search(tX, tW, Y, t(w), t(al), p, best, idx, losses)
    ref = orc.scale_search(X, W, Y.double().cpu().numpy(), w, bits, 8, al, act_bits=act)
    np.testing.assert_allclose(losses.cpu().numpy(), ref["losses"], rtol=1e-3)   # the parity bar of the search
    # the same call on dense tokens: same operands, the output's products added in the same order
    Z, Zd = torch.empty((n, co + -co % 8), dtype=tX.dtype, device=gpu), torch.empty((n, co + -co % 8), dtype=tX.dtype, device=gpu)
    tlq.apply_best(tX, tW, best, p, Z[:, :co])
    tlq.apply_best(dev(X, gpu, bf16), tW, best, p, Zd[:, :co])
    eps = 2.0 ** -7 if bf16 else 2.0 ** -10       # float sums in another order: one unit of the 16-bit result
    a, b = host(Z[:, :co]), host(Zd[:, :co])
    assert np.all(np.abs(a - b) <= eps * np.abs(b) + 1e-5)


def test_token_matrix_of_more_than_two_million_tokens(gpu):
    """The transposed tokens have rows of 2^21 elements and more: the symmetric product in the same kernel, two
    tile columns, sixteen splits."""
    import torch
    n, ci = WIDE + 5, 264
    g = torch.Generator(device=gpu)
    g.manual_seed(33)
    X = torch.randn((n, ci), generator=g, device=gpu, dtype=torch.float16)
    X[:, 5] *= 20.0
    w = torch.rand(n, generator=g, device=gpu) / n
    p = tlq.params(group=8)
    gram = torch.zeros(tlq.token_gram_bytes(ci), dtype=torch.uint8, device=gpu)
    tlq.token_gram(X, w, p, gram)
    f, cs, C = tlq.gram_views(gram, ci)
    G = f.double() * cs.double()[:, None] * cs.double()[None, :] * C.double()
    want = torch.zeros((ci, ci), dtype=torch.float64, device=gpu)
    for r in range(0, n, 1 << 18):
        x = X[r:r + (1 << 18)].double()
        want += x.t().contiguous() @ (x * w[r:r + (1 << 18)].double()[:, None])
    scale = want.diagonal().sqrt()
    # tokens times sqrt(w) and the matrix itself are rounded to fp16 once each (three roundings in a product);
    # an accumulator takes 131,136 / 16 float additions of a split: 8196 * 2^-24 = 2^-11
    assert (((G - want).abs() / (scale[:, None] * scale[None, :])).max().item()) <= 4 * 2.0 ** -11


# (tokens, channels, outputs, candidates): launches of tiles of 192 and of 320 tokens, with remainders on both sides, a
# k tail, one candidate and several
@pytest.mark.parametrize("n,ci,co,na,act,bf16", [
    (760, 136, 770, 16, 0, False), (1270, 136, 776, 16, 0, True), (760, 264, 776, 16, 8, True), (1270, 264, 776, 16, 6, False),
    (2560, 64, 1792, 6, 0, False), (1280, 192, 1024, 16, 8, False)])
def test_losses_of_narrow_and_wide_tiles(gpu, n, ci, co, na, act, bf16):
    import torch
    g = np.random.default_rng([41, n, ci, co])
    rnd = BF if bf16 else F16
    X, W = rnd(g.standard_normal((n, ci))), rnd(g.standard_normal((co, ci)) * 0.05)
    code = tlq.BF16 if bf16 else tlq.F16
    p = tlq.params(bits=4, group=0 if act else 8, symmetric=1, act_bits=act, x_dtype=code, yref_dtype=code)
    Y = torch.zeros((n, co + -co % 8), dtype=torch.bfloat16 if bf16 else torch.float16, device=gpu)[:, :co]
    tlq.ref_output(dev(X, gpu, bf16), dev(W, gpu, bf16), Y, p)
    w = g.uniform(0.1, 1.0, n).astype(np.float32) / n
    al = np.array([k / na for k in range(na)], np.float32)
    best, idx = torch.empty(ci, dtype=torch.float32, device=gpu), torch.empty(1, dtype=torch.int32, device=gpu)
    losses, table = torch.empty(na, dtype=torch.float32, device=gpu), torch.empty((na, ci), dtype=torch.float32, device=gpu)
    t = lambda a: torch.from_numpy(a).to(gpu)
    tlq.scale_search(dev(X, gpu, bf16), dev(W, gpu, bf16), Y, t(w), t(al), p, best, idx, losses, s_table_out=table)
    ref = orc.scale_search(X, W, Y.double().cpu().numpy(), w, 4, 0 if act else 8, al, s_table=table.cpu().numpy(),
                           symmetric=True, act_bits=act)
    np.testing.assert_allclose(losses.cpu().numpy(), ref["losses"], rtol=1e-3)   # the parity bar of the search


@pytest.mark.parametrize("n,co,bf16", [(2500, 4104, True), (2496, 4096, False), (4700, 4104, False), (4800, 4096, True)])
@pytest.mark.parametrize("ci", [72, 128])      # with and without a k tail
def test_stores_and_token_errors_of_narrow_and_wide_tiles(gpu, n, co, bf16, ci):
    import torch
    g = np.random.default_rng([42, n, co])
    rnd = BF if bf16 else F16
    X, W = rnd(g.standard_normal((n, ci))), rnd(g.standard_normal((co, ci)) * 0.05)
    code, dt = (tlq.BF16, torch.bfloat16) if bf16 else (tlq.F16, torch.float16)
    tX, tW = dev(X, gpu, bf16), dev(W, gpu, bf16)
    want = tX.double() @ tW.double().t()
    mag = tX.double().abs() @ tW.double().abs().t()
    for ydt, ycode, eps in ((torch.float32, tlq.F32, 0.0), (dt, code, 2.0 ** -8 if bf16 else 2.0 ** -11)):
        Y = torch.full((n, co + 8), 7.0, dtype=ydt, device=gpu)
        tlq.ref_output(tX, tW, Y[:, :co], tlq.params(x_dtype=code, yref_dtype=ycode))
        assert bool((Y[:, co:] == 7.0).all())
        # ci roundings of at most 2^-24 of the magnitude, then one to the type of the output (subnormal steps of fp16)
        bound = (ci + 2) * 2.0 ** -24 * mag + eps * want.abs() + 2.0 ** -25
        assert bool(((Y[:, :co].double() - want).abs() <= bound).all())
    target = (want + torch.randn(want.shape, generator=torch.Generator(device=gpu).manual_seed(1), device=gpu)).to(dt)
    s = np.exp2(g.integers(-2, 3, ci)).astype(np.float32)          # powers of two: folding them in is exact
    w = torch.from_numpy(g.uniform(0.1, 1.0, n).astype(np.float32) / n).to(gpu)
    loss, err = torch.empty(1, dtype=torch.float32, device=gpu), torch.empty(n, dtype=torch.float32, device=gpu)
    tlq.weighted_layer_err(tX, tW, torch.from_numpy(s).to(gpu), target, w, tlq.params(x_dtype=code, yref_dtype=code), loss,
                           per_token_err=err)
    e = ((target.double() - (tX.double() * torch.from_numpy(s).to(gpu).double()) @ tW.double().t()) ** 2).mean(1)
    np.testing.assert_allclose(err.cpu().numpy(), e.cpu().numpy(), rtol=2e-5)      # float sums of positive terms
    np.testing.assert_allclose(float(loss.item()), float((e * w.double()).sum()), rtol=2e-5)


# outputs on both sides of half a tile (128), of a quad (4) and of the first quad; tokens in one and in several waves and
# tiles, square and wide ones
@pytest.mark.parametrize("co", [1, 3, 4, 66, 124, 128, 129, 380, 386])
@pytest.mark.parametrize("n,kind", [(1, "f16"), (130, "f32"), (700, "f16"), (700, "bf16"), (33000, "f16"), (33000, "f32")])
def test_losses_where_half_a_tile_lies_past_the_edge(gpu, n, co, kind):
    import torch
    g = torch.Generator(device=gpu).manual_seed(n * 512 + co)
    ci = 64
    dt, act = {"f16": torch.float16, "f32": torch.float32, "bf16": torch.bfloat16}[kind], torch.bfloat16 if kind == "bf16" else torch.float16
    X = torch.randn((n, ci), generator=g, device=gpu).to(act)
    W = (torch.randn((co, ci), generator=g, device=gpu) * 0.05).to(act)
    prod = X.double() @ W.double().t()
    Y = torch.full((n, co + -co % 8 + 8), float("nan"), dtype=dt, device=gpu)     # what lies beside the target is not used
    Y[:, :co] = (prod + torch.randn(prod.shape, generator=g, device=gpu)).to(dt)
    w = torch.rand(n, generator=g, device=gpu) / n
    p = tlq.params(group=8, x_dtype=tlq.BF16 if kind == "bf16" else tlq.F16, yref_dtype={"f16": tlq.F16, "f32": tlq.F32, "bf16": tlq.BF16}[kind])
    e = ((Y[:, :co].double() - prod) ** 2).mean(1)
    want = float((e * w.double()).sum())
    for tok in (False, True):
        loss, err = torch.empty(1, device=gpu), torch.empty(n, device=gpu) if tok else None
        tlq.weighted_layer_err(X, W, None, Y[:, :co], w, p, loss, per_token_err=err)
        # products of 64 terms are off by 64 roundings of 2^-24 of a magnitude of about three residuals, the sums of
        # positive terms by a few more: below 2e-5
        np.testing.assert_allclose(float(loss), want, rtol=2e-5)
        if tok:
            # one output: a residual near zero keeps the absolute error of its product
            np.testing.assert_allclose(err.cpu().numpy(), e.cpu().numpy(), rtol=2e-5, atol=2e-6)


@pytest.mark.parametrize("n,co,na", [(40, 72, 1), (40, 72, 17), (300, 600, 64), (2100, 1300, 33)])
def test_selection_of_few_and_many_partial_sums(gpu, n, co, na):
    """Up to 64 partial sums a candidate are read for eight candidates at a time, more one candidate after the other; equal
    losses select the first of them; the errors of the tokens come from the launch that combines the loss."""
    import torch
    g = np.random.default_rng([27, n, na])
    ci = 64
    X, W = F16(g.standard_normal((n, ci))), F16(g.standard_normal((co, ci)) * 0.05)
    Y = orc.ref_output(X, W).astype(np.float32)
    al = np.repeat(g.uniform(0.0, 1.0, (na + 1) // 2), 2)[:na].astype(np.float32)       # every strength twice
    w = np.full(n, 1.0 / n, np.float32)
    p = tlq.params(bits=4, group=32, x_dtype=tlq.F16, yref_dtype=tlq.F32)
    tX, tW, tY, tw = dev(X, gpu, False), dev(W, gpu, False), torch.from_numpy(Y).to(gpu), torch.from_numpy(w).to(gpu)
    best, idx = torch.empty(ci, dtype=torch.float32, device=gpu), torch.empty(1, dtype=torch.int32, device=gpu)
    losses, table = (torch.empty(s, dtype=torch.float32, device=gpu) for s in ((na,), (na, ci)))
    tlq.scale_search(tX, tW, tY, tw, torch.from_numpy(al).to(gpu), p, best, idx, losses, s_table_out=table)
    got = host(losses)
    assert int(idx) == int(np.argmin(got)) and int(idx) % 2 == 0
    assert np.array_equal(got[0:na - na % 2:2], got[1::2]) and torch.equal(best, table[int(idx)])
    loss, err = torch.empty(1, dtype=torch.float32, device=gpu), torch.empty(n, dtype=torch.float32, device=gpu)
    Wq = F16(W + g.standard_normal(W.shape) * 0.01)
    tlq.weighted_layer_err(tX, dev(Wq, gpu, False), None, tY, tw, p, loss, per_token_err=err)
    ref = ((Y.astype(np.float64) - X.astype(np.float64) @ Wq.astype(np.float64).T) ** 2).mean(1)
    # squares are added in 32 bits inside a tile: at most 320 in a chain, so 320 x 2^-24, and the products' own rounding
    np.testing.assert_allclose(host(err), ref, rtol=1e-4, atol=1e-9)
    assert abs(float(loss) - ref.mean()) <= 1e-4 * ref.mean()


@pytest.mark.parametrize("n,ci,co", [(1, 8, 1), (129, 72, 127), (256, 320, 128), (511, 1096, 385), (1100, 136, 2000), (1152, 128, 2048),
                                      (2100, 200, 2100), (2048, 192, 2176)])
@pytest.mark.parametrize("bf16,float_target", [(False, False), (False, True), (True, False)])
def test_token_errors_in_small_tiles(gpu, n, ci, co, bf16, float_target):
    """Losses with token errors in tiles of 128 x 64 (up to 256 of them) and 128 x 128 (up to 512): two and four k-tiles in
    flight (more than 256 tiles and up to there), contractions that end inside a k-tile, tiles inside the matrix and at its edges."""
    import torch
    g = np.random.default_rng([28, n, ci])
    rnd = BF if bf16 else F16
    X, Wq = (np.asarray(rnd(g.standard_normal(s) * f), np.float64) for s, f in (((n, ci), 1.0), ((co, ci), 0.05)))
    Y = X @ (Wq + g.standard_normal((co, ci)) * 0.01).T
    tY = torch.zeros((n, co + -co % 8), dtype=torch.float32 if float_target else torch.bfloat16 if bf16 else torch.float16, device=gpu)[:, :co]
    tY.copy_(torch.from_numpy(Y))
    w = g.uniform(0.0, 2.0 / n, n).astype(np.float32)
    p = tlq.params(bits=4, group=8, x_dtype=tlq.BF16 if bf16 else tlq.F16, yref_dtype=tlq.F32 if float_target else tlq.BF16 if bf16 else tlq.F16)
    loss, err = torch.empty(1, dtype=torch.float32, device=gpu), torch.empty(n, dtype=torch.float32, device=gpu)
    inv = torch.ones(ci, dtype=torch.float32, device=gpu)
    tlq.weighted_layer_err(dev(X, gpu, bf16), dev(Wq, gpu, bf16), inv, tY, torch.from_numpy(w).to(gpu), p, loss, per_token_err=err)
    ref = ((host(tY).astype(np.float64) - X @ Wq.T) ** 2).mean(1)
    # (ci <= 1096 products in 32 bits, of sums about 20 times the residual; 64 squares in a chain)
    np.testing.assert_allclose(host(err), ref, rtol=2e-3, atol=1e-12)
    np.testing.assert_allclose(float(loss), (w.astype(np.float64) * ref).sum(), rtol=1e-3)
    alone = torch.empty_like(loss)
    tlq.weighted_layer_err(dev(X, gpu, bf16), dev(Wq, gpu, bf16), inv, tY, torch.from_numpy(w).to(gpu), p, alone)
    np.testing.assert_allclose(float(alone), float(loss), rtol=1e-5)


def _layer_err_room(n, ci, co, bf16):
    """Bytes of a workspace of tlq_weighted_layer_err for tiles of 256 x 256: partial sums, token sums, folded weights, a word,
    tokens in fp16, each in whole units of 256 bytes."""
    to, tt = -(-co // 256), -(-n // 256)
    return sum(-(-b // 256) * 256 for b in (4 * to * tt, 4 * to * n, 2 * co * ci, 4, 2 * n * ci if bf16 else 0))


@pytest.mark.parametrize("n,ci,co,bf16", [(1, 8, 1, True), (129, 72, 1000, False), (1948, 32, 10145, True), (1100, 136, 2000, False)])
def test_layer_error_with_the_room_of_big_tiles(gpu, n, ci, co, bf16):
    """A workspace that holds the sums of 256 x 256 tiles only, less than the query asks for where smaller ones are
    faster, is enough, and nothing behind it is written."""
    import torch
    g = np.random.default_rng([35, n, ci])
    rnd = BF if bf16 else F16
    X, Wq = (np.asarray(rnd(g.standard_normal(s) * f), np.float64) for s, f in (((n, ci), 1.0), ((co, ci), 0.05)))
    dt, code = (torch.bfloat16, tlq.BF16) if bf16 else (torch.float16, tlq.F16)
    tY = torch.zeros((n, co + -co % 8), dtype=dt, device=gpu)[:, :co]
    tY.copy_(torch.from_numpy(X @ (Wq + g.standard_normal((co, ci)) * 0.01).T))
    w = torch.from_numpy(g.uniform(0.0, 2.0 / n, n).astype(np.float32)).to(gpu)
    p = tlq.params(bits=4, group=8, x_dtype=code, yref_dtype=code)
    inv = torch.ones(ci, dtype=torch.float32, device=gpu)
    room = _layer_err_room(n, ci, co, bf16)
    assert room <= tlq.weighted_layer_err_workspace_bytes(n, ci, co, p)
    buf = torch.full((room + 4096,), 0xA5, dtype=torch.uint8, device=gpu)
    got = []
    for ws in (None, buf[:room]):
        loss, err = torch.empty(1, dtype=torch.float32, device=gpu), torch.empty(n, dtype=torch.float32, device=gpu)
        tlq.weighted_layer_err(dev(X, gpu, bf16), dev(Wq, gpu, bf16), inv, tY, w, p, loss, per_token_err=err, workspace=ws)
        got.append((float(loss), host(err)))
    assert torch.all(buf[room:] == 0xA5)
    # the same products; squares are added in another order, at most 320 in a chain of 32 bits
    np.testing.assert_allclose(got[1][1], got[0][1], rtol=320 * 2.0 ** -24, atol=1e-12)
    np.testing.assert_allclose(got[1][0], got[0][0], rtol=320 * 2.0 ** -24)
    with pytest.raises(tlq.TlqError) as e:
        tlq.weighted_layer_err(dev(X, gpu, bf16), dev(Wq, gpu, bf16), inv, tY, w, p, loss, workspace=buf[:room - 1])
    assert e.value.status == tlq.ERR_WORKSPACE


@pytest.mark.parametrize("n,ci,co", [(1, 8, 8), (63, 72, 128), (64, 64, 136), (65, 320, 248), (128, 128, 384), (1000, 1096, 2000), (64, 200, 16384)])
@pytest.mark.parametrize("bf16,float_out", [(False, False), (False, True), (True, False)])
def test_products_in_tiles_of_one_a_unit(gpu, n, ci, co, bf16, float_out):
    """Stores in tiles of 128 x 64 (up to 256 of them): one k-tile and several, ends inside a k-tile, a ring, a tile."""
    import torch
    g = np.random.default_rng([29, n, ci])
    rnd = BF if bf16 else F16
    X, W = (np.asarray(rnd(g.standard_normal(s)), np.float64) for s in ((n, ci), (co, ci)))
    dt = torch.float32 if float_out else torch.bfloat16 if bf16 else torch.float16
    p = tlq.params(bits=4, group=8, x_dtype=tlq.BF16 if bf16 else tlq.F16, yref_dtype=tlq.F32 if float_out else tlq.BF16 if bf16 else tlq.F16)
    Y = torch.full((n, co + 8), 7.0, dtype=dt, device=gpu)
    tlq.ref_output(dev(X, gpu, bf16), dev(W, gpu, bf16), Y[:, :co], p)
    want, mag = X @ W.T, np.abs(X) @ np.abs(W).T
    eps = 0.0 if float_out else 2.0 ** -8 if bf16 else 2.0 ** -11     # the output's rounding, and ci additions in 32 bits
    assert np.all(np.abs(host(Y[:, :co]) - want) <= eps * np.abs(want) + ci * 2.0 ** -24 * mag)
    assert torch.all(Y[:, co:] == 7.0)


@pytest.mark.parametrize("n,ci", [(40, 8), (300, 136), (700, 264), (9000, 392), (45000, 264), (600, 4096)])
def test_token_product_in_small_tiles(gpu, n, ci):
    """The triangle of the token product in tiles of 128 x 128 (up to 512 of them; 4096 channels have 528 and big tiles), in
    one, two and ten parts of the tokens: the matrix is symmetric to the bit, whichever side of the diagonal a block of it
    came from.  The weights' square roots are exact, and so are the weighted tokens in 16 bits."""
    import torch
    g = np.random.default_rng([30, n, ci])
    X, w = F16(g.standard_normal((n, ci))), g.choice([1.0, 0.25], n).astype(np.float32)
    w[0] = 1.0
    gram = torch.zeros(tlq.token_gram_bytes(ci), dtype=torch.uint8, device=gpu)
    tX, tw = dev(X, gpu, False), torch.from_numpy(w).to(gpu)
    tlq.token_gram(tX, tw, tlq.params(), gram)
    C = gram[256 + -(-4 * ci // 256) * 256:][:2 * ci * ci].view(torch.float16).view(ci, ci)
    assert torch.equal(C, C.t())
    Xs = (tX.float() * tw.sqrt()[:, None]).half().double()
    Xt = Xs.t().contiguous()
    G, mag = host64(Xt @ Xs), host64(Xt.abs() @ Xs.abs())
    e = np.rint(np.log2(np.diag(G)) / 2)
    unit = 2.0 ** -(e[:, None] + e[None, :])
    # one rounding to 16 bits; in 32 bits 32 products to an accumulator at a time, and up to 16 parts
    assert np.all(np.abs(host64(C) - G * unit) <= 2.0 ** -11 * np.abs(G) * unit + 2.0 ** -25 + (n / 32 + 32 + 16) * 2.0 ** -24 * mag * unit)


@pytest.mark.parametrize("n,c", [(16389, 8), (16500, 520), (33001, 2056), (30000, 5128)])
@pytest.mark.parametrize("bf16,masked", [(False, False), (True, False), (True, True)])
def test_statistic_of_long_chunks(gpu, n, c, bf16, masked):
    """Chunks of more than 128 rows in blocks of 16 waves (up to 2048 channels, 5120 without a mask) and of 4: rows in fours
    and the rest of a chunk, rows apart from each other."""
    import torch
    gen = torch.Generator(device=gpu)
    gen.manual_seed(31 + n)
    X = torch.randn((n, c + 8), generator=gen, device=gpu).to(torch.bfloat16 if bf16 else torch.float16)[:, :c]
    p = tlq.params(x_dtype=tlq.BF16 if bf16 else tlq.F16)
    out = torch.empty(c, dtype=torch.float32, device=gpu)
    if masked:
        mask = (torch.rand(n, generator=gen, device=gpu) < 0.3).to(torch.uint8)
        tlq.x_stat_masked(X, mask, p, out)
        want = X[mask.bool()].abs().amax(0).float()
        assert torch.equal(out, want)
    else:
        tlq.x_stat(X, p, out)
        want = torch.stack([part.double().abs().sum(0) for part in X.split(4096)]).sum(0) / n
        # sums in 64 bits on both sides, one rounding to 32
        assert torch.all((out.double() - want).abs() <= want * (2.0 ** -24 + 1e-12))
