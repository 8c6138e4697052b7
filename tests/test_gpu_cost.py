"""Calls whose cost must not hang on the shape that a kernel was written for: the same work in another shape may
cost a stated multiple, far from what the dispatch rules give and far from what missing them costs."""
import statistics

import pytest

from paper_2602_07899_amd import tlq

pytestmark = pytest.mark.gpu


def micros(*fns, reps=10, rounds=7):
    """Median time of each call in microseconds, the calls in turn."""
    import torch
    for f in fns:
        f()
    torch.cuda.synchronize()
    times = [[] for _ in fns]
    for _ in range(rounds):
        for f, t in zip(fns, times):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(reps):
                f()
            b.record()
            b.synchronize()
            t.append(a.elapsed_time(b) * 1e3 / reps)
    return [statistics.median(t) for t in times]


def test_attention_of_one_head_uses_the_whole_chip(gpu):
    """One (sample, head) pair of 32768 tokens is an eighth of eight pairs: 0.3 of their time when its query
    blocks run on all XCDs, 0.8 on one."""
    import torch
    seq, heads = 32768, 8
    qkv = torch.randn((seq, 3 * heads * 128), device=gpu).to(torch.bfloat16)
    out = torch.empty((seq, heads * 128), dtype=torch.bfloat16, device=gpu)
    p = tlq.params(x_dtype=tlq.BF16)

    def run(h):
        d = h * 128
        return lambda: tlq.causal_attention(qkv[:, :d], qkv[:, d:2 * d], qkv[:, 2 * d:3 * d], h, seq, p, out)
    one, eight = micros(run(1), run(8), reps=3)
    assert one < 0.65 * eight, (one, eight)


def test_token_preparation_of_few_long_rows(gpu):
    """One megabyte of tokens in 4 rows or in 128: 1.0 times the cost when long rows are split, 3.4 when a wave
    walks a row alone."""
    import torch
    p = tlq.params(group=8, x_dtype=tlq.BF16)
    X = torch.randn((4, 131072), device=gpu).to(torch.bfloat16)
    buf = torch.zeros(tlq.prepared_tokens_bytes(4, 131072, p), dtype=torch.uint8, device=gpu)
    few, many = micros(lambda: tlq.prepare_tokens(X, p, buf), lambda: tlq.prepare_tokens(X.view(128, 4096), p, buf), reps=30)
    assert few < 2.0 * many, (few, many)


def test_statistic_of_few_long_rows(gpu):
    """Rows of 262,144 channels or sixteen times as many of 16,384: twice the cost in two launches, five times where every 64
    channels have a block of their own."""
    import torch
    X = torch.randn((64, 262144), device=gpu).to(torch.float16)
    p = tlq.params(xstat_kind=1)
    out = torch.empty(262144, dtype=torch.float32, device=gpu)
    ws = torch.empty(tlq.x_stat_workspace_bytes(64, 262144), dtype=torch.uint8, device=gpu)
    few, many = micros(lambda: tlq.x_stat(X, p, out, workspace=ws),
                       lambda: tlq.x_stat(X.view(1024, 16384), p, out[:16384], workspace=ws), reps=30)
    assert few < 3.0 * many, (few, many)


def test_maximum_of_short_chunks(gpu):
    """The maximum of 3000 x 32,768 tokens takes as long as their mean with a row a wave at a time, 1.17 times that with four."""
    import torch
    X = torch.randn((3000, 32768), device=gpu).to(torch.float16)
    out = torch.empty(32768, dtype=torch.float32, device=gpu)
    ws = torch.empty(tlq.x_stat_workspace_bytes(3000, 32768), dtype=torch.uint8, device=gpu)
    run = lambda kind: lambda p=tlq.params(xstat_kind=kind): tlq.x_stat(X, p, out, workspace=ws)
    largest, mean = micros(run(1), run(0), reps=30)
    assert largest < 1.08 * mean, (largest, mean)


def test_search_of_few_tokens_prepares_them_in_time(gpu):
    """A search over 1024 tokens of 256 channels, half a megabyte, in bf16 and in fp16, which needs no preparation: 1.17 times the
    cost when the tokens are prepared beside the statistic, 1.27 with a launch that reads them all in every block."""
    import torch
    n, ci, co, na = 1024, 256, 264, 20
    w, al = torch.full((n,), 1e-3, device=gpu), torch.arange(na, device=gpu) / na
    best, idx = torch.empty(ci, device=gpu), torch.empty(1, dtype=torch.int32, device=gpu)
    losses = torch.empty(na, device=gpu)

    def captured(dt, code):
        p = tlq.params(bits=4, group=0, symmetric=1, x_dtype=code, yref_dtype=code)
        X, W = torch.randn((n, ci), device=gpu).to(dt), (torch.randn((co, ci), device=gpu) * 0.02).to(dt)
        Y = torch.empty((n, co), dtype=dt, device=gpu)
        tlq.ref_output(X, W, Y, p)
        ws = torch.empty(tlq.scale_search_workspace_bytes(n, ci, co, na, p), dtype=torch.uint8, device=gpu)
        run = lambda: tlq.scale_search(X, W, Y, w, al, p, best, idx, losses, workspace=ws)
        run()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(20):
                run()
        return graph, run          # (which keeps the buffers)
    graphs = captured(torch.bfloat16, tlq.BF16), captured(torch.float16, tlq.F16)
    prepared, plain = micros(*(g.replay for g, _ in graphs))
    assert prepared < 1.22 * plain, (prepared / 20, plain / 20)


def shifted(x):
    """A copy of x that starts one element off the 16-byte alignment of the wide paths."""
    import torch
    out = torch.empty(x.numel() + 8, dtype=x.dtype, device=x.device)[1:1 + x.numel()].view(x.shape)
    return out.copy_(x)


def test_norms_of_narrow_gradient_rows(gpu):
    """Rows of 8 channels take the element-wise form whatever their alignment: 1.0 times the cost of misaligned
    ones, 1.6 where alignment alone picked the form."""
    import torch
    n_pos = 65536
    G = torch.randn((16 * n_pos, 8), device=gpu).to(torch.float16)
    Gs, p = shifted(G), tlq.params()
    s = torch.empty(n_pos, dtype=torch.float64, device=gpu)
    ws = torch.empty(16 * n_pos * 8, dtype=torch.uint8, device=gpu)
    wide, narrow = micros(lambda: tlq.token_importance(G, 16, p, s, workspace=ws),
                          lambda: tlq.token_importance(Gs, 16, p, s, workspace=ws))
    assert wide < 1.25 * narrow, (wide, narrow)


def test_position_sums_of_one_sample(gpu):
    """As many rows in one sample or in 64 (both are mostly the row norms): 1.0 times the cost when one sample is
    added without staging, 1.2 with it."""
    import torch
    n = 1 << 22
    G = torch.randn((n, 8), device=gpu).to(torch.float16)
    p = tlq.params()
    s = torch.empty(n, dtype=torch.float64, device=gpu)
    ws = torch.empty(n * 8, dtype=torch.uint8, device=gpu)
    one, many = micros(lambda: tlq.token_importance(G, 1, p, s, workspace=ws),
                       lambda: tlq.token_importance(G, 64, p, s[:n // 64], workspace=ws), reps=5)
    assert one < 1.1 * many, (one, many)


def test_normalisation_of_narrow_rows(gpu):
    """Rows of 8 channels take the element-wise form whatever their alignment: 1.0 times the cost of misaligned
    ones, 1.3 where alignment alone picked the form."""
    import torch
    Z = torch.randn((1000000, 8), device=gpu).to(torch.float16)
    Zs, p = shifted(Z), tlq.params()
    out, outs, m = torch.empty_like(Z), shifted(Z), torch.rand(8, device=gpu)
    wide, narrow = micros(lambda: tlq.rmsnorm_mul(Z, p, out, m_a=m), lambda: tlq.rmsnorm_mul(Zs, p, outs, m_a=m))
    assert wide < 1.15 * narrow, (wide, narrow)


def test_quantiser_groups_of_24_channels(gpu):
    """The same weights in groups of 24 or of 32 channels: 1.2 times the cost with whole groups packed into a wave,
    13 with a wave to every group."""
    import torch
    co, ci = 4096, 4128
    W, s = torch.randn((co, ci), device=gpu).to(torch.float16), torch.rand(ci, device=gpu) + 0.5
    codes, wdq = torch.empty((co, ci), dtype=torch.uint8, device=gpu), torch.empty_like(W)

    def run(group):
        zp, delta = torch.empty((co, ci // group), dtype=torch.uint8, device=gpu), torch.empty((co, ci // group), device=gpu)
        p = tlq.params(group=group)
        return lambda: tlq.fake_quant(W, s, p, codes, zp, delta, wdq)
    odd, even = micros(run(24), run(32))
    assert odd < 4.0 * even, (odd, even)


def test_ragged_edge_of_a_one_round_product(gpu):
    """252 tiles, one a CU: with outputs that end inside a tile the last column's guarded store is on the
    critical path: 1.08 times the cost of whole tiles, 1.3 while that store carried the subtraction of the
    difference form."""
    import torch
    n, ci = 7168, 256
    X, W = torch.randn((n, ci), device=gpu).to(torch.float16), torch.randn((2304, ci), device=gpu).to(torch.float16)
    p = tlq.params()
    Y, Z = (torch.empty((n, co), dtype=torch.float16, device=gpu) for co in (2304, 2216))
    whole, ragged = micros(lambda: tlq.ref_output(X, W, Y, p), lambda: tlq.ref_output(X, W[:2216], Z, p), reps=50)
    assert ragged < 1.18 * whole, (ragged, whole)


def test_loss_of_few_outputs(gpu):
    """64 outputs in tiles of 256: 0.73 times the cost of 256 outputs when the rows past the edge are left out, 1.11
    when their target is read for nothing."""
    import torch
    n, ci = 100000, 64
    X, W = torch.randn((n, ci), device=gpu).to(torch.float16), torch.randn((256, ci), device=gpu).to(torch.float16)
    w, loss = torch.full((n,), 1.0 / n, device=gpu), torch.empty(1, device=gpu)
    p = tlq.params(group=8)

    def run(co):
        Y = torch.zeros((n, co), dtype=torch.float16, device=gpu)
        ws = torch.empty(tlq.weighted_layer_err_workspace_bytes(n, ci, co, p), dtype=torch.uint8, device=gpu)
        return lambda: tlq.weighted_layer_err(X, W[:co], None, Y, w, p, loss, workspace=ws)
    few, whole = micros(run(64), run(256), reps=50)
    assert few < 0.9 * whole, (few, whole)


def test_search_whose_last_patches_are_short(gpu):
    """20 candidates over 8192 and over 10,240 tokens: 0.84 times the cost when the tile is chosen by the busiest XCD's
    work, 0.95 with wide tiles, whose 26 columns leave the short patches of every candidate to the same two XCDs."""
    import torch
    ci, co, na = 4096, 1024, 20
    X, W = torch.randn((10240, ci), device=gpu).to(torch.float16), (torch.randn((co, ci), device=gpu) * 0.02).to(torch.float16)
    p, al = tlq.params(), torch.tensor([k / na for k in range(na)], device=gpu)
    best, idx, losses = torch.empty(ci, device=gpu), torch.empty(1, dtype=torch.int32, device=gpu), torch.empty(na, device=gpu)
    Y = torch.empty((10240, co), dtype=torch.float16, device=gpu)
    tlq.ref_output(X, W, Y, p)
    ws = torch.empty(tlq.scale_search_workspace_bytes(10240, ci, co, na, p), dtype=torch.uint8, device=gpu)

    def run(n):
        w = torch.full((n,), 1.0 / n, device=gpu)
        return lambda: tlq.scale_search(X[:n], W, Y[:n], w, al, p, best, idx, losses, workspace=ws)
    few, more = micros(run(8192), run(10240))
    assert few < 0.9 * more, (few, more)


def test_gate_and_the_product_behind_it(gpu):
    """An output of 113 MB that the next call reads, from inputs that do not fit the last-level cache beside it: 1.35 times
    the cost of 90 MB when only the inputs go past the cache, 1.9 when the output does too."""
    import torch
    c, co = 11008, 1024
    G, U = (torch.randn((5120, c), device=gpu).to(torch.bfloat16) for _ in range(2))
    M, W = torch.empty_like(G), (torch.randn((co, c), device=gpu) * 0.02).to(torch.bfloat16)
    Y, p = torch.empty((5120, co), dtype=torch.bfloat16, device=gpu), tlq.params(x_dtype=tlq.BF16, yref_dtype=tlq.BF16)

    def run(n):
        def calls():
            tlq.silu_mul(G[:n], U[:n], p, M[:n])
            tlq.ref_output(M[:n], W, Y[:n], p)
        return calls
    more, less = micros(run(5120), run(4096))
    assert more < 1.6 * less, (more, less)


def test_difference_form_of_few_channels(gpu):
    """The product that leaves the differences of 5000 x 128 x 13824 as floats: 0.89 times the contraction of two candidates
    with them, 1.11 in 320-token tiles."""
    import torch
    n, ci, co, na = 5000, 128, 13824, 2
    X, W = torch.randn((n, ci), device=gpu).to(torch.bfloat16), (torch.randn((co, ci), device=gpu) * 0.02).to(torch.bfloat16)
    Y, w, al = torch.empty((n, co), dtype=torch.bfloat16, device=gpu), torch.full((n,), 1.0 / n, device=gpu), torch.tensor([0.0, 0.5], device=gpu)
    best, idx, losses = torch.empty(ci, device=gpu), torch.empty(1, dtype=torch.int32, device=gpu), torch.empty(na, device=gpu)
    p = tlq.params(bits=8, group=0, symmetric=1, x_dtype=tlq.BF16, yref_dtype=tlq.BF16)
    tlq.ref_output(X, W, Y, p)
    ws = torch.empty(tlq.scale_search_workspace_bytes(n, ci, co, na, p), dtype=torch.uint8, device=gpu)
    run = lambda: tlq.scale_search(X, W, Y, w, al, p, best, idx, losses, workspace=ws)
    run()
    torch.cuda.synchronize()
    tlq.profile_enable(True)
    try:
        tlq.profile_reset()
        for _ in range(20):
            run()
        ms = {k.name: k.total_ms for k in tlq.profile_read()}
    finally:
        tlq.profile_enable(False)
    assert ms["gemm_store"] < ms["gemm_loss"], ms


def test_token_errors_beside_the_loss(gpu):
    """The loss of 14,000 x 64 x 6144 with the token errors: 1.09 times its cost without, 1.5 when the target is read in the
    layout of the accumulators for them."""
    import torch
    n, ci, co = 14000, 64, 6144
    X, W = torch.randn((n, ci), device=gpu).to(torch.float16), (torch.randn((co, ci), device=gpu) * 0.05).to(torch.float16)
    Y, w, p = torch.zeros((n, co), dtype=torch.float16, device=gpu), torch.full((n,), 1.0 / n, device=gpu), tlq.params(group=8)
    loss, err = torch.empty(1, device=gpu), torch.empty(n, device=gpu)
    ws = torch.empty(tlq.weighted_layer_err_workspace_bytes(n, ci, co, p), dtype=torch.uint8, device=gpu)
    both, alone = micros(lambda: tlq.weighted_layer_err(X, W, None, Y, w, p, loss, per_token_err=err, workspace=ws),
                         lambda: tlq.weighted_layer_err(X, W, None, Y, w, p, loss, workspace=ws), reps=30)
    assert both < 1.28 * alone, (both, alone)
