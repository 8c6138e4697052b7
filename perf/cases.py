"""The work whose speed is watched: calls that a calibration program makes, through the public
entry points (`paper_2602_07899_amd.tlq`, `paper_2602_07899_amd.stack`).

A case is one dict of plain values; `kind` names the entry points it goes through:

  search     one scale search in the token form: `scale_search` (statistic, scale table, fake
             quantisation of every candidate, contraction with the weighted loss, selection),
             weight-only or with per-token activation quantisation (`act` bits)
  gram       the second-moment form for linears that share one input: `x_stat`, `token_gram`, then
             `scale_search_gram` once per linear
  export     what follows a search for one linear: `fake_quant` with every output (the integer
             codes that are stored, zero points, steps, dequantised weights) and
             `weighted_layer_err` of those weights with the per-token errors
  propagate  one linear's full-precision target and its quantised output: `ref_output`, `apply_best`
  attention  causal attention of a decoder block, q/k/v as column slices of one matrix
  glue       the element-wise steps of a decoder block: `rmsnorm_mul`, `silu_mul`, `residual_add`
  select     the gradient-guided statistic: `token_importance`, `topk_mask`, `x_stat_masked`, beside
             the plain mean `x_stat`
  stack      `run_stack`: whole decoder blocks calibrated in sequence
"""
from __future__ import annotations

import math

import torch

from paper_2602_07899_amd import stack as gstack
from paper_2602_07899_amd import tlq

_DT = {"f16": (torch.float16, tlq.F16), "bf16": (torch.bfloat16, tlq.BF16)}
_MAX_FLOPS = 1.6e14      # no drawn search costs more than the largest listed one


def listed():
    return [
        # the smallest layer configuration of the repository (one 512 x 512 linear, 256 tokens): what
        # a test or a first try of the library runs; latency and launches count
        dict(name="search_small", kind="search", n=256, ci=512, co=512, seq=256, vis=192, bits=4, group=128,
             sym=0, act=0, dt="f16", na=20),
        # attention linear of a 7B-class decoder layer, 16 samples x 640 tokens, W4 g128: the ordinary search
        dict(name="search_7b", kind="search", n=10240, ci=4096, co=4096, seq=640, vis=576, bits=4, group=128,
             sym=0, act=0, dt="f16", na=20),
        # attention linear of a 13B-class layer with the full 128 x 1200 calibration tokens: the largest
        dict(name="search_13b", kind="search", n=153600, ci=5120, co=5120, seq=1200, vis=1152, bits=4, group=128,
             sym=0, act=0, dt="f16", na=20),
        # the method's own setting: per-channel symmetric weights, activations quantised per token, bf16,
        # a few samples with a ragged token count
        dict(name="search_w4a8", kind="search", n=3678, ci=4096, co=4096, seq=613, vis=576, bits=4, group=0,
             sym=1, act=8, dt="bf16", na=20),
        # eight bits per channel, a width that is no multiple of the tile depth, an odd number of tokens
        dict(name="search_ragged_w8", kind="search", n=1839, ci=1096, co=1400, seq=613, vis=576, bits=8, group=0,
             sym=1, act=0, dt="bf16", na=12),
        # q/k/v of a 13B-class layer in the second-moment form: one matrix, three searches
        dict(name="gram_13b_qkv", kind="gram", n=153600, ci=5120, co=5120, linears=3, seq=1200, vis=1152,
             bits=4, group=128, sym=0, dt="bf16", na=20),
        # storing a searched 7B-class down_proj and measuring it token by token
        dict(name="export_7b_down", kind="export", n=10240, ci=11008, co=4096, seq=640, vis=576, bits=4, group=128,
             sym=0, dt="f16"),
        # one sample of 1200 tokens through a 13B-class gate_proj, full precision and quantised
        dict(name="propagate_sample", kind="propagate", n=1200, ci=5120, co=13824, seq=1200, vis=1152, bits=4,
             group=128, sym=0, act=0, dt="bf16"),
        # attention of a 13B-class block over all 128 samples
        dict(name="attention_13b", kind="attention", samples=128, seq=1200, heads=40, dt="bf16"),
        # normalisation, gate and residual of a 7B-class block, 64 x 640 tokens
        dict(name="glue_7b", kind="glue", n=40960, c=4096, ffn=11008, dt="bf16"),
        # gradient-guided selection and both statistics, 128 samples x 1200 positions, 13B-class width
        dict(name="select_13b", kind="select", samples=128, seq=1200, vis=1152, c=5120, l2=0, dt="bf16"),
        # a whole calibration call: two small decoder blocks, quantisation-exposed propagation; many
        # short launches
        dict(name="stack_mini", kind="stack", layers=2, heads=2, ffn=384, samples=3, seq=72, vis=48, bits=4,
             group=128, na=6, mode="passact2", strategy="tokens", dt="bf16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi, group):
    unit = group if group else 8
    return max(unit, _log(rng, lo, hi) // unit * unit)


def draw(rng):
    kind = rng.choice(["search", "search", "search", "gram", "export", "propagate", "attention", "glue", "select",
                       "stack"])
    dt = rng.choice(["f16", "bf16"])
    group = rng.choice([128, 128, 128, 64, 32, 0])
    sym = 1 if group == 0 or rng.random() < 0.2 else 0
    seq = rng.randint(64, 1300)
    vis = seq * rng.randint(50, 96) // 100
    quant = dict(bits=rng.choice([3, 4, 4, 8]), group=group, sym=sym, dt=dt)
    if kind == "search":
        while True:
            n, ci, co = _log(rng, 128, 60000), _width(rng, 256, 13824, group), _log(rng, 256, 13824)
            na = rng.randint(6, 20)
            if 2.0 * n * ci * co * na <= _MAX_FLOPS:
                break
        return dict(kind=kind, n=n, ci=ci, co=co, seq=seq, vis=vis, act=rng.choice([0, 0, 0, 8, 6]), na=na, **quant)
    if kind == "gram":
        # the form is for many tokens per channel; its losses average over them
        ci = _width(rng, 512, 6144, group)
        n = _log(rng, max(4096, 2 * ci), 80000)
        return dict(kind=kind, n=n, ci=ci, co=_log(rng, 512, 8192), linears=rng.randint(1, 3), seq=seq, vis=vis, na=rng.randint(6, 20), **quant)
    if kind == "export":
        # (the loss of given 16-bit weights loses its meaning where their own rounding is as large as the
        # quantisation error: up to four bits)
        quant["bits"] = rng.choice([3, 4])
        return dict(kind=kind, n=_log(rng, 128, 20000), ci=_width(rng, 256, 13824, group), co=_log(rng, 256, 8192),
                    seq=seq, vis=vis, **quant)
    if kind == "propagate":
        return dict(kind=kind, n=_log(rng, 64, 40960), ci=_width(rng, 256, 13824, group),
                    co=_log(rng, 32, 1728) * 8, seq=seq, vis=vis, act=rng.choice([0, 0, 8]), **quant)
    if kind == "attention":
        return dict(kind=kind, samples=_log(rng, 1, 48), seq=_log(rng, 16, 2048), heads=rng.randint(1, 40), dt=dt)
    if kind == "glue":
        return dict(kind=kind, n=_log(rng, 64, 40960), c=_width(rng, 256, 5120, 0), ffn=_width(rng, 512, 13824, 0), dt=dt)
    if kind == "select":
        return dict(kind=kind, samples=_log(rng, 1, 64), seq=seq, vis=vis, c=_width(rng, 256, 5120, 0),
                    l2=rng.randint(0, 1), dt=dt)
    return dict(kind=kind, layers=rng.randint(1, 2), heads=rng.randint(1, 6), ffn=128 * rng.randint(2, 12),
                samples=rng.randint(2, 4), seq=rng.randint(40, 300), vis=32, bits=rng.choice([3, 4]), group=128,
                na=rng.choice([5, 6]), mode=rng.choice(["passact2", "none"]), strategy=rng.choice(["tokens", "gram"]),
                dt=dt)


# ---------------------------------------------------------------- inputs
def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 64 + stream)
    return g


def _text_rows(case, n):
    return (torch.arange(n, device="cuda") % case["seq"]) >= case["vis"]


def _tokens(case, seed, n, c, stream=0):
    """[n, c] activations in the case's type: N(0,1), 1 % of the channels x5 on visual rows and x30 on
    text rows (the outliers of vision-language activations)."""
    dt = _DT[case["dt"]][0]
    g = _gen(seed, stream)
    out = torch.empty((n, c), dtype=dt, device="cuda")
    oc = torch.randperm(c, generator=g, device="cuda")[:max(1, round(0.01 * c))]
    mult = torch.where(_text_rows(case, n), 30.0, 5.0)
    for r in range(0, n, 16384):
        x = torch.randn((min(16384, n - r), c), generator=g, device="cuda")
        x[:, oc] *= mult[r:r + 16384, None]
        out[r:r + 16384] = x.to(dt)
    return out


def _weights(case, seed, co, ci, stream):
    return (torch.randn((co, ci), generator=_gen(seed, stream), device="cuda") * 0.02).to(_DT[case["dt"]][0])


def _token_w(case, seed, n, stream=1):
    """Heavy-tailed importance weights, four times larger on text rows, normalised to sum 1."""
    w = torch.exp(torch.randn(n, generator=_gen(seed, stream), device="cuda", dtype=torch.float64))
    w = torch.where(_text_rows(case, n), 4.0 * w, w)
    return (w / w.sum()).float()


def _alphas(na):
    return torch.tensor([k / na for k in range(na)], dtype=torch.float32, device="cuda")


def _params(case):
    code = _DT[case["dt"]][1]
    return tlq.params(bits=case.get("bits", 4), group=case.get("group", 128), symmetric=case.get("sym", 0),
                      act_bits=case.get("act", 0), x_dtype=code, yref_dtype=code)


def _f32(*shape):
    return torch.empty(shape, dtype=torch.float32, device="cuda")


def _bytes(n):
    return torch.empty(max(int(n), 256), dtype=torch.uint8, device="cuda")


def _plain_scales(X):
    """A searched scale vector for the calls that take one: mean |x| ** 0.45."""
    return (X.float().abs().mean(0) if X.shape[0] <= 16384 else X[:16384].float().abs().mean(0)).clamp_min(2.0 ** -14) ** 0.45


def prepare(case, seed):
    kind, p, dt = case["kind"], _params(case), _DT[case["dt"]][0]
    st = {"case": case, "p": p}
    if kind == "search":
        n, ci, co, na = case["n"], case["ci"], case["co"], case["na"]
        X, W = _tokens(case, seed, n, ci), _weights(case, seed, co, ci, 2)
        Y = torch.empty((n, co + -co % 8), dtype=dt, device="cuda")[:, :co]
        tlq.ref_output(X, W, Y, tlq.params(x_dtype=p.x_dtype, yref_dtype=p.yref_dtype))
        st.update(X=X, W=W, Y=Y, w=_token_w(case, seed, n), al=_alphas(na),
                  out=(_f32(na), torch.empty(1, dtype=torch.int32, device="cuda"), _f32(ci), _f32(na, ci)),
                  ws=_bytes(tlq.scale_search_workspace_bytes(n, ci, co, na, p)))
    elif kind == "gram":
        n, ci, na = case["n"], case["ci"], case["na"]
        co = case["co"]
        Ws = [_weights(case, seed, co, ci, 2 + i) for i in range(case["linears"])]
        need = max(tlq.x_stat_workspace_bytes(n, ci), tlq.token_gram_workspace_bytes(n, ci),
                   tlq.scale_search_gram_workspace_bytes(ci, co, na, p))
        st.update(X=_tokens(case, seed, n, ci), Ws=Ws, w=_token_w(case, seed, n), al=_alphas(na), xs=_f32(ci),
                  gram=_bytes(tlq.token_gram_bytes(ci)), ws=_bytes(need),
                  out=[(_f32(na), torch.empty(1, dtype=torch.int32, device="cuda"), _f32(ci)) for _ in Ws])
    elif kind == "export":
        n, ci, co = case["n"], case["ci"], case["co"]
        g = case["group"] or ci
        X, W = _tokens(case, seed, n, ci), _weights(case, seed, co, ci, 2)
        Y = torch.empty((n, co + -co % 8), dtype=dt, device="cuda")[:, :co]
        tlq.ref_output(X, W, Y, p)
        s = _plain_scales(X)
        st.update(X=X, W=W, Y=Y, s=s, inv=(1.0 / s.double()).float(), w=_token_w(case, seed, n),
                  codes=torch.empty((co, ci), dtype=torch.uint8, device="cuda"),
                  zp=torch.empty((co, ci // g), dtype=torch.uint8, device="cuda"), delta=_f32(co, ci // g),
                  Wdq=torch.empty((co, ci), dtype=dt, device="cuda"), loss=_f32(1), err=_f32(n),
                  ws=_bytes(tlq.weighted_layer_err_workspace_bytes(n, ci, co, p)))
    elif kind == "propagate":
        n, ci, co = case["n"], case["ci"], case["co"]
        X = _tokens(case, seed, n, ci)
        st.update(X=X, W=_weights(case, seed, co, ci, 2), s=_plain_scales(X),
                  Y=torch.empty((n, co), dtype=dt, device="cuda"), Z=torch.empty((n, co), dtype=dt, device="cuda"),
                  ws=_bytes(tlq.apply_best_workspace_bytes(n, ci, co, p)))
    elif kind == "attention":
        n, d = case["samples"] * case["seq"], case["heads"] * 128
        # q, k, v of normalised inputs through N(0, 0.02^2) weights of a few thousand channels
        qkv = torch.empty((n, 3 * d), dtype=dt, device="cuda")
        g = _gen(seed, 0)
        for r in range(0, n, 16384):
            qkv[r:r + 16384] = (torch.randn((min(16384, n - r), 3 * d), generator=g, device="cuda") * 1.4).to(dt)
        st.update(qkv=qkv, out=torch.empty((n, d), dtype=dt, device="cuda"))
    elif kind == "glue":
        n, c, f = case["n"], case["c"], case["ffn"]
        new = lambda cols, stream, scale: (torch.randn((n, cols), generator=_gen(seed, stream), device="cuda") * scale).to(dt)
        e = lambda cols: torch.empty((n, cols), dtype=dt, device="cuda")
        gu = new(2 * f, 2, 1.4)      # gate and up come out as column slices of one matrix
        st.update(H=new(c, 0, 3.0), Z=new(c, 1, 1.0), G=gu[:, :f], U=gu[:, f:],
                  m=torch.rand(c, generator=_gen(seed, 3), device="cuda") + 0.5, out=(e(c), e(f), e(c)))
    elif kind == "select":
        n, c, per = case["samples"] * case["seq"], case["c"], case["seq"]
        amp = torch.exp(torch.randn(per, generator=_gen(seed, 3), device="cuda") * 1.5 - 4.0)
        amp[case["vis"]:] = torch.exp(torch.randn(per - case["vis"], generator=_gen(seed, 4), device="cuda") * 0.5)
        G = torch.empty((n, c), dtype=dt, device="cuda")
        g = _gen(seed, 2)
        for b in range(case["samples"]):
            G[b * per:(b + 1) * per] = (torch.randn((per, c), generator=g, device="cuda") * amp[:, None]).to(dt)
        st.update(X=_tokens(case, seed, n, c), G=G, sum_n=torch.empty(per, dtype=torch.float64, device="cuda"),
                  mask=torch.empty(per, dtype=torch.uint8, device="cuda"), xs_max=_f32(c), xs_mean=_f32(c),
                  ws=_bytes(max(8 * n + 256, tlq.x_stat_workspace_bytes(n, c))))
    else:
        d, f, n = case["heads"] * 128, case["ffn"], case["samples"] * case["seq"]
        shapes = ((d, d),) * 4 + ((f, d), (f, d), (d, f))
        Ws = [[(torch.randn(s, generator=_gen(seed, 8 + layer), device="cuda") * 0.06).to(dt) for s in shapes]
              for layer in range(case["layers"])]
        st.update(h0=_tokens(case, seed, n, d), Ws=Ws, w=_token_w(case, seed, n), al=_alphas(case["na"]))
    return st


def run(state):
    case, p, kind = state["case"], state["p"], state["case"]["kind"]
    if kind == "search":
        losses, idx, best, table = state["out"]
        tlq.scale_search(state["X"], state["W"], state["Y"], state["w"], state["al"], p, best, idx, losses,
                         s_table_out=table, workspace=state["ws"])
        return losses, idx, best, table
    if kind == "gram":
        tlq.x_stat(state["X"], p, state["xs"], workspace=state["ws"])
        tlq.token_gram(state["X"], state["w"], p, state["gram"], workspace=state["ws"])
        for W, (losses, idx, best) in zip(state["Ws"], state["out"]):
            tlq.scale_search_gram(state["gram"], W, state["al"], p, state["xs"], best, idx, losses, workspace=state["ws"])
        return state["xs"], state["out"]
    if kind == "export":
        tlq.fake_quant(state["W"], state["s"], p, state["codes"], state["zp"], state["delta"], state["Wdq"])
        tlq.weighted_layer_err(state["X"], state["Wdq"], state["inv"], state["Y"], state["w"], p, state["loss"],
                               per_token_err=state["err"], workspace=state["ws"])
        return state["codes"], state["zp"], state["delta"], state["Wdq"], state["loss"], state["err"]
    if kind == "propagate":
        tlq.ref_output(state["X"], state["W"], state["Y"], p)
        tlq.apply_best(state["X"], state["W"], state["s"], p, state["Z"], workspace=state["ws"])
        return state["Y"], state["Z"]
    if kind == "attention":
        d, qkv = case["heads"] * 128, state["qkv"]
        return tlq.causal_attention(qkv[:, :d], qkv[:, d:2 * d], qkv[:, 2 * d:], case["heads"], case["seq"], p,
                                    state["out"])
    if kind == "glue":
        x, m, h = state["out"]
        tlq.rmsnorm_mul(state["H"], p, x, m_a=state["m"])
        tlq.silu_mul(state["G"], state["U"], p, m)
        tlq.residual_add(state["H"], state["Z"], p, h)
        return x, m, h
    if kind == "select":
        ws = state["ws"]
        tlq.token_importance(state["G"], case["samples"], p, state["sum_n"], l2=bool(case["l2"]), workspace=ws)
        tlq.topk_mask(state["sum_n"], case["seq"] // 2, state["mask"])
        tlq.x_stat_masked(state["X"], state["mask"], p, state["xs_max"], workspace=ws)
        tlq.x_stat(state["X"], p, state["xs_mean"], workspace=ws)
        return state["sum_n"], state["mask"], state["xs_max"], state["xs_mean"]
    recs, hq, _ = gstack.run_stack(state["h0"], lambda layer: state["Ws"][layer], case["layers"], state["w"], state["al"],
                                   p, case["heads"], case["seq"], mode=case["mode"], strategy=case["strategy"])
    return hq, [[(r[n]["losses"], r[n]["best_idx"], r[n]["best_scales"]) for n in gstack.LINEARS] for r in recs]


def work(case):
    """Each input once, each output once; the contractions in the form that the entry point names."""
    kind = case["kind"]
    if kind == "search":
        n, ci, co, na = case["n"], case["ci"], case["co"], case["na"]
        return {"bytes": 2 * (n * ci + co * ci + n * co) + 4 * (n + na * ci), "flops": 2 * n * ci * co * na}
    if kind == "gram":
        n, ci, co, na = case["n"], case["ci"], case["co"] * case["linears"], case["na"]
        # both contractions have a symmetric operand or result: half of the full product
        return {"bytes": 2 * (n * ci + co * ci + ci * ci) + 4 * n, "flops": n * ci * ci + na * co * ci * ci}
    if kind == "export":
        n, ci, co = case["n"], case["ci"], case["co"]
        return {"bytes": 2 * (n * ci + n * co) + 5 * co * ci + 8 * n, "flops": 2 * n * ci * co}
    if kind == "propagate":
        n, ci, co = case["n"], case["ci"], case["co"]
        return {"bytes": 2 * (n * ci + co * ci + 2 * n * co), "flops": 4 * n * ci * co}
    if kind == "attention":
        b, s, h = case["samples"], case["seq"], case["heads"]
        return {"bytes": 2 * 4 * b * s * h * 128, "flops": 2 * b * h * s * (s + 1) * 128}
    if kind == "glue":
        n, c, f = case["n"], case["c"], case["ffn"]
        # the two passes over H are two calls of a program that has other work between them
        return {"bytes": 2 * n * (5 * c + 3 * f), "flops": n * (8 * c + 8 * f)}
    if kind == "select":
        n, c = case["samples"] * case["seq"], case["c"]
        # gradients once, the selected half of the tokens for the maximum, all of them for the mean
        return {"bytes": 2 * n * c + n * c + 2 * n * c, "flops": 5 * n * c}
    d, f, n, na = case["heads"] * 128, case["ffn"], case["samples"] * case["seq"], case["na"]
    params = 4 * d * d + 3 * d * f
    return {"bytes": case["layers"] * 2 * params + 4 * n * d, "flops": case["layers"] * 2 * n * params * (na + 2)}


def tolerance(case):
    """About four times what the calls show against `exact` (2-norm), over seeded draws of every kind."""
    kind, bf16 = case["kind"], case["dt"] == "bf16"
    if kind in ("search", "gram"):
        # losses: the computed operand is rounded once to fp16; 1e-5 .. 9e-5 of the loss
        return {"rel": 4e-4, "max": 1e-3, "differ": 0.0}
    if kind == "stack":
        # a 16-bit rounding that falls the other way in one linear changes a few codes in the next
        return {"rel": 2e-2, "differ": 0.0}
    if kind == "select":
        return {"rel": 1e-6, "differ": 0.0}
    # 16-bit results: half a unit of the last place is 1.7e-3 (bf16), 2.1e-4 (f16) in the 2-norm
    return {"rel": 7e-3 if bf16 else 1.6e-3, "differ": 0.0}


# ---------------------------------------------------------------- the same in 64 bits
def _grid(W, s, bits, group, sym):
    """Codes, zero points, steps and dequantised weights: the grid arithmetic is defined in 32 bits, one
    rounding per operation (torch turns a division by a Python number into a product: divide by tensors)."""
    co, ci = W.shape
    g = group or ci
    ws = W.float() if s is None else W.float() * s[None, :]
    ws = ws.view(co, ci // g, g)
    if sym:
        half = 2 ** (bits - 1)
        amax = ws.abs().amax(2).clamp_min(1e-5)
        delta = amax / torch.full_like(amax, half - 1)
        q = torch.round(ws / delta[:, :, None]).clamp(-half, half - 1)
        zp = torch.full_like(delta, half)
        return (q + half).view(co, ci), zp, delta, (q * delta[:, :, None]).view(co, ci)
    top = 2 ** bits - 1
    mx, mn = ws.amax(2), ws.amin(2)
    delta = (mx - mn).clamp_min(1e-5) / torch.full_like(mx, top)
    zp = torch.round(-mn / delta).clamp(0, top)
    q = (torch.round(ws / delta[:, :, None]) + zp[:, :, None]).clamp(0, top)
    return q.view(co, ci), zp, delta, ((q - zp[:, :, None]) * delta[:, :, None]).view(co, ci)


def _act_codes(X, inv, bits):
    """Per-token activation codes (32-bit grid arithmetic by definition) and steps."""
    half = 2 ** (bits - 1)
    xt = X.float() * inv[None, :]
    amax = xt.abs().amax(1).clamp_min(1e-5)
    sg = amax / torch.full_like(amax, half - 1)
    return torch.round(xt / sg[:, None]).clamp(-half, half - 1), sg


def _scales(x_stat, al):
    return (x_stat.clamp_min(2.0 ** -14).double()[None, :] ** al.double()[:, None]).float()


def _mean_abs(X):
    s = torch.zeros(X.shape[1], dtype=torch.float64, device="cuda")
    for r in range(0, X.shape[0], 8192):
        s += X[r:r + 8192].double().abs().sum(0)
    return (s / X.shape[0]).float()


def _exact_losses(case, X, W, target, w, table):
    """sum_t w_t mean_o (target - f_q)^2 for every candidate; target(rows) gives [rows, co] in 64 bits."""
    co, act = W.shape[0], case.get("act", 0)
    losses = torch.zeros(table.shape[0], dtype=torch.float64, device="cuda")
    folded = []
    for k in range(table.shape[0]):
        deq = _grid(W, table[k], case["bits"], case["group"], case["sym"])[3].double()
        folded.append((deq if act else deq / table[k].double()[None, :]).t().contiguous())
    step = 8192
    for r in range(0, X.shape[0], step):
        xb, y, wb = X[r:r + step], target(slice(r, r + step)), w[r:r + step].double()
        xd = xb.double()
        for k, f in enumerate(folded):
            if act:
                q, sg = _act_codes(xb, (1.0 / table[k].double()).float(), act)
                d = y - (q.double() @ f) * sg.double()[:, None]
            else:
                d = y - xd @ f
            losses[k] += (wb * (d * d).sum(1)).sum() / co
    return losses


def exact(case, seed):
    kind, st = case["kind"], None
    # the chosen index and its scales follow from the losses up to near ties: no exact value is given for them
    if kind == "search":
        if 2.0 * case["n"] * case["ci"] * case["co"] * case["na"] > 1.7e14:
            return None
        st = prepare(case, seed)
        table = _scales(_mean_abs(st["X"]), st["al"])
        return _exact_losses(case, st["X"], st["W"], lambda r: st["Y"][r].double(), st["w"], table), None, None, table
    if kind == "gram":
        st = prepare(case, seed)
        X, w, xs = st["X"], st["w"], _mean_abs(st["X"])
        table = _scales(xs, st["al"])
        G = torch.zeros((case["ci"], case["ci"]), dtype=torch.float64, device="cuda")
        for r in range(0, X.shape[0], 8192):
            xd = X[r:r + 8192].double()
            G += xd.t().contiguous() @ (xd * w[r:r + 8192].double()[:, None])
        out = []
        for W in st["Ws"]:
            ls = torch.empty(case["na"], dtype=torch.float64, device="cuda")
            for k in range(case["na"]):
                d = W.double() - _grid(W, table[k], case["bits"], case["group"], case["sym"])[3].double() / table[k].double()[None, :]
                ls[k] = ((d @ G) * d).sum() / W.shape[0]
            out.append((ls, None, None))
        return xs, out
    if kind == "export":
        st = prepare(case, seed)
        q, zp, delta, deq = _grid(st["W"], st["s"], case["bits"], case["group"], case["sym"])
        wdq = deq.to(st["W"].dtype)
        yq = (st["X"].double() * st["inv"].double()[None, :]) @ wdq.double().t().contiguous()
        err = (st["Y"].double() - yq).pow(2).mean(1)
        return (q.to(torch.uint8), zp.to(torch.uint8), delta, deq.double(), (st["w"].double() * err).sum()[None], err)
    if kind == "propagate":
        st = prepare(case, seed)
        X, W, s, act = st["X"], st["W"], st["s"], case["act"]
        deq = _grid(W, s, case["bits"], case["group"], case["sym"])[3].double()
        wt = W.double().t().contiguous()
        ft = (deq if act else deq / s.double()[None, :]).t().contiguous()
        ys, zs = [], []
        for r in range(0, X.shape[0], 8192):
            xd = X[r:r + 8192].double()
            ys.append(xd @ wt)
            if act:
                q, sg = _act_codes(X[r:r + 8192], (1.0 / s.double()).float(), act)
                zs.append((q.double() @ ft) * sg.double()[:, None])
            else:
                zs.append(xd @ ft)
        return torch.cat(ys), torch.cat(zs)
    if kind == "attention":
        st = prepare(case, seed)
        b, s, h = case["samples"], case["seq"], case["heads"]
        d = h * 128
        out = torch.empty((b * s, d), dtype=torch.float64, device="cuda")
        hide = torch.ones((s, s), dtype=torch.bool, device="cuda").triu(1)
        for i in range(b):
            rows = st["qkv"][i * s:(i + 1) * s].double()
            q, k, v = (rows[:, j * d:(j + 1) * d].view(s, h, 128).transpose(0, 1).contiguous() for j in range(3))
            sc = torch.bmm(q, k.transpose(1, 2).contiguous()) / math.sqrt(128.0)
            pr = torch.softmax(sc.masked_fill_(hide, float("-inf")), 2)
            out[i * s:(i + 1) * s] = torch.bmm(pr, v).transpose(0, 1).reshape(s, d)
        return out
    if kind == "glue":
        st = prepare(case, seed)
        H, g = st["H"].double(), st["G"].double()
        x = H / torch.sqrt(H.pow(2).mean(1, keepdim=True) + 1e-6) * st["m"].double()[None, :]
        return x, g / (1.0 + torch.exp(-g)) * st["U"].double(), H + st["Z"].double()
    if kind == "select":
        st = prepare(case, seed)
        per, X = case["seq"], st["X"]
        s = torch.zeros(per, dtype=torch.float64, device="cuda")
        for b in range(case["samples"]):
            gb = st["G"][b * per:(b + 1) * per].double()
            s += gb.pow(2).sum(1).sqrt() if case["l2"] else gb.abs().mean(1)
        order = torch.argsort(-s, stable=True)
        mask = torch.zeros(per, dtype=torch.uint8, device="cuda")
        mask[order[:per // 2]] = 1
        mx = torch.zeros(case["c"], dtype=torch.float64, device="cuda")
        for b in range(case["samples"]):
            mx = torch.maximum(mx, X[b * per:(b + 1) * per][mask.bool()].double().abs().amax(0))
        return s, mask, mx, _mean_abs(X)
    return None      # activations are rounded to 16 bits between the linears of a stack
