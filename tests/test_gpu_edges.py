"""Sizes at which a tile, a remainder or a dispatch rule of the kernels can go wrong, against the oracle."""
import numpy as np
import pytest

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
