"""The transpose and the statistic's backward over pieces of rows and strips of
bins: pieces of 4, 8 and 16 rows, last pieces and strips of every kind (one
row, one bin, one short of full), boxes across pieces and strips for every
stretch factor up to 16, cotangents that are not 16-byte aligned.

Bounds.  Every dFOP value is an fp32 sum of non-negative terms here, through at
most H additions to form G_m, m <= 16 rows, m bins, 6 pieces and strips and H
factors: fewer than 3 H + 40 roundings in a chain, each 2^-24 relative.  The
statistic's weights carry the rounding of the exponent on top (a few ulps of
log2 g, |log2 g| <= 150: 4 * 150 * 2^-24 relative; smaller weights are zero in
fp32: fewer than 10^4 of 2^-126 each).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1805_12258_amd as hs
from tests.helpers import padded_device

pytestmark = pytest.mark.gpu

SHAPES = [(1, 3, 2), (2, 257, 3), (5, 1025, 16), (17, 511, 13), (16, 512, 7), (33, 256 * 5 + 1, 9), (85, 256 * 3 + 255, 8),
          (100, 256 * 130 + 77, 11), (128, 256 * 700 + 1, 6), (3, 256 * 4200 + 255, 5), (21, 256, 1),
          (16, 256 * 2100 + 1, 8)]               # planes larger than the last-level cache


@pytest.mark.parametrize("T,N,H", SHAPES)
def test_transpose_over_pieces(T, N, H):
    print("case", T, N, H, flush=True)
    rng = np.random.default_rng(T + N + H)
    g = rng.random((H, T, N), dtype=np.float32)
    buf = torch.zeros(H * T * N + 1, device="cuda")
    for shift in (0, 1):                       # the second one not 16-byte aligned
        gd = buf[shift:shift + H * T * N].view(H, T, N)
        gd.copy_(torch.from_numpy(g))
        got = hs.Plan(T, N, H).backward(gd).cpu().numpy().astype(np.float64)
        want = oracle.vjp_f64(g)
        assert np.all(np.abs(got - want) <= (3 * H + 40) * 2.0 ** -24 * want)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("T,N,H", [s for s in SHAPES if s[0] * s[1] < 200000])
def test_statistic_over_pieces(T, N, H, dtype):
    print("case", T, N, H, dtype, flush=True)
    tau, scale = 2.0, 1.0 if dtype == "f32" else 0.125
    gen = torch.Generator().manual_seed(T * 7 + N + H)
    x = torch.empty((T, N)).exponential_(1.0, generator=gen)
    torch_type = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    dev, store = padded_device(x, dtype=torch_type, scale=scale)
    plan = hs.Plan(T, N, H, dtype=dtype, input_scale=scale)
    lse = plan.lse(dev, tau)
    got = plan.lse_backward(dev, lse, tau, gscale=-1.5).cpu().numpy().astype(np.float64)
    planes = oracle.sum_f32(store.to(torch.float32).numpy(), H).astype(np.float64) / scale
    w = np.exp(planes / tau - lse.cpu().numpy()[:, None, None])
    want = oracle.vjp_f64(w) * 1.5
    assert np.all(got <= 0)
    assert np.all(np.abs(got + want) <= (4 * 150 + 3 * H + 40) * 2.0 ** -24 * want + 1e4 * 2.0 ** -126)
