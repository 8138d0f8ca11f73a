"""Infinite, NaN and extreme powers inside a plane, and thresholds of every such
kind, through the row walk (every strip width), the fractional chains and
hs_sum: bitwise against the oracle (NaN sums are no candidates and, in the
planes, NaN of any bits)."""
import numpy as np
import pytest
import torch

import oracle
import paper_1805_12258_amd as hs
from tests.helpers import assert_same_candidates, gpu_detect, oracle_detect_sorted, padded_device, sort_cands

pytestmark = pytest.mark.gpu

TYPES = {"f32": (torch.float32, 1.0), "f16": (torch.float16, 0.125), "bf16": (torch.bfloat16, 0.125)}
THRESHOLDS = np.array([-np.inf, np.inf, np.nan, 3, 8, 20, -3e38, 3e38], dtype=np.float32)


def special_plane(T, N, dtype):
    kind, scale = TYPES[dtype]
    rng = np.random.default_rng(T * N)
    x = rng.exponential(1.0, (T, N)).astype(np.float32)
    big = float(torch.finfo(kind).max)
    put = rng.random((T, N)) < 0.02
    x[put] = rng.choice(np.array([np.inf, -np.inf, np.nan, big, -big], dtype=np.float32), int(put.sum()))
    dev, store = padded_device(torch.from_numpy(x), dtype=kind, scale=scale)
    return dev, store, scale, rng


def same_planes(got, want):
    ok = (got.view(np.uint32) == want.view(np.uint32)) | (np.isnan(got) & np.isnan(want))
    assert ok.all()


@pytest.mark.parametrize("T,N,H", [(21, 700, 8), (9, 517, 16), (40, 1030, 5), (1, 300, 4)])
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_special_powers_and_thresholds(T, N, H, dtype):
    print("case", T, N, H, dtype, flush=True)
    dev, store, scale, rng = special_plane(T, N, dtype)
    ta = rng.choice(THRESHOLDS, (H, T))
    want = oracle_detect_sorted(store, H, ta, scale=scale)
    for V in (0, 2, 4, 8):
        kw = {"schedule": 4, "bins_per_lane": V} if V else {}
        plan = hs.Plan(T, N, H, dtype=dtype, input_scale=scale, **kw)
        assert_same_candidates(gpu_detect(plan, dev, ta, capacity=H * T * N + 8), want)
    x = store.to(torch.float32).numpy()
    with np.errstate(invalid="ignore", over="ignore"):
        same_planes(plan.sum(dev).cpu().numpy(), oracle.sum_f32(x, H) * np.float32(1.0 / scale))
        frac = hs.Plan(T, N, H, dtype=dtype, input_scale=scale, mapping="fractional")
        same_planes(frac.sum(dev).cpu().numpy(), oracle.sum_frac_f32(x, H) * np.float32(1.0 / scale))
    idx, pw, cnt = oracle.detect_frac_f32(x, H, ta, scale=scale, nthreads=4)
    assert_same_candidates(gpu_detect(frac, dev, ta, capacity=H * T * N + 8), (*sort_cands(idx, pw), cnt))
