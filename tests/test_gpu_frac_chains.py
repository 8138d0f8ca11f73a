"""Fractional planes and candidates by chains (the planes K, K/2, K/4, ... of
one pass, for every K in (H/2, H]): every chain of both kernels, rows in one
piece and several, last strips of one bin, one short and none, lists too short
for their candidates; bitwise against the oracle."""
import os

import numpy as np
import pytest
import torch

import oracle
import paper_1805_12258_amd as hs
from tests.helpers import assert_same_candidates, gpu_detect, padded_device, random_thresholds, sort_cands

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("T,N,H", [(2, 257, 1), (3, 511, 2), (7, 512, 4), (40, 256 * 9 + 1, 6), (19, 256 * 3 + 255, 9),
                                   (85, 256 * 33, 10), (5, 256 * 700 + 3, 7), (21, 5, 12), (33, 256 * 5 + 2, 14),
                                   (128, 256 * 16 + 1, 16)])
def test_every_chain_matches_the_oracle(T, N, H, dtype):
    print("case", T, N, H, dtype, flush=True)
    scale = 1.0 if dtype == "f32" else 0.125
    g = torch.Generator().manual_seed(T * N + H)
    x = torch.empty((T, N)).exponential_(1.0, generator=g)
    ta = random_thresholds(H, T, T + N + H)
    torch_type = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    dev, store = padded_device(x, dtype=torch_type, scale=scale)
    plan = hs.Plan(T, N, H, dtype=dtype, input_scale=scale, mapping="fractional")
    src = store.to(torch.float32).numpy()
    ref = oracle.sum_frac_f32(src, H) * np.float32(1.0 / scale)
    assert np.array_equal(plan.sum(dev).cpu().numpy().view(np.uint32), ref.view(np.uint32))
    idx, pw, cnt = oracle.detect_frac_f32(src, H, ta, scale=scale, nthreads=min(16, os.cpu_count() or 1))
    idx, pw = sort_cands(idx, pw)
    assert_same_candidates(gpu_detect(plan, dev, ta, capacity=H * T * N + 16), (idx, pw, cnt))

    # a list for half of them: the counts are those of all, the rest is dropped
    cap = len(idx) // 2
    out = torch.zeros((cap + 64, 2), dtype=torch.int32, device="cuda")
    counts = torch.empty(H + 1, dtype=torch.int64, device="cuda")
    hs.hs_detect(plan.handle, dev, dev.stride(0), torch.from_numpy(np.ascontiguousarray(ta)).cuda(), out, cap, counts)
    assert np.array_equal(counts.cpu().numpy(), cnt)
    got = out.cpu().numpy()
    assert not got[cap:].any()
    full = set(zip(idx.view(np.uint32).tolist(), pw.view(np.uint32).tolist()))
    assert {(int(w), int(p)) for w, p in got[:cap].view(np.uint32)} <= full
