"""The register row walk's branches, bitwise against the oracle: planes whose
threshold table fits a block's LDS and taller ones (a table per wave and
piece), strips cut into several pieces, one to three rows, last strips of one
to four bins, one and many strips, fewer strips than XCDs, batches evened out
over the XCDs, and lists too short for their candidates."""
import numpy as np
import pytest
import torch

import oracle
import paper_1805_12258_amd as hs
from tests.helpers import (assert_same_candidates, batched_call, gpu_detect, make_batch, oracle_detect_sorted,
                           padded_device, random_thresholds, unpack_batched)

pytestmark = pytest.mark.gpu

TYPES = {"f32": (torch.float32, 1.0), "f16": (torch.float16, 0.125), "bf16": (torch.bfloat16, 0.125)}


@pytest.mark.parametrize("T,N,H", [(1, 300, 8), (2, 1027, 16), (3, 514, 5), (700, 513, 8), (1100, 260, 3),
                                   (255, 1282, 16), (85, 256 * 19 + 3, 12), (300, 4, 9), (21, 2049, 1), (64, 100003, 2)])
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_walk_branches(T, N, H, dtype):
    print("case", T, N, H, dtype, flush=True)
    kind, scale = TYPES[dtype]
    g = torch.Generator().manual_seed(T + 3 * N + H)
    x = torch.empty((T, N)).exponential_(1.0, generator=g)
    ta = random_thresholds(H, T, T * H + N)
    dev, store = padded_device(x, dtype=kind, scale=scale)
    want = oracle_detect_sorted(store, H, ta, scale=scale)
    plans = [hs.Plan(T, N, H, dtype=dtype, input_scale=scale)]
    if T >= 2 and T * H * 4 <= 16384:
        plans += [hs.Plan(T, N, H, dtype=dtype, input_scale=scale, schedule=4, bins_per_lane=V)
                  for V in (2, 4, 8)]
    for plan in plans:
        assert_same_candidates(gpu_detect(plan, dev, ta, capacity=H * T * N + 16), want)
    # room for half of them: the counts stay those of all, the rest is dropped
    idx, _, cnt = want
    cap = len(idx) // 2
    out = torch.zeros((cap + 64, 2), dtype=torch.int32, device="cuda")
    counts = torch.empty(H + 1, dtype=torch.int64, device="cuda")
    tat = torch.from_numpy(np.ascontiguousarray(ta)).cuda()
    for plan in plans:
        out.zero_()
        hs.hs_detect(plan.handle, dev, dev.stride(0), tat, out, cap, counts)
        assert np.array_equal(counts.cpu().numpy(), cnt)
        got = out.cpu().numpy()
        assert not got[cap:].any()
        assert set(got[:cap, 0].view(np.uint32).tolist()) <= set(idx.tolist())


@pytest.mark.parametrize("lens", [[70000], [131072, 300], [5, 70001, 1, 262144, 999]])
def test_few_lists_are_spread_over_the_xcds(lens):
    print("case", lens, flush=True)
    T, H = 43, 8
    devs, stores = make_batch(lens, T, H, 91)
    ta = random_thresholds(H, T, 92)
    plan = hs.Plan(T, 0, H, n_chans=lens)
    caps = [H * T * n + 8 for n in lens]
    (_, _, _, out, _, _, counts), offs = batched_call(plan, devs, ta, caps)
    for f, (idx, pw, cnt) in enumerate(unpack_batched(out, counts, offs, caps)):
        wi, wp, wc = oracle_detect_sorted(stores[f], H, ta)
        assert np.array_equal(cnt, wc)
        # the batch's words have fields of the longest list's width
        sr, sb = plan.info["s_row"], plan.info["s_bin"]
        r, k, b = oracle.field_bits(T, lens[f], H)
        row, low = wi >> np.uint32(k + b), wi & np.uint32((1 << b) - 1)
        pl = (wi >> np.uint32(b)) & np.uint32((1 << k) - 1)
        word = (row << np.uint32(sr)) | (pl << np.uint32(sb)) | low
        assert_same_candidates((idx, pw, cnt), (word, wp, wc))
