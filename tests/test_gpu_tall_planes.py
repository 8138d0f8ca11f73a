"""Tall planes of one to nine strips, whose pieces the waves of all XCDs share
(no list per XCD could be even): bitwise against the oracle, also as FOPs of a
batch; and a plane of one strip takes no longer than one of eight strips with
as many rows of strips in all."""
import numpy as np
import pytest
import torch

import oracle
import paper_1805_12258_amd as hs
from tests.helpers import (assert_same_candidates, batched_call, gpu_detect, oracle_detect_sorted, padded_device,
                           random_thresholds, unpack_batched)

pytestmark = pytest.mark.gpu

TYPES = {"f32": (torch.float32, 1.0), "f16": (torch.float16, 0.125), "bf16": (torch.bfloat16, 0.125)}


def plane(T, N, kind, scale):
    g = torch.Generator().manual_seed(T + N)
    return padded_device(torch.empty((T, N)).exponential_(1.0, generator=g), dtype=kind, scale=scale)


@pytest.mark.parametrize("T,N,H", [(1537, 1, 8), (4096, 5, 16), (9000, 257, 8), (1600, 2049, 5), (40001, 60, 3)])
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_tall_planes_match_the_oracle(T, N, H, dtype):
    print("case", T, N, H, dtype, flush=True)
    kind, scale = TYPES[dtype]
    dev, store = plane(T, N, kind, scale)
    ta = random_thresholds(H, T, T)
    want = oracle_detect_sorted(store, H, ta, scale=scale)
    for kw in ({}, {"persistent_blocks": 3}, {"schedule": 3}):
        plan = hs.Plan(T, N, H, dtype=dtype, input_scale=scale, **kw)
        assert_same_candidates(gpu_detect(plan, dev, ta, capacity=H * T * N + 16), want)


def test_tall_planes_of_a_batch():
    T, H, lens = 3000, 8, [300, 7, 520]
    devs, stores = zip(*(plane(T, n, torch.float32, 1.0) for n in lens))
    ta = random_thresholds(H, T, 5)
    plan = hs.Plan(T, 0, H, n_chans=lens)
    caps = [H * T * n + 8 for n in lens]
    (_, _, _, out, _, _, counts), offs = batched_call(plan, list(devs), ta, caps)
    for f, (idx, pw, cnt) in enumerate(unpack_batched(out, counts, offs, caps)):
        wi, wp, wc = oracle_detect_sorted(stores[f], H, ta)
        r, k, b = oracle.field_bits(T, lens[f], H)     # the batch's fields are the longest FOP's
        row, low = wi >> np.uint32(k + b), wi & np.uint32((1 << b) - 1)
        pl = (wi >> np.uint32(b)) & np.uint32((1 << k) - 1)
        word = (row << np.uint32(plan.info["s_row"])) | (pl << np.uint32(plan.info["s_bin"])) | low
        assert_same_candidates((idx, pw, cnt), (word, wp, wc))


def detect_us(T, N, H=8):
    x = torch.empty((T, (N + 3) // 4 * 4), device="cuda").exponential_()
    ta = torch.full((H, T), 1e9, device="cuda")
    plan = hs.Plan(T, N, H)
    out = torch.empty((16, 2), dtype=torch.int32, device="cuda")
    counts = torch.empty(H + 1, dtype=torch.int64, device="cuda")
    best = float("inf")
    for _ in range(10):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        hs.hs_detect(plan.handle, x, x.stride(0), ta, out, 16, counts)
        e1.record()
        e1.synchronize()
        best = min(best, 1e3 * e0.elapsed_time(e1))
    return best


def test_a_plane_of_one_strip_is_shared():
    tall, wide = detect_us(1 << 18, 200), detect_us(1 << 15, 2000)
    print("case us", round(tall, 1), round(wide, 1), flush=True)
    assert tall <= 2 * wide
