"""hs_sum's stores: rows at every alignment (bins not a multiple of four), full
and ragged tiles, an output that is 4-byte aligned only, planes that fit the
last-level cache and planes that do not; bitwise against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_1805_12258_amd as hs
from tests.helpers import padded_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("T,N,H", [(1, 256, 2), (33, 257, 8), (40, 1022, 5), (7, 767, 16), (85, 1536, 8), (64, 300003, 4),
                                   (16, 256 * 2100 + 3, 8)])
def test_planes_at_every_alignment(T, N, H, dtype):
    print("case", T, N, H, dtype, flush=True)
    scale = 1.0 if dtype == "f32" else 0.125
    gen = torch.Generator().manual_seed(T + N + H)
    x = torch.empty((T, N)).exponential_(1.0, generator=gen)
    kind = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}[dtype]
    dev, store = padded_device(x, dtype=kind, scale=scale)
    plan = hs.Plan(T, N, H, dtype=dtype, input_scale=scale)
    want = oracle.sum_f32(store.to(torch.float32).numpy(), H) * np.float32(1.0 / scale)
    buf = torch.full((H * T * N + 8,), -3.0, device="cuda")
    for shift in (0, 1):
        out = buf[shift:shift + H * T * N].view(H, T, N)
        plan.sum(dev, out=out)
        assert np.array_equal(out.cpu().numpy().view(np.uint32), want.view(np.uint32))
    assert bool((buf[1 + H * T * N:] == -3.0).all())
