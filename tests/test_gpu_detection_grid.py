"""The default grid of the detection against three blocks of eight waves per
compute unit, which is what the walk's registers are chosen for up to eight
planes: every block ends with atomics on the same counters, so more blocks, where
few planes leave registers for them, take longer.  The smallest of several bursts
of either, in turn, within a tenth (a burst's minimum spreads by 2 %)."""
import pytest
import torch

import paper_1805_12258_amd as hs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("H", [1, 2, 4])
def test_default_grid_is_not_slower(H, dtype):
    T, N = 85, 1 << 18
    x = torch.empty((T, N), device="cuda").exponential_(1.0, generator=torch.Generator("cuda").manual_seed(3))
    if dtype == "f16":
        x = (x / 8).half()
    ta = torch.tensor([[k + 6.0 * k ** 0.5] * T for k in range(1, H + 1)], dtype=torch.float32, device="cuda")
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    out = torch.empty((1 << 18, 2), dtype=torch.int32, device="cuda")
    counts = torch.empty(H + 1, dtype=torch.int64, device="cuda")
    scale = 1.0 if dtype == "f32" else 0.125
    plans = [hs.Plan(T, N, H, dtype=dtype, input_scale=scale, persistent_blocks=b) for b in (0, 3 * cus)]
    found, best = [], [1e9, 1e9]
    for burst in range(8):
        for i, plan in enumerate(plans):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            plan.detect(x, ta, out=out, counts=counts)
            a.record()
            for _ in range(50):
                plan.detect(x, ta, out=out, counts=counts)
            b.record()
            b.synchronize()
            if burst:                  # the first warms up
                best[i] = min(best[i], a.elapsed_time(b))
            found.append(counts.tolist())
    assert all(c == found[0] for c in found)
    assert best[0] < 1.1 * best[1], best
