"""hs_backward_workspace_bytes over the whole range of bin counts a plan takes
(host only): at least a value per target of m = 2..H and piece of rows, at most
a few planes more, and no wrap at the largest."""
import pytest

import paper_1805_12258_amd as hs


@pytest.mark.parametrize("T,N,H", [(1, 2 ** 31 - 1, 2), (1, 2 ** 31 - 2, 2), (1, 2 ** 31 - 16, 2), (2, 2 ** 30, 2), (1, 2 ** 30, 4),
                                   (1, 2 ** 28, 16), (85, 1 << 21, 8), (1 << 20, 16, 16), (5, 3, 2), (1, 1, 16)])
def test_backward_workspace(T, N, H):
    p = hs.Plan(T, N, H)
    need = hs.hs_backward_workspace_bytes(p.handle)
    least = 4 * sum(-(-N // m) for m in range(2, H + 1)) * (T // 16 + 1 if T >= 16 else 1)
    assert least <= need <= 40 * least + 4096 * H * (T + 16)
