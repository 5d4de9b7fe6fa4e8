"""A workspace sized for N tokens serves every smaller N: the sizes never fall as N
grows, whichever tiles the library picks on the way (the input gradient's per-block
sums take more blocks on some smaller N; the packed forward takes many tokens in
several passes of equal size, which are smaller than the one pass of fewer tokens)."""
import pytest
import torch

import paper_2606_10531_amd as lc


@pytest.mark.parametrize("m,n", [(64, 64), (512, 28672), (28672, 512), (4096, 4096), (6280, 10136), (8192, 28672)])
@pytest.mark.parametrize("op,dtype", [(op, dtype) for op in (lc.OP_FWD, lc.OP_BWD) for dtype in
                                      (torch.bfloat16, torch.float32)] + [(lc.OP_FWD_PACKED, torch.bfloat16)])
def test_workspace_grows_with_tokens(op, m, n, dtype):
    last = 0
    for N in list(range(1, 700, 31)) + list(range(700, 16500, 257)):
        size = lc.workspace_bytes(op, N, m, n, 8, dtype)
        assert size >= last, f"N={N}"
        last = size


def test_packed_passes_fit_one_grid():
    """A pass of the packed forward is one grid of a thread per 16 outputs (at least); even
    with the most out-features it stays below the 2^32 threads of a grid dimension, so the
    tokens of a pass, which the size tells, stop at 2^15."""
    m, n = (1 << 21) - 64, 64
    one = lc.workspace_bytes(lc.OP_FWD_PACKED, 64, m, n, 8, torch.bfloat16) / 64
    tokens = lc.workspace_bytes(lc.OP_FWD_PACKED, 1 << 20, m, n, 8, torch.bfloat16) / one
    assert tokens * m / 16 < 2 ** 32


def test_packed_long_rows_have_room_for_spans():
    """From 128 steps of 256 columns on, few rows split K over blocks: up to 32768 spans times
    rows of 16 fp32 sums.  The size does not depend on the out-features, and the split is
    left out where the 8 MiB of the call without a workspace do not hold it."""
    size = lambda m, n: lc.workspace_bytes(lc.OP_FWD_PACKED, 16, m, n, 8, torch.bfloat16)  # noqa: E731
    for n in (32768, 65536, 131072):
        assert size(64, n) >= n // 256 * 8192 + 32768 * 64
        assert size(64, n) == size(4096, n) == size(28672, n) <= 8 << 20
    assert size(64, 28672) < 112 * 8192 + 8192
    assert size(64, 262144 - 256) < (8 << 20)
