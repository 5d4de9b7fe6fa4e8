"""LC encode beyond one round of blocks (more than 2^23 elements, with a partial last
trip and a last group alone): every row's codes and packed bytes equal those of a
separate call on a slice of rows small enough for a single trip, which
test_gpu_encode.py checks against the definition."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [8, 4])
def test_encode_trips_match_slices(d, dtype):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2606_10531_amd as lc
    m, n = 1025, 8200
    g = torch.Generator(device="cuda").manual_seed(5)
    W = (0.05 * torch.randn((m, n), device="cuda", generator=g)).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    A, b = (torch.from_numpy(x).cuda() for x in synth.draw_map(d, 3))
    codes, packed = lc.encode(W, A, b, d, codes=True, packed=True)
    for r in range(0, m, 200):
        c, p = lc.encode(W[r:r + 200].contiguous(), A, b, d, codes=True, packed=True)
        assert torch.equal(codes[r:r + 200], c) and torch.equal(packed[r:r + 200], p), r
    assert len(torch.unique(codes)) == 4
