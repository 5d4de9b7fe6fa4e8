"""The packed-codes forward up to 16 tokens on each of its blocks (16 to 128 rows, 4, 8
and 16 waves, one and two rounds of blocks), with X transformed in the block (up to 2, up to 4 tokens) and by the
prepass (5 and more), K whole or split over blocks, at ragged rows and K not a multiple of a step, with fewer steps
than waves and with several per wave, against the oracle at 2e-2; a repeated call
gives the same bits."""
import numpy as np
import pytest

import oracle as orc
import synth
from helpers import assert_close, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lc():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2606_10531_amd as lc
    lc._lib.load()
    return lc


@pytest.mark.parametrize("N", [1, 2, 3, 4, 5, 16])
@pytest.mark.parametrize("m,n,d", [(24, 4160, 8), (72, 8256, 4), (5448, 320, 4), (5448, 6208, 8), (10888, 448, 8),
                                   (16360, 64, 4), (18440, 192, 8), (22536, 320, 8), (28664, 576, 4),
                                   (32760, 448, 8), (32776, 128, 8)])
def test_packed_rows(lc, N, m, n, d):
    import torch
    print(f"\npacked rows N={N} m={m} n={n} d={d}", flush=True)
    r = synth.rng(N + m + n + d)
    P = r.integers(0, 256, size=(m, n // 4), dtype=np.uint8)
    Xb = synth.draw_activations(N, n, 7 + N, "bf16")
    A, b = synth.draw_map(d, 1)
    Pd, X = torch.from_numpy(P).cuda(), to_dev(Xb, "bf16")
    Ad, bd = torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda()
    need = lc.workspace_bytes(lc.OP_FWD_PACKED, N, m, n, d, torch.bfloat16)
    got = []
    for _ in range(2):
        ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")    # NaN wherever nothing is written
        Y = torch.full((N, m), float("nan"), dtype=torch.float32, device="cuda")
        got.append(lc.linear_fwd_packed(Pd, Ad, bd, X, d, workspace=ws, out=Y))
    torch.cuda.synchronize()
    ref = orc.linear_forward_packed(P, A.astype(np.float64), b.astype(np.float64), orc.widen(Xb, "bf16"), d, n)
    assert_close(to_host(got[0]), ref, 2e-2, "Y")
    assert torch.equal(got[0].view(torch.int32), got[1].view(torch.int32))


@pytest.mark.parametrize("N", [1, 2, 3, 4])
@pytest.mark.parametrize("m,n,d", [(16376, 4096, 4), (16392, 4160, 8), (24568, 4544, 4), (28664, 8192, 8), (32776, 5184, 8),
                                   (32760, 16064, 4)])
def test_packed_rows_four_waves(lc, N, m, n, d):
    """Blocks of 64 rows and more over 16 to 63 steps of K (four waves, an odd and an even
    number of steps each), on sampled rows."""
    import torch
    print(f"\npacked rows, four waves N={N} m={m} n={n} d={d}", flush=True)
    r = synth.rng(N + m + n + d)
    P = r.integers(0, 256, size=(m, n // 4), dtype=np.uint8)
    Xb = synth.draw_activations(N, n, 7 + N, "bf16")
    A, b = synth.draw_map(d, 1)
    Pd, X = torch.from_numpy(P).cuda(), to_dev(Xb, "bf16")
    Ad, bd = torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda()
    got = []
    for _ in range(3):
        Y = torch.full((N, m), float("nan"), dtype=torch.float32, device="cuda")
        got.append(lc.linear_fwd_packed(Pd, Ad, bd, X, d, out=Y))
    torch.cuda.synchronize()
    rows = np.unique(np.concatenate([np.arange(260), np.arange(m // 2, m // 2 + 260), np.arange(m - 260, m)]))
    ref = orc.linear_forward_packed(P[rows], A.astype(np.float64), b.astype(np.float64), orc.widen(Xb, "bf16"), d, n)
    assert_close(to_host(got[0])[:, rows], ref, 2e-2, "Y")
    assert all(torch.equal(got[0].view(torch.int32), g.view(torch.int32)) for g in got[1:])


@pytest.mark.parametrize("N", [5, 16])
@pytest.mark.parametrize("m,n,d", [(136, 4096, 8), (200, 16576, 4), (136, 28736, 8), (72, 33088, 4)])
def test_parts_of_s(lc, N, m, n, d):
    """s from 16 parts of one step to 29 of four, with an offset that dominates the output,
    so that a part left out or taken twice is far beyond the tolerance."""
    import torch
    print(f"\npacked parts of s N={N} m={m} n={n} d={d}", flush=True)
    r = synth.rng(N + m + n + d)
    P = r.integers(0, 256, size=(m, n // 4), dtype=np.uint8)
    Xb = synth.draw_activations(N, n, 7 + N, "bf16")
    A, b = synth.draw_map(d, 1)
    b = (100.0 * b).astype(np.float32)
    Y = lc.linear_fwd_packed(torch.from_numpy(P).cuda(), torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda(),
                             to_dev(Xb, "bf16"), d)
    torch.cuda.synchronize()
    ref = orc.linear_forward_packed(P, A.astype(np.float64), b.astype(np.float64), orc.widen(Xb, "bf16"), d, n)
    assert_close(to_host(Y), ref, 2e-2, "Y")


@pytest.mark.parametrize("N", [1, 2, 3, 5, 16, 19])
@pytest.mark.parametrize("m,n,d", [(8, 32768, 8), (200, 33088, 4), (1032, 40960, 8), (4104, 32832, 8), (6136, 34048, 4)])
def test_long_rows(lc, N, m, n, d):
    """Few rows over 128 steps of K and more, K split over blocks (up to 16 spans, the last
    one short), on sampled rows: with a workspace of NaN, in the fixed array (the same
    bits), and unsplit in a workspace that has no room for the spans' sums."""
    import torch
    print(f"\npacked long rows N={N} m={m} n={n} d={d}", flush=True)
    r = synth.rng(N + m + n + d)
    P = r.integers(0, 256, size=(m, n // 4), dtype=np.uint8)
    Xb = synth.draw_activations(N, n, 7 + N, "bf16")
    A, b = synth.draw_map(d, 1)
    b = (100.0 * b).astype(np.float32)
    Pd, X = torch.from_numpy(P).cuda(), to_dev(Xb, "bf16")
    Ad, bd = torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda()
    need = lc.workspace_bytes(lc.OP_FWD_PACKED, N, m, n, d, torch.bfloat16)
    Y = [torch.full((N, m), float("nan"), dtype=torch.float32, device="cuda") for _ in range(4)]
    for y in Y[:2]:
        ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
        lc.linear_fwd_packed(Pd, Ad, bd, X, d, workspace=ws, out=y)
    lc.linear_fwd_packed_noalloc(Pd, Ad, bd, X, d, out=Y[2])
    small = torch.empty(-(-n // 256) * 8192 + 32 * 64, dtype=torch.uint8, device="cuda")   # X' and the parts of s
    st = lc._lib.load().lcvq_linear_fwd_packed(N, m, n, d, Pd.data_ptr(), Ad.data_ptr(), bd.data_ptr(), X.data_ptr(),
                                               Y[3].data_ptr(), lc._lib.F32, small.data_ptr(), small.numel(),
                                               torch.cuda.current_stream().cuda_stream)
    assert st == lc._lib.OK
    torch.cuda.synchronize()
    assert all(torch.equal(Y[0].view(torch.int32), y.view(torch.int32)) for y in Y[1:3])
    rows = np.unique(np.concatenate([np.arange(min(m, 136)), np.arange(m // 2, m // 2 + 64) % m,
                                     np.arange(max(m - 136, 0), m)]))
    ref = orc.linear_forward_packed(P[rows], A.astype(np.float64), b.astype(np.float64), orc.widen(Xb, "bf16"), d, n)
    assert_close(to_host(Y[0])[:, rows], ref, 2e-2, "Y")
    assert_close(to_host(Y[3])[:, rows], ref, 2e-2, "Y unsplit")
