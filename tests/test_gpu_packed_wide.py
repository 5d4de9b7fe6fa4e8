"""The packed-codes forward for more than 16 tokens (one pass over the codes per
workspace of tokens), through the C ABI, against the oracle at 2e-2: tiles of 64 and
of 128 rows, ragged rows and tokens, K shorter than the four waves' steps and not a
multiple of a step, several passes (28672 in-features at 200 tokens with 8 MiB, 33000
tokens), both output
types.  The scratch-array call must give the same bits, and a workspace sized for
fewer tokens is still accepted (16-token passes)."""
import numpy as np
import pytest

import oracle as orc
import synth
from helpers import assert_close, to_dev, to_host

pytestmark = pytest.mark.gpu

TOL = 2e-2


@pytest.fixture(scope="module")
def lc():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2606_10531_amd as lc
    lc._lib.load()
    return lc


SHAPES = [(17, 8, 64, 8), (64, 72, 320, 4), (65, 200, 4160, 8), (130, 1032, 768, 4), (300, 4104, 512, 8),
          (200, 264, 28672, 8), (33000, 72, 64, 8)]


@pytest.mark.parametrize("y_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("N,m,n,d", SHAPES)
def test_packed_wide(lc, N, m, n, d, y_dtype):
    import torch
    print(f"\npacked wide N={N} m={m} n={n} d={d} {y_dtype}", flush=True)
    tdt = torch.bfloat16 if y_dtype == "bf16" else torch.float32
    r = synth.rng(N + m + n + d)
    P = r.integers(0, 256, size=(m, n // 4), dtype=np.uint8)
    Xb = synth.draw_activations(N, n, 7 + N, "bf16")
    A, b = synth.draw_map(d, 1)
    Pd, X = torch.from_numpy(P).cuda(), to_dev(Xb, "bf16")
    Ad, bd = torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda()
    need = lc.workspace_bytes(lc.OP_FWD_PACKED, N, m, n, d, torch.bfloat16)
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")       # NaN wherever nothing is written
    Y = torch.full((N, m), float("nan"), dtype=tdt, device="cuda")
    lc.linear_fwd_packed(Pd, Ad, bd, X, d, workspace=ws, out=Y)
    Y2 = torch.full((N, m), float("nan"), dtype=tdt, device="cuda")
    lc.linear_fwd_packed_noalloc(Pd, Ad, bd, X, d, out=Y2)
    torch.cuda.synchronize()
    ref = orc.linear_forward_packed(P, A.astype(np.float64), b.astype(np.float64), orc.widen(Xb, "bf16"), d, n)
    assert_close(to_host(Y), ref, TOL, "Y")
    assert np.array_equal(to_host(Y), to_host(Y2))


def test_packed_wide_with_a_workspace_for_few_tokens(lc):
    import torch
    N, m, n, d = 40, 200, 4160, 8
    small = lc.workspace_bytes(lc.OP_FWD_PACKED, 16, m, n, d, torch.bfloat16)
    assert small < lc.workspace_bytes(lc.OP_FWD_PACKED, N, m, n, d, torch.bfloat16)
    r = synth.rng(11)
    P = r.integers(0, 256, size=(m, n // 4), dtype=np.uint8)
    Xb = synth.draw_activations(N, n, 3, "bf16")
    A, b = synth.draw_map(d, 1)
    Pd, Ad, bd = (torch.from_numpy(x).cuda() for x in (P, A, b))
    Y = lc.linear_fwd_packed(Pd, Ad, bd, to_dev(Xb, "bf16"), d, out_dtype=torch.float32,
                             workspace=torch.empty(small, dtype=torch.uint8, device="cuda"))
    torch.cuda.synchronize()
    ref = orc.linear_forward_packed(P, A.astype(np.float64), b.astype(np.float64), orc.widen(Xb, "bf16"), d, n)
    assert_close(to_host(Y), ref, TOL, "Y")


@pytest.mark.parametrize("N,m,n,d,passes", [(17, 1088, 24000, 4, True), (32, 2048, 28672, 8, True), (20, 8192, 11008, 8, True),
                                            (33, 72, 40960, 4, True), (48, 8192, 28672, 8, False), (17, 264, 1088, 8, False),
                                            (65, 1088, 24000, 8, False)])
def test_few_tokens_and_rows_over_long_k(lc, N, m, n, d, passes):
    """Where wide tiles would leave the chip idle, more than 16 tokens go 16 at a time: the same
    bits as calls of up to 16 tokens; elsewhere the wide tiles' own."""
    import torch
    print(f"\npacked passes N={N} m={m} n={n} d={d}", flush=True)
    r = synth.rng(N + m + n + d)
    P = r.integers(0, 256, size=(m, n // 4), dtype=np.uint8)
    Xb = synth.draw_activations(N, n, 7 + N, "bf16")
    A, b = synth.draw_map(d, 1)
    Pd, X = torch.from_numpy(P).cuda(), to_dev(Xb, "bf16")
    Ad, bd = torch.from_numpy(A).cuda(), torch.from_numpy(b).cuda()
    Y = lc.linear_fwd_packed(Pd, Ad, bd, X, d, out_dtype=torch.float32)
    Y2 = torch.full((N, m), float("nan"), dtype=torch.float32, device="cuda")
    lc.linear_fwd_packed_noalloc(Pd, Ad, bd, X, d, out=Y2)
    parts = torch.cat([lc.linear_fwd_packed(Pd, Ad, bd, X[i:i + 16], d, out_dtype=torch.float32) for i in range(0, N, 16)])
    torch.cuda.synchronize()
    assert torch.equal(Y.view(torch.int32), Y2.view(torch.int32))
    assert torch.equal(Y.view(torch.int32), parts.view(torch.int32)) == passes
    rows = np.unique(np.concatenate([np.arange(min(m, 136)), np.arange(max(m - 136, 0), m)]))
    ref = orc.linear_forward_packed(P[rows], A.astype(np.float64), b.astype(np.float64), orc.widen(Xb, "bf16"), d, n)
    assert_close(to_host(Y)[:, rows], ref, TOL, "Y")
