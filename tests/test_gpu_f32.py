"""The fp32 products on both of their tiles (64 and 32 columns) and both row moves
(m a multiple of 4 or not), at tile remainders, one token, K shorter than a chunk
and K not a multiple of it, through the C ABI against the oracle: 1e-5 relative
Frobenius error of the whole result, of every row and every tile."""
import numpy as np
import pytest

import oracle as orc
import synth
from helpers import assert_close, to_dev, to_host

pytestmark = pytest.mark.gpu

TOL = 1e-5


@pytest.fixture(scope="module")
def lc():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2606_10531_amd as lc
    lc._lib.load()
    return lc


# the last: 528 or more tiles of 64 columns in every product
SHAPES = [(1, 1, 4, 4), (3, 2, 8, 8), (70, 33, 40, 8), (33, 158, 1684, 4), (65, 67, 72, 8), (500, 132, 260, 4),
          (1000, 1030, 1032, 8)]


@pytest.mark.parametrize("N,m,n,d", SHAPES)
@pytest.mark.parametrize("variant", ["ste", "dge_accumulate"])
def test_f32_layer(lc, N, m, n, d, variant):
    import torch
    print(f"\nf32 N={N} m={m} n={n} d={d} {variant}", flush=True)
    inp = synth.layer_inputs(N, m, n, d, "f32", k=N + m + n + d, z_lo=-1.0, z_hi=4.0)
    Z, X, dY, A, b = (to_dev(inp[k], "f32") for k in ("Z", "X", "dY", "A", "b"))
    Y = lc.linear_fwd(Z, A, b, X, d)
    v = {k: inp[k].astype(np.float64) for k in ("Z", "X", "dY", "A", "b")}
    Yref, _ = orc.linear_forward(v["Z"], v["A"], v["b"], v["X"], d)
    assert_close(to_host(Y), Yref, TOL, "Y")
    if variant == "ste":
        got = dict(zip(("dX", "dZ", "dA", "db"), lc.linear_bwd(Z, A, b, X, dY, d)))
        ref = orc.linear_backward(v["Z"], v["A"], v["b"], v["X"], v["dY"], d)
    else:
        g0 = [torch.full(s, 0.5, device="cuda") for s in ((m, n), (d, d), (d,))]
        got = dict(zip(("dX", "dZ", "dA", "db"), lc.linear_bwd_dge(
            Z, A, b, X, dY, d, k=5.0, cap=3.0, accumulate=True, dZ=g0[0], dA=g0[1], db=g0[2])))
        ref = orc.linear_backward(v["Z"], v["A"], v["b"], v["X"], v["dY"], d, mask_mode=orc.MASK_LATENT, dge=(5.0, 3.0))
        for key in ("dZ", "dA", "db"):
            ref[key] = ref[key] + 0.5
    torch.cuda.synchronize()
    for key in ("dX", "dZ", "dA", "db"):
        assert_close(to_host(got[key]), ref[key], TOL, key)


def test_f32_rows_past_the_buffer_offsets(lc):
    """Rows of 2^22 floats take the loads with 64-bit addresses.  Only the results with
    short sums are compared: dX and dZ where the in-features are that many, Y where
    the out-features are."""
    import torch
    for N, m, n in ((2, 3, 1 << 22), (2, 1 << 22, 8)):
        print(f"\nf32 N={N} m={m} n={n}", flush=True)
        inp = synth.layer_inputs(N, m, n, 8, "f32", k=5, z_lo=-1.0, z_hi=4.0)
        Z, X, dY, A, b = (to_dev(inp[k], "f32") for k in ("Z", "X", "dY", "A", "b"))
        v = {k: inp[k].astype(np.float64) for k in ("Z", "X", "dY", "A", "b")}
        W = orc.decode(orc.quantize(v["Z"]), v["A"], v["b"], 8)
        if n == 8:
            assert_close(to_host(lc.linear_fwd(Z, A, b, X, 8)), orc.forward(v["X"], W), TOL, "Y")
        else:
            dX, dZ, _, _ = lc.linear_bwd(Z, A, b, X, dY, 8, need_map=False)
            assert_close(to_host(dX), orc.grad_input(v["dY"], W), TOL, "dX")
            assert_close(to_host(dZ), orc.grad_latent(orc.grad_weight(v["dY"], v["X"]), v["A"], 8,
                                                      orc.ste_mask(v["Z"])), TOL, "dZ")


def test_f32_output_of_more_tiles_than_one_grid_row(lc):
    """2^35 outputs and more: the tiles' threads pass 2^32, the most of one grid dimension."""
    import torch
    N, m, n, d = 4194048, 8200, 8, 8
    print(f"\nf32 N={N} m={m} n={n}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(3)
    Z = torch.empty((m, n), device="cuda").uniform_(-1.0, 4.0, generator=g)
    X = torch.randn((N, n), device="cuda", generator=g)
    A = 0.02 * (torch.eye(d, device="cuda") + 0.1 * torch.randn((d, d), device="cuda", generator=g))
    b = 0.005 * torch.randn((d,), device="cuda", generator=g)
    Y = torch.empty((N, m), device="cuda")
    Y[-1] = float("nan")
    lc.linear_fwd(Z, A, b, X, d, out=Y)
    torch.cuda.synchronize()
    rows = torch.cat([torch.arange(64), torch.arange(N // 2, N // 2 + 64), torch.arange(N - 300, N)])
    W = orc.decode(orc.quantize(to_host(Z)), to_host(A), to_host(b), d)
    got, ref = to_host(Y[rows.cuda()]), orc.forward(to_host(X[rows.cuda()]), W)
    del Y
    torch.cuda.empty_cache()
    assert_close(got, ref, TOL, "Y")
