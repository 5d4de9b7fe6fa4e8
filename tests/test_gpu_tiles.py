"""The codes products (forward, input gradient with its map gradients) on each of
their block tiles, at sizes where a tile can go wrong, against the oracle.

  * small tiles of 64 rows: one token, one step of K, ragged rows, columns and
    tokens, K not a multiple of the four waves' steps, long K;
  * small tiles of 128 rows (520 tokens, 2056 features: more than 256 tiles of 64
    rows, fewer of 128), ragged on every side;
  * wide tiles, ragged on every side (4000 tokens, 4040 x 4072: every tile of one
    round busy), on sampled rows;
  * the wide input gradient with K shorter than the 32 steps in which it fetches its X
    tile (1032 and 72 out-features), so that the rest comes behind the loop.

Each shape has to take the tiles it is there for (weight-side rows, forward and input
gradient).

Tolerance as everywhere for bf16: 2e-2 of the result, of every row and tile."""
import numpy as np
import pytest

import oracle as orc
import synth
from helpers import assert_close, product_tile, to_dev, to_host

pytestmark = pytest.mark.gpu

TOL = 2e-2


@pytest.fixture(scope="module")
def lc():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2606_10531_amd as lc
    lc._lib.load()
    return lc


SHAPES = [(1, 8, 64, 8, 64, 64), (64, 64, 64, 8, 64, 64), (65, 72, 328, 4, 64, 64), (200, 4104, 520, 8, 64, 64),
          (130, 136, 4616, 4, 64, 64), (17, 1032, 1160, 8, 64, 64), (520, 2056, 2056, 8, 128, 128),
          (520, 2056, 2056, 4, 128, 128), (4000, 4040, 4072, 4, 512, 256), (744, 1032, 11072, 8, 64, 256),
          (1232, 72, 5048, 4, 64, 256)]


@pytest.mark.parametrize("N,m,n,d,tile_fwd,tile_dx", SHAPES)
def test_products_on_every_tile(lc, N, m, n, d, tile_fwd, tile_dx):
    import torch
    assert (product_tile("fwd", N, m, n), product_tile("dx", N, m, n)) == (tile_fwd, tile_dx)
    print(f"\ntiles N={N} m={m} n={n} d={d}", flush=True)
    inp = synth.layer_inputs(N, m, n, d, "bf16", k=N + m + n + d, z_lo=-1.0, z_hi=4.0)
    Z, X, dY = (to_dev(inp[k], "bf16") for k in ("Z", "X", "dY"))
    A, b = torch.from_numpy(inp["A"]).cuda(), torch.from_numpy(inp["b"]).cuda()
    Y = torch.full((N, m), float("nan"), dtype=torch.bfloat16, device="cuda")
    dX = torch.full((N, n), float("nan"), dtype=torch.bfloat16, device="cuda")
    lc.linear_fwd(Z, A, b, X, d, out=Y)
    _, _, dA, db = lc.linear_bwd(Z, A, b, X, dY, d, dX=dX, need_dZ=False)
    dX2 = lc.linear_bwd(Z, A, b, X, dY, d, need_dZ=False, need_map=False)[0]
    torch.cuda.synchronize()
    assert torch.equal(dX.view(torch.int16), dX2.view(torch.int16))      # dX does not depend on the map gradients
    v = {k: orc.widen(inp[k], "bf16") for k in ("Z", "X", "dY")}
    A64, b64 = inp["A"].astype(np.float64), inp["b"].astype(np.float64)
    codes = orc.quantize(v["Z"])
    W = orc.decode(codes, A64, b64, d)
    tok = np.arange(N) if N <= 600 else np.unique(np.concatenate([np.arange(64), np.arange(N - 300, N)]))
    assert_close(to_host(Y)[tok], orc.forward(v["X"][tok], W), TOL, "Y")
    assert_close(to_host(dX)[tok], orc.grad_input(v["dY"][tok], W), TOL, "dX")
    dA_ref, db_ref = orc.grad_map(orc.grad_weight(v["dY"], v["X"]), codes, d)
    assert_close(to_host(dA), dA_ref, TOL, "dA")
    assert_close(to_host(db), db_ref, TOL, "db")
