"""The weight-gradient product on each of its tiles (128 x 64 with split tokens, 256 x
128, 256 x 256), ragged on every side, against the oracle on sampled out-feature rows:
both estimators, dZ in bf16 and fp32, overwritten and accumulated; each shape has to
take the tile it is there for; and the same bits
over repeated calls (the two larger tiles stage an operand through LDS with explicit
waits)."""
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


# out-features of the tile: 64, tokens split over the waves (one token, one step per wave,
# several); 128 with 4 steps of 64 tokens, where no LDS stage is refilled, and with 16; 256
# with 24 steps, about the fewest it is taken for, and with 64 (one full round of tiles)
SHAPES = [(1, 8, 8, 8, 64), (130, 72, 136, 4, 64), (600, 200, 392, 8, 64), (250, 4104, 4104, 8, 128),
          (1000, 4104, 4104, 4, 128), (1526, 28168, 264, 8, 256), (4000, 4040, 4072, 4, 256)]


@pytest.mark.parametrize("N,m,n,d,tile", SHAPES)
@pytest.mark.parametrize("est,dz,accumulate", [("ste", "bf16", False), ("ste", "f32", True), ("dge", "f32", False),
                                               ("dge", "bf16", True)])
def test_dw_on_every_tile(lc, N, m, n, d, tile, est, dz, accumulate):
    import torch
    assert product_tile("dw", N, m, n) == tile
    print(f"\ndw tiles N={N} m={m} n={n} d={d} {est} {dz} {accumulate}", flush=True)
    inp = synth.layer_inputs(N, m, n, d, "bf16", k=N + m + n + d, z_lo=-1.0, z_hi=4.0)
    Z, X, dY = (to_dev(inp[k], "bf16") for k in ("Z", "X", "dY"))
    A, b = torch.from_numpy(inp["A"]).cuda(), torch.from_numpy(inp["b"]).cuda()
    tdz = torch.bfloat16 if dz == "bf16" else torch.float32
    fn = lc.linear_bwd if est == "ste" else lc.linear_bwd_dge
    outs = []
    for _ in range(6):
        dZ = torch.full((m, n), 0.25 if accumulate else float("nan"), dtype=tdz, device="cuda")
        fn(Z, A, b, X, dY, d, mask_mode=lc.MASK_LATENT, accumulate=accumulate, need_dX=False, need_map=False, dz_dtype=tdz,
           dZ=dZ)
        outs.append(dZ)
    torch.cuda.synchronize()
    assert all(torch.equal(outs[0], o) for o in outs[1:])
    rows = np.arange(m) if m <= 400 else np.unique(np.concatenate([np.arange(64), np.arange(m // 2, m // 2 + 64),
                                                                   np.arange(m - 140, m)]))
    v = {k: orc.widen(inp[k], "bf16") for k in ("Z", "X", "dY")}
    mask = orc.ste_mask(v["Z"][rows], orc.MASK_LATENT)
    g = orc.grad_codes(orc.grad_weight(v["dY"][:, rows], v["X"]), inp["A"].astype(np.float64), d)
    if est == "dge":
        g = g * orc.dge_slope(v["Z"][rows], 5.0, 3.0)
    ref = np.where(mask, g, 0.0) + (0.25 if accumulate else 0.0)
    assert_close(to_host(outs[0])[rows], ref, TOL, "dZ")
