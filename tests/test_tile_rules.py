"""The product tiles that the rules pick where the measured times are far apart and a
model without the caches picks another one: operands beyond the 256 MB last-level cache,
on few (12000 tokens of 1040 x 20000) or many rows, next to shapes of few tiles that the
small tiles win by far.  Host arithmetic, no GPU."""
import pytest

from helpers import product_tile


@pytest.mark.parametrize("N,m,n,tile", [(12000, 1040, 20000, 256), (16000, 24120, 520, 256), (16000, 2064, 9000, 256),
                                        (4936, 1304, 28672, 256), (4096, 4096, 4096, 256), (512, 28672, 8192, 128),
                                        (1000, 11008, 4096, 128), (4096, 2048, 2048, 64), (16384, 1024, 2048, 64)])
def test_weight_gradient(N, m, n, tile):
    assert product_tile("dw", N, m, n) == tile


@pytest.mark.parametrize("N,m,n,tile", [(16000, 776, 16384, 512), (12000, 2064, 20000, 512), (4096, 4096, 4096, 512),
                                        (2048, 4096, 11008, 128), (1000, 11008, 4096, 128), (256, 4096, 4096, 64)])
def test_forward(N, m, n, tile):
    assert product_tile("fwd", N, m, n) == tile
