"""The halves of 32 columns of the MX GEMM's 64 x 64 tiles, at the edges of their ranges: as tests/test_gpu_mx_tiles.py checks a tile."""
import pytest

from test_gpu_mx_tiles import check, tile

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,M,K,N,O", [
    ("64x32, six stages", 1, 256, 33, 128),              # fewer steps than stages; a second tile of one column
    ("64x32, six stages", 65, 768, 4090, 128),
    ("64x32, six stages", 128, 4096, 4096, 128),         # one workgroup per compute unit
    ("64x32, six stages", 300, 1024, 1500, 512),         # more FP8 steps than stages
    ("64x32, eight stages", 64, 4224, 8181, 128),
    ("64x32, eight stages", 500, 4352, 970, 128),
    ("64x64", 130, 640, 4095, 128),
    ("64x64", 1664, 640, 1190, 128),                     # two to a compute unit
])
def test_mx_narrow_tiles(name, M, K, N, O):
    t64 = ((M + 63) // 64) * ((N + 63) // 64)
    assert name.split(",")[0] == ("64x32" if 2 * t64 <= 256 else "64x64")
    assert tile(M, N) == "64x64"
    check(name, M, K, N, O)
