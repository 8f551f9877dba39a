"""The halves of 32 columns of the MX GEMM's 64 x 64 tiles, at the edges of their ranges: as tests/test_gpu_mx_tiles.py checks a tile."""
import ctypes

import pytest
import torch

import paper_2310_19102_amd as atom
from test_gpu_mx_tiles import check, tile_k

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
    stages = ctypes.CDLL(atom.binding._LIB_PATH).atom_internal_mx_narrow_stages
    cus = ctypes.c_int64(torch.cuda.get_device_properties(0).multi_processor_count)
    assert tile_k(M, N, K) == "64x64"
    assert {0: "64x64", 6: "64x32, six stages", 8: "64x32, eight stages"}[stages(ctypes.c_int64(M), ctypes.c_int64(N), K, cus)] == name
    check(name, M, K, N, O)
