"""The tiles of the MX GEMM at the edges of their ranges: Y against the exact sum of the decoded operands (sampled rows, all
columns) within the tolerance of tests/test_gpu_mx.py, with rows of Y on and off the 16-byte grid, and nothing
written around the output."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2310_19102_amd as atom
from test_gpu_mx import _allowed, _dequantise, _npy, _rand_linear, _row_major

pytestmark = pytest.mark.gpu

BORDER = 3                 # guard rows and columns around Y (an odd number: off the 16-byte grid)


def tile(M, N):
    pick = ctypes.CDLL(atom.binding._LIB_PATH).atom_internal_mx_tile
    t = pick(ctypes.c_int64(M), ctypes.c_int64(N),
             ctypes.c_int64(torch.cuda.get_device_properties(0).multi_processor_count))
    return f"{t // 1000}x{t % 1000}"


@pytest.mark.parametrize("name,M,K,N", [
    ("64x64", 1, 256, 1),                # one FP4 step behind two FP8 steps: fewer steps than stages
    ("64x64", 64, 384, 64),              # one whole tile
    ("64x64", 65, 640, 4095),            # a second row tile of one row, an odd row length
    ("64x64", 250, 1024, 4096),          # one workgroup per compute unit
    ("64x128", 448, 896, 4099),          # more steps than stages by three
    ("64x128", 1100, 256, 1003),         # fewer steps than stages
    ("128x128", 100, 512, 22010),        # up to one tile per compute unit: four stages
    ("128x128", 2000, 640, 9001),        # more: three stages; an odd row length
    ("128x256", 949, 384, 21551),
    ("128x256", 2049, 256, 15001),       # a last row tile of one row
    ("256x256", 4096, 512, 8192),        # whole tiles, two rounds
    ("256x256", 3257, 384, 4099),        # ragged both ways
    ("256x256", 3269, 384, 4099),        # ... and a last wavefront of five rows
])
def test_mx_tiles(name, M, K, N):
    assert tile(M, N) == name
    check(name, M, K, N)


@pytest.mark.parametrize("name,M,K,N", [
    ("256x320", 1024, 2048, 17000),      # the fewest channels of the wide kernel; a last column tile of 40
    ("256x320", 1793, 2176, 10001),      # a last row tile of one row, an odd row length
    ("256x384", 900, 2304, 22015),       # ragged both ways
    ("256x384", 2048, 2048, 12288),      # whole tiles, one per compute unit
    ("256x384", 2999, 2048, 13823),      # more than one per compute unit
])
def test_mx_wide_tiles(name, M, K, N):
    assert tile_k(M, N, K) == name
    check(name, M, K, N)


@pytest.mark.parametrize("name,M,K,N", [
    ("128x128", 3000, 2048, 11008), ("128x128", 1300, 2048, 13824), ("128x256", 3000, 2048, 12288), ("128x256", 1300, 5120, 28672)])
def test_mx_wide_tiles_have_to_be_ahead(name, M, K, N):
    """Cheaper per step, but behind with a prologue and a store to every round."""
    assert tile_k(M, N, K) == name


# the wide kernel's loop over FP8 steps beyond its first pair: four, six and thirty of them, the last with one FP4 step behind them
@pytest.mark.parametrize("O", [256, 384, 1920])
@pytest.mark.parametrize("name,M,K,N", [("256x320", 1024, 2048, 17000), ("256x384", 2048, 2048, 12280)])
def test_mx_wide_tiles_and_outliers(name, M, K, N, O):
    assert tile_k(M, N, K) == name
    check(name, M, K, N, O)


def tile_k(M, N, K):
    pick = ctypes.CDLL(atom.binding._LIB_PATH).atom_internal_mx_tile_k
    t = pick(ctypes.c_int64(M), ctypes.c_int64(N), ctypes.c_int32(K), ctypes.c_int64(torch.cuda.get_device_properties(0).multi_processor_count))
    return f"{t // 1000}x{t % 1000}"


def check(name, M, K, N, O=128):
    print(f"[case] mx tile {name} M={M} K={K} N={N}", flush=True)
    lin = _rand_linear(M, K, N, O, seed=M + N, norm=False)
    idx = lin.idx.cuda()
    ga = atom.atom_mx_quantize_act(lin.x.cuda(), None, 0.0, idx, O, 0.9)
    gw = atom.atom_mx_quantize_weight(lin.w.cuda(), idx, O, 0.85)
    y = atom.atom_mx_gemm(*ga, *gw)
    rows = np.unique(np.concatenate([np.arange(min(M, 20)), np.arange(max(0, M - 20), M),
                                     np.random.default_rng(M).choice(M, min(M, 24), replace=False)]))
    ra, rw = tuple(t[rows] for t in _row_major(ga)), _row_major(gw)
    ref = _dequantise(ra) @ _dequantise(rw).T
    err = float((np.abs(_npy(y)[rows].astype(np.float64) - ref) / _allowed(ref, ra, rw)).max())
    assert err <= 1.0, f"Y error {err} x the allowed"
    ld = (BORDER + N + BORDER + 15) // 8 * 8                    # (rows of whole 16-byte pieces)
    for left, width in ((BORDER, ld), (8, ld), (BORDER, ld + 1), (BORDER, ld + 2)):
        wide = torch.full((BORDER + M + BORDER, width), 7.0, dtype=torch.float16, device="cuda")
        out = wide[BORDER:BORDER + M, left:left + N]
        atom.atom_mx_gemm(*ga, *gw, out=out)
        assert torch.equal(out, y)
        out.fill_(7.0)
        assert bool((wide == 7.0).all()), "written outside the output"
