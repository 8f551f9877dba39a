"""The tiles of the packed GEMM (thin 64 x 64, 64 x 128, 128 x 128; walking 128 x 128, 256 x 128) at the edges of their ranges:
Y bit-identical to the kernel that dumps the integer sums (which tests/test_gpu_packed.py holds against
the oracle), and, on the small cases, to the oracle itself, and nothing written around the output."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2310_19102_amd as atom
from _gpu_util import gpu_quantize_act, gpu_quantize_weight, npy, ref_quantize_act, ref_quantize_weight
from test_gpu_parity import _rand_linear

pytestmark = pytest.mark.gpu

TILES = {0: "64x64", 1: "64x128", 2: "128x128", 3: "walk128x128", 4: "walk256x128", -1: "general"}
BORDER = 3                 # guard rows above and below Y, and guard columns left and right of it (an odd number: off the 16-byte grid)


def tile(M, N, K):
    pick = ctypes.CDLL(atom.binding._LIB_PATH).atom_internal_packed_tile
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return TILES[pick(ctypes.c_int64(M), ctypes.c_int64(N), K, 128, ctypes.c_int64(cus))]


@pytest.mark.parametrize("name,M,K,N", [
    ("64x64", 1, 1024, 64),              # one unit of either operand, seven INT4 groups (the fewest the tiles take)
    ("64x64", 64, 1152, 65),             # whole rows, a second column unit of one column; eight groups
    ("64x64", 33, 1280, 4090),           # nine groups, columns off the 16-byte grid
    ("64x64", 250, 1408, 4096),          # one workgroup per compute unit
    ("64x128", 65, 1536, 11008),         # a second row unit of one row
    ("64x128", 60, 1024, 16428),         # 257 column units: the last tile is moved back
    ("64x128", 320, 1152, 12288),        # five row units, two rounds of tiles
    ("128x128", 512, 1024, 4160),        # 65 column units: the last tile is moved back
    ("128x128", 192, 1152, 11008),       # three row units: the last tile is moved back
    ("128x128", 150, 1280, 10937),       # three row units and 171 column units, ragged both ways
    ("walk128x128", 384, 1152, 11008),   # two tiles more than compute units
    ("general", 150, 1024, 22016),       # three row units and more tiles than compute units
    ("walk128x128", 777, 1280, 13800),   # 13 row units, ragged both ways
    ("walk128x128", 1100, 1024, 16300),  # 255 column units, ragged last units
    ("walk128x128", 2304, 2176, 8200),   # sixteen groups, 129 column units, the last of eight columns
    ("walk256x128", 1700, 1024, 2870),   # 27 row units and 45 column units, ragged: moved back both ways
    ("walk256x128", 571, 1152, 7293),    # nine row units: the last tile is moved back by three of them
    ("walk256x128", 1728, 1280, 2880),   # the same, whole units: every store is unconditional
])
def test_tiles(name, M, K, N):
    assert tile(M, N, K) == name
    lin = _rand_linear(M, K, N, 128, seed=3 * M + N, norm=False)
    print(f"[case] packed tile {name} M={M} K={K} N={N}", flush=True)
    qa, qw = gpu_quantize_act(lin), gpu_quantize_weight(lin)
    wp = atom.atom_pack_weight(*qw, lin.group_size)
    part = torch.empty((M, N, K // 128), dtype=torch.int32, device="cuda")
    want = atom.atom_w4a4_gemm_packed(*qa, wp, N, lin.group_size, partials=part)
    del part
    assert torch.equal(atom.atom_w4a4_gemm_packed(*qa, wp, N, lin.group_size), want)
    ld = (BORDER + N + BORDER + 15) // 8 * 8                    # (rows of whole 16-byte pieces)
    for left in (BORDER, 8):                                    # Y off and on the 16-byte grid
        wide = torch.full((BORDER + M + BORDER, ld), 7.0, dtype=torch.float16, device="cuda")
        out = wide[BORDER:BORDER + M, left:left + N]
        atom.atom_w4a4_gemm_packed(*qa, wp, N, lin.group_size, out=out)
        assert torch.equal(out, want)
        out.fill_(7.0)
        assert bool((wide == 7.0).all()), "written outside the output"
    if M * N <= 1 << 18:
        ref = oracle.w4a4_gemm(*ref_quantize_act(lin), *ref_quantize_weight(lin), lin.group_size)
        assert np.array_equal(npy(want).view(np.uint16), ref["y"].view(np.uint16))
