"""Rows of Y that start off the 16-byte grid (odd row lengths, views): the same bits as on the grid, and nothing written around
the output.  Canonical GEMM (128 x 128 tiles with one and two wavefront sets, 256 x 128 tiles), packed GEMM (general kernel:
two INT8 groups; its 64 x 64 tiles with few rows; the other tiles are in tests/test_gpu_packed_tiles.py)."""
import pytest
import torch

import paper_2310_19102_amd as atom
from _gpu_util import gpu_quantize_act, gpu_quantize_weight
from test_gpu_parity import _rand_linear

pytestmark = pytest.mark.gpu

BORDER = 3


@pytest.mark.parametrize("path,M,K,N,O", [
    ("canonical", 257, 256, 8193, 128),      # 128 x 128 tiles, two wavefront sets: last tiles of one row and one column
    ("canonical", 777, 384, 9003, 128),      # 128 x 128 tiles
    ("canonical", 2050, 256, 8201, 128),     # 256 x 128 tiles
    ("packed", 130, 640, 2059, 256),         # general kernel
    ("packed", 64, 512, 100, 256),
    ("packed", 8, 1024, 203, 128),           # 64 x 64 tiles: eight rows of a wavefront's 32, the most that are stored in one go
    ("packed", 9, 1024, 100, 128),           # ... and one more
    ("packed", 97, 1024, 1003, 128),         # last wavefronts of one row
    ("canonical", 265, 256, 8201, 128),      # 128 x 128 tiles: last wavefronts of nine rows
])
def test_row_starts(path, M, K, N, O):
    print(f"[case] row starts {path} M={M} K={K} N={N} O={O}", flush=True)
    lin = _rand_linear(M, K, N, O, seed=M + N, norm=False)
    qa, qw = gpu_quantize_act(lin), gpu_quantize_weight(lin)
    wp = atom.atom_pack_weight(*qw, lin.group_size) if path == "packed" else None

    def gemm(out):
        if path == "packed":
            return atom.atom_w4a4_gemm_packed(*qa, wp, N, lin.group_size, out=out)
        return atom.atom_w4a4_gemm(*qa, *qw, lin.group_size, out=out)

    ld = (N + 31) // 8 * 8
    want = gemm(torch.zeros((M, ld), dtype=torch.float16, device="cuda")[:, 8:8 + N]).clone()
    assert bool((want != 0).any())
    for left, width in ((BORDER, ld), (BORDER, ld + 1), (4, ld + 2), (7, ld + 4), (8, ld + 6)):
        wide = torch.full((BORDER + M + BORDER, width), 7.0, dtype=torch.float16, device="cuda")
        out = wide[BORDER:BORDER + M, left:left + N]
        gemm(out)
        assert torch.equal(out, want)
        out.fill_(7.0)
        assert bool((wide == 7.0).all()), "written outside the output"
