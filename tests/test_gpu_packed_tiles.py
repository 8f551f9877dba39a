"""The tiles of the packed GEMM (thin 64 x 64, 64 x 128, 128 x 128; walking 128 x 128, 256 x 128) at the edges of their ranges:
Y bit-identical to the kernel that dumps the integer sums (which tests/test_gpu_packed.py holds against
the oracle), and, on the small cases, to the oracle itself."""
import numpy as np
import pytest
import torch

import oracle
import paper_2310_19102_amd as atom
from _gpu_util import gpu_quantize_act, gpu_quantize_weight, npy, ref_quantize_act, ref_quantize_weight
from test_gpu_parity import _rand_linear

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,K,N", [
    (1, 1024, 64),         # one unit of either operand, seven INT4 groups (the fewest the tiles take)
    (64, 1152, 65),        # 64 x 64: whole rows, a second column unit of one column; eight groups
    (33, 1280, 4090),      # 64 x 64, nine groups, columns off the 16-byte grid
    (250, 1408, 4096),     # 64 x 64, one workgroup per compute unit
    (65, 1536, 11008),     # 64 x 128, a second row unit of one row
    (512, 1024, 4160),     # 64 x 128 with an odd number of column units: the last tile is moved back
    (320, 1152, 12288),    # 128 x 128, an odd number of row units
    (777, 1280, 13800),    # walking 128 x 128, ragged both ways
    (1100, 1024, 16300),   # walking 256 x 128: the last row tile is moved back by two units
    (2304, 2176, 8200),    # sixteen groups, a last column tile of eight columns
])
def test_tiles(M, K, N):
    lin = _rand_linear(M, K, N, 128, seed=3 * M + N, norm=False)
    print(f"[case] packed tiles M={M} K={K} N={N}", flush=True)
    qa, qw = gpu_quantize_act(lin), gpu_quantize_weight(lin)
    wp = atom.atom_pack_weight(*qw, lin.group_size)
    part = torch.empty((M, N, K // 128), dtype=torch.int32, device="cuda")
    want = atom.atom_w4a4_gemm_packed(*qa, wp, N, lin.group_size, partials=part)
    del part
    wide = torch.full((M, N + 24), 7.0, dtype=torch.float16, device="cuda")     # rows of Y with something behind them
    for out in (None, wide[:, :N], wide[:, 3:N + 3]):                            # (the last one off the 16-byte grid)
        y = atom.atom_w4a4_gemm_packed(*qa, wp, N, lin.group_size, out=out)
        torch.cuda.synchronize()
        assert torch.equal(y, want)
    assert bool((wide[:, N + 3:] == 7.0).all())
    if M * N <= 1 << 18:
        ref = oracle.w4a4_gemm(*ref_quantize_act(lin), *ref_quantize_weight(lin), lin.group_size)
        assert np.array_equal(npy(want).view(np.uint16), ref["y"].view(np.uint16))
