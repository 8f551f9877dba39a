"""The packed GEMM's small launches by the columns of their tile and the stages of its pipeline (64 x 32 and 64 x 64 with six, 64 x 64
and 64 x 96 with four) at the edges of their ranges: Y bit-identical to the kernel that dumps the integer sums (which
tests/test_gpu_packed.py holds against the oracle), and nothing written around the output."""
import pytest
import torch

import paper_2310_19102_amd as atom
from _gpu_util import gpu_quantize_act, gpu_quantize_weight
from test_gpu_parity import _rand_linear

pytestmark = pytest.mark.gpu

BORDER = 3                 # guard rows above and below Y, and guard columns left and right of it (an odd number: off the 16-byte grid)


@pytest.mark.parametrize("columns,M,G4,N", [
    (32, 1, 15, 40),             # one unit of either operand, the second tile nearly empty; the fewest groups of six stages
    (32, 65, 16, 1000),          # the last unit's upper half all past the end
    (32, 64, 17, 8192),          # a tile for each of 256 compute units
    (32, 130, 18, 2090),
    (32, 200, 19, 777),
    (32, 128, 20, 4096),
    (64, 250, 48, 4090),         # six stages: every remainder of the groups
    (64, 65, 49, 5000),
    (64, 700, 50, 1403),
    (64, 64, 51, 16380),
    (64, 128, 52, 4100),
    (64, 192, 47, 5120),
    (64, 256, 14, 2000),         # four stages
    (64, 256, 46, 4096),
    (96, 70, 31, 8300),          # 130 column units: the last tile is moved back by a half unit
    (96, 128, 32, 9000),         # 141: whole tiles
    (96, 300, 33, 4100),         # 65: moved back by two half units of three
    (96, 320, 34, 4096),
    (128, 60, 10, 16576),        # four stages of 64 x 128
])
def test_thin_columns(columns, M, G4, N):
    K = 128 * (G4 + 1)
    lin = _rand_linear(M, K, N, 128, seed=M + N, norm=False)
    print(f"[case] packed thin tile 64x{columns} M={M} K={K} N={N}", flush=True)
    qa, qw = gpu_quantize_act(lin), gpu_quantize_weight(lin)
    wp = atom.atom_pack_weight(*qw, lin.group_size)
    part = torch.empty((M, N, K // 128), dtype=torch.int32, device="cuda")
    want = atom.atom_w4a4_gemm_packed(*qa, wp, N, lin.group_size, partials=part)
    del part
    ld = (BORDER + N + BORDER + 15) // 8 * 8                    # (rows of whole 16-byte pieces)
    for left in (BORDER, 8):                                    # Y off and on the 16-byte grid
        wide = torch.full((BORDER + M + BORDER, ld), 7.0, dtype=torch.float16, device="cuda")
        out = wide[BORDER:BORDER + M, left:left + N]
        atom.atom_w4a4_gemm_packed(*qa, wp, N, lin.group_size, out=out)
        assert torch.equal(out, want)
        out.fill_(7.0)
        assert bool((wide == 7.0).all()), "written outside the output"
