"""The wide tiles of the packed GEMM (256 x 192, 128 x 384, 256 x 256) and those of 192 rows at the edges of their ranges: Y bit-identical to the kernel
that dumps the integer sums (which tests/test_gpu_packed.py holds against the oracle), and nothing written around the output."""
import ctypes

import pytest
import torch

import paper_2310_19102_amd as atom
from _gpu_util import gpu_quantize_act, gpu_quantize_weight
from test_gpu_parity import _rand_linear

pytestmark = pytest.mark.gpu

TILES = {5: "256x192", 6: "128x384", 7: "256x256", 8: "192x128"}
BORDER = 3                 # guard rows above and below Y, and guard columns left and right of it (an odd number: off the 16-byte grid)


@pytest.mark.parametrize("name,M,G4,N", [
    ("256x192", 449, 21, 16688),         # one round, whole units of tiles
    ("256x192", 385, 20, 16519),         # moved back both ways, ragged
    ("256x192", 965, 22, 20623),         # two rounds, the last columns cut inside a half unit
    ("256x192", 911, 20, 20512),         # two rounds, columns end on a block of 32, rows moved back
    ("128x384", 321, 21, 21877),
    ("128x384", 257, 20, 21804),         # three tiles of rows for 4.02 units
    ("128x384", 833, 22, 23374),         # two rounds
    ("128x384", 772, 20, 23324),         # two rounds, moved back both ways
    ("256x256", 706, 22, 16611),
    ("256x256", 515, 20, 19595),         # moved back both ways
    ("256x256", 1218, 21, 19666),        # two rounds
    ("256x256", 1028, 20, 21706),        # two rounds, moved back by three units of rows
    ("192x128", 150, 17, 22001),         # one tile of rows, ragged; the fewest groups
    ("192x128", 192, 19, 22050),         # whole rows; an odd number of column units
    ("192x128", 290, 21, 13851),         # moved back both ways
    ("192x128", 321, 20, 12300),
    ("192x128", 190, 18, 57000),         # two rounds
    ("192x128", 515, 22, 8200),          # 129 column units, moved back both ways
])
def test_wide_tiles(name, M, G4, N):
    K = 128 * (G4 + 1)
    pick = ctypes.CDLL(atom.binding._LIB_PATH).atom_internal_packed_tile
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert TILES[pick(ctypes.c_int64(M), ctypes.c_int64(N), K, 128, ctypes.c_int64(cus))] == name
    lin = _rand_linear(M, K, N, 128, seed=M + N, norm=False)
    print(f"[case] packed wide tile {name} M={M} K={K} N={N}", flush=True)
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
