"""Decode GEMMs with many blocks of output channels per compute unit (17 to 64 rows, canonical weights): the kernel that keeps the
activations in registers gives the bits that the same weights give a few thousand channels at a time, where the kernels for fewer
channels run (those are compared with the oracle elsewhere), and writes nothing around the output."""
import ctypes

import pytest
import torch

import paper_2310_19102_amd as atom

pytestmark = pytest.mark.gpu

SLICE = 4096               # channels of a slice
BORDER = 3                 # guard rows and columns around Y


def resident(M, N, K):
    rule = ctypes.CDLL(atom.binding._LIB_PATH).atom_internal_decode_resident
    return bool(rule(ctypes.c_int64(M), ctypes.c_int64(N), K,
                     ctypes.c_int64(torch.cuda.get_device_properties(0).multi_processor_count)))


# K: 30, 32, 34, 38 and 64 groups (an INT8 group beside one or three INT4 groups; one block of four groups per wavefront, one or two
# (34: two for the last wavefront alone), two)
@pytest.mark.parametrize("K", [3840, 4096, 4352, 4864, 8192])
# the first N past the line and one with a ragged last block; both sides of one and two sets of 32 rows
@pytest.mark.parametrize("M,N", [(17, 16400), (32, 17003), (33, 8208), (63, 9001), (64, 8999)])
def test_resident_decode_equals_slices(M, N, K):
    print(f"[case] resident decode M={M} N={N} K={K}", flush=True)
    assert resident(M, N, K) and not resident(M, SLICE, K)
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    idx = torch.randperm(K, generator=g, device="cuda").to(torch.int32)
    a = atom.atom_quantize_act(torch.randn((M, K), generator=g, device="cuda").half(), None, 0.0, idx)
    w = atom.atom_quantize_weight((0.02 * torch.randn((N, K), generator=g, device="cuda")).half(), idx)
    y = atom.atom_w4a4_gemm(*a, *w)
    for n in range(0, N, SLICE):
        part = atom.atom_w4a4_gemm(*a, *(t[n:n + SLICE].contiguous() for t in w))
        assert torch.equal(y[:, n:n + SLICE], part), n
    wide = torch.full((BORDER + M + BORDER, N + 2 * BORDER + 1), 7.0, dtype=torch.float16, device="cuda")
    out = wide[BORDER:BORDER + M, BORDER:BORDER + N]
    atom.atom_w4a4_gemm(*a, *w, out=out)
    assert torch.equal(out, y)
    out.fill_(7.0)
    assert bool((wide == 7.0).all()), "written outside the output"


@pytest.mark.parametrize("M,N,K", [(16, 57344, 4096), (65, 57344, 4096), (32, 16384, 4096), (33, 8192, 4096), (32, 57344, 3584),
                                   (32, 57344, 8448)])
def test_other_side_of_the_rule(M, N, K):
    assert not resident(M, N, K)
