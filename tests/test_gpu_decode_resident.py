"""Decode GEMMs with many blocks of output channels per compute unit (17 to 64 rows, canonical weights): the kernel that keeps the
activations in registers gives the bits that the same weights give a few thousand channels at a time, where the kernels for fewer
channels run (those are compared with the oracle elsewhere)."""
import pytest
import torch

import paper_2310_19102_amd as atom

pytestmark = pytest.mark.gpu


# K: 30, 32, 38 and 64 groups (an INT8 group beside one or three INT4 groups; one block of four groups per wavefront, one or two, two)
@pytest.mark.parametrize("K", [3840, 4096, 4864, 8192])
# the first N past the line and one with a ragged last block; both sides of one and two sets of 32 rows
@pytest.mark.parametrize("M,N", [(17, 16400), (32, 17003), (33, 8208), (64, 8999)])
def test_resident_decode_equals_slices(M, N, K):
    print(f"[case] resident decode M={M} N={N} K={K}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    idx = torch.randperm(K, generator=g, device="cuda").to(torch.int32)
    a = atom.atom_quantize_act(torch.randn((M, K), generator=g, device="cuda").half(), None, 0.0, idx)
    w = atom.atom_quantize_weight((0.02 * torch.randn((N, K), generator=g, device="cuda")).half(), idx)
    y = atom.atom_w4a4_gemm(*a, *w)
    for n in range(0, N, 4096):
        part = atom.atom_w4a4_gemm(*a, *(t[n:n + 4096].contiguous() for t in w))
        assert torch.equal(y[:, n:n + 4096], part), n
