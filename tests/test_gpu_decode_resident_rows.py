"""The decode GEMM that keeps the activations, with all of 33 to 64 rows in one workgroup (three and four blocks of 16 rows) and with two sets of 32:
the bits that the same weights give a few thousand channels at a time, and nothing written around the output."""
import pytest
import torch

import paper_2310_19102_amd as atom
from test_gpu_decode_resident import BORDER, SLICE, resident

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [3840, 4096])                       # one INT4 group beside the INT8 group, three
@pytest.mark.parametrize("M", [33, 48, 49, 64])                   # a row block of one row and whole ones
@pytest.mark.parametrize("N", [10001, 16390, 20000])              # two sets; five blocks of channels to a workgroup, the last of six channels; whole blocks
def test_rows_of_a_workgroup(M, N, K):
    print(f"[case] resident decode rows M={M} N={N} K={K}", flush=True)
    assert resident(M, N, K)
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    idx = torch.randperm(K, generator=g, device="cuda").to(torch.int32)
    a = atom.atom_quantize_act(torch.randn((M, K), generator=g, device="cuda").half(), None, 0.0, idx)
    w = atom.atom_quantize_weight((0.02 * torch.randn((N, K), generator=g, device="cuda")).half(), idx)
    wide = torch.full((BORDER + M + BORDER, N + 2 * BORDER + 1), 7.0, dtype=torch.float16, device="cuda")
    out = wide[BORDER:BORDER + M, BORDER:BORDER + N]
    atom.atom_w4a4_gemm(*a, *w, out=out)
    for n in range(0, N, SLICE):
        part = atom.atom_w4a4_gemm(*a, *(t[n:n + SLICE].contiguous() for t in w))
        assert torch.equal(out[:, n:n + SLICE], part), n
    out.fill_(7.0)
    assert bool((wide == 7.0).all()), "written outside the output"
