"""Decode GEMM where the blocks of four groups don't divide by the eight K-slices (8 n + 2 and 8 n + 4 of them: the slices are dealt to the wavefronts
out of order): each kernel, and its sets of workgroups, against the float64 sum of the integer sums of the groups, which the dumping kernel gives."""
import pytest
import torch

import paper_2310_19102_amd as atom

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1280, 4864, 5120, 5888, 6144, 9216, 10240])          # 3, 10, 10, 12, 12, 18, 20 blocks; one or three INT4 groups beside the INT8 group
@pytest.mark.parametrize("M,N", [(1, 300), (16, 4096), (8, 4112), (17, 300), (32, 8400), (33, 4200), (64, 8300),
                                 (40, 1000), (50, 2040), (200, 300)])         # sets of 16 and of 32 rows
def test_slices(M, N, K):
    print(f"[case] decode slices M={M} N={N} K={K}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    idx = torch.randperm(K, generator=g, device="cuda").to(torch.int32)
    a = atom.atom_quantize_act(torch.randn((M, K), generator=g, device="cuda").half(), None, 0.0, idx)
    w = atom.atom_quantize_weight((0.02 * torch.randn((N, K), generator=g, device="cuda")).half(), idx)
    part = torch.empty((M, N, K // 128), dtype=torch.int32, device="cuda")
    atom.atom_w4a4_gemm(*a, *w, partials=part)
    want, size = (torch.zeros((M, N), dtype=torch.float64, device="cuda") for _ in range(2))
    for i in range(K // 128):
        term = part[:, :, i].double() * a[2][:, i].double()[:, None] * w[2][:, i].double()[None, :]
        want += term
        size += term.abs()
    y = atom.atom_w4a4_gemm(*a, *w).double()
    # fp32 rounds each of the K / 128 multiply-adds and seven additions of slices by 2^-24 of a partial sum, at most `size`; fp16 the result by 2^-11
    bound = (K // 128 + 8) * 2.0 ** -24 * size + 2.0 ** -11 * want.abs() + 2.0 ** -25
    assert bool(((y - want).abs() <= bound).all())
