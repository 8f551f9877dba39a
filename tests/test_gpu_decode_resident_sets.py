"""The decode GEMM that keeps the activations on 65 to 256 rows, in sets of 32, 48 and 64, and with more than 8192 channels: the bits that the same weights give a few thousand
channels at a time, and nothing written around the output."""
import ctypes

import pytest
import torch

import paper_2310_19102_amd as atom
from test_gpu_decode_resident import BORDER

pytestmark = pytest.mark.gpu

SLICE = 2048               # channels of a slice, for which the other kernel runs


def sets(M, N, K):
    rule = ctypes.CDLL(atom.binding._LIB_PATH).atom_internal_decode_resident_sets
    return bool(rule(ctypes.c_int64(M), ctypes.c_int64(N), K,
                     ctypes.c_int64(torch.cuda.get_device_properties(0).multi_processor_count)))


@pytest.mark.parametrize("K", [3840, 4096, 4864, 5120, 8192])    # one and three INT4 groups beside the INT8 group; one block of groups per wavefront, one or two, two
@pytest.mark.parametrize("M,N", [(65, 5480), (96, 8200), (97, 11001), (130, 8192), (150, 7003), (193, 5500), (256, 5501)])
def test_sets_of_rows(M, N, K):
    assert sets(M, N, K) and not sets(M, SLICE, K)
    _check(M, N, K)


def _check(M, N, K):
    print(f"[case] resident decode sets M={M} N={N} K={K}", flush=True)
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


@pytest.mark.parametrize("K", [8448, 8704, 9216, 11008, 12288])  # 66, 68, 72, 86 and 96 groups: two or three blocks of groups per wavefront, three
@pytest.mark.parametrize("M,N", [(17, 16400), (32, 16999), (33, 8208), (64, 9001), (96, 11001), (160, 8200)])
def test_three_blocks_of_groups(M, N, K):
    _check(M, N, K)


@pytest.mark.parametrize("K", [4352, 4864, 5120, 8192])
@pytest.mark.parametrize("M,N", [(33, 10300), (48, 11001), (40, 28672)])              # 33 to 48 rows in one set
def test_one_set_of_48_rows(M, N, K):
    _check(M, N, K)


@pytest.mark.parametrize("M,N,K", [(64, 22016, 4096), (257, 8192, 4096), (65, 4096, 4096), (256, 13824, 4096), (192, 13824, 5120), (128, 13824, 12544),
                                   (128, 13824, 3584)])
def test_other_side_of_the_rule(M, N, K):
    assert not sets(M, N, K)
