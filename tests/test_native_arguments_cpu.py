"""What the native entry points ask of their arguments, without a GPU: tensors that claim to be on one (fake tensors have no
memory).  A call whose arguments pass gets as far as the device and raises RuntimeError there."""
import pytest
import torch
from torch._subclasses.fake_tensor import FakeTensorMode

import paper_2310_19102_amd as atom

M, N, K, O, G = 4, 4, 1024, 128, 8                       # (as many channels as rows: stacks of both still agree in shape)
L = 3                                                       # layers of a stack


def fake(*shape, dtype=torch.uint8):
    with FakeTensorMode():
        return torch.empty(shape, dtype=dtype, device="cuda")


def codes(*lead):
    return [fake(*lead, (K - O) // 2), fake(*lead, O, dtype=torch.int8), fake(*lead, G, dtype=torch.float16)]


X = lambda: fake(M, K, dtype=torch.float16)
CALLS = {
    "w4a4_gemm": lambda a, w: atom.atom_w4a4_gemm(*a, *w, out=fake(M, N, dtype=torch.float16)),
    "w4a4_gemm_decode_tiled": lambda a, w: atom.atom_w4a4_gemm_decode_tiled(*a, *w, out=fake(M, N, dtype=torch.float16)),
    "decode_linear": lambda a, w: atom.atom_decode_linear(X(), None, 0.0, None, *w, out=fake(M, N, dtype=torch.float16)),
    "decode_linear_coop": lambda a, w: atom.atom_decode_linear_coop(
        X(), None, 0.0, None, *w, fake(1 << 16, dtype=torch.int32), out=fake(M, N, dtype=torch.float16), codes=codes(M)),
    "pack_act": lambda a, w: atom.atom_pack_act(*a, out=fake(1 << 20)),
    "w4a4_gemm_packed": lambda a, w: atom.atom_w4a4_gemm_packed(*a, fake(1 << 20), N, out=fake(M, N, dtype=torch.float16),
                                                                workspace=fake(1 << 20)),
}


@pytest.mark.filterwarnings("ignore:Accessing the data pointer")
@pytest.mark.parametrize("name", CALLS)
def test_stacked_operands_are_refused(name):
    """Codes with a layer dimension in front: their first two sizes are not rows and outliers."""
    with pytest.raises(RuntimeError):                       # the call as it should be goes on to the device
        CALLS[name](codes(M), codes(N))
    with pytest.raises(ValueError):
        CALLS[name](codes(L, M), codes(L, N))
    with pytest.raises((ValueError, IndexError)):           # nor are those of one dimension
        CALLS[name]([t[0] for t in codes(M)], [t[0] for t in codes(N)])
