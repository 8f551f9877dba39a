"""What the native entry points ask of their arguments, without a GPU: tensors that claim to be on one (fake tensors have no
memory).  A call whose arguments pass gets as far as the device and raises RuntimeError there."""
import weakref

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


@pytest.mark.filterwarnings("ignore:Accessing the data pointer")
@pytest.mark.parametrize("static", [False, True])
def test_tensors_of_a_list_are_held_through_the_call(static):
    """A cache given as a list that changes while the call goes on (here in the conversion of a later argument, elsewhere in
    another thread): the call keeps the tensors it was given."""
    B, H, D, T = 2, 4, 128, 64
    cache = [[fake(B, H, T, D // 2), fake(B, H, T, dtype=torch.float16), fake(B, H, T, dtype=torch.int16)] for _ in "kv"]
    held = [weakref.ref(t) for c in cache for t in c]
    alive = []

    class Scale:
        def __float__(self):
            for c in cache:
                c[:] = [None] * 3
            alive.extend(r() is not None for r in held)
            raise ArithmeticError("seen")                   # (nothing is read after this)

    call = atom.atom_decode_attention_kv4_static if static else atom.atom_decode_attention_kv4
    with pytest.raises(ArithmeticError):
        call(fake(B, H, D, dtype=torch.float16), *cache, fake(B, dtype=torch.int32), Scale(),
             out=fake(B, H, D, dtype=torch.float16))
    assert alive == [True] * 6
    assert not any(r() is not None for r in held)           # and lets them go


@pytest.mark.filterwarnings("ignore:Accessing the data pointer")
@pytest.mark.parametrize("rows,shape,taken", [
    (1, (K,), True), (1, (1, 1, K), True), (1, (2, K), True), (1, (8, K // 4), True), (4, (4, K), True), (4, (5, K + 128), True),
    (4, (4, 1, K), True), (4, (4, 2, K), True), (1, (K - 128,), False), (4, (K,), False), (4, (4 * K,), False),
    (4, (1, 4, K), False), (4, (4, K - 128), False), (4, (3, K), False), (1, (), False)])
def test_second_operand_of_the_packed_front_ends(rows, shape, taken):
    """Anything that holds the rows at its first stride is taken; what would be read past its end is refused."""
    x, r = (fake(*s, dtype=torch.float16) for s in ((rows, K), shape))
    out = fake(1 << 20)
    for call in (lambda: atom.atom_add_quantize_act_packed(x, r, None, 0.0, None, sum_out=fake(rows, K, dtype=torch.float16), out=out),
                 lambda: atom.atom_swiglu_quantize_act_packed(x, r, None, out=out)):
        with pytest.raises(RuntimeError if taken else ValueError):
            call()


@pytest.mark.filterwarnings("ignore:Accessing the data pointer")
def test_codes_of_the_cooperative_linear_are_taken_by_index():
    """The first three of whatever can be indexed."""
    y, sync = fake(M, N, dtype=torch.float16), fake(1 << 16, dtype=torch.int32)
    for given, error in ((codes(M) + [None], RuntimeError), (dict(enumerate(codes(M))), RuntimeError), (codes(M)[:2], IndexError)):
        with pytest.raises(error):
            atom.atom_decode_linear_coop(X(), None, 0.0, None, *codes(N), sync, out=y, codes=given)
