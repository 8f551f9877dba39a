"""Argument forms of the native entry points: result tensors given by an iterator, a second operand of the packed
front ends with more rows than the first, and a tensor without memory (its address raises inside the call)."""
import pytest
import torch

import paper_2310_19102_amd as atom

pytestmark = pytest.mark.gpu

M, K = 5, 1024


def _inputs():
    g = torch.Generator(device="cuda").manual_seed(3)
    x, r = (torch.randn((n, K), generator=g, device="cuda").to(torch.float16) for n in (M, M + 3))
    return x, r, torch.ones(K, dtype=torch.float16, device="cuda"), torch.randperm(K, generator=g, device="cuda").to(torch.int32)


def test_results_given_by_an_iterator():
    x, _, gamma, idx = _inputs()
    want = atom.atom_quantize_act(x, gamma, 1e-5, idx)
    got = atom.atom_quantize_act(x, gamma, 1e-5, idx, out=(torch.full_like(t, 7) for t in want))
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(got, want))


def test_packed_front_ends_take_a_longer_second_operand():
    x, r, gamma, idx = _inputs()
    h, p = atom.atom_add_quantize_act_packed(x, r, gamma, 1e-5, idx)
    h0, p0 = atom.atom_add_quantize_act_packed(x, r[:M], gamma, 1e-5, idx)
    s, s0 = (atom.atom_swiglu_quantize_act_packed(x, u, idx) for u in (r, r[:M]))
    torch.cuda.synchronize()
    assert torch.equal(h, h0) and torch.equal(p, p0) and torch.equal(s, s0)


def test_a_tensor_without_memory_raises():
    x, _, gamma, idx = _inputs()
    with pytest.raises(RuntimeError):
        atom.atom_quantize_act(torch._to_functional_tensor(x), gamma, 1e-5, idx)
    want = atom.atom_quantize_act(x, gamma, 1e-5, idx)          # the interpreter goes on
    assert want[0].shape == (M, (K - 128) // 2)
