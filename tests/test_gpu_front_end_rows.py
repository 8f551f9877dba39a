"""The front ends' row routine where it can go wrong: threads past the end of a row, which load its last vector again; several rows to
a workgroup; reorder offsets of two channels in one register; groups whose scale is zero beside ordinary ones."""
import numpy as np
import pytest
import torch

import oracle
import paper_2310_19102_amd as atom
from _gpu_util import npy

pytestmark = pytest.mark.gpu


def _rows(M, K, seed):
    rng = np.random.default_rng(seed)
    x = (rng.standard_normal((M, K)) * np.exp(1.5 * rng.standard_normal(K))).astype(np.float16)
    idx = rng.permutation(K).astype(np.int32)
    x[0, idx[:128]] = 0.0                                    # a group of zeros, one whose scale rounds to zero,
    x[0, idx[128:256]] = np.float16(5.97e-8) * (rng.integers(0, 2, 128) * 2 - 1)
    x[1, idx[256]] = 65504.0
    x[2, idx[K - 128:]] = 0.0                                # outliers of zero
    return x, idx


@pytest.mark.parametrize("M,K", [(5, 4224), (5, 4992), (70, 5120), (5, 8064),       # 640 and 1024 threads, most, all and some of them
                                 (1100, 4992), (1100, 7168), (2100, 3968),         # 320, 512 and 256 threads, several rows each
                                 (800, 11008), (800, 12416), (800, 16384),         # three and four sweeps
                                 (1100, 9216), (1100, 13824)])                     # the same, several rows each also in order
def test_rows(M, K):
    print(f"[case] front end rows M={M} K={K}", flush=True)
    x, idx = _rows(M, K, M + K)
    some = sorted({0, 1, 2, 3, M // 2, M - 2, M - 1})        # (the oracle is one thread)
    dx, di = torch.from_numpy(x).cuda(), torch.from_numpy(idx).cuda()
    up = torch.from_numpy(x[::-1].copy()).cuda()
    gamma = torch.linspace(0.5, 2.0, K, device="cuda").half()

    def same(got, want, what):
        for name, a, b in zip(("q4", "q8", "scale"), got, want):
            assert np.array_equal(npy(a[some]).view(np.uint8), b.view(np.uint8)), f"{what}: {name}"

    plain = atom.atom_quantize_act(dx, None, 0.0, di)
    same(plain, oracle.quantize_act(x[some], None, 0.0, idx, 128, 128, 0.9), "plain")
    order = atom.atom_quantize_act(dx[:, di.long()].contiguous(), None, 0.0, None)
    assert all(torch.equal(a, b) for a, b in zip(plain, order))
    packed = atom.atom_quantize_act_packed(dx, None, 0.0, di)
    assert torch.equal(packed, atom.atom_pack_act(*plain))

    norm = atom.atom_quantize_act(dx, gamma, 1e-6, di)
    same(norm, oracle.quantize_act(x[some], npy(gamma), 1e-6, idx, 128, 128, 0.9), "norm")
    assert torch.equal(atom.atom_quantize_act_packed(dx, gamma, 1e-6, di), atom.atom_pack_act(*norm))

    h, *added = atom.atom_add_quantize_act(dx, up, gamma, 1e-6, di)
    same(added, oracle.quantize_act(npy(h[some]), npy(gamma), 1e-6, idx, 128, 128, 0.9), "add")
    h2, packed = atom.atom_add_quantize_act_packed(dx, up, gamma, 1e-6, di)
    assert torch.equal(h, h2) and torch.equal(packed, atom.atom_pack_act(*added))

    ordered = [t[..., di.long()].contiguous() for t in (dx, up, gamma, h)]
    norm_order = atom.atom_quantize_act(ordered[0], ordered[2], 1e-6, None)
    ho, *added_order = atom.atom_add_quantize_act(*ordered[:3], 1e-6, None)
    assert torch.equal(ho, ordered[3])
    ho, packed = atom.atom_add_quantize_act_packed(*ordered[:3], 1e-6, None)
    assert torch.equal(ho, ordered[3]) and torch.equal(packed, atom.atom_pack_act(*added_order))
    assert torch.equal(atom.atom_quantize_act_packed(ordered[0], ordered[2], 1e-6, None), atom.atom_pack_act(*norm_order))
    identity = np.arange(K, dtype=np.int32)                  # (the sum of squares of a row in another order is another sum)
    same(norm_order, oracle.quantize_act(npy(ordered[0][some]), npy(ordered[2]), 1e-6, identity, 128, 128, 0.9), "norm, in order")
    same(added_order, oracle.quantize_act(npy(ho[some]), npy(ordered[2]), 1e-6, identity, 128, 128, 0.9), "add, in order")

    glu = atom.atom_swiglu_quantize_act(dx, up, di)
    same(glu, oracle.swiglu_quantize_act(x[some], x[::-1][some], idx, 128, 128, 0.9), "SwiGLU")
    assert torch.equal(atom.atom_swiglu_quantize_act_packed(dx, up, di), atom.atom_pack_act(*glu))


@pytest.mark.parametrize("M", [1, 2])                    # 1024 (in order with a norm 512) and 640 threads
@pytest.mark.parametrize("K", [4224, 5120])
def test_packed_rows_of_a_few(M, K):
    print(f"[case] packed front end M={M} K={K}", flush=True)
    x, idx = _rows(3, K, M + K)
    dx, up, gamma = torch.from_numpy(x[:M]).cuda(), torch.from_numpy(x[3 - M:]).cuda(), torch.linspace(0.5, 2.0, K, device="cuda").half()
    for di in (torch.from_numpy(idx).cuda(), None):
        for g in (None, gamma):
            assert torch.equal(atom.atom_quantize_act_packed(dx, g, 1e-6, di), atom.atom_pack_act(*atom.atom_quantize_act(dx, g, 1e-6, di)))
        assert torch.equal(atom.atom_add_quantize_act_packed(dx, up, gamma, 1e-6, di)[1], atom.atom_pack_act(*atom.atom_add_quantize_act(dx, up, gamma, 1e-6, di)[1:]))
        assert torch.equal(atom.atom_swiglu_quantize_act_packed(dx, up, di), atom.atom_pack_act(*atom.atom_swiglu_quantize_act(dx, up, di)))


def _halves_of(denom):
    """Pairs of fp16 factors (the first in [32, 64), where silu is the identity) whose product is denom * t / 2 by a power of two, t odd
    and of twelve bits: with clip 1 the scale lies in the middle between two fp16 numbers."""
    pairs = []
    for t in range(2049, 4096, 2):
        p = next((p for p in range(3, 2048 // denom + 1, 2) if t % p == 0 and t // p < 2048), None)
        if p:
            g = denom * p
            pairs.append((g * 2.0 ** (6 - g.bit_length()), t // p * 2.0 ** -11))
    return pairs


@pytest.mark.parametrize("bits", [4, 3])
def test_scales_between_two_numbers(bits):
    inner, outer = _halves_of(15 if bits == 4 else 7), _halves_of(255)
    G, K = 128, 128 * 128
    rows = min(len(outer), -(-len(inner) // (G - 1)))
    gate, up = np.full((rows, G, 128), 32.0, np.float16), np.zeros((rows, G, 128), np.float16)
    for i, (a, b) in enumerate(inner[:rows * (G - 1)]):
        gate[i // (G - 1), i % (G - 1), i % 128], up[i // (G - 1), i % (G - 1), i % 128] = a, b
    for i, (a, b) in enumerate(outer[:rows]):
        gate[i, G - 1, 9], up[i, G - 1, 9] = a, b
    gate, up = gate.reshape(rows, K), up.reshape(rows, K)
    want = oracle.swiglu_quantize_act(gate, up, np.arange(K, dtype=np.int32), 128, 128, 1.0, bits=bits)
    assert np.array_equal(want[2][0, :3], np.float16([2 * a * b / (15 if bits == 4 else 7) for a, b in inner[:3]]))
    got = atom.atom_swiglu_quantize_act(torch.from_numpy(gate).cuda(), torch.from_numpy(up).cuda(), None, clip=1.0, bits=bits)
    for name, a, b in zip(("q4", "q8", "scale"), got, want):
        assert np.array_equal(npy(a).view(np.uint8), b.view(np.uint8)), name
