"""The front ends at the edges of their thread configurations (up to one row per compute unit: twice the threads; 5120
channels: 320 threads), the SwiGLU front end on every finite fp16 gate, and the MX front end on every thread configuration:
codes, scales and scale bytes bit-identical to the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_2310_19102_amd as atom
from _gpu_util import npy

pytestmark = pytest.mark.gpu


def _rows(M, K, seed):
    g = torch.Generator().manual_seed(seed)
    sigma = torch.exp(1.5 * torch.randn(K, generator=g))
    x = (torch.randn((M, K), generator=g) * sigma).to(torch.float16)
    gamma = (1.0 + 0.1 * torch.randn(K, generator=g)).to(torch.float16)
    return x, gamma, torch.argsort(sigma, stable=True).to(torch.int32)


def _same(got, want, what):
    for name, a, b in zip(("q4", "q8", "scale"), got, want):
        a = npy(a)
        if a.ndim == 3:                                     # the MX arrays are step-major
            a = a.transpose(1, 0, 2).reshape(a.shape[1], -1)
        assert np.array_equal(a.view(np.uint8), b.view(np.uint8)), f"{what}: {name}"


@pytest.mark.parametrize("K", [2048, 2176, 4096, 4224, 5120, 5248, 8192, 8320, 12288, 16384, 16512, 28672])
@pytest.mark.parametrize("M", [3, 258])                     # one row per workgroup with more threads; more rows than CUs
def test_front_end_configurations(M, K):
    if M > 3 and K > 8320:
        M = 257
    print(f"[case] front end M={M} K={K}", flush=True)
    x, gamma, idx = _rows(M, K, K + M)
    dx, dg, di = x.cuda(), gamma.cuda(), idx.cuda()
    xs, gs, ix = x.numpy(), gamma.numpy(), idx.numpy()
    rows = slice(0, M) if M < 10 else slice(0, M, 37)       # (the oracle is one thread)
    pick = lambda t: t[rows].contiguous() if t.dim() == 2 else t[:, rows].contiguous()
    got = atom.atom_quantize_act(dx, dg, 1e-6, di)
    _same([pick(t) for t in got], oracle.quantize_act(xs[rows], gs, 1e-6, ix, 128, 128, 0.9), "norm")
    got = atom.atom_quantize_act(dx, None, 0.0, None)
    _same([pick(t) for t in got], oracle.quantize_act(xs[rows], None, 0.0, np.arange(K, dtype=np.int32), 128, 128, 0.9), "no index")
    got = atom.atom_quantize_act(dx, dg, 1e-6, None)
    _same([pick(t) for t in got], oracle.quantize_act(xs[rows], gs, 1e-6, np.arange(K, dtype=np.int32), 128, 128, 0.9), "norm, no index")
    assert torch.equal(atom.atom_quantize_act_packed(dx, dg, 1e-6, None), atom.atom_pack_act(*got))
    got = atom.atom_mx_quantize_act(dx, dg, 1e-6, di, 128, 0.9)
    _same([pick(t) for t in got], oracle.mx_quantize_act(xs[rows], gs, 1e-6, ix, 128, 0.9), "MX")
    if 4 * K + K // 2 + 3 * (K - 128) // 4 + 128 <= 160 * 1024:
        packed = atom.atom_quantize_act_packed(dx, dg, 1e-6, di)
        assert torch.equal(packed, atom.atom_pack_act(*atom.atom_quantize_act(dx, dg, 1e-6, di)))


@pytest.mark.parametrize("up", [1.0, 0.337, -7.25])
def test_every_gate(up):
    """silu of all 65536 fp16 gates but NaN and infinity, 256 per row in an order that mixes magnitudes."""
    bits = np.arange(65536, dtype=np.uint16)
    gate = bits.view(np.float16).astype(np.float16)
    gate = np.where(np.isfinite(gate), gate, np.float16(0.5)).reshape(256, 256)
    u = np.full_like(gate, np.float16(up))
    idx = np.arange(256, dtype=np.int32)
    got = atom.atom_swiglu_quantize_act(torch.from_numpy(gate).cuda(), torch.from_numpy(u).cuda(), None)
    _same(got, oracle.swiglu_quantize_act(gate, u, idx, 128, 128, 0.9), "rows of neighbours")
    mixed = np.ascontiguousarray(gate.T)
    got = atom.atom_swiglu_quantize_act(torch.from_numpy(mixed).cuda(), torch.from_numpy(u).cuda(), torch.from_numpy(idx).cuda())
    _same(got, oracle.swiglu_quantize_act(mixed, u, idx, 128, 128, 0.9), "mixed")


@pytest.mark.parametrize("M", [4, 258])
def test_mx_of_no_number(M):
    """A NaN is a zero in FP4 and the largest value in FP8, with its sign; the scale is that of the block's numbers."""
    K, K4 = 1024, 896
    x, _, _ = _rows(M, K, M)
    x = x.numpy().copy()
    at = [(0, 3, 1.0), (0, 500, -1.0), (1, K4 + 2, 1.0), (1, K4 + 99, -1.0)] + [(2, k, 1.0) for k in range(32)]
    for i, k, sign in at:
        x[i, k] = np.copysign(np.float16(np.nan), np.float16(sign))
    idx = torch.arange(K, dtype=torch.int32)
    got = [npy(t) for t in atom.atom_mx_quantize_act(torch.from_numpy(x).cuda(), None, 0.0, idx.cuda(), 128, 0.9)]
    numbers = np.where(np.isnan(x), np.copysign(np.float16(0.0), x), x)
    q4, q8, e8 = oracle.mx_quantize_act(numbers, None, 0.0, idx.numpy(), 128, 0.9)
    q8 = q8.copy()
    for i, k, sign in at:
        if k >= K4:
            q8.view(np.uint8)[i, k - K4] = 0x7E if sign > 0 else 0xFE
    for name, a, b in zip(("q4", "q8", "e8"), got, (q4, q8, e8)):
        a = a.transpose(1, 0, 2).reshape(a.shape[1], -1)
        assert np.array_equal(a.view(np.uint8), b.view(np.uint8)), name


def _around_ties(a, u, rng):
    """128 pairs of fp16 factors for a group of the scale 2 a u: their products are all 16 ties (k + 1/2) of INT4 (the outermost
    two are the group's maximum), values next to them, and values in between."""
    t = 2.0 * np.arange(-8, 8) + 1.0
    a = np.float16(a)
    below, above = np.nextafter(a, np.float16(0.0)), np.nextafter(a, np.float16(np.inf))
    first = np.repeat(np.array([a, below, above, a]), (16, 16, 14, 82))
    second = u * np.concatenate([t, t, t[1:-1], np.round(rng.uniform(-14.8, 14.8, 82) * 8.0) / 8.0])
    return first, second.astype(np.float16)


def test_every_scale():
    """Every positive fp16 scale: all codes of a group share the scale's reciprocal, and an exact tie has to stay one.  The
    values are exact products of two fp16 numbers: a gate whose sigma is 1 and the up operand, or, for the 63 smallest scales, a row and
    gamma where the factor of the norm is 1."""
    rng = np.random.default_rng(5)
    scales = [(m, e) for e in range(-24, 6) for m in range(1024, 2048)] + [(m, -24) for m in range(64, 1024)]
    rows = -(-len(scales) // 127)
    K = 128 * 128                                            # 127 INT4 groups per row, and the outliers
    gate, up = np.full((rows, K), 32.0, np.float16), np.full((rows, K), 0.25, np.float16)
    for i, (m, e) in enumerate(scales):
        b = m.bit_length()                                   # gates in [32, 64)
        at = np.s_[i // 127, 128 * (i % 127):128 * (i % 127) + 128]
        gate[at], up[at] = _around_ties(m * 2.0 ** (6 - b), 2.0 ** (e + b - 7), rng)
    ident = np.arange(K, dtype=np.int32)
    want = oracle.swiglu_quantize_act(gate, up, ident, 128, 128, 1.0)
    stored = want[2][:, :127].reshape(-1)[:len(scales)]
    assert np.array_equal(stored.astype(np.float64), [m * 2.0 ** e for m, e in scales])
    dg, du = torch.from_numpy(gate).cuda(), torch.from_numpy(up).cuda()
    _same(atom.atom_swiglu_quantize_act(dg, du, None, 128, 128, 1.0), want, "in order")
    _same(atom.atom_swiglu_quantize_act(dg, du, torch.from_numpy(ident).cuda(), 128, 128, 1.0), want, "gathered")

    K = 64 * 128
    x, gamma = np.full((1, K), 2.0 ** -15, np.float16), np.ones(K, np.float16)
    for m in range(1, 64):
        at = np.s_[128 * (m - 1):128 * m]
        x[0, at], gamma[at] = _around_ties(m * 2.0 ** -20, 2.0 ** -5, rng)
    ident = np.arange(K, dtype=np.int32)
    want = oracle.quantize_act(x, gamma, 1.0, ident, 128, 128, 1.0)
    assert np.array_equal(want[2][0, :63].astype(np.float64), np.arange(1, 64) * 2.0 ** -24)
    got = atom.atom_quantize_act(*(torch.from_numpy(v).cuda() for v in (x, gamma)), 1.0, torch.from_numpy(ident).cuda(), 128, 128, 1.0)
    _same(got, want, "norm")
