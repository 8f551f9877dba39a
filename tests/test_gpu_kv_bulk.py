"""The bulk form of the KV quantiser (from 16384 rows) at the edges of its wavefronts' and workgroups' rows, with rows of
every kind among them: bit-identical to the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2310_19102_amd as atom
from _gpu_util import npy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("R", [16383, 16384, 16385, 16384 + 63, 20001])
def test_kv_quantize_bulk_edges(R, D):
    print(f"[case] kv bulk R={R} D={D}", flush=True)
    g = torch.Generator().manual_seed(R + D)
    x = torch.randn((R, D), generator=g) * torch.exp(4.0 * torch.randn((R, 1), generator=g)) + 50.0 * torch.randn((R, 1), generator=g)
    x = x.clamp(-65504.0, 65504.0).to(torch.float16)
    x[5] = 3.25                                             # scale 0
    x[6, ::2], x[6, 1::2] = -65504.0, 65504.0               # the widest range
    x[7] = torch.linspace(0, 1e-7, D).to(torch.float16)
    x[R - 1] = 1000.0 + (torch.arange(D) % 7).to(torch.float16)
    x[R - 2] = (torch.arange(D) % 31) * 0.5 - 7.5       # ties
    out = atom.atom_kv_quantize(x.cuda(), 0.95)
    want = oracle.kv_quantize(x.numpy(), 0.95)
    for name, a, b in zip(("codes", "scale", "zero"), out, want):
        assert np.array_equal(npy(a).view(np.uint8), b.view(np.uint8)), name


@pytest.mark.parametrize("clip", [0.0, -0.0, -0.75, 1e-30, 7.5])
@pytest.mark.parametrize("R", [37, 16385])
def test_kv_quantize_any_clip(R, clip):
    """The equations hold for every factor: a zero scale has the sign of its quotient, a large one saturates."""
    g = torch.Generator().manual_seed(R)
    x = (torch.randn((R, 128), generator=g) * torch.exp(3.0 * torch.randn((R, 1), generator=g))).clamp(-65504.0, 65504.0).to(torch.float16)
    x[0] = 0.0
    x[1] = -3.25
    x[2, ::2], x[2, 1::2] = -65504.0, 65504.0
    out = atom.atom_kv_quantize(x.cuda(), clip)
    want = oracle.kv_quantize(x.numpy(), clip)
    for name, a, b in zip(("codes", "scale", "zero"), out, want):
        assert np.array_equal(npy(a).view(np.uint8), b.view(np.uint8)), name


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("R", [37, 16385])
def test_kv_quantize_infinities(R, D):
    """A row of one infinity has no span: its scale is no number and its codes are zero.  An infinity among numbers gives the
    largest scale; the other rows are untouched."""
    g = torch.Generator().manual_seed(R)
    x = torch.randn((R, D), generator=g).to(torch.float16)
    x[0], x[1], x[2, 3], x[3, D - 1] = float("inf"), -float("inf"), float("inf"), -float("inf")
    codes, scale, zero = (npy(t) for t in atom.atom_kv_quantize(x.cuda()))
    want = oracle.kv_quantize(x[4:].numpy(), 1.0)
    for name, a, b in zip(("codes", "scale", "zero"), (codes[4:], scale[4:], zero[4:]), want):
        assert np.array_equal(a.view(np.uint8), b.view(np.uint8)), name
    assert np.isnan(scale[:2]).all() and (scale[2:4] == 65504.0).all()
    assert (codes[:4] == 0).all() and zero[:4].tolist() == [-32768, -32768, 0, -32768]


@pytest.mark.parametrize("R", [37, 16385])
def test_kv_quantize_scale_below_fp16(R):
    """A scale below every fp16 number is minus infinity, whether the span that gives it is finite in 32 bits or not."""
    g = torch.Generator().manual_seed(R)
    x = torch.randn((R, 128), generator=g).to(torch.float16)
    for clip in (-1e7, -1e38, -float("inf")):
        scale = npy(atom.atom_kv_quantize(x.cuda(), clip)[1])
        assert (scale == -np.inf).all(), clip
    x[::2, 3] = float("inf")
    scale = npy(atom.atom_kv_quantize(x.cuda(), -0.75)[1])
    assert (scale[::2] == -np.inf).all() and np.isfinite(scale[1::2]).all()


@pytest.mark.parametrize("clip", [1.0, 15.0])
def test_kv_quantize_every_scale(clip):
    """Every positive fp16 scale s that a row can have at this clip factor (spans 15 s / clip, from s to 16 s or from 0 to s): the
    nine quotients of a row share the scale's reciprocal.  Values next to the ties (k + 1/2) s and in between."""
    s = np.arange(1, 0x7c00, dtype=np.uint16).view(np.float16).astype(np.float64)
    s = s[s <= (65504.0 / 16.0 if clip == 1.0 else 65504.0)][:, None]
    lo, hi = (s, 16.0 * s) if clip == 1.0 else (0.0 * s, s)
    rng = np.random.default_rng(3)
    ties = ((np.arange(1, 16) + 0.5) * s if clip == 1.0 else np.repeat(0.5 * s, 15, 1)).astype(np.float16)
    inside = (lo + (hi - lo) * rng.random((len(s), 128 - 47))).astype(np.float16)
    x = np.concatenate([np.nextafter(ties, np.float16(0.0)), ties, np.nextafter(ties, np.float16(np.inf)), inside,
                        lo.astype(np.float16), hi.astype(np.float16)], 1)
    x = np.clip(x, lo, hi).astype(np.float16)
    want = oracle.kv_quantize(x, clip)
    assert np.array_equal(want[1].astype(np.float64), s[:, 0])
    for step in (1, 2):                                      # the bulk form, the form of few rows
        out = atom.atom_kv_quantize(torch.from_numpy(np.ascontiguousarray(x[::step])).cuda(), clip)
        for name, a, b in zip(("codes", "scale", "zero"), out, want):
            assert np.array_equal(npy(a).view(np.uint8), np.ascontiguousarray(b[::step]).view(np.uint8)), (name, step)
