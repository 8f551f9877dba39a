"""Decode attention at the edges of its 64-token groups and 16-token steps, over caches written by hand: value scales among
fp16's subnormals, zero points near the end of int16's range, key codes all 0 or all 15."""
import numpy as np
import pytest
import torch

import oracle
import paper_2310_19102_amd as atom

pytestmark = pytest.mark.gpu

LENS = [0, 1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 255, 256, 257, 320, 400]


@pytest.mark.parametrize("H,Hkv", [(2, 2), (4, 2)])
@pytest.mark.parametrize("kind", ["plain", "subnormal"])
def test_attention_at_group_edges(H, Hkv, kind):
    B, T, D = len(LENS), 400, 128
    print(f"[case] attention at group edges H={H} Hkv={Hkv} {kind}", flush=True)
    rng = np.random.default_rng(7 * H + Hkv)
    codes = lambda: rng.integers(0, 256, (B, Hkv, T, D // 2), dtype=np.uint8)
    k = [codes(), (0.05 + 0.05 * rng.random((B, Hkv, T))).astype(np.float16), rng.integers(0, 16, (B, Hkv, T)).astype(np.int16)]
    v = [codes(), (0.01 + 0.1 * rng.random((B, Hkv, T))).astype(np.float16), rng.integers(0, 16, (B, Hkv, T)).astype(np.int16)]
    k[0][:, :, 5::64], k[0][:, :, 6::64] = 0x00, 0xFF
    if kind == "subnormal":       # outputs of about 30000 * 2^-23: normal fp16, all of it from the zero points
        v[1] = (rng.integers(1, 4, (B, Hkv, T)) * 2.0 ** -24).astype(np.float16)
        v[2] = rng.integers(-32768, -30000, (B, Hkv, T)).astype(np.int16)
    q = rng.standard_normal((B, H, D)).astype(np.float16)
    lens = np.array(LENS, dtype=np.int32)
    dev = lambda a: torch.from_numpy(a).cuda()
    out = atom.atom_decode_attention_kv4(dev(q), [dev(a) for a in k], [dev(a) for a in v], dev(lens), D ** -0.5).cpu().numpy()
    ref = oracle.decode_attention_kv4(q, *k, *v, lens, D ** -0.5)
    assert not out[0].any()
    # fp16 rounds by 2^-11 of a value; what is summed in fp32 adds less than that again
    floor = 1e-2 * np.abs(ref).max(axis=(1, 2), keepdims=True)
    err = np.abs(out.astype(np.float64) - ref)[1:] / np.maximum(np.abs(ref), floor)[1:]
    assert err.max() <= 2.0 ** -10, err.max(axis=(1, 2))


@pytest.mark.parametrize("H,Hkv", [(2, 2), (4, 2)])
def test_nothing_behind_the_end_counts(H, Hkv):
    """The last group of a sequence: whatever its other rows hold (codes, scales that are no numbers, zero points), the bits are those
    of a cache without them."""
    B, T, D = len(LENS), 400, 128
    print(f"[case] attention behind the end H={H} Hkv={Hkv}", flush=True)
    rng = np.random.default_rng(H)
    lens = np.array(LENS, dtype=np.int32)
    behind = np.arange(T)[None, None, :] >= lens[:, None, None]
    cache = []
    for _ in range(2):
        cache += [rng.integers(0, 256, (B, Hkv, T, D // 2), dtype=np.uint8), (0.05 + 0.05 * rng.random((B, Hkv, T))).astype(np.float16),
                  rng.integers(0, 16, (B, Hkv, T)).astype(np.int16)]
    other = [np.where(behind[..., None], 255 - cache[i], cache[i]) if i % 3 == 0 else
             np.where(behind, np.float16("nan") if i == 1 else np.float16("inf"), cache[i]) if i % 3 == 1 else
             np.where(behind, np.int16(-32768), cache[i]) for i in range(6)]
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    q = dev(rng.standard_normal((B, H, D)).astype(np.float16))
    outs = [atom.atom_decode_attention_kv4(q, [dev(a) for a in c[:3]], [dev(a) for a in c[3:]], dev(lens), D ** -0.5) for c in (cache, other)]
    assert bool(torch.isfinite(outs[1]).all())
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))


@pytest.mark.parametrize("B,H,Hkv,T", [(64, 32, 32, 512), (1, 32, 32, 32768), (128, 64, 8, 1024), (64, 34, 2, 8192)])
def test_attention_over_a_large_cache(B, H, Hkv, T):
    """From 2^27 bytes of codes on the rows are loaded with another hint (four wavefronts, sixteen, grouped query; not where 17 query heads
    share a cache head): the bits are those of the cache of one row less per sequence, which has as many groups and so the same splits."""
    D = 128
    assert B * Hkv * T * D == 1 << 27
    print(f"[case] attention over a large cache B={B} H={H} Hkv={Hkv} T={T}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(B + H)
    rnd = lambda lo, hi, *shape, dtype: torch.randint(lo, hi, shape, generator=g, device="cuda").to(dtype)
    cache = [[rnd(0, 256, B, Hkv, T, D // 2, dtype=torch.uint8),
              (torch.rand((B, Hkv, T), generator=g, device="cuda") * 0.05 + 0.05).half(),
              rnd(0, 16, B, Hkv, T, dtype=torch.int16)] for _ in range(2)]
    lens = rnd(1, T, B, dtype=torch.int32)
    lens[B // 2] = T - 1
    q = torch.randn((B, H, D), generator=g, device="cuda").half()
    less = [[t[:, :, :T - 1].contiguous() for t in c] for c in cache]
    large, small = (atom.atom_decode_attention_kv4(q, k, v, lens, D ** -0.5) for k, v in (cache, less))
    assert bool(torch.isfinite(small).all())
    assert torch.equal(large.view(torch.int16), small.view(torch.int16))
