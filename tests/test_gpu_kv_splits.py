"""Decode attention where the workgroups of one more split would be a second round: the number of splits (by the workspace that it asks for), and a
sample of (sequence, head) pairs against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2310_19102_amd as atom
from test_gpu_kv import O_TOL, _npy, _rel_err

pytestmark = pytest.mark.gpu

D = 128


@pytest.mark.parametrize("B,H,T,splits", [
    (1, 40, 7200, 6),            # a lone sequence: 240 workgroups, not 280
    (1, 96, 3100, 2),
    (1, 200, 2049, 1),
    (1, 40, 2048, 2),            # up to 2048 tokens as ever
    (2, 40, 4200, 4),            # several sequences: one more than fits
    (7, 32, 2100, 1),            # more than 200 heads in all
    (7, 32, 2048, 2),
    (5, 40, 6144, 1),            # 200 heads: up to 96 groups
    (5, 40, 6145, 2),
    (12, 16, 2500, 2),           # 192 heads
    (19, 16, 2500, 1),           # more heads than compute units
])
def test_splits(B, H, T, splits):
    print(f"[case] attention splits B={B} H={H} T={T}", flush=True)
    need = atom.atom_decode_attention_kv4_workspace_bytes(B, H, H, D, T)
    assert need == (B * H * splits * (D + 2) * 4 if splits > 1 else 0)
    g = torch.Generator(device="cuda").manual_seed(B + H + T)
    rnd = lambda lo, hi, *shape, dtype: torch.randint(lo, hi, shape, generator=g, device="cuda").to(dtype)
    kc, vc = ([rnd(0, 256, B, H, T, D // 2, dtype=torch.uint8),
               (torch.rand((B, H, T), generator=g, device="cuda") * 0.05 + 0.05).half(),
               rnd(0, 16, B, H, T, dtype=torch.int16)] for _ in range(2))
    lens = rnd(1, T + 1, B, dtype=torch.int32)
    lens[B // 2] = T
    q = torch.randn((B, H, D), generator=g, device="cuda").half()
    ws = torch.empty(max(16, need), dtype=torch.uint8, device="cuda")
    out = _npy(atom.atom_decode_attention_kv4(q, kc, vc, lens, D ** -0.5, workspace=ws))
    for b, h in [(0, 0), (B // 2, H - 1), (B - 1, H // 2)]:
        one = lambda c: [np.ascontiguousarray(_npy(t[b:b + 1, h:h + 1])) for t in c]
        ref = oracle.decode_attention_kv4(_npy(q)[b:b + 1, h:h + 1], *one(kc), *one(vc), _npy(lens)[b:b + 1], D ** -0.5)
        err = _rel_err(out[b:b + 1, h:h + 1], ref)
        assert err <= O_TOL, f"(b={b}, h={h}): rel err {err}"
