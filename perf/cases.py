"""The work a user of this library has it do, as measurable cases.

Each case is a pass through the public entry points on inputs that already are on the GPU, with the
weights quantised (and, where the path wants it, packed) beforehand, as a serving process keeps
them.  Sizes are those of the benchmark's configurations (Llama-7B, -13B and -70B shaped linears,
group 128, 128 outlier channels, clip 0.9 / 0.85) and of the ranges around them.
"""
import math

import torch

import paper_2310_19102_amd as atom
from paper_2310_19102_amd.synth import CLIP_ACT, CLIP_WEIGHT, EPS, GROUP_SIZE, N_OUTLIER

D = 128                                  # head dimension
# hidden size, query heads, cache heads, intermediate size of the decoder shapes used here
SHAPES = {"7b": (4096, 32, 32, 11008), "13b": (5120, 40, 40, 13824), "70b": (8192, 64, 8, 28672)}


def listed():
    return [
        # one token of one user: a single projection in the one-launch form, bound by the call itself
        {"name": "one_call_m1_attn", "kind": "linear", "path": "one", "M": 1, "K": 4096, "N": 4096, "norm": True},
        # a small decoding batch through the two plain calls (front end, GEMM)
        {"name": "decode_m8_up", "kind": "linear", "path": "canonical", "M": 8, "K": 4096, "N": 11008, "norm": True},
        # a large decoding batch, fused gate/up projection
        {"name": "decode_m64_gate_up", "kind": "linear", "path": "canonical", "M": 64, "K": 4096, "N": 22016,
         "norm": True},
        # a short prompt or a very large decoding batch: fused QKV projection on packed weights
        {"name": "prompt_m256_qkv", "kind": "linear", "path": "packed", "M": 256, "K": 4096, "N": 12288, "norm": True},
        # an odd number of tokens on canonical weights (a process that keeps one copy of its weights)
        {"name": "ragged_m777_13b_up", "kind": "linear", "path": "canonical", "M": 777, "K": 5120, "N": 13824,
         "norm": True},
        # the hardware-scaled variant on the gate/up projection of a 1024-token prompt
        {"name": "mx_m1024_gate_up", "kind": "linear", "path": "mx", "M": 1024, "K": 4096, "N": 22016, "norm": True},
        # the MLP block of a 1024-token prompt: every quantisation fused into the operator before it
        {"name": "mlp_7b_m1024", "kind": "mlp", "shape": "7b", "M": 1024, "in_order": False},
        # the same block at the largest size: a 4096-token batch through the 70B-shaped MLP
        {"name": "mlp_70b_m4096", "kind": "mlp", "shape": "70b", "M": 4096, "in_order": False},
        # a decoding step of two whole layers, captured once in a graph as a serving loop does
        {"name": "layers_7b_b8", "kind": "layers", "shape": "7b", "B": 8, "T": 1024, "layers": 2},
        # the attention step of a decoding batch: append the new token, attend over ragged caches
        {"name": "attend_7b_b64_t2048", "kind": "attend", "H": 32, "Hkv": 32, "B": 64, "T": 2048},
        # grouped-query heads with long contexts
        {"name": "attend_70b_b16_t4096", "kind": "attend", "H": 64, "Hkv": 8, "B": 16, "T": 4096},
        # filling the cache from the keys and values of a batch of prompts
        {"name": "fill_cache_7b_4x2048", "kind": "fill", "Hkv": 32, "B": 4, "T": 2048},
    ]


def _log(rng, lo, hi):
    """An integer spread evenly over the logarithm of [lo, hi]."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: the kinds in the proportion in which they are listed."""
    kind = rng.choice(["decode", "decode", "decode", "prompt", "prompt", "mx", "mlp", "mlp", "layers", "attend", "attend",
                       "fill"])
    if kind == "decode":                         # 1 to 64 rows, weights streamed
        M = _log(rng, 1, 64)
        K = rng.choice([4096, 5120, 8192, 11008, 256 * rng.randint(4, 48)])
        N = rng.choice([4096, 11008, 22016, _log(rng, 1000, 28672)])
        path = rng.choice(["one", "coop", "canonical"] if M <= 8 else ["coop", "canonical"] if M <= 16 else ["canonical"])
        return {"kind": "linear", "path": path, "M": M, "K": K, "N": N, "norm": rng.random() < 0.7}
    if kind in ("prompt", "mx"):                 # 65 to 4096 rows, ragged row and column counts
        M = _log(rng, 65, 4096)
        K = rng.choice([4096, 5120, 8192, 11008, 128 * rng.randint(8, 112)])
        N = rng.choice([4096, 12288, 13824, _log(rng, 1000, 22016)])
        path = "mx" if kind == "mx" else rng.choice(["packed", "canonical"])
        return {"kind": "linear", "path": path, "M": M, "K": K, "N": N, "norm": rng.random() < 0.7}
    if kind == "mlp":
        return {"kind": "mlp", "shape": rng.choice(["7b", "13b", "70b"]), "M": _log(rng, 65, 4096),
                "in_order": rng.random() < 0.5}
    if kind == "layers":
        shape = rng.choice(["7b", "13b", "70b"])
        return {"kind": "layers", "shape": shape, "B": _log(rng, 1, 64), "T": _log(rng, 100, 2048),
                "layers": 1 if shape == "70b" else 2}
    if kind == "attend":
        H, Hkv = rng.choice([(32, 32), (40, 40), (64, 8)])
        B = _log(rng, 1, 128)
        return {"kind": "attend", "H": H, "Hkv": Hkv, "B": B, "T": _log(rng, 100, min(16384, 262144 // B))}
    B = _log(rng, 1, 16)
    return {"kind": "fill", "Hkv": rng.choice([8, 32, 40]), "B": B, "T": _log(rng, 50, 16384 // B)}


# ---- inputs ---------------------------------------------------------------------------------------


class _Inputs:
    """Seeded inputs on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(self, *shape, std=1.0):
        t = torch.empty(shape, dtype=torch.float16, device="cuda").normal_(generator=self.g)
        return t if std == 1.0 else t.mul_(std)

    def channels(self, K):
        """Heavy-tailed channel magnitudes (lognormal, sigma 1.5) and the index that puts the
        largest last."""
        sigma = torch.exp(1.5 * torch.randn(K, generator=self.g, device="cuda"))
        return sigma, torch.argsort(sigma, stable=True).to(torch.int32)

    def rows(self, M, sigma):
        return (torch.randn((M, sigma.numel()), generator=self.g, device="cuda") * sigma).to(torch.float16)

    def gamma(self, K):
        return (1.0 + 0.1 * torch.randn(K, generator=self.g, device="cuda")).to(torch.float16)

    def weight(self, N, K, idx, rows=None):
        """Quantised weight of a linear layer; `rows`: the order its output channels come in."""
        w = self.normal(N, K, std=0.02)
        if rows is not None:
            w = atom.atom_permute_rows(w, rows)
        return atom.atom_quantize_weight(w, idx, GROUP_SIZE, N_OUTLIER, CLIP_WEIGHT)

    def cache(self, B, Hkv, T):
        mu = torch.randn((1, Hkv, 1, D), generator=self.g, device="cuda").to(torch.float16)
        sigma = torch.exp(0.5 * torch.randn((1, Hkv, 1, D), generator=self.g, device="cuda")).to(torch.float16)
        k = self.normal(B, Hkv, T, D).mul_(sigma).add_(mu)
        v = self.normal(B, Hkv, T, D, std=0.5)
        return k, v

    def lengths(self, B, T):
        """Ragged sequence lengths, spread evenly from T/4 to T, in an order of this seed."""
        n = torch.tensor(_lengths(B, T), dtype=torch.int32, device="cuda")
        return n[torch.randperm(B, generator=self.g, device="cuda")].contiguous()


def _lengths(B, T):
    lo = max(1, T // 4)
    return [T if B == 1 else lo + (T - lo) * b // (B - 1) for b in range(B)]


def _empty(*shape):
    return torch.empty(shape, dtype=torch.float16, device="cuda")


def _packed_bytes(M, N, K):
    return torch.empty(atom.atom_w4a4_gemm_packed_workspace_bytes(M, N, K), dtype=torch.uint8, device="cuda")


def prepare(case, seed):
    return {"linear": _prepare_linear, "mlp": _prepare_mlp, "layers": _prepare_layers, "attend": _prepare_attend,
            "fill": _prepare_fill}[case["kind"]](case, _Inputs(seed))


def run(state):
    return state["run"](state)


# ---- one linear layer: front end and GEMM -----------------------------------------------------------


def _prepare_linear(case, r):
    M, K, N = case["M"], case["K"], case["N"]
    sigma, idx = r.channels(K)
    s = {"run": {"one": _run_one, "coop": _run_coop, "canonical": _run_canonical, "packed": _run_packed,
                 "mx": _run_mx}[case["path"]],
         "M": M, "K": K, "N": N, "x": r.rows(M, sigma), "gamma": r.gamma(K) if case["norm"] else None, "idx": idx}
    if case["path"] == "mx":
        s["w"] = atom.atom_mx_quantize_weight(r.normal(N, K, std=0.02), idx, N_OUTLIER, CLIP_WEIGHT)
        return s
    s["w"] = r.weight(N, K, idx)
    if case["path"] == "packed":
        s["w"] = atom.atom_pack_weight(*s["w"], GROUP_SIZE)
        s["a"] = _packed_bytes(M, N, K)
        s["y"] = _empty(M, N)
    elif case["path"] == "coop":
        s["sync"] = atom.atom_decode_linear_coop_sync()
        s["codes"] = tuple(torch.empty_like(t) for t in atom.atom_quantize_act(s["x"], s["gamma"], EPS, idx))
        s["y"] = _empty(M, N)
    return s


def _run_one(s):
    return atom.atom_decode_linear(s["x"], s["gamma"], EPS, s["idx"], *s["w"], GROUP_SIZE, CLIP_ACT)


def _run_coop(s):
    y, codes = atom.atom_decode_linear_coop(s["x"], s["gamma"], EPS, s["idx"], *s["w"], s["sync"], GROUP_SIZE, CLIP_ACT,
                                            out=s["y"], codes=s["codes"])
    return [y, *codes]


def _run_canonical(s):
    codes = atom.atom_quantize_act(s["x"], s["gamma"], EPS, s["idx"], GROUP_SIZE, N_OUTLIER, CLIP_ACT)
    return [atom.atom_w4a4_gemm(*codes, *s["w"], GROUP_SIZE), *codes]


def _run_packed(s):
    atom.atom_quantize_act_packed(s["x"], s["gamma"], EPS, s["idx"], GROUP_SIZE, N_OUTLIER, CLIP_ACT, out=s["a"])
    return atom.atom_w4a4_gemm_prepacked(s["a"], s["M"], s["w"], s["N"], s["K"], GROUP_SIZE, N_OUTLIER, out=s["y"])


def _run_mx(s):
    codes = atom.atom_mx_quantize_act(s["x"], s["gamma"], EPS, s["idx"], N_OUTLIER, CLIP_ACT)
    return [atom.atom_mx_gemm(*codes, *s["w"]), *codes]


# ---- the MLP block of a prompt ----------------------------------------------------------------------


def _prepare_mlp(case, r):
    M = case["M"]
    K, _, _, F = SHAPES[case["shape"]]
    sigma, idx = r.channels(K)
    _, idx_f = r.channels(F)
    # the down projection's reorder either happens in its front end, or was fused into the rows of
    # the gate and up weights
    rows = torch.cat([idx_f, idx_f + F]).to(torch.int32) if case["in_order"] else None
    s = {"run": _run_mlp, "M": M, "K": K, "F": F, "x": r.rows(M, sigma), "res": r.rows(M, 0.5 * sigma),
         "gamma": r.gamma(K), "idx": idx, "idx_f": None if case["in_order"] else idx_f}
    s["w1"] = atom.atom_pack_weight(*r.weight(2 * F, K, idx, rows), GROUP_SIZE)
    s["w2"] = atom.atom_pack_weight(*r.weight(K, F, idx_f), GROUP_SIZE)
    # the benchmark's rule: small activations are tiled by their front end, large ones in a pass
    s["fused"] = [M * K <= 1 << 24, M * F <= 1 << 24]
    s["a1"], s["a2"] = _packed_bytes(M, 2 * F, K), _packed_bytes(M, K, F)
    s["h"], s["gu"], s["y"] = _empty(M, K), _empty(M, 2 * F), _empty(M, K)
    s["q1"], s["q2"] = (None if fused else _codes(M, k) for fused, k in zip(s["fused"], (K, F)))
    return s


def _codes(M, K):
    return (torch.empty((M, (K - N_OUTLIER) // 2), dtype=torch.uint8, device="cuda"),
            torch.empty((M, N_OUTLIER), dtype=torch.int8, device="cuda"), _empty(M, K // GROUP_SIZE))


def _run_mlp(s):
    M, K, F = s["M"], s["K"], s["F"]
    if s["fused"][0]:
        atom.atom_add_quantize_act_packed(s["x"], s["res"], s["gamma"], EPS, s["idx"], sum_out=s["h"], out=s["a1"])
    else:
        atom.atom_add_quantize_act(s["x"], s["res"], s["gamma"], EPS, s["idx"], sum_out=s["h"], out=s["q1"])
        atom.atom_pack_act(*s["q1"], GROUP_SIZE, out=s["a1"])
    gu = atom.atom_w4a4_gemm_prepacked(s["a1"], M, s["w1"], 2 * F, K, out=s["gu"])
    if s["fused"][1]:
        atom.atom_swiglu_quantize_act_packed(gu[:, :F], gu[:, F:], s["idx_f"], out=s["a2"])
    else:
        atom.atom_swiglu_quantize_act(gu[:, :F], gu[:, F:], s["idx_f"], out=s["q2"])
        atom.atom_pack_act(*s["q2"], GROUP_SIZE, out=s["a2"])
    y = atom.atom_w4a4_gemm_prepacked(s["a2"], M, s["w2"], K, F, out=s["y"])
    return [y, gu, s["h"]]


# ---- whole decoder layers at decode time, in a graph --------------------------------------------------


def _prepare_layers(case, r):
    B, T = case["B"], case["T"]
    K, H, Hkv, F = SHAPES[case["shape"]]
    sigma, idx = r.channels(K)
    _, idx_f = r.channels(F)
    stack = []
    for _ in range(case["layers"]):
        w = {name: r.weight(n, k, i) for name, n, k, i in (
            ("q", K, K, idx), ("k", Hkv * D, K, idx), ("v", Hkv * D, K, idx), ("o", K, K, idx),
            ("gu", 2 * F, K, idx), ("down", K, F, idx_f))}
        w["gamma"] = (r.gamma(K), r.gamma(K))
        w["kc"], w["vc"] = (atom.atom_kv_quantize(t) for t in r.cache(B, Hkv, T))
        w["out"] = (_empty(B, K), _empty(B, K))
        stack.append(w)
    s = {"run": _run_layers, "x": r.rows(B, sigma), "res": r.rows(B, 0.5 * sigma), "stack": stack, "idx": idx,
         "idx_f": idx_f, "shape": (B, H, Hkv, K, F), "len": r.lengths(B, T)}
    s["pos"] = (s["len"] - 1).contiguous()
    s["ws"] = torch.empty(max(16, atom.atom_decode_attention_kv4_workspace_bytes(B, H, Hkv, D, T)), dtype=torch.uint8,
                          device="cuda")
    _layers(s)                                   # once outside the capture, as a server warms up
    torch.cuda.synchronize()
    s["graph"] = torch.cuda.CUDAGraph()
    with torch.cuda.graph(s["graph"]):
        _layers(s)
    return s


def _layers(s):
    B, H, Hkv, K, F = s["shape"]
    x, res = s["x"], s["res"]
    for w in s["stack"]:
        y, h2 = w["out"]
        h, *qa = atom.atom_add_quantize_act(x, res, w["gamma"][0], EPS, s["idx"])
        q, k, v = (atom.atom_w4a4_gemm(*qa, *w[n]) for n in ("q", "k", "v"))
        atom.atom_kv_quantize_pair(k.view(B, Hkv, D), v.view(B, Hkv, D), w["kc"], w["vc"], s["pos"])
        o = atom.atom_decode_attention_kv4(q.view(B, H, D), w["kc"], w["vc"], s["len"], D ** -0.5, workspace=s["ws"])
        o = atom.atom_w4a4_gemm(*atom.atom_quantize_act(o.view(B, K), None, 0.0, s["idx"]), *w["o"])
        _, *qa = atom.atom_add_quantize_act(o, h, w["gamma"][1], EPS, s["idx"], sum_out=h2)
        gu = atom.atom_w4a4_gemm(*qa, *w["gu"])
        qd = atom.atom_swiglu_quantize_act(gu[:, :F], gu[:, F:], s["idx_f"])
        atom.atom_w4a4_gemm(*qd, *w["down"], out=y)
        x, res = y, h2


def _run_layers(s):
    s["graph"].replay()
    return [[w["out"], w["kc"], w["vc"]] for w in s["stack"]]


# ---- the KV cache -----------------------------------------------------------------------------------


def _prepare_attend(case, r):
    B, H, Hkv, T = case["B"], case["H"], case["Hkv"], case["T"]
    k, v = r.cache(B, Hkv, T)
    s = {"run": _run_attend, "kc": atom.atom_kv_quantize(k), "vc": atom.atom_kv_quantize(v), "q": r.normal(B, H, D),
         "len": r.lengths(B, T), "out": _empty(B, H, D)}
    del k, v
    s["k"], s["v"] = (t[:, :, 0].contiguous() for t in r.cache(B, Hkv, 1))
    s["pos"] = (s["len"] - 1).contiguous()
    s["ws"] = torch.empty(max(16, atom.atom_decode_attention_kv4_workspace_bytes(B, H, Hkv, D, T)), dtype=torch.uint8,
                          device="cuda")
    return s


def _run_attend(s):
    atom.atom_kv_quantize_pair(s["k"], s["v"], s["kc"], s["vc"], s["pos"])
    o = atom.atom_decode_attention_kv4(s["q"], s["kc"], s["vc"], s["len"], D ** -0.5, out=s["out"], workspace=s["ws"])
    return [o, s["kc"], s["vc"]]


def _prepare_fill(case, r):
    k, v = r.cache(case["B"], case["Hkv"], case["T"])
    return {"run": _run_fill, "k": k, "v": v}


def _run_fill(s):
    return [atom.atom_kv_quantize(s["k"]), atom.atom_kv_quantize(s["v"])]


# ---- what a pass cannot do without ------------------------------------------------------------------


def _row(K):
    """Bytes of a quantised row: INT4 codes, INT8 outliers, fp16 scales."""
    return (K - N_OUTLIER) // 2 + N_OUTLIER + 2 * (K // GROUP_SIZE)


def work(case):
    """Inputs and weights read once, outputs written once; two operations per multiply-add."""
    kind = case["kind"]
    if kind == "linear":
        M, K, N = case["M"], case["K"], case["N"]
        row = (K - N_OUTLIER) // 2 + N_OUTLIER + K // 32 if case["path"] == "mx" else _row(K)
        codes = M * row if case["path"] in ("canonical", "coop", "mx") else 0
        return {"bytes": 2 * M * K + 4 * K + (2 * K if case["norm"] else 0) + N * row + 2 * M * N + codes,
                "flops": 2 * M * N * K}
    if kind == "mlp":
        M = case["M"]
        K, _, _, F = SHAPES[case["shape"]]
        return {"bytes": 2 * M * (2 * K + K + 2 * F + K) + 2 * F * _row(K) + K * _row(F),
                "flops": 2 * M * 3 * F * K}
    if kind == "layers":
        B, n = case["B"], case["layers"]
        K, H, Hkv, F = SHAPES[case["shape"]]
        weights = (2 * K + 2 * Hkv * D + 2 * F) * _row(K) + K * _row(F)
        tokens = sum(_lengths(B, case["T"]))
        return {"bytes": n * (weights + 2 * Hkv * tokens * (D // 2 + 4) + 2 * B * 4 * K),
                "flops": n * (2 * B * ((2 * K + 2 * Hkv * D + 2 * F) * K + K * F) + 4 * H * D * tokens)}
    if kind == "attend":
        B, H, Hkv = case["B"], case["H"], case["Hkv"]
        tokens = sum(_lengths(B, case["T"]))
        return {"bytes": 2 * Hkv * tokens * (D // 2 + 4) + 2 * B * (2 * H + 2 * Hkv) * D, "flops": 4 * H * D * tokens}
    n = 2 * case["B"] * case["Hkv"] * case["T"]
    return {"bytes": n * (2 * D + D // 2 + 4), "flops": 10 * n * D}


def tolerance(case):
    """fp32 sums rounded to fp16 outputs; codes and scales of given inputs are exact.  Behind a
    rounding to fp16 a value on the border of two codes may take the other one."""
    if case["kind"] == "fill":
        return "exact"
    if case["kind"] == "layers":
        return {"rel": 5e-3, "max": 0.2, "differ": 1e-3}
    return {"rel": 1e-3, "max": 2e-2}
