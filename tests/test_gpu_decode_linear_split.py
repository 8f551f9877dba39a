"""atom_decode_linear on both sides of the line between one launch and two: the same codes and the same bits of Y (shapes whose sum over
groups is the same tree in both), and the one-launch kernel where a caller gives no arrays of codes, or some off their boundaries."""
import ctypes

import pytest
import torch

import paper_2310_19102_amd as atom

pytestmark = pytest.mark.gpu


def _case(M, K, N, norm, seed=0):
    g = torch.Generator(device="cuda").manual_seed(seed + 31 * M + K + N)
    idx = torch.randperm(K, generator=g, device="cuda").to(torch.int32)
    x = torch.randn((M, K), generator=g, device="cuda").half()
    gamma = (1 + 0.1 * torch.randn(K, generator=g, device="cuda")).half() if norm else None
    w = atom.atom_quantize_weight(torch.randn((N, K), generator=g, device="cuda").half() * 0.02, idx)
    qa = atom.atom_quantize_act(x, gamma, 1e-5, idx)
    return x, gamma, idx, w, qa, atom.atom_w4a4_gemm(*qa, *w)


def _wants(M, N, K, norm=True):
    from paper_2310_19102_amd.binding import _desc
    return atom.load_library().atom_decode_linear_wants_codes(M, N, ctypes.byref(_desc(K, 128, 128)), int(norm))


@pytest.mark.parametrize("M,K,N,norm,two", [
    (1, 4096, 8192, True, False), (1, 4096, 11008, True, True), (1, 11008, 512, False, True), (2, 4096, 4096, True, False),
    (3, 4096, 4096, True, True), (4, 1024, 1000, False, False), (16, 1024, 40, True, True), (9, 5120, 1300, False, True),
    (4, 4096, 4096, False, False), (5, 4096, 4096, False, True), (1, 5120, 4096, True, False), (1, 5120, 5120, True, True),
    (2, 2048, 8192, True, False)])
def test_both_sides_of_the_line(M, K, N, norm, two):
    print(f"[case] decode linear, {'two launches' if two else 'one launch'} M={M} K={K} N={N} norm={norm}", flush=True)
    assert bool(_wants(M, N, K, norm)) == two
    x, gamma, idx, w, qa, want = _case(M, K, N, norm)
    wide = torch.full((M, N + 3), 7.0, dtype=torch.float16, device="cuda")
    atom.atom_decode_linear(x, gamma, 1e-5, idx, *w, out=wide[:, :N])
    assert torch.equal(wide[:, :N], want) and bool((wide[:, N:] == 7.0).all())
    y, codes = atom.atom_decode_linear(x, gamma, 1e-5, idx, *w, debug=True)
    assert torch.equal(y, want) and all(torch.equal(c, q) for c, q in zip(codes, qa))


@pytest.mark.parametrize("M,K,N", [(3, 4096, 4096), (8, 4096, 11008), (16, 1024, 1000)])
def test_one_launch_without_arrays_on_their_boundaries(M, K, N):
    from paper_2310_19102_amd.binding import _desc
    print(f"[case] decode linear, one launch M={M} K={K} N={N}", flush=True)
    assert _wants(M, N, K)
    x, gamma, idx, w, qa, want = _case(M, K, N, True)
    L, d, P = atom.load_library(), _desc(K, 128, 128), lambda t: ctypes.c_void_p(t.data_ptr())
    room = [torch.zeros(4 + q.numel() * q.element_size(), dtype=torch.uint8, device="cuda")[4:] for q in qa]    # 4-byte boundaries
    for codes in (None, room):
        y = torch.zeros((M, N), dtype=torch.float16, device="cuda")
        rc = L.atom_decode_linear(P(x), M, K, P(gamma), ctypes.c_float(1e-5), P(idx), ctypes.byref(d), ctypes.c_float(0.9), *map(P, w), N,
                                  P(y), N, *(map(P, codes) if codes else (None, None, None)), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == 0 and torch.equal(y, want)
    assert all(torch.equal(r, q.view(-1).view(torch.uint8)) for r, q in zip(room, qa))


def test_refused_as_before():
    x, gamma, idx, w, _, _ = _case(16, 512, 64, True)
    for bad in (dict(clip=1e-9), dict(group_size=64), dict(bits=5)):
        with pytest.raises(atom.AtomError):
            atom.atom_decode_linear(x, gamma, 1e-5, idx, *w, **bad)
    with pytest.raises(atom.AtomError):
        atom.atom_decode_linear(torch.cat([x, x]), gamma, 1e-5, idx, *w)


@pytest.mark.parametrize("M,K,N,O,bits", [
    (8, 4096, 11008, 128, 4), (8, 5376, 8200, 128, 4),       # a multiple of four groups, two groups left over
    (12, 4224, 5000, 128, 4), (12, 4096, 8192, 256, 4),      # an odd number of groups, two INT8 groups
    (16, 512, 16400, 128, 4), (16, 384, 16400, 128, 4),      # fewer than eight groups
    (16, 256, 30000, 128, 4), (9, 4096, 8192, 128, 3)])      # one INT4 group, W3A3
def test_scales_off_the_grid_keep_the_bits(M, K, N, O, bits):
    """Y of a call that gives arrays for the codes is Y of the one launch, also where one of the scale arrays stands on an odd half-word."""
    from paper_2310_19102_amd.binding import _desc
    print(f"[case] decode linear, scales off the grid M={M} K={K} N={N} O={O} bits={bits}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(M + K + N)
    idx = torch.randperm(K, generator=g, device="cuda").to(torch.int32)
    x = torch.randn((M, K), generator=g, device="cuda").half()
    gamma = (1 + 0.1 * torch.randn(K, generator=g, device="cuda")).half()
    w = list(atom.atom_quantize_weight(torch.randn((N, K), generator=g, device="cuda").half() * 0.02, idx, 128, O, bits=bits))
    L, d, P = atom.load_library(), _desc(K, 128, O, bits), lambda t: ctypes.c_void_p(t.data_ptr())

    def off(t, by):                                          # the same numbers `by` bytes past a 256-byte boundary
        b = torch.empty(t.numel() + 4, dtype=t.dtype, device="cuda")[by // t.element_size():][:t.numel()].view(t.shape)
        return b.copy_(t)

    def call(scale, codes):
        y = torch.zeros((M, N), dtype=torch.float16, device="cuda")
        rc = L.atom_decode_linear(P(x), M, K, P(gamma), ctypes.c_float(1e-5), P(idx), ctypes.byref(d), ctypes.c_float(0.9), P(w[0]), P(w[1]),
                                  P(scale), N, P(y), N, *(map(P, codes) if codes else (None, None, None)),
                                  ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        assert rc == 0
        return y

    want = call(w[2], None)
    for by in (0, 2, 4):
        scale = off(w[2], by)
        assert torch.equal(call(scale, None), want)
        codes = [torch.empty((M, n), dtype=t, device="cuda") for n, t in (((K - O) // 2, torch.uint8), (O, torch.int8), (K // 128, torch.half))]
        assert torch.equal(call(scale, codes), want), f"weight scales {by} bytes off"
        codes[2] = off(codes[2], by)
        assert torch.equal(call(w[2], codes), want), f"activation scales {by} bytes off"
    assert torch.equal(atom.atom_decode_linear(x, gamma, 1e-5, idx, *w, bits=bits), want)


def test_no_memory_for_the_codes():
    """A call with an output of the caller's needs no memory: where the allocator has none for the codes it is one launch, the same bits."""
    M, K, N = 8, 4096, 4096
    assert _wants(M, N, K)
    x, gamma, idx, w, _, want = _case(M, K, N, True)
    y = torch.zeros((M, N), dtype=torch.float16, device="cuda")
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    try:
        torch.cuda.set_per_process_memory_fraction(1e-6)
        with pytest.raises(torch.OutOfMemoryError):
            while True:                                      # what the allocator still has of its small blocks
                held.append(torch.empty(16384, dtype=torch.uint8, device="cuda"))
        atom.atom_decode_linear(x, gamma, 1e-5, idx, *w, out=y)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.equal(y, want)
