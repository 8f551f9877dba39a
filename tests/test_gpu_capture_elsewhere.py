"""Calls with an output of the caller's inside a capture that PyTorch's allocator does not know of (hipStreamBeginCapture on a stream): what a
call takes for its own length must not be part of the graph, since other tensors have that memory when the graph is replayed."""
import ctypes

import pytest
import torch

import paper_2310_19102_amd as atom

pytestmark = pytest.mark.gpu

RELAXED = 2                                                  # hipStreamCaptureModeRelaxed


def _hip():
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    return ctypes.CDLL(path)


def _gemm():
    M, N, K = 777, 3001, 4224
    assert atom.atom_w4a4_gemm_scratch_bytes(M, N, K) > 0
    g = torch.Generator(device="cuda").manual_seed(1)
    idx = torch.randperm(K, generator=g, device="cuda").to(torch.int32)
    qa = atom.atom_quantize_act(torch.randn((M, K), generator=g, device="cuda").half(), None, 0.0, idx)
    qw = atom.atom_quantize_weight(torch.randn((N, K), generator=g, device="cuda").half() * 0.02, idx)
    none = torch.empty(0, dtype=torch.uint8, device="cuda")
    return (M, N), lambda y: atom.atom_w4a4_gemm(*qa, *qw, out=y), lambda: atom.atom_w4a4_gemm(*qa, *qw, workspace=none)


def _linear():
    M, N, K = 8, 4096, 4096
    g = torch.Generator(device="cuda").manual_seed(2)
    idx = torch.randperm(K, generator=g, device="cuda").to(torch.int32)
    x = torch.randn((M, K), generator=g, device="cuda").half()
    gamma = (1 + 0.1 * torch.randn(K, generator=g, device="cuda")).half()
    w = atom.atom_quantize_weight(torch.randn((N, K), generator=g, device="cuda").half() * 0.02, idx)
    return (M, N), lambda y: atom.atom_decode_linear(x, gamma, 1e-5, idx, *w, out=y), lambda: atom.atom_decode_linear(x, gamma, 1e-5, idx, *w)


@pytest.mark.parametrize("case", [_gemm, _linear])
def test_replays_write_nothing_but_the_output(case):
    shape, call, reference = case()
    want = reference()
    y, hip, stream = torch.zeros(shape, dtype=torch.float16, device="cuda"), _hip(), torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        call(y)                                              # (the allocator has blocks of this stream now)
        stream.synchronize()
        handle, graph, run = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p(), ctypes.c_void_p()
        assert hip.hipStreamBeginCapture(handle, RELAXED) == 0
        try:
            call(y)
        finally:
            assert hip.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
        assert hip.hipGraphInstantiate(ctypes.byref(run), graph, None, None, ctypes.c_size_t(0)) == 0
        free = torch.cuda.memory_stats()["reserved_bytes.all.current"] - torch.cuda.memory_stats()["allocated_bytes.all.current"]
        # everything that is free goes to others before the replays
        others = [torch.full((1 << 20,), 0x5A, dtype=torch.uint8, device="cuda") for _ in range(free // (1 << 20) + 8)]
        others += [torch.full((1 << 12,), 0x5A, dtype=torch.uint8, device="cuda") for _ in range(1024)]
        for _ in range(3):
            y.zero_()
            assert hip.hipGraphLaunch(run, handle) == 0
            stream.synchronize()
            assert torch.equal(y, want)
            assert all(bool((t == 0x5A).all()) for t in others)
        assert hip.hipGraphExecDestroy(run) == 0 and hip.hipGraphDestroy(graph) == 0
