"""hilore_dequant_wgrad_ws: tiles past the last whole round split over tokens.

Integer-valued operands make every partial sum an integer below 2^24, so the
split and the unsplit call must agree bit for bit; a guard behind the workspace
and a NaN-filled dW show writes out of place and elements left out.
"""
import ctypes

import numpy as np
import pytest
import torch

from paper_2609_33570_amd import hilore as hl_mod

GUARD = 4096


def test_workspace_sizes():
    """256 KB slots, at most 512 of them; none where the tiles fill whole rounds or K is short."""
    need = hl_mod.hilore_wgrad_workspace_bytes
    assert need(16384, 4096, 4096) == 0   # 256 tiles
    assert need(16384, 8192, 4096) == 0   # 512 tiles
    assert need(128, 512, 512) == 0       # one pair of stages
    assert need(0, 512, 512) == 0 and need(16384, 0, 512) == 0
    for K, M, N in [(16384, 3584, 512), (1024, 896, 256), (16384, 3584, 18944),
                    (11987, 4096, 14336), (2 ** 20, 256, 8), (16384, 4104, 4096)]:
        b = need(K, M, N)
        tiles = -(-M // 256) * -(-N // 256)
        assert 0 < b <= 512 << 18 and b % ((tiles % 256) << 18) == 0, (K, M, N, b)


def test_workspace_errors():
    """Checked on the host before anything is enqueued."""
    L = hl_mod.load()
    p = ctypes.c_void_p(1 << 20)
    call = lambda ws, n: L.hilore_dequant_wgrad_ws(p, p, 1, 128, p, p, 16384, 3584, 512, 0,  # noqa: E731
                                                   ws, n, None)
    need = hl_mod.hilore_wgrad_workspace_bytes(16384, 3584, 512)
    assert call(None, 0) == hl_mod.HILORE_ERR_INVALID_ARG
    assert call(ctypes.c_void_p((1 << 20) + 8), need) == hl_mod.HILORE_ERR_ALIGNMENT
    assert call(p, need - 1) == hl_mod.HILORE_ERR_WORKSPACE


@pytest.mark.gpu
@pytest.mark.parametrize("code,block", [(0, 64), (1, 128), (2, 0)], ids=["int8", "e4m3fn", "cast"])
@pytest.mark.parametrize("K,M,N", [
    (1025, 256, 8),       # the last part one token, 8 columns of a tile
    (1000, 768, 272),     # ragged in K and N
    (4095, 128, 1032),    # half a tile of rows
    (16384, 3584, 512),   # 28 tiles
    (2000, 4352, 4096),   # 272 tiles: 256 whole, 16 split
    (2100, 3968, 4360),   # 288 tiles, ragged
])
@pytest.mark.parametrize("accumulate", [False, True], ids=["write", "add"])
def test_split_matches_unsplit(hl, code, block, K, M, N, accumulate):
    g = torch.Generator(device="cuda").manual_seed(K + M + N)
    x = torch.randint(-7, 8, (K, M), generator=g, device="cuda").to(torch.bfloat16)
    dy = torch.randint(-8, 9, (K, N), generator=g, device="cuda").to(torch.bfloat16)
    if code == 0:
        codes = (x.to(torch.int8) * 16).view(torch.uint8)
        scales = torch.full((K, M // block), 1 / 16, device="cuda")
    else:
        codes = x.to(torch.float8_e4m3fn).view(torch.uint8)
        scales = torch.full((K, M // block), 1.0, device="cuda") if block else None
    need = hl.hilore_wgrad_workspace_bytes(K, M, N)
    assert need > 0
    dw0 = (torch.randint(-50, 51, (M, N), generator=g, device="cuda").float() if accumulate
           else torch.full((M, N), float("nan"), device="cuda"))
    buf = torch.full((need + GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
    want, given, auto, side = dw0.clone(), dw0.clone(), dw0.clone(), dw0.clone()
    torch.cuda.synchronize()
    st = hl.load().hilore_dequant_wgrad(  # the unsplit call
        codes.data_ptr(), scales.data_ptr() if block else None, code, block, dy.data_ptr(),
        want.data_ptr(), K, M, N, int(accumulate), torch.cuda.current_stream().cuda_stream)
    assert st == hl.HILORE_OK
    hl.hilore_dequant_wgrad(codes, scales, code, block, dy, given, K, M, N, accumulate,
                            workspace=buf[:need])
    hl.hilore_dequant_wgrad(codes, scales, code, block, dy, auto, K, M, N, accumulate)
    stream = torch.cuda.Stream()
    hl.hilore_dequant_wgrad(codes, scales, code, block, dy, side, K, M, N, accumulate,
                            stream=stream.cuda_stream)
    torch.cuda.synchronize()
    ref = x[:, :8].double().t().contiguous() @ dy.double()
    if accumulate:
        ref += dw0[:8].double()
    assert np.array_equal(want[:8].double().cpu().numpy(), ref.cpu().numpy())
    assert torch.equal(given, want) and torch.equal(auto, want) and torch.equal(side, want)
    assert bool((buf[need:] == 0xA5).all())


def general(hl, K, M, N):
    assert hl.hilore_wgrad_workspace_bytes(K, M, N) > 0
    g = torch.Generator(device="cuda").manual_seed(5)
    codes = torch.randn((K, M), generator=g, device="cuda").to(torch.float8_e4m3fn).view(torch.uint8)
    scales = torch.rand((K, M // 128), generator=g, device="cuda") + 0.1
    return codes, scales, torch.randn((K, N), generator=g, device="cuda").to(torch.bfloat16)


def unsplit(hl, codes, scales, dy, K, M, N):
    dw = torch.full((M, N), float("nan"), device="cuda")
    st = hl.load().hilore_dequant_wgrad(codes.data_ptr(), scales.data_ptr(), 1, 128, dy.data_ptr(),
                                        dw.data_ptr(), K, M, N, 0,
                                        torch.cuda.current_stream().cuda_stream)
    assert st == hl.HILORE_OK
    return dw


@pytest.mark.gpu
def test_streams_and_capture(hl):
    """General operands: default and explicit streams give the same bits, as does a
    graph replayed from either."""
    K, M, N = 2048, 896, 896
    codes, scales, dy = general(hl, K, M, N)
    out = [torch.full((M, N), float("nan"), device="cuda") for _ in range(4)]
    torch.cuda.synchronize()
    call = lambda dw, **kw: hl.hilore_dequant_wgrad(codes, scales, 1, 128, dy, dw, K, M, N, **kw)  # noqa: E731
    call(out[0])
    side = torch.cuda.Stream()
    call(out[1], stream=side.cuda_stream)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(out[2])
        call(out[3], stream=torch.cuda.current_stream().cuda_stream)
    for _ in range(3):
        out[2].fill_(float("nan"))
        out[3].fill_(float("nan"))
        graph.replay()
        call(out[1])
        torch.cuda.synchronize()
        for o in out[1:]:
            assert torch.equal(out[0], o)


@pytest.mark.gpu
@pytest.mark.parametrize("explicit", [False, True], ids=["current", "explicit"])
def test_capture_not_begun_by_torch(hl, explicit):
    """hipStreamBeginCapture: torch gives the graph no pool of its own, so the call takes no
    memory and runs unsplit; a tensor in the memory it would have been given stays whole."""
    K, M, N = 2048, 896, 896
    codes, scales, dy = general(hl, K, M, N)
    want = unsplit(hl, codes, scales, dy, K, M, N)
    need = hl.hilore_wgrad_workspace_bytes(K, M, N)
    dw = torch.full((M, N), float("nan"), device="cuda")
    L, P = hl.load(), ctypes.c_void_p
    side, graph, run = torch.cuda.Stream(), P(), P()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        torch.empty(need, dtype=torch.uint8, device="cuda")  # a free block of this size
        torch.cuda.synchronize()
        assert L.hipStreamBeginCapture(P(side.cuda_stream), 0) == 0
        try:
            hl.hilore_dequant_wgrad(codes, scales, 1, 128, dy, dw, K, M, N,
                                    **({"stream": side.cuda_stream} if explicit else {}))
        finally:
            assert L.hipStreamEndCapture(P(side.cuda_stream), ctypes.byref(graph)) == 0
        nodes = ctypes.c_size_t(0)
        assert L.hipGraphGetNodes(graph, None, ctypes.byref(nodes)) == 0 and nodes.value == 1
        other = torch.full((need,), 0xA5, dtype=torch.uint8, device="cuda")
        assert L.hipGraphInstantiate(ctypes.byref(run), graph, None, None, ctypes.c_size_t(0)) == 0
        try:
            for _ in range(3):
                dw.fill_(float("nan"))
                assert L.hipGraphLaunch(run, P(side.cuda_stream)) == 0
                torch.cuda.synchronize()
                assert torch.equal(dw, want) and bool((other == 0xA5).all())
        finally:
            assert L.hipGraphExecDestroy(run) == 0 and L.hipGraphDestroy(graph) == 0


@pytest.mark.gpu
def test_out_of_memory(hl):
    """No memory left for the partial sums: the unsplit call, with a warning."""
    K, M, N = 2048, 896, 896
    codes, scales, dy = general(hl, K, M, N)
    want = unsplit(hl, codes, scales, dy, K, M, N)
    dw = torch.full((M, N), float("nan"), device="cuda")
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    try:
        torch.cuda.set_per_process_memory_fraction(
            (torch.cuda.memory_reserved() + 1) / torch.cuda.mem_get_info()[1])
        need, held = hl.hilore_wgrad_workspace_bytes(K, M, N), []
        with pytest.raises(torch.cuda.OutOfMemoryError):  # what earlier tests left in the pool
            while True:
                held.append(torch.empty(need, dtype=torch.uint8, device="cuda"))
        with pytest.warns(RuntimeWarning, match="unsplit"):
            hl.hilore_dequant_wgrad(codes, scales, 1, 128, dy, dw, K, M, N)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    torch.cuda.synchronize()
    assert torch.equal(dw, want)
