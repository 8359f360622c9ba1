"""Transposed pass of max, gradients sorted by winner (n * d >= 2^20): edges of its tiles of 512 rows, blocks of 512 nodes and chunks of 32 columns, blocks
that are cut into parts, and the calls around it.  Sums of small whole numbers, so that every order of addition gives the same floats."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1906_03707_amd import binding
    binding.lib()
    return binding


def ring(B, n):
    col = ((np.arange(n) + 1) % n).astype(np.int32)
    return B.hag_from_merges(np.arange(n + 1, dtype=np.int64), col, np.zeros(0, np.int32), np.zeros(0, np.int32)).upload()


def winners(n, d, kind, seed):
    rng = np.random.default_rng(seed)
    am = rng.integers(0, n, (n, d), dtype=np.int32)
    if kind == "hubs":                     # one node wins a third of everything, 40 others most of the rest: blocks of several parts
        am[::3] = n - 1
        am[1::3] = am[1::3] % 40
    elif kind == "one":
        am[:] = n // 2
    am[rng.random((n, d)) < 0.05] = -1     # empty lists
    return am


@pytest.mark.parametrize("n,d,kind,dtype", [
    (16384, 64, "any", "f32"), (16385, 64, "any", "i32"), (16383, 68, "any", "f32"), (29789, 36, "any", "f32"), (52429, 20, "hubs", "f32"),
    (262145, 4, "any", "f32"), (8192, 132, "hubs", "i32"), (1000, 1052, "any", "f32"), (511, 2056, "hubs", "f32"), (16384, 64, "one", "f32"), (40000, 100, "hubs", "f32")])
def test_every_gradient_reaches_its_winner(B, n, d, kind, dtype):
    h = ring(B, n)
    dt, code = (torch.float32, B.HAG_F32) if dtype == "f32" else (torch.int32, B.HAG_I32)
    am = winners(n, d, kind, n + d)
    gy = np.random.default_rng(n).integers(-8, 9, (n, d))
    v, f = np.nonzero(am >= 0)
    want = np.zeros(n * d, np.int64)
    np.add.at(want, am[v, f].astype(np.int64) * d + f, gy[v, f])
    assert np.abs(want).max() < 1 << 24    # exact in fp32
    want = torch.from_numpy(want.reshape(n, d)).to(dt).cuda()
    am, gy = torch.from_numpy(am).cuda(), torch.from_numpy(gy).to(dt).cuda()
    assert h.workspace_bytes("max", code, d) > 6 * n * d
    assert torch.equal(h.backward(gy, "max", argmax=am, gx=torch.full_like(gy, 7)), want)
    # without a workspace: device-wide atomics
    gx = torch.full_like(gy, 7)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert B.lib().hag_backward(h._h, B.HAG_MAX, code, d, gy.data_ptr(), am.data_ptr(), gx.data_ptr(), None, stream) == 0
    assert torch.equal(gx, want)


def test_replays_of_a_captured_call_and_what_the_forward_pass_needs(B):
    n, d = 65536, 272
    h = ring(B, n)
    # the sorted gradients do not fit the fixed scratch array, but a forward pass over this handle needs none
    assert h.workspace_bytes("max", B.HAG_F32, d) > B.HAG_STATIC_SCRATCH_BYTES
    x = torch.randn(n, d, device="cuda")
    y, am = h.forward_static_scratch(x, "max")
    assert torch.equal(y, x.roll(-1, 0)) and bool((am == (torch.arange(n, device="cuda", dtype=torch.int32)[:, None] + 1) % n).all())
    gy, gx = torch.empty_like(x), torch.empty_like(x)
    ws = torch.empty(h.workspace_bytes("max", B.HAG_F32, d), dtype=torch.uint8, device="cuda")
    gy.copy_(x)
    h.backward(gy, "max", argmax=am, gx=gx, workspace=ws)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        h.backward(gy, "max", argmax=am, gx=gx, workspace=ws)
    for k in range(3):
        gy.copy_(x * (k + 1))
        gx.fill_(7.0)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(gx, (x * (k + 1)).roll(1, 0))


def test_forward_passes_hold_no_room_for_sorted_gradients(B):
    n, d = 65536, 64
    h = ring(B, n)
    x = torch.randn(n, d, device="cuda")
    assert B.lib().hag_forward_workspace_bytes(h._h, B.HAG_MAX, B.HAG_F32, d) == 0 and h.workspace_bytes("max", B.HAG_F32, d) > 6 * n * d
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    y, am = h.forward(x, "max")
    assert torch.cuda.memory_allocated() - before <= 2 * 4 * n * d + 4096           # the results
    # a captured forward pass keeps its workspace when a transposed one needs more
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        h.forward(x, "max", y=y, argmax=am)
    kept = dict(h._ws)
    gx = h.backward(y, "max", argmax=am)
    assert all(h._ws[k] is w for k, w in kept.items())
    x.copy_(torch.randn(n, d, device="cuda"))
    graph.replay()
    assert torch.equal(y, x.roll(-1, 0)) and torch.equal(h.backward(y, "max", argmax=am), y.roll(1, 0)) and gx.shape == y.shape
