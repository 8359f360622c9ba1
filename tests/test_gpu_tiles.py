"""Sums over lists split into dense tiles and a rest (HAG_TILES=2: wherever there are tiles): tiles of 128 rows and their remainder, units of 24 steps of 32 sources, chunks of 16, 32
and 64 columns.  Small whole numbers, so that every order of addition gives the same floats and an entry dropped or taken twice shows."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1906_03707_amd import binding
    binding.lib()
    return binding


def groups(n, size, density, cross, symmetric, seed):
    """Dense groups of `size` neighbouring nodes and `cross` further edges; some rows are empty."""
    rng = np.random.default_rng(seed)
    r, c = np.repeat(np.arange(n), size), np.repeat(np.arange(n) // size * size, size) + np.tile(np.arange(size), n)
    keep = (rng.random(r.size) < density) & (c < n)
    r, c = np.concatenate([r[keep], rng.integers(0, n, cross)]), np.concatenate([c[keep], rng.integers(0, n, cross)])
    if symmetric:
        r, c = np.concatenate([r, c]), np.concatenate([c, r])
    else:
        keep = r % 50 != 7
        r, c = r[keep], c[keep]
    keys = np.unique((r.astype(np.int64) * n + c)[r != c])
    return np.concatenate([[0], np.cumsum(np.bincount(keys // n, minlength=n))]).astype(np.int64), (keys % n).astype(np.int32)


def handles(B, monkeypatch, rowptr, col, cut):
    monkeypatch.setenv("HAG_COMPONENT", "0")
    monkeypatch.setenv("HAG_PARTITION_MIN_ROWS", "0" if cut else "16384")
    monkeypatch.setenv("HAG_TILES_MIN_ENTRIES", "0")
    monkeypatch.setenv("HAG_TILES_SHARE_PCT", "0")
    none = np.zeros(0, np.int32)
    out = []
    for tiles in ("2", "0"):
        monkeypatch.setenv("HAG_TILES", tiles)
        out.append(B.hag_from_merges(rowptr, col, none, none).upload())
    assert out[0].route("sum", d=64) == "lists"
    return out


@pytest.mark.parametrize("n,size,density,cross,symmetric,cut", [
    (128, 128, 0.5, 0, True, False),       # one tile
    (129, 40, 0.9, 300, False, False),     # a tile of one row
    (1500, 64, 0.6, 4000, False, True),
    (2048, 700, 0.4, 3000, True, False),   # tiles of several units
    (5003, 1100, 0.2, 20000, False, True)])
@pytest.mark.parametrize("d", [4, 16, 20, 36, 64, 68, 132])
def test_every_entry_once(B, monkeypatch, n, size, density, cross, symmetric, cut, d):
    rowptr, col = groups(n, size, density, cross, symmetric, seed=n + d)
    h, plain = handles(B, monkeypatch, rowptr, col, cut)
    x = np.random.default_rng(d).integers(-8, 9, (n, d)).astype(np.float32)
    xd = torch.from_numpy(x).cuda()
    want, size_f, _ = oracle.naive_forward(rowptr, col, x, "sum")
    assert size_f.max() < 1 << 23          # exact in fp32
    y, ws = torch.full_like(xd, 7), torch.full((max(h.workspace_bytes("sum", B.HAG_F32, d), 16),), 255, dtype=torch.uint8, device="cuda")
    h.forward(xd, "sum", y=y, workspace=ws)
    assert np.array_equal(y.cpu().numpy(), want.astype(np.float32))
    back, _ = oracle.naive_backward(rowptr, col, x, "sum")
    assert np.array_equal(h.backward(xd, "sum", gx=torch.full_like(xd, 7), workspace=ws).cpu().numpy(), back.astype(np.float32))
    for op in ("mean", "gcn"):
        ref, s, _ = oracle.naive_forward(rowptr, col, x, op)
        assert np.all(np.abs(h.forward(xd, op).cpu().numpy() - ref) <= 1e-5 * s)
        ref, s = oracle.naive_backward(rowptr, col, x, op)
        assert np.all(np.abs(h.backward(xd, op).cpu().numpy() - ref) <= 1e-5 * s)
    # what is not a sum of floats, and single phases, go over the lists as before
    xi = xd.to(torch.int32)
    assert torch.equal(h.forward(xi, "sum"), plain.forward(xi, "sum"))
    assert all(torch.equal(a, b) for a, b in zip(h.forward(xd, "max"), plain.forward(xd, "max")))
    h.set_option(B.HAG_OPT_LIST_FORMS, 1)
    assert torch.equal(h.forward(xd, "sum"), plain.forward(xd, "sum"))


def test_numbers_that_are_not_finite_or_huge_reach_their_neighbours_only(B, monkeypatch):
    n, d = 1000, 72
    rowptr, col = groups(n, 200, 0.5, 2000, True, seed=3)
    h, plain = handles(B, monkeypatch, rowptr, col, False)
    x = torch.randn(n, d, device="cuda")
    x[5, 3], x[300, 10], x[301, 10], x[700, 70], x[701, 71], x[702, 71], x[40, 0] = float("inf"), float("inf"), float("-inf"), float("nan"), 3e38, -3e38, 1e-42
    got, want = h.forward(x, "sum"), plain.forward(x, "sum")
    assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.equal(torch.isinf(got), torch.isinf(want))
    fine = torch.isfinite(want)
    size = plain.forward(torch.where(torch.isfinite(x), x.abs() / 2 ** 40, torch.zeros_like(x)), "sum") * 2 ** 40
    assert bool(((got - want).abs()[fine] <= 1e-5 * size[fine]).all())


@pytest.mark.parametrize("kind", ["normal", "positive"])
def test_sums_lean_to_no_side(B, monkeypatch, kind):
    # rounded additions err to either side: the mean of N errors is within a few of their standard deviations / sqrt(N) (10: columns of a row share its order
    # of additions).  Products that are cut to the size of their accumulator leave more than that.
    n, d = 6000, 128
    rowptr, col = groups(n, 1500, 0.3, 60000, False, seed=8)
    h, plain = handles(B, monkeypatch, rowptr, col, False)
    x = torch.randn(n, d, device="cuda", generator=torch.Generator(device="cuda").manual_seed(9))
    x = x.abs() if kind == "positive" else x
    to = torch.repeat_interleave(torch.arange(n, device="cuda"), torch.from_numpy(np.diff(rowptr)).cuda())
    want = torch.zeros(n, d, dtype=torch.float64, device="cuda").index_add_(0, to, x.double()[torch.from_numpy(col).cuda().long()])
    error = h.forward(x, "sum").double() - want
    assert abs(error.mean().item()) <= 10 * error.std().item() / error.numel() ** 0.5
    # and they are of the size of the lists' errors: a chain of m additions of positive numbers errs by about sqrt(m / 3) roundings of its sum.  Here two units of 24 steps
    # (2.8 of half a row each) and their fold, 2.2 in all; the lists 8 streams of 54 entries, four at a time (2.1 of an eighth), and their fold, 1.8
    assert error.norm().item() <= 1.5 * (plain.forward(x, "sum").double() - want).norm().item()


def test_replays_of_a_captured_pass(B, monkeypatch):
    n, d = 3000, 64
    rowptr, col = groups(n, 700, 0.4, 9000, False, seed=4)
    h, _ = handles(B, monkeypatch, rowptr, col, True)
    x, y, gx = torch.randn(n, d, device="cuda"), torch.empty(n, d, device="cuda"), torch.empty(n, d, device="cuda")
    ws = torch.empty(max(h.workspace_bytes("gcn", B.HAG_F32, d), 16), dtype=torch.uint8, device="cuda")
    call = lambda: (h.forward(x, "sum", y=y, workspace=ws), h.backward(y, "gcn", gx=gx, workspace=ws))   # noqa: E731
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for k in range(3):
        x.copy_(torch.randn(n, d, device="cuda"))
        graph.replay()
        torch.cuda.synchronize()
        a, b = y.clone(), gx.clone()
        call()
        assert torch.equal(a, y) and torch.equal(b, gx)


def test_without_room_for_the_partial_rows_a_sum_goes_over_the_lists(B, monkeypatch):
    import ctypes
    n = 2048
    rowptr, col = groups(n, 700, 0.4, 3000, True, seed=5)
    h, plain = handles(B, monkeypatch, rowptr, col, False)
    need = lambda a, d: a.workspace_bytes("sum", B.HAG_F32, d)   # noqa: E731
    assert need(plain, 64) == 0 < need(h, 64) and h.workspace_bytes("sum", B.HAG_I32, 64) == 0
    x = torch.randn(n, 64, device="cuda")
    y = torch.full_like(x, 7)
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert B.lib().hag_forward(h._h, B.HAG_SUM, B.HAG_F32, 64, x.data_ptr(), y.data_ptr(), None, None, stream) == 0
    assert torch.equal(y, plain.forward(x, "sum"))
    y.fill_(7)
    assert B.lib().hag_backward(h._h, B.HAG_SUM, B.HAG_F32, 64, x.data_ptr(), None, y.data_ptr(), None, stream) == 0
    assert torch.equal(y, plain.backward(x, "sum"))
    assert torch.equal(h.forward_static_scratch(x, "sum"), h.forward(x, "sum"))
    # more than the fixed scratch array holds: not refused, as the lists need none of it
    d = 8192
    assert need(h, d) > B.HAG_STATIC_SCRATCH_BYTES and need(plain, d) == 0
    x = torch.randn(n, d, device="cuda")
    assert torch.equal(h.forward_static_scratch(x, "sum"), plain.forward(x, "sum"))


def test_the_fixed_scratch_array_serves_what_a_forward_pass_needs(B, monkeypatch):
    # seven partial rows per node.  They fit the array, but not together with the scaled copy of a transposed mean
    n, d = 12000, 200
    rowptr, col = groups(n, 1500, 0.15, 0, True, seed=11)
    h, plain = handles(B, monkeypatch, rowptr, col, False)
    need = {op: h.workspace_bytes(op, B.HAG_F32, d) for op in ("sum", "mean")}
    assert need["sum"] <= B.HAG_STATIC_SCRATCH_BYTES < need["mean"]
    x = torch.randn(n, d, device="cuda")
    for op in ("sum", "mean"):
        want = h.forward(x, op)
        assert not torch.equal(want, plain.forward(x, op))    # another order of additions: tiles ran
        assert torch.equal(h.forward_static_scratch(x, op), want)


@pytest.mark.parametrize("kind", ["batch", "blocks"])
def test_handles_that_take_no_tiles_keep_none(B, monkeypatch, kind):
    # dense products serve the batch at every width, and the lists the blocks (12 of 1300 nodes: d = 128 50 us, as tiles and a rest 100; 512 184 and 262)
    from paper_1906_03707_amd import synth
    rowptr, col = synth.er_batch(1000, 74, 0.9, seed=104)[:2] if kind == "batch" else synth.sbm(12, 1300, 0.1, 0.0005, seed=5)[:2]
    none, held = np.zeros(0, np.int32), []
    for tiles in ("1", "0"):
        monkeypatch.setenv("HAG_TILES", tiles)
        h = B.hag_from_merges(rowptr, col, none, none)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        h.upload()
        held.append(before - torch.cuda.mem_get_info()[0])
        del h
    assert held[0] <= held[1] + 4 * col.size // 4          # (a quarter of what a second copy of the lists would take)
