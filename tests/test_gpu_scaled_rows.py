"""Transposed mean and gcn over long lists: rows multiplied by 1 / degree once before the gather (hag_backward with a workspace) give the sums of the gather
that multiplies every row it reads (the same call without one) bit for bit, over the lists and over a HAG, in whole and by phases."""
import ctypes

import numpy as np
import pytest

import oracle
from paper_1906_03707_amd import synth

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1906_03707_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("d", [4, 20, 64, 132, 260])
@pytest.mark.parametrize("way", ["lists", "hag"])
def test_scaled_rows(B, monkeypatch, way, d):
    monkeypatch.setenv("HAG_COMPONENT", "0")
    monkeypatch.setenv("HAG_ROUTE", "0")
    rowptr, col = synth.random_graph(3001, 0.25, seed=d)
    n = rowptr.size - 1
    h = B.hag_search(rowptr, col, 60 if way == "hag" else 0).upload()
    gy = torch.randn(n, d, device="cuda")
    for op in ("mean", "gcn"):
        with_copy = h.workspace_bytes(op, B.HAG_F32, d) - h.workspace_bytes("sum", B.HAG_F32, d)
        assert with_copy >= 4 * n * d
        got = h.backward(gy, op)
        ref, size = oracle.naive_backward(rowptr, col, gy.cpu().numpy(), op)
        assert np.all(np.abs(got.cpu().numpy() - ref) <= 1e-5 * size)
        ws = torch.empty(h.workspace_bytes(op, B.HAG_F32, d), dtype=torch.uint8, device="cuda")
        gx = torch.full_like(gy, 7)
        for phase in (B.HAG_PHASE_LEVELS, B.HAG_PHASE_GATHER, B.HAG_PHASE_FOLD):
            h.backward_phases(gy, phase, op, gx=gx, workspace=ws)
        assert torch.equal(gx, got)
        if way == "lists" and h.workspace_bytes("sum", B.HAG_F32, d) == 0:
            gx.fill_(7)
            stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
            assert B.lib().hag_backward(h._h, B.OPS[op], B.HAG_F32, d, gy.data_ptr(), None, gx.data_ptr(), None, stream) == 0
            assert torch.equal(gx, got)


def test_no_copy_over_a_hag_that_scales_few_entries(B):
    # complete groups of shuffled nodes: a million list entries, of which a HAG with a balanced tree per group names a destination 10000 times
    size, n, d = 100, 10000, 64
    members = np.sort(np.random.default_rng(4).permutation(n).astype(np.int32).reshape(-1, size), axis=1)
    group = np.empty(n, np.int64)
    group[members.ravel()] = np.repeat(np.arange(n // size), size)
    rowptr, col = np.arange(n + 1, dtype=np.int64) * size, members[group].reshape(-1)
    merges, at = [], n
    trees = [list(m) for m in members]
    while len(trees[0]) > 1:
        for t in trees:
            pairs = [(t[i], t[i + 1]) for i in range(0, len(t) - 1, 2)]
            t[:] = list(range(at, at + len(pairs))) + t[2 * len(pairs):]
            merges += pairs
            at += len(pairs)
    h = B.hag_from_merges(rowptr, col, *np.array(merges, np.int32).T).upload()
    assert h.stats()["h"] == n and h.route("mean", d=d, backward=True) == "hag"
    gy = torch.randn(n, d, device="cuda")
    for op in ("mean", "gcn"):
        rows = h.workspace_bytes("sum", B.HAG_F32, d)      # the copy's place is behind what a sum needs (lists alone make one: their rows are long)
        ws = torch.full((h.workspace_bytes(op, B.HAG_F32, d),), 171, dtype=torch.uint8, device="cuda")
        assert ws.numel() >= rows + 4 * n * d
        got = h.backward(gy, op, workspace=ws)
        assert bool((ws[rows:] == 171).all())
        assert bool(((got - h.naive_backward(gy, op, workspace=ws)).abs() <= 1e-5 * gy.abs().max() * 2).all())
        assert not bool((ws[rows:] == 171).all())
