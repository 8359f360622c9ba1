"""The gather's items at the edges of their lane groups, and the choice between the HAG and the plain lists.

Rows of up to 16 / 32 columns are walked by 4 / 2 streams of lanes per item, 16 ids at a time: list lengths around 1, 4, 16 and 64 entries, with aggregation nodes in
the lists, with ties for max (small integers as features) and without.  Bars: int32 and max bit-exact, fp32 sums within 1e-5 * sum|terms|."""
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


def edge_graph(seed):
    """Directed graph whose lists have the lengths at which chunks, streams and unrolled steps end; shared runs of ids, so that a HAG has nodes."""
    rng = np.random.default_rng(seed)
    n, rows = 520, []
    shared = rng.permutation(n)
    for v in range(n):
        k = [0, 1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 31, 32, 33, 63, 64, 65, 129, 300][v % 20]
        own = rng.choice(n, k, replace=False)
        if v % 3 == 0 and k >= 8:
            own = np.unique(np.concatenate([shared[:k // 2], own]))[:max(k, 1)]
        rows.append(np.sort(np.unique(own)))
    return np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64), np.concatenate(rows).astype(np.int32)


@pytest.mark.parametrize("d", [4, 12, 16, 20, 32, 36, 132, 260])
@pytest.mark.parametrize("route", ["0", "1"])
def test_list_lengths(B, d, route, monkeypatch):
    monkeypatch.setenv("HAG_ROUTE", route)
    rowptr, col = edge_graph(d)
    h = B.hag_search(rowptr, col, 130).upload()
    assert h.stats()["a"] > 20 and h.route("sum", d=d) == h.route("max", d=d) == ("lists" if route == "1" else "hag")
    check_against_oracle(h, rowptr, col, d)


@pytest.mark.parametrize("d", [4, 16, 32, 128, 132, 256, 260])
@pytest.mark.parametrize("route", ["0", "1"])
def test_rows_cut_by_source(B, d, route, monkeypatch):
    # every row of 8 and more entries cut into the eight source classes, wide rows in chunks of 128 columns: pieces of one entry, folds of partial rows
    # whose winners may still be aggregation nodes
    for k, v in dict(HAG_PARTITION_MIN_ROWS="0", HAG_PART_MIN="8", HAG_PART_SHARE_PCT="0", HAG_PART_MEAN_MIN="0", HAG_ROUTE=route).items():
        monkeypatch.setenv(k, v)
    rowptr, col = edge_graph(d)
    h = B.hag_search(rowptr, col, 130).upload()
    monkeypatch.setenv("HAG_PARTITION", "0")
    whole = B.hag_search(rowptr, col, 130)
    assert h.workspace_bytes("sum", 0, d) > whole.workspace_bytes("sum", 0, d)       # the cut is in effect: partial rows
    if route == "0":
        assert h.route("sum", d=d) == h.route("max", d=d) == "hag"
    check_against_oracle(h, rowptr, col, d)


def check_against_oracle(h, rowptr, col, d):
    n = rowptr.size - 1
    real, ties = synth.features_f32(n, d, 1), np.random.default_rng(2).integers(-2, 3, (n, d)).astype(np.float32)
    ints = synth.features_i32(n, d, 3)
    for x, ops in ((real, ("sum", "mean", "gcn", "max")), (ties, ("max",)), (ints, ("sum", "max"))):
        xd = torch.from_numpy(x).cuda()
        for op in ops:
            want, s, am = oracle.naive_forward(rowptr, col, x, op)
            y = h.forward(xd, op)
            if op == "max":
                assert np.array_equal(y[0].cpu().numpy(), want.astype(x.dtype)) and np.array_equal(y[1].cpu().numpy(), am)
                continue
            gx = h.backward(xd, op)
            gw, gs = oracle.naive_backward(rowptr, col, x, op)
            if x is ints:
                assert np.array_equal(y.cpu().numpy(), want) and np.array_equal(gx.cpu().numpy(), gw)
            else:
                assert np.all(np.abs(y.cpu().numpy() - want) <= 1e-5 * s) and np.all(np.abs(gx.cpu().numpy() - gw) <= 1e-5 * gs)


@pytest.mark.parametrize("d", [16, 64])
def test_both_graphs_give_the_same(B, d, monkeypatch):
    # a whole pass may run over the plain lists: it is the naive pass bit for bit, and what single phases give up to rounding
    rowptr, col = synth.holme_kim(2000, 8, 0.5, seed=5)
    h = B.hag_search(rowptr, col, 500).upload()
    monkeypatch.setenv("HAG_ROUTE", "0")
    over_hag = B.hag_search(rowptr, col, 500).upload()
    x = torch.from_numpy(synth.features_f32(2000, d, 6)).cuda()
    assert torch.equal(h.forward(x, "sum"), h.naive_forward(x, "sum")) and torch.equal(h.backward(x, "mean"), h.naive_backward(x, "mean"))
    for a, b in ((h, over_hag), (over_hag, h)):
        y, am = a.forward(x, "max")
        z, bm = b.forward(x, "max")
        assert torch.equal(y, z) and torch.equal(am, bm)
        assert torch.equal(a.forward_phases(x, B.HAG_PHASE_ALL, "sum"), a.forward(x, "sum"))
        _, s, _ = oracle.naive_forward(rowptr, col, x.cpu().numpy(), "sum")
        assert np.all(np.abs((a.forward(x, "sum") - b.forward(x, "sum")).cpu().numpy()) <= 1e-5 * s)
    out = torch.zeros_like(x)
    for phase in (B.HAG_PHASE_LEVELS, B.HAG_PHASE_GATHER, B.HAG_PHASE_FOLD):   # phase by phase: over the HAG
        h.forward_phases(x, phase, "sum", y=out)
    assert torch.equal(out, over_hag.forward(x, "sum"))


@pytest.mark.parametrize("d", [4, 16, 32])
def test_one_launch_max_with_ties(B, d, monkeypatch):
    # several dependent phases in one launch: an item's streams settle their ties on winners that an earlier phase of the launch wrote,
    # whose narrow rows share cache lines with rows that are written later
    monkeypatch.setenv("HAG_FUSE_MAX_ITEMS", "262144")
    monkeypatch.setenv("HAG_STAGE_EXTRA_ROWS", "-1000000")            # one phase per level
    rowptr, col = synth.sbm(n_blocks=4, block=60, p_in=0.5, p_out=0.02, seed=82)
    n = rowptr.size - 1
    h = B.hag_search(rowptr, col, n).upload()
    assert 3 <= h.stats()["stages"] == h.stats()["levels"] <= 7
    for seed in range(6):
        x = np.random.default_rng(seed).integers(0, 2 + seed, (n, d)).astype(np.float32)
        want, _, am = oracle.naive_forward(rowptr, col, x, "max")
        xd = torch.from_numpy(x).cuda()
        for _ in range(3):
            y, who = h.forward(xd, "max")
            assert np.array_equal(y.cpu().numpy(), want) and np.array_equal(who.cpu().numpy(), am), seed
            gy = synth.features_f32(n, d, seed)
            gw, gs = oracle.naive_backward(rowptr, col, gy, "max", am)
            assert np.all(np.abs(h.backward(torch.from_numpy(gy).cuda(), "max", argmax=who).cpu().numpy() - gw) <= 1e-5 * gs)
        h.check()                                                     # no wait gave up


@pytest.mark.parametrize("d", [4, 16, 20, 32])
@pytest.mark.parametrize("route", ["0", "1"])
def test_lists_too_short_for_several_streams(B, d, route, monkeypatch):
    # mean length below 8: one stream of 4 or 8 lanes per item, 64 or 32 items per workgroup, the last workgroup partly filled
    monkeypatch.setenv("HAG_ROUTE", route)
    rng = np.random.default_rng(d)
    n = 1203
    rows = [np.sort(rng.choice(n // 8, [0, 1, 2, 3, 4, 5, 7, 8, 9, 12][v % 10], replace=False)) for v in range(n)]
    rowptr, col = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64), np.concatenate(rows).astype(np.int32)
    h = B.hag_search(rowptr, col, 200).upload()
    assert h.stats()["a"] > 20 and h.route("sum", d=d) == ("lists" if route == "1" else "hag")
    check_against_oracle(h, rowptr, col, d)


@pytest.mark.parametrize("longest", [8, 31])                          # one stream per item, several
@pytest.mark.parametrize("d", [4, 16, 32, 64])
def test_max_passes_over_nan_in_short_lists(B, d, longest):
    # the scan takes the first entry and then whatever is greater: a NaN stays if it comes first and hides nothing anywhere else, however many
    # streams of lanes share the list
    rng = np.random.default_rng(d)
    n = 400
    rows = [np.sort(rng.choice(n, k, replace=False)) for k in rng.integers(1, longest + 1, n)]
    rowptr, col = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64), np.concatenate(rows).astype(np.int32)
    h = B.hag_search(rowptr, col, 0).upload()
    x = rng.integers(-3, 4, (n, d)).astype(np.float32)
    x[rng.random((n, d)) < 0.3] = np.nan
    x[rng.random((n, d)) < 0.2] = -np.inf
    want, who = np.empty_like(x), np.empty((n, d), np.int32)
    for v, r in enumerate(rows):
        best, at = x[r[0]].copy(), np.full(d, r[0])
        for u in r[1:]:
            take = x[u] > best                              # (False beside a NaN)
            best, at = np.where(take, x[u], best), np.where(take, u, at)
        want[v], who[v] = best, at
    y, am = h.forward(torch.from_numpy(x).cuda(), "max")
    assert np.array_equal(y.cpu().numpy(), want, equal_nan=True) and np.array_equal(am.cpu().numpy(), who)
