"""Which way a pass takes (hag_route): a host decision, checked without a GPU."""
import numpy as np
import pytest

from paper_1906_03707_amd import binding as B
from paper_1906_03707_amd import synth


def test_one_launch_option_leaves_nothing_behind():
    # switching the one-launch schedule on and off again gives the handle's own way back, whatever came before
    rowptr, col = synth.holme_kim(3000, 8, 0.5, seed=81)
    h = B.hag_search(rowptr, col, 750)
    ways = lambda: [h.route(op, dt, d, back) for op, dt in (("sum", B.HAG_F32), ("max", B.HAG_F32), ("sum", B.HAG_I32)) for d in (16, 64, 256)   # noqa: E731
                    for back in (False, True)]
    before = ways()
    assert "one_launch" not in before
    h.set_option(B.HAG_OPT_ONE_LAUNCH_MAX_ITEMS, 262144)
    on = ways()
    assert set(on) == {"one_launch", "scatter"}
    h.set_option(B.HAG_OPT_ONE_LAUNCH_MAX_ITEMS, 0)
    assert ways() == before


def test_route_refuses_what_the_calls_refuse():
    rowptr, col = synth.random_graph(20, 0.3, seed=1)
    h = B.hag_search(rowptr, col, 4)
    for args in (("mean", B.HAG_I32, 8), ("sum", B.HAG_F32, 6), ("sum", B.HAG_F32, 0), ("sum", 7, 8)):
        with pytest.raises(B.HagError) as e:
            h.route(*args)
        assert e.value.code == B.HAG_EINVAL
    assert h.route("max", backward=True) == "scatter"
    h.set_option(B.HAG_OPT_DETERMINISTIC_MAX_BACKWARD, 1)
    assert h.route("max", backward=True) == "lists"


def dense_groups(n, size, cross, seed):
    """Complete groups of `size` consecutive nodes and `cross` random edges: a HAG of |V| nodes saves nearly every row read."""
    rng = np.random.default_rng(seed)
    g = np.arange(n) // size
    rows = np.repeat(np.arange(n), size)
    cols = np.repeat(g * size, size) + np.tile(np.arange(size), n)
    a, b = rng.integers(0, n, cross), rng.integers(0, n, cross)
    keys = np.unique(np.concatenate([rows, a, b]).astype(np.int64) * n + np.concatenate([cols, b, a]))
    r, c = keys // n, keys % n
    r, c = r[r != c], c[r != c]
    return np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))]).astype(np.int64), c.astype(np.int32)


def ways(h, op="sum", dtype=B.HAG_F32, widths=(16, 64, 128, 512)):
    return [[h.route(op, dtype, d, back) for back in (False, True)] for d in widths]


def test_a_hag_that_saves_most_rows_is_used_whatever_the_graph_size():
    # 2 M edges, 95 % fewer row reads; measured on a graph of twice the size, d = 128: 25 against 83 us for a sum, 35 against 114 us for a max
    rowptr, col = dense_groups(10000, 200, 10000, 3)
    h = B.hag_search(rowptr, col, 10000)
    st = h.stats()
    assert st["e"] < 16_000_000 and st["h"] + 2 * st["a"] < 0.1 * st["e"]
    assert ways(h, widths=(64, 128, 512)) == [["hag", "hag"]] * 3
    assert ways(h, dtype=B.HAG_I32, widths=(64, 128, 512)) == [["hag", "hag"]] * 3
    assert ways(h, "max", widths=(64, 128, 512)) == [["hag", "scatter"]] * 3
    few = h.prefix(600)                                     # 6 % fewer: 82 against 82 us forward, 90 against 82 transposed, at d = 128
    assert few.stats()["h"] > 0.9 * st["e"] and ways(few)[2][1] == "lists"


def test_a_hag_that_saves_little_of_a_small_graph_is_not():
    # launches: 10 against 7 us (1025 nodes); rows that miss either way: 105 against 88 us (57 k nodes, 6 % fewer reads)
    for rowptr, col in (synth.sbm(25, 41, 0.2, 0.001, seed=101), synth.holme_kim(6000, 14, 0.5, seed=102)):
        h = B.hag_search(rowptr, col, (rowptr.size - 1) // 4)
        assert {w[0] for w in ways(h)} == {w[1] for w in ways(h)} == {"lists"}


def test_batches():
    # time of both passes, us: dense products, LDS lists over the HAG, over the plain lists
    def batch(count, size, density, frac):
        rowptr, col, gp = synth.er_batch(count, size, density, seed=104)
        return B.hag_search_batched(rowptr, col, gp, frac)
    full = batch(1500, 74, 0.9, 1.0)
    assert ways(full, widths=(64,)) == [["dense", "dense"]]                                    # 31, 72, 64
    assert ways(full, dtype=B.HAG_I32, widths=(20,)) == [["component_hag", "component_hag"]]   # -, 38, 61
    sparse = batch(100, 250, 0.02, 0.25)
    # few large sparse graphs: at d = 128 no form fits in LDS; 37, 32 (over the HAG, from L2), 23
    assert ways(sparse, widths=(128,)) == [["lists", "lists"]]
    assert "dense" not in ways(sparse, widths=(64,))[0]                                        # 35, 22, 38
    few = batch(200, 128, 0.04, 0.25)
    assert ways(few, widths=(64, 128, 256)) == [["dense", "dense"]] * 3                        # 22, 27, 23; 24, 34, 24; 34, 54, 42


def test_knobs_that_shape_a_form_keep_it(monkeypatch):
    rowptr, col, gp = synth.er_batch(150, 40, 0.6, seed=5)
    search = lambda: B.hag_search_batched(rowptr, col, gp, 0.25)   # noqa: E731
    for expand in ("0", "1"):
        monkeypatch.setenv("HAG_COMPONENT_EXPAND", expand)
        assert ways(search(), widths=(16, 64)) == [["component_hag"] * 2] * 2
    monkeypatch.delenv("HAG_COMPONENT_EXPAND")
    want = ways(search(), widths=(32, 64, 128))
    monkeypatch.setenv("HAG_COMPONENT_PARTS", "2")
    assert ways(search(), widths=(32, 64, 128)) == want
    monkeypatch.setenv("HAG_ROUTE", "0")
    monkeypatch.setenv("HAG_COMPONENT_DENSE", "0")
    assert ways(search(), widths=(32, 64, 128)) == [["component_hag"] * 2] * 3
    monkeypatch.delenv("HAG_COMPONENT_PARTS")
    monkeypatch.delenv("HAG_COMPONENT_DENSE")
    rowptr, col = synth.holme_kim(2000, 8, 0.5, seed=6)
    h = B.hag_search(rowptr, col, 500)
    assert ways(h) == [["hag", "hag"]] * 4 and ways(h, "max") == [["hag", "scatter"]] * 4


def test_the_way_depends_on_the_handle_alone():
    rowptr, col = dense_groups(1000, 50, 500, 7)
    h = B.hag_search(rowptr, col, 1000)
    left, right, _ = h.get_merges()
    again = B.hag_from_merges(rowptr, col, left, right)
    for op in ("sum", "max", "gcn"):
        assert ways(h, op, widths=range(4, 300, 28)) == ways(again, op, widths=range(4, 300, 28)) == ways(h.prefix(left.size), op, widths=range(4, 300, 28))


def test_list_forms_option():
    # what a comparison of the HAG with the plain lists needs: each over its own lists, and the handle's own choice back afterwards
    rowptr, col = synth.holme_kim(3000, 8, 0.5, seed=81)
    graph = B.hag_search(rowptr, col, 750)
    rowptr, col, gp = synth.er_batch(150, 40, 0.6, seed=5)
    batch = B.hag_search_batched(rowptr, col, gp, 0.25)
    for h, own, hag, lists in ((graph, "lists", "hag", "lists"), (batch, "dense", "component_hag", "component_lists")):
        both = lambda **k: [h.route("sum", d=64, backward=b, **k) for b in (False, True)]   # noqa: E731
        assert both() == [own] * 2 == both(naive=True)
        h.set_option(B.HAG_OPT_LIST_FORMS, 1)
        assert both() == [hag] * 2 and both(naive=True) == [lists] * 2
        h.set_option(B.HAG_OPT_LIST_FORMS, 0)
        assert both() == [own] * 2 == both(naive=True)


def test_workspace_of_a_batch_holds_nothing_for_lists():
    # 2.4 M entries, enough for a scaled copy of the gradients if a transposed mean went over the lists: it runs as dense products, which need none
    rowptr, col, gp = synth.er_batch(500, 74, 0.9, seed=104)
    h = B.hag_search_batched(rowptr, col, gp, 0.0)
    for op in ("sum", "mean", "gcn"):
        for naive in (False, True):
            assert {h.route(op, d=64, backward=b, naive=naive) for b in (False, True)} == {"dense"}
        assert h.workspace_bytes(op, B.HAG_F32, 64) == 0
    # and an option given later does not need more than was told before
    h.set_option(B.HAG_OPT_LIST_FORMS, 1)
    assert h.workspace_bytes("mean", B.HAG_F32, 64) == 0


@pytest.mark.parametrize("n,degree,tiles,lists", [
    # forward sums timed over the lists and as tiles and a rest, us, at the widths where the line lies:
    (65536, 128, (132, 192, 256, 320, 512), (8, 16, 32, 64, 100, 128)),   # 389 / 340, 369 / 302, 412 / 374, 583 / 473, 821 / 748; 55 / 75, 58 / 77, 74 / 94, 118 / 145, 206 / 260, 211 / 216
    (30000, 150, (192, 320, 512), (16, 64, 128)),                         # 203 / 168, 314 / 249, 422 / 370; 37 / 59, 71 / 106, 117 / 136
    (65536, 60, (), (16, 64, 128, 132, 256, 512)),                        # 45 / 61, 66 / 118, 111 / 156, 196 / 227, 207 / 235, 408 / 435
    (131072, 120, (132, 256, 512), (16, 64, 100))])                       # 760 / 691, 835 / 789, 1664 / 1553; 103 / 108, 211 / 229, 394 / 513
def test_widths_where_a_sum_runs_as_tiles(n, degree, tiles, lists):
    rowptr, col = synth.dcsbm(n=n, mean_degree=float(degree), seed=103 if n < 131072 else 22)[:2]
    h = B.hag_from_merges(rowptr, col, np.zeros(0, np.int32), np.zeros(0, np.int32))
    # (what a sum of floats needs beyond one of integers is the tiles' partial rows)
    takes = lambda d: h.workspace_bytes("sum", B.HAG_F32, d) > h.workspace_bytes("sum", B.HAG_I32, d)   # noqa: E731
    assert [d for d in tiles if not takes(d)] == [] == [d for d in lists if takes(d)]
    assert {h.route("sum", d=d) for d in tiles} <= {"lists"}


def test_max_sorts_its_gradients_only_where_the_runs_are_long_enough():
    # a ring of nodes needs no other workspace: sorted gradients (6 bytes an element and tables), or none where atomics are faster.  Times, us, atomics / sorted:
    # f32 106 / 99, 140 / 158, 391 / 651, 390 / 281, 774 / 796, 1157 / 897, 55 / 46; i32 84 / 98, 307 / 281, 456 / 508, 681 / 566
    for dt, sorts, adds in ((B.HAG_F32, ((524288, 4), (1000003, 8), (2000000, 12), (16384, 64)), ((700000, 4), (2000000, 4), (2000000, 8))),
                            (B.HAG_I32, ((1000003, 8), (1500000, 12)), ((524288, 4), (1500000, 8)))):
        for n, d in sorts + adds:
            h = B.hag_from_merges(np.arange(n + 1, dtype=np.int64), ((np.arange(n) + 1) % n).astype(np.int32), np.zeros(0, np.int32), np.zeros(0, np.int32))
            assert (h.workspace_bytes("max", dt, d) >= 6 * n * d) == ((n, d) in sorts), (dt, n, d)
