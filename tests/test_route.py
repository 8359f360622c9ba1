"""Which way a pass takes (hag_route): a host decision, checked without a GPU."""
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
