"""The dense form of the component pass (adjacency bits times feature rows in bf16 pieces) against the CPU oracle, at the edges
of its tiles: 16 output rows, 32 nodes per product step, 80 rows per wavefront, 16 / 32 / 64 columns per wavefront.

Tolerance: the pieces add up to the fp32 features exactly and every product is exact, so the result differs from the oracle by the rounding of an
fp32 sum of at most 3 * 256 terms: within 1e-5 * sum|terms| with a wide margin, the bar of the other sums."""
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


def directed_batch(sizes, p, seed):
    """Disjoint directed random graphs (self-loops allowed) of the given sizes; block-diagonal CSR."""
    rng = np.random.default_rng(seed)
    rows, cols, off = [], [], 0
    for sz in sizes:
        r, c = np.nonzero(rng.random((sz, sz)) < p)
        rows.append(r + off)
        cols.append(c + off)
        off += sz
    rows, cols = np.concatenate(rows), np.concatenate(cols)
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=off))]).astype(np.int64)
    return rowptr, cols.astype(np.int32), np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)


SIZES = {"small": [1, 2, 3, 7, 8, 9, 15, 16, 17, 24] * 12,
         "middle": [31, 32, 33, 47, 48, 49, 63, 64, 65, 74] * 7,
         "large": [79, 80, 81, 95, 96, 97, 128, 161, 255, 256] * 7}


@pytest.mark.parametrize("sizes", SIZES)
@pytest.mark.parametrize("d", [4, 16, 20, 32, 36, 64, 68, 132])
def test_tile_edges(B, sizes, d, monkeypatch):
    monkeypatch.setenv("HAG_COMPONENT_DENSE", "2")          # at every width
    rowptr, col, gp = directed_batch(SIZES[sizes], 0.4, seed=d)
    h = B.hag_search_batched(rowptr, col, gp, 0.25).upload()
    assert h.stats()["components"] >= 64
    x = synth.features_f32(rowptr.size - 1, d, d + 1)
    xd = torch.from_numpy(x).cuda()
    for op in ("sum", "mean", "gcn"):
        y, s, _ = oracle.naive_forward(rowptr, col, x, op)
        gx, gs = oracle.naive_backward(rowptr, col, x, op)
        for fwd, bwd in ((h.forward, h.backward), (h.naive_forward, h.naive_backward)):
            assert np.all(np.abs(fwd(xd, op).cpu().numpy() - y) <= 1e-5 * s), op
            assert np.all(np.abs(bwd(xd, op).cpu().numpy() - gx) <= 1e-5 * gs), op


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3e38, 1e-40, -1e-33])
@pytest.mark.parametrize("d", [12, 64])
def test_values_that_the_pieces_cannot_hold(B, value, d, monkeypatch):
    # one such feature must reach its neighbours as an fp32 sum would and nobody else: the same results as the list form
    rowptr, col, gp = directed_batch([5, 40, 70] * 30, 0.3, seed=3)
    monkeypatch.setenv("HAG_COMPONENT_DENSE", "2")
    dense = B.hag_search_batched(rowptr, col, gp, 0.0).upload()
    monkeypatch.setenv("HAG_COMPONENT_DENSE", "0")
    lists = B.hag_search_batched(rowptr, col, gp, 0.0).upload()
    x = synth.features_f32(rowptr.size - 1, d, 4)
    if abs(value) < 1:
        x[:] = np.float32(value) * np.random.default_rng(5).integers(-3, 4, x.shape)   # sums of such values, nothing to hide them
    else:
        x[20, 3] = x[60, d - 1] = value
    xd = torch.from_numpy(x).cuda()
    for op in ("sum", "mean", "gcn"):
        for a, b in ((dense.forward(xd, op), lists.forward(xd, op)), (dense.backward(xd, op), lists.backward(xd, op))):
            a, b = a.cpu().numpy().astype(np.float64), b.cpu().numpy().astype(np.float64)
            assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isinf(a), np.isinf(b))
            fine = np.isfinite(b)
            assert np.array_equal(a[~fine & ~np.isnan(b)], b[~fine & ~np.isnan(b)])
            # two fp32 sums of at most 70 terms: 70 * 2^-24 of the sum of magnitudes each (subnormal results: half a unit in the last place per term)
            assert np.all(np.abs(a[fine] - b[fine]) <= 1e-5 * np.abs(x[np.isfinite(x)]).max() * 70)


@pytest.mark.parametrize("parts", ["0", "2", "4"])
def test_list_form(B, parts, monkeypatch):
    # what sparse batches of larger graphs run at narrow widths, and int32 features always
    monkeypatch.setenv("HAG_COMPONENT_DENSE", "0")
    monkeypatch.setenv("HAG_COMPONENT_PARTS", parts)
    rowptr, col, gp = directed_batch([3, 20, 40] * 25, 0.3, seed=8)
    h = B.hag_search_batched(rowptr, col, gp, 0.25).upload()
    x = synth.features_f32(rowptr.size - 1, 64, 9)
    xd = torch.from_numpy(x).cuda()
    for op in ("sum", "mean", "gcn"):
        y, s, _ = oracle.naive_forward(rowptr, col, x, op)
        gx, gs = oracle.naive_backward(rowptr, col, x, op)
        assert np.all(np.abs(h.forward(xd, op).cpu().numpy() - y) <= 1e-5 * s), op
        assert np.all(np.abs(h.backward(xd, op).cpu().numpy() - gx) <= 1e-5 * gs), op


@pytest.mark.parametrize("d", [12, 64])
def test_small_values_are_summed_like_any_other(B, d, monkeypatch):
    # features and gradients that have underflowed partly or all the way (down to the smallest subnormal) beside ordinary ones
    rowptr, col, gp = directed_batch([5, 40, 70, 256] * 20, 0.3, seed=6)
    monkeypatch.setenv("HAG_COMPONENT_DENSE", "2")
    h = B.hag_search_batched(rowptr, col, gp, 0.0).upload()
    rng = np.random.default_rng(7)
    n = rowptr.size - 1
    ordinary = synth.features_f32(n, d, 8)
    spread = (rng.normal(size=(n, d)) * 2.0 ** rng.integers(-149, 1, (n, d))).astype(np.float32)
    below = (rng.integers(-5, 6, (n, d)) * 2.0 ** -149).astype(np.float32)
    assert np.count_nonzero(below) > 0 and h.route("sum", d=d) == "dense"
    for x in (spread, np.where(rng.random((n, d)) < 0.1, below, ordinary), below):
        xd = torch.from_numpy(x).cuda()
        for op in ("sum", "mean", "gcn"):
            y, s, _ = oracle.naive_forward(rowptr, col, x, op)
            gx, gs = oracle.naive_backward(rowptr, col, x, op)
            # fp32 rounding as in the other tests; below 2^-126 fp32 has units of 2^-149, so there a rounding is off by up to half of that: one for the
            # sum and one for its factor going forward, one per factor times gradient (257 terms at most) and one for the sum going back
            assert np.all(np.abs(h.forward(xd, op).cpu().numpy() - y) <= 1e-5 * s + 1.01 * 2.0 ** -149), op
            assert np.all(np.abs(h.backward(xd, op).cpu().numpy() - gx) <= 1e-5 * gs + 258 * 2.0 ** -150), op
