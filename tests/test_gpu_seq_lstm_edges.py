"""LSTM aggregator: sizes at the edges of the kernels' tiles, and numbers at the edges of the fp16 and bf16 pieces that its products run in.

Forward: gate tiles of 8 hidden units, 16 columns per product step, variants for hidden up to 32, 64 and 128; the input half of the gates runs
over 64 nodes at a time, d padded to 8.  Backward: node sums over ranges of cells that cut through a node's cells (one node in every list)."""
import numpy as np
import pytest

from oracle import lstm

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1906_03707_amd import binding
    binding.lib()
    return binding


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()


def lists(n, seed, hub=False):
    rng = np.random.default_rng(seed)
    rows = [rng.integers(0, n, int(k)) for k in rng.integers(0, 7, n)]
    if hub:
        rows = [np.concatenate([[3], r]) for r in rows]       # node 3 starts every list: its cells fill many ranges of the node sums
    rowptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int64)
    return rowptr, np.concatenate(rows).astype(np.int32)


@pytest.mark.parametrize("d,hidden", [(4, 8), (12, 24), (20, 32), (8, 40), (248, 8), (188, 64), (60, 56), (8, 72), (132, 88), (12, 120), (128, 128)])
@pytest.mark.parametrize("hub", [False, True])
def test_sizes(B, d, hidden, hub):
    n = 700 if hub else 131
    rowptr, col = lists(n, d + hidden, hub)
    rng = np.random.default_rng(hidden)
    x, w_ih, w_hh, b, g = (dev(rng.normal(0, s, shape)) for s, shape in ((1, (n, d)), (0.3, (4 * hidden, d)), (0.3, (4 * hidden, hidden)), (0.3, 4 * hidden), (1, (n, hidden))))
    f64 = lambda t: t.cpu().numpy().astype(np.float64)
    want_a, _ = lstm.naive_aggregate(rowptr, col, f64(x), f64(w_ih), f64(w_hh), f64(b))
    want = lstm.naive_aggregate_backward(rowptr, col, f64(x), f64(w_ih), f64(w_hh), f64(b), f64(g))
    for cap in (0, int(col.size)):
        h = B.SeqHag(rowptr, col, cap).upload()
        # pre-activations of up to 256 terms of size 1 carry 256 * 2^-24 = 1.5e-5 at most, the gates' slopes are below 1
        assert np.abs(f64(h.lstm_forward(x, w_ih, w_hh, b)) - want_a).max() <= 1.5e-5
        a, ws = h.lstm_forward_train(x, w_ih, w_hh, b)
        for got, ref in zip(h.lstm_backward(x, w_ih, w_hh, g, ws), want):
            # norm-wise, the bar of the other gradient tests
            assert np.linalg.norm(f64(got) - ref) <= 2e-5 * max(np.linalg.norm(ref), 1e-30)
        h.check()


def test_infinite_and_nan_features_stay_with_their_readers(B):
    # an infinite feature saturates the gates of the cells that read it, a NaN spreads to the lists that hold it, and to nobody else
    n, d, hidden = 200, 16, 40
    rowptr, col = lists(n, 5)
    rng = np.random.default_rng(6)
    x, w_ih, w_hh, b = rng.normal(0, 1, (n, d)), rng.normal(0, 0.3, (4 * hidden, d)), rng.normal(0, 0.3, (4 * hidden, hidden)), rng.normal(0, 0.3, 4 * hidden)
    h = B.SeqHag(rowptr, col, int(col.size)).upload()
    clean = h.lstm_forward(dev(x), dev(w_ih), dev(w_hh), dev(b)).cpu().numpy()
    x[7, 2], x[9, 0] = np.inf, np.nan
    got = h.lstm_forward(dev(x), dev(w_ih), dev(w_hh), dev(b)).cpu().numpy()
    x32 = [a.astype(np.float32).astype(np.float64) for a in (x, w_ih, w_hh, b)]
    with np.errstate(all="ignore"):
        want, _ = lstm.naive_aggregate(rowptr, col, *x32)
    holds = lambda u: np.array([u in col[rowptr[v]:rowptr[v + 1]] for v in range(n)])   # noqa: E731
    assert holds(7).any() and holds(9).any()
    assert np.array_equal(np.isnan(got).any(1), holds(9))
    untouched = ~holds(7) & ~holds(9)
    assert np.array_equal(got[untouched], clean[untouched])
    fine = holds(7) & ~holds(9)
    assert np.abs(got[fine] - want[fine]).max() <= 1e-5


@pytest.mark.parametrize("d,hidden", [(4, 8), (36, 32), (68, 56), (132, 64), (64, 72), (128, 128)])
def test_gradients_scale_with_the_gradient_they_come_from(B, d, hidden):
    # The backward pass is linear in g: over the plain lists (no atomics, so bit-reproducible) a power of two passes through every product, piece
    # and sum unchanged.  2^60 and 2^-60 leave the smallest pieces of a product (2^-16 of it) far from the ends of the fp32 range.
    n = 173
    rowptr, col = lists(n, hidden)
    rng = np.random.default_rng(d)
    x, w_ih, w_hh, b, g = (dev(rng.normal(0, s, shape)) for s, shape in ((1, (n, d)), (0.3, (4 * hidden, d)), (0.3, (4 * hidden, hidden)), (0.3, 4 * hidden), (1, (n, hidden))))
    h = B.SeqHag(rowptr, col, 0).upload()

    def grads(g_a):
        _, ws = h.lstm_forward_train(x, w_ih, w_hh, b)
        return h.lstm_backward(x, w_ih, w_hh, g_a, ws)

    plain = grads(g)
    for k in (60, -60):
        for one, other in zip(plain, grads(g * 2.0 ** k)):
            assert torch.equal(one * 2.0 ** k, other)
    # an infinite gradient of one node reaches what that node's list reads, and no other row of g_x
    v = int(np.argmax(np.diff(rowptr)))
    g[v, 1] = float("inf")
    g_x, g_w_ih, g_w_hh, g_b = grads(g)
    read = np.unique(col[rowptr[v]:rowptr[v + 1]])
    others = np.setdiff1d(np.arange(n), read)
    assert not torch.isfinite(g_x[read]).all(1).any() and not torch.isfinite(g_b).any()
    assert torch.equal(g_x[others], plain[0][others])


@pytest.mark.parametrize("d,hidden", [(8, 8), (16, 40), (20, 64), (12, 120)])
def test_units_of_very_different_weights(B, d, hidden):
    # Every gate row's weights are brought to a common size by a power of two of their own.  Side by side: units of ordinary weights, units whose rows are 2^-12 throughout, units of
    # recurrent weights 2^-60 and 0, a weight that fp16 cannot hold (1e5, on a unit whose output gate lets e^-11 through), and features outside fp16's range in both directions.
    n = 150
    rowptr, col = lists(n, hidden)
    rng = np.random.default_rng(d)
    kind = np.arange(hidden) % 4
    x, w_ih, w_hh, b = rng.normal(0, 1, (n, d)), rng.normal(0, 0.3, (4 * hidden, d)), rng.normal(0, 0.3, (4 * hidden, hidden)), rng.normal(0, 0.3, 4 * hidden)
    w_hh *= np.tile(np.array([1.0, 2.0 ** -12, 2.0 ** -60, 0.0])[kind], 4)[:, None]
    w_ih *= np.tile(np.where(kind == 1, 2.0 ** -12, 1.0), 4)[:, None]
    b *= np.tile(np.where(kind == 1, 2.0 ** -12, 1.0), 4)
    b[3 * hidden + 7] -= 11
    w_hh[2 * hidden + 4, 7] = 1e5
    x[3, 1], x[5, 2] = 1e25, 1e-25
    f32 = [a.astype(np.float32).astype(np.float64) for a in (x, w_ih, w_hh, b)]
    want, _ = lstm.naive_aggregate(rowptr, col, *f32)
    without = [a.copy() for a in f32]
    without[2][np.tile(kind == 1, 4)] = 0
    fine = ~np.array([3 in col[rowptr[v]:rowptr[v + 1]] for v in range(n)])     # (the feature of 1e25 times 2^-12 saturates a small unit too)
    # Gate functions leave absolute errors of about 1e-7, and six cells at most add them up: 2e-6 as in the test of gates below.  A small unit's are multiplied by gates of one half
    # (c is 2^-13, h half of it): 5e-7, a hundredth of what its recurrent weights bring about.
    bar = np.where(kind == 1, 5e-7, 2e-6)
    assert np.abs(lstm.naive_aggregate(rowptr, col, *without)[0] - want)[fine][:, kind == 1].max() > 20 * 5e-7
    for cap in (0, int(col.size)):
        h = B.SeqHag(rowptr, col, cap).upload()
        got = h.lstm_forward(dev(x), dev(w_ih), dev(w_hh), dev(b))
        error = np.abs(got.cpu().numpy() - want)
        assert error.max() <= 2e-6 and (error[fine].max(0) <= bar).all()
        a, _ = h.lstm_forward_train(dev(x), dev(w_ih), dev(w_hh), dev(b))
        assert torch.equal(a, got)


@pytest.mark.parametrize("d,hidden", [(8, 8), (16, 32), (16, 40), (20, 64), (12, 72), (8, 128)])
def test_gradients_of_very_different_sizes(B, d, hidden):
    # The product of the reverse pass brings a path's gradients and a column of weights to a common size each.  Side by side: nodes of gradients of 2^-40, 1, 0 and 2^20, which read nodes
    # of their own kind only, so that every kind's rows of g_x are held against their own norm; and units whose columns of weights are 2^3, 1, 2^-12, 2^-60 and 0 times the others and
    # whose own outputs have no gradient but for the first two: what reaches the small ones went through those columns, and so did their rows of the weight gradients.
    n = 152
    rowptr, col = lists(n, hidden)
    kind = np.arange(n) % 4
    col = (col // 4 * 4 + np.repeat(kind, np.diff(rowptr))).astype(np.int32)
    rng = np.random.default_rng(d)
    x, w_ih, w_hh, b, g = rng.normal(0, 1, (n, d)), rng.normal(0, 0.3, (4 * hidden, d)), rng.normal(0, 0.3, (4 * hidden, hidden)), rng.normal(0, 0.3, 4 * hidden), rng.normal(0, 1, (n, hidden))
    unit = np.arange(hidden) % 5
    w_hh *= np.array([8.0, 1.0, 2.0 ** -12, 2.0 ** -60, 0.0])[unit]
    g *= np.array([2.0 ** -40, 1.0, 0.0, 2.0 ** 20])[kind][:, None] * (unit < 2)
    f32 = [a.astype(np.float32).astype(np.float64) for a in (x, w_ih, w_hh, b, g)]
    want = lstm.naive_aggregate_backward(rowptr, col, *f32)
    for cap in (0, int(col.size)):
        h = B.SeqHag(rowptr, col, cap).upload()
        _, ws = h.lstm_forward_train(dev(x), dev(w_ih), dev(w_hh), dev(b))
        g_x, *weights = (t.cpu().numpy() for t in h.lstm_backward(dev(x), dev(w_ih), dev(w_hh), dev(g), ws))
        # norm-wise, the bar of the other gradient tests (columns of weights of 2.4 hand errors on that much larger)
        for k in range(4):
            assert np.linalg.norm(g_x[kind == k] - want[0][kind == k]) <= 2e-5 * np.linalg.norm(want[0][kind == k])
        for got, ref in zip(weights, want[1:]):
            for k in range(5):
                rows = np.tile(unit == k, 4)
                assert np.linalg.norm(got[rows] - ref[rows]) <= 2e-5 * np.linalg.norm(ref[rows])
        h.check()


@pytest.mark.parametrize("d,hidden", [(8, 8), (16, 32), (16, 40), (20, 64), (12, 72), (12, 120)])
def test_gates_of_very_different_weights(B, d, hidden):
    # Every gate row has a factor of its own: forget gates that stay open (f = 1) with weights a million times those of the other gates leave the others all their bits.
    n = 150
    rowptr, col = lists(n, hidden)
    rng = np.random.default_rng(d)
    x, w_ih, w_hh, b = rng.normal(0, 1, (n, d)), rng.normal(0, 0.3, (4 * hidden, d)), rng.normal(0, 0.3, (4 * hidden, hidden)), rng.normal(0, 0.3, 4 * hidden)
    w_hh[hidden:2 * hidden] *= 1e6
    b[hidden:2 * hidden] = 1e9
    want, _ = lstm.naive_aggregate(rowptr, col, *(a.astype(np.float32).astype(np.float64) for a in (x, w_ih, w_hh, b)))
    for cap in (0, int(col.size)):
        h = B.SeqHag(rowptr, col, cap).upload()
        got = h.lstm_forward(dev(x), dev(w_ih), dev(w_hh), dev(b))
        # six cells at most, each adding i g (an error of about 3e-7: two gate functions and pre-activations of size 3) to c; |h| changes by less than c
        assert np.abs(got.cpu().numpy() - want).max() <= 2e-6
        a, _ = h.lstm_forward_train(dev(x), dev(w_ih), dev(w_hh), dev(b))
        assert torch.equal(a, got)


@pytest.mark.parametrize("d,hidden", [(8, 8), (16, 40), (12, 120)])
def test_pre_activations_have_the_range_of_fp32(B, d, hidden):
    # features of 1e36 whose terms have opposite signs, rows of large weights in either matrix: finite sums that saturate the gates
    n = 150
    rowptr, col = lists(n, hidden)
    rng = np.random.default_rng(d)
    x, w_ih, w_hh, b = rng.normal(0, 1, (n, d)), rng.normal(0, 0.3, (4 * hidden, d)), rng.normal(0, 0.3, (4 * hidden, hidden)), rng.normal(0, 0.3, 4 * hidden)
    x[:40, 1], x[:40, 2] = 1e36, -1e36
    w_ih[3, 3:] *= 1e34
    w_hh[hidden + 5] *= 1e36
    with np.errstate(over="ignore"):
        want, _ = lstm.naive_aggregate(rowptr, col, *(a.astype(np.float32).astype(np.float64) for a in (x, w_ih, w_hh, b)))
    assert np.isin(col, np.arange(40)).sum() > 30
    for cap in (0, int(col.size)):
        h = B.SeqHag(rowptr, col, cap).upload()
        assert np.abs(h.lstm_forward(dev(x), dev(w_ih), dev(w_hh), dev(b)).cpu().numpy() - want).max() <= 1e-5


@pytest.mark.parametrize("d,hidden", [(8, 8), (16, 32), (16, 40), (20, 64), (12, 72), (8, 128)])
def test_gradients_of_units_that_do_not_see_each_other(B, d, hidden):
    # even units read even features and even units, odd ones the others, and the even ones' gradients are 2^26 times as large: the odd ones keep all their bits, although
    # a path's gradients are brought into range together
    n = 150
    rowptr, col = lists(n, hidden)
    rng = np.random.default_rng(d)
    x, w_ih, w_hh, b, g = rng.normal(0, 1, (n, d)), rng.normal(0, 0.3, (4 * hidden, d)), rng.normal(0, 0.3, (4 * hidden, hidden)), rng.normal(0, 0.3, 4 * hidden), rng.normal(0, 1, (n, hidden))
    odd, odd_x = np.arange(hidden) % 2, np.arange(d) % 2
    w_ih *= np.tile(odd[:, None] == odd_x[None, :], (4, 1))
    w_hh *= np.tile(odd[:, None] == odd[None, :], (4, 1))
    g *= np.where(odd, 1.0, 2.0 ** 26)
    want = lstm.naive_aggregate_backward(rowptr, col, *(a.astype(np.float32).astype(np.float64) for a in (x, w_ih, w_hh, b, g)))
    of_odd = ((slice(None), odd_x == 1), *[np.tile(odd == 1, 4)] * 3)
    for cap in (0, int(col.size)):
        h = B.SeqHag(rowptr, col, cap).upload()
        _, ws = h.lstm_forward_train(dev(x), dev(w_ih), dev(w_hh), dev(b))
        for got, ref, rows in zip(h.lstm_backward(dev(x), dev(w_ih), dev(w_hh), dev(g), ws), want, of_odd):
            # gradients that see no larger ones beside them have errors of up to 6e-7 here
            assert np.linalg.norm(got.cpu().numpy()[rows] - ref[rows]) <= 2e-6 * np.linalg.norm(ref[rows])


@pytest.mark.parametrize("d,hidden", [(8, 8), (16, 40), (12, 120)])
def test_weights_and_gradients_near_the_ends_of_fp32(B, d, hidden):
    # a column of weights that saturates the gates (3e38) under gradients of 1e-20, and gradients of 2^122
    n = 150
    rowptr, col = lists(n, hidden)
    rng = np.random.default_rng(d)
    x, w_ih, w_hh, b, g = rng.normal(0, 1, (n, d)), rng.normal(0, 0.3, (4 * hidden, d)), rng.normal(0, 0.3, (4 * hidden, hidden)), rng.normal(0, 0.3, 4 * hidden), rng.normal(0, 1, (n, hidden))
    large = w_hh.copy()
    large[:, 0] = 0
    large[:hidden // 2, 0] = 3e38
    h = B.SeqHag(rowptr, col, 0).upload()
    for w, scale in ((large, 1e-20), (w_hh, 2.0 ** 122)):
        with np.errstate(over="ignore"):
            want = lstm.naive_aggregate_backward(rowptr, col, *(a.astype(np.float32).astype(np.float64) for a in (x, w_ih, w, b, g * scale)))
        _, ws = h.lstm_forward_train(dev(x), dev(w_ih), dev(w), dev(b))
        for got, ref in zip(h.lstm_backward(dev(x), dev(w_ih), dev(w), dev(g * scale), ws), want):
            size = np.abs(ref).max()
            assert np.linalg.norm(got.cpu().numpy() / size - ref / size) <= 2e-5 * np.linalg.norm(ref / size)


@pytest.mark.parametrize("d,hidden", [(8, 8), (36, 32), (64, 72), (132, 64)])
def test_weight_gradients_of_features_at_the_ends_of_fp32(B, d, hidden):
    # g_w_ih is cut into pieces that neither hold features above 3.39e38 nor all bits of a column of features of 1e-36, or of gradients of 1e-35: those take fp32
    # products.  The large feature's weights are zero, so that it changes nothing else; the other columns are as they are without it.
    n = 150
    rowptr, col = lists(n, hidden)
    rng = np.random.default_rng(d)
    x, w_ih, w_hh, b, g = rng.normal(0, 1, (n, d)), rng.normal(0, 0.3, (4 * hidden, d)), rng.normal(0, 0.3, (4 * hidden, hidden)), rng.normal(0, 0.3, 4 * hidden), rng.normal(0, 1, (n, hidden))
    w_ih[:, 2] = 0
    small, huge = x.copy(), x.copy()
    small[:, 1] *= 1e-36
    huge[int(col[0]), 2] = 3.4e38
    h = B.SeqHag(rowptr, col, 0).upload()
    for feats, scale in ((small, 1.0), (small, 2.0 ** 100), (huge, 1e-3), (x, 1e-35)):
        want = lstm.naive_aggregate_backward(rowptr, col, *(a.astype(np.float32).astype(np.float64) for a in (feats, w_ih, w_hh, b, g * scale)))[1]
        _, ws = h.lstm_forward_train(dev(feats), dev(w_ih), dev(w_hh), dev(b))
        got = h.lstm_backward(dev(feats), dev(w_ih), dev(w_hh), dev(g * scale), ws)[1].cpu().numpy().astype(np.float64)
        # other columns have errors of up to 6e-7
        assert (np.linalg.norm(got - want, axis=0) <= 2e-6 * np.linalg.norm(want, axis=0)).all()


@pytest.mark.parametrize("d,hidden", [(8, 8), (16, 32), (16, 40), (20, 64), (12, 72), (12, 120)])
@pytest.mark.parametrize("closed", [6, 12, 18, 30])
def test_recurrent_weight_gradients_of_nearly_closed_units(B, d, hidden, closed):
    # output gates of every second unit e^-6 to e^-30 open: their h, and with it the columns of g_w_hh that belong to them, are that much smaller than the others and keep their bits
    n = 150
    rowptr, col = lists(n, hidden)
    rng = np.random.default_rng(d)
    x, w_ih, w_hh, b, g = rng.normal(0, 1, (n, d)), rng.normal(0, 0.3, (4 * hidden, d)), rng.normal(0, 0.3, (4 * hidden, hidden)), rng.normal(0, 0.3, 4 * hidden), rng.normal(0, 1, (n, hidden))
    b[3 * hidden + 1::2] -= closed
    want = lstm.naive_aggregate_backward(rowptr, col, *(a.astype(np.float32).astype(np.float64) for a in (x, w_ih, w_hh, b, g)))[2]
    for cap in (0, int(col.size)):
        h = B.SeqHag(rowptr, col, cap).upload()
        _, ws = h.lstm_forward_train(dev(x), dev(w_ih), dev(w_hh), dev(b))
        got = h.lstm_backward(dev(x), dev(w_ih), dev(w_hh), dev(g), ws)[2].cpu().numpy()
        # exp of a pre-activation of -closed - 4 at most in size: its rounding, half of 2^-24 of that and as much from the sum and the scaling, is a relative error of h
        bar = 2e-6 + 3 * (closed + 4) * 2.0 ** -24
        for cols in (slice(0, None, 2), slice(1, None, 2)):
            assert np.linalg.norm(got[:, cols] - want[:, cols]) <= bar * np.linalg.norm(want[:, cols])


@pytest.mark.parametrize("hidden", [8, 64, 72])
def test_an_infinite_gradient_stays_infinite_in_the_weight_gradients(B, hidden):
    # lists of one: dG of node v is infinite where g is, and a sum of one infinite and many finite products has its sign; h before the step is zero, so that g_w_hh has no number there
    n, d = 96, 8
    rng = np.random.default_rng(hidden)
    rowptr, col = np.arange(n + 1, dtype=np.int64), rng.permutation(n).astype(np.int32)
    x, w_ih, w_hh, b, g = rng.normal(0, 1, (n, d)), rng.normal(0, 0.3, (4 * hidden, d)), rng.normal(0, 0.3, (4 * hidden, hidden)), rng.normal(0, 0.3, 4 * hidden), rng.normal(0, 1, (n, hidden))
    g[5, 1] = np.inf
    h = B.SeqHag(rowptr, col, 0).upload()
    _, ws = h.lstm_forward_train(dev(x), dev(w_ih), dev(w_hh), dev(b))
    _, g_w_ih, g_w_hh, g_b = (t.cpu().numpy() for t in h.lstm_backward(dev(x), dev(w_ih), dev(w_hh), dev(g), ws))
    rows = np.arange(4) * hidden + 1
    rows = rows[[0, 2, 3]]       # (the forget gate's is infinity times the zero state)
    assert np.isinf(g_b[rows]).all() and np.isinf(g_w_ih[rows]).all()
    assert np.array_equal(np.sign(g_w_ih[rows]), np.sign(g_b[rows])[:, None] * np.sign(x[col[5]]))
    others = np.setdiff1d(np.arange(4 * hidden), np.arange(4) * hidden + 1)
    assert np.isfinite(g_w_ih[others]).all() and np.isfinite(g_w_hh[others]).all() and np.isfinite(g_b[others]).all()


@pytest.mark.parametrize("hidden", [8, 32, 64])
@pytest.mark.parametrize("masked", [False, True])
def test_no_error_adds_up_over_many_cells(B, hidden, masked):
    # The matrix cores cut sums downwards; the sign of the power of two that brings gradients into range alternates over paths, tiles, steps and chunks, so that cuts cancel.  Gradients that go
    # with it, of every second node over lists of one length, which come as paths in order: as good as all of them.
    n, d, length = 60000, 16, 8
    gen = torch.Generator(device="cuda").manual_seed(hidden)
    normal = lambda s, *shape: torch.randn(*shape, generator=gen, device="cuda") * s   # noqa: E731
    idx = torch.randint(0, n, (n, length), generator=gen, device="cuda")
    x, w_ih, w_hh, b, g = normal(1, n, d), normal(0.3, 4 * hidden, d), normal(0.3, 4 * hidden, hidden), normal(0.3, 4 * hidden), normal(1, n, hidden)
    if masked:
        g[1::2] = 0
    h = B.SeqHag(np.arange(n + 1, dtype=np.int64) * length, idx.cpu().numpy().astype(np.int32).ravel(), 0).upload()
    _, ws = h.lstm_forward_train(x, w_ih, w_hh, b)
    got = h.lstm_backward(x, w_ih, w_hh, g, ws)
    leaves = [t.double().requires_grad_() for t in (x, w_ih, w_hh, b)]
    gates = leaves[0] @ leaves[1].t() + leaves[3]
    hs = cs = torch.zeros(n, hidden, dtype=torch.float64, device="cuda")
    for t in range(length):
        i, f, u, o = (gates[idx[:, t]] + hs @ leaves[2].t()).split(hidden, 1)
        cs = torch.sigmoid(f) * cs + torch.sigmoid(i) * torch.tanh(u)
        hs = torch.sigmoid(o) * torch.tanh(cs)
    # Errors are 2e-7 to 4e-7 here (with fp32 products up to 8e-7); with one sign throughout those of g_w_hh and g_b reach 1e-6 at 32 units and 3e-6 at 64.
    for one, ref in zip(got, torch.autograd.grad(hs, leaves, g.double())):
        assert ((one.double() - ref).norm() <= 8e-7 * ref.norm()).item()
