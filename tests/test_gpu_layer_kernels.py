"""hag_weight_grad and hag_softmax_loss against 64-bit sums: edges of their tiles (4 rows, 64 columns of x, 16 and 64 of g; 16 and 64 lanes per row of the
loss), and the functions of layers.py around them where autograd is used in other ways than a plain backward pass."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
EPS = 2.0 ** -24


@pytest.fixture(scope="module")
def B():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1906_03707_amd import binding
    binding.lib()
    return binding


@pytest.mark.parametrize("n", [0, 1, 3, 5, 64, 515, 4099, 70001])
@pytest.mark.parametrize("d,k", [(4, 1), (60, 7), (64, 16), (68, 17), (128, 33), (132, 65), (4, 4096), (4096, 5)])
def test_weight_grad(B, n, d, k):
    gen = torch.Generator(device="cuda").manual_seed(n + d)
    x, g = torch.randn(n, d, device="cuda", generator=gen), torch.randn(n, k, device="cuda", generator=gen)
    want, size = x.double().t() @ g.double(), x.double().abs().t() @ g.double().abs()
    # any order of n fp32 additions of rounded products: n + 1 roundings at most on the way of a term
    assert bool(((B.weight_grad(x, g).double() - want).abs() <= (n + 1) * EPS * size).all())


@pytest.mark.parametrize("n", [1, 31, 33, 128, 129, 5001])
@pytest.mark.parametrize("d,k", [(4, 1), (16, 16), (20, 17), (64, 33), (132, 64), (256, 65), (512, 32), (1024, 7)])
def test_narrow_product(B, n, d, k):
    gen = torch.Generator(device="cuda").manual_seed(n + d)
    x, w, a = (torch.randn(*s, device="cuda", generator=gen) for s in ((n, d), (d, k), (n, k)))
    a[0, 0] = float("nan")                                 # (a ReLU passes a NaN on, and its gradient)
    for relu, mask in ((False, None), (True, None), (False, a), (True, a)):
        z = torch.relu(x) if relu else x
        want, size = z.double() @ w.double(), z.double().abs() @ w.double().abs()
        if mask is not None:
            want = torch.where(mask <= 0, 0.0, want)
        for got in (B.narrow_product(x, w, relu=relu, mask=mask), B.narrow_product(x, w.t().contiguous(), transposed=True, relu=relu, mask=mask)):
            assert bool(((got.double() - want).abs() <= (d + 1) * EPS * size).all())
    g = torch.randn(n, k, device="cuda", generator=gen)
    z = torch.relu(x).double()
    assert bool(((B.weight_grad(x, g, relu=True).double() - z.t() @ g.double()).abs() <= (n + 1) * EPS * (z.t() @ g.double().abs())).all())


@pytest.mark.parametrize("n", [1, 17, 1000, 40001])
@pytest.mark.parametrize("classes", [1, 2, 16, 63, 64, 65, 256, 257, 1000])
def test_softmax_loss(B, n, classes):
    gen = torch.Generator(device="cuda").manual_seed(n + classes)
    z = 5 * torch.randn(n, classes, device="cuda", generator=gen)
    z[0] += 1e4                                            # far from where exp() is finite
    labels = torch.randint(0, classes, (n,), device="cuda", generator=gen)
    labels[1::5] = -100
    ref = z.double().requires_grad_()
    want = torch.nn.functional.cross_entropy(ref, labels)
    want.backward()
    loss, counted = B.softmax_loss(z, labels)
    # a row's loss is a difference of numbers of the size of its logits (top + log-sum and the label's): a few roundings of those
    assert abs(loss.item() - want.item()) <= 8 * EPS * (abs(want.item()) + z.abs().max(1).values.sub(z[:, 0].abs()).abs().max().item() + 40)
    assert counted.item() == (labels != -100).sum().item()
    g = B.softmax_loss_grad(z, labels, counted, torch.tensor(3.0, device="cuda"))
    # probabilities: exp of a difference that is exact to half an ulp of up to 40, times a reciprocal of a sum
    assert bool(((g.double() - 3 * ref.grad).abs() <= 3 / counted.item() * EPS * 100).all())


def test_softmax_loss_of_what_is_no_number(B):
    z = torch.randn(40, 16, device="cuda")
    labels = torch.arange(40, device="cuda") % 16
    ce = torch.nn.functional.cross_entropy
    for value in (float("nan"), float("inf"), float("-inf")):
        y = z.clone()
        y[7, 3] = value
        assert torch.equal(torch.isfinite(B.softmax_loss(y, labels)[0]), torch.isfinite(ce(y, labels))), value
    assert torch.isnan(B.softmax_loss(z, torch.full_like(labels, -100))[0])
    labels[5] = 16                                         # no class
    assert torch.isnan(B.softmax_loss(z, labels)[0])


def test_products_and_loss_under_autograd(B):
    from paper_1906_03707_amd import layers
    gen = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen)   # noqa: E731
    x, w, labels = rnd(900, 20), rnd(20, 6), torch.randint(0, 6, (900,), device="cuda", generator=gen)
    labels[::9] = -100

    def model(product, loss, xx, ww):
        return loss(product(xx, ww), labels)

    own = (layers.product, layers.softmax_loss)
    lib = (torch.matmul, torch.nn.functional.cross_entropy)
    for x_grad in (False, True):
        results = []
        for how in (own, lib):
            xx, ww = x.clone().requires_grad_(x_grad), w.clone().requires_grad_()
            inputs = (xx, ww) if x_grad else (ww,)
            value = model(*how, xx, ww)
            first = torch.autograd.grad(value, inputs, create_graph=True)
            second = torch.autograd.grad(sum((g ** 2).sum() for g in first), inputs)
            plain = torch.autograd.grad(model(*how, xx, ww) * 2, inputs)
            kept = []
            with torch.autograd.graph.saved_tensors_hooks(lambda t: kept.append(t) or t.cpu(), lambda t: t.cuda()):
                hooked = model(*how, xx, ww)
            assert kept
            results.append((value, *first, *second, *plain, *torch.autograd.grad(hooked, inputs)))
        for a, b in zip(*results):
            assert a.shape == b.shape and (a - b).norm().item() <= 1e-5 * b.norm().item()
    with torch.no_grad():
        assert torch.equal(layers.product(x, w), x @ w)
    assert torch.equal(layers.product(x.to_sparse(), w.requires_grad_()), x.to_sparse() @ w)
    value = layers.softmax_loss(x, labels.clamp(min=0))
    value += 1                                             # in place, as with the library's
    with pytest.raises(RuntimeError):
        layers.product(x, w[:19])
    probabilities = torch.softmax(rnd(900, 20), 1)
    assert torch.equal(layers.softmax_loss(x, probabilities), torch.nn.functional.cross_entropy(x, probabilities))


@pytest.mark.parametrize("naive", [False, True])
@pytest.mark.parametrize("x_grad", [False, True])
def test_gcn_loss_as_one_node_equals_the_composed_form(B, naive, x_grad):
    from paper_1906_03707_amd import layers, synth
    rowptr, col = synth.holme_kim(900, 6, 0.5, seed=5)
    h = B.hag_search(rowptr, col, 200).upload()
    n = rowptr.size - 1
    gen = torch.Generator(device="cuda").manual_seed(6)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen)   # noqa: E731
    data = rnd(n, 20), rnd(20, 12), rnd(12, 8)
    labels = torch.randint(0, 8, (n,), device="cuda", generator=gen)
    labels[::7] = -100
    results = []
    for form in (lambda *a: layers.gcn2_loss(*a, naive=naive), lambda *a: layers._gcn2_composed(*a, naive, None)):
        x, w1, w2 = (t.clone().requires_grad_(k > 0 or x_grad) for k, t in enumerate(data))
        inputs = (x, w1, w2) if x_grad else (w1, w2)
        loss = form(h, x, w1, w2, labels)
        plain = torch.autograd.grad(loss, inputs, retain_graph=True)
        again = torch.autograd.grad(3 * loss, inputs)
        loss = form(h, x, w1, w2, labels)
        first = torch.autograd.grad(loss, inputs, create_graph=True)
        second = torch.autograd.grad(sum((g ** 2).sum() for g in first), inputs, allow_unused=True)
        only = torch.autograd.grad(form(h, x.detach(), w1.detach(), w2, labels), (w2,))
        with torch.autograd.graph.saved_tensors_hooks(lambda t: t.cpu(), lambda t: t.cuda()):
            hooked = form(h, x, w1, w2, labels)
        results.append((loss, *plain, *again, *first, *second, *only, *torch.autograd.grad(hooked, inputs)))
    for a, b in zip(*results):
        assert (a is None) == (b is None) and (a is None or (a - b).norm().item() <= 1e-5 * b.norm().item())
    with torch.no_grad():
        assert not layers.gcn2_loss(h, *data, labels).requires_grad
    for bad in ((data[0][:-1], *data[1:]), (data[0], data[2], data[2])):
        with pytest.raises((ValueError, RuntimeError)):
            layers.gcn2_loss(h, *bad, labels)


def test_gradients_keep_no_graph_when_hooks_return_saved_tensors_as_something_else(B):
    from paper_1906_03707_amd import layers, synth
    rowptr, col = synth.holme_kim(600, 6, 0.5, seed=5)
    h = B.hag_search(rowptr, col, 100).upload()
    n = rowptr.size - 1
    gen = torch.Generator(device="cuda").manual_seed(8)
    x, w1, w2 = (torch.randn(*s, device="cuda", generator=gen) for s in ((n, 20), (20, 12), (12, 8)))
    labels = torch.randint(0, 8, (n,), device="cuda", generator=gen)
    w1.requires_grad_()
    w2.requires_grad_()
    turned = lambda t: t.t().contiguous().t() if t.dim() == 2 else t   # noqa: E731  (the same numbers, columns first)
    with torch.autograd.graph.saved_tensors_hooks(lambda t: t.detach(), turned):
        loss = layers.gcn2_loss(h, x, w1, w2, labels)
    got, want = torch.autograd.grad(loss, (w1, w2)), torch.autograd.grad(layers.gcn2_loss(h, x, w1, w2, labels), (w1, w2))
    for a, b in zip(got, want):
        assert not a.requires_grad and (a - b).norm().item() <= 1e-5 * b.norm().item()


@pytest.mark.parametrize("n,d,k", [(70001, 64, 16), (70001, 68, 33), (200003, 12, 70), (40000, 132, 5)])
@pytest.mark.parametrize("relu", [False, True])
def test_weight_grad_takes_every_row_once(B, n, d, k, relu):
    # small whole numbers: sums below 2^24 are exact in any order, so a row left out or taken twice shows (wavefronts go many times round their stride here)
    gen = torch.Generator(device="cuda").manual_seed(n + d + k)
    x = torch.randint(-3, 4, (n, d), device="cuda", generator=gen).float()
    g = torch.randint(1, 4, (n, k), device="cuda", generator=gen).float()
    z = torch.relu(x) if relu else x
    want = z.double().t() @ g.double()
    assert (z.double().abs().t() @ g.double()).max().item() < 1 << 24
    assert torch.equal(B.weight_grad(x, g, relu=relu), want.float())


def test_small_calls_take_the_library_and_large_ones_are_the_same_under_autograd(B):
    # (what a node of the graph in Python costs the host is more than small calls gain)
    from paper_1906_03707_amd import layers
    gen = torch.Generator(device="cuda").manual_seed(4)
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=gen)   # noqa: E731
    name = lambda t: type(t.grad_fn).__name__   # noqa: E731
    for n, d, k, own in ((1000, 64, 16, False), (16384, 64, 16, False), (8192, 128, 64, True), (32768, 16, 16, True), (1000, 256, 256, True)):
        assert (name(layers.product(rnd(n, d), rnd(d, k).requires_grad_())) == "_ProductBackward") == own, (n, d, k)
    for n, k, own in ((1000, 16, False), (16384, 16, False), (32768, 16, True), (16384, 40, True)):
        assert (name(layers.softmax_loss(rnd(n, k).requires_grad_(), torch.zeros(n, dtype=torch.int64, device="cuda"))) == "_SoftmaxLossBackward") == own, (n, k)
    x, w, labels = rnd(90000, 20), rnd(20, 6), torch.randint(0, 6, (90000,), device="cuda", generator=gen)
    labels[::9] = -100
    results = []
    for product, loss in ((layers.product, layers.softmax_loss), (torch.matmul, torch.nn.functional.cross_entropy)):
        xx, ww = x.clone().requires_grad_(), w.clone().requires_grad_()
        value = loss(product(xx, ww), labels)
        first = torch.autograd.grad(value, (xx, ww), create_graph=True)
        second = torch.autograd.grad(sum((g ** 2).sum() for g in first), (xx, ww))
        with torch.autograd.graph.saved_tensors_hooks(lambda t: t.cpu(), lambda t: t.cuda()):
            hooked = loss(product(xx, ww), labels)
        results.append((value, *first, *second, *torch.autograd.grad(loss(product(xx, ww), labels) * 2, (xx, ww)), *torch.autograd.grad(hooked, (xx, ww))))
    for a, b in zip(*results):
        assert a.shape == b.shape and (a - b).norm().item() <= 1e-5 * b.norm().item()


def test_forward_mode_derivatives_of_the_last_product_and_the_loss(B):
    # what comes after the last aggregation can be differentiated forwards, as with the library's product and loss
    from paper_1906_03707_amd import layers
    import torch.autograd.forward_ad as fw
    gen = torch.Generator(device="cuda").manual_seed(12)
    x, w, v = (torch.randn(*s, device="cuda", generator=gen) for s in ((40000, 20), (20, 16), (20, 16)))
    labels = torch.randint(0, 16, (40000,), device="cuda", generator=gen)
    tangents = []
    for product, loss in ((layers.product, layers.softmax_loss), (torch.matmul, torch.nn.functional.cross_entropy)):
        for grad in (False, True):
            with fw.dual_level():
                tangents.append(fw.unpack_dual(loss(product(x, fw.make_dual(w.clone().requires_grad_(grad), v)), labels)).tangent)
    assert all(t is not None and (t - tangents[-1]).abs().item() <= 1e-5 * tangents[-1].abs().item() for t in tangents)
