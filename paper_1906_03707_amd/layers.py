"""The two GNN layers of the paper's Table 1 around the library's aggregation calls.

The aggregation (and, for GCN, the normalisation fused into it), the gradients of the weight matrices
and the SoftMax loss are this library's kernels; the other dense parts (products with the weight
matrices, ReLU) are plain torch.  Each aggregation call can be recorded (its input and
output tensors), so that a test can hand exactly those inputs to the CPU oracle.

GCN (Table 1, GCN row; the model of Section 5.3):  h'_v = relu(W . (a_v + h_v) / (|N(v)| + 1)) with
a_v the sum over N(v).  W is linear, so the layer transforms first and aggregates at the narrow width:
h' = relu(gcn_agg(h W)), gcn_agg being op "gcn" of hag_forward.
GraphSAGE-P (Table 1, pooling row):  a_v = max over N(v) of relu(W1 h_u),  h'_v = relu(W2 [a_v, h_v]).
"""
from __future__ import annotations

import torch

from . import binding


def _plain(t):
    """A contiguous float32 matrix of the ordinary kind on the current device: what the library's kernels take."""
    return (type(t) in (torch.Tensor, torch.nn.Parameter) and t.is_cuda and t.layout == torch.strided and t.dtype == torch.float32 and t.dim() == 2
            and t.is_contiguous() and t.get_device() == torch.cuda.current_device())


def _no_tangent(*tensors):
    """None of them carries a forward-mode derivative, which the nodes below do not pass on."""
    return all(torch.autograd.forward_ad.unpack_dual(t).tangent is None for t in tensors)


def _plain_labels(labels, z):
    return (type(labels) is torch.Tensor and labels.dtype == torch.int64 and labels.dim() == 1 and labels.device == z.device and labels.is_contiguous()
            and labels.shape[0] == z.shape[0])


class _Product(torch.autograd.Function):
    """x @ w with the gradient of w, a contraction over all rows of x, by hag_weight_grad."""

    @staticmethod
    def forward(ctx, x, w):
        ctx.save_for_backward(x, w if ctx.needs_input_grad[0] else None)
        return x @ w

    @staticmethod
    def backward(ctx, g):
        x, w = ctx.saved_tensors
        g_x = g @ w.t() if w is not None else None
        if not ctx.needs_input_grad[1]:
            return g_x, None
        g = g.contiguous()
        # a backward pass that is itself differentiated needs operations that are; and x comes back from whatever hooks keep saved tensors
        own = not torch.is_grad_enabled() and _plain(x) and _plain(g) and x.data_ptr() % 16 == 0
        return g_x, binding.weight_grad(x, g) if own else x.t() @ g


def product(x, w):
    """x @ w for a tall x [n, d] and a small w [d, k].

    The gradient of w is the library's up to d * k = 65536: 65536 rows, 64 x 16 14 us against the BLAS's 82, 16 x 16 15 and 174, 256 x 256 144 and 217 (its
    error against 64 bits 2e-7 and 2e-6); beyond, it reads x and g too many times (370000 rows, 256 x 256: 784 and 878).  Below 32768 rows and 2^25 products it
    saves less than a node of the graph in Python costs the host (forward and backward 57 us, torch's 53: 16384 rows, 64 x 16; 57 and 66: 8192 rows, 128 x 64)."""
    if (torch.is_grad_enabled() and w.requires_grad and _plain(x) and _plain(w) and x.shape[1] == w.shape[0] and x.shape[1] % 4 == 0
            and 0 < w.numel() <= 65536 and max(w.shape) <= 4096 and (x.shape[0] >= 32768 or x.shape[0] * w.numel() >= 1 << 25)
            and not torch.is_autocast_enabled() and _no_tangent(x, w)):
        return _Product.apply(x, w)
    return x @ w


class _SoftmaxLoss(torch.autograd.Function):
    @staticmethod
    def forward(ctx, z, labels):
        loss, counted = binding.softmax_loss(z, labels)
        ctx.save_for_backward(z, labels, counted)
        return loss

    @staticmethod
    def backward(ctx, g):
        z, labels, counted = ctx.saved_tensors
        if torch.is_grad_enabled() or not (_plain(z) and labels.is_contiguous()):   # (as above)
            kept = (labels != -100)[:, None]
            one_hot = torch.nn.functional.one_hot(torch.where(kept[:, 0], labels, 0), z.shape[1])
            return torch.where(kept, (torch.softmax(z, 1) - one_hot) * (g / counted), 0.0), None
        return binding.softmax_loss_grad(z, labels, counted, g.contiguous()), None


def softmax_loss(z, labels):
    """torch.nn.functional.cross_entropy(z, labels) by hag_softmax_loss where the arguments are of the ordinary kind (65536 rows, 16 classes, both
    passes: 27 us against 113, 300 classes 100 and 234) and there are 2^19 logits or more (as above: 16384 rows of 40 a whole step 496 us against 532, below
    49 us against torch's 43)."""
    if _plain(z) and _plain_labels(labels, z) and 0 < z.shape[1] <= 1 << 20 and z.numel() >= 1 << 19 and not torch.is_autocast_enabled() and _no_tangent(z):
        return _SoftmaxLoss.apply(z, labels)
    return torch.nn.functional.cross_entropy(z, labels)


def aggregation(h, op, naive=False, record=None):
    """torch.autograd.Function around hag_forward / hag_backward (or the naive-CSR kernels) for `op`.

    record: optional list; every call appends (kind, input tensor, output tensor[, argmax]).  Its backward pass is not itself differentiable: second derivatives
    leave out what passes through it."""
    fwd = h.naive_forward if naive else h.forward
    bwd = h.naive_backward if naive else h.backward

    class Agg(torch.autograd.Function):
        @staticmethod
        def forward(ctx, z):
            z = z.contiguous()
            if op == "max":
                y, am = fwd(z, "max")
                ctx.am = am
                if record is not None:
                    record.append(("forward", z.detach().clone(), y.detach().clone(), am.clone()))
                return y
            y = fwd(z, op)
            if record is not None:
                record.append(("forward", z.detach().clone(), y.detach().clone()))
            return y

        @staticmethod
        def backward(ctx, g):
            g = g.contiguous()
            gx = bwd(g, "max", argmax=ctx.am) if op == "max" else bwd(g, op)
            if record is not None:
                record.append(("backward", g.detach().clone(), gx.detach().clone()) + ((ctx.am.clone(),) if op == "max" else ()))
            return gx

    return Agg.apply


def _gcn2_composed(h, x, w1, w2, labels, naive, record):
    agg = aggregation(h, "gcn", naive, record)
    h1 = torch.relu(agg(product(x, w1)))
    logits = agg(product(h1, w2))
    return softmax_loss(logits, labels)


class _Gcn2Loss(torch.autograd.Function):
    """gcn2_loss as one node of the graph: the same calls as the composed form, with the ReLU inside the products on both sides of it."""

    @staticmethod
    def forward(ctx, x, w1, w2, labels, h, naive):
        agg = h.naive_forward if naive else h.forward
        a1 = agg(binding.narrow_product(x, w1), "gcn")
        logits = agg(binding.narrow_product(a1, w2, relu=True), "gcn")
        loss, counted = binding.softmax_loss(logits, labels)
        ctx.save_for_backward(x, w1, w2, labels, a1, logits, counted)
        ctx.h, ctx.naive = h, naive
        return loss

    @staticmethod
    def backward(ctx, g):
        x, w1, w2, labels, a1, logits, counted = ctx.saved_tensors
        need_x, need_1, need_2 = ctx.needs_input_grad[:3]
        if torch.is_grad_enabled() or not (_plain(x) and _plain(w1) and _plain(w2) and _plain(a1) and _plain(logits) and x.data_ptr() % 16 == 0
                                           and a1.data_ptr() % 16 == 0 and labels.is_contiguous()):
            # to be differentiated itself (as far as the composed form is: not through an aggregation), or the saved tensors came back from hooks as something else
            wanted = [t for t, need in ((x, need_x), (w1, need_1), (w2, need_2)) if need]
            again = torch.is_grad_enabled()
            with torch.enable_grad():
                inner = iter(torch.autograd.grad(_gcn2_composed(ctx.h, x, w1, w2, labels, ctx.naive, None), wanted, g, create_graph=again))
            return (*(next(inner) if need else None for need in (need_x, need_1, need_2)), None, None, None)
        back = ctx.h.naive_backward if ctx.naive else ctx.h.backward
        g_z2 = back(binding.softmax_loss_grad(logits, labels, counted, g.contiguous()), "gcn")
        g_w2 = binding.weight_grad(a1, g_z2, relu=True) if need_2 else None
        if not (need_x or need_1):
            return None, None, g_w2, None, None, None
        g_z1 = back(binding.narrow_product(g_z2, w2, transposed=True, mask=a1), "gcn")
        g_w1 = binding.weight_grad(x, g_z1) if need_1 else None
        g_x = binding.narrow_product(g_z1, w1, transposed=True) if need_x else None
        return g_x, g_w1, g_w2, None, None, None


def _narrow(d, k):
    """What hag_narrow_product takes both ways round.  A step as one node was faster than one of the library's products, ReLU and loss at every size timed (8000 to 370000 rows, weights up to
    256 x 256: 126 / 238 us at 8000 rows, 128 x 128 and 128 x 16; 5202 / 5903 at 370000, 256 x 256 twice); the wide products by themselves are not (x is read once per 64 columns of the
    weight: 65536 rows, 256 x 256 139 us, the BLAS library 75), the weight gradients and the passes left out make up for it."""
    return d % 4 == 0 and k % 4 == 0 and 0 < d <= 256 and 0 < k <= 256


def gcn2_loss(h, x, w1, w2, labels, naive=False, record=None):
    """SoftMax cross-entropy of a 2-layer GCN (Section 5.3's model) on features x."""
    if (record is None and _plain(x) and _plain(w1) and _plain(w2) and _plain_labels(labels, x) and x.data_ptr() % 16 == 0 and x.shape[1] == w1.shape[0]
            and w1.shape[1] == w2.shape[0] and _narrow(*w1.shape) and _narrow(*w2.shape) and not torch.is_autocast_enabled()):
        return _Gcn2Loss.apply(x, w1, w2, labels, h, naive)
    return _gcn2_composed(h, x, w1, w2, labels, naive, record)


def sage_pool2_loss(h, x, pool, comb, labels, naive=False, record=None):
    """SoftMax cross-entropy of a 2-layer GraphSAGE with the pooling aggregator of Table 1.

    pool[i]: [d_i, hidden] (W1 of layer i), comb[i]: [hidden + d_i, d_{i+1}] (W2 of layer i)."""
    agg = aggregation(h, "max", naive, record)
    hcur = x
    for i in range(2):
        a = agg(torch.relu(product(hcur, pool[i])))
        hcur = product(torch.cat([a, hcur], dim=1), comb[i])
        if i == 0:
            hcur = torch.relu(hcur)
    return softmax_loss(hcur, labels)


def sage_lstm2_logits(seq, x, cells, comb):
    """Logits of a 2-layer GraphSAGE with LSTM aggregators over ordered neighbour lists (inference; training would wrap
    SeqHag.lstm_forward_train / lstm_backward the way `aggregation` wraps the set aggregates).  seq: binding.SeqHag (a prefix HAG or the plain lists);
    cells[i] = (w_ih, w_hh, b) of layer i; comb[i] = W2 of layer i, [hidden_i + d_i, d_{i+1}].
    a_v = LSTM over (h_u : u in N(v)), h'_v = relu(W2 [a_v, h_v]); the second layer has no ReLU."""
    with torch.no_grad():
        h = x
        for i in range(2):
            a = seq.lstm_forward(h.contiguous(), *cells[i])
            h = torch.cat([a, h], dim=1) @ comb[i]
            if i == 0:
                h = torch.relu(h)
        return h


def lstm_aggregation(seq):
    """torch.autograd.Function around SeqHag.lstm_forward_train / lstm_backward: a = f(x, w_ih, w_hh, b)."""
    class Agg(torch.autograd.Function):
        @staticmethod
        def forward(ctx, x, w_ih, w_hh, b):
            x, w_ih, w_hh = x.contiguous(), w_ih.contiguous(), w_hh.contiguous()
            a, ws = seq.lstm_forward_train(x, w_ih, w_hh, b.contiguous())
            ctx.save_for_backward(x, w_ih, w_hh)
            ctx.ws = ws
            return a

        @staticmethod
        def backward(ctx, g):
            x, w_ih, w_hh = ctx.saved_tensors
            out = seq.lstm_backward(x, w_ih, w_hh, g.contiguous(), ctx.ws)
            ctx.ws = None
            return out

    return Agg.apply


def sage_lstm2_loss(seq, x, cells, comb, labels):
    """SoftMax cross-entropy of the 2-layer GraphSAGE with LSTM aggregators of sage_lstm2_logits, differentiable:
    the aggregator's forward and backward passes are the library's, the dense parts torch."""
    agg = lstm_aggregation(seq)
    h = x
    for i in range(2):
        a = agg(h, *cells[i])
        h = product(torch.cat([a, h], dim=1), comb[i])
        if i == 0:
            h = torch.relu(h)
    return softmax_loss(h, labels)
