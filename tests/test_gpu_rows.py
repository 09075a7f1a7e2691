"""The kernels with several matrix rows per wavefront (forward, and backward with the gradient) at the sizes where their
layout changes: batches around 16, 32, 64, 128 and 256 samples (lanes per row), batches that are no multiple of four (zero
samples fill the last group), tiles of samples, row lengths around the 16-entry groups, rows left over at the end."""
import numpy as np
import pytest

from paper_2104_11805_amd import workloads as wl
from tests import parity as P

pytestmark = pytest.mark.gpu


def _layer(seed, n_out, n_in, lengths):
    """Row r holds lengths[r % len(lengths)] distinct random columns."""
    rng = np.random.default_rng(seed)
    deg = np.resize(np.asarray(lengths), n_out)
    row_ptr = np.zeros(n_out + 1, np.int32)
    np.cumsum(deg, out=row_ptr[1:])
    cols = np.concatenate([np.sort(rng.choice(n_in, size=d, replace=False)) for d in deg]).astype(np.int32)
    vals = (rng.standard_normal(cols.size) * 0.4).astype(np.float32)
    return wl.Layer(n_out, n_in, row_ptr, cols, vals, (rng.standard_normal(n_out) * 0.2).astype(np.float32))


def _step(layers, b, seed, fuse, activation="relu"):
    work = wl.Workload("rows", layers, 3.0, wl.normal_inputs(seed, layers[0].n_in, b), b, "mse", 0.05,
                       targets=wl.uniform_targets(seed + 1, layers[-1].n_out, b), activation=activation)
    g = P.gpu_train_step(work, work.x_infer, fuse_gradient=fuse)
    o = P.oracle_train_step(work, work.x_infer)
    st = P.compare_step(g, o, f"rows b={b} fuse={fuse} {activation}", exact_fwd=(activation == "relu"))
    assert st["live_g"] == len(layers)
    if activation == "relu":
        assert st["bitexact_d"] == len(layers)


@pytest.mark.parametrize("b", [2, 3, 4, 15, 17, 31, 33, 63, 66, 97, 127, 129, 200, 255, 257])
def test_batch_sizes_around_the_lanes_per_row(b):
    layers = [_layer(9300, 2113, 250, (0, 1, 3, 15, 16, 17, 31, 33, 40)), _layer(9301, 75, 2113, (70, 16, 5, 90))]
    _step(layers, b, 9310, fuse=1)


def _turned(lay):
    """The layer whose W is the other one's W^T."""
    rows = np.repeat(np.arange(lay.n_out), np.diff(lay.row_ptr))
    order = np.lexsort((rows, lay.col_idx))
    row_ptr = np.zeros(lay.n_in + 1, np.int32)
    np.cumsum(np.bincount(lay.col_idx, minlength=lay.n_in), out=row_ptr[1:])
    return wl.Layer(lay.n_in, lay.n_out, row_ptr, rows[order].astype(np.int32), lay.values[order], np.linspace(-0.5, 0.5, lay.n_in, dtype=np.float32))


@pytest.mark.parametrize("b,activation", [(129, "relu"), (130, "sigmoid"), (192, "relu"), (255, "relu"), (256, "relu"), (256, "sigmoid")])
def test_long_columns_and_more_than_128_samples(b, activation):
    """The sweep with a wavefront per row: columns of W around its groups of sixteen entries, empty ones and very long ones;
    layers whose columns have just under and just over 64 entries on average."""
    layers = [_turned(_layer(9430, 301, 1700, (0, 1, 15, 16, 17, 31, 33, 250, 1700))), _turned(_layer(9431, 1700, 203, (62, 64, 65, 66))),
              _turned(_layer(9432, 203, 150, (63, 64)))]
    _step(layers, b, 9440, 1, activation)


@pytest.mark.parametrize("b,fuse,activation", [(5, -1, "relu"), (99, -1, "relu"), (30, 1, "sigmoid"), (99, 1, "sigmoid")])
def test_separate_update_and_sigmoid(b, fuse, activation):
    layers = [_layer(9320, 2113, 250, (2, 9, 16, 40)), _layer(9321, 75, 2113, (70, 16, 5, 90))]
    _step(layers, b, 9330, fuse, activation)


@pytest.mark.parametrize("n_in,n_mid,b", [(9001, 2500, 128), (17003, 6500, 256), (17003, 6500, 130)])
def test_tiles_of_samples_on_operands_larger_than_l2(n_in, n_mid, b):
    """Forward tiles of 64 and 32 samples (operands of 4.6 and 17 MB), backward over operands of 2 to 8 MB."""
    layers = [_layer(9340, n_mid, n_in, (4, 20)), _layer(9341, 8001, n_mid, (3, 6)), _layer(9342, 33, 8001, (200, 17))]
    _step(layers, b, 9350, fuse=1)


@pytest.mark.parametrize("b", [124, 125, 126, 127, 129])
def test_gradient_is_rounded_once(b):
    """Batches next to 128 (which are two rounded windows).  Samples 64 and up cancel the first 64 but for one part in 2^20: a sum over all samples in fp64, rounded once, is within
    half a unit in the last place (2^-24) of the exact one, plus 2^-53 per term; rounded halves are off by about 2^-24 * 2^20."""
    import torch
    from paper_2104_11805_amd import sdnn
    lay = _layer(9390, 2113, 250, (2, 9, 16, 40))
    lay.values[:], lay.bias[:] = 0.0, 1.0          # every neuron is active: Delta is the loss gradient
    x, d = wl.normal_inputs(9391, 250, 64), wl.normal_inputs(9392, 2113, 64)
    x = np.concatenate([x, x, x], axis=1)[:, :b].copy()
    d = np.concatenate([d, (-d * (1 + 2.0 ** -20)).astype(np.float32), d], axis=1)[:, :b].copy()
    net = sdnn.Net([lay], float("inf"), b, training=True, fuse_gradient=1)
    net.sdnn_forward(P.dev(x), torch.empty(2113, b, device=P.DEV))
    net.sdnn_backward(P.dev(d))
    got = P.host(net.sdnn_weight_grad(1)[0]).astype(np.float64)
    rows = np.repeat(np.arange(2113), np.diff(lay.row_ptr))
    terms = d[rows].astype(np.float64) * x[lay.col_idx].astype(np.float64)
    ref = terms.sum(axis=1)
    assert (np.abs(got - ref) <= 2.0 ** -24 * np.abs(ref) + 2 * b * 2.0 ** -53 * np.abs(terms).sum(axis=1)).all()
    net.close()


@pytest.mark.parametrize("n_out,offset", [(3670, 0), (3670, 1), (3671, 3), (3674, 2)])
def test_gradient_of_a_million_entries_in_csr_order(n_out, offset):
    """Entries just under 7 2^18 (a scatter), and just over (two passes; the last chunk and span part-filled), into an array that
    starts at any float; what lies before and after it stays."""
    import ctypes as C
    import torch
    from paper_2104_11805_amd import sdnn
    lay = _layer(9395, n_out, 600, (500,))
    nnz, b = lay.col_idx.size, 5
    assert (nnz >= 7 << 18) == (n_out > 3670)
    x, d = wl.normal_inputs(9396, 600, b), wl.normal_inputs(9397, n_out, b)
    lay.values[:], lay.bias[:] = 0.0, 1.0          # every neuron is active: Delta is the loss gradient
    net = sdnn.Net([lay], float("inf"), b, training=True, fuse_gradient=1)
    net.sdnn_forward(P.dev(x), torch.empty(n_out, b, device=P.DEV))
    net.sdnn_backward(P.dev(d))
    out = torch.full((nnz + 16,), 7.0, device=P.DEV)
    for _ in range(2):
        rc = sdnn.lib().sdnn_weight_grad(net._handle, 1, C.c_void_p(out.data_ptr() + 4 * offset), None, None)
        assert rc == 0
    torch.cuda.synchronize()
    got = P.host(out)
    assert (got[:offset] == 7.0).all() and (got[offset + nnz:] == 7.0).all()
    rows = np.repeat(np.arange(n_out), 500)
    terms = d[rows].astype(np.float64) * x[lay.col_idx].astype(np.float64)
    assert (np.abs(got[offset:offset + nnz] - terms.sum(axis=1)) <= 2.0 ** -24 * np.abs(terms.sum(axis=1)) + 2 * b * 2.0 ** -53 * np.abs(terms).sum(axis=1)).all()
    new = lay.values.astype(np.float64) - 0.5 * got[offset:offset + nnz]
    net.sdnn_sgd_step(0.5)
    assert np.array_equal(P.host(net.sdnn_get_weights(1)[0]), new.astype(np.float32))
    net.close()


def test_a_smaller_batch_after_a_larger_one():
    """The arrays' row pitch follows the batch: nothing of the earlier, wider batch may show."""
    import torch
    from paper_2104_11805_amd import sdnn
    layers = [_layer(9360, 2113, 250, (2, 9, 16, 40)), _layer(9361, 75, 2113, (70, 16, 5, 90))]
    net = sdnn.Net(layers, 3.0, 131, training=True, fuse_gradient=1)
    for b in (131, 6, 50, 1, 99):
        x, y = wl.normal_inputs(9370 + b, 250, b), wl.uniform_targets(9380 + b, 75, b)
        xl = torch.empty(75, b, device=P.DEV)
        net.sdnn_forward(P.dev(x), xl)
        net.sdnn_backward(sdnn.sdnn_mse_dloss(xl, P.dev(y)))
        xs, deltas, grads, _ = P.O32.train_step(layers, x, 3.0, lambda v: P.mse_dloss(v, y), 0.0)
        assert np.array_equal(P.host(xl), xs[-1]), b
        assert np.array_equal(P.host(net.sdnn_get_activation(1, b)), xs[1]), b
        for k in (1, 2):
            assert np.array_equal(P.host(net.sdnn_get_delta(k, b)), deltas[k]), b
            for got, ref in zip(net.sdnn_weight_grad(k), grads[k - 1]):
                P.assert_grad_close(P.host(got), ref, f"b={b} layer {k}")
        net.sdnn_sgd_step(0.0)
    net.close()


@pytest.mark.parametrize("b", [148, 212])
def test_last_narrow_block_on_a_narrow_last_layer(b):
    """Inference in blocks of 64 samples for the panel sweep, the last one of 20 samples; a last layer of few rows."""
    import torch
    from paper_2104_11805_amd import sdnn
    layers = [_layer(9400, 65536, 65536, (2, 16, 7)), _layer(9401, 1000, 65536, (40, 5))]
    x = wl.normal_inputs(9402, 65536, b)
    ref = P.O32.forward(layers, x, 2.0)[-1]
    net = sdnn.Net(layers, 2.0, b, training=False)
    out = torch.full((1000, b), -1.0, device=P.DEV)
    net.sdnn_forward(P.dev(x), out)
    assert np.array_equal(P.host(out), ref) and (ref > 0).any()
    net.close()


@pytest.mark.parametrize("fuse", [-1, 1])
def test_rows_that_are_not_filled_up(fuse):
    """17e6 neurons x 63 samples: below 4 GiB only with rows of 63 floats (no wide loads).  The two narrow ends of the net make
    the reference small: the middle neurons that the last layer reads, in fp64."""
    import torch
    from paper_2104_11805_amd import sdnn
    n, b, lr = 17_000_000, 63, 0.5
    rng = np.random.default_rng(9410)
    rp = (np.arange(n + 1, dtype=np.int64) + 3) // 4                           # one entry in every fourth row
    first = wl.Layer(n, 8, rp.astype(np.int32), rng.integers(0, 8, rp[-1]).astype(np.int32),
                     rng.standard_normal(rp[-1]).astype(np.float32), np.full(n, 0.25, np.float32))
    cols = np.sort(rng.choice(n, (8, 50), replace=False).astype(np.int32) // 4 * 4, axis=1)   # rows of the first layer with an entry
    cols[:, -1] = n - 4
    assert (np.diff(cols, axis=1) > 0).all()
    last = wl.Layer(8, n, np.arange(0, 401, 50, dtype=np.int32), cols.ravel(), rng.standard_normal(400).astype(np.float32),
                    np.full(8, 1.0, np.float32))
    x, d = wl.normal_inputs(9411, 8, b), wl.normal_inputs(9412, 8, b)
    # reference: the neurons `used` of the middle layer, whose entries are at used // 4
    used, at = np.unique(cols, return_inverse=True)
    w1, c1, w2, at = first.values[used // 4].astype(np.float64), first.col_idx[used // 4], last.values.astype(np.float64), at.ravel()
    row2 = np.repeat(np.arange(8), 50)
    x1 = np.minimum(np.maximum(w1[:, None] * x[c1] + 0.25, 0.0), 8.0).astype(np.float32)
    x2 = np.ones((8, b))
    np.add.at(x2, row2, w2[:, None] * x1[at])
    x2 = np.minimum(np.maximum(x2, 0.0), 8.0).astype(np.float32)
    d2 = np.where((x2 > 0) & (x2 < 8), d, np.float32(0.0))
    back = np.zeros((used.size, b))
    np.add.at(back, at, w2[:, None] * d2[row2])
    d1 = np.where((x1 > 0) & (x1 < 8), back, 0.0).astype(np.float32)
    g1 = (d1.astype(np.float64) * x[c1]).sum(axis=1)
    g2 = (d2[row2].astype(np.float64) * x1[at]).sum(axis=1)
    net = sdnn.Net([first, last], 8.0, b, training=True, fuse_gradient=fuse)
    xl = torch.empty(8, b, device=P.DEV)
    net.sdnn_forward(P.dev(x), xl)
    P.assert_forward_close(P.host(xl), x2)
    net.sdnn_backward(P.dev(d))
    mid = torch.from_numpy(used.astype(np.int64)).to(P.DEV)
    P.assert_forward_close(P.host(net.sdnn_get_activation(1, b)[mid]), x1)
    P.assert_grad_close(P.host(net.sdnn_get_delta(1, b)[mid]), d1)
    net.sdnn_sgd_step(lr)
    v1, v2 = net.sdnn_get_weights(1)[0], P.host(net.sdnn_get_weights(2)[0])
    P.assert_grad_close(P.host(v1[mid // 4]), (w1 - lr * g1).astype(np.float32))
    rest = torch.ones(v1.numel(), dtype=torch.bool, device=P.DEV)
    rest[mid // 4] = False                                                     # nobody reads those neurons: no gradient
    assert torch.equal(v1[rest], P.dev(first.values)[rest])
    P.assert_grad_close(v2, (w2 - lr * g2).astype(np.float32))
    net.close()
