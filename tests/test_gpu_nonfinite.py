"""Infinite and NaN activations stay with the rows that gather them: the slots that fill up a row's last group of entries
carry weight 0, and 0 times infinity is NaN, so they must not read a neuron's value.  One case per kernel that fills up
rows; row lengths around the groups of 8 and 16 entries, bad values at the first and the last neuron.  Exact: a row that
does not gather a bad value has the bits that it has without bad values anywhere."""
import numpy as np
import pytest
import torch

from paper_2104_11805_amd import sdnn, workloads as wl
from tests import parity as P

pytestmark = pytest.mark.gpu

LENGTHS = (0, 1, 7, 8, 9, 15, 16, 17, 31, 33)


def _layer(seed, n_out, n_in):
    rng = np.random.default_rng(seed)
    deg = np.resize(np.asarray(LENGTHS), n_out)
    row_ptr = np.zeros(n_out + 1, np.int32)
    np.cumsum(deg, out=row_ptr[1:])
    cols = np.concatenate([np.sort(rng.choice(n_in, size=d, replace=False)) for d in deg]).astype(np.int32)
    cols[row_ptr[3]], cols[row_ptr[6] - 1] = 0, n_in - 1  # rows of 8 and 15 entries
    vals = (rng.standard_normal(cols.size) * 0.4).astype(np.float32)
    return wl.Layer(n_out, n_in, row_ptr, cols, vals, (-0.1 * rng.random(n_out)).astype(np.float32))


def _gathers(layer, neurons):
    """Whether a row of the layer has one of the columns."""
    hit = np.isin(layer.col_idx, neurons)
    return np.add.reduceat(np.append(hit, False), layer.row_ptr[:-1]).astype(bool) & (np.diff(layer.row_ptr) > 0)


@pytest.mark.parametrize("bad", [np.inf, np.nan])
@pytest.mark.parametrize("mode,n_in,b", [("infer", 2050, 1), ("infer", 2050, 7), ("infer", 2050, 600), ("skip_dead", 2050, 7),
                                         ("layers", 2050, 70), ("train", 2050, 1), ("train", 65536, 1), ("train", 65537, 1),
                                         ("train", 2050, 6), ("train", 2050, 70), ("train", 2050, 130)])
def test_forward(mode, n_in, b, bad):
    n_out = 2113
    layer = _layer(9500, n_out, n_in)
    lds = {"infer": sdnn.SDNN_LDS_ON, "skip_dead": sdnn.SDNN_LDS_ON}.get(mode, sdnn.SDNN_LDS_OFF)
    x = wl.normal_inputs(9501, n_in, b)
    x_bad = x.copy()
    x_bad[[0, -1], :] = bad
    outs = []
    for v in (x, x_bad):
        net = sdnn.Net([layer], 2.0, b, training=(mode == "train"), lds_forward=lds)
        out = torch.empty(n_out, b, device=P.DEV)
        if mode == "skip_dead":
            net.sdnn_forward_skip_dead(P.dev(v), out, 1)
        else:
            net.sdnn_forward(P.dev(v), out)
        outs.append(P.host(out))
        net.close()
    touched = _gathers(layer, [0, n_in - 1])
    assert touched.any() and not touched.all()
    assert np.array_equal(outs[0][~touched], outs[1][~touched])
    if np.isnan(bad):
        assert np.isnan(outs[1][touched]).all()
    else: # one infinite term: the cap or zero by its weight's sign (both of them: perhaps NaN)
        both = _gathers(layer, [0]) & _gathers(layer, [n_in - 1])
        assert np.isin(outs[1][touched & ~both], [0.0, 2.0]).all()


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_one_sample_with_a_launch_per_layer(bad):
    """Inference with one sample where the single launch does not pay (tests/test_routes.py checks the kernel): both layers'
    slots past the end of a row lie past the widest layer's positions, and the second layer's rows among them."""
    layers = [_layer(9503, 30000, 2050), _layer(9504, 2113, 30000)]
    x = wl.normal_inputs(9505, 2050, 1)
    x_bad = x.copy()
    x_bad[[0, -1], :] = bad
    outs = []
    for v in (x, x_bad):
        net = sdnn.Net(layers, np.inf, 1, training=False)
        out = torch.empty(2113, 1, device=P.DEV)
        net.sdnn_forward(P.dev(v), out)
        outs.append(P.host(out))
        net.close()
    assert np.array_equal(outs[0], P.O32.forward(layers, x, np.inf)[-1])
    touched = _gathers(layers[1], np.flatnonzero(_gathers(layers[0], [0, 2049])))
    assert touched.any() and not touched.all()
    assert np.isfinite(outs[0]).all() and np.array_equal(outs[0][~touched], outs[1][~touched])
    assert not np.isfinite(outs[1][touched]).all()


@pytest.mark.parametrize("b", [1, 6, 70, 130, 200])
def test_backward(b):
    layers = [_layer(9510, 7001, 300), _layer(9511, 2113, 7001)]
    x = wl.normal_inputs(9512, 300, b)
    d = wl.normal_inputs(9513, 2113, b)
    d_bad = d.copy()
    d_bad[[0, 9], :] = np.inf
    deltas = []
    for v in (d, d_bad):
        net = sdnn.Net(layers, 1e30, b, training=True, fuse_gradient=1, activation="sigmoid")
        xl = torch.empty(2113, b, device=P.DEV)
        net.sdnn_forward(P.dev(x), xl)
        net.sdnn_backward(P.dev(v))
        deltas.append(P.host(net.sdnn_get_delta(1, b)))
        net.close()
    touched = np.zeros(7001, bool)
    for r in (0, 9):
        touched[layers[1].col_idx[layers[1].row_ptr[r]:layers[1].row_ptr[r + 1]]] = True
    assert touched.any()
    assert np.isfinite(deltas[0]).all()
    assert np.array_equal(deltas[0][~touched], deltas[1][~touched])
    assert not np.isfinite(deltas[1][touched]).any()


@pytest.mark.parametrize("b", [130, 256])
def test_gradient_on_long_columns(b):
    """An infinite delta is in the gradient of its own row's entries and in no other: the others' sums differ from those of the
    run without it by the order of fp64 additions at most, i.e. by no more than their last bit."""
    lay = _layer(9514, 900, 120)
    rng = np.random.default_rng(9515)
    cols = np.stack([np.sort(rng.choice(120, 30, replace=False)) for _ in range(900)]).astype(np.int32)
    lay = wl.Layer(900, 120, np.arange(0, 900 * 30 + 1, 30, dtype=np.int32), cols.ravel(), rng.standard_normal(27000).astype(np.float32), lay.bias)
    x = wl.normal_inputs(9516, 120, b)
    grads = []
    for bad in (0.0, np.inf, np.nan):
        d = wl.normal_inputs(9517, 900, b)
        d[[0, 9, 500], 3] += bad
        net = sdnn.Net([lay], 1e30, b, training=True, fuse_gradient=1, activation="sigmoid")
        net.sdnn_forward(P.dev(x), torch.empty(900, b, device=P.DEV))
        net.sdnn_backward(P.dev(d))
        grads.append(P.host(net.sdnn_weight_grad(1)[0]).reshape(900, 30))
        net.close()
    touched = np.zeros(900, bool)
    touched[[0, 9, 500]] = True
    for g in grads[1:]:
        assert not np.isfinite(g[touched]).any()
        assert (np.abs(g[~touched] - grads[0][~touched]) <= 2.0 ** -23 * np.abs(grads[0][~touched])).all()


def _hot_and_cold(n, degree, n_layers):
    """The first half of the neurons is exactly zero for inputs of 1 and grows without bound for inputs of 0; the other half
    stays alive.  A row's links lie in its own half."""
    half = n // 2
    cols = np.sort((np.arange(half)[:, None] + np.arange(degree)) % half, axis=1)
    cols = np.concatenate([cols, cols + half]).astype(np.int32).ravel()
    row_ptr = np.arange(0, n * degree + 1, degree, dtype=np.int32)
    layers = []
    for l in range(n_layers):
        vals = np.full((n, degree), 0.9 / degree, np.float32)
        vals[:half] = -1.0 / degree if l == 0 else 10.0
        bias = np.zeros(n, np.float32)
        bias[:half] = l == 0
        layers.append(wl.Layer(n, n, row_ptr, cols, vals.ravel(), bias))
    return layers


@pytest.mark.parametrize("n,degree,b,fuse", [(64, 1, 3, 1), (64, 1, 3, -1), (256, 128, 3, -1), (256, 128, 67, 1), (256, 128, 130, -1),
                                             (2050, 1, 67, -1), (7000, 1, 3, 1), (7000, 1, 67, 1), (7000, 1, 130, -1),
                                             (33000, 1, 43, -1), (33000, 1, 43, 1)])
def test_samples_that_fill_up_a_batch_add_nothing(n, degree, b, fuse):
    """Batches that are no multiple of four on an uncapped ReLU: a sample with zero input would reach infinity, and infinity
    times its zero delta is NaN.  One case per kernel that forms gradients or stores activations."""
    layers = _hot_and_cold(n, degree, 42 if degree == 1 else 15)
    x = np.ones((n, b), np.float32)
    x[n // 2:] = np.abs(wl.normal_inputs(9520, n - n // 2, b)) + 0.1
    work = wl.Workload("fill", layers, np.inf, x, b, "mse", 0.05, targets=wl.uniform_targets(9521, n, b), activation="relu")
    with np.errstate(over="ignore"):
        zero_input = P.O32.forward(layers, np.zeros((n, 1), np.float32), np.inf)[-1]
    assert np.isinf(zero_input[:n // 2]).all()
    g = P.gpu_train_step(work, x, fuse_gradient=fuse)
    st = P.compare_step(g, P.oracle_train_step(work, x), f"n={n} b={b} fuse={fuse}")
    assert st["live_g"] == st["live_d"] == len(layers) and st["bitexact_d"] == len(layers)
