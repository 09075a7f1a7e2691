"""Nets made for one sample per step (lane-major copies of W and W^T) at the edges of their layout: blocks of 64 rows, chunks
of eight entries and rounds of four chunks (back: eight), the longest row they take and the first they do not, more than 65536 neurons
(4-byte columns), vectors that do and do not fit LDS in the step; weights replaced in between and read back."""
import numpy as np
import pytest
import torch

from paper_2104_11805_amd import sdnn, workloads as wl
from tests import parity as P
from tests.test_gpu_rows import _layer

pytestmark = pytest.mark.gpu


def _steps(layers, seed, activation="relu", n_steps=3, replace=True):
    net = sdnn.Net(layers, 3.0, 1, training=True, activation=activation)
    n0, nl = layers[0].n_in, layers[-1].n_out
    orc = P.ORACLES[activation]
    for s in range(n_steps):
        x, y = wl.normal_inputs(seed + s, n0, 1), wl.uniform_targets(seed + 50 + s, nl, 1)
        if s == 2 and replace:
            lay = layers[0]
            lay.values = (lay.values * np.random.default_rng(seed).uniform(0.5, 1.5, lay.nnz)).astype(np.float32)
            net.sdnn_set_weights(1, P.dev(lay.values), P.dev(lay.bias))
        xl = torch.empty(nl, 1, device=P.DEV)
        net.sdnn_forward(P.dev(x), xl)
        net.sdnn_backward(sdnn.sdnn_mse_dloss(xl, P.dev(y)))
        grads_got = [tuple(P.host(t) for t in net.sdnn_weight_grad(k + 1)) for k in range(len(layers))]
        deltas_got = [P.host(net.sdnn_get_delta(k + 1, 1)) for k in range(len(layers))]
        net.sdnn_sgd_step(0.05)
        xs, deltas, grads, new = orc.train_step(layers, x, 3.0, lambda v: P.mse_dloss(v, y), 0.05)
        P.assert_forward_close(P.host(xl), xs[-1], f"step {s}")
        if activation == "relu":
            assert np.array_equal(P.host(xl), xs[-1])
        for k, lay in enumerate(layers):
            P.assert_grad_close(deltas_got[k], deltas[k + 1], f"step {s} delta {k + 1}")
            for got, ref in zip(grads_got[k], grads[k]):
                P.assert_grad_close(got, ref, f"step {s} gradient {k + 1}")
            v, b = (P.host(t) for t in net.sdnn_get_weights(k + 1))
            P.assert_grad_close(v, new[k][0], f"step {s} values {k + 1}")
            P.assert_grad_close(b, new[k][1], f"step {s} bias {k + 1}")
            lay.values, lay.bias = v, b     # both sides go on from the GPU's weights
        assert (new[0][0] != 0).any()
    net.close()


@pytest.mark.parametrize("activation", ["relu", "sigmoid"])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 1000])
def test_blocks_and_chunks(n, activation):
    lengths = [min(n, k) for k in (0, 1, 7, 8, 9, 31, 32, 33, 40)]
    _steps([_layer(9500 + n, 130, n, lengths), _layer(9501 + n, n, 130, (0, 5, 8, 17, 33)), _layer(9502 + n, 17, n, [min(n, 20)])], 9510, activation)


@pytest.mark.parametrize("longest", [512, 513])
def test_longest_row(longest):
    """513 entries in one row: the net takes the kernels that share a row among lanes."""
    _steps([_layer(9520, 600, 700, (longest,) + (3,) * 599), _layer(9521, 40, 600, (9, 30))], 9530)


@pytest.mark.parametrize("rows", [200, 360, 435, 900, 1300])
def test_long_columns(rows):
    """Columns of about 30, 54, 65, 135 and 195 entries: one round of eight chunks in the backward pass, and several; layers
    whose numbers of blocks of 64 rows (4 to 21, and 1) do not fit each other's."""
    _steps([_layer(9590, rows, 20, (3,)), _layer(9591, 20, rows, (9, 1)), _layer(9592, rows, 20, (3,)), _layer(9593, 5, rows, (40,))], 9595)


def test_wide_layers():
    _steps([_layer(9540, 65600, 60, (1, 3)), _layer(9541, 50, 65600, (2, 9, 33))], 9550, n_steps=2, replace=False)
    _steps([_layer(9542, 41000, 60, (1, 3)), _layer(9543, 50, 41000, (2, 9, 33))], 9560, n_steps=2, replace=False)


@pytest.mark.parametrize("n,long_columns", [(49152, 300), (49153, 300), (65536, 300), (65536, 33)])
def test_long_columns_of_wide_layers(n, long_columns):
    """On both sides of three wavefronts per CU: the first 64 columns have an entry in every row, the others one or none."""
    rng = np.random.default_rng(9545)
    cols = np.concatenate([np.tile(np.arange(64), (long_columns, 1)), 64 + np.sort(rng.choice(n - 64, (long_columns, 9), replace=False), axis=1)], axis=1)
    y = wl.Layer(long_columns, n, np.arange(0, cols.size + 1, 73, dtype=np.int32), cols.astype(np.int32).ravel(),
                 (rng.standard_normal(cols.size) * 0.1).astype(np.float32), (rng.standard_normal(long_columns) * 0.1).astype(np.float32))
    _steps([_layer(9546, n, 60, (1, 3)), y], 9565, n_steps=2, replace=False)


@pytest.mark.parametrize("n", [64, 1025, 16400])
def test_one_sample_inference_on_the_lane_major_copy(n):
    layers = [_layer(9570, n, 90, (0, 1, 9, 16, 17, 33)), _layer(9571, n, n, (3, 16, 33)), _layer(9572, 70, n, (5, 40))]
    x = wl.normal_inputs(9580, 90, 1)
    ref = P.O32.forward(layers, x, 2.0)[-1]
    net = sdnn.Net(layers, 2.0, 4, training=False)
    out = torch.full((70, 1), -1.0, device=P.DEV)
    net.sdnn_forward(P.dev(x), out)
    assert np.array_equal(P.host(out), ref) and (ref > 0).any()
    out.fill_(-1.0)
    net.sdnn_forward_noalloc(P.dev(x), out)
    assert np.array_equal(P.host(out), ref)
    net.close()


# widths of nets of which tests/test_routes.py checks that one sample takes a launch per layer on the copy of the LDS forward
LANE_MAJOR_NETS = [(90, 64, 30000, 70), (90, 1025, 30000, 1024, 70), (2050, 30000, 63)]
LANE_MAJOR_LENGTHS = (0, 1, 9, 16, 17, 33)


@pytest.mark.parametrize("sizes", LANE_MAJOR_NETS)
def test_one_sample_inference_with_a_launch_per_layer(sizes):
    """Narrow layers next to one that is too wide for the single launch to pay: positions and slots past the end of a row
    are those of the widest layer."""
    layers = [_layer(9590 + l, n_out, n_in, LANE_MAJOR_LENGTHS) for l, (n_in, n_out) in enumerate(zip(sizes, sizes[1:]))]
    x = wl.normal_inputs(9599, sizes[0], 1)
    ref = P.O32.forward(layers, x, 2.0)[-1]
    net = sdnn.Net(layers, 2.0, 4, training=False)
    for call in (net.sdnn_forward, net.sdnn_forward_noalloc):
        out = torch.full((sizes[-1], 1), -1.0, device=P.DEV)
        call(P.dev(x), out)
        assert np.array_equal(P.host(out), ref) and (ref > 0).any()
    net.close()
