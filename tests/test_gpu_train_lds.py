"""Training on narrow nets with one launch per pass: widths around the blocks of 64 rows and the 1024 and 2048 positions, rows of
W and of W^T around the chunks of sixteen entries and up to 512, batches that are filled up and batches of a net made for more.  Forward and deltas the same bits as the oracle's,
over two steps, so that the copies have followed the first one's values."""
import numpy as np
import pytest
import torch

from paper_2104_11805_amd import sdnn, workloads as wl
from tests import pan_nets, parity as P

pytestmark = pytest.mark.gpu


def _two_steps(layers, b, cap, lr=0.05, activation="relu", lds_forward=0, replace=False):
    """X_l, Delta_l and the weights after each of two steps (with replaced weights of layer 2 in between)."""
    net = sdnn.Net(layers, cap, b, training=True, activation=activation, lds_forward=lds_forward)
    x, y = P.dev(wl.normal_inputs(8000, layers[0].n_in, b)), P.dev(np.abs(wl.normal_inputs(8001, layers[-1].n_out, b)))
    xl = torch.empty(layers[-1].n_out, b, device=P.DEV)
    out = []
    for step in range(2):
        net.sdnn_forward(x, xl)
        net.sdnn_backward(sdnn.sdnn_mse_dloss(xl, y))
        out += [xl.clone()] + [net.sdnn_get_activation(k, b) for k in range(1, len(layers) + 1)] + [net.sdnn_get_delta(k, b) for k in range(1, len(layers) + 1)]
        net.sdnn_sgd_step(lr)
        out += [t for k in range(1, len(layers) + 1) for t in net.sdnn_get_weights(k)]
        if replace:
            v, bias = net.sdnn_get_weights(2)
            net.sdnn_set_weights(2, v * 0.5, bias + 0.1)
    net.close()
    return out


@pytest.mark.parametrize("widths,b,lengths", [((1024, 1024, 1024, 1024, 1024), 64, (32,)), ((50, 1025, 63, 1000, 7), 5, (0, 1, 16, 17, 33)),
                                              ((300, 1400, 1300, 64, 1), 255, (7, 8, 9)), ((1024, 65, 1023, 129, 1024, 40), 2, (15, 31, 64))])
def test_single_launch_passes_against_a_launch_per_layer(widths, b, lengths):
    layers = pan_nets.layers(widths, lengths, seed=8100)
    for replace in (False, True):
        single, per_layer = (_two_steps(layers, b, 2.0, lds_forward=o, replace=replace) for o in (sdnn.SDNN_LDS_AUTO, sdnn.SDNN_LDS_OFF))
        assert all(torch.equal(u, v) for u, v in zip(single, per_layer))
    assert float(single[len(widths) - 1].abs().max()) > 0


def _steps(layers, max_batch, batches, **options):
    """X_l, Delta_l and the weights of one net after each of its steps over so many samples."""
    net = sdnn.Net(layers, 2.0, max_batch, training=True, **options)
    out = []
    for step, b in enumerate(batches):
        xl = torch.empty(layers[-1].n_out, b, device=P.DEV)
        net.sdnn_forward(P.dev(wl.normal_inputs(8600 + step, layers[0].n_in, b)), xl)
        net.sdnn_backward(sdnn.sdnn_mse_dloss(xl, P.dev(np.abs(wl.normal_inputs(8700 + step, layers[-1].n_out, b)))))
        out += [xl.clone()] + [net.sdnn_get_activation(k, b) for k in range(1, len(layers) + 1)] + [net.sdnn_get_delta(k, b) for k in range(1, len(layers) + 1)]
        net.sdnn_sgd_step(0.05)
        out += [t for k in range(1, len(layers) + 1) for t in net.sdnn_get_weights(k)]
    net.close()
    return out


def test_steps_of_different_batches():
    """A net whose steps over 2 and 1 samples take a launch per layer, those over 33 and 64 a single one (tests/test_routes.py)."""
    layers = pan_nets.layers((1600,) * 13, (32,), seed=8400)
    batches = (64, 2, 33, 1, 64, 2)
    single, per_layer = (_steps(layers, 64, batches, lds_forward=o) for o in (sdnn.SDNN_LDS_AUTO, sdnn.SDNN_LDS_OFF))
    assert all(torch.equal(u, v) for u, v in zip(single, per_layer))


@pytest.mark.parametrize("widths,max_batch,lengths,full,batches", pan_nets.TRAIN_NETS)
def test_single_launch_passes_at_their_limits(widths, max_batch, lengths, full, batches):
    layers = pan_nets.layers(widths, lengths, seed=8500, full=full)
    single, per_layer = (_steps(layers, max_batch, batches, lds_forward=o) for o in (sdnn.SDNN_LDS_AUTO, sdnn.SDNN_LDS_OFF))
    assert all(torch.equal(u, v) for u, v in zip(single, per_layer))
    assert all(float(t.abs().max()) > 0 for t in single[:2 * len(layers) + 1])


def test_all_weights_replaced_before_a_step():
    layers, other = (pan_nets.layers((700,) * 7, (16, 40), seed=s) for s in (8900, 8950))
    x, y = P.dev(wl.normal_inputs(8960, 700, 9)), P.dev(np.abs(wl.normal_inputs(8961, 700, 9)))
    outs = []
    for o in (sdnn.SDNN_LDS_AUTO, sdnn.SDNN_LDS_OFF):
        net = sdnn.Net(layers, 2.0, 9, training=True, lds_forward=o)
        xl = torch.empty(700, 9, device=P.DEV)
        for rounds in range(2):
            for k, (l, v) in enumerate(zip(layers, other), 1):
                net.sdnn_set_weights(k, P.dev(np.resize(v.values, l.nnz) * (0.5 + rounds)), P.dev(v.bias))
            net.sdnn_forward(x, xl)
            net.sdnn_backward(sdnn.sdnn_mse_dloss(xl, y))
            outs.append([xl.clone()] + [net.sdnn_get_delta(k, 9) for k in range(1, 7)])
            net.sdnn_sgd_step(0.05)
        net.close()
    assert all(torch.equal(u, v) for u, v in zip(outs[0] + outs[1], outs[2] + outs[3])) and not torch.equal(outs[0][0], outs[1][0])


def test_captured_steps_between_steps_of_few_samples():
    """A graph of a step over 64 samples (the copies are read) and steps over 2 (they are not), in turn, against a net that runs all
    of them eagerly with a launch per layer."""
    layers = pan_nets.layers((1600,) * 13, (32,), seed=8400)
    nets = [sdnn.Net(layers, 2.0, 64, training=True, lds_forward=o) for o in (sdnn.SDNN_LDS_AUTO, sdnn.SDNN_LDS_OFF)]
    data = {b: [P.dev(wl.normal_inputs(8800 + b, 1600, b)), P.dev(np.abs(wl.normal_inputs(8900 + b, 1600, b))), torch.empty(1600, b, device=P.DEV),
                torch.empty(1600, b, device=P.DEV)] for b in (2, 64)}

    def step(net, b):
        x, y, xl, dl = data[b]
        net.sdnn_forward(x, xl)
        sdnn.sdnn_mse_dloss(xl, y, out=dl)
        net.sdnn_backward(dl)
        net.sdnn_sgd_step(0.05)

    for net in nets:
        step(net, 2)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        step(nets[0], 64)
    for b in (64, 2, 64, 64, 2):
        if b == 64:
            graph.replay()
        else:
            step(nets[0], b)
        step(nets[1], b)
        torch.cuda.synchronize()
        for k in (1, 7, 12):
            assert all(torch.equal(u, v) for u, v in zip(*(net.sdnn_get_weights(k) for net in nets))), (b, k)
    step(nets[0], 64)
    step(nets[1], 64)
    assert torch.equal(nets[0].sdnn_get_activation(12, 64), nets[1].sdnn_get_activation(12, 64))
    for net in nets:
        net.close()


def test_single_launch_passes_sigmoid():
    layers = pan_nets.layers((200, 900, 800, 700, 100), (20, 40), seed=8200)
    single, per_layer = (_two_steps(layers, 9, np.inf, activation="sigmoid", lds_forward=o) for o in (sdnn.SDNN_LDS_AUTO, sdnn.SDNN_LDS_OFF))
    assert all(torch.equal(u, v) for u, v in zip(single, per_layer))


def test_single_launch_passes_against_the_oracle():
    work = wl.make_config(1, n=1024, n_layers=6, density=0.40)
    st = P.compare_step(P.gpu_train_step(work, work.x_train), P.oracle_train_step(work, work.x_train), "single launch")
    assert st["bitexact_x"] == 7 and st["bitexact_d"] == 6 and st["live_g"] == 6


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_infinite_samples_stay_to_themselves(bad):
    """A sample that is not finite, next to those that fill up a batch of five."""
    layers = pan_nets.layers((300, 1024, 1024, 1024, 50), (0, 5, 17, 40), seed=8300)
    x = wl.normal_inputs(8301, 300, 5)
    x[17, 4] = bad
    res = []
    for o in (sdnn.SDNN_LDS_AUTO, sdnn.SDNN_LDS_OFF):
        net = sdnn.Net(layers, np.inf, 5, training=True, lds_forward=o)
        xl = torch.empty(50, 5, device=P.DEV)
        net.sdnn_forward(P.dev(x), xl)
        net.sdnn_backward(xl * 0.1)
        res.append([P.host(xl)] + [P.host(net.sdnn_get_activation(k, 5)) for k in range(1, 5)] + [P.host(net.sdnn_get_delta(k, 5)) for k in range(1, 5)] +
                   [P.host(t) for k in range(1, 5) for t in net.sdnn_weight_grad(k)])
        net.close()
    assert all(np.array_equal(u, v, equal_nan=True) for u, v in zip(*res))
