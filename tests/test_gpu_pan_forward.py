"""The forward in panels (layers wider than LDS) at the edges of its panels, ranges and blocks: same bits as the oracle."""
import numpy as np
import pytest
import torch

from paper_2104_11805_amd import sdnn, workloads as wl
from tests import pan_nets, parity as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("widths,b,lengths", pan_nets.NETS)
def test_pan_forward_at_the_edges_of_its_layout(widths, b, lengths):
    layers = pan_nets.layers(widths, lengths)
    x = wl.normal_inputs(7100, widths[0], b)
    ref = P.O32.forward(layers, x, 1.5)[-1]
    assert (ref > 0).any() and (ref == 1.5).any()
    net = sdnn.Net(layers, 1.5, b, training=False)
    out = torch.full((widths[-1], b), -1.0, device=P.DEV)
    net.sdnn_forward(P.dev(x), out)
    assert np.array_equal(P.host(out), ref)
    net.close()


def test_pan_forward_after_the_weights_were_replaced():
    widths, b, lengths = pan_nets.NETS[3]
    layers, other = pan_nets.layers(widths, lengths), pan_nets.layers(widths, lengths, seed=7000)
    for y in other[1:2]:
        y.values = (y.values * 0.5 + 0.1).astype(np.float32)
        y.bias = (y.bias + 0.3).astype(np.float32)
    x = wl.normal_inputs(7200, widths[0], b)
    net = sdnn.Net(layers, np.inf, b, training=False)
    net.sdnn_set_weights(2, P.dev(other[1].values), P.dev(other[1].bias))
    out = torch.full((widths[-1], b), -1.0, device=P.DEV)
    net.sdnn_forward(P.dev(x), out)
    assert np.array_equal(P.host(out), P.O32.forward(other, x, np.inf)[-1])
    net.close()


@pytest.mark.parametrize("b", [129, 341])
def test_pan_forward_sigmoid(b):
    widths, _, lengths = pan_nets.NETS[3]
    layers = pan_nets.layers(widths, lengths)
    x = wl.normal_inputs(7300, widths[0], b)
    nets = [sdnn.Net(layers, np.inf, b, training=False, activation="sigmoid", lds_forward=o) for o in (sdnn.SDNN_LDS_AUTO, sdnn.SDNN_LDS_OFF)]
    outs = [net.sdnn_forward(P.dev(x), torch.empty((widths[-1], b), device=P.DEV)) for net in nets]
    assert torch.equal(outs[0], outs[1]) and float(outs[0].std()) > 0


@pytest.mark.parametrize("shift", [0, 7, -(40000 * 3 + 1)])
def test_pan_forward_over_its_input(shift):
    widths, b, lengths = pan_nets.NETS[3]
    layers = pan_nets.layers(widths, lengths)
    x = wl.normal_inputs(7400, widths[0], b)
    net = sdnn.Net(layers, 1.5, b, training=False)
    pad = 1 << 17
    room = torch.empty(x.size + 2 * pad, device=P.DEV)
    x0, out = room[pad:pad + x.size].view(-1, b), room[pad + shift:pad + shift + x.size].view(-1, b)
    x0.copy_(P.dev(x))
    net.sdnn_forward(x0, out)
    assert np.array_equal(P.host(out), P.O32.forward(layers, x, 1.5)[-1])
    net.close()


@pytest.mark.parametrize("bad,b", [(np.inf, 129), (-np.inf, 129), (np.nan, 129), (np.inf, 341), (np.nan, 341)])
def test_infinities_stay_with_the_rows_that_gather_them(bad, b):
    """Slots past a row's entries, and rows of other panels, take nothing from a neuron that is not finite, nor does the next piece of a
    workgroup (341 samples: 171 pairs, of which three XCDs have one more than the others) from one whose sums are not."""
    widths, _, lengths = pan_nets.NETS[3]
    layers = pan_nets.layers(widths, lengths)
    x = wl.normal_inputs(7500, widths[0], b)
    hit = x.copy()
    hit[[0, 13375, 13376, 39999], 5] = bad             # ends of the first and last panel
    net = sdnn.Net(layers[:1] + layers[1:], 1.5, b, training=False)
    outs = [P.host(net.sdnn_forward(P.dev(v), torch.empty((widths[-1], b), device=P.DEV))) for v in (x, hit)]
    others = np.arange(b) != 5
    assert np.array_equal(outs[0][:, others], outs[1][:, others])
    touched = np.isin(np.arange(widths[0]), [0, 13375, 13376, 39999])
    for y in layers:                                   # neurons that a path leads to from one of those
        rows = np.repeat(np.arange(y.n_out), np.diff(y.row_ptr))
        nxt = np.zeros(y.n_out, bool)
        nxt[rows[touched[y.col_idx]]] = True
        touched = nxt
    assert 0 < touched.sum() < touched.size
    assert np.array_equal(outs[0][~touched, 5], outs[1][~touched, 5])
    net.close()


def test_pan_forward_in_a_graph():
    """Captured and replayed, with eager passes of another input between the replays."""
    widths, b, lengths = pan_nets.NETS[3]
    layers = pan_nets.layers(widths, lengths)
    net = sdnn.Net(layers, 1.5, b, training=False)
    xs = [P.dev(wl.normal_inputs(7600 + k, widths[0], b)) for k in range(2)]
    ref = [net.sdnn_forward(x, torch.empty((widths[-1], b), device=P.DEV)).clone() for x in xs]
    x, out = torch.empty_like(xs[0]), torch.empty_like(ref[0])
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        net.sdnn_forward(x, out)
    for k in (0, 1, 0):
        x.copy_(xs[k])
        out.fill_(-1.0)
        g.replay()
        assert torch.equal(out, ref[k])
        assert torch.equal(net.sdnn_forward(xs[1 - k], torch.empty_like(out)), ref[1 - k])
    net.close()
