"""The single-launch forward with activations in LDS at the sizes where its layout changes: widths around the limits of
4, 2 and 1 samples per workgroup (8192, 16384, 32768 positions), blocks of 64 rows and 1024 positions, rows around the
16-entry chunks, samples that do not fill a workgroup.  Same bits as the oracle."""
import numpy as np
import pytest
import torch

from paper_2104_11805_amd import sdnn, workloads as wl
from tests import parity as P

pytestmark = pytest.mark.gpu


def _ragged(seed, n_out, n_in, lengths):
    """Row r holds lengths[r % len(lengths)] distinct random columns."""
    rng = np.random.default_rng(seed)
    deg = np.resize(np.asarray(lengths), n_out)
    row_ptr = np.zeros(n_out + 1, np.int32)
    np.cumsum(deg, out=row_ptr[1:])
    cols = np.concatenate([np.sort(rng.choice(n_in, size=d, replace=False)) for d in deg]).astype(np.int32)
    vals = (rng.standard_normal(cols.size) * 0.4).astype(np.float32)
    return wl.Layer(n_out, n_in, row_ptr, cols, vals, (rng.standard_normal(n_out) * 0.2).astype(np.float32))


@pytest.mark.parametrize("n,b", [(63, 9), (1024, 3), (1025, 6), (8192, 7), (8193, 5), (16384, 2), (16385, 3), (32768, 3)])
def test_lds_forward_at_the_limits_of_its_layout(n, b):
    lengths = (0, 1, 7, 8, 9, 15, 16, 17, 31, 33)
    layers = [_ragged(9000 + n, n, 50, lengths), _ragged(9001 + n, n, n, lengths), _ragged(9002 + n, 70, n, (0, 5, 40))]
    x = wl.normal_inputs(9003 + n, 50, b)
    ref = P.O32.forward(layers, x, 2.0)[-1]
    assert (ref > 0).any()
    net = sdnn.Net(layers, 2.0, b, training=False, lds_forward=sdnn.SDNN_LDS_ON)
    out = torch.full((70, b), -1.0, device=P.DEV)
    net.sdnn_forward(P.dev(x), out)
    assert np.array_equal(P.host(out), ref)
    net.close()


@pytest.mark.parametrize("b", [1, 255, 257, 511, 513, 1027, 2050])
def test_lds_forward_samples_per_workgroup(b):
    """Batches on both sides of one, two and four samples for each of the 256 CUs."""
    layers = [_ragged(9100 + l, 300, 300, (3, 20, 34)) for l in range(3)]
    x = wl.normal_inputs(9110, 300, b)
    ref = P.O32.forward(layers, x, 1.5)[-1]
    net = sdnn.Net(layers, 1.5, b, training=False, lds_forward=sdnn.SDNN_LDS_ON)
    out = torch.full((300, b), -1.0, device=P.DEV)
    net.sdnn_forward(P.dev(x), out)
    assert np.array_equal(P.host(out), ref)
    net.close()


@pytest.mark.parametrize("activation", ["relu", "sigmoid"])
@pytest.mark.parametrize("n", [2100, 4200, 2048])
def test_lds_forward_with_loads_in_either_order(n, activation):
    """One sample per workgroup on layers whose loads of W are in the compiler's order (2100: by age, 4200: in turns) and in their own."""
    layers = [_ragged(9400 + n + l, n, n, (3, 20, 34)) for l in range(3)]
    for y in layers[1:]:
        y.bias = -np.abs(y.bias)
    x = wl.normal_inputs(9410, n, 5)
    nets = [sdnn.Net(layers, 1.5, 5, training=False, activation=activation, lds_forward=o) for o in (sdnn.SDNN_LDS_ON, sdnn.SDNN_LDS_OFF)]
    outs = [net.sdnn_forward(P.dev(x), torch.empty(n, 5, device=P.DEV)) for net in nets]
    assert torch.equal(outs[0], outs[1]) and float(outs[0].std()) > 0
    if activation == "relu":
        skip = torch.full_like(outs[0], -1.0)
        nets[0].sdnn_forward_skip_dead(P.dev(x), skip, check_every=1)
        assert torch.equal(skip, outs[1])
    for net in nets:
        net.close()


@pytest.mark.parametrize("shift", [0, 1, -5, 600 * 3 + 2, -(600 * 2 + 1)])
def test_lds_forward_over_its_input(shift):
    """The result over the input, or shifted against it by some floats, as the per-layer launches take it."""
    layers = [_ragged(9200 + l, 5000, 5000, (3, 20, 34)) for l in range(2)]
    x = wl.normal_inputs(9210, 5000, 600)
    ref = P.O32.forward(layers, x, 1.5)[-1]
    net = sdnn.Net(layers, 1.5, 600, training=False, lds_forward=sdnn.SDNN_LDS_ON)
    room = torch.empty(x.size + 2 * 4096, device=P.DEV)
    x0, out = room[4096:4096 + x.size].view(-1, 600), room[4096 + shift:4096 + shift + x.size].view(-1, 600)
    x0.copy_(P.dev(x))
    net.sdnn_forward(x0, out)
    assert np.array_equal(P.host(out), ref)
    net.close()


@pytest.mark.parametrize("shift", [1, 2100 * 3 + 2])
def test_forward_across_a_large_input(shift):
    """Blocks that a launch per layer takes through the net in sub-blocks of samples where the result does not lie across the input."""
    layers = [_ragged(9300 + l, 5000, 5000, (3, 20)) for l in range(2)]
    x = wl.normal_inputs(9310, 5000, 2100)
    net = sdnn.Net(layers, 1.5, 2100, training=False, lds_forward=sdnn.SDNN_LDS_OFF)
    ref = net.sdnn_forward(P.dev(x), torch.empty(5000, 2100, device=P.DEV)).clone()
    room = torch.empty(x.size + 2 * 8192, device=P.DEV)
    x0, out = room[8192:8192 + x.size].view(-1, 2100), room[8192 + shift:8192 + shift + x.size].view(-1, 2100)
    x0.copy_(P.dev(x))
    net.sdnn_forward(x0, out)
    assert torch.equal(out, ref)
    net.close()


@pytest.mark.parametrize("sizes", [(4096, 4095, 1, 4096, 1025, 3000), (4097, 1024, 1023, 300), (17, 4096, 4097, 40, 40)])
@pytest.mark.parametrize("b", [1, 70, 300, 1100])
def test_two_buffers_up_to_4096_positions(sizes, b):
    """Layers alternate between two LDS buffers where the net's positions fit twice with four samples, and share one beyond: the widest
    of either kind, odd and even numbers of layers, one, two and four samples per workgroup, stretches that start at either buffer."""
    rng = np.random.default_rng(9700)
    layers = []
    for l, (n_in, n_out) in enumerate(zip(sizes, sizes[1:])):
        d = min(n_in, 24)
        cols = np.stack([np.sort(rng.choice(n_in, d, replace=False)) for _ in range(n_out)]).astype(np.int32)
        layers.append(wl.Layer(n_out, n_in, np.arange(0, n_out * d + 1, d, dtype=np.int32), cols.ravel(), (rng.standard_normal(n_out * d) * 0.4).astype(np.float32),
                               -0.05 * rng.random(n_out).astype(np.float32)))
    x = np.maximum(wl.normal_inputs(9701, sizes[0], b), 0.0)
    ref = P.O32.forward(layers, x, 8.0)[-1]
    net = sdnn.Net(layers, 8.0, b, training=False, lds_forward=sdnn.SDNN_LDS_ON)
    out = torch.empty(sizes[-1], b, device=P.DEV)
    for _ in range(2):
        assert np.array_equal(P.host(net.sdnn_forward(P.dev(x), out)), ref)
    for every in (1, 3):
        n_live = torch.zeros(1, dtype=torch.int32, device=P.DEV)
        out.fill_(-1.0)
        net.sdnn_forward_skip_dead(P.dev(x), out, check_every=every, n_live=n_live)
        assert np.array_equal(P.host(out), ref), every
    v, bias = net.sdnn_get_weights(2)
    net.sdnn_set_weights(2, values=v.clone(), bias=bias.clone())
    assert np.array_equal(P.host(net.sdnn_forward(P.dev(x), out)), ref)
    net.close()
