"""Training on layers of long rows with the forward pass in LDS, four samples per workgroup (k_fwd_long), at the sizes where it can go
wrong: the smallest batch that takes it, batches that fill no group of four and no stretch of an XCD, more than 256 samples; row lengths
around the halves of eight entries, empty rows, blocks that are not full, the widest operand; the copy of W after steps of
narrower batches, after sdnn_set_weights and under graph replay.  Against the oracle, or bit for bit against the same net
without the copies."""
import numpy as np
import pytest
import torch

from paper_2104_11805_amd import sdnn, workloads as wl
from tests import parity as P

pytestmark = pytest.mark.gpu


def _layer(seed, n_out, n_in, lengths):
    rng = np.random.default_rng(seed)
    deg = np.minimum(np.resize(np.asarray(lengths), n_out), n_in)
    row_ptr = np.zeros(n_out + 1, np.int32)
    np.cumsum(deg, out=row_ptr[1:])
    cols = np.concatenate([np.sort(rng.choice(n_in, size=d, replace=False)) for d in deg]).astype(np.int32)
    vals = (rng.standard_normal(cols.size) * 0.1).astype(np.float32)
    return wl.Layer(n_out, n_in, row_ptr, cols, vals, (rng.standard_normal(n_out) * 0.2).astype(np.float32))


def _net(layers, b, lds, **kw):
    return sdnn.Net(layers, 3.0, b, training=True, lds_forward=lds, **kw)


LENGTHS = (0, 1, 7, 8, 9, 15, 16, 17, 250, 300, 511, 512, 513)


@pytest.mark.parametrize("b,activation,fuse", [(64, "relu", 0), (65, "relu", 0), (66, "sigmoid", 1), (99, "relu", -1), (128, "relu", 0), (129, "relu", 0),
                                               (255, "sigmoid", 0), (256, "relu", 0), (301, "relu", 0)])
def test_step_against_the_oracle(b, activation, fuse):
    layers = [_layer(9600, 1089, 1500, LENGTHS), _layer(9601, 1281, 1089, (129, 130, 127)), _layer(9602, 1025, 1281, LENGTHS)]
    assert _net(layers, 65, 0).workspace_bytes > _net(layers, 65, sdnn.SDNN_LDS_OFF).workspace_bytes
    work = wl.Workload("long", layers, 3.0, wl.normal_inputs(9603, 1500, b), b, "mse", 0.05,
                       targets=wl.uniform_targets(9604, 1025, b), activation=activation)
    st = P.compare_step(P.gpu_train_step(work, work.x_infer, fuse_gradient=fuse), P.oracle_train_step(work, work.x_infer),
                        f"b={b} {activation} fuse={fuse}", exact_fwd=(activation == "relu"))
    assert st["live_g"] == len(layers)


@pytest.mark.parametrize("n_out,n_in,lengths", [(8192, 8192, (2048, 64, 20, 8)), (8193, 8191, (300, 9, 200)), (300, 8192, (8192, 700, 3)), (8192, 8193, (130,))])
def test_widths(n_out, n_in, lengths):
    """The widest operand, one just past it (no copy), few rows of every column."""
    layers, x = [_layer(9610, n_out, n_in, lengths)], wl.normal_inputs(9611, n_in, 70)
    nets = [_net(layers, 70, lds) for lds in (0, sdnn.SDNN_LDS_OFF)]
    assert (nets[0].workspace_bytes > nets[1].workspace_bytes) == (n_in <= 8192)
    outs = [net.sdnn_forward(P.dev(x), torch.full((n_out, 70), -1.0, device=P.DEV)) for net in nets]
    assert torch.equal(*outs) and float(outs[0].std()) > 0


@pytest.mark.parametrize("b", [1021, 1024, 1601, 2301])
def test_more_samples_than_a_round_of_workgroups(b):
    """All groups of four at once on 256 compute units, and in two and three rounds; some places stay empty."""
    layers, x = [_layer(9615, 1000, 700, (150, 160, 170)), _layer(9616, 961, 1000, (150, 160, 170))], wl.normal_inputs(9617, 700, b)
    outs = [_net(layers, b, lds).sdnn_forward(P.dev(x), torch.full((961, b), -1.0, device=P.DEV)) for lds in (0, sdnn.SDNN_LDS_OFF)]
    assert torch.equal(*outs) and float(outs[0].std()) > 0


def test_copy_follows_steps_of_other_batches_and_replaced_values():
    layers = [_layer(9620, 1100, 900, (300, 130, 9)), _layer(9621, 1100, 1100, (280, 150))]
    nets = [_net(layers, 200, lds) for lds in (0, sdnn.SDNN_LDS_OFF)]
    for it, b in enumerate((200, 64, 8, 65, 1, 200, 131)):
        x, y = P.dev(wl.normal_inputs(9622 + it, 900, b)), P.dev(wl.uniform_targets(9632 + it, 1100, b))
        outs = []
        for net in nets:
            if it in (2, 5):
                v, bias = net.sdnn_get_weights(1)
                net.sdnn_set_weights(1, values=v.flip(0).contiguous(), bias=bias + 0.125)
            xl = net.sdnn_forward(x, torch.empty(1100, b, device=P.DEV))
            net.sdnn_backward(sdnn.sdnn_mse_dloss(xl, y))
            net.sdnn_sgd_step(0.5)
            outs.append([xl, *net.sdnn_get_weights(1), *net.sdnn_get_weights(2)])
        assert all(torch.equal(u, v) for u, v in zip(*outs)), it


def test_graph_replays_between_eager_steps_of_another_batch():
    layers = [_layer(9640, 1100, 900, (300, 130, 9)), _layer(9641, 1100, 1100, (280, 150))]
    b = 96
    x, y = P.dev(wl.normal_inputs(9642, 900, b)), P.dev(wl.uniform_targets(9643, 1100, b))
    xs, ys = x[:, :20].contiguous(), y[:, :20].contiguous()
    nets = [_net(layers, b, lds) for lds in (0, sdnn.SDNN_LDS_OFF)]
    xl, d = torch.empty(1100, b, device=P.DEV), torch.empty(1100, b, device=P.DEV)

    def step(net, xin, yin, xl, d):
        net.sdnn_forward(xin, xl)
        sdnn.sdnn_mse_dloss(xl, yin, out=d)
        net.sdnn_backward(d)
        net.sdnn_sgd_step(0.5)

    def small(net):
        step(net, xs, ys, torch.empty(1100, 20, device=P.DEV), torch.empty(1100, 20, device=P.DEV))

    step(nets[0], x, y, xl, d)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step(nets[0], x, y, xl, d)
    xr, dr = torch.empty_like(xl), torch.empty_like(d)
    step(nets[1], x, y, xr, dr)                   # (the captured step has not run)
    for it in range(4):
        small(nets[0])
        graph.replay()
        small(nets[1])
        step(nets[1], x, y, xr, dr)
        torch.cuda.synchronize()
        assert torch.equal(xl, xr), it
        for k in (1, 2):
            assert all(torch.equal(u, v) for u, v in zip(nets[0].sdnn_get_weights(k), nets[1].sdnn_get_weights(k))), (it, k)


@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_infinite_and_nan_activations(bad):
    """They stay with the rows that gather them: the slots past the end of a row read zeros."""
    layers = [_layer(9650, 1100, 1000, LENGTHS + (300, 300))]
    x = wl.normal_inputs(9651, 1000, 67)
    x_bad = x.copy()
    x_bad[[0, 500, 999], 3] = bad
    net = _net(layers, 67, 0, activation="relu")
    outs = [P.host(net.sdnn_forward(P.dev(v), torch.empty(1100, 67, device=P.DEV))) for v in (x, x_bad)]
    hit = np.isin(layers[0].col_idx, [0, 500, 999])
    touched = np.add.reduceat(np.append(hit, False), layers[0].row_ptr[:-1]).astype(bool) & (np.diff(layers[0].row_ptr) > 0)
    assert touched.any() and not touched.all()
    assert np.array_equal(outs[0][~touched], outs[1][~touched])
    others = np.arange(67) != 3
    assert np.array_equal(outs[0][:, others], outs[1][:, others])
