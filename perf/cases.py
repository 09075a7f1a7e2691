"""The work that users of this framework have it do, as cases that can be timed and compared.

Every case is one net and one call sequence through the public binding (paper_2104_11805_amd.sdnn):

  infer        sdnn_forward on an inference net (a block of input vectors in, the last layer's activations out)
  skip_dead    sdnn_forward_skip_dead: inference on thresholded nets in which many samples die on the way
  train        one SGD step on a minibatch: forward, loss gradient, backward, update; the loop also looks at the
               gradient of the first layer before the update and reads back every 16th layer and the last
  train_single the paper's own training setup (Section 6.1): sigmoid, weights uniform in [-1, 1], one vector per step

Two kinds of topology: "even" (32 links per neuron at distinct uniformly random sources, as in configurations 1 to 4)
and "pruned" (heavy-tailed row degrees with a mean of a tenth of the columns, as in configuration 5).  The sizes are those
of the five configurations (depths shortened where a pass would only repeat itself), of the tests, and ragged ones
between them.  Nets are drawn on the GPU from the seed (creating them is part of prepare(), not of the pass).
"""
import math

import torch

from paper_2104_11805_amd import sdnn

DEV = "cuda:0"


# ---- the cases ---------------------------------------------------------------------------------------------------

def listed():
    return [
        # configuration 1: the smallest net, a short block of inputs; launches and latency count
        dict(name="infer-n1024-b64", kind="infer", topo="even", n=1024, layers=120, batch=64),
        # configuration 2: bulk inference on a narrow net
        dict(name="infer-n4096-b1024", kind="infer", topo="even", n=4096, layers=120, batch=1024),
        # configuration 3: bulk inference on a mid-width net
        dict(name="infer-n16384-b4096", kind="infer", topo="even", n=16384, layers=48, batch=4096),
        # configuration 4: the widest net, one of the blocks that its samples are streamed in
        dict(name="infer-n65536-b1024", kind="infer", topo="even", n=65536, layers=24, batch=1024),
        # configuration 5: bulk inference on an irregularly pruned net
        dict(name="infer-pruned-n8192-b2048", kind="infer", topo="pruned", n=8192, layers=6, batch=2048),
        # samples that die next to samples that live, sizes that are multiples of nothing
        dict(name="skip-dead-n3001-b777", kind="skip_dead", topo="even", n=3001, layers=120, batch=777),
        # configuration 1: training on the smallest net
        dict(name="train-n1024-b64", kind="train", topo="even", n=1024, layers=120, batch=64),
        # configuration 2: its minibatch of 128
        dict(name="train-n4096-b128", kind="train", topo="even", n=4096, layers=120, batch=128),
        # a minibatch that fits no tile on a width that fits none either
        dict(name="train-n10007-b99", kind="train", topo="even", n=10007, layers=48, batch=99),
        # configuration 4: the headline training step
        dict(name="train-n65536-b64", kind="train", topo="even", n=65536, layers=24, batch=64),
        # configuration 5: irregular rows, softmax cross-entropy on the last ten neurons
        dict(name="train-pruned-n8192-b256", kind="train", topo="pruned", n=8192, layers=6, batch=256),
        # the paper's training experiment: one vector per step
        dict(name="train-single-n16384", kind="train_single", topo="even", n=16384, layers=120, batch=1),
    ]


# no drawn case visits more edges than the largest listed one of its kind does
_MOST_EDGE_VISITS = {("infer", "even"): 10.0e10, ("infer", "pruned"): 8.0e10, ("skip_dead", "even"): 1.2e10,
                     ("train", "even"): 3.2e9, ("train", "pruned"): 1.0e10, ("train_single", "even"): 6.4e7}


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _degree(topo, n):
    return 32.0 if topo == "even" else 0.1 * n


def _depth(topo, n):
    if topo == "pruned":
        return 6
    return 120 if n < 8192 else 48 if n < 32768 else 24


def draw(rng):
    """One more case of the same ranges: widths from 1024 to 65536 (pruned: 1024 to 8192), batches from one vector
    to bulk blocks, both spread over their logarithm, half of the widths odd."""
    kind, topo = rng.choice([("infer", "even")] * 4 + [("train", "even")] * 4 + [("train_single", "even")] * 2 +
                            [("infer", "pruned"), ("train", "pruned"), ("skip_dead", "even")])
    n = _log_uniform(rng, 1024, {"skip_dead": 16384}.get(kind, 65536 if topo == "even" else 8192))
    n = n | 1 if rng.random() < 0.5 else n // 32 * 32
    layers_of_edges = _MOST_EDGE_VISITS[(kind, topo)] / (n * _degree(topo, n))  # one sample through this many layers
    if kind == "train_single":
        layers, batch = min(120, int(layers_of_edges)), 1
    else:
        layers = _depth(topo, n)
        hi = {"infer": 4096, "skip_dead": 2048, "train": 256}[kind]
        batch = _log_uniform(rng, 64 if kind == "skip_dead" else 1, min(hi, int(layers_of_edges / layers)))
    return dict(kind=kind, topo=topo, n=n, layers=layers, batch=batch)


# ---- nets and inputs -----------------------------------------------------------------------------------------------

class _Layer:
    """What sdnn.Net takes: CSR arrays on the host."""

    def __init__(self, n, row_ptr, col_idx, values, bias):
        self.n_out = self.n_in = n
        self.row_ptr, self.col_idx, self.values, self.bias = row_ptr, col_idx, values, bias


def _even_columns(gen, rows, n, d):
    """[rows][d] int32: d distinct, ascending, uniformly random columns per row."""
    cols = torch.randint(n, (rows, d), generator=gen, device=DEV, dtype=torch.int32).sort(dim=1).values
    while True:
        bad = (cols[:, 1:] == cols[:, :-1]).any(dim=1).nonzero().flatten()
        if bad.numel() == 0:
            return cols
        cols[bad] = torch.randint(n, (bad.numel(), d), generator=gen, device=DEV, dtype=torch.int32).sort(dim=1).values


def _even_layers(gen, case, scale, uniform, bias_mean, bias_sd):
    n, d = case["n"], 32
    row_ptr = torch.arange(0, n * d + 1, d, dtype=torch.int32).numpy()
    out = []
    for _ in range(case["layers"]):
        cols = _even_columns(gen, n, n, d).flatten().cpu().numpy()
        if uniform == "constant":
            vals = torch.full((n * d,), scale, device=DEV)
        elif uniform == "uniform":
            vals = (2.0 * torch.rand(n * d, generator=gen, device=DEV) - 1.0) * scale
        else:
            vals = torch.randn(n * d, generator=gen, device=DEV) * scale
        bias = bias_mean + bias_sd * torch.randn(n, generator=gen, device=DEV)
        out.append(_Layer(n, row_ptr, cols, vals.cpu().numpy(), bias.cpu().numpy()))
    return out


def _pruned_degrees(n):
    """The n quantiles of a Pareto tail of shape 1.2, scaled to a mean of n/10 and clipped to 1 .. n/4: the same degrees
    for every seed, dealt to the rows anew."""
    tail = ((torch.arange(n, dtype=torch.float64) + 0.5) / n).pow(-1.0 / 1.2)
    lo, hi = 0.0, float(n)
    for _ in range(60):
        mid = 0.5 * (lo + hi)
        if float((tail * mid).round().clamp(1, n // 4).mean()) < 0.1 * n:
            lo = mid
        else:
            hi = mid
    return (tail * hi).round().clamp(1, n // 4).to(torch.int64)


def _pruned_layers(gen, case):
    """Every row keeps its degree's number of uniformly random links; weights normal(0, 1/sqrt(degree)), no biases."""
    n, out = case["n"], []
    degrees = _pruned_degrees(n).to(DEV)
    for _ in range(case["layers"]):
        deg = degrees[torch.randperm(n, generator=gen, device=DEV)]
        row_ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
        row_ptr[1:] = deg.cumsum(0)
        key = torch.rand(n, n, generator=gen, device=DEV, dtype=torch.float64)
        last = key.sort(dim=1).values.gather(1, deg[:, None] - 1)  # the largest key that a row keeps
        row, col = (key <= last).nonzero(as_tuple=True)
        vals = torch.randn(col.numel(), generator=gen, device=DEV) / deg[row].float().sqrt()
        out.append(_Layer(n, row_ptr.to(torch.int32).cpu().numpy(), col.to(torch.int32).cpu().numpy(), vals.cpu().numpy(),
                          torch.zeros(n).numpy()))
    return out


def prepare(case, seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    kind, n, batch = case["kind"], case["n"], case["batch"]
    if case["topo"] == "pruned":
        layers, cap, act = _pruned_layers(gen, case), float("inf"), "relu"
        x = torch.randn(n, batch, generator=gen, device=DEV)
    elif kind == "skip_dead":
        # the benchmark nets themselves: weight 1/16, one negative bias, cap 32; samples of several densities, so that
        # some die in the first layers, some over the first dozen and some never
        layers, cap, act = _even_layers(gen, case, 0.0625, "constant", -0.32, 0.0), 32.0, "relu"
        dens = torch.tensor([0.10, 0.20, 0.30, 0.40], device=DEV)[torch.arange(batch, device=DEV) % 4]
        x = (torch.rand(n, batch, generator=gen, device=DEV) < dens).float()
    elif kind == "train_single":
        layers, cap, act = _even_layers(gen, case, 1.0, "uniform", 0.0, 0.0), float("inf"), "sigmoid"
        x = (torch.rand(n, batch, generator=gen, device=DEV) < 0.19).float()
    else:
        # weights that neither blow the activations up nor let them die over 120 layers of 32 links
        layers, cap, act = _even_layers(gen, case, 0.25, "normal", 0.0, 0.1), 32.0, "relu"
        x = (torch.rand(n, batch, generator=gen, device=DEV) < 0.19).float()
    training = kind in ("train", "train_single")
    state = dict(kind=kind, x=x, net=sdnn.Net(layers, cap, batch, training=training, activation=act),
                 xl=torch.empty(n, batch, device=DEV))
    if training:
        state["dloss"] = torch.empty(n, batch, device=DEV)
        if case["topo"] == "pruned":
            state["labels"] = torch.randint(10, (batch,), generator=gen, device=DEV, dtype=torch.int32)
            state["lr"] = 0.005
        else:
            state["target"] = torch.rand(n, batch, generator=gen, device=DEV)
            state["lr"] = 0.01
    if kind == "skip_dead":
        state["n_live"] = torch.zeros(1, dtype=torch.int32, device=DEV)
    return state


# ---- one pass -------------------------------------------------------------------------------------------------------

def run(state):
    net, x, xl = state["net"], state["x"], state["xl"]
    if state["kind"] == "infer":
        return net.sdnn_forward(x, xl)
    if state["kind"] == "skip_dead":
        net.sdnn_forward_skip_dead(x, xl, check_every=4, n_live=state["n_live"])
        return xl, state["n_live"]
    net.sdnn_forward(x, xl)
    if "labels" in state:
        sdnn.sdnn_softmax_ce_dloss(xl, state["labels"], 10, out=state["dloss"])
    else:
        sdnn.sdnn_mse_dloss(xl, state["target"], out=state["dloss"])
    net.sdnn_backward(state["dloss"])
    grad = net.sdnn_weight_grad(1)
    net.sdnn_sgd_step(state["lr"])
    look = sorted({*range(1, net.n_layers + 1, 16), net.n_layers})
    return [xl, state["dloss"], grad, [net.sdnn_get_weights(k) for k in look]]


def work(case):
    """Per layer with nnz entries: forward reads index and value of every entry and the biases (the activations between
    the layers are the library's own); a training step reads index and value for the forward pass and for
    back-propagation and writes the values, and keeps and reads back each layer's activations and deltas once.  Two
    operations per entry and sample and product (training: forward, back-propagation, gradient)."""
    n, batch, layers = case["n"], case["batch"], case["layers"]
    nnz = n * _degree(case["topo"], n)
    if case["kind"] in ("infer", "skip_dead"):
        return {"bytes": layers * (8 * nnz + 4 * n) + 8 * n * batch, "flops": 2 * layers * nnz * batch}
    return {"bytes": layers * (20 * nnz + 12 * n + 16 * n * batch), "flops": 6 * layers * nnz * batch}


def tolerance(case):
    """fp32 storage, every sum accumulated in fp64 and rounded once: another order of the sums shows in the last bit of a
    stored value now and then.  Whole values (the live-sample count) are exact."""
    return {"rel": 1e-5}
