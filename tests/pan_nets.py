"""Nets that take the forward in panels: the same for tests/test_gpu_pan_forward.py (on the GPU, against the oracle) and
tests/test_routes.py (which launches they take)."""
import numpy as np

from paper_2104_11805_amd import workloads as wl

# widths of the layers, samples, lengths of the rows in turn: one to four panels, layers on both sides of a panel and of a block
# of 64 rows, a last range that is nearly empty, rows past a half of eight slots
NETS = [((20001, 16385, 33000, 17000), 999, (0, 1, 40, 64, 90)), ((65536, 49153, 16384, 70), 200, (33, 31, 64)),
        ((50, 32769, 1025, 32768, 16449), 511, (7, 60, 25, 0, 129)), ((40000, 40000, 40000, 40000), 129, (32,))]


def layers(widths, lengths, seed=7000):
    """Row r of a layer holds lengths[r % len(lengths)] random columns (duplicates dropped)."""
    out = []
    for k, (n_in, n_out) in enumerate(zip(widths, widths[1:])):
        rng = np.random.default_rng(seed + k)
        deg = np.minimum(np.resize(np.asarray(lengths), n_out), n_in)
        rows = np.repeat(np.arange(n_out), deg)
        key = np.unique(rows * np.int64(n_in) + rng.integers(0, n_in, rows.size))
        row_ptr = np.searchsorted(key, np.arange(n_out + 1, dtype=np.int64) * n_in).astype(np.int32)
        cols = (key % n_in).astype(np.int32)
        vals = (rng.standard_normal(cols.size) * 0.3).astype(np.float32)
        out.append(wl.Layer(n_out, n_in, row_ptr, cols, vals, (rng.standard_normal(n_out) * 0.2).astype(np.float32)))
    return out
