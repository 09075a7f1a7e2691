"""Nets that take the forward in panels, or train with one launch per pass: the same for tests/test_gpu_pan_forward.py and
tests/test_gpu_train_lds.py (on the GPU) and tests/test_routes.py (which launches they take)."""
import numpy as np

from paper_2104_11805_amd import workloads as wl

# widths of the layers, samples, lengths of the rows in turn: one to four panels, layers on both sides of a panel and of a block
# of 64 rows, a last range that is nearly empty, rows past a half of eight slots
NETS = [((20001, 16385, 33000, 17000), 999, (0, 1, 40, 64, 90)), ((65536, 49153, 16384, 70), 200, (33, 31, 64)),
        ((50, 32769, 1025, 32768, 16449), 511, (7, 60, 25, 0, 129)), ((40000, 40000, 40000, 40000), 129, (32,))]

# training with one launch per pass: widths, max_batch, lengths of the rows in turn, columns that every row has, samples of the steps
# one after the other.  2048 positions (all of a buffer) next to narrow layers; 2047; batches of a net made for more; rows and columns
# of up to the 512 entries that are taken; a long row among short ones in every block
TRAIN_NETS = [((2048, 300, 2048, 300, 2048), 64, (8, 3), 0, (64, 2)), ((2047,) * 9, 200, (8,), 0, (200, 67)),
              ((1024, 1025, 640, 1024, 100), 200, (32, 0, 16), 0, (7, 130, 1, 7)), ((512, 512, 500, 512, 512, 512), 33, (1, 6, 2, 512), 1, (33, 9)),
              ((700,) * 6, 64, (16,) * 20 + (100,), 0, (64, 3)), ((511, 300, 511, 511, 400), 256, (4,) * 60 + (500,), 2, (256, 250))]


def layers(widths, lengths, seed=7000, full=0):
    """Row r of a layer holds lengths[r % len(lengths)] random columns (duplicates dropped; from 500 on all of them)
    and the first `full`."""
    out = []
    for k, (n_in, n_out) in enumerate(zip(widths, widths[1:])):
        rng = np.random.default_rng(seed + k)
        deg = np.minimum(np.resize(np.asarray(lengths), n_out), n_in)
        rows = np.repeat(np.arange(n_out), deg)
        key = rows * np.int64(n_in) + rng.integers(0, n_in, rows.size)
        whole = np.flatnonzero(deg >= 500)[:, None] * np.int64(n_in) + np.arange(n_in if deg.max() >= 500 else 0)
        key = np.unique(np.concatenate([key, whole.ravel(), (np.arange(n_out)[:, None] * np.int64(n_in) + np.arange(full)).ravel()]))
        row_ptr = np.searchsorted(key, np.arange(n_out + 1, dtype=np.int64) * n_in).astype(np.int32)
        cols = (key % n_in).astype(np.int32)
        vals = (rng.standard_normal(cols.size) * 0.3).astype(np.float32)
        out.append(wl.Layer(n_out, n_in, row_ptr, cols, vals, (rng.standard_normal(n_out) * 0.2).astype(np.float32)))
    return out
