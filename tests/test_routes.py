"""Which calls are launched and which are refused, at sizes that the GPU tests do not reach (no GPU: see tests/routes.py)."""
import pytest

from tests import routes


@pytest.mark.parametrize("links", [2, 40])
def test_last_narrow_block_of_a_wide_net(links):
    """A pass cut into blocks of 64 samples for the panel sweep; the last block, of 40 samples or fewer, does not take that
    sweep, nor (1000 rows) the kernel with several rows per wavefront."""
    routes.run(f"""
        net = Net([layer(65536, 65536, ({links},)), layer(1000, 65536, ({links},))], 1200)
        for B in [*range(129, 257), 340, 1100]:
            rc, log = net("sdnn_forward", X0, B, XL, None)
            assert rc == 0, (B, sdnn.last_error(net.h))
            assert len(log) == 2 * -(-B // 64), (B, log)
            if 0 < B % 64 <= 40:
                assert log[-1].startswith("k_spmm<") and B // 64 * 64 % (64 * int(log[-1][7])) == 0, (B, log)
    """)


def test_result_across_the_input():
    """A result that overlaps the input without being the same block: a launch per layer, which has read the input by then."""
    routes.run("""
        net = Net([layer(5000, 5000, (8,))] * 3, 2000, lds_forward=1)
        for shift, lds in [(0, True), (4, False), (-4, False), (4 * 5000 * 2000 - 4, False), (4 * 5000 * 2000, True), (-4 * 5000 * 2000, True)]:
            rc, log = net("sdnn_forward", X0, 2000, X0 + shift, None)
            assert rc == 0 and (len(log) == 1 and log[0].startswith("k_fwd_lds")) == lds, (shift, log)
    """)


def test_result_across_the_input_in_one_piece():
    """Blocks of activations past the memory-side cache go through all layers in sub-blocks of samples, whose results must not replace
    inputs of the later ones."""
    routes.run("""
        net = Net([layer(5000, 5000, (8,))] * 3, 2000, lds_forward=-1)
        for shift, pieces in [(0, 3), (4, 1), (-4, 1), (4 * 5000 * 2000 - 4, 1), (4 * 5000 * 2000, 3)]:
            rc, log = net("sdnn_forward", X0, 2000, X0 + shift, None)
            assert rc == 0 and len(log) == 3 * pieces, (shift, log)
    """)


def test_gradient_over_two_windows_of_samples():
    """Two rounded windows only where the batch itself is 128 samples on up to 16384 neurons (two partial gradients from 6.5 MB on):
    not for the batches that are filled up to 128."""
    routes.run("""
        for n, B, kernel, rows, tiles in [(12695, 128, "<32, true>", 8, 1), (12696, 128, "<16, false>", 16, 2), (16384, 128, "<16, false>", 16, 2),
                                          (16385, 128, "<32, false>", 8, 1), (16384, 124, "<32, false>", 8, 1), (16384, 125, "<32, false>", 8, 1),
                                          (16384, 127, "<32, false>", 8, 1), (16384, 129, "<64, false>", 4, 1), (4096, 128, "<32, true>", 8, 1),
                                          (4096, 125, "<32, false>", 8, 1), (4096, 127, "<32, false>", 8, 1)]:
            net = Net([layer(n, n, (32,))], 300, training=True)
            assert net("sdnn_forward", X0, B, XL, None)[0] == 0
            rc, log = net("sdnn_backward", DL, None)
            assert rc == 0 and log[-1] == f"k_bwd_rows{kernel} {tiles * -(-n // rows)} 1 1", (n, B, log)
    """)


def test_backward_refuses_an_operand_of_4_gib():
    """The last layer's own block is an operand of the sweep that forms the gradient (and of back-propagation, where there is a
    layer below): byte offsets into it are 32 bits.  Nothing is launched."""
    routes.run("""
        n = 17000000                                   # x 64 samples x 4 bytes: just over 4 GiB
        wide = layer(n, 8, (1, 0, 0, 0))
        for layers, fuse, refused in [([wide], 1, True), ([wide], -1, False), ([layer(8, 4, (2,)), wide], -1, True)]:
            net = Net(layers, 64, training=True, fuse_gradient=fuse)
            assert net("sdnn_forward", X0, 64, XL, None)[0] == 0, sdnn.last_error(net.h)
            rc, log = net("sdnn_backward", DL, None)
            assert (rc, log) == (sdnn.SDNN_EINVAL, []) if refused else (rc == 0 and log), (rc, log)
            assert not refused or "4 GiB" in sdnn.last_error(net.h)
            lib.sdnn_destroy(net.h)
    """)


@pytest.mark.parametrize("training", [False, True])
@pytest.mark.parametrize("fuse", [-1, 1])
def test_blocks_below_4_gib_are_taken_whatever_their_row_pitch(training, fuse):
    """17e6 neurons: 63 samples fit 32-bit offsets, 64 do not; 33 would not with rows of 64 floats."""
    routes.run(f"""
        n = 17000000
        layers = [layer(n, 8, (1, 0, 0, 0)), layer(8, n, (5, 40))]
        for max_batch, batches in [(63, (33, 63, 2, 61, 50)), (33, (33, 32, 5)), (64, (64, 60))]:
            net = Net(layers, max_batch, training={training}, fuse_gradient={fuse})
            rows = n + 8 + ({training} and n + 8 + 8 or n)             # X_0, X_l, Delta_l or two activation buffers
            assert net.bytes < 4 * rows * (max_batch + 3) + 300 * n, net.bytes
            for B in batches:
                rc, log = net("sdnn_forward", X0, B, XL, None)
                assert rc == (sdnn.SDNN_EINVAL if B == 64 else 0), (B, sdnn.last_error(net.h))
                if B == 64 or not {training}:
                    continue
                rc, log = net("sdnn_backward", DL, None)
                assert rc == 0 and (B != 63 or not any("k_bwd_rows" in l for l in log)), (B, log)
                rc, log = net("sdnn_sgd_step", C.c_float(0.1), None)
                assert rc == 0 and ({fuse} == 1 or ("<1, 0>" in log[0]) == (B > 60)), (B, log)
            lib.sdnn_destroy(net.h)
    """)


@pytest.mark.parametrize("n_out,n_in,lengths", [(64, 64, (64,)), (300, 300, (1, 0, 7)), (1000, 64, (33,)), (64, 1000, (9, 100)),
                                                (700, 90, (88, 3, 16)), (5, 3, (0,)), (513, 2, (1,)), (3000, 70000, (40, 64)),
                                                (70000, 3000, (2, 5))])
def test_workspace_sized_without_the_columns(n_out, n_in, lengths):
    """A net of one sample per step: what the sizes alone give is enough for sdnn_create, whatever the columns are (here as
    uneven as the row lengths allow: every row starts at column 0)."""
    routes.run(f"""
        layers = [layer({n_out}, {n_in}, {lengths}), layer({n_in}, {n_out}, {lengths[:1]})]
        for max_batch, training in [(1, True), (7, True), (1, False)]:
            a, b = Net(layers, max_batch, training=training, col_idx=False), Net(layers, max_batch, training=training)
            assert a.bytes >= b.bytes and (a.bytes == b.bytes or (max_batch, training) == (1, True)), (a.bytes, b.bytes)
            assert a("sdnn_forward", X0, 1, XL, None) == b("sdnn_forward", X0, 1, XL, None)
    """)


def test_one_sample_takes_a_launch_per_layer_on_the_lane_major_copy():
    """The nets of tests/test_gpu_single_sample.py and tests/test_gpu_nonfinite.py."""
    routes.run("""
        for sizes in [(90, 64, 30000, 70), (90, 1025, 30000, 1024, 70), (2050, 30000, 63), (2050, 30000, 2113)]:
            net = Net([layer(o, i, (0, 1, 9, 16, 17, 33)) for i, o in zip(sizes, sizes[1:])], 4)
            for call in ("sdnn_forward", "sdnn_forward_noalloc"):
                rc, log = net(call, X0, 1, XL, None)
                assert rc == 0 and len(log) == len(sizes) - 1 and all(l.startswith("k_spmv_lm<0, false, false>") for l in log), log
    """)


def test_single_launch_or_a_launch_per_layer():
    """Where one of the two paths was measured at least 7 % faster than the other (32 entries per row; uneven rows: a tenth of
    the columns in the mean), that one is taken."""
    routes.run("""
        for n, layers, single, per_layer in [(1500, 24, (16, 100, 1100), ()), (3001, 24, (100, 450), (2, 33, 64)), (5000, 24, (150, 700), (2, 64, 100)),
                                             (8000, 24, (200, 450), (1, 100, 150)), (16384, 24, (300, 1100), (1, 64, 100, 150, 200)),
                                             (20000, 24, (450, 700), (1, 100, 150, 300)), (32000, 24, (200, 256, 450, 700), (1, 33, 100, 150, 300))]:
            net = Net([layer(n, n, (32,))] * layers, 1100)
            for B in single + per_layer:
                rc, log = net("sdnn_forward", X0, B, XL, None)
                assert rc == 0 and (len(log) == 1) == (B in single), (n, B, log)
        tail = (np.arange(4097) + 0.5) ** (-1 / 1.2)
        for n, single, per_layer in [(1024, (1, 2, 64, 100, 450), ()), (2000, (100, 200, 450, 1100), (1, 2, 64)), (4097, (450,), (1, 2, 64, 200))]:
            deg = np.clip(np.round(tail[:n] / tail[:n].mean() * 0.12 * n), 1, n // 4).astype(int)
            net = Net([layer(n, n, deg)] * 6, 1100)
            for B in single + per_layer:
                rc, log = net("sdnn_forward", X0, B, XL, None)
                assert rc == 0 and (len(log) == 1) == (B in single), (n, B, deg.mean(), log)
    """)


def test_more_results_than_a_launch_has_threads():
    """Layers of 2^34 results in a launch and more: the kernel that walks its blocks.  (The stand-in refuses launches of 2^32
    threads.)"""
    routes.run("""
        net = Net([layer(68000000, 8, (1, 0, 0, 0))], 256)
        for B, kernel in [(100, "k_rows<"), (256, "k_spmm<")]:
            rc, log = net("sdnn_forward", X0, B, XL, None)
            assert rc == 0 and len(log) == 1 and log[0].startswith(kernel), (B, log, sdnn.last_error(net.h))
    """)


def test_forward_in_panels():
    """Which passes go in panels: those of tests/test_gpu_pan_forward.py, and where that path was measured faster than the others
    by 7 % and more (32 entries per row, 24 layers); not with links that stay within one panel, over two layers, in the fixed
    staging array, where the caller asks for other layouts, or with one sample."""
    routes.run("""
        from tests import pan_nets
        def spread(n, n_in, links):
            ci = np.sort((np.arange(links) * (n_in // links) + np.random.default_rng(n).integers(0, n_in // links, (n, links))), axis=1)
            return n, n_in, np.arange(0, n * links + 1, links, dtype=np.int32), ci.astype(np.int32).ravel(), np.ones(n * links, np.float32), None
        def pans(net, B, call="sdnn_forward"):
            rc, log = net(call, X0, B, XL, None)
            assert rc == 0, sdnn.last_error(net.h)
            n = sum(l.startswith("k_fwd_pan<") for l in log)
            assert n in (0, len(net.keep)) and (n == 0 or (len(log) == n + 2 and log[0].startswith("k_pan_turn<true>"))), log
            return n > 0
        for widths, b, lengths in pan_nets.NETS:
            net = Net([(y.n_out, y.n_in, y.row_ptr, y.col_idx, y.values, y.bias) for y in pan_nets.layers(widths, lengths)], b)
            assert pans(net, b) and not pans(net, 1)
            lib.sdnn_destroy(net.h)
        for n, yes, no in [(16384, (), (512, 1024)), (20001, (512, 700, 1024), (1, 33, 64, 100)), (25000, (200, 512, 700, 1024), (33, 64)),
                           (32768, (100, 150, 256, 300, 400, 512, 1024), (33, 64)), (40000, (100, 200, 512, 1024), (33, 64)), (65536, (100, 150, 256, 1024), (33, 64))]:
            net = Net([spread(n, n, 32)] * 24, 1024)
            assert [pans(net, B) for B in yes + no] == [True] * len(yes) + [False] * len(no), (n, [(B, pans(net, B)) for B in yes + no])
            lib.sdnn_destroy(net.h)
        assert not pans(Net([layer(40000, 40000, (32,))] * 4, 512), 512)
        assert not pans(Net([spread(40000, 40000, 32)] * 2, 512), 512)
        assert not pans(Net([spread(40000, 40000, 32)] * 4, 512), 50, "sdnn_forward_noalloc")
        for options in (dict(lds_forward=-1), dict(panel_cols=8192), dict(reorder_rows=1), dict(training=True)):
            assert not pans(Net([spread(40000, 40000, 32)] * 3, 512, **options), 512)
    """)


def test_forward_in_panels_beside_the_single_launch():
    """A result that lies across the input cannot take the single launch: what the panels are compared with is a launch per layer.
    lds_forward = ON takes the single launch with every batch and holds no copy for panels; layers too wide for it still do."""
    routes.run("""
        def spread(n, n_in, links):
            ci = np.sort((np.arange(links) * (n_in // links) + np.random.default_rng(n).integers(0, n_in // links, (n, links))), axis=1)
            return n, n_in, np.arange(0, n * links + 1, links, dtype=np.int32), ci.astype(np.int32).ravel(), np.ones(n * links, np.float32), None
        def kernel(net, B, xl=XL):
            rc, log = net("sdnn_forward", X0, B, xl, None)
            assert rc == 0
            return log[len(log) // 2].split("<")[0]
        net = Net([spread(18000, 18000, 32)] * 24, 1024)
        for B in (507, 729, 951):
            assert [kernel(net, B), kernel(net, B, X0 + 4)] == ["k_fwd_lds", "k_fwd_pan"], B
        auto, on, off = (Net([spread(32768, 32768, 32)] * 4, 1024, lds_forward=o) for o in (0, 1, -1))
        assert [kernel(n, 512) for n in (auto, on)] == ["k_fwd_pan", "k_fwd_lds"]
        entries = 4 * 32 * 32768
        assert on.bytes - off.bytes < 7 * entries and auto.bytes - on.bytes > 6 * entries
        rc, log = on("sdnn_set_weights", 2, X0, XL, None)
        assert rc == 0 and not any(l.startswith("k_pan") for l in log), (rc, log)
        assert kernel(Net([spread(40000, 40000, 32)] * 4, 1024, lds_forward=1), 512) == "k_fwd_pan"
    """)


def test_training_with_one_launch_per_pass():
    """Narrow nets of short rows and at least four layers: not with one sample, more samples than compute units, long rows or
    columns, the gradient formed in the sweep, or lds_forward off."""
    routes.run("""
        from tests import pan_nets
        def nets(widths, lengths, max_batch, **options):
            ls = pan_nets.layers(widths, lengths, seed=8100)
            return Net([(y.n_out, y.n_in, y.row_ptr, y.col_idx, y.values, y.bias) for y in ls], max_batch, training=True, **options)
        def passes(net, B):
            rc, f = net("sdnn_forward", X0, B, XL, None)
            assert rc == 0
            rc, b = net("sdnn_backward", DL, None)
            assert rc == 0
            rc, u = net("sdnn_sgd_step", C.c_float(0.1), None)
            assert rc == 0
            n = sum(l.startswith("k_train_fill") for l in u)
            return any("k_train_lds<0" in l for l in f), any("k_train_lds<1" in l for l in b), n
        for widths, b, lengths in [((1024,) * 5, 64, (32,)), ((50, 1025, 63, 1000, 7), 5, (0, 1, 16, 17, 33)), ((300, 1400, 1300, 64, 1), 255, (7, 8, 9)),
                                   ((1024, 65, 1023, 129, 1024, 40), 2, (15, 31, 64)), ((200, 900, 800, 700, 100), 9, (20, 40)), ((300, 1024, 1024, 1024, 50), 5, (0, 5, 17, 40))]:
            assert passes(nets(widths, lengths, b), b) == (True, True, 2), widths
        n = (1024,) * 5
        assert passes(nets(n, (32,), 64), 1)[:2] == (False, False)
        for net, B in [(nets(n[:4], (32,), 64), 64), (nets(n, (32,), 64, lds_forward=-1), 64), (nets(n, (32,), 64, fuse_gradient=1), 64), (nets(n, (32,), 300), 64),
                       (nets((2049,) + n, (32,), 64), 64), (nets((1024,) * 5, (1, 600), 64, fuse_gradient=-1), 64)]:
            assert passes(net, B) == (False, False, 0), (net.keep[0][0], passes(net, B))
        rc, log = nets(n, (32,), 64)("sdnn_set_weights", 2, X0, XL, None)
        assert rc == 0 and sum(l.startswith("k_train_fill") for l in log) == 2
    """)


def test_training_with_one_launch_per_pass_by_the_batch():
    """The same net steps in either way: with a launch per layer where wide layers meet few samples, or more samples than compute
    units; on half of a chip's compute units they are not idle while the copies come."""
    routes.run("""
        from tests import pan_nets
        def batches(n, links, max_batch, cus=256, depth=12, **options):
            stub.stub_cus(cus)
            ls = pan_nets.layers((n,) * 13, links if isinstance(links, tuple) else (links,), seed=8400)
            net = Net([(y.n_out, y.n_in, y.row_ptr, y.col_idx, y.values, y.bias) for y in ls * (depth // 12)], max_batch, training=True, **options)
            single = []
            for B in (2, 16, 33, 64, 96, 127, 128, 200, 256):
                if B > max_batch:
                    break
                rc, f = net("sdnn_forward", X0, B, XL, None)
                assert rc == 0
                rc, b = net("sdnn_backward", DL, None)
                assert rc == 0
                f, b = ([l.startswith("k_train_lds") for l in log] for log in (f, b))
                assert any(f) == any(b), (n, B)
                single += [B] * any(f)
            lib.sdnn_destroy(net.h)
            return single
        every = [2, 16, 33, 64, 96, 127, 128, 200, 256]
        for n, links, max_batch, want in [(300, 32, 256, every), (1024, 32, 256, every), (1201, 32, 256, every), (1600, 32, 64, [33, 64]), (1800, 32, 64, []),
                                          (2048, 32, 64, []), (1024, 64, 64, every[:4]), (512, 160, 64, every[:4]), (2048, 8, 200, every[:-1])]:
            got = batches(n, links, max_batch)
            assert got == want, (n, links, max_batch, got)
        assert batches(2048, 32, 127, fuse_gradient=-1) == [96, 127]
        for n, want in [(1500, [2, 16, 33, 64]), (1600, [16, 33, 64]), (1850, [64]), (2048, [])]: # W does not stay in the L2s
            got = batches(n, 32, 64, depth=120)
            assert got == want, (n, got)
        # a longer row in every block of 64: W follows the order of the rows of the W^T above, and the room for it is not that of sorted rows
        for n, links in [(700, (16,) * 20 + (100,)), (512, (8,) * 63 + (200,)), (300, (4,) * 60 + (500,))]:
            assert batches(n, links, 64) == every[:4], (n, links)
        assert batches(300, 32, 256, cus=128) == every[:7]
    """)


def test_training_with_one_launch_per_pass_at_its_limits():
    """The nets of tests/test_gpu_train_lds.py go through it; a row or a column of 513 entries, and more samples than compute units,
    do not."""
    routes.run("""
        from tests import pan_nets
        def single(widths, max_batch, lengths, full, batches):
            ls = pan_nets.layers(widths, lengths, seed=8500, full=full)
            net = Net([(y.n_out, y.n_in, y.row_ptr, y.col_idx, y.values, y.bias) for y in ls], max_batch, training=True)
            out = []
            for B in batches:
                rc, log = net("sdnn_forward", X0, B, XL, None)
                assert rc == 0
                out.append(any(l.startswith("k_train_lds") for l in log))
            return out
        for case in pan_nets.TRAIN_NETS:
            assert single(*case) == [B > 1 for B in case[4]], (case, single(*case))
        assert single((600,) * 6, 33, (1, 6, 2, 5), 0, (33,)) == [True]
        assert single((600,) * 6, 33, (1, 6, 2, 5), 1, (33,)) == [False]
        assert single((513,) * 6, 33, (1, 6, 2, 513), 0, (33,)) == [False]
        stub.stub_cus(128)
        assert single((300,) * 6, 256, (8,), 0, (127, 128, 129, 256)) == [True, True, False, False]
    """)


def test_copies_of_narrow_training_nets_follow_when_they_are_read():
    """A step that does not read the copies leaves them behind; the next pass that reads them brings them up to date first.  Not in
    a graph, and not once a graph reads them: its replays have to find them current."""
    routes.run("""
        from tests import pan_nets
        def net(n=1600, max_batch=64):
            ls = pan_nets.layers((n,) * 13, (32,), seed=8400)
            return Net([(y.n_out, y.n_in, y.row_ptr, y.col_idx, y.values, y.bias) for y in ls], max_batch, training=True)
        def fills(net, B, capture=()):
            out = []
            for k, (name, args) in enumerate([("sdnn_forward", (X0, B, XL, None)), ("sdnn_backward", (DL, None)), ("sdnn_sgd_step", (C.c_float(0.1), None))]):
                stub.stub_capture(k in capture)
                rc, log = net(name, *args)
                assert rc == 0
                out.append(sum(l.startswith("k_train_fill") for l in log))
                assert not out[-1] or k == 2 or log[0].startswith("k_train_fill") or log[1].startswith("k_train_fill"), log
            stub.stub_capture(0)
            return out
        a = net()
        assert [fills(a, B) for B in (64, 2, 1, 2, 64, 64)] == [[0, 0, 2], [0, 0, 0], [0, 0, 0], [0, 0, 0], [2, 0, 2], [0, 0, 2]]
        for B in (1, 2):                               # a captured step, and what follows it
            b = net()
            assert [fills(b, B, (0, 1, 2)), fills(b, B), fills(b, 64), fills(b, B)] == [[0, 0, 2], [0, 0, 0], [2, 0, 2], [0, 0, 0]]
        c = net()                                      # a graph that reads copies which are behind, and a pass after it
        assert [fills(c, 2), fills(c, 64, (0, 1)), fills(c, 2), fills(c, 64), fills(c, 2), fills(c, 64)] == [[0, 0, 0], [2, 2, 2], [0, 0, 2], [2, 0, 2], [0, 0, 2], [0, 0, 2]]
        d = net()
        assert [fills(d, 64, (0, 1, 2)), fills(d, 1), fills(d, 64)] == [[0, 0, 2], [0, 0, 2], [0, 0, 2]]
        def replaced(net, layers, capture=0):
            stub.stub_capture(capture)
            out = []
            for k in layers:
                rc, log = net("sdnn_set_weights", k, X0, XL, None)
                assert rc == 0
                out.append(sum(l.startswith("k_train_fill") for l in log))
            stub.stub_capture(0)
            return out
        e = net()                                      # all layers replaced: the first one's copy (W_1^T has none) at once, the others' with the next pass
        assert replaced(e, range(1, 5)) == [1, 0, 0, 0] and fills(e, 64) == [2, 0, 2] and replaced(e, (3,)) == [2] and fills(e, 64) == [0, 0, 2]
        assert replaced(e, (2, 3)) == [2, 0] and replaced(e, (3, 4), 1) == [2, 2] and fills(e, 64, (0, 1)) == [2, 2, 2]
        assert replaced(e, (2, 3)) == [2, 2] and fills(e, 64) == [2, 0, 2] and replaced(e, (2, 3)) == [2, 2] and fills(e, 64) == [0, 0, 2]
    """)


def test_back_propagation_of_one_sample():
    """In rounds of eight chunks up to three wavefronts per CU, of four in wider layers and with 4-byte columns."""
    routes.run("""
        for n, kernel in [(3000, "<1, false, true>"), (49152, "<1, false, true>"), (49153, "<2, false, true>"), (65536, "<2, false, true>"), (65537, "<1, true, true>")]:
            ci = np.sort((np.arange(n)[:, None] + 17 * np.arange(8)) % n, axis=1).astype(np.int32).ravel()
            net = Net([(n, n, np.arange(0, 8 * n + 1, 8, dtype=np.int32), ci, np.ones(8 * n, np.float32), None)] * 2, 1, training=True)
            assert net("sdnn_forward", X0, 1, XL, None)[0] == 0
            rc, log = net("sdnn_backward", DL, None)
            assert rc == 0 and [l for l in log if l.startswith("k_spmv_lm")] == [f"k_spmv_lm{kernel} {-(-n // 64)} 1 1"], (n, log)
    """)


def test_turns_at_priority_between_equal_shares():
    """With 1, 2 and 4 samples per workgroup of the LDS forward: the wavefronts do not take turns where the blocks left over, or one
    deep block, make the shares of a few of them longer than the others', nor on the longest rows."""
    routes.run("""
        def turns(deg):
            n = len(deg)
            net = Net([layer(n, n, deg)] * 2, 1024, lds_forward=1)
            out = {}
            for B in (200, 500, 1000):
                rc, log = net("sdnn_forward", X0, B, XL, None)
                assert rc == 0 and len(log) == 1
                out[int(log[0][10])] = stub.stub_arg()[22]           # LdsForward::turns
            return out
        def uneven(n):
            # a tenth of the columns in the mean, at most a quarter
            tail, lo, hi = ((np.arange(n) + 0.5) / n) ** (-1 / 1.2), 0.0, n
            while hi - lo > 1e-6:
                mid = (lo + hi) / 2
                lo, hi = (mid, hi) if np.clip(np.round(tail * mid), 1, n // 4).mean() < 0.1 * n else (lo, mid)
            return np.clip(np.round(tail * hi), 1, n // 4).astype(int)
        none, every, four = {1: 0, 2: 0, 4: 0}, {1: 1, 2: 1, 4: 1}, {1: 0, 2: 0, 4: 1}
        for n, want in [(300, none), (1024, none), (1025, none), (1089, none), (1565, none), (1792, none), (1793, every), (2048, every),
                        (2100, four), (2432, four), (2433, every), (3001, every), (3100, every), (4096, every), (7000, every)]:
            assert turns([32] * n) == want, (n, turns([32] * n))
        for n, want in [(1300, none), (2000, none), (3001, every), (4097, every), (6000, {1: 0, 2: 1, 4: 1}), (8192, {1: 0, 2: 1, 4: 1})]:
            assert turns(uneven(n)) == want, (n, turns(uneven(n)))
        assert turns([820] * 8192) == four
        net = Net([layer(4096, 4096, (32,)), layer(10, 4096, (32,))], 1024, lds_forward=1) # a narrow layer does not matter
        assert net("sdnn_forward", X0, 1000, XL, None)[0] == 0 and stub.stub_arg()[22] == 1
        net = Net([layer(1300, 1300, (32,))] * 3, 1024, act_cap=32.0, lds_forward=1)
        assert net("sdnn_forward_skip_dead", X0, 1000, XL, 1, DL, None)[0] == 0 and stub.stub_arg()[22] & 7 == 0
    """)


def test_order_of_the_loads_with_one_sample():
    """The LDS forward with one sample per workgroup requests its loads strictly in order where there are few rounds of blocks or the
    layers are larger than an L2."""
    routes.run("""
        def order(deg, activation=0):
            n = len(deg)
            net = Net([layer(n, n, deg)] * 2, 1024, lds_forward=1, activation=activation)
            rc, log = net("sdnn_forward", X0, 1 if n == 16384 else 2, XL, None)
            assert rc == 0 and len(log) == 1 and log[0].startswith(f"k_fwd_lds<1, {activation}, "), (n, log)
            return log[0].split(", ")[2].startswith("true")
        def uneven(n):
            tail, lo, hi = ((np.arange(n) + 0.5) / n) ** (-1 / 1.2), 0.0, n
            while hi - lo > 1e-6:
                mid = (lo + hi) / 2
                lo, hi = (mid, hi) if np.clip(np.round(tail * mid), 1, n // 4).mean() < 0.1 * n else (lo, mid)
            return np.clip(np.round(tail * hi), 1, n // 4).astype(int)
        for n, links, want in [(300, 32, True), (1024, 200, True), (1025, 33, True), (1216, 33, True), (1217, 33, False), (1300, 32, True), (1856, 64, True),
                               (2048, 32, True), (2049, 32, False), (2500, 32, True), (3072, 64, True), (3500, 32, False), (4096, 32, False), (4096, 128, False),
                               (4097, 33, False), (8192, 96, False), (8192, 128, True), (16384, 16, False), (16384, 64, True), (9000, 256, True)]:
            for activation in (0, 1):
                assert order([links] * n, activation) == want, (n, links, activation)
        assert [order(uneven(n)) for n in (1000, 1180, 1249, 2000, 6000, 8192)] == [True, True, False, False, True, True]
    """)


def test_long_forward_requests_nothing_past_its_copy():
    """A wavefront requests two halves of eight slots past the last one of its block: also those of the last layer, whose copy ends the
    workspace, have room in it."""
    routes.run("""
        for widths, lengths in [((1024, 1024, 1024), (256,)), ((8192, 300), (8192, 700, 3)), ((1500, 1089, 1281), (0, 1, 250, 512, 300)), ((8192, 8192), (2048, 64, 20, 8))]:
            net = Net([layer(o, i, np.minimum(np.resize(lengths, o), i)) for i, o in zip(widths, widths[1:])], 100, training=True)
            rc, log = net("sdnn_forward", X0, 100, XL, None)
            assert rc == 0 and sum(l.startswith("k_fwd_long<") for l in log) == len(widths) - 1, log
            rp = net.keep[-1][2]
            deg = np.sort(np.diff(rp))[::-1]
            halves = int(((deg[::64] + 7) // 8).sum())
            lm, sizes = stub.stub_long_arg()[2], stub.stub_long_arg()[6]
            assert 3072 * (halves + 2) <= sizes & 0xffffffff and lm + (sizes & 0xffffffff) <= ADDR + net.bytes, (widths, lm - ADDR, net.bytes)
    """)


def test_long_forward_by_the_batch():
    """From 65 samples on; more groups of four samples than compute units only where the rounds are three quarters full and every layer
    has blocks for all wavefronts, none much deeper than the others."""
    routes.run("""
        def batches(net):
            out = []
            for B in (1, 64, 65, 255, 1024, 1025, 1532, 1533, 2048, 2049, 2300, 2301, 3072, 3073):
                rc, log = net("sdnn_forward", X0, B, XL, None)
                n = sum(l.startswith("k_fwd_long<") for l in log)
                assert rc == 0 and n in (0, len(net.keep)) and all(not l.startswith("k_fwd_long<") or int(l.split()[1]) * 4 >= B for l in log), (B, log)
                out += [B] * (n > 0)
            lib.sdnn_destroy(net.h)
            return out
        few, many = [65, 255, 1024], [1533, 2048, 2301, 3072, 3073]
        for widths, lengths, want in [((1024, 1024), (256,), few + many), ((1000, 961), (256,), few + many), ((1000, 960), (256,), few), ((8192, 64), (2400,), few),
                                      ((2048, 2048), (632,) + (140,) * 63, few + many), ((2048, 2048), (633,) + (140,) * 63, few)]:
            got = batches(Net([layer(o, i, lengths) for i, o in zip(widths, widths[1:])], 3073, training=True))
            assert got == want, (widths, got)
        stub.stub_cus(128)
        assert batches(Net([layer(1024, 1024, (256,))], 3073, training=True)) == [65, 255, 1024, 1532, 1533, 2048, 2049, 2300, 2301, 3072, 3073]
    """)


def test_long_forward_refuses_an_operand_of_4_gib():
    """As the kernel that it stands in for does: 8192 neurons, 131072 samples."""
    routes.run("""
        for n, B, want in [(8192, 131068, 0), (8192, 131072, sdnn.SDNN_EINVAL), (8191, 131072, 0)]:
            net = Net([layer(n, n, (128,))], B, training=True)
            rc, log = net("sdnn_forward", X0, B, None, None)
            assert rc == want and (rc == 0 or "4 GiB" in sdnn.last_error(net.h)) and (rc == 0) == any(l.startswith(("k_fwd_long", "k_spmm")) for l in log), (n, B, rc, log)
            lib.sdnn_destroy(net.h)
    """)


def test_sweep_of_long_rows():
    """129 to 256 samples and 64 entries per row of W^T and more; more than that on operands over 10.7 MB, and not over 26 MB (225 samples and
    more: 16 MB)."""
    routes.run("""
        def kernel(n, deg, B):
            net = Net([layer(n, n, deg)], 256, training=True, fuse_gradient=1)
            assert net("sdnn_forward", X0, B, XL, None)[0] == 0
            rc, log = net("sdnn_backward", DL, None)
            lib.sdnn_destroy(net.h)
            assert rc == 0 and (not log[-1].startswith("k_bwd_long") or log[-1] == f"k_bwd_long {-(-n // 4)} 1 1"), log
            return log[-1].split()[0].split("<")[0]
        for n, k, B, want in [(1000, 64, 128, 0), (1000, 64, 129, 1), (1000, 64, 256, 1), (1000, 63, 256, 0), (10449, 64, 256, 1), (10450, 64, 256, 0), (12000, 95, 256, 0), (12000, 96, 256, 1),
                              (12000, 64, 192, 1), (15625, 170, 256, 1), (15626, 170, 256, 0), (15626, 170, 225, 0), (15626, 170, 224, 1), (29017, 369, 224, 0), (29017, 370, 224, 1),
                              (29018, 400, 224, 0)]:
            assert kernel(n, (k,), B) == ("k_bwd_long" if want else "k_bwd_rows"), (n, k, B)
        assert [kernel(1000, (64,) * 999 + (c,), 200) for c in (64, 63)] == ["k_bwd_long", "k_bwd_rows"]
    """)


def test_workgroups_that_stay_in_the_forward_in_panels():
    """With the clamped ReLU and at least eight pieces for five places of an XCD a workgroup takes one piece after the other; else there is
    a workgroup for every piece.  The nets of tests/test_gpu_pan_forward.py take both."""
    routes.run("""
        from tests import pan_nets
        def pans(widths, lengths, batches, max_batch=800, **options):
            net = Net([(y.n_out, y.n_in, y.row_ptr, y.col_idx, y.values, y.bias) for y in pan_nets.layers(widths, lengths)], max_batch, **options)
            out = []
            for B in batches:
                rc, log = net("sdnn_forward", X0, B, XL, None)
                assert rc == 0
                out.append([l.split("<")[1].replace(">", "").replace(",", "").split()[:3] for l in log if l.startswith("k_fwd_pan<")])
            return out
        n = (40000,) * 4                               # three ranges; 256 samples: 16 pairs for an XCD
        got = pans(n, (32,), (129, 256, 272, 273, 341))
        assert got == [[["0", "false", "216"]] * 3, [["0", "false", "384"]] * 3, [["0", "false", "408"]] * 3, [["0", "true", "256"]] * 3, [["0", "true", "256"]] * 3], got
        assert pans(n, (32,), (341,), activation=1) == [[["1", "false", "528"]] * 3]
        widths, b, lengths = pan_nets.NETS[0]
        assert [p[1] for p in pans(widths, lengths, (b,), b)[0]] == ["true"] * 3
    """)


def test_gradient_in_csr_order():
    """Large layers in two passes: not where the columns of short rows lie close together, nor with two partial gradients."""
    routes.run("""
        def passes(n, k, B, columns, n_in=None):
            n_in = n_in or n
            rng = np.random.default_rng(n)
            step = n_in // k
            ci = dict(random=lambda: np.arange(k) * step + rng.integers(0, step, (n, k)), diagonal=lambda: np.sort((np.arange(n)[:, None] + np.arange(k)) % n_in, axis=1),
                      window=lambda: np.sort((np.arange(n)[:, None] + 128 * np.arange(k)) % n_in, axis=1))[columns]()
            net = Net([(n, n_in, np.arange(0, n * k + 1, k, dtype=np.int32), ci.astype(np.int32).ravel(), np.ones(n * k, np.float32), None)], B, training=True, fuse_gradient=1)
            assert net("sdnn_forward", X0, B, XL, None)[0] == 0 and net("sdnn_backward", DL, None)[0] == 0
            rc, log = net("sdnn_weight_grad", 1, X0, None, None)
            lib.sdnn_destroy(net.h)
            names = [l.split()[0] for l in log]
            assert rc == 0 and names in (["k_sum_parts"], ["k_apply<true>", "k_spread_vals<true>"]), log
            return len(names)
        for n, k, B, columns, want in [(57343, 32, 64, "random", 1), (57344, 32, 64, "random", 2), (16384, 112, 64, "random", 2), (16384, 112, 128, "random", 1),
                                       (65536, 32, 64, "diagonal", 1), (65536, 32, 64, "window", 2), (40000, 63, 64, "diagonal", 1), (40000, 64, 64, "diagonal", 2)]:
            assert passes(n, k, B, columns) == want, (n, k, B, columns)
    """)


def test_long_forward_by_the_net():
    """Operands of up to 8192 neurons, 128 entries per row in the mean of every layer, 150000 per layer in the mean of all, made for more than
    64 samples; not for inference or where the caller asks for other layouts.  No copies, no room for them."""
    routes.run("""
        def longs(layers, max_batch=65, **options):
            options = {"training": True, **options}
            net, off = Net(layers, max_batch, **options), Net(layers, max_batch, **{**options, "lds_forward": -1})
            rc, log = net("sdnn_forward", X0, max_batch, XL, None)
            n = sum(l.startswith("k_fwd_long<") for l in log)
            assert rc == 0 and n in (0, len(layers)) and (net.bytes > off.bytes) == (n > 0), log
            for h in (net.h, off.h):
                lib.sdnn_destroy(h)
            return n > 0
        one_less = (128,) * 1199 + (127,)
        for layers, want in [([layer(8192, 8192, (128,))], True), ([layer(8192, 8193, (128,))], False), ([layer(8193, 8192, (128,))], True),
                             ([layer(1200, 1200, (128,))], True), ([layer(1200, 1200, one_less)], False), ([layer(8192, 1200, (128,) * 8191 + (127,))], False),
                             ([layer(1171, 1200, (128,))], False), ([layer(1172, 1200, (128,))], True),
                             ([layer(1200, 1200, (128,)), layer(1144, 1200, (128,))], True), ([layer(1200, 1200, (128,)), layer(1143, 1200, (128,))], False),
                             ([layer(2000, 2000, (400,)), layer(2000, 2000, (127,))], False), ([layer(2000, 2000, (0, 1, 500)), layer(10, 2000, (128,))], True)]:
            assert longs(layers) == want, [(l[0], l[1], len(l[3])) for l in layers]
        net = [layer(2000, 2000, (200,))]
        assert longs(net, 64) is False and longs(net, 300) and longs(net, fuse_gradient=1) and longs(net, fuse_gradient=-1) and longs(net, lds_forward=1)
        for options in (dict(training=False, lds_forward=-1), dict(panel_cols=512), dict(reorder_rows=1)):
            assert not longs(net, **options), options
    """)


def test_copies_for_the_long_forward_follow_when_they_are_read():
    """After a step whose batch reads them, at once; else before the next pass that does.  In a graph, and once a graph reads
    them, always.  Replaced values of a layer likewise, that layer alone."""
    routes.run("""
        def net():
            return Net([layer(2000, 2000, (200,))] * 3, 256, training=True)
        def fills(net, B, capture=()):
            out = []
            for k, (name, args) in enumerate([("sdnn_forward", (X0, B, XL, None)), ("sdnn_backward", (DL, None)), ("sdnn_sgd_step", (C.c_float(0.1), None))]):
                stub.stub_capture(k in capture)
                rc, log = net(name, *args)
                assert rc == 0
                lines = [l for l in log if l.startswith("k_long_fill")]
                assert lines in ([], ["k_long_fill<false> 32 16 3"]) and (not lines or k == 2 or [l.split("<")[0] for l in log[-4:]] == ["k_long_fill"] + ["k_fwd_long"] * 3 or
                                                                          log[-1].startswith("memcpy") or log[-1].startswith("k_copy")), log
                out.append(len(lines))
            stub.stub_capture(0)
            return out
        a = net()
        assert [fills(a, B) for B in (65, 64, 1, 256, 256, 8, 64, 65)] == [[0, 0, 1], [0, 0, 0], [0, 0, 0], [1, 0, 1], [0, 0, 1], [0, 0, 0], [0, 0, 0], [1, 0, 1]]
        b = net()                                      # a captured step of few samples: its replays keep the copies current, a later pass need not
        assert [fills(b, 64, (0, 1, 2)), fills(b, 256)] == [[0, 0, 1], [0, 0, 1]]
        c = net()                                      # a graph reads copies that are behind
        assert [fills(c, 64), fills(c, 65, (0, 1)), fills(c, 64), fills(c, 65), fills(c, 64)] == [[0, 0, 0], [1, 0, 1], [0, 0, 1], [1, 0, 1], [0, 0, 1]]
        def replaced(net, layers, capture=0):
            stub.stub_capture(capture)
            out = []
            for k, values in layers:
                rc, log = net("sdnn_set_weights", k, X0 if values else None, XL, None)
                assert rc == 0
                out += [l for l in log if l.startswith("k_long_fill")]
            stub.stub_capture(0)
            rc, log = net("sdnn_forward", X0, 65, XL, None)
            assert rc == 0
            return out, [l for l in log if l.startswith("k_long_fill")]
        one, two, three = (f"k_long_fill<false> 32 16 {n}" for n in (1, 2, 3))
        assert replaced(a, [(2, 1)]) == ([], [one]) and replaced(a, [(2, 0)]) == ([], []) and replaced(a, [(3, 1), (2, 1)]) == ([], [two])
        assert replaced(a, [(1, 1), (3, 1)]) == ([], [one, one]) and replaced(a, [(1, 1), (2, 1), (3, 1)]) == ([], [three]) and replaced(a, []) == ([], [])
        assert replaced(a, [(2, 1)], 1) == ([one], []) # captured: its replays are not seen
        assert replaced(c, [(2, 1), (1, 1)]) == ([one, one], []) # a graph reads the copies
    """)
