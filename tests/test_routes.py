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
