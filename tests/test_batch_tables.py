"""The room a batch's tables take in the pool's front: a pool that was sized
for a number of channels and nodes goes on holding them."""
import pytest

from paper_2112_13930_amd._lib import lib


# bytes that pools have been sized with since the batch's tables were laid out
@pytest.mark.parametrize("channels,nodes,size", [(1, 1, 8960), (256, 1 << 24, 50757120),
                                                 (65535, 1 << 20, 110367744)])
def test_overhead_has_not_grown(channels, nodes, size):
    assert lib().lks_mhd_batch_overhead_bytes(channels, nodes) <= size
