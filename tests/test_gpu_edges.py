"""Kernels and dispatch branches at the sizes where they can go wrong (needs an MI355X): edges of tiles, remainders,
the smallest and largest of a range.  Same bars as the other parity tests: integers bit for bit, products under the
norm and element-wise bounds of tests/parity_util.py against the fp64 oracle."""
import pytest

from tests import test_gpu_ragged as ragged

pytestmark = pytest.mark.gpu


# tiles of 32 x 64, eight wavefronts that take chunks of 32 k in turn: one token, one row more than a tile, less than
# one chunk, one chunk per wavefront and a remainder, the largest rank
@pytest.mark.parametrize("b,d_out,d_in,r", [(1, 8, 8, 32), (33, 72, 264, 512), (257, 1000, 136, 160), (31, 136, 1000, 32)])
def test_ragged_adapter_products(b, d_out, d_in, r):
    ragged.test_every_call_on_a_ragged_layer(b, d_out, d_in, r)
