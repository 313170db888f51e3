"""The surrogate network's narrow layers against the oracle: every input count of
the first layer's own kernels, and products whose terms are less than one chunk of
32, or one chunk and a short or long rest, on both tile sizes."""
import pytest

import test_gpu_mlp_shapes as shapes

pytestmark = pytest.mark.gpu


# hidden widths 8 .. 16: one group of 16 terms; 20 .. 31: two; 40: a chunk and a
# group; 300: two workgroups along the first layer's outputs; rows of whole and of
# broken quads of four terms; 1275 outputs of 2000 or more samples: 64 x 64 tiles
@pytest.mark.parametrize("n_in, hidden, n_out, B", [
    (1, 16, 70, 100), (2, 20, 33, 65), (3, 28, 130, 200), (4, 12, 1275, 3000), (5, 24, 40, 50), (6, 31, 66, 95),
    (7, 300, 41, 530), (4, 40, 1275, 2000), (2, 8, 1275, 2100), (5, 22, 1275, 2000)])
def test_narrow_products_match_oracle(n_in, hidden, n_out, B):
    # the bounds of the other shapes: sums of at most 3000 terms
    shapes.test_products_match_oracle(n_in, hidden, n_out, B)
