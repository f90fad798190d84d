"""The network's products in the forms that batches of 17 to 65 rows, deep or wide
layers and long batches take, each checked as the edges of the products are."""
import pytest

from tests.test_gpu_mlp import test_product_edges as check
from tests.test_gpu_mlp import qg  # noqa: F401  (its fixture)

pytestmark = pytest.mark.gpu

# tiles of 32 rows, ragged, over slices (d_in 1100) and, transposed, over slices
# (d_out 300); of 32 rows in one slice with the loss (d_out 17000) and transposed
# (4100 inputs, 300 deep); of 64 rows, ragged and with a second tile of one row, in
# one slice with the loss and over slices; weight gradients of more than 8 and 64
# chains of 32 rows, with and without a remainder
SHAPES = [(1100, 70, 1, 300, 17), (1300, 90, 2, 17000, 31), (40, 4100, 1, 300, 31),
          (1200, 64, 1, 11000, 33), (1200, 72, 1, 11000, 65), (33, 40, 1, 50, 600),
          (20, 17, 1, 30, 256), (20, 17, 1, 30, 257), (20, 17, 1, 30, 2049)]


@pytest.mark.parametrize("shape", SHAPES)
def test_product_forms(qg, shape):  # noqa: F811
    check(qg, shape)
