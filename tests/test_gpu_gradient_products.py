"""GPU parity of the loss's gradients (section 2.4) at the edges of the products that read their operands as they are: rows of a
contraction that end inside a slab of 64 and columns that end inside a tile of 256 or a 16-byte piece, one sequence and several, a
contraction over the vocabulary that is cut into parts.  Bars and oracle as in test_gpu_nll_backward.py."""
import pytest

from test_gpu_nll_backward import test_gradients_match_oracle as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,N,V,d,M,cap,pool,use_grad", [
    (1, 9, 256, 64, 3, 1, "mean", True),
    (2, 63, 257, 64, 3, 63, "mean", True),
    (3, 64, 512, 256, 3, 256, "mean", False),
    (2, 65, 511, 320, 3, 65, "mean", True),
    (4, 257, 775, 448, 4, 129, "weighted", True),
    (2, 40, 5003, 128, 3, 30, "mean", True),                 # 79 slabs over the vocabulary, one row tile
    (1, 2100, 600, 64, 3, 300, "mean", True),                # 33 slabs over the rows
    # more sequences than one launch takes the hyper part of (2048)
    (2100, 66, 200, 64, 3, 30, "mean", True),
    (300, 70, 300, 64, 3, 300, "mean", True),
])
def test_gradients(B, N, V, d, M, cap, pool, use_grad):
    check(B, N, V, d, M, cap, pool, use_grad, 0)
