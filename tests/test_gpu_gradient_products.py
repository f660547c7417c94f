"""GPU parity of the loss's gradients (section 2.4) at the edges of the products that read their operands as they are: rows of a
contraction that end inside a slab of 64 and columns that end inside a tile of 256 or a 16-byte piece, one sequence and several, a
contraction over the vocabulary that is cut into parts; products of many sequences in one launch, cut too; dZ of up to 192 rows on the
streaming kernel with tiles of 256 columns.  Bars and oracle as in test_gpu_nll_backward.py."""
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
    # a product per sequence, cut along K: the hyper part of dH over 32 slabs (its residual is its output) ...
    (3, 300, 300, 64, 3, 2048, "mean", True),                # 6 tiles, over all workgroups
    (64, 40, 300, 64, 3, 2048, "mean", True),                # 64 tiles, 8 an XCD
    (272, 20, 300, 64, 3, 2000, "mean", False),              # 34 an XCD: a whole round and two tiles
    # ... and dW_hyper over the rows of a sequence
    (2, 2100, 300, 64, 3, 300, "mean", True),                # 4 tiles, over all workgroups
    (32, 2000, 200, 64, 3, 500, "mean", True),               # 64 tiles, 8 an XCD; a last slab of 16 rows
    # up to 64, 128 and 192 rows, more than 128 tiles of 256 columns, vocabularies and codebooks that end inside one
    (1, 50, 33000, 64, 3, 300, "mean", True),
    (2, 25, 32833, 128, 4, 257, "weighted", True),
    (1, 100, 33300, 64, 3, 513, "mean", True),
    (2, 50, 32769, 192, 3, 100, "mean", False),
    (1, 190, 32900, 64, 3, 40, "mean", True),
    (2, 95, 33333, 128, 3, 320, "mean", True),
    (9, 20, 33000, 64, 3, 65, "mean", True),
    # more sequences than one launch takes the hyper part of (2048)
    (2100, 66, 200, 64, 3, 30, "mean", True),
    (300, 70, 300, 64, 3, 300, "mean", True),
])
def test_gradients(B, N, V, d, M, cap, pool, use_grad):
    check(B, N, V, d, M, cap, pool, use_grad, 0)
