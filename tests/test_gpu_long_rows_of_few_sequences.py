"""GPU parity of extended_logits where up to 192 hidden rows belong to one or two sequences (section 2.3, steps 7-9; a chunk of a prompt):
the streaming kernel takes the hyper part along, tile by tile against its sequence's rows.  Both tile widths, codebooks that end in every
tile and at an edge, rows that fill each build; every row against the oracle as in test_gpu_logits_mid.py."""
import pytest

from test_gpu_logits_mid import test_streaming_kernel_every_row_ragged as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,rows_per_seq,V,d,M,cap,pool", [
    (1, 65, 400, 128, 3, 128, "mean"),           # tiles of 128 columns; one, full
    (1, 128, 700, 320, 3, 400, "mean"),          # four hyper tiles, every row of the 128-row build
    (2, 66, 513, 192, 4, 257, "weighted"),       # 132 rows in the 192-row build
    (2, 96, 300, 576, 3, 129, "mean"),           # 192 rows
    (1, 192, 33000, 256, 3, 600, "mean"),        # tiles of 256 columns
    (2, 70, 33300, 448, 3, 256, "mean"),
])
def test_every_row(B, rows_per_seq, V, d, M, cap, pool):
    check(B, rows_per_seq, V, d, M, cap, pool)
