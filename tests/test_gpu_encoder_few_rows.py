"""GPU parity of hyper_encode where the dense layers are split over K and what follows them adds up the parts: rows
of d that do not fill the row kernels' workgroups, attention-only layers, every slot count, the tile kernel's split,
and the plain kernels behind a last layer that is not split.  Section 2.2; bar and oracle as in test_gpu_encoder.py."""
import pytest

from test_gpu_encoder import test_hyper_encode_matches_oracle_every_entry as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,N,V,d,M,cap,n_layers,n_heads,d_ff,attn_only,with_pos", [
    (1, 200, 40, 576, 8, 15, 2, 9, 0, True, True),           # 120 rows at most, attention layers, up to 8 slots
    (3, 100, 200, 1088, 3, 13, 2, 17, 1152, False, False),   # 117 rows: widths that are no multiple of 256
    (2, 200, 300, 4096, 2, 9, 1, 32, 512, False, True),      # rows that fill the workgroups; 36 rows
    (1, 60, 300, 64, 3, 10, 2, 2, 64, False, True),          # one K slab: no layer is split
    (1, 60, 300, 2112, 3, 30, 3, 33, 4224, False, True),     # 90 rows laid out; weights past the caches
    (1, 200, 40, 192, 8, 16, 1, 3, 128, False, True),        # 128 rows laid out: three and two slabs
    (2, 500, 300, 1024, 5, 60, 2, 8, 0, True, False),        # 600 rows: the tile kernel's split, attention layers
])
def test_few_rows(B, N, V, d, M, cap, n_layers, n_heads, d_ff, attn_only, with_pos):
    check(B, N, V, d, M, cap, n_layers, n_heads, d_ff, attn_only, with_pos)
