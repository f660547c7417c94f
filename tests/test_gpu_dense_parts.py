"""GPU parity of the learned hyper-encoder (section 2.2) where the device cuts the last round of a dense layer's tiles along K:
fewer rows than the codebook has room for, one and several row tiles, widths that end inside a tile, a tail behind whole
rounds, contractions short of what a cut is worth.  Bars and oracle as in test_gpu_encoder.py and test_gpu_encoder_backward.py."""
import pytest

from test_gpu_encoder import test_hyper_encode_matches_oracle_every_entry as check
from test_gpu_encoder_backward import test_hyper_encode_backward_matches_oracle as check_backward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,N,V,d,M,cap,n_layers,n_heads,d_ff,attn_only,with_pos", [
    (1, 60, 300, 2048, 3, 400, 2, 16, 4096, False, True),      # under 128 rows of 1200 laid out: every layer in parts
    (1, 950, 900, 2176, 4, 700, 1, 17, 4352, False, True),     # 9 tiles wide, several row tiles: more parts over all CUs than in an XCD
    (2, 200, 500, 2112, 3, 300, 1, 33, 2112, False, True),     # 33 slabs, widths that end inside a tile, two row tiles
    (1, 300, 700, 1984, 3, 400, 1, 31, 2048, False, False),    # 31 slabs: only the second feed-forward layer may be cut
    (2, 900, 800, 2048, 2, 900, 1, 16, 0, True, True),         # q | k | v in more than one round, the tail in parts
])
def test_forward(B, N, V, d, M, cap, n_layers, n_heads, d_ff, attn_only, with_pos):
    check(B, N, V, d, M, cap, n_layers, n_heads, d_ff, attn_only, with_pos)


@pytest.mark.parametrize("B,N,V,d,M,cap,n_layers,n_heads,d_ff,attn_only,with_pos", [
    (1, 60, 300, 2048, 3, 400, 1, 16, 2112, False, True),      # gradients over a contraction of 2 slabs of 19 laid out
    (2, 700, 500, 512, 3, 800, 1, 8, 2048, False, True),       # few tiles, ~2000 rows: weight gradients in parts
])
def test_backward(B, N, V, d, M, cap, n_layers, n_heads, d_ff, attn_only, with_pos):
    check_backward(B, N, V, d, M, cap, n_layers, n_heads, d_ff, attn_only, with_pos)
