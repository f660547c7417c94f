"""GPU parity of the learned hyper-encoder (section 2.2) where the device cuts the last round of a dense layer's tiles along K:
fewer rows than the codebook has room for, one and several row tiles, widths that end inside a tile, a tail behind whole
rounds, contractions short of what a cut is worth.  Bars and oracle as in test_gpu_encoder.py and test_gpu_encoder_backward.py."""
import numpy as np
import pytest

import oracle
from paper_2506_01084_amd import workloads as wl

from helpers import encoder_to_device, storage_to_host
from test_gpu_encoder import _compare, _setup, test_hyper_encode_matches_oracle_every_entry as check
from test_gpu_encoder_backward import test_hyper_encode_backward_matches_oracle as check_backward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,N,V,d,M,cap,n_layers,n_heads,d_ff,attn_only,with_pos", [
    (1, 60, 300, 2048, 3, 400, 2, 16, 4096, False, True),      # under 128 rows of 1200 laid out: every layer in parts
    (1, 950, 900, 2176, 4, 380, 1, 17, 4352, False, True),     # 9 tiles wide, several row tiles: more parts over all CUs than in an XCD
    (2, 200, 500, 2112, 3, 300, 1, 33, 2112, False, True),     # 33 slabs, widths that end inside a tile, two row tiles
    (1, 300, 700, 1984, 3, 400, 1, 31, 2048, False, False),    # 31 slabs: only the second feed-forward layer may be cut
    (8, 900, 800, 2048, 2, 900, 1, 16, 0, True, True),         # q | k | v: 24 x 14 tiles, a whole round and a tail in parts
])
def test_forward(B, N, V, d, M, cap, n_layers, n_heads, d_ff, attn_only, with_pos):
    check(B, N, V, d, M, cap, n_layers, n_heads, d_ff, attn_only, with_pos)


@pytest.mark.parametrize("B,N,V,d,M,cap,n_layers,n_heads,d_ff,attn_only,with_pos", [
    (1, 60, 300, 2048, 3, 400, 1, 16, 2112, False, True),      # gradients over a contraction of 2 slabs of 19 laid out
    (2, 700, 500, 512, 3, 800, 1, 8, 2048, False, True),       # few tiles, ~2000 rows: weight gradients in parts
])
def test_backward(B, N, V, d, M, cap, n_layers, n_heads, d_ff, attn_only, with_pos):
    check_backward(B, N, V, d, M, cap, n_layers, n_heads, d_ff, attn_only, with_pos)


def test_entries_in_two_passes():
    """75 x 600 x 3 = 135000 slot rows, more than one pass takes (131072): passes of 582 and 18 entries per sequence.  The second
    feed-forward layer is cut in both: about 73000 rows, the 35 or 36 tiles of an XCD less a whole round of 32; about 1500, 7 tiles in all."""
    import torch

    B, N, V, d, M, cap = 75, 1500, 3000, 64, 3, 600
    cfg = wl.scaled(wl.CONFIGS["c2"], B=B, N=N, V=V, d=d, M=M, cap=cap, zipf_s=1.2, seed=78)
    print("[case] hyper_encode in two passes", flush=True)
    lens = wl.make_lens(cfg, ragged=True)
    ctx, ref, E, d_E = _setup(cfg, lens)
    enc = wl.make_encoder(cfg, n_layers=1, n_heads=2, d_ff=2048)
    d_W = torch.full((B, cap, d), 3.0, dtype=torch.bfloat16, device="cuda")
    ctx.hyper_encode(d_E, encoder_to_device(enc, "bf16"), d_W)
    torch.cuda.synchronize()
    W = storage_to_host(d_W, "bf16")
    longest = int(np.argmax([len(r[1]) for r in ref]))
    assert len(ref[longest][1]) > 582, "the case must reach the second pass"
    rows = [sum(len(e) for r in ref for e in part(r[1])) for part in (lambda e: e[:582], lambda e: e[582:])]
    assert 8 <= (rows[0] + 255) // 256 - 256 <= 128 and 2 <= (rows[1] + 255) // 256 <= 128, rows
    for b in (0, longest, B - 1):
        entries = ref[b][1]
        want = oracle.hyper_encode(E, "bf16", entries, cap, enc, rounded=False)
        if entries:
            _compare(W[b, :len(entries)], want[:len(entries)], f"two passes, seq {b}")
        assert (W[b, len(entries):] == 0).all()
    ctx.close()
