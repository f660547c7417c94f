"""The tile kernel's workgroup mapping for row counts behind whole blocks of 16 row tiles: every tile is computed once,
so the automatic mapping leaves what a mapping of one block shape over everything leaves, bit for bit
(that one is compared with the oracle elsewhere).  Joint logits: section 2.3, steps 7-9."""
import numpy as np
import pytest

from paper_2506_01084_amd import workloads as wl

from helpers import gpu_encode, torch_storage

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("row_tiles", [16, 17, 20, 23, 24, 29, 30, 31])
def test_pieces_behind_the_whole_blocks(row_tiles):
    import torch

    from paper_2506_01084_amd import api

    B, V, d, M, cap, N = 2, 9300, 64, 3, 300, 900
    rows_per_seq = row_tiles * 128 - 3
    cfg = dict(name="map", B=B, N=N, V=V, d=d, dtype="bf16", M=M, cap=cap, zipf_s=1.2, copy_frac=0.4, span=(2, 7),
               mode="motif", pool="mean", seed=9700)
    print(f"[case] {row_tiles} row tiles", flush=True)
    ctx = api.Context(B=B, V=V, M=M, cap=cap, d=d, dtype="bf16", pool="mean")
    gpu_encode(ctx, wl.make_tokens(cfg), np.full(B, N, dtype=np.int32))
    d_E = torch_storage(wl.make_embeddings(cfg), "bf16")
    d_W = torch.empty((B, cap, d), dtype=torch.bfloat16, device="cuda")
    ctx.hyper_embed(d_E, d_W)
    rows = B * rows_per_seq
    d_H = torch_storage(wl.make_hidden(cfg, rows), "bf16")
    got = []
    for mapping in (0, 4 | 8 << 8 | 4 << 16 | 2 << 24):
        ctx.set_option(api.OPT_LOGITS_MAP, mapping)
        am = torch.full((rows,), -5, dtype=torch.int32, device="cuda")
        mx = torch.full((rows,), 777.0, device="cuda")
        lse = torch.full((rows,), 777.0, device="cuda")
        ctx.extended_logits(d_H, rows_per_seq, d_E, d_W, am, mx, lse, None)
        torch.cuda.synchronize()
        got.append([x.cpu().numpy() for x in (am, mx, lse)])
        # the parts of the next call start from other values
        ctx.extended_logits(torch.zeros_like(d_H), rows_per_seq, d_E, d_W, am, mx, lse, None)
    for x, y in zip(*got):
        assert np.array_equal(x, y)
    ctx.close()


@pytest.mark.parametrize("row_tiles,V", [
    (2, 17921),         # 71 weight tiles, walked in blocks along the vocabulary; the last with one column
    (5, 9300),          # five row tiles: an odd short side, dealt out whole
    (6, 8192),          # an even one, two ways
    (33, 300),          # more row tiles than weight tiles: blocks along the rows, one behind whole blocks of 32
    (9, 513),           # three weight tiles under nine row tiles
])
def test_lists_hold_every_tile_once(row_tiles, V):
    """The automatic order along either side against single row tiles dealt out eight ways: the same bits."""
    import torch

    from paper_2506_01084_amd import api

    rows, d = row_tiles * 256 - 5, 64
    print(f"[case] {row_tiles} row tiles x {V} columns", flush=True)
    ctx = api.Context(B=1, V=V, M=3, cap=0, d=d, dtype="bf16", pool="mean")
    ctx.reset()
    gen = torch.Generator(device="cuda").manual_seed(V)
    W, H = (torch.randn((n, d), generator=gen, device="cuda").bfloat16() for n in (V, rows))
    none = torch.zeros((1, 0, d), dtype=torch.bfloat16, device="cuda")
    got = []
    for mapping in (0, 1 | 1 << 8 | 8 << 16 | 1 << 24):
        ctx.set_option(api.OPT_LOGITS_MAP, mapping)
        am = torch.full((rows,), -5, dtype=torch.int32, device="cuda")
        mx, lse = torch.full((rows,), 777.0, device="cuda"), torch.full((rows,), 777.0, device="cuda")
        ctx.extended_logits(H, rows, W, none, am, mx, lse)
        torch.cuda.synchronize()
        got.append((am, mx, lse))
        # the parts of the next call start from other values
        ctx.extended_logits(torch.zeros_like(H), rows, W, none, am.clone(), mx.clone(), lse.clone())
    for x, y in zip(*got):
        assert torch.equal(x, y)
    want = (H.float() @ W.float().t()).max(1).values          # 64 products of bf16 values in fp32: 1e-5 of the size
    assert torch.allclose(got[0][1], want, rtol=1e-5, atol=1e-4)
    ctx.close()
