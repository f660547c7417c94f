"""GPU parity of the general tile kernel of extended_logits (fp32, and bf16 shapes the other kernels do not take), with
and without the full-logits output: section 2.3, steps 7-9.

Shapes sit at the edges of its tiles (128 rows x 64 columns, 128 columns in bf16 where those of 64 would be more than 768), of its blocks of eight row tiles, of a K slab (32 floats or 64
bf16) and of a vocabulary tile; both instances must leave the same picks and maxima."""
import numpy as np
import pytest

import oracle
from paper_2506_01084_amd import workloads as wl

from helpers import check_logits_rows, gpu_encode, oracle_encode_batch, torch_storage

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,rows_per_seq,V,d,cap", [
    ("f32", 1, 1153, 300, 36, 40),      # ten row tiles (a block of eight and one of two), the last with one row
    ("f32", 2, 129, 129, 4, 257),       # one chunk of K; a vocabulary tile with one column; three hyper tiles
    ("f32", 9, 3, 1000, 100, 130),      # few rows of many sequences; a K slab with one chunk
    ("f32", 3, 128, 2049, 64, 0),       # no hyper part; whole slabs
    ("bf16", 2, 200, 700, 72, 150),     # d no multiple of 64
    ("bf16", 1, 1, 50, 8, 5),           # a single row
    ("bf16", 2, 700, 4353, 200, 300),   # 759 tiles of 64 columns, 819 with the hyper part: 128 columns, one in the last tile; a part of a slab
    ("bf16", 1, 129, 24512, 64, 0),     # 766: the most (an even number) that stay at 64; a second row tile with one row
    ("bf16", 1, 129, 24577, 64, 0),     # 770; one slab; strips of one tile
    ("f32", 2, 130, 65, 68, 66),        # tiles with one and two columns behind a whole one; two K slabs and a chunk
    ("f32", 1, 300, 6400, 32, 64),      # one slab: nothing is fetched ahead; strips of one tile
])
def test_general_kernel(dtype, B, rows_per_seq, V, d, cap):
    import torch

    from paper_2506_01084_amd import api

    M, N = 3, 700
    cfg = dict(name="general", B=B, N=N, V=V, d=d, dtype=dtype, M=M, cap=cap, zipf_s=1.2, copy_frac=0.4, span=(2, 7),
               mode="motif", pool="mean", seed=9500 + V + d)
    print(f"[case] general kernel {dtype} B={B} rows/seq={rows_per_seq} V={V} d={d} cap={cap}", flush=True)
    tokens = wl.make_tokens(cfg)
    lens = np.full(B, N, dtype=np.int32)
    if B > 2:
        lens[1], lens[2] = 0, 9
    E = wl.make_embeddings(cfg)
    rows = B * rows_per_seq
    H = wl.make_hidden(cfg, rows)
    ctx = api.Context(B=B, V=V, M=M, cap=cap, d=d, dtype=dtype, pool="mean")
    gpu_encode(ctx, tokens, lens)
    ref = oracle_encode_batch(tokens, lens, V, M, cap)
    d_E, d_H = torch_storage(E, dtype), torch_storage(H, dtype)
    d_W = torch.zeros((B, cap, d), dtype=ctx.torch_dtype, device="cuda")
    if cap:
        ctx.hyper_embed(d_E, d_W)
        for b in range(B):
            d_W[b, len(ref[b][1]):] = 900.0        # rows that do not exist
    ctx.set_option(api.OPT_LOGITS_KERNEL, 1)
    ctx.set_option(api.OPT_DECODE_KERNEL, 1)
    got = []
    for full in (False, True):
        am = torch.full((rows,), -5, dtype=torch.int32, device="cuda")
        mx = torch.full((rows,), 777.0, device="cuda")
        lse = torch.full((rows,), 777.0, device="cuda")
        logits = torch.full((rows, V + cap), 777.0, device="cuda") if full else None
        before = ctx.read_launches()["general"]
        ctx.extended_logits(d_H, rows_per_seq, d_E, d_W, am, mx, lse, logits)
        torch.cuda.synchronize()
        assert ctx.read_launches()["general"] == before + 1
        got.append([x.cpu().numpy() for x in (am, mx, lse)] + [logits.cpu().numpy() if full else None])
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
    # (the same sums in the same order; a multiply and an add may be contracted in one instance alone: ulps)
    assert np.allclose(got[0][2], got[1][2], rtol=1e-6, atol=1e-6)
    am, mx, lse, logits = got[1]
    for b in range(B):
        Wr = oracle.hyper_embed(E, dtype, ref[b][1], cap, "mean") if cap else np.zeros((0, d), E.dtype)
        sl = slice(b * rows_per_seq, (b + 1) * rows_per_seq)
        want = oracle.extended_logits(H[sl], E, Wr, len(ref[b][1]), dtype)
        check_logits_rows(want, am[sl], mx[sl], lse[sl], logits[sl])
    ctx.close()


def test_strips_lengthen_where_the_static_array_would_not_hold_the_parts():
    """32768 rows x 32769 columns: strips of 4 x 64 columns would leave 129 parts a row, more than the static array's 2^22 in all
    (Z2Z_ELIMIT).  Through the allocation-free entry point, every row against float64 products (four terms each: 1e-6 of the largest
    logit); the allocating one cuts the same way: the same bits."""
    import torch

    from paper_2506_01084_amd import api

    rows, V, d = 32768, 32769, 4
    ctx = api.Context(B=1, V=V, M=3, cap=0, d=d, dtype="f32", pool="mean")
    ctx.reset()
    gen = torch.Generator(device="cuda").manual_seed(4)
    W, H = torch.randn((V, d), generator=gen, device="cuda"), torch.randn((rows, d), generator=gen, device="cuda")
    W[-1] = 9.0                                   # the column of a tile of its own decides many rows
    am = torch.full((rows,), -5, dtype=torch.int32, device="cuda")
    mx, lse = torch.zeros(rows, device="cuda"), torch.zeros(rows, device="cuda")
    none = torch.zeros((1, 0, d), device="cuda")
    ctx.extended_logits_static(H, rows, W, none, am, mx, lse)
    grown = torch.full_like(am, -5), torch.zeros_like(mx), torch.zeros_like(lse)
    ctx.extended_logits(H, rows, W, none, *grown)
    torch.cuda.synchronize()
    for a, b in zip((am, mx, lse), grown):
        assert torch.equal(a, b)
    for r in range(0, rows, 4096):
        z = H[r:r + 4096].double() @ W.double().t()
        top = z.topk(2, dim=1)
        sl = slice(r, r + 4096)
        assert torch.allclose(mx[sl].double(), top.values[:, 0], rtol=1e-6, atol=1e-6)
        assert torch.allclose(lse[sl].double(), z.logsumexp(1), rtol=1e-5, atol=1e-5)
        clear = top.values[:, 0] - top.values[:, 1] > 1e-4
        assert torch.equal(am[sl][clear].long(), top.indices[:, 0][clear])
    ctx.close()
