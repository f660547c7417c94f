"""GPU parity of decode steps of 5..64 sequences over a vocabulary of at least 65281 columns (256 tiles; with more
than 16 sequences only where there are more than 512 tiles, or the rounds of 256 tiles are 7/8 full, or hyper units would
open another): the base part on the weight-streaming kernel (sums in three levels), the hyper units alone, in units of
64..512 rows.  Section 2.3, steps 7-9.

Bound of the largest logit: fp32 sums of d products, 8 at most in one run of the accumulators: 1e-5 of its size."""
import numpy as np
import pytest

import oracle
from paper_2506_01084_amd import workloads as wl

from helpers import check_logits_rows, gpu_encode, oracle_encode_batch, torch_storage

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,V,d,cap,split", [
    (5, 65281, 128, 40, 1),       # two slabs: fewer than the ring's slots; one unit per sequence
    (9, 65290, 768, 700, 1),      # twelve slabs: the second level is flushed at the end alone
    (33, 65500, 1664, 100, 1),    # 26 slabs: the second level is flushed after 16 and at the end
    (64, 65281, 256, 520, 1),     # every row valid; nine units of 64 per sequence
    (4, 65281, 128, 40, 0),       # (four sequences stay on the dot-product units)
    (4, 65500, 1152, 40, 0),      # (... past the caches with more than 128 MB of weights)
    (40, 65000, 128, 40, 0),      # (254 tiles stay on the decode kernel)
    (16, 66000, 128, 40, 1),      # 258 tiles, half of the second round idle: up to 16 sequences
    (17, 66000, 128, 40, 0),
    (17, 114433, 128, 40, 1),     # 448 tiles of 512
    (17, 114432, 128, 40, 0),     # 447
    (17, 131073, 128, 40, 1),     # 513: a third round, nearly empty
    (32, 66000, 128, 4000, 1),    # 258 tiles and 256 hyper units
    (37, 28432, 128, 2000, 1),    # 112 tiles, 148 hyper units: above 256 in all
    (36, 28432, 128, 2000, 0),    # 256
    (37, 28416, 256, 2000, 0),    # 111 tiles
    (64, 49200, 128, 100, 1),     # 193 tiles and 64 units: 257
    (63, 49500, 128, 100, 0),     # 194 tiles, 63 units
    (9, 50000, 256, 3600, 1),     # 196 tiles, 72 units, the last of a sequence nearly empty
    (20, 32700, 384, 500, 1),     # 128 tiles, halved; 20 units: 148
    (40, 28500, 1664, 700, 1),    # 112 tiles, halved, 80 units: 192
    (41, 32768, 256, 700, 0),     # 128 tiles and 82 units: 210
    (8, 32769, 128, 40, 0),       # 129 tiles
])
def test_split_step(B, V, d, cap, split):
    import torch

    from paper_2506_01084_amd import api

    M, N = 3, 900
    cfg = dict(name="split", B=B, N=N, V=V, d=d, dtype="bf16", M=M, cap=cap, zipf_s=1.4, copy_frac=0.5, span=(2, 7),
               mode="motif", pool="mean", seed=9100 + B)
    print(f"[case] step of {B} sequences, V={V} d={d} cap={cap}", flush=True)
    tokens = wl.make_tokens(cfg)
    lens = np.full(B, N, dtype=np.int32)
    lens[1] = 0
    E, H = wl.make_embeddings(cfg), wl.make_hidden(cfg, B)
    ctx = api.Context(B=B, V=V, M=M, cap=cap, d=d, dtype="bf16", pool="mean")
    gpu_encode(ctx, tokens, lens)
    ref = oracle_encode_batch(tokens, lens, V, M, cap)
    d_E = torch_storage(E, "bf16")
    d_W = torch.empty((B, cap, d), dtype=torch.bfloat16, device="cuda")
    ctx.hyper_embed(d_E, d_W)
    for b in range(B):
        d_W[b, len(ref[b][1]):] = 900.0
    am = torch.full((B,), -5, dtype=torch.int32, device="cuda")
    mx = torch.full((B,), 777.0, device="cuda")
    lse = torch.full((B,), 777.0, device="cuda")
    before = ctx.read_launches()
    ctx.extended_logits(torch_storage(H, "bf16"), 1, d_E, d_W, am, mx, lse, None)
    torch.cuda.synchronize()
    after = ctx.read_launches()
    assert after["mid"] - before["mid"] == split
    am, mx, lse = am.cpu().numpy(), mx.cpu().numpy(), lse.cpu().numpy()
    for b in range(B):
        Wr = oracle.hyper_embed(E, "bf16", ref[b][1], cap, "mean")
        want = oracle.extended_logits(H[b:b + 1], E, Wr, len(ref[b][1]), "bf16")
        check_logits_rows(want, am[b:b + 1], mx[b:b + 1], lse[b:b + 1], None)
        assert abs(mx[b] - want["max"][0]) <= 1e-5 * abs(want["max"][0])
    ctx.close()


@pytest.mark.parametrize("B,V,d,cap,top_k,top_p", [
    (5, 65281, 128, 40, 0, 1.0),        # two slabs, fewer than the ring's slots; a last tile of one column
    (33, 65500, 1664, 100, 0, 1.0),     # weights past the caches; a second block of rows with one row
    (64, 65500, 384, 520, 0, 1.0),      # six slabs: half of the steps behind the loop
    (9, 65290, 768, 700, 50, 0.9),
    (32, 65281, 1152, 40, 50, 0.9),     # (one block of rows: the second is left out)
    (64, 65500, 256, 100, 0, 0.8),
    (17, 131073, 128, 40, 0, 1.0),      # 513 tiles
    (33, 131073, 128, 40, 50, 0.9),
    (20, 32700, 384, 500, 0, 1.0),      # tiles of 128 columns
    (33, 32768, 256, 2000, 50, 0.9),    # ... whose parts the filters' kernels read
    (64, 33000, 1024, 700, 0, 1.0),     # weights past the caches by those of the codebooks
    (32, 50000, 1152, 1000, 50, 0.9),   # 196 tiles, 64 units
    (43, 50000, 1024, 1100, 50, 0.9),   # ... 129, rows of 2 KB
])
def test_split_draws_match_one_launch(B, V, d, cap, top_k, top_p):
    """Draws of a split step against those of the decode kernel in one launch (both oracle-tested on smaller vocabularies):
    the same numbers perturb logits that differ by fp32 rounding, at most 1e-5 of a size below 10: picks agree unless two
    perturbed values are that close, and log-probabilities to 1e-4."""
    import torch

    from paper_2506_01084_amd import api

    print(f"[case] draws of {B} sequences, V={V} d={d} cap={cap} top_k={top_k} top_p={top_p}", flush=True)
    ctx = api.Context(B=B, V=V, M=3, cap=cap, d=d, dtype="bf16", pool="mean")
    gen = torch.Generator(device="cuda").manual_seed(V + B)
    tokens = torch.randint(0, V, (B, 300), generator=gen, device="cuda").to(torch.int32)
    codes, n, st = torch.empty_like(tokens), *(torch.empty(B, dtype=torch.int32, device="cuda") for _ in range(2))
    ctx.lzw_encode(tokens, None, codes, n, st, api.RESET)
    E = (torch.randn((V, d), generator=gen, device="cuda") * d ** -0.5).bfloat16()
    W = (torch.randn((B, cap, d), generator=gen, device="cuda") * d ** -0.5).bfloat16()
    H = torch.randn((B, d), generator=gen, device="cuda").bfloat16()
    got = {}
    for kernel in (0, 4):               # automatic; not the streaming kernel
        ctx.set_option(api.OPT_LOGITS_KERNEL, kernel)
        token, lp = torch.full((B,), -5, dtype=torch.int32, device="cuda"), torch.full((B,), 777.0, device="cuda")
        before = ctx.read_launches()["mid"]
        ctx.extended_sample(H, 1, E, W, 0.8, 77, 5, token, lp, top_k=top_k, top_p=top_p)
        torch.cuda.synchronize()
        assert ctx.read_launches()["mid"] - before == (1 if kernel == 0 else 0)
        got[kernel] = token, lp
    same = got[0][0] == got[4][0]
    assert int((~same).sum()) <= 1
    assert torch.allclose(got[0][1][same], got[4][1][same], atol=1e-4, rtol=0)
    ctx.close()


def test_greedy_step_is_captured_behind_an_eager_draw():
    """(the draw's kernels leave fewer parts per row; every kind of step sizes the scratch for all of them)"""
    import torch

    from paper_2506_01084_amd import api

    B, V, d, cap = 6, 65281, 128, 300
    ctx = api.Context(B=B, V=V, M=3, cap=cap, d=d, dtype="bf16", pool="mean")
    ctx.reset()
    gen = torch.Generator(device="cuda").manual_seed(5)
    E = (torch.randn((V, d), generator=gen, device="cuda") * 0.1).bfloat16()
    W = torch.zeros((B, cap, d), dtype=torch.bfloat16, device="cuda")
    H = torch.randn((B, d), generator=gen, device="cuda").bfloat16()
    token = torch.zeros(B, dtype=torch.int32, device="cuda")
    am, mx, lse, lp = torch.zeros_like(token), *(torch.zeros(B, device="cuda") for _ in range(3))
    ctx.extended_sample(H, 1, E, W, 0.8, 1, 2, token, lp)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ctx.extended_logits(H, 1, E, W, am, mx, lse)
    want = (H.float() @ E.float().t()).max(1)
    for _ in range(3):
        am.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(am.long(), want.indices) and torch.allclose(mx, want.values, rtol=1e-4)
    ctx.close()


def test_sums_keep_the_decode_kernels_precision():
    """The largest logits of a step at d = 4096 against float64 products of the stored operands: the streaming kernel's sums
    in three levels leave 4.4e-8 to 5.2e-8 of their size (root mean square), one accumulator over all of K 2.7e-7 to
    3.3e-7.  The bound lies between the two, a factor of two from either."""
    import torch

    from paper_2506_01084_amd import api

    B, V, d, cap = 16, 65500, 4096, 16
    ctx = api.Context(B=B, V=V, M=3, cap=cap, d=d, dtype="bf16", pool="mean")
    ctx.reset()
    gen = torch.Generator(device="cuda").manual_seed(3)
    E = (torch.randn((V, d), generator=gen, device="cuda") * 0.02).bfloat16()
    W = torch.zeros((B, cap, d), dtype=torch.bfloat16, device="cuda")
    am, mx, lse = torch.zeros(B, dtype=torch.int32, device="cuda"), torch.zeros(B, device="cuda"), torch.zeros(B, device="cuda")
    err = []
    for _ in range(4):
        H = torch.randn((B, d), generator=gen, device="cuda").bfloat16()
        before = ctx.read_launches()["mid"]
        ctx.extended_logits(H, 1, E, W, am, mx, lse)
        torch.cuda.synchronize()
        assert ctx.read_launches()["mid"] == before + 1
        want = (H.double() * E[am.long()].double()).sum(1)
        err.append(((mx.double() - want) / want).cpu())
    rms = float(torch.cat(err).square().mean().sqrt())
    print(f"[case] largest logits of 64 rows: relative error {rms:.2e}", flush=True)
    assert rms <= 1.2e-7
    ctx.close()


@pytest.mark.parametrize("B,V,d,cap", [(32, 50000, 1024, 1000), (64, 50000, 256, 1000), (20, 32700, 384, 500)])
def test_filtered_steps_in_one_launch(B, V, d, cap):
    """Filtered steps that a draw splits and they do not: rows of up to 2 KB until the hyper units fill half of another round, and
    whatever fits one round."""
    import torch

    from paper_2506_01084_amd import api

    ctx = api.Context(B=B, V=V, M=3, cap=cap, d=d, dtype="bf16", pool="mean")
    ctx.reset()
    gen = torch.Generator(device="cuda").manual_seed(V + B)
    E = (torch.randn((V, d), generator=gen, device="cuda") * d ** -0.5).bfloat16()
    W = torch.zeros((B, cap, d), dtype=torch.bfloat16, device="cuda")
    H = torch.randn((B, d), generator=gen, device="cuda").bfloat16()
    token, lp = torch.full((B,), -5, dtype=torch.int32, device="cuda"), torch.full((B,), 777.0, device="cuda")
    for filters, split in ((dict(top_k=1), 0), (dict(), 1)):
        before = ctx.read_launches()["mid"]
        ctx.extended_sample(H, 1, E, W, 0.8, 77, 5, token, lp, **filters)
        torch.cuda.synchronize()
        assert ctx.read_launches()["mid"] - before == split
        if filters:                     # one column is kept: the largest logit, whose log-probability is 0
            assert torch.equal(token.long(), (H.float() @ E.float().t()).argmax(1)) and (lp == 0).all()
    ctx.close()
