"""GPU parity of the per-sequence part of extended_logits for calls with a few hidden rows per sequence at every size
its units take (64, 128 or 256 rows of W_hyper, chosen by how many there are): section 2.3, steps 7-9.

Small widths, so that the oracle can take every row; codebooks that end inside the first unit, at a unit's edge
and inside the last one; W_hyper rows behind the codebook hold values that would win every maximum."""
import numpy as np
import pytest

import oracle
from paper_2506_01084_amd import workloads as wl

from helpers import check_logits_rows, gpu_encode, oracle_encode_batch, torch_storage

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows_per_seq", [2, 5, 17])
@pytest.mark.parametrize("B,cap,unit", [(3, 257, 64), (20, 1500, 128), (33, 1500, 256), (130, 300, 256), (1, 64, 64),
                                        (130, 4200, 256)])   # more than 128 MB of weights: streamed past the caches
def test_units_of_every_size(B, cap, unit, rows_per_seq):
    import torch

    from paper_2506_01084_amd import api

    V, d, M, N = 300, 128, 3, 1600
    cfg = dict(name="units", B=B, N=N, V=V, d=d, dtype="bf16", M=M, cap=cap, zipf_s=1.2, copy_frac=0.4, span=(2, 7),
               mode="motif", pool="mean", seed=9300 + B)
    print(f"[case] units of {unit} rows: B={B} cap={cap} rows/seq={rows_per_seq}", flush=True)
    tokens = wl.make_tokens(cfg)
    lens = np.full(B, N, dtype=np.int32)
    if B > 2:
        lens[1], lens[2] = 0, 66         # an empty codebook and one that ends about a unit's edge
    E = wl.make_embeddings(cfg)
    rows = B * rows_per_seq
    H = wl.make_hidden(cfg, rows)
    ctx = api.Context(B=B, V=V, M=M, cap=cap, d=d, dtype="bf16", pool="mean")
    gpu_encode(ctx, tokens, lens)
    ref = oracle_encode_batch(tokens, lens, V, M, cap)
    d_E = torch_storage(E, "bf16")
    d_W = torch.empty((B, cap, d), dtype=torch.bfloat16, device="cuda")
    ctx.hyper_embed(d_E, d_W)
    for b in range(B):
        d_W[b, len(ref[b][1]):] = 900.0
    am = torch.full((rows,), -5, dtype=torch.int32, device="cuda")
    mx = torch.full((rows,), 777.0, device="cuda")
    lse = torch.full((rows,), 777.0, device="cuda")
    before = ctx.read_launches()["decode"]
    ctx.extended_logits(torch_storage(H, "bf16"), rows_per_seq, d_E, d_W, am, mx, lse, None)
    torch.cuda.synchronize()
    assert ctx.read_launches()["decode"] == before + 1
    am, mx, lse = am.cpu().numpy(), mx.cpu().numpy(), lse.cpu().numpy()
    for b in range(B):
        Wr = oracle.hyper_embed(E, "bf16", ref[b][1], cap, "mean")
        sl = slice(b * rows_per_seq, (b + 1) * rows_per_seq)
        check_logits_rows(oracle.extended_logits(H[sl], E, Wr, len(ref[b][1]), "bf16"), am[sl], mx[sl], lse[sl], None)
    ctx.close()
