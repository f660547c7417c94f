"""GPU parity of hyper_embed at every entry length (one instance of the row kernel each) and at row lengths about the
chunks it requests together: section 2.2.  Bound, relative to sum_j a_j |E[t_j]|: 8 fp32 additions (1e-6), or one ulp
of the storage type, 2^-7 for bf16: a sixth or a seventh of a sum of bf16 values often lies half way between two of
them, where a quotient (here) and a product with a rounded 1/L (the oracle) go to different sides."""
import numpy as np
import pytest

import oracle
from paper_2506_01084_amd import workloads as wl

from helpers import gpu_encode, hyper_embed_bound, oracle_encode_batch, storage_to_host, torch_storage

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pool", ["mean", "weighted"])
@pytest.mark.parametrize("dtype,d,cap", [("bf16", 8, 600), ("bf16", 520, 600), ("bf16", 2056, 600), ("f32", 4, 600), ("f32", 260, 600),
                                         ("f32", 1028, 600),
                                         ("bf16", 2056, 17000), ("f32", 1028, 17000)])   # over 128 MB: past the caches
def test_every_length(dtype, d, cap, pool):
    import torch

    from paper_2506_01084_amd import api

    B, V, M, N = 2, 3, 8, 4000                      # three tokens: entries grow to M quickly
    cfg = dict(name="lengths", B=B, N=N, V=V, d=d, dtype=dtype, M=M, cap=cap, zipf_s=1.5, copy_frac=0.4, span=(4, 12),
               mode="motif", pool=pool, seed=9900 + d)
    print(f"[case] {dtype} d={d} cap={cap} {pool}", flush=True)
    tokens = wl.make_tokens(cfg)
    E = wl.make_embeddings(cfg)
    w = wl.make_pool_weights(cfg)
    ctx = api.Context(B=B, V=V, M=M, cap=cap, d=d, dtype=dtype, pool=pool, w=w.tolist())
    gpu_encode(ctx, tokens, np.full(B, N, dtype=np.int32))
    ref = oracle_encode_batch(tokens, np.full(B, N), V, M, cap)
    assert {len(e) for _, entries, *_ in ref for e in entries} == set(range(2, M + 1))
    d_W = torch.full((B, cap, d), 3.0, dtype=ctx.torch_dtype, device="cuda")
    ctx.hyper_embed(torch_storage(E, dtype), d_W)
    torch.cuda.synchronize()
    got = storage_to_host(d_W, dtype)
    for b in range(B):
        entries = ref[b][1]
        want = oracle.to_f64(oracle.hyper_embed(E, dtype, entries, cap, pool, w), dtype)
        bound = hyper_embed_bound(E, dtype, entries, pool, w, cap)
        err = np.abs(oracle.to_f64(got[b], dtype) - want)
        assert (err <= (1e-6 if dtype == "f32" else 2.0 ** -7) * bound + 1e-30).all()
        assert (err[len(entries):] == 0).all()
    ctx.close()


def test_infinite_embedding_stays_infinite():
    """(the quotient of the mean is a product and a correction: an infinite sum must not become NaN)"""
    import torch

    from paper_2506_01084_amd import api

    V, d, M, cap = 4, 64, 3, 16
    ctx = api.Context(B=1, V=V, M=M, cap=cap, d=d, dtype="f32", pool="mean")
    codes, n_codes, status = gpu_encode(ctx, np.array([[0, 1, 2, 0, 1, 2, 3, 0, 1, 2]], dtype=np.int32), None)
    E = torch.ones((V, d), device="cuda")
    E[2] = float("inf")
    d_W = torch.zeros((1, cap, d), device="cuda")
    ctx.hyper_embed(E, d_W)
    entries, lengths, sizes = ctx.codebook()
    n = int(sizes[0])
    has = (entries[0, :n] == 2).any(1)
    assert lengths[0, :n].max() == 3
    assert torch.isinf(d_W[0, :n][has]).all() and (d_W[0, :n][~has] == 1).all()
    ctx.close()
