"""GPU parity of filtered draws (top-k, nucleus) with the hyper part in units of every size (64 to 512 rows, by how many there are):
with one column kept the draw is the largest logit, wherever among the units it lies, and the short-list pass agrees with the passes over
the whole row.  Section 2.3, steps 7-9; codebooks that end in every unit, W_hyper rows behind them that would win."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,cap,unit", [
    (66, 130, 64),        # three units of 64, the last of two rows
    (66, 330, 64),        # 198 units of 128 would be too few
    (110, 500, 256),      # 110 units of 512
    (70, 600, 128),       # 140: those of 256 would be more than a round
    (110, 1000, 512),     # 220
    (70, 2100, 512),      # 350 units, roomy but enough of them
    (66, 64, 64),
])
def test_units_of_every_size(B, cap, unit):
    import torch

    from paper_2506_01084_amd import api

    V, d, N = 300, 256, 2300
    print(f"[case] filtered draws, units of {unit} rows: B={B} cap={cap}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(B + cap)
    ctx = api.Context(B=B, V=V, M=3, cap=cap, d=d, dtype="bf16", pool="mean")
    tokens = torch.randint(0, V, (B, N), generator=gen, device="cuda").to(torch.int32)
    lens = torch.randint(0, N + 1, (B,), generator=gen, device="cuda").to(torch.int32)
    lens[0], lens[1], lens[2] = N, 0, 66
    codes, n, st = torch.empty_like(tokens), *(torch.empty(B, dtype=torch.int32, device="cuda") for _ in range(2))
    ctx.lzw_encode(tokens, lens, codes, n, st, api.RESET)
    sizes = ctx.codebook()[2].long()
    E = (torch.randn((V, d), generator=gen, device="cuda") * d ** -0.5).bfloat16()
    W = (torch.randn((B, cap, d), generator=gen, device="cuda") * 1.5 * d ** -0.5).bfloat16()
    H = torch.randn((B, d), generator=gen, device="cuda").bfloat16()
    exists = torch.arange(cap, device="cuda") < sizes[:, None]
    hyper = torch.bmm(W.float(), H.float().unsqueeze(2).contiguous()).squeeze(2)
    z = torch.cat([H.float() @ E.float().t(), torch.where(exists, hyper, float("-inf"))], 1)
    W[~exists] = 900.0
    token, lp = torch.full((B,), -5, dtype=torch.int32, device="cuda"), torch.full((B,), 777.0, device="cuda")

    def draw(step, **filters):
        token.fill_(-5)
        ctx.extended_sample(H, 1, E, W, 0.8, 77, step, token, lp, **filters)
        torch.cuda.synchronize()
        return token.clone(), lp.clone()

    got, gl = draw(1, top_k=1)
    top = z.topk(2, 1)
    clear = top.values[:, 0] - top.values[:, 1] > 1e-4       # (fp32 sums of 256 products of size 1: 1e-6)
    assert torch.equal(got.long()[clear], top.indices[clear, 0]) and (gl == 0).all()
    assert int((got >= V).sum()) > B // 4                     # (draws among the units)
    for step, filters in ((2, dict(top_k=50)), (3, dict(top_k=40, top_p=0.9)), (4, dict(top_p=0.3))):
        ctx.set_option(api.OPT_SAMPLE_KERNEL, 0)
        a, la = draw(step, **filters)
        ctx.set_option(api.OPT_SAMPLE_KERNEL, 1)              # the passes over the whole row
        b, lb = draw(step, **filters)
        ctx.set_option(api.OPT_SAMPLE_KERNEL, 0)
        same = a == b
        assert int((~same).sum()) <= 1 and torch.allclose(la[same], lb[same], atol=1e-4, rtol=0)
    ctx.close()
