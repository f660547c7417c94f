"""A hidden row of NaN: its log-sum-exp, or the log-probability of what is drawn for it, reads NaN on every kernel (softmax over
NaN), and the other rows read the bits they have without it.  Codebooks are empty unless a case says otherwise: one part that
reads NaN would do for the row."""
import pytest

pytestmark = pytest.mark.gpu


def _setup(B, rows_per_seq, V, d, cap, dtype, fill=False):
    import torch

    from paper_2506_01084_amd import api

    storage = torch.float32 if dtype == "f32" else torch.bfloat16
    ctx = api.Context(B=B, V=V, M=3, cap=cap, d=d, dtype=dtype, pool="mean")
    gen = torch.Generator(device="cuda").manual_seed(V + d)
    ctx.reset()
    if fill:
        tokens = torch.randint(0, V, (B, 100), generator=gen, device="cuda").to(torch.int32)
        codes, n, st = torch.empty_like(tokens), *(torch.empty(B, dtype=torch.int32, device="cuda") for _ in range(2))
        ctx.lzw_encode(tokens, None, codes, n, st, api.RESET)
    E, W, H = (torch.randn(shape, generator=gen, device="cuda").to(storage)
               for shape in ((V, d), (B, cap, d), (B * rows_per_seq, d)))
    return ctx, E, W, H


def _check(H, run):
    import torch

    row = H.shape[0] // 2
    want = run(H)
    bad = H.clone()
    bad[row] = float("nan")
    got = run(bad)
    assert torch.isnan(got[-1][row])
    others = torch.arange(H.shape[0], device="cuda") != row
    for w, g in zip(want, got):
        assert not torch.isnan(w).any()
        assert torch.equal(w[others], g[others])


@pytest.mark.parametrize("dtype,B,rows_per_seq,V,d,cap,fill", [
    ("bf16", 2, 1, 600, 128, 40, False),        # decode kernel
    ("bf16", 200, 1, 600, 128, 40, False),      # tile kernel
    ("bf16", 1, 300, 600, 64, 300, True),       # ... for both parts; a last tile that is partly there
    ("bf16", 2, 150, 5, 64, 3, True),           # ... and nothing but partial groups of columns
    ("bf16", 2, 20, 600, 64, 40, False),        # weight-streaming kernel
    ("bf16", 2, 20, 5, 64, 40, False),          # ... a partial group of columns
    ("f32", 2, 20, 600, 36, 40, False),         # general kernel
    ("f32", 2, 20, 3, 36, 40, True),            # ... partial groups of columns
    ("bf16", 2, 400, 9000, 72, 40, False),      # ... tiles of 128 columns
])
def test_log_sum_exp(dtype, B, rows_per_seq, V, d, cap, fill):
    import torch

    print(f"[case] {dtype} B={B} x {rows_per_seq} V={V} d={d} cap={cap}", flush=True)
    ctx, E, W, H = _setup(B, rows_per_seq, V, d, cap, dtype, fill)

    def run(h):
        am = torch.full((h.shape[0],), -5, dtype=torch.int32, device="cuda")
        mx, lse = torch.zeros(h.shape[0], device="cuda"), torch.zeros(h.shape[0], device="cuda")
        ctx.extended_logits(h, rows_per_seq, E, W, am, mx, lse)
        torch.cuda.synchronize()
        return am, mx, lse

    _check(H, run)
    ctx.close()


@pytest.mark.parametrize("B,V,d,top_k,top_p", [
    (2, 600, 128, 0, 1.0),          # decode kernel
    (5, 65281, 128, 0, 1.0),        # weight-streaming kernel, sums in levels; a last tile of one column
    (70, 600, 128, 0, 1.0),         # weight-streaming kernel
    (200, 600, 128, 0, 1.0),        # tile kernel
    (200, 3, 128, 0, 1.0),          # ... one partial group of columns
    (2, 600, 128, 50, 0.9),         # filtered: a short list, then the row's passes in the same launch
    (5, 65281, 128, 0, 0.9),        # ... the passes in launches of their own
])
def test_log_probability(B, V, d, top_k, top_p):
    import torch

    print(f"[case] draws of {B} sequences, V={V} d={d} top_k={top_k} top_p={top_p}", flush=True)
    ctx, E, W, H = _setup(B, 1, V, d, 40, "bf16")

    def run(h):
        token, lp = torch.full((B,), -5, dtype=torch.int32, device="cuda"), torch.zeros(B, device="cuda")
        ctx.extended_sample(h, 1, E, W, 0.8, 77, 5, token, lp, top_k=top_k, top_p=top_p)
        torch.cuda.synchronize()
        return token, lp

    _check(H, run)
    ctx.close()


@pytest.mark.parametrize("B,rows_per_seq,V,d,cap", [
    (1, 70, 600, 64, 40),           # weight-streaming kernel, both parts
    (4, 30, 33000, 64, 40),         # ... tiles of 256 columns, several sequences
    (2, 150, 600, 64, 40),          # tile kernel
])
@pytest.mark.parametrize("bits", [0x7FC00000, 0x7FFFFFFF, -1])
def test_gradient_of_a_loss_whose_weight_is_nan(B, rows_per_seq, V, d, cap, bits):
    """A row whose loss has a NaN, of any bits, for its weight has NaN for its gradient; the other rows read the bits they have without it."""
    import torch

    print(f"[case] gradient, B={B} x {rows_per_seq} V={V} d={d} cap={cap} NaN {bits & 0xFFFFFFFF:#x}", flush=True)
    ctx, E, W, H = _setup(B, rows_per_seq, V, d, cap, "bf16", fill=True)
    E, W = E * d ** -0.5, W * d ** -0.5
    rows = B * rows_per_seq
    targets = torch.arange(rows, device="cuda", dtype=torch.int32) % V
    nll, lse, weight = torch.zeros(rows, device="cuda"), torch.zeros(rows, device="cuda"), torch.ones(rows, device="cuda")
    ctx.extended_nll(H, rows_per_seq, E, W, targets, nll, lse)

    def run():
        dH, dE, dW = torch.zeros_like(H), torch.zeros_like(E), torch.zeros_like(W)
        ctx.extended_nll_backward(H, rows_per_seq, E, W, targets, lse, weight, dH, dE, dW)
        torch.cuda.synchronize()
        return dH, dE, dW

    want = run()
    assert not any(torch.isnan(x).any() for x in want)
    row = rows // 2
    weight.view(torch.int32)[row] = bits
    dH, dE, dW = run()
    others = torch.arange(rows, device="cuda") != row
    assert torch.isnan(dH[row]).all() and torch.equal(dH[others], want[0][others])
    assert torch.isnan(dE).all()
    ctx.close()
