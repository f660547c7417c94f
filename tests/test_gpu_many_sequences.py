"""What a hidden row costs in extended_logits must not depend on how many sequences the rows belong to: the hyper part's items are found
in a time that does not grow with the sequences.  The same rows and entries in many sequences of 66 rows and in a few long ones.  (Rows of 66 fill a
quarter of a hyper tile, hence the room: 1.6 times the time is what that takes; with the items counted out from the first sequence on, it was 7.5.)"""
import pytest

pytestmark = pytest.mark.gpu


def _time(B, rows_per_seq, V, d, cap):
    import torch
    from paper_2506_01084_amd import api

    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    ctx = api.Context(B=B, V=V, M=3, cap=cap, d=d, dtype="bf16")
    i32 = lambda *s: torch.empty(s, dtype=torch.int32, device="cuda")
    tokens = torch.randint(0, 24, (B, 3 * cap), generator=gen, device="cuda").to(torch.int32)
    ctx.lzw_encode(tokens, None, i32(B, 3 * cap), i32(B), i32(B), api.RESET)
    rand = lambda *s: (torch.randn(s, generator=gen, device="cuda") * 0.02).bfloat16()
    rows = B * rows_per_seq
    E, W, H = rand(V, d), rand(B, cap, d), rand(rows, d)
    am, mx, lse = i32(rows), torch.empty(rows, device="cuda"), torch.empty(rows, device="cuda")
    times = []
    for _ in range(12):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        ctx.extended_logits(H, rows_per_seq, E, W, am, mx, lse)
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b))
    assert (ctx.codebook()[2] == cap).all()
    ctx.close()
    return min(times)


def test_time_does_not_grow_with_the_sequences():
    many, few = _time(2000, 66, 1024, 512, 300), _time(8, 16500, 1024, 512, 300)
    print(f"2000 x 66 rows {many * 1e3:.0f} us, 8 x 16500 rows {few * 1e3:.0f} us", flush=True)
    assert many < 2.5 * few
