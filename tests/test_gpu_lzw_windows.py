"""GPU parity of the window kernels of lzw_encode / lzw_decode (up to 1024 elements of a sequence at once, iterated until
they agree with the entries they make) at the sizes where a window can go wrong, against the oracle, bit for bit."""
import numpy as np
import pytest

import oracle
from helpers import assert_codebook_equal, gpu_decode, gpu_encode, oracle_encode_batch

pytestmark = pytest.mark.gpu


def _ctx(B, V, M, cap, kernel=0):
    from paper_2506_01084_amd import api

    ctx = api.Context(B=B, V=V, M=M, cap=cap, d=64, dtype="bf16")
    ctx.set_option(api.OPT_LZW_KERNEL, kernel)
    return ctx


def _round_trip(tokens, lens, V, M, cap, kernel=0):
    B, N = tokens.shape
    ref = oracle_encode_batch(tokens, lens, V, M, cap)
    ctx, ctx2 = _ctx(B, V, M, cap, kernel), _ctx(B, V, M, cap, kernel)
    codes, n_codes, status = gpu_encode(ctx, tokens, lens)
    assert (status == 0).all()
    for b, (rc, _, _) in enumerate(ref):
        assert codes[b, :n_codes[b]].tolist() == rc, f"codes of sequence {b}"
    assert_codebook_equal(ctx, [r[1] for r in ref], M, cap)
    toks, n_tok, st = gpu_decode(ctx2, codes, n_codes, out_stride=N)
    assert (st == 0).all() and (n_tok == lens).all()
    for b in range(B):
        assert (toks[b, :lens[b]] == tokens[b, :lens[b]]).all(), f"tokens of sequence {b}"
    assert_codebook_equal(ctx2, [r[1] for r in ref], M, cap)
    ctx.close()
    ctx2.close()


@pytest.mark.parametrize("M,cap", [(2, 90), (3, 5000), (4, 1500), (5, 700), (8, 3000)])
@pytest.mark.parametrize("N", [65, 511, 513, 1023, 1024, 1025, 2049, 3100])
def test_window_edges(N, M, cap):
    """Lengths around the windows of 64, 512 and 1024; streams that depend on the window's own entries everywhere (tiny
    alphabets, runs, periods) or rarely (Zipf); codebooks that fill inside a window, or never."""
    rng = np.random.default_rng(N * 16 + M)
    V = 60
    rows = [rng.integers(0, 2, N), rng.integers(0, 9, N), np.minimum(rng.zipf(1.3, N) - 1, V - 1), np.zeros(N, np.int64),
            np.tile(rng.integers(0, V, 7), N // 7 + 1)[:N], np.repeat(rng.integers(0, V, N // 11 + 1), 11)[:N]]
    tokens = np.stack(rows).astype(np.int32)
    lens = np.full(len(rows), N, dtype=np.int32)
    lens[1] = N - 1
    _round_trip(tokens, lens, V, M, cap)
    if N in (1024, 2049):
        for kernel in (2, 4):                                # table in memory; one wave, windows of 64
            _round_trip(tokens, lens, V, M, cap, kernel)


@pytest.mark.parametrize("B,cap", [(300, 500), (300, 4096)])
def test_more_sequences_than_compute_units(B, cap):
    """Several workgroups per CU: eight waves each, or four where the tables are larger."""
    rng = np.random.default_rng(B + cap)
    tokens = np.minimum(rng.zipf(1.2, (B, 700)) - 1, 199).astype(np.int32)
    lens = rng.integers(0, 701, B).astype(np.int32)
    lens[0] = 700
    _round_trip(tokens, lens, 200, 3, cap)


@pytest.mark.parametrize("B,N,cap", [(3, 300, 5000), (3, 300, 8192), (3, 300, 11208), (3, 300, 11209), (256, 600, 4957),
                                     (256, 600, 4965), (3, 700, 2478), (3, 700, 2479)])
def test_tables_beside_wide_round_sets(B, N, cap):
    """Tables of the sizes up to which LDS has room for them beside the encoder's sets of eight slots per position (one window
    of eight waves, or windows of sixteen), and beside any of its sets: a launch must not ask for more than is declared."""
    rng = np.random.default_rng(N + cap)
    tokens = np.minimum(rng.zipf(1.2, (B, N)) - 1, 199).astype(np.int32)
    _round_trip(tokens, np.full(B, N, np.int32), 200, 3, cap)


@pytest.mark.parametrize("B,M,cap", [(520, 3, 2048), (1100, 4, 1500), (800, 5, 3000), (1030, 8, 40), (2700, 3, 200)])
def test_several_workgroups_of_a_compute_unit(B, M, cap):
    """More than two sequences per CU: three or four workgroups on one, tables cut to what that leaves of the LDS, one round
    set for all iterations of a window, sequences taken longest first (lengths of 0, of all of a row, all alike, of every class),
    or as they come where there are too many of them for their length."""
    rng = np.random.default_rng(B + cap)
    N = {520: 2100, 1100: 700, 2700: 700}.get(B, 300)   # (in order of length from 640 tokens, 2048 codes on; 2700: as they come)
    tokens = np.where(rng.random((B, 1)) < 0.5, rng.integers(0, 4, (B, N)), np.minimum(rng.zipf(1.3, (B, N)) - 1, 99)).astype(np.int32)
    lens = rng.integers(0, N + 1, B).astype(np.int32)
    lens[rng.integers(0, B, 40)] = 0
    lens[:30] = N
    lens[100:200] = 150
    _round_trip(tokens, lens, 100, M, cap)


def test_largest_ids():
    """V + cap = 2^24: parents and tokens use all their bits in the table's slots and the round's keys."""
    rng = np.random.default_rng(7)
    cap = 1200
    V = (1 << 24) - cap
    tokens = (V - 1 - rng.integers(0, 5, (3, 1500))).astype(np.int32)
    _round_trip(tokens, np.full(3, 1500, np.int32), V, 6, cap)


def _random_codes(rng, V, M, cap, n, hot):
    """A code stream no greedy parse made: any code that is legal when its turn comes, with many repeated pairs."""
    s, codes = oracle.LZWStream(V, M, cap), []
    while len(codes) < n:
        C = len(s.entries)
        u = rng.random()
        k = int(rng.integers(0, hot)) if u < 0.5 or C == 0 else V + C if u < 0.53 else V + int(rng.integers(max(0, C - 40), C))
        _, st = s.decode_chunk([k]) if k < V + C else (None, 1)
        if k == V + C:                                       # the entry this code makes itself, where that is legal
            t = oracle.LZWStream(V, M, cap)
            if t.decode_chunk(codes + [k])[1] != 0:
                continue
            s.decode_chunk([k])
        codes.append(k)
    return codes


@pytest.mark.parametrize("M,cap", [(3, 5000), (5, 400), (4, 12000)])
def test_decode_of_arbitrary_codes(M, cap):
    """Windows whose codes repeat edges, meet edges of the table and name the window's own entries: cut where they
    must be; then a code that names nothing, and an output row that ends, at places in different windows."""
    from paper_2506_01084_amd import api

    V, n = 25, 1300
    rng = np.random.default_rng(M)
    streams = [_random_codes(rng, V, M, cap, n, hot) for hot in (2, 6, 25)]
    B = len(streams)
    rows = np.asarray(streams, dtype=np.int32)
    cnt = np.full(B, n, np.int32)
    ref = [oracle.lzw_decode(s, V, M, cap) for s in streams]
    longest = max(len(r[0]) for r in ref)
    for kernel in (0, 2, 4):
        ctx = _ctx(B, V, M, cap, kernel)
        toks, n_tok, st = gpu_decode(ctx, rows, cnt, out_stride=longest)
        assert (st == 0).all()
        for b in range(B):
            assert toks[b, :n_tok[b]].tolist() == ref[b][0]
        assert_codebook_equal(ctx, [r[1] for r in ref], M, cap)
        for at in (0, 1, 511, 512, 1023, 1030):
            bad = rows.copy()
            bad[:, at] = V + cap + 5
            toks, n_tok, st = gpu_decode(ctx, bad, cnt, out_stride=longest)
            for b in range(B):
                rt, re, rst = oracle.lzw_decode(bad[b].tolist(), V, M, cap)
                assert int(st[b]) == rst == api.ST_BAD_CODE and toks[b, :n_tok[b]].tolist() == rt
            assert_codebook_equal(ctx, [oracle.lzw_decode(bad[b].tolist(), V, M, cap)[1] for b in range(B)], M, cap)
        for room in (1, 700, 1500):
            toks, n_tok, st = gpu_decode(ctx, rows, cnt, out_stride=room)
            for b in range(B):
                if len(ref[b][0]) > room:
                    assert int(st[b]) == api.ST_OVERFLOW and room - M < int(n_tok[b]) <= room
                assert toks[b, :n_tok[b]].tolist() == ref[b][0][:n_tok[b]]
        ctx.close()


@pytest.mark.parametrize("M,cap,kernel", [(3, 9000, 0), (5, 9000, 2), (4, 12000, 0), (3, 9000, 4)])
def test_windows_behind_a_cut_window(M, cap, kernel):
    """Stretches of a parse's codes, of arbitrary ones and of a parse's with one in sixty replaced, longer and shorter than a
    window, in turn: windows that are inserted at once, taken back, looked through first, and inserted at once again."""
    V = 200
    rng = np.random.default_rng(M)
    streams = []
    for b in range(3):
        s, codes = oracle.LZWStream(V, M, cap), []
        for part, n in enumerate((1500, 700, 2600, 300, 1100, 60, 1500)):
            if (part + b) % 3 == 0:                          # pairs that repeat all the time
                chunk = rng.integers(0, 12, n).tolist()
            else:                                            # what a parse of these tokens gives, as the codebook stands
                t = oracle.LZWStream(V, M, cap)
                t.decode_chunk(codes)
                chunk = t.encode_chunk(np.minimum(rng.zipf(1.3, n) - 1, V - 1).tolist())[0]
                if (part + b) % 3 == 2:
                    chunk = [int(rng.integers(0, 12)) if rng.random() < 1 / 60 else c for c in chunk]
            for c in chunk:
                if c < V + len(s.entries):                   # (a replaced code moves the entries behind it)
                    assert s.decode_chunk([c])[1] == 0
                    codes.append(c)
        streams.append(codes)
    n = min(len(c) for c in streams)
    rows = np.asarray([c[:n] for c in streams], dtype=np.int32)
    ref = [oracle.lzw_decode(r.tolist(), V, M, cap) for r in rows]
    ctx = _ctx(len(rows), V, M, cap, kernel)
    toks, n_tok, st = gpu_decode(ctx, rows, None, out_stride=M * n)
    for b in range(len(rows)):
        assert int(st[b]) == ref[b][2] == 0 and toks[b, :n_tok[b]].tolist() == ref[b][0]
    assert_codebook_equal(ctx, [r[1] for r in ref], M, cap)
    ctx.close()


@pytest.mark.parametrize("M,cap", [(3, 400), (5, 40), (8, 1500), (2, 0)])
def test_codes_behind_a_full_codebook(M, cap):
    """Rows so long that the codes behind a full codebook go to a launch of their own, in parts: ragged rows (one too short for
    it), no output, a code that names nothing and an output row that ends in any part, appended calls behind it."""
    from paper_2506_01084_amd import api

    V, n = 25, 12000
    rng = np.random.default_rng(M + cap)
    streams = []
    for b in range(4):
        head = oracle.lzw_encode(rng.integers(0, V, 4 * cap + 64).tolist(), V, M, cap)
        assert len(head[1]) == cap
        streams.append(head[0] + rng.integers(0, V + cap, n - len(head[0])).tolist())
    rows = np.asarray(streams, dtype=np.int32)
    cnt = np.array([n, n - 1, 2500, 9217], dtype=np.int32)
    B = len(cnt)
    ref = [oracle.lzw_decode(streams[b][:cnt[b]], V, M, cap) for b in range(B)]
    longest = max(len(r[0]) for r in ref)
    ctx = _ctx(B, V, M, cap)
    toks, n_tok, st = gpu_decode(ctx, rows, cnt, out_stride=longest)
    assert (st == 0).all()
    for b in range(B):
        assert toks[b, :n_tok[b]].tolist() == ref[b][0] and (toks[b, n_tok[b]:] == -7).all()
    assert_codebook_equal(ctx, [r[1] for r in ref], M, cap)
    # appended: all codes of the second call stand behind a full codebook; then a few, then a tokenized chunk
    s = [oracle.LZWStream(V, M, cap) for _ in range(B)]
    for b in range(B):
        s[b].decode_chunk(streams[b][:cnt[b]])
    more = rng.integers(0, V + cap, (B, 7000)).astype(np.int32)
    for chunk, width in ((more, M * 7000), (more[:, :5], 0)):
        toks, n_tok, st = gpu_decode(ctx, chunk, None, out_stride=width, flags=api.APPEND)
        for b in range(B):
            want, rst = s[b].decode_chunk(chunk[b].tolist())
            assert int(st[b]) == rst == 0 and int(n_tok[b]) == len(want)
            assert toks is None or toks[b, :n_tok[b]].tolist() == want
    _, n_tok, st = gpu_decode(ctx, rows, cnt, out_stride=0)
    assert (st == 0).all() and n_tok.tolist() == [len(r[0]) for r in ref]
    for at in (0, 3000, 6143, 6144, 7168, 9215, 9216, n - 1):
        bad = rows.copy()
        bad[:, at] = (V + cap, -1, V + cap + 7, -2**31)
        toks, n_tok, st = gpu_decode(ctx, bad, cnt, out_stride=longest)
        for b in range(B):
            rt, _, rst = oracle.lzw_decode(bad[b, :cnt[b]].tolist(), V, M, cap)
            assert int(st[b]) == rst and toks[b, :n_tok[b]].tolist() == rt and (toks[b, n_tok[b]:] == -7).all()
    for room in (longest - 1, longest - 1500, len(ref[3][0]), len(ref[3][0]) - 1, 5000):
        toks, n_tok, st = gpu_decode(ctx, rows, cnt, out_stride=room)
        for b in range(B):
            rt, _, rst = oracle.lzw_decode(streams[b][:cnt[b]], V, M, cap, max_tokens=room)
            assert int(st[b]) == rst and toks[b, :n_tok[b]].tolist() == rt and (toks[b, n_tok[b]:] == -7).all()
    ctx.close()


def test_lengths_overwritten_by_the_counts_of_a_long_decode():
    """One tensor for the lengths and the token counts of a decode call in two launches: the second takes the lengths that
    the first one read (expanding codes, so that the counts are larger; one row ends behind its full codebook, one before)."""
    import torch

    from paper_2506_01084_amd import api

    V, M, cap, n = 25, 3, 400, 9000
    rng = np.random.default_rng(11)
    streams = []
    for b in range(3):
        head = oracle.lzw_encode(rng.integers(0, V, 4 * cap + 64).tolist(), V, M, cap)[0]
        streams.append(head + rng.integers(V, V + cap, n - len(head)).tolist())
    cnt = [n - 2000, n, 300]
    ref = [oracle.lzw_decode(streams[b][:cnt[b]], V, M, cap) for b in range(3)]
    assert max(len(r[0]) for r in ref) > n
    ctx = _ctx(3, V, M, cap)
    codes = torch.tensor(streams, dtype=torch.int32, device="cuda")
    for counts_first in (True, False):
        tokens = torch.full((3, M * n), -7, dtype=torch.int32, device="cuda")
        shared = torch.tensor(cnt, dtype=torch.int32, device="cuda")
        other = torch.empty_like(shared)
        ctx.lzw_decode(codes, shared, tokens, *((shared, other) if counts_first else (other, shared)), api.RESET)
        n_tok, st = (shared, other) if counts_first else (other, shared)
        assert st.tolist() == [0, 0, 0] and n_tok.tolist() == [len(r[0]) for r in ref]
        got = tokens.cpu().numpy()
        for b in range(3):
            assert got[b, :len(ref[b][0])].tolist() == ref[b][0] and (got[b, len(ref[b][0]):] == -7).all()
    ctx.close()


@pytest.mark.parametrize("shared_with", ["counts", "status", "neither"])
def test_lengths_overwritten_by_many_sequences(shared_with):
    """One tensor for the lengths and the counts (or the status words) of a call that has more sequences than run at once and
    would take them in order of length, in both directions."""
    import torch

    from paper_2506_01084_amd import api

    B, N, V, M, cap = 1300, 2100, 100, 3, 300
    rng = np.random.default_rng(17)
    lens = rng.integers(1, 200, B).astype(np.int32)
    lens[rng.integers(0, B, 12)] = N
    tokens = np.minimum(rng.zipf(1.3, (B, N)) - 1, V - 1).astype(np.int32)
    ref = oracle_encode_batch(tokens, lens, V, M, cap)
    n_ref = [len(r[0]) for r in ref]
    ctx = _ctx(B, V, M, cap)
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    outputs = lambda n: dict(counts=(n, torch.empty_like(n)), status=(torch.empty_like(n), n),
                             neither=(torch.empty_like(n), torch.empty_like(n)))[shared_with]
    d_tok, d_codes, d_back = t(tokens), t(np.full((B, N), -7, np.int32)), t(np.full((B, N), -7, np.int32))
    d_len = t(lens)
    n_codes, st = outputs(d_len)
    ctx.lzw_encode(d_tok, d_len, d_codes, n_codes, st, api.RESET)
    assert (st == 0).all() and n_codes.tolist() == n_ref
    codes = d_codes.cpu().numpy()
    for b in range(B):
        assert codes[b, :n_ref[b]].tolist() == ref[b][0]
    assert_codebook_equal(ctx, [r[1] for r in ref], M, cap)
    d_n = t(np.asarray(n_ref, np.int32))
    n_tok, st = outputs(d_n)
    ctx.lzw_decode(d_codes, d_n, d_back, n_tok, st, api.RESET)
    assert (st == 0).all() and n_tok.tolist() == lens.tolist()
    back = d_back.cpu().numpy()
    assert all((back[b, :lens[b]] == tokens[b, :lens[b]]).all() and (back[b, lens[b]:] == -7).all() for b in range(B))
    ctx.close()


@pytest.mark.parametrize("M,cap,kernel", [(3, 12000, 0), (5, 20000, 0), (8, 23000, 0), (8, 28136, 0), (4, 28137, 0), (5, 3000, 0), (5, 3000, 2)])
def test_calls_on_one_codebook(M, cap, kernel):
    """A codebook emptied twice, then appended to by long, short and single-element calls in both directions: tables in LDS,
    in memory with their tags in LDS (more than 11000 entries), in memory alone (more than 28136, or as an option)."""
    from paper_2506_01084_amd import api

    V, B = 3000, 3
    rng = np.random.default_rng(cap + M)
    draw = lambda n: np.where(rng.random((B, n)) < 0.3, rng.integers(0, 6, (B, n)), np.minimum(rng.zipf(1.2, (B, n)) - 1, V - 1)).astype(np.int32)
    enc, dec = _ctx(B, V, M, cap, kernel), _ctx(B, V, M, cap, kernel)
    s = d = None
    for n, flags in ((2500, api.RESET), (3100, api.RESET), (2048, api.APPEND), (40, api.APPEND), (1, api.APPEND), (700, api.APPEND)):
        if flags == api.RESET:
            s, d = ([oracle.LZWStream(V, M, cap) for _ in range(B)] for _ in range(2))
        tokens = draw(n)
        codes, n_codes, st = gpu_encode(enc, tokens, None, flags=flags)
        toks, n_tok, st2 = gpu_decode(dec, codes, n_codes, out_stride=n, flags=flags)
        for b in range(B):
            want, rst = s[b].encode_chunk(tokens[b].tolist())
            assert int(st[b]) == rst == 0 and codes[b, :n_codes[b]].tolist() == want, (n, flags, b)
            assert d[b].decode_chunk(want) == (tokens[b].tolist(), 0)
            assert int(st2[b]) == 0 and toks[b, :n_tok[b]].tolist() == tokens[b].tolist(), (n, flags, b)
        assert_codebook_equal(enc, [x.entries for x in s], M, cap)
        assert_codebook_equal(dec, [x.entries for x in d], M, cap)
    enc.close()
    dec.close()


@pytest.mark.parametrize("M", [3, 6])
def test_ragged_appends_to_a_table_in_memory(M):
    """Appended rows of one call on both sides of the length, and of the room, from which the tags of a table in memory are
    made for it."""
    from paper_2506_01084_amd import api

    V, cap, N = 500, 12000, 2100
    lens = np.array([N, 2048, 2047, 700, 65, 64, 0], dtype=np.int32)
    B, rng = len(lens), np.random.default_rng(M)
    enc, dec = _ctx(B, V, M, cap), _ctx(B, V, M, cap)
    s = [oracle.LZWStream(V, M, cap) for _ in range(B)]
    for flags in (api.RESET, api.APPEND, api.APPEND, "room", api.APPEND, api.APPEND):
        if flags == "room":                                  # room for 500 to 1900 entries
            N, flags = 12000, api.RESET
            lens = (10300 + 250 * np.arange(B)).astype(np.int32)
            s = [oracle.LZWStream(V, M, cap) for _ in range(B)]
            tokens = rng.integers(0, V, (B, N)).astype(np.int32)
        else:
            N = 2100
            tokens = np.minimum(rng.zipf(1.2, (B, N)) - 1, V - 1).astype(np.int32)
        codes, n_codes, st = gpu_encode(enc, tokens, lens, flags=flags)
        toks, n_tok, st2 = gpu_decode(dec, codes, n_codes, out_stride=N, flags=flags)
        for b in range(B):
            want, rst = s[b].encode_chunk(tokens[b, :lens[b]].tolist())
            assert int(st[b]) == int(st2[b]) == rst == 0 and codes[b, :n_codes[b]].tolist() == want
            assert int(n_tok[b]) == lens[b] and (toks[b, :lens[b]] == tokens[b, :lens[b]]).all()
        lens = lens[::-1].copy() if N == 2100 else np.full(B, 2100, dtype=np.int32)
    assert_codebook_equal(enc, [x.entries for x in s], M, cap)
    assert_codebook_equal(dec, [x.entries for x in s], M, cap)
    enc.close()
    dec.close()


def _edge_hash(p, t):
    """The kernel's hash of an edge (arrays of uint64)."""
    h = (p * np.uint64(0x9E3779) + t * np.uint64(0xC2B2AF)) & np.uint64(0xFFFFFFFF)
    h ^= h >> np.uint64(15)
    return (h * np.uint64(0x2C1B3C6D)) & np.uint64(0xFFFFFFFF)


def _groups(h, bits):
    a = h >> np.uint64(32 - bits)
    return a, a ^ (((h >> np.uint64(2)) & np.uint64((1 << bits) - 1)) | np.uint64(1))


def _crowded_pairs(V, bits):
    """Pairs of tokens, the most found, whose edges share both of their groups of the round's set (2^bits groups of four):
    beyond eight of them in a window the rest find no slot."""
    p, t = np.divmod(np.arange(V * V, dtype=np.uint64), np.uint64(V))
    a, b = _groups(_edge_hash(p, t), bits)
    _, at, count = np.unique((a << np.uint64(16)) | b, return_inverse=True, return_counts=True)
    best = np.nonzero(at == count.argmax())[0]
    return np.stack([p[best], t[best]], 1).astype(np.int32).reshape(-1)


def _edges_without_slot(tokens, bits):
    """Edges of neighbours that find both of their groups full, inserted in order (the first iteration of a first window)."""
    groups, lost = {}, 0
    for p, t in dict.fromkeys(zip(tokens[:-1].tolist(), tokens[1:].tolist())):
        h = _edge_hash(np.uint64(p), np.uint64(t))
        for g in map(int, _groups(h, bits)):
            if groups.get(g, 0) < 4:
                groups[g] = groups.get(g, 0) + 1
                break
        else:
            lost += 1
    return lost


# sequences, tokens, groups of the round's set (log2) of the kernel that takes them, its waves, sets and slots per position
@pytest.mark.parametrize("B,N,cap,bits,kernel", [
    pytest.param(4, 500, 2500, 10, 0, id="8 waves, two sets of 8"),
    pytest.param(4, 3000, 2500, 11, 0, id="16 waves, two sets of 8"),
    pytest.param(4, 3000, 6000, 10, 0, id="16 waves, two sets of 4"),
    pytest.param(4, 3000, 12000, 10, 0, id="16 waves, two sets of 4, tags"),
    pytest.param(4, 3000, 2500, 10, 2, id="16 waves, two sets of 4, table in memory"),
    pytest.param(4, 400, 2500, 6, 4, id="one wave"),
    pytest.param(900, 500, 2048, 9, 0, id="8 waves, one set of 4"),
    pytest.param(300, 500, 2048, 9, 0, id="8 waves, two sets of 4"),
])
def test_windows_whose_edges_find_no_slot(B, N, cap, bits, kernel):
    """Windows cut because an edge finds both of its groups full, with whole windows between and behind them; then a token
    out of range, and an output row that ends, in windows of either kind."""
    import torch

    from paper_2506_01084_amd import api

    V, M = 4000 if bits == 11 else 1800, 3
    rng = np.random.default_rng(N + bits)
    crowd = _crowded_pairs(V, bits)[:60]
    assert len(crowd) >= 24 and _edges_without_slot(crowd, bits) >= 4
    tokens = np.minimum(rng.zipf(1.25, (B, N)) - 1, V - 1).astype(np.int32)
    tokens[0, :len(crowd)] = crowd
    tokens[1, N // 2:N // 2 + len(crowd)] = crowd
    tokens[2, N - len(crowd):] = crowd
    lens = np.full(B, N, dtype=np.int32)
    if B > 256:
        lens[3:] = rng.integers(0, 120, B - 3)
    _round_trip(tokens, lens, V, M, cap, kernel)
    ctx = _ctx(B, V, M, cap, kernel)

    # the kernel cuts a window for it: more rounds than for a stream of the same structure, its tokens under other names (in which
    # all edges find a slot), or there would be nothing to test here
    named = np.concatenate([tokens[0], tokens[0]]).reshape(2, N)
    named[1] = rng.permutation(V)[tokens[0]]
    for _ in range(20):
        if _edges_without_slot(named[1][:64 if kernel == 4 else 1024], bits) == 0:
            break
        named[1] = rng.permutation(V)[tokens[0]]
    pair = np.tile(named, (B // 2 + 1, 1))[:B]
    gpu_encode(ctx, pair, np.where(np.arange(B) < 2, N, 0).astype(np.int32))
    torch.cuda.synchronize()
    rounds = ctx.lzw_rounds()[:2].tolist()
    assert rounds[0] > rounds[1], rounds

    for at in (5, 40, N // 3, N // 2 + 30, N - 1):
        bad = tokens.copy()
        bad[:, at] = V + 7
        codes, n_codes, status = gpu_encode(ctx, bad, lens)
        ref = oracle_encode_batch(bad, lens, V, M, cap)
        for b in range(B):
            assert int(status[b]) == ref[b][2] and codes[b, :n_codes[b]].tolist() == ref[b][0]
            assert lens[b] <= at or int(status[b]) == api.ST_BAD_TOKEN
        assert_codebook_equal(ctx, [r[1] for r in ref], M, cap)
    ref = oracle_encode_batch(tokens, lens, V, M, cap)
    for room in (3, 35, N // 2):
        codes, n_codes, status = gpu_encode(ctx, tokens, lens, out_stride=room)
        for b in range(B):
            want = ref[b][0][:room]
            assert int(n_codes[b]) == len(want) and codes[b, :n_codes[b]].tolist() == want
            assert int(status[b]) == (api.ST_OVERFLOW if len(ref[b][0]) > room else 0)
    ctx.close()
