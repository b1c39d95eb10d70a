"""GPU launch shapes against the CPU oracle, at the sizes where a launch
changes: counts of (sequence, head) slices around the multiples of 8 that the
work order deals to the XCDs, the split and one-workgroup decode, and the
rounds of the bookkeeping kernels."""
import numpy as np
import pytest
import torch

from oracle import sckv_oracle as O

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
# the output's bf16 rounding (2^-9 of values below 4) and that of the
# probabilities (2^-9 of each, values below 5) stay under half of this
TOL = 2e-2


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2310_08152_amd import binding  # noqa: F401  (fails loudly without the library)


def P():
    from paper_2310_08152_amd import path
    return path


def W():
    from paper_2310_08152_amd import workload
    return workload


def f64(t):
    return t.detach().to("cpu", torch.float64).numpy()


def rnd(shape, seed, dtype="bf16"):
    return W().randn(shape, seed=seed, dtype=dtype).to(DEV)


@pytest.mark.parametrize("b,H", [(1, 1), (1, 7), (2, 4), (3, 3), (1, 17), (5, 16)])
def test_prefill_covers_every_slice(b, H):
    """Every slice's every block is computed whatever the number of slices
    (left-over slices alone, whole groups alone, both, a partial group)."""
    print(f"prefill b={b} H={H}", flush=True)
    L, d = 300, 64
    rng = np.random.default_rng(b * 100 + H)
    spans = [W().spans_uniform_lengths(L, 0.4, 4, 24, rng) for _ in range(b)]
    q, k, v = (rnd((b, H, L, d), 200 + i) for i in range(3))
    o = torch.full_like(q, float("nan"))
    P().prefill_layer(q, k, v, o, P().SpanMeta(spans, L, DEV), P().Workspace(b, H, L, L, d, DEV), L)
    torch.cuda.synchronize()
    Q, K, V, Og = f64(q), f64(k), f64(v), f64(o)
    assert np.isfinite(Og).all()
    for s in range(b):
        ref = O.masked_attention(Q[s], K[s], V[s], O.attention_mask(O.token_types(spans[s], L)))
        assert np.abs(Og[s] - ref).max() <= TOL, s


# (b, H, L_cap): split launches whose chunks are cut finer than 1024 rows (8,
# 32, 96, 188, 192, 256 slices) and one workgroup per slice (a short cache)
@pytest.mark.parametrize("finer", [True, False], ids=["room", "least"])
@pytest.mark.parametrize("d,theta", [(64, 0.0), (80, 10000.0)])
@pytest.mark.parametrize("b,H,L_cap", [(4, 2, 2400), (4, 8, 1400), (4, 24, 1500), (4, 16, 1000),
                                       (4, 47, 2100), (4, 48, 2100), (4, 64, 2100), (4, 64, 1100),
                                       (4, 72, 1100)])
def test_decode_launch_shapes(b, H, L_cap, d, theta, finer):
    """One decode step against the oracle, at chunk edges, with the workspace
    path.Workspace allocates and with the least one the library accepts."""
    print(f"decode b={b} H={H} L_cap={L_cap} d={d} finer={finer}", flush=True)
    from paper_2310_08152_amd import binding as B
    lens = [0, 129, 1024, L_cap - 1] if L_cap > 1024 else [1, 127, 128, L_cap - 1]
    T = L_cap + 8
    meta = P().SpanMeta([[] for _ in range(b)], T, DEV)
    cache = P().KVCache(1, b, H, L_cap, d, torch.bfloat16, DEV)
    cache.kv.copy_(rnd(cache.kv.shape, 71))
    cache.kv_len.copy_(torch.tensor(lens, dtype=torch.int32))
    cache.cur_tok.copy_(torch.tensor(lens, dtype=torch.int32))
    ws = P().Workspace(b, H, 1, L_cap, d, DEV)
    if not finer:
        ws.decode = ws.decode[:B.sckv_decode_workspace_bytes(b, H, L_cap, d)].contiguous()
    q, kn, vn = (rnd((b, H, d), 72 + i) for i in range(3))
    o = torch.full_like(q, float("nan"))
    K, V = f64(cache.kv[0, 0]), f64(cache.kv[0, 1])
    P().decode_layer(q, kn, vn, cache, 0, meta, ws, o, theta=theta)
    torch.cuda.synchronize()
    assert int(cache.status) == 0
    Q, KN, VN, Og = f64(q), f64(kn), f64(vn), f64(o)
    for s in range(b):
        qs, ks = Q[s], KN[s]
        if theta > 0:
            qs, ks = (np.stack([O.rope_rotate_half(x[h][None], [lens[s]], theta)[0]
                                for h in range(H)]) for x in (qs, ks))
        ref = O.decode_attention(qs, ks, VN[s], K[s], V[s], lens[s], False)
        # fp32 sums; the output's bf16 rounding, and the new key's
        assert np.abs(Og[s] - ref).max() <= TOL, (s, np.abs(Og[s] - ref).max())
        assert np.array_equal(f64(cache.kv[0, 1, s, :, lens[s]]), VN[s])


# (slices, L_cap, one): the line between one workgroup per slice and the split
@pytest.mark.parametrize("d", [64, 80])
@pytest.mark.parametrize("slices,L_cap,one", [(32, 768, True), (32, 769, False), (160, 1536, True),
                                              (192, 1537, False), (256, 3000, False),
                                              (511, 1536, True), (511, 1537, False),
                                              (512, 1537, True)])
def test_decode_splits_long_slices(slices, L_cap, one, d):
    """Below 512 slices a long cache is split, so that one long slice among
    short ones does not stay on one CU; a launch of one workgroup per slice
    leaves the workspace alone."""
    print(f"decode split slices={slices} L_cap={L_cap} d={d}", flush=True)
    b = slices if slices == 511 else 8
    H = slices // b
    lens = [L_cap - 1] + [40 + s % 200 for s in range(b - 1)]
    meta = P().SpanMeta([[]] * b, L_cap + 8, DEV)
    cache = P().KVCache(1, b, H, L_cap, d, torch.bfloat16, DEV)
    cache.kv.copy_(rnd((1, 2, 1, 1, L_cap, d), 91).expand_as(cache.kv))
    cache.kv_len.copy_(torch.tensor(lens, dtype=torch.int32))
    cache.cur_tok.copy_(cache.kv_len)
    ws = P().Workspace(b, H, 1, L_cap, d, DEV)
    ws.decode.fill_(0x5a)
    q, kn, vn = (rnd((b, H, d), 92 + i) for i in range(3))
    o = torch.full_like(q, float("nan"))
    K, V = (f64(x[:1].expand(H, -1, -1)) for x in (cache.kv[0, 0, 0], cache.kv[0, 1, 0]))
    P().decode_layer(q, kn, vn, cache, 0, meta, ws, o)
    torch.cuda.synchronize()
    assert bool((ws.decode == 0x5a).all()) == one
    Q, KN, VN, Og = f64(q), f64(kn), f64(vn), f64(o)
    for s in sorted({0, 1, b // 2, b - 1}):
        ref = O.decode_attention(Q[s], KN[s], VN[s], K, V, lens[s], False)
        # fp32 sums; the output's bf16 rounding, and the new key's
        assert np.abs(Og[s] - ref).max() <= TOL, s


@pytest.mark.parametrize("L", [1, 255, 256, 1023, 1024, 1025, 4096, 4097, 9000])
def test_span_metadata_plan_and_scan_round_sizes(L):
    """Span metadata, compaction indices and (through the attention's last
    rows) the prompt's plan at the edges of their rounds (256 tokens a
    workgroup, 1024 columns and 256, 1024 or 4096 rows a round)."""
    print(f"meta, plan, scan L={L}", flush=True)
    rng = np.random.default_rng(L)
    spans = [W().spans_uniform_lengths(L, 0.5, 2, 25, rng) if L > 60 else [], [(0, L + 3)]]
    T = L + 4
    meta = P().SpanMeta(spans, T, DEV)
    d, H = 64, 1
    cache = P().KVCache(1, 2, H, L + 1, d, torch.bfloat16, DEV)
    cache.kv.copy_(rnd(cache.kv.shape, 81))
    cache.start_prompt(L, meta)
    cache.compact(meta)
    kept = cache.kept_src.cpu().numpy()
    q, k, v = (rnd((2, H, L, d), 82 + i) for i in range(3))
    o = torch.empty_like(q)
    P().prefill_layer(q, k, v, o, meta, P().Workspace(2, H, L, 1, d, DEV), L)
    torch.cuda.synchronize()
    Og = f64(o)
    rows = sorted({0, L // 2, max(0, L - 2), L - 1})
    for s in range(2):
        types = O.token_types(spans[s], T)
        assert np.array_equal(meta.pos[s].cpu().numpy(), O.tie_positions(types)), s
        keep = np.flatnonzero(O.keep_rows(types, L)[:L])
        assert int(cache.kv_len[s]) == len(keep)
        assert np.array_equal(kept[s, :len(keep)], keep) and (kept[s, len(keep):] == -1).all()
        m = O.attention_mask_rows(O.token_types(spans[s], L), rows)
        ref = O.masked_attention(f64(q)[s][:, rows], f64(k)[s], f64(v)[s], m)
        assert np.abs(Og[s][:, rows] - ref).max() <= TOL, s


# one workgroup's tiles shared among groups of waves (few workgroups: three
# groups at d = 80, two or, for long lists, four at d = 64), with fewer tiles
# than groups (the first blocks), as many, and a remainder; one group (short
# prompts, many workgroups), on both sides of each line; and three
# (d = 80) or two (d = 64) in more workgroups where the slices are few and long
@pytest.mark.parametrize("d,H,L", [(80, 2, 1), (80, 2, 64), (80, 2, 130), (80, 2, 400), (80, 3, 901),
                                   (80, 2, 511), (80, 2, 512), (64, 2, 255), (64, 2, 256),
                                   (64, 2, 1408), (64, 2, 1409), (64, 70, 511), (64, 70, 512),
                                   (64, 2, 1), (64, 2, 65), (64, 2, 700), (64, 2, 1600),
                                   (80, 140, 129), (64, 260, 129), (80, 48, 700), (64, 96, 700),
                                   (80, 8, 4224), (64, 8, 8320)])
def test_prefill_wave_groups(d, H, L):
    print(f"prefill d={d} H={H} L={L}", flush=True)
    rng = np.random.default_rng(L + d)
    spans = [W().spans_uniform_lengths(L, 0.4, 4, 40, rng) if L > 60 else []]
    q, k, v = (rnd((1, H, L, d), 300 + i) for i in range(3))
    k[:, :, L // 2] *= 8  # one key whose scores jump: the running maxima of the groups differ
    o = torch.full_like(q, float("nan"))
    P().prefill_layer(q, k, v, o, P().SpanMeta(spans, L, DEV), P().Workspace(1, H, L, 1, d, DEV), L)
    torch.cuda.synchronize()
    heads = sorted({0, 1, H // 2, H - 1})
    Q, K, V, Og = (f64(x)[0][heads] for x in (q, k, v, o))
    assert np.isfinite(f64(o)).all()
    ref = O.masked_attention(Q, K, V, O.attention_mask(O.token_types(spans[0], L)))
    assert np.abs(Og - ref).max() <= TOL, np.abs(Og - ref).max()


# launches of groups of waves (three at d = 80; two and, for long lists, four at
# d = 64) against one of a single group (the same heads, repeated)
@pytest.mark.parametrize("d,H,L,many", [(80, 2, 777, 80), (64, 2, 777, 160), (64, 2, 1600, 160),
                                        (80, 8, 4224, 16)])
def test_prefill_rounds_alike_in_every_launch(d, H, L, many):
    """A row's probabilities are rounded to bf16 relative to its running
    maximum: with the same one in every launch, outputs differ by the order of
    32-bit sums alone.  Those are within some 1e-6 of each other, against a
    spacing of 2^-8 in bf16: one output in 500 may round the other way, one in
    50 where sums cancel to a tenth (maxima of their own move a quarter)."""
    print(f"prefill launches d={d} H={H} L={L}", flush=True)
    rng = np.random.default_rng(L + d)
    spans = [W().spans_uniform_lengths(L, 0.3, 2, 25, rng)]
    meta = P().SpanMeta(spans, L, DEV)
    q, k, v = (rnd((1, H, L, d), 320 + i) for i in range(3))
    few, all_ = torch.zeros_like(q), torch.zeros(1, many, L, d, dtype=q.dtype, device=DEV)
    P().prefill_layer(q, k, v, few, meta, P().Workspace(1, H, L, 1, d, DEV), L)
    Q, K, V = (x.repeat(1, many // H, 1, 1) for x in (q, k, v))
    P().prefill_layer(Q, K, V, all_, meta, P().Workspace(1, many, L, 1, d, DEV), L)
    torch.cuda.synchronize()
    share = float((few != all_[:, :H]).double().mean())
    assert share <= 0.02, share
    assert float((few.double() - all_[:, :H].double()).abs().max()) <= TOL


# fp32: the keys split over the waves (32 query rows a workgroup) on one side of
# each line, 128 rows on the other (one tile of keys, many workgroups)
@pytest.mark.parametrize("d,H,L", [(64, 3, 64), (80, 3, 64), (64, 3, 65), (80, 3, 65),
                                   (64, 73, 200), (64, 74, 200), (80, 36, 200), (80, 37, 200),
                                   (80, 73, 256), (64, 130, 200), (80, 130, 200), (64, 24, 1000),
                                   (64, 80, 127), (64, 81, 127), (80, 39, 400), (80, 40, 400),
                                   (64, 20, 1200), (80, 16, 1200), (64, 16, 2048), (80, 9, 2100)])
def test_prefill_f32_launches(d, H, L):
    print(f"prefill f32 d={d} H={H} L={L}", flush=True)
    rng = np.random.default_rng(L + d)
    spans = [W().spans_uniform_lengths(L, 0.4, 4, 40, rng)]
    q, k, v = (rnd((1, H, L, d), 330 + i, "f32") for i in range(3))
    k[:, :, L // 2] *= 8
    o = torch.full_like(q, float("nan"))
    P().prefill_layer(q, k, v, o, P().SpanMeta(spans, L, DEV), P().Workspace(1, H, L, 1, d, DEV), L)
    torch.cuda.synchronize()
    assert torch.isfinite(o).all()
    heads = sorted({0, 1, H // 2, H - 1})
    Q, K, V, Og = (f64(x)[0][heads] for x in (q, k, v, o))
    ref = O.masked_attention(Q, K, V, O.attention_mask(O.token_types(spans[0], L)))
    # 32-bit sums and exponentials of weights that add to 1, values below 5
    assert np.abs(Og - ref).max() <= 1e-5, np.abs(Og - ref).max()


# over a cache: one group of waves (many workgroups, short caches), two (d = 64, up
# to 512 where the cache is long) and four (d = 64, few over 1409 rows and more),
# three (d = 80, few); fp32 with the keys split and with 128 rows a workgroup
@pytest.mark.parametrize("dtype,d,H,L,block", [
    ("bf16", 80, 130, 630, 200), ("bf16", 80, 2, 630, 200), ("bf16", 64, 260, 450, 200),
    ("bf16", 64, 130, 450, 200), ("bf16", 64, 2, 450, 200), ("bf16", 64, 2, 1900, 300),
    ("bf16", 64, 130, 630, 200), ("bf16", 64, 130, 895, 200), ("bf16", 64, 130, 896, 200),
    ("bf16", 80, 2, 640, 200), ("bf16", 64, 2, 383, 200), ("f32", 64, 130, 300, 130), ("f32", 64, 5, 300, 130),
    ("f32", 80, 130, 300, 130), ("f32", 80, 5, 300, 130)])
def test_prefill_block_launches(dtype, d, H, L, block):
    """Blocks with a ragged last one, spans freed between them and one that
    stays open across them, against the oracle over the whole prompt."""
    print(f"blocks {dtype} d={d} H={H} L={L} block={block}", flush=True)
    rng = np.random.default_rng(L + d + H)
    a = block - 30
    spans = [[(c, r) for c, r in W().spans_uniform_lengths(a - 1, 0.4, 4, 24, rng)]
             + [(a, a + 60), (a + 61, L + 2)]]
    meta = P().SpanMeta(spans, L + 4, DEV)
    q, k, v = (rnd((1, 1, H, L, d), 350 + i, dtype) for i in range(3))
    o = torch.full_like(q, float("nan"))
    cache = P().KVCache(1, 1, H, L, d, q.dtype, DEV)
    P().prefill_progressive(q, k, v, o, cache, meta, P().Workspace(1, H, 1, L, d, DEV, block=block),
                            L, block)
    torch.cuda.synchronize()
    assert int(cache.status) == 0 and torch.isfinite(o).all()
    heads = sorted({0, 1, H // 2, H - 1})
    Q, K, V, Og = (f64(x)[0, 0][heads] for x in (q, k, v, o))
    ref = O.masked_attention(Q, K, V, O.attention_mask(O.token_types(spans[0], L)))
    assert np.abs(Og - ref).max() <= (TOL if dtype == "bf16" else 1e-5), np.abs(Og - ref).max()


# groups of waves, a single group; fp32 with 32 query rows a workgroup and 128
@pytest.mark.parametrize("dtype,d,H", [("bf16", 80, 2), ("bf16", 64, 2), ("bf16", 80, 140),
                                       ("bf16", 64, 270), ("f32", 80, 2), ("f32", 64, 2),
                                       ("f32", 80, 130), ("f32", 64, 130)])
def test_prefill_reads_only_its_rows(dtype, d, H):
    """Rows behind the prompt's, within the stride to the next slice, are not
    read, even where a longer prompt's plan lists them."""
    print(f"prefill rows {dtype} d={d} H={H}", flush=True)
    L, room = 600, 640
    meta = P().SpanMeta([[(3, 40)]], room, DEV)
    ws = P().Workspace(1, H, room, 1, d, DEV)
    q = rnd((1, H, L, d), 340, dtype)
    k, v = (torch.full((1, H, room, d), float("nan"), dtype=q.dtype, device=DEV) for _ in range(2))
    k[:, :, :L], v[:, :, :L] = rnd((1, H, L, d), 341, dtype), rnd((1, H, L, d), 342, dtype)
    o = [torch.full_like(q, float("nan")) for _ in range(2)]
    for out, n in zip(o, (L, room)):
        P().prefill_plan(meta, ws, 1, n)
        P().prefill_layer(q, k[:, :, :L], v[:, :, :L], out, meta, ws, L, planned=True)
    torch.cuda.synchronize()
    assert torch.isfinite(o[0]).all() and torch.equal(o[0], o[1])


@pytest.mark.parametrize("dtype,d,theta,H,n", [("bf16", 80, 10000.0, 3, 37), ("bf16", 64, 0.0, 4, 300),
                                               ("f32", 80, 10000.0, 1, 1), ("f32", 64, 10000.0, 5, 129)])
def test_rope_block_is_its_three_calls(dtype, d, theta, H, n):
    """One launch gives bit for bit what the three calls give, a sequence
    without room included."""
    print(f"rope_block {dtype} d={d} theta={theta} H={H} n={n}", flush=True)
    from paper_2310_08152_amd import binding as B
    b, L, L_cap, tok0 = 3, 400, 500, 23
    meta = P().SpanMeta([[(3, 40)], [(30, 200), (210, 211)], []], L, DEV)
    q, k, v = (rnd((b, H, n + 5, d), 400 + i, dtype)[:, :, 2:2 + n] for i in range(3))
    row0 = torch.tensor([0, -1, L_cap - n], dtype=torch.int32, device=DEV)
    got = []
    for one in (False, True):
        cache = torch.zeros((2, b, H, L_cap, d), dtype=q.dtype, device=DEV)
        qr = torch.zeros((b, H, n + 1, d), dtype=q.dtype, device=DEV)
        st = torch.zeros(1, dtype=torch.int32, device=DEV)
        s, c = q.stride(1), cache.stride(2)
        if one:
            B.rope_block(q, k, v, qr, cache[0], cache[1], row0, L_cap, b, H, n, s, s, s,
                         qr.stride(1), c, d, meta.pos, L, tok0, theta, status=st)
        else:
            for x, y, th in ((k, cache[0], theta), (v, cache[1], 0.0)):
                B.rope_apply_at(x, y, row0, L_cap, b, H, n, s, c, d, meta.pos, L, tok0, th,
                                status=st)
            B.rope_apply(q, qr, b, H, n, s, qr.stride(1), d, meta.pos, L, tok0, theta)
        torch.cuda.synchronize()
        assert int(st) == B.STATUS_CAP
        got.append((cache, qr))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    assert not got[0][0][:, 1].any() and got[0][0][0, 2, :, L_cap - n:].any()


@pytest.mark.parametrize("L", [1, 256, 257, 300])
def test_start_prompt_bookkeeping(L):
    """Rows past the prompt keep what they held; a prompt longer than the
    cache or the metadata is refused; an empty one is accepted."""
    print(f"start_prompt L={L}", flush=True)
    b, cap = 3, 300
    meta = P().SpanMeta([[(0, 9)], [], [(20, 290)]], 320, DEV)
    cache = P().KVCache(1, b, 1, cap, 64, torch.bfloat16, DEV)
    cache.tok_idx.fill_(-7)
    cache.pos_ids.fill_(-7)
    cache.start_prompt(L, meta)
    t = torch.arange(cap, dtype=torch.int32)
    rows = (t < L).expand(b, cap)
    assert torch.equal(cache.tok_idx.cpu(), torch.where(rows, t, -7))
    assert torch.equal(cache.pos_ids.cpu(), torch.where(rows, meta.pos.cpu()[:, :cap], -7))
    assert cache.kv_len.tolist() == cache.cur_tok.tolist() == [L] * b
    with pytest.raises(RuntimeError):
        cache.start_prompt(cap + 1, meta)
    with pytest.raises(RuntimeError):
        cache.start_prompt(300, P().SpanMeta([[]] * b, 200, DEV))
    cache.start_prompt(0, meta)
    assert cache.kv_len.tolist() == [0] * b
