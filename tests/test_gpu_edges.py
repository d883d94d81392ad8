"""Kernels at the sizes where their tiling changes: remainders of pieces, waves and tiles, the smallest and
the largest of a range, against the oracle or against the general path."""
import numpy as np
import pytest

from oracle import cassandra_oracle as O
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2605_26558_amd import binding as B
    return torch, B, B.Context()


def _dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda()


@pytest.mark.parametrize("rows,cols", [(40, 77), (33, 2049), (16, 5001), (20, 8203)])
@pytest.mark.parametrize("ncols", [1, 8, 9, 20, 32])
def test_verify_gemm_with_rows_of_x_at_odd_offsets(env, rows, cols, ncols):
    """An odd number of columns: the rows of X start at odd multiples of 2 bytes and end inside a piece.
    Bound: fp32 sums of exact products, cols * 2^-24 * |W||x| at worst, far less in practice."""
    torch, B, ctx = env
    W, X = synth.weight_matrix(rows, cols, seed=5), synth.activations(cols, ncols, seed=6)
    ew = B.cas_encode_weight(ctx, _dev(torch, W), 600, 4)
    Y = B.cas_gemm_verify(ctx, ew, _dev(torch, X))
    one = torch.cat([B.cas_gemm_verify(ctx, ew, _dev(torch, X[c:c + 1])) for c in range(ncols)])
    assert torch.equal(Y, one)
    w, x = O.bf16_to_f64(W), O.bf16_to_f64(X)
    err = np.abs(Y.cpu().numpy() - x @ w.T)
    assert (err <= cols * 2.0 ** -24 * np.linalg.norm(x, axis=1)[:, None] * np.linalg.norm(w, axis=1)[None, :]).all()


def _streams(ew):
    d = ew.desc
    sp, vf = ew.spec.cpu().numpy(), ew.verif.cpu().numpy()
    def reg(buf, off, w):
        return buf[off: off + d.rows * w * 4].view("<u4").reshape(d.rows, w)
    return reg(sp, d.off_bitmap, d.bw), reg(sp, d.off_spec, d.sw), reg(vf, d.off_lo, d.lw), reg(vf, d.off_pruned, d.pw)


@pytest.mark.parametrize("cols,keep", [(9, 500), (600, 3), (1030, 997), (4096, 600), (4096, 1000), (4099, 2), (9000, 900)])
@pytest.mark.parametrize("act", [False, True])
def test_encoder_finds_the_threshold_in_any_distribution(env, cols, keep, act):
    """Rows on which a search between two counts has little to go by: two values, one in a thousand, ramps and
    powers of two, subnormal and infinite values, few distinct values.  Streams are compared bit for bit."""
    torch, B, ctx = env
    rng = np.random.default_rng(cols + keep)
    i = np.arange(cols)
    W = np.stack([
        np.where(i % 2, 0x3F80, 0x0001), np.where(i % 1000 == 7, 0x4000, 0x3C23), i % 0x7F80, (cols - i) % 0x7F80,
        (i % 255) << 7, rng.integers(0, 128, cols), np.where(rng.random(cols) < 0.3, 0x7F80, 0xFF80),
        rng.choice([0x3F80, 0xBF81, 0x3F82], cols), np.sort(rng.integers(0, 0x10000, cols)), np.zeros(cols, np.int64),
    ]).astype(np.uint16)
    a = np.where(i % 3 == 1, 1.0, np.exp2(rng.integers(-60, 60, cols))).astype(np.float32) if act else None
    ew = B.cas_encode_weight(ctx, _dev(torch, W), keep, 4, None if a is None else torch.from_numpy(a).cuda())
    p = O.encode_weight(W, keep, 4, a)
    for got, want in zip(_streams(ew), (p.bitmap, p.spec, p.lo, p.pruned)):
        np.testing.assert_array_equal(got, want)


@pytest.mark.parametrize("cols", [64, 511, 512, 513, 1000, 1024])
@pytest.mark.parametrize("keep", [1, 250, 600, 1000])
def test_encoder_finds_the_same_threshold_by_either_search(env, cols, keep):
    """4097 rows with norms are searched along a line between two counts from 512 columns on, 4096 rows and less bit by
    bit: the streams of the whole matrix are those of its parts, and of the oracle where a distribution comes first."""
    torch, B, ctx = env
    rows = 4097
    rng = np.random.default_rng(cols * 7 + keep)
    W = (rng.standard_normal((rows, cols)) * 0.02).astype(np.float32).view(np.uint32) >> 16
    kinds = [np.where(rng.random(cols) < 0.5, 0, 0x3F80), np.zeros(cols), rng.choice([0x3F80, 0xBF81, 0x3F82], cols),
             np.round(rng.standard_normal(cols) * 3).astype(np.float32).view(np.uint32) >> 16, np.full(cols, 0x7F80),
             rng.integers(0, 128, cols), np.arange(cols) % 0x7F80, np.where(np.arange(cols) % 100 == 7, 0x4000, 0)]
    for k, row in enumerate(kinds):
        W[k::97] = row
    W = W.astype(np.uint16)
    a = np.exp2(rng.integers(-3, 4, cols)).astype(np.float32)
    ad, Wd = torch.from_numpy(a).cuda(), _dev(torch, W)
    whole = _streams(B.cas_encode_weight(ctx, Wd, keep, 4, ad))
    parts = [_streams(B.cas_encode_weight(ctx, Wd[i:j], keep, 4, ad)) for i, j in ((0, 4096), (4096, rows))]
    p = O.encode_weight(W[:len(kinds)], keep, 4, a)
    for got, one, two, want in zip(whole, *parts, (p.bitmap, p.spec, p.lo, p.pruned)):
        np.testing.assert_array_equal(got, np.concatenate([one, two]))
        np.testing.assert_array_equal(got[:len(kinds)], want)


@pytest.mark.parametrize("cols", [1, 7, 9, 1024, 1025, 2048, 2049, 4096, 4097, 8193, 28672, 65536, 65543])
@pytest.mark.parametrize("keep,t,act", [(600, 4, True), (333, 0, False), (999, 7, True)])
def test_encoder_around_the_sizes_of_its_pieces_and_waves(env, cols, keep, t, act):
    """Rows just below and above the columns of a wave, of a piece and of all waves; equal keys at the
    threshold in another wave than the ones above it; norms with 0, -1, Inf and NaN among them."""
    torch, B, ctx = env
    rows = 5
    W = synth.weight_matrix(rows, cols, seed=cols)
    W[1, :] = 0x3F80                                        # all equal
    W[2, cols // 2:] = 0x3C00                               # equal keys from the middle of the row on
    W[3, ::3] = 0
    a = None
    if act:
        a = synth.act_norm(cols, seed=7)
        a[::11] = 0.0
        a[5::97], a[6::101], a[8::103] = -1.0, np.inf, np.nan
    buf = torch.zeros((rows, cols + 3), dtype=torch.int16, device="cuda")  # rows at odd offsets
    buf[:, :cols] = _dev(torch, W)
    ew = B.cas_encode_weight(ctx, buf[:, :cols], keep, t, None if a is None else torch.from_numpy(a).cuda())
    p = O.encode_weight(W, keep, t, a)
    for got, want in zip(_streams(ew), (p.bitmap, p.spec, p.lo, p.pruned)):
        np.testing.assert_array_equal(got, want)


def test_encoder_of_more_rows_than_a_grid_holds(env):
    """2^26 workgroups of 64 threads are one more than a launch may have."""
    torch, B, ctx = env
    rows = (1 << 26) + 3
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    W = torch.randint(-32768, 32768, (rows, 2), device="cuda", generator=gen, dtype=torch.int16)
    W[-1] = 0x3F80                                          # equal magnitudes: the lower column
    ew = B.cas_encode_weight(ctx, W, 500, 4)
    d = ew.desc
    assert (d.K, d.bw, d.sw, d.lw, d.pw) == (1, 1, 1, 1, 1)
    right = (W[:, 1] & 0x7FFF) > (W[:, 0] & 0x7FFF)
    kept, other = torch.where(right, W[:, 1], W[:, 0]).int(), torch.where(right, W[:, 0], W[:, 1]).int()
    for buf, off, want in ((ew.spec, d.off_bitmap, 1 + right.int()), (ew.spec, d.off_spec, (kept >> 4) & 0xFFF),
                           (ew.verif, d.off_lo, kept & 15), (ew.verif, d.off_pruned, other & 0xFFFF)):
        assert torch.equal(buf[off: off + 4 * rows].view(torch.int32), want)


WIDE_SHAPES = {  # hidden, query heads, kv heads, feed-forward: 4 parts per row, 8 (down); 4 and 16 (out, down)
    "a": (264, 4, 2, 520, 400 << 10),
    "b": (200, 14, 2, 8200, 1200 << 10),
    # 16 parts (qkv, out), 4 (gate/up, 64 rows a workgroup, 89 groups of them), 8 (down); the last run of a row is a part of one
    "c": (3900, 16, 4, 2840, 1600 << 10),
    # down: groups of rows for 64 a workgroup, whose LDS does not hold the counts of 61000 columns beside the sums
    "d": (5472, 4, 2, 61000, 8 << 20, 256 << 20),
}


@pytest.fixture(scope="module")
def wide_models(env):
    """(context, model, cache) with a workspace that holds the chunks of a prompt and with one that does not."""
    from types import SimpleNamespace
    torch, B, _ = env
    cache = {}

    def get(shape, form, kv_form, keep, t):
        key = (shape, form, kv_form, keep, t)
        if key in cache:
            return cache[key]
        hidden, n_q, n_kv, ffn, small, *big = WIDE_SHAPES[shape]
        gen = torch.Generator(device="cuda")
        gen.manual_seed(17)
        bits = lambda x: x.to(torch.bfloat16).view(torch.int16)  # noqa: E731
        rnd = lambda *s: torch.randn(s, device="cuda", generator=gen)  # noqa: E731
        sh = SimpleNamespace(hidden=hidden, n_layers=2, n_q_heads=n_q, n_kv_heads=n_kv, head_dim=128, ffn=ffn, vocab=301,
                             rms_eps=1e-5)
        dims = (("wqkv", (n_q + 2 * n_kv) * 128, hidden), ("wo", hidden, n_q * 128), ("wgu", 2 * ffn, hidden),
                ("wd", hidden, ffn), ("head", 301, hidden))
        raw = [{n: bits(rnd(r, c) * c ** -0.5) for n, r, c in dims} for _ in range(2)]
        gains = [bits(1 + 0.1 * rnd(hidden)) for _ in range(5)]
        embed = bits(rnd(301, hidden))
        rope = torch.from_numpy(synth.rope_table(640, 128, 500000.0)).cuda()
        out = []
        for ws in (small, *(big or [64 << 20])):
            ctx = B.Context(workspace=torch.empty(ws, dtype=torch.uint8, device="cuda"))
            enc = [{n: B.cas_encode_weight(ctx, w, keep, t) for n, w in L.items()} for L in raw]
            layers = [dict(e, g_attn=gains[2 * i], g_ffn=gains[2 * i + 1]) for i, e in enumerate(enc)]
            model = B.Model(ctx, sh, layers, enc[0]["head"], embed, gains[4], rope, max_cols=16)
            if form != "raw":
                recode, use = (B.cas_mx_encode, model.use_mx) if form == "shared" else (B.cas_unary_encode, model.use_unary)
                big = B.Context(workspace=torch.empty(8 << 20, dtype=torch.uint8, device="cuda"))
                for i in range(2):
                    for which, n in enumerate(("wqkv", "wo", "wgu", "wd")):
                        use(i, which, recode(big, enc[i][n]))
            kv = B.KVCache(ctx, 2, n_kv, n_pages=10, max_seqs=1, max_pages_per_seq=10, keep_permille=keep, trunc_bits=t,
                           exp_mode=B.CAS_EXP_SHARED if kv_form == "shared" else B.CAS_EXP_RAW)
            out.append((ctx, model, kv))
        cache[key] = out
        return out

    return get


@pytest.mark.parametrize("shape,form,kv_form,keep,t", [("a", "raw", "raw", 600, 4), ("b", "raw", "raw", 600, 4),
                                                       ("a", "raw", "raw", 1000, 0), ("b", "shared", "shared", 400, 3),
                                                       ("a", "shared", "raw", 600, 5), ("b", "unary", "raw", 600, 4)])
@pytest.mark.parametrize("before,n", [(0, 47), (0, 48), (5, 63), (9, 128), (0, 130), (70, 257), (3, 513)])
def test_prompt_in_chunks_leaves_the_bits_of_narrow_passes(env, wide_models, shape, form, kv_form, keep, t, before, n):
    torch, B, _ = env
    tokens = torch.from_numpy(synth.token_ids(before + n + 1, 301, seed=3)).cuda()
    got = []
    for ctx, model, kv in wide_models(shape, form, kv_form, keep, t):
        kv.spec_pool.zero_()
        kv.verif_pool.zero_()
        B.cas_kv_set_len(kv, 0, 0)
        if before:
            B.cas_prefill(ctx, model, kv, 0, tokens[:before])
        B.cas_prefill(ctx, model, kv, 0, tokens[before:before + n])
        assert B.cas_kv_len(kv, 0) == before + n
        logits = torch.empty((1, 301), device="cuda")
        B.cas_verify_step(ctx, model, kv, 0, tokens[-1:], 0, torch.empty(1, dtype=torch.int32, device="cuda"), logits)
        assert bool(torch.isfinite(logits).all())
        got.append((kv.spec_pool.clone(), kv.verif_pool.clone(), logits))
    for narrow, wide in zip(*got):
        assert torch.equal(narrow, wide)


@pytest.mark.parametrize("form,kv_form,keep,t", [("raw", "raw", 600, 4), ("shared", "raw", 700, 1)])
@pytest.mark.parametrize("before,n", [(0, 113), (0, 128), (0, 129), (70, 257), (3, 500)])
def test_prompt_in_chunks_over_all_numbers_of_parts(env, wide_models, form, kv_form, keep, t, before, n):
    """Rows cut into 4, 8 and 16 parts, one and two column blocks, workgroups of 32 and of 64 rows: the bits of narrow passes."""
    test_prompt_in_chunks_leaves_the_bits_of_narrow_passes(env, wide_models, "c", form, kv_form, keep, t, before, n)


def test_prompt_in_chunks_over_rows_too_long_for_64_in_a_workgroup(env, wide_models):
    test_prompt_in_chunks_leaves_the_bits_of_narrow_passes(env, wide_models, "d", "raw", "raw", 600, 4, 0, 300)


@pytest.mark.parametrize("ws", [4 << 20, 5 << 20, 6 << 20, 8 << 20])
@pytest.mark.parametrize("shape,kv_form", [("a", "raw"), ("b", "shared")])
def test_runs_of_a_prompt_in_one_launch_and_in_several(env, wide_models, shape, kv_form, ws):
    """The workspace decides how many runs of columns attention takes together and how long the chunks and the runs
    are: logits and cache are those of the workspace that holds everything at once."""
    torch, B, _ = env
    tokens = torch.from_numpy(synth.token_ids(521, 301, seed=4)).cuda()
    big, model, kv = wide_models(shape, "raw" if kv_form == "raw" else "shared", kv_form, *((600, 4) if kv_form == "raw" else (400, 3)))[1]
    small = B.Context(workspace=torch.empty(ws, dtype=torch.uint8, device="cuda"))
    got = []
    for ctx in (big, small):
        kv.spec_pool.zero_()
        kv.verif_pool.zero_()
        B.cas_kv_set_len(kv, 0, 0)
        B.cas_prefill(ctx, model, kv, 0, tokens[:-1])
        logits = torch.empty((1, 301), device="cuda")
        B.cas_verify_step(ctx, model, kv, 0, tokens[-1:], 0, torch.empty(1, dtype=torch.int32, device="cuda"), logits)
        torch.cuda.synchronize()
        got.append((kv.spec_pool.clone(), kv.verif_pool.clone(), logits))
    for one, several in zip(*got):
        assert torch.equal(one, several)


def _prompt_model(env, n_q, n_kv, kv_form, ctx, positions, layers=1, ffn=520):
    """A small model whose cache holds `positions` vectors that nothing computed, and room for 520 more."""
    from types import SimpleNamespace
    torch, B, _ = env
    gen = torch.Generator(device="cuda")
    gen.manual_seed(23)
    bits = lambda x: x.to(torch.bfloat16).view(torch.int16)  # noqa: E731
    rnd = lambda *s: torch.randn(s, device="cuda", generator=gen)  # noqa: E731
    hidden = 264
    sh = SimpleNamespace(hidden=hidden, n_layers=layers, n_q_heads=n_q, n_kv_heads=n_kv, head_dim=128, ffn=ffn, vocab=301,
                         rms_eps=1e-5)
    dims = (("wqkv", (n_q + 2 * n_kv) * 128, hidden), ("wo", hidden, n_q * 128), ("wgu", 2 * ffn, hidden), ("wd", hidden, ffn))
    enc = lambda r, c: B.cas_encode_weight(ctx, bits(rnd(r, c) * c ** -0.5), 600, 4)  # noqa: E731
    gain = lambda: bits(1 + 0.1 * rnd(hidden))  # noqa: E731
    weights = [{**{n: enc(r, c) for n, r, c in dims}, "g_attn": gain(), "g_ffn": gain()} for _ in range(layers)]
    rope = torch.from_numpy(synth.rope_table(positions + 640, 128, 500000.0)).cuda()
    model = B.Model(ctx, sh, weights, enc(301, hidden), bits(rnd(301, hidden)), gain(), rope, max_cols=16)
    pages = (positions + 520 + 63) // 64
    kv = B.KVCache(ctx, layers, n_kv, n_pages=pages, max_seqs=1, max_pages_per_seq=pages,
                   exp_mode=B.CAS_EXP_SHARED if kv_form == "shared" else B.CAS_EXP_RAW)
    kv.spec_pool.zero_()
    kv.verif_pool.zero_()
    for layer in range(layers):
        if positions:
            B.cas_kv_append(ctx, kv, layer, 0, bits(rnd(positions, n_kv, 128)), bits(rnd(positions, n_kv, 128)))
    return model, kv


def _attention_of(env, ctx, call):
    """(launches, milliseconds) of the exact attention of one call"""
    _, B, _ = env
    B.cas_prof_reset(ctx)
    B.cas_prof_enable(ctx, True)
    call()
    launches, ms, _ = B.cas_prof_read(ctx, B.PROF_ATTN_VERIFY)
    B.cas_prof_enable(ctx, False)
    return launches, ms


@pytest.mark.parametrize("kv_form,heads,ws", [("shared", 32, 256 << 20), ("raw", 32, 100 << 20)])
def test_runs_of_few_query_rows_take_no_longer_than_calls_of_their_own(env, kv_form, heads, ws):
    """One query head per kv head, and runs of 16 columns (shared exponents, or a workspace too small for runs of 64):
    16 query rows.  The best of five timings of a prompt's attention against the same columns in cas_attention, 16 at a
    time: 0.87 and 0.92 of it; 1.30 and 1.37 with products for 64 query rows.  The bound lies between."""
    torch, B, _ = env
    before, n = 8000, 256
    ctx = B.Context(workspace=torch.empty(ws, dtype=torch.uint8, device="cuda"))
    model, kv = _prompt_model(env, heads, heads, kv_form, ctx, before)
    tokens = torch.from_numpy(synth.token_ids(n, 301, seed=3)).cuda()
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    q, k, v = (torch.randn((16, heads, 128), device="cuda", generator=gen).to(torch.bfloat16).view(torch.int16) for _ in range(3))
    out = torch.empty_like(q)

    def prompt():
        B.cas_kv_set_len(kv, 0, before)
        B.cas_prefill(ctx, model, kv, 0, tokens)

    def calls():
        for c in range(0, n, 16):
            B.cas_kv_set_len(kv, 0, before + c)
            B.cas_attention(ctx, kv, 0, 0, True, q, k, v, out)

    prompt()
    calls()
    runs = [_attention_of(env, ctx, prompt) for _ in range(5)]
    own = min(_attention_of(env, ctx, calls)[1] for _ in range(5))
    assert runs[0][0] < n // 16, "the prompt went through narrow passes"
    ratio = min(ms for _, ms in runs) / own
    print(f"runs / calls: {ratio:.3f} in {runs[0][0]} launches", flush=True)
    assert ratio < 1.1


@pytest.mark.parametrize("n_q,n,columns", [(6, 64, 72), (4, 48, 56), (2, 130, 140), (8, 64, 72)])
def test_runs_waste_no_workspace(env, n_q, n, columns):
    """A workspace for the partial results of a few columns more than the prompt has takes them in one launch: runs of
    one length, and no longer ones that only a part of them would fit (groups of 3, 2, 1 and 4 query heads)."""
    torch, B, _ = env
    before, n_kv, hidden = 1930, 2, 264
    pages = -(-(before + n) // 64)
    front = n * 2 * (hidden + 2 * n_q * 128 + 2 * n_kv * 128) + 8 * 256  # what outlives attention, with its alignment
    ctx = B.Context(workspace=torch.empty(front + pages * n_q * columns * 132 * 4, dtype=torch.uint8, device="cuda"))
    model, kv = _prompt_model(env, n_q, n_kv, "raw", ctx, before)
    B.cas_kv_set_len(kv, 0, before)
    tokens = torch.from_numpy(synth.token_ids(n, 301, seed=3)).cuda()
    launches, _ = _attention_of(env, ctx, lambda: B.cas_prefill(ctx, model, kv, 0, tokens))
    assert launches == 1


@pytest.mark.parametrize("kv_form,n_q,n_kv", [("raw", 2, 2), ("raw", 4, 2), ("raw", 6, 2), ("raw", 8, 2), ("shared", 2, 2),
                                              ("shared", 4, 2), ("shared", 6, 2), ("shared", 8, 2), ("shared", 10, 2)])
@pytest.mark.parametrize("before,n", [(0, 203), (1930, 490)])
def test_runs_of_every_group_size_leave_the_bits_of_narrow_passes(env, kv_form, n_q, n_kv, before, n):
    """16 to 80 query rows in a run (the longer prompt has 64 for the groups of one and two), with a workspace for all of
    them at once and with a small one, on few pages and with the 32nd and 33rd page (where the merge changes its form) in
    one launch: logits and cache are those of the same columns a pass at a time."""
    torch, B, _ = env
    tokens = torch.from_numpy(synth.token_ids(n + 1, 301, seed=4)).cuda()
    big = B.Context(workspace=torch.empty(160 << 20, dtype=torch.uint8, device="cuda"))
    model, kv = _prompt_model(env, n_q, n_kv, kv_form, big, before, layers=2)
    piece = min(16, 80 // (n_q // n_kv))  # a pass of its own: too short for a chunk

    def once(ctx, step):
        B.cas_kv_set_len(kv, 0, before)
        for c in range(0, n, step):
            B.cas_prefill(ctx, model, kv, 0, tokens[c:min(c + step, n)])

    def result(ctx, step):
        launches, _ = _attention_of(env, ctx, lambda: once(ctx, step))
        logits = torch.empty((1, 301), device="cuda")
        B.cas_verify_step(ctx, model, kv, 0, tokens[-1:], 0, torch.empty(1, dtype=torch.int32, device="cuda"), logits)
        torch.cuda.synchronize()
        return launches, (kv.spec_pool.clone(), kv.verif_pool.clone(), logits)

    passes, want = result(big, piece)
    assert passes == 2 * -(-n // piece) and bool(torch.isfinite(want[2]).all())
    wide, got = result(big, n)
    assert wide == 2
    for x, y in zip(got, want):
        assert torch.equal(x, y)
    # the smallest workspace that takes a chunk has room for the partial results of the shortest runs only
    for ws in range(1 << 19, 16 << 20, 1 << 17):
        if ws < -(-(before + n) // 64) * n_q * piece * 132 * 4:
            continue
        short, got = result(B.Context(workspace=torch.empty(ws, dtype=torch.uint8, device="cuda")), n)
        for x, y in zip(got, want):
            assert torch.equal(x, y)
        if short < passes:
            break
    assert wide < short < passes


@pytest.mark.parametrize("piece", [16, 500])
def test_rounding_to_bf16_of_every_exponent(env, piece):
    """Ties, subnormals, numbers that round up to the next power or to infinity, NaNs with a payload in the low half
    alone, of both signs: one column of the projection is 1, so the rotated key is the cosine of the rotary table, any
    fp32 pattern, rounded.  In passes of 16 columns (split by the attention kernel) and in a chunk (by a kernel of
    its own), against the oracle's rounding."""
    from types import SimpleNamespace
    torch, B, _ = env
    low = [0, 1, 0x7FFF, 0x8000, 0x8001, 0xFFFF, 0x10000, 0x17FFF, 0x18000, 0x18001, 0x400000, 0x7F7FFF, 0x7F8000, 0x7FFFFF]
    pat = np.array([s << 31 | e << 23 | m for e in range(256) for s in (0, 1) for m in low], dtype=np.uint32)
    n = len(pat) // 64
    cos = pat.view(np.float32).reshape(n, 64)
    want = O.f64_to_bf16(cos)
    hidden = 264
    ctx = B.Context(workspace=torch.empty(16 << 20, dtype=torch.uint8, device="cuda"))
    sh = SimpleNamespace(hidden=hidden, n_layers=1, n_q_heads=2, n_kv_heads=2, head_dim=128, ffn=520, vocab=301, rms_eps=1e-5)
    one = 0x3F80
    zeros = lambda *s: torch.zeros(s, dtype=torch.int16, device="cuda")  # noqa: E731
    ones = lambda *s: torch.full(s, one, dtype=torch.int16, device="cuda")  # noqa: E731
    qkv = zeros(768, hidden)
    qkv[256:512].view(2, 128, hidden)[:, :64, 0] = one  # keys: 1 in the lower half of the channels, 0 in the upper
    enc = lambda w: B.cas_encode_weight(ctx, w, 600, 4)  # noqa: E731
    layer = {"wqkv": enc(qkv), "wo": enc(zeros(hidden, 256)), "wgu": enc(zeros(1040, hidden)), "wd": enc(zeros(hidden, 520)),
             "g_attn": ones(hidden), "g_ffn": ones(hidden)}
    rope = torch.zeros((n, 64, 2), device="cuda")
    rope[:, :, 0] = torch.from_numpy(pat.view(np.int32).reshape(n, 64)).cuda().view(torch.float32)
    model = B.Model(ctx, sh, [layer], enc(zeros(301, hidden)), ones(301, hidden), ones(hidden), rope, max_cols=16)
    kv = B.KVCache(ctx, 1, 2, n_pages=2, max_seqs=1, max_pages_per_seq=2)
    tokens = torch.zeros(n, dtype=torch.int32, device="cuda")
    for c in range(0, n, piece):
        B.cas_prefill(ctx, model, kv, 0, tokens[c:c + piece])
    got = B.cas_kv_read(ctx, kv, 0, 0, 0, n, full=True)[0].cpu().numpy().view(np.uint16)
    for head in (0, 1):
        np.testing.assert_array_equal(got[:, head, :64], want)


@pytest.mark.parametrize("rows,cols,keep", [(5, 1, 1000), (7, 31, 1000), (70, 33, 1000), (9, 64, 500), (1030, 4096, 600),
                                            (66, 5001, 333), (1030, 14336, 700)])
@pytest.mark.parametrize("t", [0, 4, 7])
def test_unary_rows_recoded_in_the_workspace(env, rows, cols, keep, t):
    """Rows of few exponents, rows with more than 16 of them (codes longer than a window takes), a row whose
    codes are long throughout; kept counts around a group of 32.  The verification product has the bits that
    the raw form gives, and so has the draft product, which reads the codes itself (the draft product through
    re-coded rows is a pass of a model: test_unary_draft_values_depend_on_neither_company_nor_workspace)."""
    torch, B, _ = env
    rng = np.random.Generator(np.random.Philox(rows + cols))
    W = synth.weight_matrix(rows, cols, seed=8)
    wide = rng.integers(100, 140, size=(rows, cols)).astype(np.uint16) << 7
    W[1::5] = (W[1::5] & 0x807F) | wide[1::5]                      # 40 exponents in every fifth row
    W[2] = (W[2] & 0x807F) | (98 << 7)                             # the rarest exponent throughout
    x, X = _dev(torch, synth.activations(cols, 1, seed=9)), _dev(torch, synth.activations(cols, 3, seed=10))
    with_ws = B.Context(workspace=torch.empty(8 << 20, dtype=torch.uint8, device="cuda"))
    ew = B.cas_encode_weight(with_ws, _dev(torch, W), keep, t)
    ue = B.cas_unary_encode(with_ws, ew)
    want = B.cas_gemm_verify(with_ws, ew, X)
    assert torch.equal(B.cas_gemm_verify_unary(with_ws, ue, X), want)
    assert torch.equal(B.cas_gemv_draft_unary(with_ws, ue, x).reshape(-1), B.cas_gemv_draft(with_ws, ew, x)[0])


@pytest.mark.parametrize("rows,cols", [(3, 33), (70, 300), (4101, 300), (2050, 700), (9, 4096), (6, 14336)])
@pytest.mark.parametrize("keep,t", [(1000, 0), (600, 4), (1000, 7)])
def test_unary_rows_with_a_few_long_codes(env, rows, cols, keep, t):
    """Most values share a few exponents, one in a hundred has any of 254: codes of up to 255 bits between short
    ones, over word boundaries and at the end of a row.  The verification product has the raw form's bits."""
    torch, B, _ = env
    rng = np.random.Generator(np.random.Philox(rows + cols + t))
    W = synth.weight_matrix(rows, cols, seed=12)
    rare = rng.random((rows, cols)) < 0.01
    rare[0] = False                                           # a row without any
    rare[-1, -1] = True                                       # the last value of a row
    W = np.where(rare, (W & 0x807F) | (rng.integers(1, 255, size=(rows, cols)).astype(np.uint16) << 7), W)
    ctx = B.Context(workspace=torch.empty(8 << 20, dtype=torch.uint8, device="cuda"))
    X = _dev(torch, synth.activations(cols, 3, seed=10))
    ew = B.cas_encode_weight(ctx, _dev(torch, W.astype(np.uint16)), keep, t)
    assert torch.equal(B.cas_gemm_verify_unary(ctx, B.cas_unary_encode(ctx, ew), X), B.cas_gemm_verify(ctx, ew, X))


def test_unary_draft_pass_through_the_workspace_and_without(env, wide_models):
    """The down projection of shape b (8200 columns) leaves the unary draft kernel one workgroup per CU and goes
    through re-coded rows where the workspace holds them; the small workspace does not.  The logits are the same."""
    torch, B, _ = env
    tokens = torch.from_numpy(synth.token_ids(40, 301, seed=3)).cuda()
    got = []
    for ctx, model, kv in wide_models("b", "unary", "raw", 600, 4):
        B.cas_kv_set_len(kv, 0, 0)
        B.cas_prefill(ctx, model, kv, 0, tokens[:-1])
        logits = torch.empty((1, 301), device="cuda")
        B.cas_draft_step(ctx, model, kv, 0, tokens[-1:], 0, torch.empty(1, dtype=torch.int32, device="cuda"), logits)
        got.append(logits)
    assert torch.equal(*got)


def _unary_draft_model(env, hidden, n_q, n_kv, ffn, ws, unary, keep=600):
    """Two layers and a head on unary-coded (or raw) weights, a context with a workspace of ws bytes."""
    from types import SimpleNamespace
    torch, B, _ = env
    gen = torch.Generator(device="cuda")
    gen.manual_seed(5)
    bits = lambda x: x.to(torch.bfloat16).view(torch.int16)  # noqa: E731
    rnd = lambda *s: torch.randn(s, device="cuda", generator=gen)  # noqa: E731
    sh = SimpleNamespace(hidden=hidden, n_layers=2, n_q_heads=n_q, n_kv_heads=n_kv, head_dim=128, ffn=ffn, vocab=301,
                         rms_eps=1e-5)
    dims = (("wqkv", (n_q + 2 * n_kv) * 128, hidden), ("wo", hidden, n_q * 128), ("wgu", 2 * ffn, hidden),
            ("wd", hidden, ffn))
    big = B.Context(workspace=torch.empty(8 << 20, dtype=torch.uint8, device="cuda"))
    layers = []
    for _ in range(2):
        L = {n: B.cas_encode_weight(big, bits(rnd(r, c) * c ** -0.5), keep, 4) for n, r, c in dims}
        layers.append(dict(L, g_attn=bits(1 + 0.1 * rnd(hidden)), g_ffn=bits(1 + 0.1 * rnd(hidden))))
    head = B.cas_encode_weight(big, bits(rnd(301, hidden) * hidden ** -0.5), keep, 4)
    embed, gain = bits(rnd(301, hidden)), bits(1 + 0.1 * rnd(hidden))
    rope = torch.from_numpy(synth.rope_table(64, 128, 500000.0)).cuda()
    ctx = B.Context(workspace=torch.empty(ws, dtype=torch.uint8, device="cuda"))
    model = B.Model(ctx, sh, layers, head, embed, gain, rope, max_cols=16, max_seqs=4)
    if unary:
        for i in range(2):
            for which, (n, _, _) in enumerate(dims):
                model.use_unary(i, which, B.cas_unary_encode(big, layers[i][n]))
        model.use_unary(-1, 0, B.cas_unary_encode(big, head))
    kv = B.KVCache(ctx, 2, n_kv, n_pages=4, max_seqs=4, max_pages_per_seq=1, keep_permille=600, trunc_bits=4)
    return ctx, model, kv


def _draft_kv(env, ctx, model, kv, n_seqs):
    """The last layer's keys and values of 48 draft passes, sequence by sequence."""
    torch, B, _ = env
    tokens = torch.from_numpy(synth.token_ids(48, 301, seed=3)).cuda()
    out = torch.empty(4, dtype=torch.int32, device="cuda")
    for seq in range(n_seqs):
        B.cas_kv_set_len(kv, seq, 0)
    for i in range(48):
        if n_seqs == 1:
            B.cas_draft_step(ctx, model, kv, 0, tokens[i:i + 1], i % 16, out)
        else:
            B.cas_draft_step_multi(ctx, model, kv, list(range(n_seqs)), [i % 16] * n_seqs, tokens[i].repeat(n_seqs), out)
        if i % 16 == 15:
            for seq in range(n_seqs):
                B.cas_commit(ctx, model, kv, seq, 15)
    return [torch.stack(B.cas_kv_read(ctx, kv, 1, seq, 0, 48, True)) for seq in range(n_seqs)]


@pytest.mark.parametrize("hidden,n_q,n_kv,ffn,keep,blocks,raw", [(264, 4, 2, 520, 600, 400 << 10, True),
                                                                 (2056, 14, 2, 1100, 600, 2500 << 10, True),
                                                                 (8192, 8, 2, 1024, 600, 8 << 20, False),
                                                                 (8199, 16, 4, 1031, 600, 12 << 20, False),
                                                                 (264, 4, 2, 19000, 250, 1 << 20, False),
                                                                 (2600, 64, 8, 14339, 600, 17 << 20, True)])
def test_unary_draft_values_depend_on_neither_company_nor_workspace(env, hidden, n_q, n_kv, ffn, keep, blocks, raw):
    """One, two and four columns through a workspace that holds whole matrices, through one that holds some of them
    (2600: cuts the projection, the gate/up and the down matrix into blocks with smaller last ones, outputs of all
    three kinds) and through one that holds none: the same bits (19000: x of four columns does not fit the LDS).  For a hidden size in eights
    up to 4096 the raw form's fused norm adds in the same order too, so the raw form gives these bits as well."""
    torch = env[0]
    want = None
    for ws, unary in [(80 << 20, True), (blocks, True), (256 << 10, True)] + ([(80 << 20, False)] if raw else []):
        ctx, model, kv = _unary_draft_model(env, hidden, n_q, n_kv, ffn, ws, unary, keep)
        for n_seqs in (1, 2, 4):
            for got in _draft_kv(env, ctx, model, kv, n_seqs):
                want = got if want is None else want
                assert torch.equal(got, want), (ws, unary, n_seqs)


@pytest.mark.parametrize("hidden,n_seqs", [(264, 1), (264, 2), (8199, 1), (8199, 4)])
@pytest.mark.parametrize("field,by", [("smw", 1), ("off_sm", 256), ("off_table", -256), ("off_rowoff", 4), ("off_ue", 256),
                                      ("ue_words", 64), ("spec_bytes", 256)])
def test_unary_draft_pass_refuses_a_layout_that_is_not_the_matrix_s(env, hidden, n_seqs, field, by):
    """Every route of a unary draft product (264 / 8199: with one column the kernel that reads the codes / re-coded
    rows) refuses a descriptor whose layout does not follow from the shape, before a kernel reads by it."""
    torch, B, _ = env
    ctx, model, kv = _unary_draft_model(env, hidden, 4, 2, 520, 32 << 20, True)
    bad = model._unary[(0, 0)]
    setattr(bad.desc, field, getattr(bad.desc, field) + by)
    model.use_unary(0, 0, bad)
    out = torch.empty(4, dtype=torch.int32, device="cuda")
    token = torch.zeros(n_seqs, dtype=torch.int32, device="cuda")
    with pytest.raises(B.CasError) as err:
        if n_seqs == 1:
            B.cas_draft_step(ctx, model, kv, 0, token, 0, out)
        else:
            B.cas_draft_step_multi(ctx, model, kv, list(range(n_seqs)), [0] * n_seqs, token, out)
    assert err.value.code == B.CAS_EINVAL


@pytest.mark.parametrize("keep,t,exp_mode", [(5, 0, 0), (117, 3, 0), (600, 5, 0), (631, 1, 0), (992, 7, 0), (996, 2, 0),
                                             (5, 1, 2), (250, 6, 2), (605, 3, 2), (992, 0, 2)])
@pytest.mark.parametrize("pos0,ntok", [(0, 1), (3, 2), (14, 5), (62, 67), (47, 17)])
def test_online_encoder_at_any_row_of_a_page(env, keep, t, exp_mode, pos0, ntok, heads=3):
    """One to 127 kept values, fields of any width, runs that begin and end inside the four rows of a wave and the
    sixteen of a workgroup: the rows of the run bit for bit like the oracle's, every other byte of the pools as before;
    and the same from vectors that lie at odd multiples of two bytes."""
    torch, B, ctx = env
    rng = np.random.default_rng(keep + 7 * pos0 + ntok)
    K, V = (synth.kv_tensor(ntok, heads, 128, seed=s) for s in (31, 32))
    K[0, 0, :] = 0x3F81                                              # equal magnitudes: the first columns are kept
    K[0, 1, :] = rng.choice([0x3F80, 0xBF80, 0x3F81], 128)           # the line falls among equals, with either sign
    K[0, 2, :] = rng.integers(0, 0x10000, 128)                       # any pattern: NaN, infinities, subnormal values
    V[0, 0, :] = rng.choice([0x7F80, 0xFF80, 0x7FFF, 0xFFFF, 0x0000, 0x8000], 128)
    kv = B.KVCache(ctx, 1, heads, n_pages=4, max_seqs=1, max_pages_per_seq=3, keep_permille=keep, trunc_bits=t,
                   page_table=torch.tensor([[2, 0, 3]], dtype=torch.int32), exp_mode=exp_mode)
    d, page_of = kv.desc, [2, 0, 3]
    packed = [O.encode_kv(x.reshape(-1, 128), keep, t) for x in (K, V)]
    coded = [O.to_mx(p) for p in packed] if exp_mode else None
    for shift in (0, 1):
        kv.spec_pool.fill_(0xA5)
        kv.verif_pool.fill_(0xA5)
        spec, verif = kv.spec_pool.cpu().numpy(), kv.verif_pool.cpu().numpy()
        for tok in range(ntok):
            page, row = page_of[(pos0 + tok) // 64], (pos0 + tok) % 64
            for which in range(2):
                for head in range(heads):
                    tile, i = (page * 2 + which) * heads + head, tok * heads + head
                    ts = spec[tile * d.tile_spec_bytes: (tile + 1) * d.tile_spec_bytes].view("<u4")
                    tv = verif[tile * d.tile_verif_bytes: (tile + 1) * d.tile_verif_bytes].view("<u4")
                    ts[row * 4: row * 4 + 4] = packed[which].bitmap[i]
                    off = 256
                    if exp_mode:
                        ts[256 + row: 257 + row] = np.ascontiguousarray(coded[which].sexp[i]).view("<u4")
                        off = 320
                    fields, lo = (coded[which].field, coded[which].lo) if exp_mode else (packed[which].spec, packed[which].lo)
                    ts[off + row * d.sw: off + (row + 1) * d.sw] = fields[i]
                    tv[row * d.lw: (row + 1) * d.lw] = lo[i]
                    tv[64 * d.lw + row * d.pw: 64 * d.lw + (row + 1) * d.pw] = packed[which].pruned[i]
        def at(x):
            buf = torch.empty(x.size + 1, dtype=torch.int16, device="cuda")
            buf[shift: shift + x.size] = _dev(torch, x).flatten()
            return buf[shift: shift + x.size].view(x.shape)
        B.cas_kv_set_len(kv, 0, pos0)
        B.cas_kv_append(ctx, kv, 0, 0, at(K), at(V))
        np.testing.assert_array_equal(kv.spec_pool.cpu().numpy(), spec)
        np.testing.assert_array_equal(kv.verif_pool.cpu().numpy(), verif)


@pytest.mark.parametrize("keep,t,exp_mode", [(5, 0, 0), (117, 3, 0), (605, 5, 0), (631, 1, 0), (992, 7, 0), (996, 2, 0),
                                             (5, 1, 2), (250, 6, 2), (605, 3, 2), (992, 0, 2)])
@pytest.mark.parametrize("pos0,ntok,heads", [(14, 5, 310), (62, 67, 24), (47, 17, 92)])
def test_online_encoder_of_many_vectors_at_any_row_of_a_page(env, keep, t, exp_mode, pos0, ntok, heads):
    """The same with enough vectors that a wave takes four of them."""
    assert 2 * ntok * heads > 12 * env[0].cuda.get_device_properties(0).multi_processor_count
    test_online_encoder_at_any_row_of_a_page(env, keep, t, exp_mode, pos0, ntok, heads)


@pytest.mark.parametrize("vocab", [1, 2, 63, 65, 1024, 1025, 4095, 4096, 4097, 9001])
def test_token_is_the_first_of_the_largest_logits(env, vocab):
    """One launch up to 4096 tokens, two above: with every row of the head present several times, the first of equal
    maxima, infinite ones too; logits that are NaN beside numbers and infinities are never chosen, nor where all others
    are -Inf; token 0 where all are NaN."""
    from types import SimpleNamespace
    torch, B, _ = env
    hidden, n_q, n_kv, ffn = 256, 4, 2, 256
    gen = torch.Generator(device="cuda")
    gen.manual_seed(vocab)
    bits = lambda x: x.to(torch.bfloat16).view(torch.int16)  # noqa: E731
    rnd = lambda *s: torch.randn(s, device="cuda", generator=gen)  # noqa: E731
    ctx = B.Context(workspace=torch.empty(8 << 20, dtype=torch.uint8, device="cuda"))
    sh = SimpleNamespace(hidden=hidden, n_layers=1, n_q_heads=n_q, n_kv_heads=n_kv, head_dim=128, ffn=ffn, vocab=vocab, rms_eps=1e-5)
    dims = (("wqkv", (n_q + 2 * n_kv) * 128, hidden), ("wo", hidden, n_q * 128), ("wgu", 2 * ffn, hidden), ("wd", hidden, ffn))
    layer = {n: B.cas_encode_weight(ctx, bits(rnd(r, c) * c ** -0.5), 600, 4) for n, r, c in dims}
    layer.update(g_attn=bits(1 + 0.1 * rnd(hidden)), g_ffn=bits(1 + 0.1 * rnd(hidden)))
    rows = rnd(max(1, vocab // 3), hidden)
    rope = torch.from_numpy(synth.rope_table(64, 128, 500000.0)).cuda()
    embed, g = bits(rnd(vocab, hidden)), bits(1 + 0.1 * rnd(hidden))
    for special in ("none", "all", "mixed", "one +", "one -"):
        head = bits(rows[torch.arange(vocab, device="cuda") % rows.shape[0]] * hidden ** -0.5)
        if special == "all":
            head[:] = 0x7F80  # infinities of one sign: products of either sign, sums that are NaN
        elif special == "mixed":  # NaN, infinities of either sign (that of a hidden value) and numbers
            head[1::4] = 0x7F80
            for i in range(4):
                head[4 * i + 2::16, i] = 0x7F80
        elif special != "none":  # all logits infinities of one sign, -Inf with one of the two, but for a NaN in front
            head[:, 5] = 0x7F80 if special == "one +" else -0x80  # 0xFF80
            head[0] = 0x7F80
        head = B.cas_encode_weight(ctx, head.contiguous(), 1000, 0)
        model = B.Model(ctx, sh, [layer], head, embed, g, rope, max_cols=8)
        kv = B.KVCache(ctx, 1, n_kv, n_pages=1, max_seqs=1, max_pages_per_seq=1)
        B.cas_kv_set_len(kv, 0, 0)
        out, logits = torch.full((3,), -7, dtype=torch.int32, device="cuda"), torch.empty((3, vocab), device="cuda")
        tokens = torch.tensor([0, vocab // 2, vocab - 1], dtype=torch.int32, device="cuda")
        B.cas_verify_step(ctx, model, kv, 0, tokens, 2, out, logits)
        seen = logits.cpu().numpy()
        if special == "mixed" and vocab >= 63:
            assert np.isnan(seen).any() and np.isfinite(seen).any() and (seen == np.inf).any() and (seen == -np.inf).any()
        if special.startswith("one"):
            assert np.isnan(seen[:, 0]).all() and np.isinf(seen[:, 1:]).all() and (seen[:, 1:] == seen[:, 1:2]).all()
            if special == "one +":
                first = seen[:, 1:2]
            else:
                np.testing.assert_array_equal(seen[:, 1:2], -first)
        for lg, got in zip(seen, out.cpu().numpy()):
            ok = ~np.isnan(lg)
            want = int(np.flatnonzero(ok & (lg == lg[ok].max()))[0]) if ok.any() else 0
            assert got == want, (special, got, want)
