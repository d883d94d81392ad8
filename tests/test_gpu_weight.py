"""GPU parity of the weight path (encode, decode, draft GEMV, verify GEMM) against the oracle,
through the C ABI."""
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


def _regions(ew):
    d = ew.desc
    sp = ew.spec.cpu().numpy()
    vf = ew.verif.cpu().numpy()
    def reg(buf, off, rows, w):
        return buf[off: off + rows * w * 4].view("<u4").reshape(rows, w) if w else np.zeros((rows, 0), np.uint32)
    return (reg(sp, d.off_bitmap, d.rows, d.bw), reg(sp, d.off_spec, d.rows, d.sw),
            reg(vf, d.off_lo, d.rows, d.lw), reg(vf, d.off_pruned, d.rows, d.pw))


CASES = [
    # rows, cols, keep, t, act
    (37, 77, 600, 4, False),
    (16, 128, 600, 4, False),
    (5, 1, 1000, 4, False),
    (64, 4096, 600, 4, True),
    (33, 2500, 250, 4, True),
    (20, 4100, 600, 0, False),
    (20, 300, 0, 4, False),
    (20, 300, 1000, 7, True),
    (19, 2048, 500, 3, False),
    (8, 14336, 600, 4, True),
]


@pytest.mark.parametrize("rows,cols,keep,t,act", CASES)
def test_encode_decode_bit_exact(env, rows, cols, keep, t, act):
    torch, B, ctx = env
    print(f"case rows={rows} cols={cols} keep={keep} t={t} act={act}", flush=True)
    W = synth.weight_matrix(rows, cols, seed=rows + cols)
    if cols >= 8:
        W[:, 3] = W[:, 5]           # ties inside rows
        W[0, :] = W[0, 0]           # a row of equal magnitudes
    a = synth.act_norm(cols, seed=7) if act else None
    ew = B.cas_encode_weight(ctx, _dev(torch, W), keep, t, None if a is None else torch.from_numpy(a).cuda())
    torch.cuda.synchronize()
    p = O.encode_weight(W, keep, t, a)
    assert (ew.desc.K, ew.desc.bw, ew.desc.sw, ew.desc.lw, ew.desc.pw) == (p.K, *O.stream_words(cols, p.K, t))
    bm, sp, lo, pr = _regions(ew)
    np.testing.assert_array_equal(bm, p.bitmap)
    np.testing.assert_array_equal(sp, p.spec)
    np.testing.assert_array_equal(lo, p.lo)
    np.testing.assert_array_equal(pr, p.pruned)
    full = B.cas_decode_weight(ctx, ew, full=True).cpu().numpy().view(np.uint16)
    draft = B.cas_decode_weight(ctx, ew, full=False).cpu().numpy().view(np.uint16)
    np.testing.assert_array_equal(full, W)
    np.testing.assert_array_equal(draft, O.decode_draft(p))


def _tol(W, X):
    wn = np.linalg.norm(O.bf16_to_f64(W), axis=1)
    xn = np.linalg.norm(O.bf16_to_f64(X), axis=1)
    return wn[None, :] * xn[:, None] + 1e-30


@pytest.mark.parametrize("rows,cols,keep,t,act", CASES)
@pytest.mark.parametrize("batch", [1, 3, 4])
def test_gemv_draft_matches_oracle(env, rows, cols, keep, t, act, batch):
    torch, B, ctx = env
    print(f"case rows={rows} cols={cols} keep={keep} t={t} batch={batch}", flush=True)
    W = synth.weight_matrix(rows, cols, seed=rows + cols)
    a = synth.act_norm(cols, seed=7) if act else None
    X = synth.activations(cols, batch, seed=11)
    ew = B.cas_encode_weight(ctx, _dev(torch, W), keep, t, None if a is None else torch.from_numpy(a).cuda())
    try:
        y = B.cas_gemv_draft(ctx, ew, _dev(torch, X)).cpu().numpy()
    except B.CasError as e:
        if e.code == B.CAS_ENOTSUP:
            pytest.skip("x block does not fit LDS at this width and batch")
        raise
    p = O.encode_weight(W, keep, t, a)
    ref = np.stack([O.gemv_draft(p, X[b]) for b in range(batch)])
    err = np.abs(y - ref) / _tol(W, X)
    # spec bar 2e-3 |W||x|; fp32 accumulation of exact bf16 products stays far below it
    assert err.max() < 2e-3
    assert err.max() < 2e-5, err.max()


@pytest.mark.parametrize("rows,cols,keep,t,act", CASES)
def test_gemm_verify_matches_oracle_and_is_column_invariant(env, rows, cols, keep, t, act):
    torch, B, ctx = env
    print(f"case rows={rows} cols={cols} keep={keep} t={t}", flush=True)
    W = synth.weight_matrix(rows, cols, seed=rows + cols)
    a = synth.act_norm(cols, seed=7) if act else None
    X = synth.activations(cols, 5, seed=12)
    ew = B.cas_encode_weight(ctx, _dev(torch, W), keep, t, None if a is None else torch.from_numpy(a).cuda())
    Xd = _dev(torch, X)
    Y = B.cas_gemm_verify(ctx, ew, Xd).cpu().numpy()
    ref = (O.bf16_to_f64(X) @ O.bf16_to_f64(W).T)          # exact reconstruction => GEMM of W itself
    err = np.abs(Y - ref) / _tol(W, X)
    assert err.max() < 2e-3
    assert err.max() < 2e-5, err.max()
    # a column's value does not depend on how many columns ride along (Sec. 2.2)
    for c in (0, 4):
        y1 = B.cas_gemm_verify(ctx, ew, Xd[c:c + 1].contiguous()).cpu().numpy()
        np.testing.assert_array_equal(y1[0], Y[c])
    Y9 = B.cas_gemm_verify(ctx, ew, torch.cat([Xd, Xd[:4]]).contiguous()).cpu().numpy()
    np.testing.assert_array_equal(Y9[:5], Y)


@pytest.mark.parametrize("rows,cols,keep,t", [(70, 4096, 600, 4), (33, 2500, 250, 0), (300, 300, 1000, 7), (20, 9000, 600, 3)])
@pytest.mark.parametrize("ncols", [9, 16, 20, 32])
def test_gemm_verify_many_columns(env, rows, cols, keep, t, ncols):
    """9 to 32 columns (a second block of output columns above 16):
    against the oracle, and every column bit-identical to the one-column call."""
    torch, B, ctx = env
    print(f"case rows={rows} cols={cols} keep={keep} t={t} ncols={ncols}", flush=True)
    W = synth.weight_matrix(rows, cols, seed=rows + cols)
    X = synth.activations(cols, ncols, seed=13)
    ew = B.cas_encode_weight(ctx, _dev(torch, W), keep, t)
    Xd = _dev(torch, X)
    Y = B.cas_gemm_verify(ctx, ew, Xd).cpu().numpy()
    ref = O.bf16_to_f64(X) @ O.bf16_to_f64(W).T
    err = np.abs(Y - ref) / _tol(W, X)
    assert err.max() < 2e-3
    assert err.max() < 2e-5, err.max()
    for c in sorted({0, 7, 8, 15, 16, ncols - 1} & set(range(ncols))):
        y1 = B.cas_gemm_verify(ctx, ew, Xd[c:c + 1].contiguous()).cpu().numpy()
        np.testing.assert_array_equal(y1[0], Y[c])


def test_config0_full_size_linear_layer(env):
    """W 4096x4096, 0.5 % outlier input columns, 25 % kept, t = 4, one draft GEMV and a
    verify GEMM with k = 4 extra columns."""
    torch, B, ctx = env
    W = synth.weight_matrix(4096, 4096, seed=1)
    X = synth.activations(4096, 5, seed=2)
    ew = B.cas_encode_weight(ctx, _dev(torch, W), 250, 4)
    p = O.encode_weight(W, 250, 4)
    bm, sp, lo, pr = _regions(ew)
    assert np.array_equal(bm, p.bitmap) and np.array_equal(sp, p.spec)
    assert np.array_equal(lo, p.lo) and np.array_equal(pr, p.pruned)
    Xd = _dev(torch, X)
    y = B.cas_gemv_draft(ctx, ew, Xd[:1].contiguous()).cpu().numpy()[0]
    Y = B.cas_gemm_verify(ctx, ew, Xd).cpu().numpy()
    tol = _tol(W, X)
    assert (np.abs(y - O.gemv_draft(p, X[0])) / tol[0]).max() < 2e-5
    assert (np.abs(Y - O.gemm_verify(p, X)) / tol).max() < 2e-5


def test_accept_matches_oracle(env):
    _, B, _ = env
    rng = np.random.default_rng(0)
    for _ in range(200):
        k = int(rng.integers(0, 7))
        d = rng.integers(0, 3, size=k).tolist()
        t = rng.integers(0, 3, size=k + 1).tolist()
        assert B.cas_accept(d, t) == O.accept_greedy(d, t)


@pytest.mark.parametrize("rows,cols", [(64, 300), (96, 4096), (30, 2500)])
def test_fused_draft_gemv_variants_match_oracle(env, rows, cols):
    """RMSNorm prologue, residual epilogue and SwiGLU epilogue of the draft GEMV against the
    oracle's separate operations."""
    torch, B, ctx = env
    W = synth.weight_matrix(rows, cols, seed=5)
    x = synth.normal_bf16((1, cols), 2.0, seed=6)
    g = synth.f32_to_bf16_bits(1.0 + 0.1 * np.random.default_rng(0).standard_normal(cols).astype(np.float32))
    h0 = synth.normal_bf16((1, rows), 1.0, seed=7)
    ew = B.cas_encode_weight(ctx, _dev(torch, W), 600, 4)
    p = O.encode_weight(W, 600, 4)
    xn = O.rmsnorm(x[0], g, 1e-5)
    yref = O.gemv_draft(p, xn)
    tol = _tol(W, xn[None])[0]
    # epilogue 0 with the norm prologue
    y = B.cas_gemv_draft_fused(ctx, ew, _dev(torch, x), y=torch.empty((1, rows), device="cuda"), gain=_dev(torch, g),
                               eps=1e-5).cpu().numpy()[0]
    assert (np.abs(y - yref) / tol).max() < 2e-3
    # epilogue 1: residual update of a bf16 vector (no norm)
    h = _dev(torch, h0.copy())
    B.cas_gemv_draft_fused(ctx, ew, _dev(torch, x), epilogue=1, out16=h)
    href = O.add_bf16(h0[0], O.gemv_draft(p, x[0]))
    got = O.bf16_to_f64(h.cpu().numpy().view(np.uint16)[0])
    assert np.abs(got - O.bf16_to_f64(href)).max() <= 2.0 ** -7 * np.abs(O.bf16_to_f64(href)).max()
    assert (h.cpu().numpy().view(np.uint16)[0] != href).mean() < 0.02     # rare 1-ulp rounding flips only
    # epilogue 2: SwiGLU over row pairs with the norm prologue
    act = torch.zeros((1, rows // 2), dtype=torch.int16, device="cuda")
    B.cas_gemv_draft_fused(ctx, ew, _dev(torch, x), gain=_dev(torch, g), eps=1e-5, epilogue=2, out16=act)
    aref = O.swiglu(yref[0::2], yref[1::2])
    ga = O.bf16_to_f64(act.cpu().numpy().view(np.uint16)[0]); ra = O.bf16_to_f64(aref)
    assert np.abs(ga - ra).max() <= 2.0 ** -6 * np.abs(ra).max() + 1e-6
    assert (act.cpu().numpy().view(np.uint16)[0] != aref).mean() < 0.05


@pytest.mark.parametrize("rows,cols,batch", [(96, 4096, 4), (40, 14336, 3), (64, 300, 2)])
def test_fused_draft_gemv_batch_equals_single_columns(env, rows, cols, batch):
    """Every column of a batched fused call (norm prologue; fp32, residual and SwiGLU epilogues)
    has exactly the bits of the one-column call: sequences decoded together do not influence
    each other.  (One column stages x as fp32, a batch as bf16: the staged values are
    bf16-representable, so nothing changes.)"""
    torch, B, ctx = env
    W = synth.weight_matrix(rows, cols, seed=9)
    X = _dev(torch, synth.normal_bf16((batch, cols), 2.0, seed=10))
    g = _dev(torch, synth.f32_to_bf16_bits(1.0 + 0.1 * np.random.default_rng(1).standard_normal(cols).astype(np.float32)))
    H0 = _dev(torch, synth.normal_bf16((batch, rows), 1.0, seed=12))
    ew = B.cas_encode_weight(ctx, _dev(torch, W), 600, 4)
    yb = B.cas_gemv_draft_fused(ctx, ew, X, y=torch.empty((batch, rows), device="cuda"), gain=g, eps=1e-5)
    hb = H0.clone(); B.cas_gemv_draft_fused(ctx, ew, X, epilogue=1, out16=hb)
    ab = torch.zeros((batch, rows // 2), dtype=torch.int16, device="cuda")
    B.cas_gemv_draft_fused(ctx, ew, X, gain=g, eps=1e-5, epilogue=2, out16=ab)
    for b in range(batch):
        x1 = X[b:b + 1].contiguous()
        y1 = B.cas_gemv_draft_fused(ctx, ew, x1, y=torch.empty((1, rows), device="cuda"), gain=g, eps=1e-5)
        h1 = H0[b:b + 1].clone(); B.cas_gemv_draft_fused(ctx, ew, x1, epilogue=1, out16=h1)
        a1 = torch.zeros((1, rows // 2), dtype=torch.int16, device="cuda")
        B.cas_gemv_draft_fused(ctx, ew, x1, gain=g, eps=1e-5, epilogue=2, out16=a1)
        assert torch.equal(yb[b:b + 1], y1) and torch.equal(hb[b:b + 1], h1) and torch.equal(ab[b:b + 1], a1)


@pytest.mark.parametrize("batch,cols", [(2, 18432), (2, 18433), (3, 12288), (3, 12289), (4, 8192), (4, 8193), (4, 31)])
def test_draft_gemv_batch_keeps_its_bits_on_both_sides_of_the_lds(env, batch, cols):
    """x of a batch is staged as fp32 up to the first of each pair of sizes and as bf16 above it: every column has
    the bits of the one-column call."""
    torch, B, ctx = env
    ew = B.cas_encode_weight(ctx, _dev(torch, synth.weight_matrix(19, cols, seed=9)), 600, 3)
    X = _dev(torch, synth.normal_bf16((batch, cols), 2.0, seed=10))
    got = B.cas_gemv_draft(ctx, ew, X)
    for b in range(batch):
        assert torch.equal(got[b:b + 1], B.cas_gemv_draft(ctx, ew, X[b:b + 1].contiguous()))


def _special_patterns(rows, cols, seed):
    """bf16 words that exercise the selection order and the bit split: +-0, subnormals, the
    largest finite values, +-Inf and NaNs with several payloads, among ordinary values."""
    W = synth.weight_matrix(rows, cols, seed=seed)
    specials = np.array([0x0000, 0x8000, 0x0001, 0x8001, 0x007F, 0x0080, 0x7F7F, 0xFF7F, 0x7F80, 0xFF80,
                         0x7F81, 0x7FC0, 0xFFFF, 0x7FFF, 0x3F80, 0xBF80], dtype=np.uint16)
    rng = np.random.Generator(np.random.Philox(seed))
    idx = rng.integers(0, W.size, size=min(W.size, 6 * len(specials)))
    W.reshape(-1)[idx] = np.resize(specials, idx.shape)
    return W


@pytest.mark.parametrize("rows,cols,keep,t,act", [(24, 200, 600, 4, True), (9, 2100, 250, 0, False),
                                                   (12, 64, 500, 7, True)])
def test_encode_decode_special_values_bit_exact(env, rows, cols, keep, t, act):
    """Selection keys are the raw patterns of the scores (NaN largest, -0 == +0 by magnitude):
    the GPU encoder must pick the same sets as the oracle for every pattern, and the exact
    reconstruction must give back every word, NaN payloads included."""
    torch, B, ctx = env
    print(f"case rows={rows} cols={cols} keep={keep} t={t} act={act}", flush=True)
    W = _special_patterns(rows, cols, seed=91 + cols)
    a = synth.act_norm(cols, seed=3) if act else None
    ew = B.cas_encode_weight(ctx, _dev(torch, W), keep, t, None if a is None else torch.from_numpy(a).cuda())
    torch.cuda.synchronize()
    p = O.encode_weight(W, keep, t, a)
    bm, sp, lo, pr = _regions(ew)
    np.testing.assert_array_equal(bm, p.bitmap)
    np.testing.assert_array_equal(sp, p.spec)
    np.testing.assert_array_equal(lo, p.lo)
    np.testing.assert_array_equal(pr, p.pruned)
    np.testing.assert_array_equal(B.cas_decode_weight(ctx, ew, full=True).cpu().numpy().view(np.uint16), W)
    np.testing.assert_array_equal(B.cas_decode_weight(ctx, ew, full=False).cpu().numpy().view(np.uint16),
                                  O.decode_draft(p))


def test_empty_matrix_is_accepted(env):
    """rows = 0: the descriptor has empty streams and every call returns without launching."""
    torch, B, ctx = env
    W = torch.empty((0, 256), dtype=torch.int16, device="cuda")
    ew = B.cas_encode_weight(ctx, W, 600, 4)
    assert ew.desc.rows == 0 and ew.desc.K == O.kept_count(256, 600)
    x = _dev(torch, synth.activations(256, 2, seed=1))
    assert B.cas_gemv_draft(ctx, ew, x[:1].contiguous()).shape == (1, 0)
    assert B.cas_gemm_verify(ctx, ew, x).shape == (2, 0)
    assert B.cas_decode_weight(ctx, ew, full=True).shape == (0, 256)


@pytest.mark.parametrize("rows,cols", [(40, 4096), (7, 14336), (300, 64), (5, 8), (1000, 1032), (33, 28672)])
def test_dense_bf16_baseline_gemv(env, rows, cols):
    """The uncompressed baseline kernel against the plain definition y = W x."""
    torch, B, ctx = env
    W = synth.weight_matrix(rows, cols, seed=rows + cols)
    x = synth.activations(cols, 1, seed=3)
    y = B.cas_gemv_bf16(ctx, _dev(torch, W), _dev(torch, x[0])).cpu().numpy()
    ref = O.gemv(W, x[0])
    err = np.abs(y - ref) / _tol(W, x)[0]
    assert err.max() < 2e-5, err.max()


def test_dense_bf16_baseline_rejects_unaligned_rows(env):
    torch, B, ctx = env
    W = _dev(torch, synth.weight_matrix(4, 77, seed=1))
    x = _dev(torch, synth.activations(77, 1, seed=2)[0])
    with pytest.raises(B.CasError) as e:
        B.cas_gemv_bf16(ctx, W, x)
    assert e.value.code == B.CAS_ENOTSUP
    assert B.cas_gemv_bf16(ctx, torch.empty((0, 64), dtype=torch.int16, device="cuda"),
                           torch.zeros(64, dtype=torch.int16, device="cuda")).shape == (0,)


@pytest.mark.parametrize("cols,keep,t", [(96, 600, 4), (160, 250, 3), (2112, 600, 4), (72, 500, 1)])
def test_draft_gemv_rows_do_not_see_their_neighbours(env, cols, keep, t):
    """A lane that has walked all of its kept values keeps forming products with the zero entry of x;
    the weight bits it pairs with must come from its own row (or be zero).  Rows whose field stream
    does not end on a word boundary (K (16 - t) not a multiple of 32), followed by rows full of
    Inf / NaN / large values: the finite rows must give the oracle's finite result."""
    torch, B, ctx = env
    rows = 48
    K = O.kept_count(cols, keep)
    assert (K * (16 - t)) % 32 != 0
    W = synth.weight_matrix(rows, cols, seed=31)
    W[1::3] = 0x7F80                       # +Inf rows
    W[2::3] = 0x7FC1                       # NaN rows
    W[2::3, ::2] = 0xFF7F                  # ... mixed with the largest finite magnitude, negative
    X = synth.activations(cols, 1, seed=32)
    ew = B.cas_encode_weight(ctx, _dev(torch, W), keep, t)
    y = B.cas_gemv_draft(ctx, ew, _dev(torch, X)).cpu().numpy()[0]
    ref = O.gemv_draft(O.encode_weight(W, keep, t), X[0])
    good = np.arange(0, rows, 3)
    assert np.isfinite(ref[good]).all() and np.isfinite(y[good]).all()
    wn = np.linalg.norm(O.bf16_to_f64(W[good]), axis=1) * np.linalg.norm(O.bf16_to_f64(X[0]))
    assert (np.abs(y[good] - ref[good]) <= 2e-5 * wn).all()
    assert not np.isfinite(y[1::3]).any() and np.isnan(y[2::3]).all()


@pytest.mark.parametrize("rows,cols", [(4803, 131), (4800, 640), (40, 7), (40, 129), (40, 1026), (33, 8199), (16, 8192 + 136)])
@pytest.mark.parametrize("ncols", [1, 5, 17, 32])
def test_verification_gemm_at_the_ends_of_x(rows, cols, ncols):
    """Rows cut into 4, 8 and 16 parts, row lengths around words, pieces of 8 and blocks of 128, X from an aligned
    address and from the middle of a word: the reference's products, the same bits from both addresses, and nothing of
    a column's neighbours (its last pieces are read across its end; the neighbour is set to NaN)."""
    import torch
    from paper_2605_26558_amd import binding as B
    ctx = B.Context()
    W = synth.weight_matrix(rows, cols, seed=rows + cols)
    X = synth.activations(cols, ncols, seed=cols + ncols)
    ew = B.cas_encode_weight(ctx, torch.from_numpy(W.view(np.int16)).cuda(), 600, 4)
    xd = torch.from_numpy(X.view(np.int16)).cuda()
    y = B.cas_gemm_verify(ctx, ew, xd).cpu().numpy()
    w64, x64 = O.bf16_to_f64(W), O.bf16_to_f64(X)
    bar = 2e-5 * np.linalg.norm(w64, axis=1)[None, :] * np.linalg.norm(x64, axis=1)[:, None] + 1e-30
    assert (np.abs(y - x64 @ w64.T) <= bar).all()
    buf = torch.full((ncols * cols + 1,), 0x7FC0, dtype=torch.int16, device="cuda")
    buf[1:] = xd.reshape(-1)
    np.testing.assert_array_equal(B.cas_gemm_verify(ctx, ew, buf[1:].view(ncols, cols)).cpu().numpy(), y)
    if ncols > 1:
        for c in (0, ncols - 1):
            xn = xd.clone()
            xn[[k for k in range(ncols) if k != c]] = 0x7FC0
            np.testing.assert_array_equal(B.cas_gemm_verify(ctx, ew, xn).cpu().numpy()[c], y[c])


@pytest.mark.parametrize("cols", [1, 63, 257, 1000, 1024, 1025, 2048, 2049, 4095, 4096, 4097])
@pytest.mark.parametrize("keep,t", [(600, 4), (1000, 0), (3, 7), (250, 3)])
def test_draft_gemv_of_one_column_whatever_form_its_x_has(env, cols, keep, t):
    """The form for one column of up to 4096 values and the one beside it, words with all, some and no kept values:
    the bits of the same column in company."""
    torch, B, ctx = env
    rows = 37
    W = synth.weight_matrix(rows, cols, seed=41)
    W[3, :] = 0x3F80                         # equal scores: the first columns are kept, the words behind them are empty
    x = synth.activations(cols, 2, seed=42)
    ew = B.cas_encode_weight(ctx, _dev(torch, W), keep, t)
    pair = B.cas_gemv_draft(ctx, ew, _dev(torch, x))
    one = B.cas_gemv_draft(ctx, ew, _dev(torch, x[:1]))
    assert torch.equal(one[0], pair[0])
    assert torch.equal(B.cas_gemv_draft(ctx, ew, _dev(torch, x[1:]))[0], pair[1])
    ref = O.gemv_draft(O.encode_weight(W, keep, t), x[0])
    wn, xn = np.linalg.norm(O.bf16_to_f64(W), axis=1), np.linalg.norm(O.bf16_to_f64(x[0]))
    # fp32 sums of exact products: cols * 2^-24 |W| |x| at worst
    assert (np.abs(one.cpu().numpy()[0] - ref) <= cols * 2.0 ** -24 * wn * xn).all()
