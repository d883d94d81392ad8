"""GPU parity of the compressed KV cache (online encode, read-back) and of draft / verify
attention against the oracle, through the C ABI."""
import numpy as np
import pytest

from oracle import cassandra_oracle as O
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    from paper_2605_26558_amd import binding as B
    ws = torch.empty(64 << 20, dtype=torch.uint8, device="cuda")
    return torch, B, B.Context(workspace=ws)


def _dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).cuda()


def _host(t):
    return t.cpu().numpy().view(np.uint16)


@pytest.mark.parametrize("keep,t", [(600, 4), (1000, 4), (250, 0), (0, 4), (500, 7)])
def test_kv_append_is_bit_exact(env, keep, t):
    torch, B, ctx = env
    print(f"case keep={keep} t={t}", flush=True)
    heads, layers, ntok = 2, 2, 75
    perm = torch.tensor([[3, 0, 2, 1]], dtype=torch.int32)          # a non-trivial page table
    kv = B.KVCache(ctx, layers, heads, n_pages=4, max_seqs=1, max_pages_per_seq=4, keep_permille=keep,
                   trunc_bits=t, page_table=perm)
    Kh = synth.kv_tensor(ntok, heads, 128, seed=1)
    Vh = synth.kv_tensor(ntok, heads, 128, seed=2, outlier_channels=0)
    Kh[5, 0, :] = Kh[5, 0, 0]                                        # all-equal magnitudes: tie rule
    Kh[6, 1, 10] = Kh[6, 1, 90]
    for layer in range(layers):
        B.cas_kv_append(ctx, kv, layer, 0, _dev(torch, Kh[:70]), _dev(torch, Vh[:70]))
    B.cas_kv_set_len(kv, 0, 70)
    for layer in range(layers):
        B.cas_kv_append(ctx, kv, layer, 0, _dev(torch, Kh[70:]), _dev(torch, Vh[70:]))
    B.cas_kv_set_len(kv, 0, ntok)
    assert B.cas_kv_len(kv, 0) == ntok
    for layer in range(layers):
        Kf, Vf = B.cas_kv_read(ctx, kv, layer, 0, 0, ntok, full=True)
        np.testing.assert_array_equal(_host(Kf), Kh)
        np.testing.assert_array_equal(_host(Vf), Vh)
        Kd, Vd = B.cas_kv_read(ctx, kv, layer, 0, 0, ntok, full=False)
        pk = O.encode_kv(Kh.reshape(-1, 128), keep, t)
        pv = O.encode_kv(Vh.reshape(-1, 128), keep, t)
        np.testing.assert_array_equal(_host(Kd).reshape(-1, 128), O.decode_draft(pk))
        np.testing.assert_array_equal(_host(Vd).reshape(-1, 128), O.decode_draft(pv))
    # raw streams of one tile against the oracle's packing (layer 1, K, head 1, page slot 0 -> page 3)
    d = kv.desc
    spec = kv.spec_pool.cpu().numpy()
    verif = kv.verif_pool.cpu().numpy()
    tile = ((1 * d.n_pages + 3) * 2 + 0) * heads + 1
    ts = spec[tile * d.tile_spec_bytes: (tile + 1) * d.tile_spec_bytes].view("<u4")
    tv = verif[tile * d.tile_verif_bytes: (tile + 1) * d.tile_verif_bytes].view("<u4")
    p = O.encode_kv(Kh[:64, 1, :], keep, t)
    np.testing.assert_array_equal(ts[: 64 * 4].reshape(64, 4), p.bitmap)
    np.testing.assert_array_equal(ts[64 * 4: 64 * (4 + d.sw)].reshape(64, d.sw), p.spec)
    np.testing.assert_array_equal(tv[: 64 * d.lw].reshape(64, d.lw), p.lo)
    np.testing.assert_array_equal(tv[64 * d.lw: 64 * (d.lw + d.pw)].reshape(64, d.pw), p.pruned)
    assert (d.K, d.sw, d.lw, d.pw) == (p.K, *O.stream_words(128, p.K, t)[1:])


def _ref_attention(Q, Kc, Vc, Kn, Vn, ncols, nq, nkv):
    """Column c sees the cache and in-flight vectors 0 .. n_new - ncols + c."""
    out = np.zeros((ncols, nq, 128), dtype=np.uint16)
    n_new = Kn.shape[0]
    for c in range(ncols):
        vis = n_new - ncols + c + 1
        k = np.concatenate([Kc, Kn[:vis]], axis=0)
        v = np.concatenate([Vc, Vn[:vis]], axis=0)
        out[c] = O.attention(Q[c], k, v, nq, nkv)
    return out


def _attn_tol(Q, Kc, Vc, Kn, Vn, ncols, nq, nkv, ref):
    """2e-3 |p| |V_d| per channel plus half a bf16 ulp of the rounded output."""
    grp = nq // nkv
    n_new = Kn.shape[0]
    tol = np.zeros(ref.shape)
    for c in range(ncols):
        vis = n_new - ncols + c + 1
        k = O.bf16_to_f64(np.concatenate([Kc, Kn[:vis]], axis=0))
        v = O.bf16_to_f64(np.concatenate([Vc, Vn[:vis]], axis=0))
        q = O.bf16_to_f64(Q[c])
        for h in range(nq):
            s = k[:, h // grp, :] @ q[h] / np.sqrt(128.0)
            p = np.exp(s - s.max()); p /= p.sum()
            tol[c, h] = 2e-3 * np.linalg.norm(p) * np.linalg.norm(v[:, h // grp, :], axis=0)
    return tol + 2.0 ** -8 * np.abs(ref)


@pytest.mark.parametrize("len_cache,ncols,n_new,full", [
    (150, 1, 1, False), (150, 1, 3, False), (0, 1, 1, False), (64, 1, 2, False), (1, 1, 1, False),
    (150, 5, 5, True), (0, 3, 3, True), (130, 7, 7, True), (200, 9, 9, True), (63, 1, 1, True),
])
def test_attention_matches_oracle(env, len_cache, ncols, n_new, full):
    torch, B, ctx = env
    print(f"case len={len_cache} ncols={ncols} n_new={n_new} full={full}", flush=True)
    nq, nkv, layers = 8, 2, 2
    kv = B.KVCache(ctx, layers, nkv, n_pages=8, max_seqs=2, max_pages_per_seq=4,
                   page_table=torch.tensor([[5, 1, 7, 2], [0, 3, 4, 6]], dtype=torch.int32))
    seq, layer = 1, 1
    Kh = synth.kv_tensor(max(len_cache, 1), nkv, 128, seed=3)
    Vh = synth.kv_tensor(max(len_cache, 1), nkv, 128, seed=4, outlier_channels=0)
    if len_cache:
        B.cas_kv_append(ctx, kv, layer, seq, _dev(torch, Kh[:len_cache]), _dev(torch, Vh[:len_cache]))
    B.cas_kv_set_len(kv, seq, len_cache)
    Q = synth.normal_bf16((ncols, nq, 128), 1.0, seed=5)
    Kn = synth.kv_tensor(n_new, nkv, 128, seed=6)
    Vn = synth.kv_tensor(n_new, nkv, 128, seed=7, outlier_channels=0)
    out = _host(B.cas_attention(ctx, kv, layer, seq, full, _dev(torch, Q), _dev(torch, Kn), _dev(torch, Vn)))
    if len_cache:
        pk = O.encode_kv(Kh[:len_cache].reshape(-1, 128), 600, 4)
        pv = O.encode_kv(Vh[:len_cache].reshape(-1, 128), 600, 4)
        dec = O.decode_full if full else O.decode_draft
        Kc = dec(pk).reshape(len_cache, nkv, 128)
        Vc = dec(pv).reshape(len_cache, nkv, 128)
    else:
        Kc = np.zeros((0, nkv, 128), np.uint16); Vc = Kc.copy()
    ref = _ref_attention(Q, Kc, Vc, Kn, Vn, ncols, nq, nkv)
    reff = O.bf16_to_f64(ref)
    err = np.abs(O.bf16_to_f64(out) - reff)
    tol = _attn_tol(Q, Kc, Vc, Kn, Vn, ncols, nq, nkv, reff)
    assert (err <= tol).all(), float((err / tol).max())
    print("max err / tol", float((err / tol).max()), flush=True)
    if full and ncols > 1:
        # a column's output does not depend on how many columns are verified together
        for c in (0, ncols - 1):
            vis = n_new - ncols + c + 1
            o1 = _host(B.cas_attention(ctx, kv, layer, seq, True, _dev(torch, Q[c:c + 1]),
                                       _dev(torch, Kn[:vis]), _dev(torch, Vn[:vis])))
            np.testing.assert_array_equal(o1[0], out[c])


@pytest.mark.parametrize("length", [2047, 2048, 16383, 16384, 32767, 32768])
def test_attention_merge_of_few_and_of_many_pages(env, length):
    """Partial results of 32 / 33, 256 / 257 and 512 / 513 pages, the ends of what a merge takes in one go, against
    the oracle; next to another sequence of the same launch the bits are the same (the two forms of the merge are
    compared in the next test)."""
    torch, B, ctx = env
    nq, nkv = 4, 2
    kv = B.KVCache(ctx, 1, nkv, n_pages=1100, max_seqs=2, max_pages_per_seq=550)
    Kh, Vh = synth.kv_tensor(length, nkv, 128, seed=3), synth.kv_tensor(length, nkv, 128, seed=4, outlier_channels=0)
    for seq in (0, 1):
        B.cas_kv_append(ctx, kv, 0, seq, _dev(torch, Kh), _dev(torch, Vh))
    B.cas_kv_set_len(kv, 0, length)
    B.cas_kv_set_len(kv, 1, 1 if length > 4000 else length)
    Q, Kn, Vn = (synth.normal_bf16((1, n, 128), 1.0, seed=5 + n) for n in (nq, nkv, nkv))
    args = [_dev(torch, x) for x in (Q, Kn, Vn)]
    out = _host(B.cas_attention(ctx, kv, 0, 0, True, *args))
    ref = _ref_attention(Q, Kh, Vh, Kn, Vn, 1, nq, nkv)
    reff = O.bf16_to_f64(ref)
    assert (np.abs(O.bf16_to_f64(out) - reff) <= _attn_tol(Q, Kh, Vh, Kn, Vn, 1, nq, nkv, reff)).all()
    alone = [_host(B.cas_attention(ctx, kv, 0, seq, True, *args)) for seq in (0, 1)]
    both = B.cas_attention_multi(ctx, kv, 0, [0, 1], True, [args[0]] * 2, [args[1]] * 2, [args[2]] * 2)
    for one, two in zip(alone, both):
        np.testing.assert_array_equal(one, _host(two))


@pytest.mark.parametrize("full,ncols", [(False, 1), (False, 9), (True, 1), (True, 9)])
@pytest.mark.parametrize("pages", [2, 8, 9, 31, 32])
def test_a_row_has_the_same_bits_from_the_merge_of_few_and_of_many_pages(env, pages, full, ncols):
    """Up to 32 pages a call alone takes the merge for few pages; next to a sequence of 40 pages the other form combines
    the same partial results.  The pages of a pair cancel (equal keys, opposite values) and what is left is 2^-12 of
    them, so that the order of the additions shows in the outputs: from 9 pages on, adding the splits one after the
    other, in parts of neighbours or in four parts instead of eight changes 3 to 6 % of them (in numpy)."""
    torch, B, ctx = env
    nq, nkv, length = 8, 2, 64 * pages - ncols
    kv = B.KVCache(ctx, 1, nkv, n_pages=96, max_seqs=2, max_pages_per_seq=48)
    K, V = synth.normal_bf16((length, nkv, 128), 1.0, seed=3), synth.normal_bf16((length, nkv, 128), 2.0 ** -12, seed=4)
    for first in range(0, (pages - 1) // 2 * 128, 128):
        K[first + 64:first + 128] = K[first:first + 64]
        V[first:first + 64] = synth.normal_bf16((64, nkv, 128), 1.0, seed=5 + first)
        V[first + 64:first + 128] = V[first:first + 64] ^ 0x8000
    B.cas_kv_append(ctx, kv, 0, 0, _dev(torch, K), _dev(torch, V))
    B.cas_kv_set_len(kv, 0, length)
    other = synth.normal_bf16((40 * 64 - ncols, nkv, 128), 1.0, seed=6)
    B.cas_kv_append(ctx, kv, 0, 1, _dev(torch, other), _dev(torch, other))
    B.cas_kv_set_len(kv, 1, len(other))
    args = [_dev(torch, x) for x in (synth.normal_bf16((ncols, nq, 128), 0.3, seed=7),
                                     synth.normal_bf16((ncols, nkv, 128), 1.0, seed=8),
                                     synth.normal_bf16((ncols, nkv, 128), 2.0 ** -12, seed=9))]
    alone = [_host(B.cas_attention(ctx, kv, 0, seq, full, *args)) for seq in (0, 1)]
    both = B.cas_attention_multi(ctx, kv, 0, [0, 1], full, [args[0]] * 2, [args[1]] * 2, [args[2]] * 2)
    for one, two in zip(alone, both):
        np.testing.assert_array_equal(one, _host(two))


def test_attention_llama70b_head_grouping(env):
    """64 query heads on 8 kv heads (group of 8), 9 verification columns = 72 query rows per
    kv head, and the matching one-column draft call."""
    torch, B, ctx = env
    nq, nkv = 64, 8
    kv = B.KVCache(ctx, 1, nkv, n_pages=3, max_seqs=1, max_pages_per_seq=3)
    L = 100
    Kh = synth.kv_tensor(L, nkv, 128, seed=13)
    Vh = synth.kv_tensor(L, nkv, 128, seed=14, outlier_channels=0)
    B.cas_kv_append(ctx, kv, 0, 0, _dev(torch, Kh), _dev(torch, Vh))
    B.cas_kv_set_len(kv, 0, L)
    pk = O.encode_kv(Kh.reshape(-1, 128), 600, 4); pv = O.encode_kv(Vh.reshape(-1, 128), 600, 4)
    for ncols, full in ((9, True), (1, False)):
        Q = synth.normal_bf16((ncols, nq, 128), 0.5, seed=15)
        Kn = synth.kv_tensor(ncols, nkv, 128, seed=16)
        Vn = synth.kv_tensor(ncols, nkv, 128, seed=17, outlier_channels=0)
        out = _host(B.cas_attention(ctx, kv, 0, 0, full, _dev(torch, Q), _dev(torch, Kn), _dev(torch, Vn)))
        dec = O.decode_full if full else O.decode_draft
        Kc = dec(pk).reshape(L, nkv, 128); Vc = dec(pv).reshape(L, nkv, 128)
        ref = _ref_attention(Q, Kc, Vc, Kn, Vn, ncols, nq, nkv)
        reff = O.bf16_to_f64(ref)
        err = np.abs(O.bf16_to_f64(out) - reff)
        tol = _attn_tol(Q, Kc, Vc, Kn, Vn, ncols, nq, nkv, reff)
        assert (err <= tol).all(), float((err / tol).max())


def test_kv_append_special_values_and_empty_append(env):
    """Vectors holding +-0, subnormals, Inf and NaN patterns go through the online encoder bit
    for bit like the oracle's; appending zero tokens changes nothing."""
    torch, B, ctx = env
    heads, ntok = 2, 9
    kv = B.KVCache(ctx, 1, heads, n_pages=1, max_seqs=1, max_pages_per_seq=1)
    Kh = synth.kv_tensor(ntok, heads, 128, seed=21)
    Vh = synth.kv_tensor(ntok, heads, 128, seed=22, outlier_channels=0)
    specials = np.array([0x0000, 0x8000, 0x0001, 0x807F, 0x7F7F, 0x7F80, 0xFF80, 0x7FC0, 0xFFFF, 0x7F81],
                        dtype=np.uint16)
    Kh[1, 0, 5:15] = specials
    Vh[2, 1, 100:110] = specials
    Kh[3, 1, :] = 0x8000                       # a vector of negative zeros: all keys equal
    Vh[4, 0, :] = 0x7FC0                       # a vector of NaNs
    empty = torch.empty((0, heads, 128), dtype=torch.int16, device="cuda")
    B.cas_kv_append(ctx, kv, 0, 0, empty, empty)
    B.cas_kv_append(ctx, kv, 0, 0, _dev(torch, Kh), _dev(torch, Vh))
    B.cas_kv_set_len(kv, 0, ntok)
    B.cas_kv_append(ctx, kv, 0, 0, empty, empty)
    Kf, Vf = B.cas_kv_read(ctx, kv, 0, 0, 0, ntok, full=True)
    np.testing.assert_array_equal(_host(Kf), Kh)
    np.testing.assert_array_equal(_host(Vf), Vh)
    Kd, Vd = B.cas_kv_read(ctx, kv, 0, 0, 0, ntok, full=False)
    np.testing.assert_array_equal(_host(Kd).reshape(-1, 128), O.decode_draft(O.encode_kv(Kh.reshape(-1, 128), 600, 4)))
    np.testing.assert_array_equal(_host(Vd).reshape(-1, 128), O.decode_draft(O.encode_kv(Vh.reshape(-1, 128), 600, 4)))


@pytest.mark.parametrize("nq,nkv,ncols,full,keep,t", [
    (3, 3, 1, False, 600, 4),      # one query head per kv head, odd head count
    (3, 3, 16, True, 600, 4),      # the largest number of columns
    (6, 3, 4, False, 600, 4),      # four draft columns of a group of two (a multi-sequence draft shape)
    (16, 1, 5, True, 1000, 0),     # one kv head for sixteen query heads = 80 query rows; nothing pruned or truncated
    (16, 1, 3, False, 250, 4),     # 48 draft rows; a quarter kept
    (8, 2, 7, True, 500, 7),       # sign and exponent only in the speculation data
])
def test_attention_head_layouts_and_cache_formats(env, nq, nkv, ncols, full, keep, t):
    torch, B, ctx = env
    print(f"case nq={nq} nkv={nkv} ncols={ncols} full={full} keep={keep} t={t}", flush=True)
    L = 200
    kv = B.KVCache(ctx, 1, nkv, n_pages=5, max_seqs=1, max_pages_per_seq=5, keep_permille=keep, trunc_bits=t)
    Kh = synth.kv_tensor(L, nkv, 128, seed=23)
    Vh = synth.kv_tensor(L, nkv, 128, seed=24, outlier_channels=0)
    B.cas_kv_append(ctx, kv, 0, 0, _dev(torch, Kh), _dev(torch, Vh))
    B.cas_kv_set_len(kv, 0, L)
    Q = synth.normal_bf16((ncols, nq, 128), 0.7, seed=25)
    Kn = synth.kv_tensor(ncols, nkv, 128, seed=26)
    Vn = synth.kv_tensor(ncols, nkv, 128, seed=27, outlier_channels=0)
    out = _host(B.cas_attention(ctx, kv, 0, 0, full, _dev(torch, Q), _dev(torch, Kn), _dev(torch, Vn)))
    pk = O.encode_kv(Kh.reshape(-1, 128), keep, t); pv = O.encode_kv(Vh.reshape(-1, 128), keep, t)
    dec = O.decode_full if full else O.decode_draft
    Kc = dec(pk).reshape(L, nkv, 128); Vc = dec(pv).reshape(L, nkv, 128)
    ref = _ref_attention(Q, Kc, Vc, Kn, Vn, ncols, nq, nkv)
    reff = O.bf16_to_f64(ref)
    err = np.abs(O.bf16_to_f64(out) - reff)
    tol = _attn_tol(Q, Kc, Vc, Kn, Vn, ncols, nq, nkv, reff)
    assert (err <= tol).all(), float((err / tol).max())
    # the last column alone gets the bits it gets in company
    o1 = _host(B.cas_attention(ctx, kv, 0, 0, full, _dev(torch, Q[ncols - 1:]), _dev(torch, Kn), _dev(torch, Vn)))
    np.testing.assert_array_equal(o1[0], out[ncols - 1])


# ---- the cache in the shared-exponent form (Sec. 4.2, the MX approach; Sec. 5.1 encoder) ----------

@pytest.mark.parametrize("keep,t", [(600, 4), (1000, 4), (250, 0), (0, 4), (500, 7)])
def test_kv_append_shared_exponents_is_bit_exact(env, keep, t):
    """Online formatting with shared exponents: every region of a tile against the oracle's
    re-coding of the same vectors, and both read-backs (converted vector / draft view)."""
    torch, B, ctx = env
    print(f"case keep={keep} t={t}", flush=True)
    heads, layers, ntok = 2, 2, 75
    perm = torch.tensor([[3, 0, 2, 1]], dtype=torch.int32)
    kv = B.KVCache(ctx, layers, heads, n_pages=4, max_seqs=1, max_pages_per_seq=4, keep_permille=keep,
                   trunc_bits=t, page_table=perm, exp_mode=B.CAS_EXP_SHARED)
    Kh = synth.kv_tensor(ntok, heads, 128, seed=1)
    Vh = synth.kv_tensor(ntok, heads, 128, seed=2, outlier_channels=0)
    Kh[5, 0, :] = Kh[5, 0, 0]
    specials = np.array([0x0000, 0x8000, 0x0001, 0x807F, 0x7F7F, 0x7F80, 0xFF80, 0x7FC0, 0xFFFF, 0x0080],
                        dtype=np.uint16)
    Kh[7, 1, 30:40] = specials                                       # spans two blocks
    Vh[8, 0, :] = 0x0003                                             # a vector of subnormals
    for layer in range(layers):
        B.cas_kv_append(ctx, kv, layer, 0, _dev(torch, Kh[:70]), _dev(torch, Vh[:70]))
    B.cas_kv_set_len(kv, 0, 70)
    for layer in range(layers):
        B.cas_kv_append(ctx, kv, layer, 0, _dev(torch, Kh[70:]), _dev(torch, Vh[70:]))
    B.cas_kv_set_len(kv, 0, ntok)
    mk = O.to_mx(O.encode_kv(Kh.reshape(-1, 128), keep, t))
    mv = O.to_mx(O.encode_kv(Vh.reshape(-1, 128), keep, t))
    for layer in range(layers):
        Kf, Vf = B.cas_kv_read(ctx, kv, layer, 0, 0, ntok, full=True)
        np.testing.assert_array_equal(_host(Kf).reshape(-1, 128), O.decode_full_mx(mk))
        np.testing.assert_array_equal(_host(Vf).reshape(-1, 128), O.decode_full_mx(mv))
        Kd, Vd = B.cas_kv_read(ctx, kv, layer, 0, 0, ntok, full=False)
        np.testing.assert_array_equal(_host(Kd).reshape(-1, 128), O.decode_draft_mx(mk))
        np.testing.assert_array_equal(_host(Vd).reshape(-1, 128), O.decode_draft_mx(mv))
    d = kv.desc
    spec = kv.spec_pool.cpu().numpy()
    verif = kv.verif_pool.cpu().numpy()
    tile = ((1 * d.n_pages + 3) * 2 + 0) * heads + 1                  # layer 1, K, head 1, page slot 0 -> page 3
    ts = spec[tile * d.tile_spec_bytes: (tile + 1) * d.tile_spec_bytes].view("<u4")
    tv = verif[tile * d.tile_verif_bytes: (tile + 1) * d.tile_verif_bytes].view("<u4")
    p = O.encode_kv(Kh[:64, 1, :], keep, t)
    m = O.to_mx(p)
    assert d.sw == m.field.shape[1] and d.lw == m.lo.shape[1]
    np.testing.assert_array_equal(ts[: 64 * 4].reshape(64, 4), p.bitmap)
    np.testing.assert_array_equal(ts[64 * 4: 64 * 5].view(np.uint8).reshape(64, 4), m.sexp)
    np.testing.assert_array_equal(ts[64 * 5: 64 * (5 + d.sw)].reshape(64, d.sw), m.field)
    np.testing.assert_array_equal(tv[: 64 * d.lw].reshape(64, d.lw), m.lo)
    np.testing.assert_array_equal(tv[64 * d.lw: 64 * (d.lw + d.pw)].reshape(64, d.pw), p.pruned)


@pytest.mark.parametrize("len_cache,ncols,n_new,full", [
    (150, 1, 1, False), (150, 1, 3, False), (64, 1, 2, False), (1, 1, 1, False),
    (150, 5, 5, True), (130, 7, 7, True), (200, 9, 9, True), (63, 1, 1, True),
])
def test_attention_over_a_shared_exponent_cache_matches_oracle(env, len_cache, ncols, n_new, full):
    torch, B, ctx = env
    print(f"case len={len_cache} ncols={ncols} n_new={n_new} full={full}", flush=True)
    nq, nkv, layers = 8, 2, 2
    kv = B.KVCache(ctx, layers, nkv, n_pages=8, max_seqs=2, max_pages_per_seq=4,
                   page_table=torch.tensor([[5, 1, 7, 2], [0, 3, 4, 6]], dtype=torch.int32),
                   exp_mode=B.CAS_EXP_SHARED)
    seq, layer = 1, 1
    Kh = synth.kv_tensor(len_cache, nkv, 128, seed=3)
    Vh = synth.kv_tensor(len_cache, nkv, 128, seed=4, outlier_channels=0)
    B.cas_kv_append(ctx, kv, layer, seq, _dev(torch, Kh), _dev(torch, Vh))
    B.cas_kv_set_len(kv, seq, len_cache)
    Q = synth.normal_bf16((ncols, nq, 128), 1.0, seed=5)
    Kn = synth.kv_tensor(n_new, nkv, 128, seed=6)
    Vn = synth.kv_tensor(n_new, nkv, 128, seed=7, outlier_channels=0)
    out = _host(B.cas_attention(ctx, kv, layer, seq, full, _dev(torch, Q), _dev(torch, Kn), _dev(torch, Vn)))
    mk = O.to_mx(O.encode_kv(Kh.reshape(-1, 128), 600, 4))
    mv = O.to_mx(O.encode_kv(Vh.reshape(-1, 128), 600, 4))
    dec = O.decode_full_mx if full else O.decode_draft_mx
    Kc = dec(mk).reshape(len_cache, nkv, 128)
    Vc = dec(mv).reshape(len_cache, nkv, 128)
    ref = _ref_attention(Q, Kc, Vc, Kn, Vn, ncols, nq, nkv)
    reff = O.bf16_to_f64(ref)
    err = np.abs(O.bf16_to_f64(out) - reff)
    tol = _attn_tol(Q, Kc, Vc, Kn, Vn, ncols, nq, nkv, reff)
    assert (err <= tol).all(), float((err / tol).max())
    if full and ncols > 1:
        for c in (0, ncols - 1):
            vis = n_new - ncols + c + 1
            o1 = _host(B.cas_attention(ctx, kv, layer, seq, True, _dev(torch, Q[c:c + 1]),
                                       _dev(torch, Kn[:vis]), _dev(torch, Vn[:vis])))
            np.testing.assert_array_equal(o1[0], out[c])


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("full", [False, True])
def test_a_query_row_has_the_same_bits_whatever_rows_ride_along(env, full, shared):
    """Row counts on both sides of every line between the forms of the products (4, 8, 16, 24, 32, 48, 64 rows of a kv
    head): the rows of the widest call, which has one form, are those of every narrower one.  A page of committed
    positions alone and one with positions in flight."""
    torch, B, ctx = env
    length, most = 119, 80 if full else 48
    kv = B.KVCache(ctx, 1, 1, n_pages=2, max_seqs=1, max_pages_per_seq=2,
                   exp_mode=B.CAS_EXP_SHARED if shared else B.CAS_EXP_RAW)
    g = torch.Generator().manual_seed(11)
    bits = lambda *s: torch.randn(s, generator=g).to(torch.bfloat16).view(torch.int16).cuda()
    B.cas_kv_append(ctx, kv, 0, 0, bits(length, 1, 128), bits(length, 1, 128))
    B.cas_kv_set_len(kv, 0, length)
    q, k, v = bits(1, most, 128), bits(3, 1, 128), bits(3, 1, 128)
    wide = B.cas_attention(ctx, kv, 0, 0, full, q, k, v)
    for rows in (1, 3, 4, 5, 8, 9, 16, 17, 24, 25, 32, 33, 48, 49, 64, 65):
        if rows <= most:
            assert torch.equal(B.cas_attention(ctx, kv, 0, 0, full, q[:, :rows].contiguous(), k, v), wide[:, :rows]), rows
