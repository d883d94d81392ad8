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
