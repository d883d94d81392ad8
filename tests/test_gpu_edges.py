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
