"""Block products whose set-up sorts stay below and go beyond 2^18 pairs (two
sorting methods), against scipy: pattern, values in graph order, products of
both directions and the block-sampled product of the result."""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

from oracle import expand_op
from workloads.core import Operator

from paper_2609_04397_amd.matrix import Matrix

pytestmark = pytest.mark.gpu


def banded(n, offsets, bset, seed):
    """Blocks at i + offsets; sizes drawn from bset."""
    rng = np.random.default_rng(seed)
    b = rng.choice(np.asarray(bset, np.int32), n).astype(np.int32)
    cols = np.arange(n)[:, None] + np.asarray(offsets)[None, :]
    keep = (cols >= 0) & (cols < n)
    rp = np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int64)
    ci = cols[keep].astype(np.int32)
    rows = np.repeat(np.arange(n), np.diff(rp))
    nnz = int((b[rows].astype(np.int64) * b[ci]).sum())
    return Operator("banded", b, rp, ci, rng.uniform(-1, 1, nnz), np.zeros(ci.size))


@pytest.mark.parametrize("n,bset", [(9000, (1, 2, 5)), (15400, (1,)), (15500, (3, 4)), (40000, (1, 2))])
def test_pattern_and_values(n, bset):
    """17 blocks a row of the product: 153,000, 261,800 and 263,500 (just below
    and above 2^18), 680,000.  A value is a sum of at most 9 * 5 terms, a row of
    C X of 17 * 5 such sums: 1e-13 of the sum of magnitudes."""
    op = banded(n, (-10, -7, -3, -1, 0, 2, 5, 8, 11), bset, n)
    print("case", n, bset, flush=True)
    A = Matrix.from_operator(op)
    C, st = A.spgemm(A)
    E = expand_op(op)
    S = sp.csr_matrix((E.va, E.ci, E.rp), shape=(E.N, E.N))
    P = sp.csr_matrix((np.ones(op.col_idx.size), op.col_idx, op.row_ptr), shape=(n, n))
    P = (P @ P).tocsr()
    P.sort_indices()
    assert np.array_equal(C.row_ptr, P.indptr) and np.array_equal(C.col_idx, P.indices)
    rng = np.random.default_rng(1)
    X, G = rng.standard_normal((E.N, 3)), rng.standard_normal((E.N, 3))
    ref, absS = S @ S, abs(S)
    mag = absS @ absS
    for T in (False, True):
        M, m = (ref.T, mag.T) if T else (ref, mag)
        got = C.spmm(torch.from_numpy(X).cuda(), transpose=T).cpu().numpy()
        assert (np.abs(got - M @ X) <= 1e-13 * (m @ np.abs(X))).all()
    # graph-order values (unpacked pages): they rebuild the same operator
    D = Matrix(op.b, C.row_ptr, C.col_idx, C.values().cpu().numpy())
    got = D.spmm(torch.from_numpy(X).cuda()).cpu().numpy()
    assert (np.abs(got - ref @ X) <= 1e-13 * (mag @ np.abs(X))).all()
    assert torch.equal(C.sddmm(torch.from_numpy(G).cuda(), torch.from_numpy(X).cuda()),
                       D.sddmm(torch.from_numpy(G).cuda(), torch.from_numpy(X).cuda()))
