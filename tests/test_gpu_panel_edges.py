"""Products at every panel width around the kernels' load groups.

Row atoms of many heights reference 0 .. 80 one-orbital atoms, so panels end
at every position of a group of slices.  Atom 0 is referenced by no row and
its X rows are NaN: a padding column that read X (instead of zeros) would
show.  Tolerances are the parity tests' (FP64 componentwise 1e-12, FP32 1e-5
and BF16x3 5e-5 in the Frobenius norm).
"""
import numpy as np
import pytest

import oracle
from gpu_util import check, dev, host, rounded
from workloads.core import Operator

from paper_2609_04397_amd.matrix import Matrix

pytestmark = pytest.mark.gpu

HEIGHTS = (1, 3, 4, 5, 8, 9, 12, 13, 16, 17, 20, 32, 33)


def edge_operator(widths=tuple(range(0, 81))):
    rng = np.random.default_rng(11)
    nc = 1 + max(widths)                      # one-orbital atoms, atom 0 unreferenced
    b = np.concatenate([np.ones(nc, np.int32),
                        np.array([HEIGHTS[i % len(HEIGHTS)] for i in range(len(widths))], np.int32)])
    rows = [np.empty(0, np.int64)] * nc
    rows += [np.sort(rng.choice(np.arange(1, nc), size=w, replace=False)) for w in widths]
    row_ptr = np.concatenate([[0], np.cumsum([r.size for r in rows])]).astype(np.int64)
    col = np.concatenate(rows).astype(np.int32)
    nnz = int(sum(int(b[i]) * r.size for i, r in enumerate(rows)))
    return Operator("edges", b, row_ptr, col, rng.uniform(-1, 1, nnz), np.zeros(col.size))


@pytest.fixture(scope="module")
def op():
    return edge_operator()


@pytest.mark.parametrize("prec,nrhs", [("fp64", 2), ("fp64", 3), ("fp64", 8), ("fp64", 12), ("fp64", 16),
                                       ("fp64", 24), ("fp64", 32), ("fp64", 33), ("fp64", 64),
                                       ("fp32", 5), ("fp32", 12), ("fp32", 16), ("fp32", 20),
                                       ("fp32", 32), ("fp32", 50), ("fp32", 64),
                                       ("bf16x3", 16), ("bf16x3", 64)])
def test_product_at_every_width(op, prec, nrhs):
    print("case", prec, nrhs, flush=True)
    A = Matrix.from_operator(op, prec=prec)
    X = rounded(np.random.default_rng(nrhs).standard_normal((op.N, nrhs)), prec)
    X[0] = 0.0
    ref = oracle.spmm(op, X)
    scale = oracle.abs_product(op, X)
    Xn = X.copy()
    Xn[0] = np.nan
    check(host(A.spmm(dev(Xn, prec))), ref, prec, scale, "forward %s %d" % (prec, nrhs))
    # the adjoint's panels have the heights' widths; its unused row stays zero
    ref = oracle.spmm_t(op, X)
    got = host(A.spmm_t(dev(X, prec)))
    check(got, ref, prec, oracle.abs_product(op, X, transpose_op=True), "adjoint %s %d" % (prec, nrhs))
    assert not got[0].any()


@pytest.mark.parametrize("prec,nrhs", [("fp64", 3), ("fp64", 6), ("fp64", 13), ("fp32", 5), ("fp32", 9),
                                       ("fp32", 13), ("fp32", 22), ("fp32", 50), ("bf16x3", 1),
                                       ("bf16x3", 13), ("bf16x3", 50)])
def test_columns_beside_the_vectors_do_not_matter(op, prec, nrhs):
    """X and Y are column slices of wider arrays: what lies beside X (NaN) is
    read at most into columns that are not stored, what lies beside Y stays."""
    print("case slices", prec, nrhs, flush=True)
    A = Matrix.from_operator(op, prec=prec)
    X = rounded(np.random.default_rng(nrhs).standard_normal((op.N, nrhs)), prec)
    ref = oracle.spmm(op, X)
    for lead, tail in ((3, 2), (4, 0), (0, 7)):
        wide = np.full((op.N, lead + nrhs + tail), np.nan)
        wide[:, lead:lead + nrhs] = X
        Xd = dev(wide, prec)[:, lead:lead + nrhs]
        Yw = dev(np.full_like(wide, 7.0), prec)
        A.spmm(Xd, Yw[:, lead:lead + nrhs])
        got = host(Yw)
        check(got[:, lead:lead + nrhs], ref, prec, oracle.abs_product(op, X), "slice %d" % lead)
        assert (got[:, :lead] == 7.0).all() and (got[:, lead + nrhs:] == 7.0).all()
