"""Rounding error of the FP64 products against sums in extended precision: the
matrix-core tiles split a row's sum at least as finely as the kernels that
they take the place of."""
import numpy as np
import pytest
import torch

from gpu_util import dev
from workloads import random_cube, sc_lattice

from paper_2609_04397_amd.kspace import KMatrix
from paper_2609_04397_amd.matrix import Matrix

pytestmark = pytest.mark.gpu

OPS = {
    "1_4_9": lambda: random_cube(1500, 0.1, [(1, 300), (4, 600), (9, 600)], 5.2, 2.0, seed=3),
    "5": lambda: random_cube(2000, 0.1, [(5, 2000)], 5.2, 2.0, seed=8),
    "28": lambda: random_cube(400, 0.1, [(28, 400)], 5.2, 2.0, seed=9),
    "8": lambda: random_cube(1200, 0.1, [(8, 1200)], 5.2, 2.0, seed=4),
    "13": lambda: sc_lattice(10, 13, seed=5),
}


def row_sums(op, transpose, values, X):
    """op(A) X in the precision of the arguments, from scalar entries."""
    b = op.b.astype(np.int64)
    off = np.concatenate([[0], np.cumsum(b)])
    rows = np.repeat(np.arange(b.size), np.diff(op.row_ptr))
    size = b[rows] * b[op.col_idx]
    blk = np.repeat(np.arange(rows.size), size)
    loc = np.arange(size.sum()) - (np.cumsum(size) - size)[blk]
    bj = b[op.col_idx][blk]
    r, c = off[rows[blk]] + loc // bj, off[op.col_idx[blk]] + loc % bj
    if transpose:
        r, c = c, r
    o = np.argsort(r, kind="stable")
    r = r[o]
    first = np.flatnonzero(np.concatenate([[True], r[1:] != r[:-1]]))
    Y = np.zeros((off[-1], X.shape[1]), X.dtype)
    Y[r[first]] = np.add.reduceat(values[o][:, None] * X[c[o]], first, axis=0)
    return Y


def rel(y, ref):
    d = y - ref
    return float(np.sqrt((np.abs(d) ** 2).sum() / (np.abs(ref) ** 2).sum()))


# About 10^4 output rows times up to 4 columns are compared, so that the two
# root-mean-square errors are known to about 1 %: 10 % is well outside of it.
@pytest.mark.parametrize("transpose", [False, True])
@pytest.mark.parametrize("name", list(OPS))
def test_few_right_hand_sides_sum_like_the_vector_kernel(name, transpose):
    op = OPS[name]()
    rng = np.random.default_rng(7)
    N = int(op.b.sum())
    v = rng.uniform(-1, 1, op.values.size)
    X = rng.standard_normal((N, 8))
    ref = row_sums(op, transpose, v.astype(np.longdouble), X[:, :4].astype(np.longdouble))
    A = Matrix.from_operator(op, values=v)
    B = Matrix.from_operator(op, values=v, path="vec")
    for n in (2, 3, 4, 5, 8):
        k = min(n, 4)
        Xd = dev(X[:, :n], "fp64")
        ea, eb = (rel(M.spmm(Xd, transpose=transpose).cpu().numpy()[:, :k], ref[:, :k])
                  for M in (A, B))
        assert ea <= 1.1 * eb, (n, ea, eb)


# A component of a complex product is the sum of two real ones over the same
# rows: split alike it has the relative error of one of them (measured 1.00 to
# 1.08 of it); 1.25 is below the 1.4 of chains twice as long.
@pytest.mark.parametrize("adjoint", [False, True])
@pytest.mark.parametrize("name", ["1_4_9", "8", "13"])
def test_complex_products_sum_like_the_real_ones(name, adjoint):
    op = OPS[name]()
    rng = np.random.default_rng(9)
    N = int(op.b.sum())
    v = rng.uniform(-1, 1, op.values.size)
    K = KMatrix(op.b, op.row_ptr, op.col_idx, np.zeros(op.col_idx.size, np.int32),
                np.array([[1, 2, 3]], np.int32), prec="fp64", values=v)
    K.sample((0.11, 0.23, 0.07))
    w = K.values().cpu().numpy()
    X = rng.standard_normal((N, 48)) + 1j * rng.standard_normal((N, 48))
    ref = row_sums(op, adjoint, (w.conj() if adjoint else w).astype(np.clongdouble),
                   X[:, :4].astype(np.clongdouble))
    real = row_sums(op, adjoint, w.real.astype(np.longdouble), X[:, :4].real.astype(np.longdouble))

    def real_error(path, n):
        A = Matrix.from_operator(op, values=np.ascontiguousarray(w.real), path=path)
        y = A.spmm(dev(X[:, :n].real, "fp64"), transpose=adjoint)
        return rel(y.cpu().numpy()[:, :4], real)

    few, many = real_error("vec", 4), real_error("mfma", 16)
    for n in (1, 4, 8, 11, 15, 16, 24, 48):
        k = min(n, 4)
        y = K.spmm(torch.from_numpy(np.ascontiguousarray(X[:, :n])).cuda(), adjoint=adjoint)
        e = rel(y.cpu().numpy()[:, :k], ref[:, :k])
        assert e <= 1.25 * (few if n < 16 else many), (n, e, few, many)
