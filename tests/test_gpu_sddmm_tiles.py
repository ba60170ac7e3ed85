"""Block-sampled dY X^T on every route of its dispatch against the oracle:
panel widths around the 16-column tiles, blocks that run over tile borders,
heights on both sides of the staged and the direct stores, right-hand sides
around every chunk, strided inputs, outputs at odd alignment."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from workloads import random_pattern

from paper_2609_04397_amd import _lib
from paper_2609_04397_amd.matrix import Matrix

pytestmark = pytest.mark.gpu

OPS = {"ones": dict(seed=41, n=120, bset=(1,), density=0.2),
       "small": dict(seed=42, n=90, bset=(1, 2, 3, 4, 5), density=0.2, empty_rows=3, unsorted=True),
       "sp": dict(seed=43, n=80, bset=(1, 4, 9), density=0.3, empty_rows=2, unsorted=True),
       "ten": dict(seed=44, n=50, bset=(7, 8, 10, 11), density=0.3),
       "dzp": dict(seed=45, n=40, bset=(12, 13, 16), density=0.4, unsorted=True),
       "wide": dict(seed=46, n=24, bset=(1, 5, 17, 33, 64), density=0.4, unsorted=True)}
DT = {"fp64": torch.float64, "fp32": torch.float32}
EPS = {"fp64": 2.0**-53, "fp32": 2.0**-24}
MARK = -77.0


def strided(a, ld, prec):
    """Rows at a leading dimension, NaN between them."""
    t = torch.full((a.shape[0], ld), float("nan"), dtype=DT[prec], device="cuda")
    t[:, :a.shape[1]] = torch.from_numpy(a).to("cuda", DT[prec])
    return t


def call(A, dY, lddy, X, ldx, nrhs, size, lead, prec, pages):
    """The C entry into the middle of a marked buffer; the marks survive."""
    buf = torch.full((lead + size + 64,), MARK, dtype=DT[prec], device="cuda")
    fn = _lib.load().vbcsr_sddmm_pages if pages else _lib.load().vbcsr_sddmm
    _lib.check(fn(A._h, ctypes.c_void_p(dY.data_ptr()), lddy, ctypes.c_void_p(X.data_ptr()), ldx, nrhs,
                  ctypes.c_void_p(buf[lead:].data_ptr()),
                  ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    got = buf.cpu().numpy().astype(np.float64)
    assert (got[:lead] == MARK).all() and (got[lead + size:] == MARK).all()
    return got[lead:lead + size]


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("name", sorted(OPS))
def test_routes_against_oracle(name, prec):
    """Componentwise within (nrhs + 8) eps of |dY||X|: products and sums of
    nrhs terms in the working precision, the inputs exact."""
    op = random_pattern(**OPS[name])
    A = Matrix.from_operator(op, prec=prec)
    # page position of every value of graph order
    A.set_values(torch.arange(1, op.nnz + 1, dtype=DT[prec], device="cuda"))
    held = A.get_pages().cpu().numpy().astype(np.int64)
    where = np.argsort(np.where(held > 0, held, op.nnz + 1), kind="stable")[:op.nnz]
    for nrhs in (1, 2, 4, 7, 8, 9, 16, 17, 31, 32, 33, 48, 63, 64, 65):
        print("case", name, prec, nrhs, flush=True)
        rng = np.random.default_rng(nrhs)
        X, G = (rng.standard_normal((op.N, nrhs)).astype(np.float32).astype(np.float64) for _ in range(2))
        ref = oracle.sddmm(op, G, X)
        tol = (nrhs + 8) * EPS[prec] * oracle.sddmm(op, np.abs(G), np.abs(X))
        for ldx, lddy, lead in ((nrhs, nrhs, 4), (nrhs + 3, nrhs + 1, 1)):
            Xd, Gd = strided(X, ldx, prec), strided(G, lddy, prec)
            got = call(A, Gd, lddy, Xd, ldx, nrhs, op.nnz, lead, prec, False)
            assert (np.abs(got - ref) <= tol).all()
            got = call(A, Gd, lddy, Xd, ldx, nrhs, A.page_size, lead, prec, True)
            assert (np.abs(got[where] - ref) <= tol).all()
            rest = np.ones(A.page_size, bool)
            rest[where] = False
            assert (got[rest] == 0).all()


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("which", ["X", "dY"])
def test_spans_beyond_one_descriptor(which, prec):
    """Inputs spread over more memory than 32-bit offsets reach take the
    general kernels and give what the packed ones give, to both roundings."""
    op = random_pattern(seed=47, n=16, bset=(1, 4, 9, 17), density=0.5)
    A = Matrix.from_operator(op, prec=prec)
    far = 2**31 // (8 if prec == "fp64" else 4) // (op.N - 1) + 1 if which == "X" else 2**22
    for nrhs in (5, 32, 40):
        rng = np.random.default_rng(nrhs)
        X, G = rng.standard_normal((op.N, nrhs)), rng.standard_normal((op.N, nrhs))
        tol = 2 * (nrhs + 8) * EPS[prec] * oracle.sddmm(op, np.abs(G), np.abs(X))
        ref = call(A, strided(G, nrhs, prec), nrhs, strided(X, nrhs, prec), nrhs, nrhs, op.nnz, 0, prec, False)
        ldx, lddy = (far, nrhs) if which == "X" else (nrhs, far)
        got = call(A, strided(G, lddy, prec), lddy, strided(X, ldx, prec), ldx, nrhs, op.nnz, 0, prec, False)
        assert (np.abs(got - ref) <= tol).all()
