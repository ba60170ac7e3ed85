"""FP64 products that the library routes to small matrix-core tiles, against
the kernels that a forced path takes, over the forms both accept."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host
from metrics import comp
from workloads import random_pattern
from workloads.core import inf_norm_scale, scaled

from paper_2609_04397_amd.matrix import Matrix

pytestmark = pytest.mark.gpu

# mean heights that pad little, some and much in 16-row tiles
OPS = {"wide": dict(seed=31, n=40, bset=(13, 16), density=0.3, empty_rows=2, unsorted=True),
       "mixed": dict(seed=32, n=36, bset=(9, 13, 17, 20, 33, 64), density=0.25, unsorted=True),
       "narrow": dict(seed=33, n=150, bset=(1, 2, 4, 5, 8), density=0.08, empty_rows=4)}


@pytest.mark.parametrize("name", sorted(OPS))
@pytest.mark.parametrize("nrhs", [2, 3, 4, 5, 8, 9, 13, 16, 17, 31, 32])
def test_routed_path_agrees_with_the_forced_ones(name, nrhs):
    """Both directions, alpha and beta, aligned and odd column slices, three
    processing orders: within 1e-13 of (|A||X|), as two FP64 summation orders
    of at most 600 terms are."""
    op = random_pattern(**OPS[name])
    print("case", name, nrhs, flush=True)
    rng = np.random.default_rng(nrhs)
    X, Y0 = rng.standard_normal((op.N, nrhs)), rng.standard_normal((op.N, nrhs))
    general = Matrix.from_operator(op, path="mfma" if nrhs > 8 else "vec")
    for order in ("auto", "atom", "rcm"):
        A = Matrix.from_operator(op, row_order=order)
        for T in (False, True):
            scale = 1.5 * oracle.abs_product(op, X, transpose_op=T) + 0.5 * np.abs(Y0)
            Yg = dev(Y0, "fp64")
            general.spmm(dev(X, "fp64"), Yg, alpha=1.5, beta=-0.5, transpose=T)
            want = host(Yg)
            for lead, tail in ((0, 0), (1, 2), (2, 0)):
                wide = np.full((op.N, lead + nrhs + tail), np.nan)
                wide[:, lead:lead + nrhs] = X
                Xd = dev(wide, "fp64")[:, lead:lead + nrhs]
                wide[:, lead:lead + nrhs] = Y0
                Yw = dev(wide, "fp64")
                A.spmm(Xd, Yw[:, lead:lead + nrhs], alpha=1.5, beta=-0.5, transpose=T)
                got = host(Yw)
                assert comp(got[:, lead:lead + nrhs], want, scale) <= 1e-13
                assert np.isnan(got[:, :lead]).all() and np.isnan(got[:, lead + nrhs:]).all()


@pytest.mark.parametrize("nrhs", [2, 3, 7, 12, 16, 24])
def test_moments_of_the_small_tiles(nrhs):
    op = random_pattern(seed=34, n=60, bset=(1, 4, 9, 20), density=0.1, symmetric=True, empty_rows=2)
    op = scaled(op, inf_norm_scale(op))
    R = np.random.default_rng(nrhs).standard_normal((op.N, nrhs))
    ref = oracle.cheb_moments(op, R, 12)
    A = Matrix.from_operator(op)
    mu = A.cheb_moments(dev(R, "fp64"), 12)
    assert np.max(np.abs(mu - ref)) <= 1e-12 * np.max(np.abs(ref[0]))
    assert np.array_equal(mu, A.cheb_moments(dev(R, "fp64"), 12))


def test_rows_beyond_one_buffer_descriptor():
    """X spanning more than 2 GiB takes the kernels with 64-bit addresses."""
    op = random_pattern(seed=35, n=64, bset=(1, 4, 9), density=0.2)
    for nrhs in (3, 8, 12, 20):
        ld = (1 << 31) // 8 // op.N + 64
        X = np.random.default_rng(nrhs).standard_normal((op.N, nrhs))
        big = torch.empty((op.N, ld), dtype=torch.float64, device="cuda")
        big[:, :nrhs] = torch.from_numpy(X).cuda()
        got = host(Matrix.from_operator(op).spmm(big[:, :nrhs]))
        assert comp(got, oracle.spmm(op, X), oracle.abs_product(op, X)) <= 1e-12
        del big
