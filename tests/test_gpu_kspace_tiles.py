"""Complex products on small and on 16-row matrix-core tiles: panel heights
around multiples of 4 and 16, panel widths around the 16- and 4-column steps
and the register ring, right-hand sides around every tile, leading dimensions
beyond the right-hand sides, and an X whose span takes the vector kernel."""
import ctypes

import numpy as np
import pytest
import torch

from oracle.kspace import KOperator
from workloads.periodic import random_images

pytestmark = pytest.mark.gpu

from paper_2609_04397_amd import _lib
from paper_2609_04397_amd.kspace import KMatrix

# Componentwise, times |O(k)||X|: at most ~2000 FP64 terms of four products
# (2000 * 4 * 1.1e-16 = 9e-13 at worst, its root over random signs 2e-14) on
# sampled values good to 1e-15; FP32 rounds the values and X once (1.2e-7).
TOL = {"fp64": 1e-13, "fp32": 2e-5}


def product(KM, X, ldx, ldy, alpha, beta, Y0, adjoint):
    """C entry with leading dimensions; columns past nrhs of X hold NaN, those
    of Y a mark that has to survive."""
    n, nrhs = X.shape
    Xd = torch.full((n, ldx), complex(float("nan"), float("nan")), dtype=KM.dtype, device="cuda")
    Xd[:, :nrhs] = torch.from_numpy(X).to("cuda", KM.dtype)
    Yd = torch.full((n, ldy), 7 - 3j, dtype=KM.dtype, device="cuda")
    Yd[:, :nrhs] = torch.from_numpy(Y0).to("cuda", KM.dtype)
    a = np.array([alpha.real, alpha.imag])
    b = np.array([beta.real, beta.imag])
    _lib.check(_lib.load().vbcsr_zmat_spmm(
        KM._h, ctypes.c_void_p(Xd.data_ptr()), ldx, ctypes.c_void_p(Yd.data_ptr()), ldy, nrhs,
        a.ctypes.data, b.ctypes.data, int(adjoint),
        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)))
    assert bool((Yd[:, nrhs:] == 7 - 3j).all())
    return Yd[:, :nrhs].cpu().numpy().astype(np.complex128)


SETS = {"heights": (1, 3, 4, 5, 8, 9, 12, 13), "wide": (15, 16, 17, 20, 32, 33),
        "ones": (1,), "tall": (48, 49, 64)}


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("blocks", sorted(SETS))
def test_tiles_against_oracle(blocks, prec):
    n = 14 if blocks == "tall" else 40
    Z = random_images(31, n, bset=SETS[blocks], density=0.2, hermitian=False, empty_rows=2)
    rng = np.random.default_rng(6)
    KM = KMatrix.from_images(Z, prec=prec)
    k = rng.uniform(-1, 1, 3)
    KM.sample(k, "R+tau")
    K = KOperator(Z, k, "R+tau")
    alpha, beta = 0.75 - 0.5j, -0.25 + 1j
    for nrhs in (1, 2, 4, 5, 8, 9, 15, 16, 17, 31, 32, 33, 65):
        print("case", blocks, prec, nrhs, flush=True)
        X = rng.standard_normal((Z.N, nrhs)) + 1j * rng.standard_normal((Z.N, nrhs))
        Y0 = rng.standard_normal((Z.N, nrhs)) + 1j * rng.standard_normal((Z.N, nrhs))
        for adj in (False, True):
            got = product(KM, X, nrhs + 3, nrhs + 2, alpha, beta, Y0, adj)
            ref = (K.spmm_h(X) if adj else K.spmm(X)) * alpha + beta * Y0
            scale = abs(alpha) * K.abs_scale(X, adjoint=adj) + abs(beta) * np.abs(Y0)
            err = (np.abs(got - ref) / np.maximum(scale, 1e-300)).max()
            assert err <= TOL[prec], "%s nrhs %d adjoint %s: %.2e" % (blocks, nrhs, adj, err)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_span_of_x_beyond_one_descriptor(prec):
    """The same product with X spread over more than 2 GiB (vector kernel)
    and just within it agrees with the packed one."""
    Z = random_images(8, 30, bset=(1, 4, 9, 17), density=0.3, hermitian=False)
    rng = np.random.default_rng(2)
    KM = KMatrix.from_images(Z, prec=prec).sample(rng.uniform(-1, 1, 3), "R")
    es = 16 if prec == "fp64" else 8
    for nrhs in (1, 7, 21):
        X = rng.standard_normal((Z.N, nrhs)) + 1j * rng.standard_normal((Z.N, nrhs))
        Y0 = np.zeros((Z.N, nrhs), complex)
        near = (2**31 - 4096 - 1) // es // Z.N
        for adj in (False, True):
            ref = product(KM, X, nrhs, nrhs, 1 + 0j, 0j, Y0, adj)
            scale = np.abs(ref).max()
            for ld in (near, near + near // 8):
                got = product(KM, X, ld, nrhs, 1 + 0j, 0j, Y0, adj)
                assert np.abs(got - ref).max() <= TOL[prec] * scale
