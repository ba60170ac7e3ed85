"""Device memory kept between calls: bounded, returned with the last handle,
never relied on for its contents, safe from several threads and streams."""
import gc
import threading

import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host
from workloads import random_pattern, sc_lattice

from paper_2609_04397_amd.matrix import Matrix

pytestmark = pytest.mark.gpu


def free_bytes():
    gc.collect()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return torch.cuda.mem_get_info()


def test_kept_memory_is_bounded_and_returned():
    gc.collect()
    op = sc_lattice(4, 5, seed=3)
    m = 30                                        # 2 x 1.1 GB of pages per handle
    big = sc_lattice(6, 1, seed=1)                # structure only, for the anchor
    n = m ** 3
    nb = np.full(n, 20, np.int32)
    rp = np.arange(0, 13 * n + 1, 13, dtype=np.int64)
    ci = ((np.arange(n)[:, None] + np.arange(13)[None, :] * 7) % n).astype(np.int32).ravel()
    Matrix.from_operator(op).close()              # library and context loaded
    start, total = free_bytes()
    anchor = Matrix.from_operator(big)
    hs = [Matrix(nb, rp, ci) for _ in range(4)]
    used = start - free_bytes()[0]
    assert used > total // 64                     # more than may be kept
    for h in hs:
        h.close()
    kept = start - free_bytes()[0]
    assert kept <= total // 64 + (64 << 20)
    # a kept block serves the next handle
    again = Matrix(nb, rp, ci)
    assert start - free_bytes()[0] <= kept + (3 << 30)
    again.close()
    anchor.close()
    assert start - free_bytes()[0] <= 64 << 20    # all returned with the last handle


def test_products_from_threads_and_streams_over_kept_memory():
    ops = [random_pattern(seed=20 + t, n=60, bset=(1, 4, 9, 13, 17), density=0.1, symmetric=True)
           for t in range(3)]
    refs, errs = [], []
    for op in ops:
        D = np.zeros((op.N, op.N))
        X = np.eye(op.N)
        D[:] = oracle.spmm(op, oracle.spmm(op, X))
        refs.append(D)
    anchors = [Matrix.from_operator(op) for op in ops]
    torch.cuda.synchronize()

    def work(t):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                X = dev(np.eye(ops[t].N), "fp64")
                for k in range(12):
                    C, _ = anchors[t].spgemm(anchors[t], eps=0.0)
                    Y = C.spmm(X)
                    s.synchronize()
                    C.close()
                    e = np.abs(Y.cpu().numpy() - refs[t]).max() / np.abs(refs[t]).max()
                    if not e <= 1e-12:
                        errs.append((t, k, e))
        except Exception as ex:  # reported by the main thread
            errs.append((t, repr(ex)))

    th = [threading.Thread(target=work, args=(t,)) for t in range(3)]
    for x in th:
        x.start()
    for x in th:
        x.join()
    assert not errs, errs[:3]
    assert host(anchors[0].values()).size == ops[0].nnz
