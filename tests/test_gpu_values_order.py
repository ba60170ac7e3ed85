"""Values back in graph order, bit for bit, where several waves share a run of
blocks: few large blocks, one large block size among small ones, a last run
that is not full, and enough blocks for one wave a run."""
import numpy as np
import pytest

from workloads import random_pattern

from paper_2609_04397_amd.matrix import Matrix

pytestmark = pytest.mark.gpu

CASES = {
    "one block": (1, (64,), 0.0),
    "few of 64": (5, (64,), 0.6),
    "64 among small": (40, (1, 2, 64), 0.3),
    "runs of 1,024 values and more": (70, (11, 12, 13), 0.5),
    "many": (420, (1, 3), 0.4),
}


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
@pytest.mark.parametrize("name", list(CASES))
def test_values_come_back(name, prec):
    n, bset, density = CASES[name]
    op = random_pattern(seed=n, n=n, bset=bset, density=density)
    v = np.random.default_rng(n).uniform(-1, 1, op.values.size)
    got = Matrix.from_operator(op, prec=prec, values=v).values().cpu().numpy()
    assert np.array_equal(got, v.astype(got.dtype))
