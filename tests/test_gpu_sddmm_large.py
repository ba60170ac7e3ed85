"""Block-sampled products whose outputs are large enough to leave through the
ring in LDS, and panels of more than 16 rows in the page layout: graph order
and page layout take different ways out of the same sums, so they agree bit
for bit, and a sample of the values is checked against FP64 sums."""
import numpy as np
import pytest
import torch

from paper_2609_04397_amd.matrix import Matrix

pytestmark = pytest.mark.gpu


def graph(n, near, bset, seed):
    """Blocks at up to 2 near + 1 columns around the diagonal, some left out."""
    rng = np.random.default_rng(seed)
    b = rng.choice(np.asarray(bset, np.int32), n)
    cols = np.arange(n)[:, None] + np.arange(-near, near + 1)[None, :]
    keep = (cols >= 0) & (cols < n) & (rng.random(cols.shape) < 0.9)
    rp = np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int64)
    return b, rp, cols[keep].astype(np.int32)


def check(b, rp, ci, prec, counts, least):
    A = Matrix(b, rp, ci, prec=prec)
    assert A.n_values * (8 if prec == "fp64" else 4) >= least
    rng = np.random.default_rng(1)
    dt = torch.float64 if prec == "fp64" else torch.float32
    off = np.concatenate([[0], np.cumsum(b.astype(np.int64))])
    rows = np.repeat(np.arange(b.size), np.diff(rp))
    size = b[rows].astype(np.int64) * b[ci]
    base = np.concatenate([[0], np.cumsum(size)])
    e = np.sort(rng.choice(base[-1], 20000))
    k = np.searchsorted(base, e, side="right") - 1
    p, q = np.divmod(e - base[k], b[ci[k]])
    for nrhs in counts:
        print("case", prec, nrhs, flush=True)
        X = torch.from_numpy(rng.standard_normal((A.N, nrhs))).to("cuda", dt)
        G = torch.from_numpy(rng.standard_normal((A.N, nrhs))).to("cuda", dt)
        out = torch.full((A.n_values,), float("nan"), dtype=dt, device="cuda")
        A.sddmm(G, X, out)
        A.use_pages(A.sddmm_pages(G, X))
        assert torch.equal(A.values(), out), nrhs
        x, g = X.double().cpu().numpy()[off[ci[k]] + q], G.double().cpu().numpy()[off[rows[k]] + p]
        # nrhs roundings of at most the sum of magnitudes
        eps = nrhs * (1.2e-16 if prec == "fp64" else 6e-8)
        d = np.abs(out.cpu().numpy()[e].astype(np.float64) - (g * x).sum(1))
        assert (d <= eps * np.abs(g * x).sum(1)).all(), nrhs


# widths that the ring holds beside panels that it does not (b = 11 with a
# block of 12, b above 12), panels of more than 16 rows, and single columns
@pytest.mark.parametrize("prec,n", [("fp64", 4500), ("fp32", 9000)])
def test_graph_order_through_the_ring(prec, n):
    b, rp, ci = graph(n, 45, (1, 2, 3, 4, 5, 8, 9, 10, 11, 12, 13, 13, 16, 17, 33), 3)
    check(b, rp, ci, prec, (1, 7, 16, 32, 33, 64), 192 << 20)


def test_ring_with_narrow_panels_beside_wide_ones():
    """Panels whose widest block decides: b = 12 with columns up to 9 beside
    b = 12 with one of 40."""
    n = 40000
    b, rp, ci = graph(n, 40, (1, 3, 4, 9), 4)
    b[::500] = 40
    b[7::100] = 12
    check(b, rp, ci, "fp32", (5, 32, 64), 192 << 20)


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_tall_panels_in_both_layouts(prec):
    b, rp, ci = graph(60, 12, (1, 15, 16, 17, 20, 31, 32, 33, 47, 63, 64), 5)
    check(b, rp, ci, prec, (1, 3, 8, 31, 32, 33, 63, 64), 0)


@pytest.mark.parametrize("prec,full,part", [("fp64", 16, 10), ("fp64", 64, 34), ("fp32", 32, 20),
                                            ("fp32", 64, 40)])
def test_staged_pieces_past_the_right_hand_sides_read_zero(prec, full, part):
    """LDS holds NaN from a call that used all pieces of a row; one that uses
    fewer of them, whole, gives the sums of its own."""
    b, rp, ci = graph(3000, 12, (4, 9, 13), 6)
    A = Matrix(b, rp, ci, prec=prec)
    dt = torch.float64 if prec == "fp64" else torch.float32
    rng = np.random.default_rng(2)
    X = torch.from_numpy(rng.standard_normal((A.N, part))).to("cuda", dt)
    G = torch.from_numpy(rng.standard_normal((A.N, part))).to("cuda", dt)
    bad = torch.full((A.N, full), float("nan"), dtype=dt, device="cuda")
    first = A.sddmm(G, X), A.sddmm_pages(G, X)
    assert bool(torch.isnan(A.sddmm(bad, bad)).all())
    again = A.sddmm(G, X)
    A.sddmm_pages(bad, bad)
    pages = A.sddmm_pages(G, X)
    assert bool(torch.isfinite(again).all()) and torch.equal(again, first[0])
    assert bool(torch.isfinite(pages[:-2]).all()) and torch.equal(pages[:-2], first[1][:-2])
