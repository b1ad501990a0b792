"""The 64x64 FP64 tile at its edges: rows and columns that end inside a tile,
odd leading dimensions, bases that are not 16-byte aligned, with and without a
ragged block of K.  1021x1019 takes it on 256 CUs (one tile of 64x64 a CU
against five of 32x32), as the dispatch's figures have it."""
import numpy as np
import pytest

import oracle
from paper_1608_05265_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _offset(x, off):
    """The same storage `off` elements into a larger buffer of NaN."""
    import torch
    buf = torch.full((x.size + off + 4,), float("nan"), dtype=torch.float64, device="cuda:0")
    buf[off:off + x.size] = torch.from_numpy(x)
    return buf[off:off + x.size]


@pytest.mark.parametrize("ta,tb", [("N", "N"), ("N", "T"), ("T", "N"), ("T", "T")])
@pytest.mark.parametrize("k", [7, 16, 64, 69])
@pytest.mark.parametrize("pad", [0, 3])
def test_dgemm_large_tile_edges(ta, tb, k, pad):
    import torch
    import paper_1608_05265_amd as mg
    m, n = 1021, 1019
    p = wl.make_problem_d(ta, tb, m, n, k, 1.5, -0.5, wl.seed_for(9, 700 + 8 * k + pad), pad=pad)
    A, B, C = _offset(p.A, 1), _offset(p.B, 3), _offset(p.C0, 1)
    mg.dgemm(ta, tb, m, n, k, p.alpha, A, p.lda, B, p.ldb, p.beta, C, p.ldc)
    torch.cuda.synchronize()
    out = C.cpu().numpy()
    rng = np.random.default_rng(k)
    r, c = np.arange(m), np.arange(n)
    # the last rows and columns whole, and a sample of the rest
    rows = np.concatenate([r, np.full(n, m - 1), np.full(n, m - 2), r, rng.integers(0, m, 2000)])
    cols = np.concatenate([np.full(m, n - 1), c, c, np.full(m, n - 2), rng.integers(0, n, 2000)])
    cref, den = oracle.dgemm_f128_entries(ta, tb, m, n, k, p.alpha, p.A, p.lda, p.B, p.ldb, p.beta,
                                          p.C0, p.ldc, rows.astype(np.int64), cols.astype(np.int64))
    err = np.abs(out[rows + cols * p.ldc] - cref)
    assert np.all(err <= max(2 * k, k + 3) * 2.0 ** -53 * den)
    pad_rows = lambda x: np.ascontiguousarray(x.reshape(n, p.ldc)[:, m:]).view(np.uint64)
    assert np.array_equal(pad_rows(out), pad_rows(p.C0)), "padding rows written"
