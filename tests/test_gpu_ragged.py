"""Ragged sizes, odd leading dimensions and unaligned bases through every
configuration: the edges of the tiles (one row or column past, short of and
fewer than a vector), the ragged end of K (shorter and longer than a K block,
absent), in both forms and in double precision, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1608_05265_amd import workloads as wl
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu

# (m, n, k): below one vector; one past and one short of the 16, 32, 64, 128
# and 256 tile sides, each residue of a chunk of four; k around the K blocks
SIZES = [(1, 1, 1), (3, 2, 5), (2, 65, 33), (17, 15, 64), (33, 63, 65), (66, 129, 31),
         (127, 131, 130), (257, 259, 47), (254, 62, 16)]


def _offset(x, off):
    """The same storage `off` elements into a larger buffer of NaN: base
    addresses that are not multiples of 16 bytes."""
    import torch
    buf = torch.full((x.size + off + 4,), float("nan"), dtype=torch.from_numpy(x[:0]).dtype,
                     device="cuda:0")
    buf[off:off + x.size] = torch.from_numpy(x)
    return buf[off:off + x.size]


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("size", SIZES, ids=lambda s: "%dx%dx%d" % s)
def test_every_config_ragged(size, mode):
    import torch
    import paper_1608_05265_amd as mg
    m, n, k = size
    for t, (ta, tb) in enumerate(wl.TRANS_PAIRS):
        p = wl.make_problem(ta, tb, m, n, k, 1.5, -0.5, wl.seed_for(9, 4 * SIZES.index(size) + t),
                            pad=t)
        A, B = _offset(p.A, 1 + t), _offset(p.B, 3)
        cref, den = oracle.sgemm_f64(ta, tb, m, n, k, p.alpha, p.A, p.lda, p.B, p.ldb, p.beta,
                                     p.C0, p.ldc)
        for cfg in mg.configs(mode):
            C = _offset(p.C0, 1)
            mg.sgemm_config(ta, tb, m, n, k, p.alpha, A, p.lda, B, p.ldb, p.beta, C, p.ldc, mode,
                            cfg["id"])
            torch.cuda.synchronize()
            out = C.cpu().numpy()
            ok, mx, mean, ratio = oracle.check(gu.c_dense(p, out), cref, den, k)
            label = "%s %s%s %dx%dx%d" % (cfg["name"], ta, tb, m, n, k)
            assert ok, "%s: max normalized error %.3e" % (label, mx)
            assert gu.padding_untouched(p, out), label


@pytest.mark.parametrize("size", SIZES + [(2100, 2050, 37)], ids=lambda s: "%dx%dx%d" % s)
def test_dgemm_ragged(size):
    """The last size takes the large tile."""
    import torch
    import paper_1608_05265_amd as mg
    m, n, k = size
    for t, (ta, tb) in enumerate(wl.TRANS_PAIRS):
        p = wl.make_problem_d(ta, tb, m, n, k, 1.5, -0.5, wl.seed_for(9, 500 + m + t), pad=t)
        A, B, C = _offset(p.A, 1), _offset(p.B, t), _offset(p.C0, 1)
        mg.dgemm(ta, tb, m, n, k, p.alpha, A, p.lda, B, p.ldb, p.beta, C, p.ldc)
        torch.cuda.synchronize()
        out = C.cpu().numpy()
        rng = np.random.default_rng(m)
        rows = np.concatenate([rng.integers(0, m, 64), np.full(64, m - 1)]).astype(np.int64)
        cols = np.concatenate([np.full(64, n - 1), rng.integers(0, n, 64)]).astype(np.int64)
        cref, den = oracle.dgemm_f128_entries(ta, tb, m, n, k, p.alpha, p.A, p.lda, p.B, p.ldb,
                                              p.beta, p.C0, p.ldc, rows, cols)
        err = np.abs(out[rows + cols * p.ldc] - cref)
        assert np.all(err <= max(2 * k, k + 3) * 2.0 ** -53 * den), "%s%s %s" % (ta, tb, size)
