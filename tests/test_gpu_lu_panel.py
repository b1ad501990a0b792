"""The LU's panel kernel: its workgroups' start, together or not, and what a
panel's arithmetic is, whichever way its workgroups met."""
import ctypes

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

EPS32 = 2.0 ** -24
PANEL_WAIT = 1 << 16  # the library's own bounds
WORD_WAIT = 1 << 18
GROUPS = 64


def _limited():
    import paper_1608_05265_amd as mg
    fn = mg._load().misgemm_sgetrf_limited
    fn.argtypes = [ctypes.c_int64, ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p,
                   ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_int,
                   ctypes.c_void_p]
    return fn


class Factors:
    """The factorization of a (queued on `stream`, not waited for)."""

    def __init__(self, a, stream=None, wait_polls=PANEL_WAIT, word_polls=WORD_WAIT, groups=GROUPS,
                 sync=True):
        import torch
        n = a.shape[0]
        self.A = torch.from_numpy(np.ascontiguousarray(a.T)).to("cuda:0")
        self.piv = torch.empty(n, dtype=torch.int64, device="cuda:0")
        self.inf = torch.empty(1, dtype=torch.int32, device="cuda:0")
        s = stream or torch.cuda.current_stream()
        s.wait_stream(torch.cuda.current_stream())  # the copy
        if sync:
            torch.cuda.synchronize()
        rc = _limited()(n, self.A.data_ptr(), n, self.piv.data_ptr(), self.inf.data_ptr(), 0,
                        wait_polls, word_polls, groups, s.cuda_stream)
        assert rc == 0

    def get(self):
        import torch
        torch.cuda.synchronize()
        return self.A.cpu().numpy().T, self.piv.cpu().numpy(), int(self.inf.item())


def _dominant(n, seed):
    """A matrix whose pivots are unique by a wide margin, and its factors."""
    rng = np.random.default_rng(seed)
    d = rng.uniform(-1, 1, (n, n)) + np.diag(rng.uniform(n, 2 * n, n))
    a = d[rng.permutation(n)].astype(np.float32)
    return a, oracle.getrf_f64(n, a.T.reshape(-1), n)


def _check(got, want, n):
    lu, ipiv, info = got
    lu_o, ipiv_o, _ = want
    assert info == 0 and np.array_equal(ipiv, ipiv_o)
    assert np.max(np.abs(lu - lu_o)) <= 8 * n * EPS32 * np.max(np.abs(lu_o))


@pytest.mark.parametrize("n", [513, 1025, 2500])
def test_panels_called_off_by_the_other_workgroups(n):
    """The other workgroups do not wait for the first one's word: they call
    the panel off, or find that it goes on.  Nobody leaves a panel that does."""
    a, want = _dominant(n, 61)
    _check(Factors(a, word_polls=0).get(), want, n)
    _check(Factors(a, wait_polls=-1, word_polls=0).get(), want, n)


def test_factorizations_on_several_streams():
    """Four factorizations at once, on a stream each."""
    import torch
    n = 1600
    cases = [_dominant(n, 62 + i) for i in range(4)]
    streams = [torch.cuda.Stream() for _ in cases]
    runs = [Factors(a, s) for (a, _), s in zip(cases, streams)]
    for r, (_, want) in zip(runs, cases):
        _check(r.get(), want, n)


def test_factorization_beside_a_product_that_fills_the_card():
    import torch
    import paper_1608_05265_amd as mg
    n, k = 1600, 8192
    a, want = _dominant(n, 66)
    B = torch.empty(k * k, device="cuda:0").uniform_(-1, 1)
    C = torch.empty_like(B)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(3):
        mg.sgemm("N", "N", k, k, k, 1.0, B, k, B, k, 0.0, C, k, stream=side)
    _check(Factors(a).get(), want, n)


def _fma(a, b, c):
    """a * b + c in float32, rounded once: exact product, the sum rounded to
    odd in double (its last bit set where it is not exact), then to float."""
    p = a.astype(np.float64) * b.astype(np.float64)
    c = np.broadcast_to(c, p.shape).astype(np.float64)
    t = p + c
    bv = t - p
    err = (p - (t - bv)) + (c - bv)
    bits = t.view(np.int64)
    toward = np.where((err > 0) == (t > 0), 1, -1)  # away from zero or towards it
    bits = np.where((err != 0) & (bits & 1 == 0), bits + toward, bits)
    return bits.view(np.float64).astype(np.float32)


def _panel(a):
    """The factored panel and its pivots, in float32: columns in blocks of
    eight, a pivot row subtracted at once from the block's own columns and the
    block's eight together, summed apart in order, from the later ones."""
    a = a.copy()
    m, w = a.shape
    piv = np.empty(w, np.int64)
    for b in range(0, w, 8):
        e = min(b + 8, w)
        for j in range(b, e):
            p = j + int(np.argmax(np.abs(a[j:, j])))
            piv[j] = p
            a[[j, p]] = a[[p, j]]
            a[j + 1:, j] *= np.float32(1) / a[j, j]
            a[j + 1:, j + 1:e] = _fma(-a[j + 1:, j, None], a[None, j, j + 1:e], a[j + 1:, j + 1:e])
        for r in range(b + 1, e):
            s = np.zeros(w - e, np.float32)
            for k in range(b, r):
                s = _fma(-a[r, k, None], a[k, e:], s)
            a[r, e:] += s
        s = np.zeros((m - e, w - e), np.float32)
        for k in range(b, e):
            s = _fma(-a[e:, k, None], a[None, k, e:], s)
        a[e:, e:] += s
    return a, piv


@pytest.mark.parametrize("n", [5, 50, 64, 200, 512, 513, 1024, 1025, 2600, 6144, 6145, 12289, 16385])
def test_first_panel_bit_for_bit(n):
    """Against the same sums in numpy: whole and partial blocks, one workgroup
    of one (to 512 rows) and two rows per thread (to 1024), up to 12 workgroups
    of one row per thread (to 6144), two rows per thread again (from 6145), more
    than the 12 whose messages come in one round trip (from 12289), all XCDs
    (from 16385)."""
    a = np.random.default_rng(68).random((n, n), np.float32) - np.float32(0.5)
    w = min(n, 64)
    want, piv = _panel(a[:, :w])
    lu, ipiv, info = Factors(a).get()
    for j in range(w, n):  # the later panels' interchanges
        want[[j, ipiv[j]]] = want[[ipiv[j], j]]
    assert info == 0 and np.array_equal(ipiv[:w], piv)
    assert np.array_equal(lu[:, :w], want)


# significands after which a Newton step from a reciprocal an ulp off would
# round the wrong way
HARD_PIVOTS = [0x069913, 0x07cc45, 0x0efa43, 0x109909, 0x186799, 0x1beaaf, 0x20ddd1, 0x224cf7,
               0x26449f, 0x2aaaac, 0x2b8be1, 0x2d1367, 0x384a93, 0x423dc3, 0x50ac19, 0x50dd0d,
               0x525d25, 0x543d43, 0x5c23dd, 0x5e86a9, 0x605475, 0x61368b, 0x625473, 0x6c7ec7,
               0x6e4bc5, 0x700ff1, 0x702a3b, 0x70ff0f, 0x7c3237, 0x7e01ff, 0x7ffffd, 0x7fffff]


def test_multipliers_are_the_entries_times_the_rounded_reciprocal():
    """A lower triangular matrix whose diagonal holds the pivots: nothing is
    updated, so L is each column times its pivot's reciprocal, rounded twice
    (divided by a subnormal pivot), bit for bit."""
    rng = np.random.default_rng(67)
    n = 700
    piv = (0x3f800000 | rng.integers(0, 1 << 23, n)).astype(np.uint32)
    piv[:32] = np.uint32(0x3f800000) | np.array(HARD_PIVOTS, np.uint32)
    piv = piv.view(np.float32) * np.exp2(rng.integers(-100, 100, n)).astype(np.float32)
    piv[40], piv[41], piv[42] = 2.0 ** -140, 1.5 * 2.0 ** 126, np.finfo(np.float32).max
    piv[50::2] *= -1
    a = np.tril(rng.uniform(-0.99, 0.99, (n, n)).astype(np.float32), -1) * np.abs(piv)
    a[np.arange(n), np.arange(n)] = piv
    with np.errstate(over="ignore", invalid="ignore"):
        want = np.where(np.abs(piv) >= np.float32(2.0 ** -126), a * (np.float32(1) / piv), a / piv)
    want = np.tril(want.astype(np.float32), -1)
    want[np.arange(n), np.arange(n)] = piv
    lu, ipiv, info = Factors(a).get()
    assert info == 0 and np.array_equal(ipiv, np.arange(n))
    assert np.array_equal(lu, want)


@pytest.mark.parametrize("kind", ["uniform", "ties", "scaled", "subnormal", "huge", "nan"])
@pytest.mark.parametrize("n", [600, 1100, 2500])
def test_bits_do_not_depend_on_whether_the_workgroups_met(n, kind):
    """Panels called off by the first workgroup or by the others, factored in
    memory, give the same factors as those that go on, bit for bit."""
    rng = np.random.default_rng(69)
    a = rng.uniform(-1, 1, (n, n))
    if kind == "ties":
        a = rng.integers(-2, 3, (n, n))
        a[:, 3] = a[:, 70] = 0
    elif kind == "scaled":
        a = a * np.exp2(rng.integers(-60, 60, (n, n)))
    elif kind == "subnormal":
        a = a * 2.0 ** -130
    elif kind == "huge":
        a = a * 2.0 ** 126
    elif kind == "nan":
        a[:, 3], a[:, 20], a[5, 21], a[7, 22] = 0, np.nan, np.inf, np.nan
    a = a.astype(np.float32)
    lu, ipiv, info = Factors(a).get()
    for limits in (dict(wait_polls=-1), dict(word_polls=0)):
        lu2, ipiv2, info2 = Factors(a, **limits).get()
        assert info == info2 and np.array_equal(ipiv, ipiv2), limits
        assert np.array_equal(lu, lu2, equal_nan=True), limits


def test_bits_do_not_depend_on_what_else_runs():
    """Six factorizations on streams of their own beside products that fill
    the card, against each alone; panels over one XCD (n = 1600) and over all
    of them (16500)."""
    import torch
    import paper_1608_05265_amd as mg
    rng = np.random.default_rng(70)
    big = torch.empty(8192 * 8192, device="cuda:0").uniform_(-1, 1)
    out = torch.empty_like(big)
    for n, count in ((1600, 6), (16500, 1)):
        mats = [rng.random((n, n), np.float32) - np.float32(0.5) for _ in range(count)]
        alone = []
        for a in mats:
            f = Factors(a)
            torch.cuda.synchronize()
            alone.append((f.A, f.piv))
        side = torch.cuda.Stream()
        streams = [torch.cuda.Stream() for _ in mats]
        for _ in range(2):
            mg.sgemm("N", "N", 8192, 8192, 8192, 1.0, big, 8192, big, 8192, 0.0, out, 8192, stream=side)
        runs = [Factors(a, s, sync=False) for a, s in zip(mats, streams)]
        torch.cuda.synchronize()
        for (A, piv), r in zip(alone, runs):
            assert torch.equal(A, r.A) and torch.equal(piv, r.piv) and int(r.inf.item()) == 0, n


def test_a_column_of_nan_stays_out_of_the_panel():
    """A column with no pivot has no multipliers: NaN in it reaches no other
    column of its panel, whichever way that is factored."""
    rng = np.random.default_rng(71)
    a = rng.uniform(-1, 1, (64, 64)).astype(np.float32)
    b = a.copy()
    for col in (0, 5, 18):
        a[:, col], b[:, col] = 0, np.nan
    lu, ipiv, info = Factors(a).get()
    lu2, ipiv2, info2 = Factors(b).get()
    assert info == info2 == 1 and np.array_equal(ipiv, ipiv2)
    keep = [c for c in range(64) if c not in (0, 5, 18)]
    assert np.array_equal(lu[:, keep], lu2[:, keep])


@pytest.mark.parametrize("groups", [0, 1, 3])
def test_panels_taller_than_the_workgroups_hold(groups):
    """With fewer workgroups allowed to a panel, one that would need more is 8
    columns factored in memory; the factorization goes over to 64 columns in
    registers where the rest fits (at 1024 and 1536 rows; never with none)."""
    n = 3000
    a, want = _dominant(n, 75)
    _check(Factors(a, groups=groups).get(), want, n)
    a = np.random.default_rng(76).uniform(-1, 1, (n, n)).astype(np.float32)
    lu, ipiv, info = Factors(a, groups=groups).get()
    lu = lu.astype(np.float64)
    assert info == 0 and np.all(ipiv >= np.arange(n)) and np.all(ipiv < n)
    L, U = np.tril(lu, -1) + np.eye(n), np.triu(lu)
    assert np.max(np.abs(L)) <= 1.0 + 1e-6
    pa = a.astype(np.float64)
    for j, p in enumerate(ipiv):
        pa[[j, p]] = pa[[p, j]]
    # entry by entry the backward-error bound of LU, about n eps, as the other
    # sizes' tests take it
    assert np.all(np.abs(pa - L @ U) <= 4 * n * EPS32 * (np.abs(L) @ np.abs(U)))
