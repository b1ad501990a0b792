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


def _limited():
    import paper_1608_05265_amd as mg
    fn = mg._load().misgemm_sgetrf_limited
    fn.argtypes = [ctypes.c_int64, ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p,
                   ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    return fn


class Factors:
    """The factorization of a (queued on `stream`, not waited for)."""

    def __init__(self, a, stream=None, wait_polls=PANEL_WAIT, word_polls=WORD_WAIT):
        import torch
        n = a.shape[0]
        self.A = torch.from_numpy(np.ascontiguousarray(a.T)).to("cuda:0")
        self.piv = torch.empty(n, dtype=torch.int64, device="cuda:0")
        self.inf = torch.empty(1, dtype=torch.int32, device="cuda:0")
        torch.cuda.synchronize()
        s = stream or torch.cuda.current_stream()
        rc = _limited()(n, self.A.data_ptr(), n, self.piv.data_ptr(), self.inf.data_ptr(), 0,
                        wait_polls, word_polls, s.cuda_stream)
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
