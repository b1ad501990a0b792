"""Problems of few rows and so many columns that a launch of the smallest
tiles would hold 2^32 threads or more."""
import pytest

pytestmark = pytest.mark.gpu


def _vectors(n, dtype):
    import torch
    g = torch.Generator("cuda").manual_seed(n & 0xFFFF)
    b = torch.randint(-8, 9, (n,), generator=g, device="cuda", dtype=torch.int8).to(dtype)
    c = torch.randint(-8, 9, (n,), generator=g, device="cuda", dtype=torch.int8).to(dtype)
    return b, c


@pytest.mark.parametrize("wide", ["n", "m"])
@pytest.mark.parametrize("size", [1 << 27, (1 << 30) + 5], ids=["2^27", "2^30+5"])
def test_dgemm_wide(size, wide):
    """One launch of larger tiles, and a call cut in two (integers: exact)."""
    import torch
    import paper_1608_05265_amd as mg
    b, c = _vectors(size, torch.float64)
    a = torch.tensor([3.0], dtype=torch.float64, device="cuda")
    want = 6.0 * b
    want -= c
    if wide == "n":
        mg.dgemm("N", "N", 1, size, 1, 2.0, a, 1, b, 1, -1.0, c, 1)
    else:
        mg.dgemm("N", "N", size, 1, 1, 2.0, b, size, a, 1, -1.0, c, size)
    assert torch.equal(c, want)


@pytest.mark.parametrize("mode", [0, 1])
def test_sgemm_wide(mode):
    import torch
    import paper_1608_05265_amd as mg
    n = 1 << 27
    b, c = _vectors(n, torch.float32)
    a = torch.tensor([3.0], device="cuda")
    want = 6.0 * b
    want -= c
    mg.sgemm("N", "N", 1, n, 1, 2.0, a, 1, b, 1, -1.0, c, 1, mode=mode)
    assert torch.equal(c, want)
