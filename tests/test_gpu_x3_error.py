"""The split form's default choice around 2048 is no further off than the tile
that once was the tuned one there, with the leading products in a sum of their
own."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k", [(2348, 4032, 1664), (2048, 2048, 2048)])
def test_default_choice_error(m, n, k):
    """rms over four million entries and more: two of the same order differ by a
    few thousandths, one sum instead of two by a factor of 2.75."""
    import torch
    import paper_1608_05265_amd as mg
    cfg = {c["name"]: c["id"] for c in mg.configs(1)}["x3d_128x128x32_w64x64"]
    g = torch.Generator("cuda").manual_seed(73)
    A = torch.empty(k, m, device="cuda").uniform_(-1, 1, generator=g)  # column-major m x k
    B = torch.empty(n, k, device="cuda").uniform_(-1, 1, generator=g)
    exact = B.double() @ A.double()
    C = torch.empty(n, m, device="cuda")
    rms = lambda: float((C.double() - exact).pow(2).mean().sqrt())
    mg.sgemm_config("N", "N", m, n, k, 1.0, A, m, B, k, 0.0, C, m, 1, cfg)
    other = rms()
    mg.sgemm("N", "N", m, n, k, 1.0, A, m, B, k, 0.0, C, m, mode=1)
    assert rms() <= 1.05 * other, (rms(), other)
