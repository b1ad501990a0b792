"""Long inner products over few outputs: the error of the default choice is no
larger than that of sixteen partial sums per output, each a chain of fused
multiply-adds in float32, added at the end."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k", [(128, 512, 8192), (200, 96, 4096), (61, 300, 11264)])
def test_skinny_error(m, n, k):
    """The measured rms over an output block of 64 x 64 may be a tenth above
    the chains' (4096 entries: its own spread is 1 %; one chain less per pair
    would be 1.4 times as far off)."""
    import torch
    import paper_1608_05265_amd as mg
    rng = np.random.default_rng(72)
    a, b = rng.uniform(-1, 1, (m, k)).astype(np.float32), rng.uniform(-1, 1, (k, n)).astype(np.float32)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    C = torch.zeros(m * n, device="cuda")
    mg.sgemm("N", "N", m, n, k, 1.0, dev(a.T), m, dev(b.T), k, 0.0, C, m)
    got = C.cpu().numpy().reshape(n, m).T[:61, :64]
    a, b = a[:61], b[:, :64]
    exact = a.astype(np.float64) @ b.astype(np.float64)
    chains = np.zeros((16, 61, 64), np.float32)
    ac, bc = a.reshape(61, 16, k // 16), b.reshape(16, k // 16, 64)
    for s in range(k // 16):
        prod = ac[:, :, s].T[:, :, None].astype(np.float64) * bc[:, s, None, :]
        chains = (prod + chains).astype(np.float32)
    total = chains[0]
    for c in chains[1:]:
        total = total + c
    rms = lambda x: float(np.sqrt(np.mean((x - exact) ** 2)))
    assert rms(got) <= 1.1 * rms(total), (rms(got), rms(total))
