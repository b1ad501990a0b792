"""K loops of none to eight blocks, with and without a ragged one, through
every configuration, split or not, and through a batched plan: the straight-line
part of the loop, its last blocks and the reuse of the LDS stages.  Entries
are integers of at most 8, so every product, part product and partial sum is
exact in any order and the results must be equal."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _operands(rng, ta, tb, m, n, k):
    import torch
    a, b, c = (rng.integers(-8, 9, size=s).astype(np.float32) for s in ((m, k), (k, n), (m, n)))
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()
    return (dev(a if ta == "T" else a.T), dev(b if tb == "T" else b.T), dev(c.T),
            2.0 * (a.astype(np.float64) @ b) - c)


def _lengths(bk):
    return [1, bk, 2 * bk, 2 * bk + 3, 3 * bk, 4 * bk + 1, 5 * bk, 6 * bk, 7 * bk + 2]


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("ta,tb", [("N", "N"), ("N", "T"), ("T", "N"), ("T", "T")])
def test_every_config_exact(mode, ta, tb):
    import paper_1608_05265_amd as mg
    rng = np.random.default_rng(5)
    for cfg in mg.configs(mode):
        m, n = cfg["bm"] + 5, cfg["bn"] * 2 - 3
        for k in _lengths(cfg["bk"]):
            A, B, C, want = _operands(rng, ta, tb, m, n, k)
            lda, ldb = (m if ta == "N" else k), (k if tb == "N" else n)
            first = C.clone()
            mg.sgemm_config(ta, tb, m, n, k, 2.0, A, lda, B, ldb, -1.0, C, m, mode, cfg["id"])
            assert np.array_equal(C.cpu().numpy().T, want), (cfg["name"], ta, tb, m, n, k)
            if cfg["splitk"] and k >= 2 * cfg["bk"]:
                mg.sgemm_split(ta, tb, m, n, k, 2.0, A, lda, B, ldb, -1.0, first, m, mode, cfg["id"], 8, 2)
                assert np.array_equal(first.cpu().numpy().T, want), ("split", cfg["name"], ta, tb, m, n, k)


@pytest.mark.parametrize("mode", [0, 1])
def test_batch_exact(mode):
    import paper_1608_05265_amd as mg
    rng = np.random.default_rng(6)
    problems, wants = [], []
    for i, k in enumerate(_lengths(16) + _lengths(32)):
        ta, tb = [("N", "N"), ("N", "T"), ("T", "N"), ("T", "T")][i % 4]
        m, n = int(rng.integers(1, 300)), int(rng.integers(1, 300))
        A, B, C, want = _operands(rng, ta, tb, m, n, k)
        problems.append((ta, tb, m, n, k, 2.0, A, m if ta == "N" else k, B, k if tb == "N" else n, -1.0, C, m))
        wants.append(want)
    plan = mg.Batch(problems, mode=mode)
    plan.launch()
    for p, want in zip(problems, wants):
        assert np.array_equal(p[11].cpu().numpy().T, want), p[:5]
