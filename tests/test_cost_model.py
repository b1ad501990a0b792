"""The built-in choice of a configuration (no tuning table): every size gets
one of its mode that runs without a workspace, and the choice follows what
the model is made of -- whole cards of tiles take large tiles, few tiles small
ones, and a ragged size the same as its neighbours."""
import numpy as np
import pytest

import paper_1608_05265_amd as mg


@pytest.fixture(autouse=True)
def no_table():
    mg.load_tuning(None)
    yield
    mg.load_tuning(mg.TUNING_PATH)


@pytest.mark.parametrize("mode", [0, 1])
def test_every_size_has_a_choice(mode):
    rng = np.random.default_rng(3)
    cfgs = {c["id"]: c for c in mg.configs(mode)}
    sizes = [(0, 5, 5), (5, 0, 5), (5, 5, 0), (1, 1, 1), (1, 1, 1 << 24), (1 << 20, 1, 1), (1, 1 << 20, 3)]
    sizes += [tuple(int(v) for v in np.exp(rng.uniform(0, 10, 3))) for _ in range(300)]
    for m, n, k in sizes:
        c = cfgs[mg.select_config("N", "T", m, n, k, mode)]
        assert not c["packed"], (m, n, k, c["name"])


@pytest.mark.parametrize("mode,large,small", [(0, 128 * 128, 32 * 32), (1, 256 * 256, 32 * 32)])
def test_tile_follows_the_size(mode, large, small):
    cfgs = {c["id"]: c for c in mg.configs(mode)}
    area = lambda m, n, k: (lambda c: c["bm"] * c["bn"])(cfgs[mg.select_config("N", "N", m, n, k, mode)])
    for s in (8192, 8191, 10000):
        assert area(s, s, s) >= large
    for s in (64, 100, 200, 256):
        assert area(s, s, s) <= small
    for s in (900, 1000, 1024):
        assert small < area(s, s, 2048) < large or area(s, s, 2048) == 64 * 64


@pytest.mark.parametrize("mode", [0, 1])
def test_choice_fits_a_launch(mode):
    """A launch holds less than 2^32 threads: thin and very wide problems take
    a tile whose launch does."""
    cfgs = {c["id"]: c for c in mg.configs(mode)}
    for m, n, k in ((1, 1 << 27, 16), (16, 1 << 27, 16), (1, 1 << 28, 64), (1 << 28, 1, 64),
                    (32, 1 << 29, 8), (1 << 29, 1, 300), (1, (1 << 31) - 1024, 1)):
        c = cfgs[mg.select_config("N", "N", m, n, k, mode)]
        tiles = -(-m // c["bm"]) * -(-n // c["bn"])
        assert tiles * c["threads"] < 1 << 32, (m, n, k, c["name"])
