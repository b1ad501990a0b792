"""The built-in choice of a configuration (no tuning table): every size gets
one of its mode that runs without a workspace, and the choice follows what
the model is made of -- whole cards of tiles take large tiles, few tiles small
ones, and a ragged size the same as its neighbours."""
import os
import re

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


def test_every_row_names_a_configuration():
    """A row whose configuration is gone would be left out without a word."""
    src = open(os.path.join(os.path.dirname(mg.__file__), "csrc", "api.cpp")).read()
    for mode, table in ((0, "FP32_ROWS"), (1, "X3_ROWS")):
        body = re.search(r"const CostRow %s\[\] = \{(.*?)\n\};" % table, src, re.S).group(1)
        rows = re.findall(r'\{"(\w+)"', body)
        names = {c["name"] for c in mg.configs(mode)}
        assert len(rows) >= 10 and set(rows) <= names, set(rows) - names


@pytest.mark.parametrize("mode", [0, 1])
def test_tuner_times_each_kernel_once(mode):
    from paper_1608_05265_amd import autotune
    shape = lambda c: tuple(v for k, v in c.items() if k not in ("id", "name"))
    kept, every = autotune.kernels(mode), mg.configs(mode)
    assert {shape(c) for c in kept} == {shape(c) for c in every}
    if mode == 0:
        assert len(kept) == len({shape(c) for c in every}) < len(every)
    else:
        assert kept == every
