"""The build's sorts and plan at the sizes where another way of doing them
begins, the blob checked section by section as in test_gpu_build."""
import os
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import test_gpu_build as tb  # noqa: E402


def _check(monkeypatch, meshes, width, leaf, builder=0):
    monkeypatch.setattr(tb, "_case", lambda name: meshes)
    tb.test_blob_sections("given", width, leaf, builder)


@pytest.mark.parametrize("width,leaf", [(2, 1), (4, 4), (8, 8)])
def test_meshes_that_one_wave_sorts(monkeypatch, width, leaf):
    """Up to 64 faces, up to 64 half-edges (21 faces), and the next sizes; shared and repeated edges."""
    rng = np.random.default_rng(width)
    meshes = [tb._soup(rng, n) for n in (1, 2, 20, 21, 22, 63, 64, 65)]
    meshes += [tb._book(n) for n in (5, 21, 22)] + [tb._surface(n) for n in (8, 18, 32)]
    # equal centroids and midpoints: codes that tie
    v = np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0], [1, 1, 0], [0.5, 0.5, 1], [0.5, 0.5, -1]], np.float32)
    meshes.append((v, np.array([[0, 3, 4], [3, 0, 5], [1, 2, 4], [2, 1, 5], [0, 3, 5], [1, 2, 5]], np.int32)))
    _check(monkeypatch, meshes, width, leaf)


@pytest.mark.parametrize("n", [2047, 2048, 2049, 4097])
def test_plans_of_one_block_and_of_several(monkeypatch, n):
    rng = np.random.default_rng(n)
    meshes = [tb._soup(rng, int(k)) for k in rng.integers(1, 6, n)]
    for k in (0, 1023, 1024, 2047, n - 1):
        if k < n:
            meshes[k] = tb._soup(rng, 700)
    for k in (5, 2040):
        meshes[k] = (np.zeros((0, 3), np.float32), np.zeros((0, 3), np.int32))
    _check(monkeypatch, meshes, 4, 2)
