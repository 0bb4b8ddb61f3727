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
    meshes = [(v.astype(np.float32), f.astype(np.int32)) for v, f in meshes]
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


def _far(v, f, stretch):
    """The mesh with a triangle that stretches its box."""
    far = np.array([[0, 0, 0], [0.9, 1, 0.8], [1, 0.9, 1]]) * stretch
    return (np.concatenate([v, far]).astype(np.float32),
            np.concatenate([f, [[len(v), len(v) + 1, len(v) + 2]]]).astype(np.int32))


def _unit(mesh):
    v, f = mesh
    v = v.astype(np.float64) - v.min(0)
    return v / v.max(), f


def _join(*meshes):
    n = np.cumsum([0] + [m[0].shape[0] for m in meshes])
    return (np.concatenate([m[0] for m in meshes]).astype(np.float32),
            np.concatenate([m[1] + k for m, k in zip(meshes, n)]).astype(np.int32))


def _fan(n):
    """n faces about one vertex."""
    a = 2 * np.pi * np.arange(n + 1) / (n + 1)
    v = np.concatenate([[[0, 0, 0.3]], np.stack([np.cos(a), np.sin(a), 0 * a], 1)])
    i = 1 + np.arange(n)
    return v, np.stack([0 * i, i, i + 1], 1)


def _clustered(name):
    rng = np.random.default_rng(sum(map(ord, name)))
    if name == "stretched":  # cells of a few codes, of one, and a mesh of several such cells
        out = [_far(*_unit(tb._surface(n)), s) for n, s in ((20_000, 30), (20_000, 3000), (5000, 300), (1500, 1e4))]
        return out + [_far(*_unit(tb._soup(rng, 12_000)), 1e4)]
    if name == "nested":     # a part far smaller than its neighbours in the cell, twice over
        a, b, c = (_unit(tb._surface(n)) for n in (6000, 8000, 9000))
        return [_far(*_join((a[0] * 1e-2, a[1]), (b[0] * 1e-4, b[1]), (c[0] * 1e-6, c[1])), 50)]
    if name == "copies":     # one edge of thousands of faces, alone in its cell and among others
        b = tb._book(9000)
        return [tb._book(20_000), _far(*b, 1e4), _far(*_join(b, _unit(tb._surface(4000))), 1e5)]
    if name == "fan":        # equal codes and equal first vertices
        return [_far(*_fan(6000), 1e5), _fan(3000)]
    if name == "limits":     # cells of 2,046 to 2,052 half-edges, of 2,047 to 2,049 triangles
        return [_far(*_unit(tb._soup(rng, n)), 1e5) for n in (682, 683, 684, 2047, 2048, 2049)]
    # two full cells that start in one unit
    a, b = _unit(tb._soup(rng, 400)), _unit(tb._soup(rng, 682))
    c, d = _unit(tb._soup(rng, 1200)), _unit(tb._soup(rng, 2048))
    return [_far(*_join((x[0], x[1]), (y[0] + 400.0, y[1])), 1000) for x, y in ((a, b), (b, a), (c, d), (d, c))]


@pytest.mark.parametrize("width,leaf", [(4, 4), (8, 1)])
@pytest.mark.parametrize("name", ["stretched", "nested", "copies", "fan", "limits", "two_cells"])
def test_detail_packed_into_few_cells(monkeypatch, name, width, leaf):
    _check(monkeypatch, _clustered(name), width, leaf)
