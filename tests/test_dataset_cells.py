"""The estimate's grid resolution against its definition in numpy, also where
extent / (4 mean sides) is next to a whole number and the order of the sum decides."""
import numpy as np
import pytest


class _Boxes:
    def __init__(self, b):
        self.b = np.ascontiguousarray(b, np.float32)

    def boxes(self):
        import torch
        return torch.from_numpy(self.b.reshape(-1, 6))


def _cells(a, b, per_side=4.0, max_cells=64):
    x = np.concatenate([a.b.reshape(-1, 6), b.b.reshape(-1, 6)]).astype(np.float64)
    x = x[np.all(x[:, 3:] >= x[:, :3], axis=1)]
    if x.shape[0] == 0:
        return 1
    side = float((x[:, 3:] - x[:, :3]).mean())
    extent = float((x[:, 3:].max(axis=0) - x[:, :3].min(axis=0)).max())
    return int(min(max_cells, max(1, np.floor(extent / max(per_side * side, 1e-30)))))


@pytest.mark.parametrize("n", [100, 1000, 3000])
@pytest.mark.parametrize("m", [2, 5, 10])
def test_next_to_a_whole_number(n, m):
    from paper_2609_24513_amd import dataset
    for e in range(-56, -44):
        rng = np.random.default_rng(e + 100)
        lo, hi = np.zeros((2 * n, 3)), np.full((2 * n, 3), 2.0 ** e)  # half of the boxes are tiny
        pos = rng.integers(0, 2 * m, (n, 3))
        pos[0], pos[1] = 0, 2 * m - 1
        lo[:n], hi[:n] = pos, pos + 1
        b = np.concatenate([lo, hi], 1)[rng.permutation(2 * n)]
        A, B = _Boxes(b[:n]), _Boxes(b[n:])
        assert dataset.auto_cells(A, B) == _cells(A, B)


@pytest.mark.parametrize("n,scale", [(0, 1.0), (1, 1.0), (7, 1e-30), (500, 1e20), (500, 0.3)])
def test_drawn_boxes_with_empty_meshes(n, scale):
    from paper_2609_24513_amd import dataset
    rng = np.random.default_rng(n)
    lo = rng.uniform(0, 30, (2 * n, 3))
    b = np.concatenate([lo, lo + rng.uniform(0, 2, (2 * n, 3))], 1) * scale
    b[3::11, :3], b[3::11, 3:] = np.inf, -np.inf
    A, B = _Boxes(b[:n]), _Boxes(b[n:])
    assert dataset.auto_cells(A, B) == _cells(A, B)
