"""The query-box filter, one box and batches, against a brute-force count of
the closed-box definition: dataset sizes at the edges of the ballot words and
tiles, shares of one to several row tiles, several column tiles, empty meshes,
boxes that keep nothing or everything, and regions too small for their pairs."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _cubes(rng, n, side):
    from paper_2609_24513_amd import synth
    v = rng.uniform(0, side, size=(n, 1, 3)) + rng.uniform(0.5, 1.5, size=(n, 1, 1)) * synth._CUBE_V[None]
    meshes = [(v[k].astype(np.float32), synth._CUBE_F) for k in range(n)]
    for k in range(7, n, 50):
        meshes[k] = (np.zeros((0, 3), np.float32), np.zeros((0, 3), np.int32))
    return synth.concat_meshes(meshes)


def _want(a, b, q):
    ka = np.nonzero(np.all(a[:, :3] <= q[3:], 1) & np.all(a[:, 3:] >= q[:3], 1))[0]
    kb = np.nonzero(np.all(b[:, :3] <= q[3:], 1) & np.all(b[:, 3:] >= q[:3], 1))[0]
    out = []
    for i in ka:
        lo = np.maximum(np.maximum(b[kb, :3], a[i, :3]), q[:3])
        hi = np.minimum(np.minimum(b[kb, 3:], a[i, 3:]), q[3:])
        j = kb[np.all(lo <= hi, 1)]
        out.append(np.stack([np.full(j.size, i), j], 1))
    return np.concatenate(out).astype(np.int32) if out else np.zeros((0, 2), np.int32)


@pytest.mark.parametrize("ma,mb,side", [(1, 1, 2.0), (63, 65, 6.0), (64, 1, 5.0), (1025, 1023, 14.0), (300, 2600, 14.0),
                                        (9000, 1100, 24.0)])
def test_query_boxes(ma, mb, side):
    import torch
    import paper_2609_24513_amd as pa
    from paper_2609_24513_amd import _lib
    rng = np.random.default_rng(ma + mb)
    A, B = _cubes(rng, ma, side), _cubes(rng, mb, side)
    ga, gb = pa.MeshBlob.build(A), pa.MeshBlob.build(B)
    ba, bb = A.aabbs(), B.aabbs()
    inf = 1e30
    boxes = [np.array([-inf] * 3 + [inf] * 3), np.array([side + 50] * 6), np.array([side / 2] * 6)]
    for _ in range(9):
        c, h = rng.uniform(0, side, 3), rng.uniform(0.1, side / 2)
        boxes.append(np.concatenate([c - h, c + h]))
    boxes = np.asarray(boxes, np.float32)
    want = [_want(ba, bb, q) for q in boxes]
    assert want[1].shape[0] == 0 and (ma == 1 or want[0].shape[0] > 0)
    for q, w in zip(boxes, want):
        assert np.array_equal(pa.filter_pairs(ga, gb, query_box=q).cpu().numpy(), w)
    lib = _lib.load()
    for n, cap in ((len(boxes), max(w.shape[0] for w in want) + 3), (3, 5)):
        wb = ctypes.c_size_t(0)
        _lib.check(lib.filter_aabb_pairs_batch_ws_bytes(ma, mb, n, ctypes.byref(wb)))
        ws = torch.empty(wb.value, dtype=torch.uint8, device="cuda")
        dq = torch.as_tensor(boxes[:n]).cuda()
        out = torch.full((n * cap, 2), -7, dtype=torch.int32, device="cuda")
        cnt = torch.empty(n, dtype=torch.int64, device="cuda")
        for _ in range(2):  # the control words are cleared by every call
            _lib.check(lib.filter_aabb_pairs_batch(ga.ptr, ma, gb.ptr, mb, dq.data_ptr(), n, out.data_ptr(), cap,
                                                   cnt.data_ptr(), ws.data_ptr(), ws.numel(), None))
        torch.cuda.synchronize()
        assert cnt.tolist() == [w.shape[0] for w in want[:n]]
        got = out.cpu().numpy().reshape(n, cap, 2)
        for k in range(n):
            m = min(cap, want[k].shape[0])
            assert np.array_equal(got[k, :m], want[k][:m]) and np.all(got[k, m:] == -7)
