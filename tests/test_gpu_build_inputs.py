"""What the build does with inputs that it refuses: nothing is written outside
the blob and the workspace, and the status names the first bad face."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GUARD = 1 << 16


def _build(verts, faces, vert_off, face_off, width=4, leaf=4):
    """build_mesh_bvh with guard bytes on both sides of the blob and of the
    workspace: (status, guards untouched)."""
    import torch
    from paper_2609_24513_amd import _lib
    lib = _lib.load()
    prm = _lib.BvhParams(width, leaf, 0, 0)
    M, F, V = len(face_off) - 1, faces.shape[0], verts.shape[0]
    bb, wb = ctypes.c_size_t(0), ctypes.c_size_t(0)
    _lib.check(lib.build_mesh_bvh_sizes(M, F, V, ctypes.byref(prm), ctypes.byref(bb), ctypes.byref(wb)))
    bufs = [torch.full((2 * GUARD + n.value,), 0xA5, dtype=torch.uint8, device="cuda") for n in (bb, wb)]
    dev = [torch.as_tensor(x).cuda() for x in (verts, vert_off, faces, face_off)]
    status = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    _lib.check(lib.build_mesh_bvh(dev[0].data_ptr(), dev[1].data_ptr(), dev[2].data_ptr(), dev[3].data_ptr(), M, V, F,
                                  ctypes.byref(prm), bufs[0].data_ptr() + GUARD, bb.value, bufs[1].data_ptr() + GUARD,
                                  wb.value, status.data_ptr(), None))
    torch.cuda.synchronize()
    clean = all(bool((b[:GUARD] == 0xA5).all()) and bool((b[-GUARD:] == 0xA5).all()) for b in bufs)
    return int(status.item()), clean


def _faces(n):
    f = np.stack([np.arange(n), np.arange(n) + 1, np.arange(n) + 2], 1).astype(np.int32)
    v = np.random.default_rng(n).uniform(-1, 1, size=(n + 2, 3)).astype(np.float32)
    return v, f


@pytest.mark.parametrize("name", ["alternating", "one_after", "past_the_end", "negative", "not_from_zero", "vertices"])
def test_offsets_that_overlap_or_leave_the_arrays(name):
    v, f = _faces(1000)
    F, V = f.shape[0], v.shape[0]
    fo = {"alternating": [0, F] * 20 + [F], "one_after": [0, F] * 20 + [0, 1, F], "past_the_end": [0, F + 5, F],
          "negative": [0, -4, F], "not_from_zero": [3, 500, F], "vertices": [0, 500, F]}[name]
    vo = np.array([0] + [V] * (len(fo) - 1), np.int64)
    if name == "vertices":
        vo = np.array([0, V + 1, V], np.int64)
    fo = np.array(fo, np.int64)
    status, clean = _build(v, f, vo, fo)
    assert clean and status == 0


def test_sound_offsets_with_the_same_helper():
    v, f = _faces(1000)
    assert _build(v, f, np.array([0, 1002], np.int64), np.array([0, 1000], np.int64)) == (-1, True)


@pytest.mark.parametrize("check", [True, False])
def test_build_on_another_stream_is_waited_for(check):
    """The status and the exponent range are read behind the build, though its
    stream is busy when it is enqueued."""
    import torch
    import paper_2609_24513_amd as pa
    from paper_2609_24513_amd import synth
    rng = np.random.default_rng(5)
    v = np.array([[0, 0, 0], [1, 0, 0], [0, 2, 0], [0, 0, 8]], np.float32)
    f = np.array([[0, 2, 1], [0, 1, 3], [0, 3, 2], [1, 2, 3]], np.int32)
    good = synth.concat_meshes([(v, f)] * 40)
    bad = synth.MeshSet(good.verts, good.faces.copy(), good.vert_off, good.face_off)
    bad.faces[77, 1] = 99
    pa.MeshBlob.build(good)  # the kernels are loaded
    s = torch.cuda.Stream()
    for k in range(3):
        torch.cuda.synchronize()
        # the words' memory holds what an earlier build left: neither -1 nor a face, nor a range
        junk = torch.full((1 << 16,), -1000 - k, dtype=torch.int32, device="cuda")
        torch.cuda.synchronize()
        del junk
        with torch.cuda.stream(s):
            torch.cuda._sleep(int(rng.integers(20_000_000, 60_000_000)))
        if check:
            assert pa.MeshBlob.build(good, stream=s).exp_range() == (0, 3)
            with torch.cuda.stream(s):
                torch.cuda._sleep(20_000_000)
            with pytest.raises(pa.PierceError):
                pa.MeshBlob.build(bad, stream=s)
        else:
            g = pa.MeshBlob.build(good, stream=s, check_status=False)
            assert g.exp_range() == (0, 3) and g.status() == -1
            b = pa.MeshBlob.build(bad, stream=s, check_status=False)
            assert b.status() == 77


def test_more_meshes_than_one_grid_dimension_takes():
    """2^23 + 5 meshes of one triangle: a block each of 512 threads is beyond 2^32 threads."""
    import torch
    import paper_2609_24513_amd as pa
    from paper_2609_24513_amd import synth
    M = (1 << 23) + 5
    g = torch.Generator(device="cuda").manual_seed(1)
    v = torch.rand(M, 3, 3, generator=g, device="cuda")
    f = torch.arange(3, dtype=torch.int32, device="cuda").expand(M, 3).contiguous()
    off = torch.arange(M + 1, device="cuda")
    blob = pa.MeshBlob.build(synth.MeshSet(v.reshape(-1, 3), f, 3 * off, off), width=8, leaf_size=1)
    want = torch.cat([v.amin(dim=1), v.amax(dim=1)], dim=1)
    assert torch.equal(blob.boxes(), want)
    assert bool((blob.edge_counts() == 3).all())
    # the last meshes meet themselves and their neighbours as the first do
    k = 600
    pairs = torch.cat([torch.arange(k), torch.arange(M - k, M)]).int()[:, None].expand(-1, 2).cuda()
    flags, _, status = pa.refine(blob, blob, pairs)
    torch.cuda.synchronize()
    assert int(status.item()) == 0 and bool(flags.bool().all())


@pytest.mark.parametrize("at", [0, 1500, 2600, 4999])
def test_bad_offsets_among_many_meshes(at):
    v, f = _faces(10_000)
    fo, vo = 2 * np.arange(5001, dtype=np.int64), np.full(5001, v.shape[0], np.int64)
    vo[0] = 0
    f = f % 3  # every mesh after the first has no vertices of its own, so its faces are bad too
    ok_status, clean = _build(v, f, vo, fo)
    assert clean and ok_status == 2
    fo[at + 1 if at < 4999 else at] = 3 if at else 9_000
    status, clean = _build(v, f, vo, fo)
    assert clean and status == 0
