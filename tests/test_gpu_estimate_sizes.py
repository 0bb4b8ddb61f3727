"""The estimate over datasets of many small meshes with large ones among them:
those a wave takes, those it leaves to its block, and more than a block's list."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,large", [(700, {3: 4, 5: 5, 600: 5}), (700, {0: 5, 1: 5, 2: 5, 3: 5}),
                                     (41_000, {4 * b + w + 8192 * i: 5 for b in (0, 7) for w in range(4) for i in range(5)})])
def test_estimate_with_large_meshes_among_small_ones(n, large):
    import oracle
    import paper_2609_24513_amd as pa
    from paper_2609_24513_amd import dataset, synth
    rng = np.random.default_rng(n + len(large))
    ico = {k: synth.icosphere(k) for k in (4, 5)}  # 5,120 and 20,480 triangles
    side = n ** (1 / 3)

    def meshes():
        c = rng.uniform(0, side, (n, 3))
        out = []
        for k in range(n):
            if k in large:
                v, f = ico[large[k]]
                out.append(((c[k] + rng.uniform(1, 2) * v).astype(np.float32), f))
            else:
                out.append(((c[k] + rng.uniform(0.5, 1.0) * synth._CUBE_V).astype(np.float32), synth._CUBE_F))
        return synth.concat_meshes(out)

    A, B = meshes(), meshes()
    assert max(np.diff(A.face_off)) > 4096 and A.faces.shape[0] <= 512 * n
    ga, gb = pa.MeshBlob.build(A), pa.MeshBlob.build(B)
    got = dataset.estimate(ga, gb, 8)
    want = oracle.estimate.estimate(A, B, oracle.mesh_boxes(A), oracle.mesh_boxes(B), 8)["estimate"]
    assert want > 0
    # FP64 sums in another order
    assert got == pytest.approx(want, rel=1e-9, abs=1e-9)
