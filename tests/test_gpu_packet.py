"""The default packet traversal at the edges of its work distribution: queues of
one entry up to several pop batches, fewer blocks than queues, waves that only
help, roots with leaf children, and leaves of up to eight triangles.  Flags
are bit-exact with the CPU oracle."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _shapes(rng, n, kinds):
    from paper_2609_24513_amd import synth
    cube_v, cube_f = synth._CUBE_V, synth._CUBE_F
    out = []
    for k in range(n):
        kind = kinds[k % len(kinds)]
        c = rng.uniform(0.0, 2.2, size=3)
        if kind == 0:      # 12 triangles: a root whose children are all leaves
            v, f = 0.9 * cube_v, cube_f
        else:              # 80 / 320 / 1,280 triangles
            v, f = synth.icosphere(kind)
        out.append(((c + rng.uniform(0.4, 0.8) * v).astype(np.float32), f))
    return synth.concat_meshes(out)


@pytest.mark.parametrize("width,leaf", [(2, 1), (4, 4), (8, 1), (8, 8)])
@pytest.mark.parametrize("kinds", [(0,), (1, 0), (2, 3)])
def test_packet_distribution_matches_oracle(oracle_mod, width, leaf, kinds):
    import torch
    import paper_2609_24513_amd as pa
    rng = np.random.default_rng(100 * width + 10 * leaf + len(kinds) + kinds[0])
    n = 18
    A, B = _shapes(rng, n, kinds), _shapes(rng, n, kinds[::-1])
    every = np.array([(i, j) for i in range(n) for j in range(n)], np.int32)
    want = oracle_mod.join(A, B, every, mode=1)
    assert 0 < want.sum() < want.size
    ga, gb = pa.MeshBlob.build(A, width=width, leaf_size=leaf), pa.MeshBlob.build(B, width=width, leaf_size=leaf)
    for count in (1, 2, 15, 16, 17, 33, every.shape[0]):
        for kw in (dict(), dict(grid_blocks=1), dict(grid_blocks=7), dict(grid_blocks=64), dict(trace_budget=-1),
                   dict(precision=1), dict(precision=2)):
            sel = rng.permutation(every.shape[0])[:count]
            flags, _, status = pa.refine(ga, gb, every[sel], pa.RefineConfig(**kw))
            torch.cuda.synchronize()
            assert int(status.item()) == 0, (count, kw)
            got = flags.cpu().numpy()
            assert np.array_equal(got, want[sel]), (count, kw, np.nonzero(got != want[sel])[0][:5])
