"""A request that fails ends the run only when no batch writes the server's
buffers any more (they may die with it)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("graphs", [True, False])
def test_a_failing_batch_leaves_nothing_in_flight(monkeypatch, graphs):
    import torch
    import paper_2609_24513_amd as pa
    from paper_2609_24513_amd import serve, synth
    A, B = synth.make_c1()
    ga, gb = pa.MeshBlob.build(A), pa.MeshBlob.build(B)
    srv = serve.JoinServer(ga, gb, max_req_per_batch=2, max_pairs=64, slots=3, graphs=graphs)
    start = srv._start

    def slow_start(slot, reqs):
        start(slot, reqs)
        if slot is not srv.slots[0]:
            with torch.cuda.stream(slot.stream):
                torch.cuda._sleep(400_000_000)  # some tenths of a second

    def fail(slot, now):
        raise ValueError("no")

    box = np.array([-9] * 3 + [9] * 3, np.float32)
    trace = [serve.Request(k, 0.0, box) for k in range(6)]
    assert all(r.t_done >= 0 for r in srv.run(trace, realtime=False))
    monkeypatch.setattr(srv, "_start", slow_start)
    monkeypatch.setattr(srv, "_finish", fail)
    with pytest.raises(ValueError):
        srv.run([serve.Request(k, 0.0, box) for k in range(6)], realtime=False)
    assert all(slot.stream.query() for slot in srv.slots)
