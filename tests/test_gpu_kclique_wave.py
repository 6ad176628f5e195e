"""Split k-clique bodies run by the whole wavefront, at the sizes where their
paths change: out-degrees around multiples of 64 (words per row), 384 (the
largest matrix kept in LDS) and beyond, clique sizes on both sides of the
register search (five members inside an edge's candidates), thresholds that
send a vertex to its in-place, row and edge forms, hubs whose out-lists are
longer and shorter than their neighbours'.  Counts equal the oracle's."""
import numpy as np
import pytest

import oracle
from synth import graphs

pytestmark = pytest.mark.gpu


def hub_graph(d, p, seed, fringe=40):
    """Vertex 0 with d out-neighbours, those joined with probability p, and a
    fringe of low-degree vertices in front of them."""
    rng = np.random.default_rng(seed)
    i, j = np.triu_indices(d, 1)
    keep = rng.random(i.size) < p
    core = np.stack([i[keep], j[keep]], 1) + 1 + fringe
    hub = np.stack([np.full(d, fringe), np.arange(d) + 1 + fringe], 1)
    ends = rng.integers(fringe, d + 1 + fringe, size=(fringe * 6, 2))
    ends[:, 0] = rng.integers(0, fringe, size=fringe * 6)
    return graphs.oriented_from_edges(d + 1 + fringe, np.concatenate([core, hub, ends]), order="id")


CASES = [(20, 0.8), (63, 0.6), (64, 0.6), (65, 0.55), (128, 0.4), (129, 0.4), (192, 0.33), (256, 0.28), (321, 0.25),
         (384, 0.22), (385, 0.22), (600, 0.15)]


@pytest.mark.parametrize("algorithm", ["orient", "pivot"])
@pytest.mark.parametrize("threshold", [0, 20, 64])
def test_hub_graphs(algorithm, threshold):
    import torch
    from paper_2604_05982_amd import gtap
    alg = gtap.GTAP_KCLIQUE_PIVOT if algorithm == "pivot" else gtap.GTAP_KCLIQUE_ORIENT
    built = [hub_graph(d, p, 7 * d) for d, p in CASES]
    with gtap.Runtime(waves_per_group=4, small_frames=1 << 22, big_frames=1 << 20, deque_capacity=1 << 17,
                      big_frame_ints=gtap.kclique_split_buffer_ints(1024), timeout_ms=60000) as rt:
        for k in (4, 5, 7, 8):
            jobs = []
            for g in built:  # one launch: lanes of a wavefront hold tasks of different jobs
                rp, col = torch.as_tensor(g.row_ptr32).cuda(), torch.as_tensor(g.col).cuda()
                jobs.append((g, rt.submit_kclique_split(rp, col, k, threshold=threshold, algorithm=alg,
                                                        max_outdeg=g.max_outdeg)))
            print(f"{algorithm} threshold {threshold} k {k}", flush=True)
            rt.run()
            for g, job in jobs:
                assert rt.result(job) == oracle.kclique(g.row_ptr, g.col, k).value, (g.max_outdeg, k)
