"""Split k-clique searches that end early: edges whose rows hold fewer candidates
than a clique needs (finished by their own lanes), and pivoting nodes counted in
place with one or two members still to be chosen, with pivots held and without.
One- and multi-word rows, matrices in LDS and beyond it.  Counts and task counts
equal the oracle's."""
import numpy as np
import pytest

import oracle
from synth import graphs
from test_gpu_kclique_split import assert_tree

pytestmark = pytest.mark.gpu


def core(d, p, seed):
    """Vertex 0 joined to the next d, those with probability p: sparse rows at
    small p, cliques throughout at 1."""
    rng = np.random.default_rng(seed)
    i, j = np.triu_indices(d, 1)
    keep = rng.random(i.size) < p
    e = np.concatenate([np.stack([i[keep], j[keep]], 1) + 1, np.stack([np.zeros(d, int), np.arange(d) + 1], 1)])
    return graphs.oriented_from_edges(d + 1, e, order="id")


@pytest.mark.parametrize("algorithm", ["orient", "pivot"])
@pytest.mark.parametrize("threshold", [0, 3, 16, 64])
def test_few_candidates(algorithm, threshold):
    import torch
    from paper_2604_05982_amd import gtap
    alg = gtap.GTAP_KCLIQUE_PIVOT if algorithm == "pivot" else gtap.GTAP_KCLIQUE_ORIENT
    built = [core(12, 1.0, 1), core(30, 0.1, 2), core(40, 0.7, 3), core(65, 0.05, 4), core(70, 0.4, 5), core(130, 0.2, 6),
             core(400, 0.02, 7), graphs.chung_lu(500, 16, 2.3, 1.0, 4)]
    with gtap.Runtime(waves_per_group=4, small_frames=1 << 22, big_frames=1 << 20, deque_capacity=1 << 17,
                      big_frame_ints=gtap.kclique_split_buffer_ints(1024), timeout_ms=60000) as rt:
        for k in (4, 5, 6, 8):
            for g in built:
                want = oracle.kclique_split(g.row_ptr, g.col, k, threshold=threshold, algorithm=algorithm)
                print(f"{algorithm} threshold {threshold} k {k} vertices {g.n}", flush=True)
                job = rt.submit_kclique_split(torch.as_tensor(g.row_ptr32).cuda(), torch.as_tensor(g.col).cuda(), k,
                                              threshold=threshold, algorithm=alg, max_outdeg=g.max_outdeg)
                rt.run()
                assert rt.result(job) == want.value == oracle.kclique(g.row_ptr, g.col, k).value
                assert_tree(rt.stats(), want, g, k, threshold)
