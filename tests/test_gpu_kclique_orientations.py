"""Split k-clique search on acyclic orientations whose vertex ids do not ascend
along the edges: out-lists are sorted by id, as the contract asks, but hold ids
below their own vertex (vertex 0 among them).  Rows of matrices and vertices
counted in place, out-degrees around a word and beyond the matrices kept in
LDS.  Counts equal the oracle's and those of the ascending labelling."""
import numpy as np
import pytest

import oracle
from synth import graphs

pytestmark = pytest.mark.gpu


def relabelled(g, ids):
    """g with vertex v named ids[v]: the same edges and directions, out-lists
    sorted by the new names."""
    ids = np.asarray(ids)
    src = np.repeat(np.arange(g.n), np.diff(g.row_ptr))
    u, w = ids[src], ids[g.col[: src.size]]
    at = np.lexsort((w, u))
    row_ptr = np.concatenate([[0], np.cumsum(np.bincount(u, minlength=g.n))])
    return row_ptr.astype(np.int32), w[at].astype(np.int32)


def clique(n):
    return graphs.oriented_from_edges(n, np.array([(a, b) for a in range(n) for b in range(a + 1, n)]), order="id")


def hub(d, p, seed):
    """Vertex 0 with d out-neighbours, those joined with probability p."""
    rng = np.random.default_rng(seed)
    i, j = np.triu_indices(d, 1)
    keep = rng.random(i.size) < p
    e = np.concatenate([np.stack([i[keep], j[keep]], 1) + 1, np.stack([np.zeros(d, int), np.arange(d) + 1], 1)])
    return graphs.oriented_from_edges(d + 1, e, order="id")


@pytest.mark.parametrize("algorithm", ["orient", "pivot"])
@pytest.mark.parametrize("threshold", [0, 20, 64])
def test_any_acyclic_orientation(algorithm, threshold):
    import torch
    from paper_2604_05982_amd import gtap
    alg = gtap.GTAP_KCLIQUE_PIVOT if algorithm == "pivot" else gtap.GTAP_KCLIQUE_ORIENT
    built = [clique(4), clique(6), clique(12), graphs.chung_lu(400, 20, 2.3, 1.0, 3)]
    built += [hub(d, p, d) for d, p in ((20, 0.8), (64, 0.5), (65, 0.5), (130, 0.35), (385, 0.15))]
    rng = np.random.default_rng(11)
    with gtap.Runtime(waves_per_group=4, small_frames=1 << 22, big_frames=1 << 20, deque_capacity=1 << 17,
                      big_frame_ints=gtap.kclique_split_buffer_ints(1024), timeout_ms=60000) as rt:
        for k in (4, 5, 6, 7, 8):
            jobs = []
            for g in built:
                want = oracle.kclique(g.row_ptr, g.col, k).value
                for name, ids in (("descending", np.arange(g.n)[::-1]), ("random", rng.permutation(g.n)),
                                  ("rotated", (np.arange(g.n) + g.n // 2) % g.n)):
                    rp, col = relabelled(g, ids)
                    assert oracle.kclique(rp, col, k).value == want
                    jobs.append(((g.n, k, name), want,
                                 rt.submit_kclique_split(torch.as_tensor(rp).cuda(), torch.as_tensor(col).cuda(), k,
                                                         threshold=threshold, algorithm=alg, max_outdeg=g.max_outdeg)))
            print(f"{algorithm} threshold {threshold} k {k}", flush=True)
            rt.run()
            for what, want, job in jobs:
                assert rt.result(job) == want, what
