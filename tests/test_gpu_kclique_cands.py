"""The plain k-clique search's candidate tasks, whose intersections the
wavefront runs together: candidate streams around its 64-element chunks and
its 256-element rounds, empty lists, long lists next to short ones, one queue
and several (the candidates' vertices are then kept between the two passes
over the children, up to 1024 of them).  Counts and task counts equal the
oracle's."""
import numpy as np
import pytest

import oracle
from synth import graphs

pytestmark = pytest.mark.gpu


def clique_with_tail(n, tail):
    """A clique of n vertices followed by a path of `tail` vertices."""
    e = [(a, b) for a in range(n) for b in range(a + 1, n)]
    e += [(n - 1 + i, n + i) for i in range(tail)]
    return graphs.oriented_from_edges(n + tail, np.array(e), order="id")


@pytest.mark.parametrize("queues", [1, 4])
def test_candidate_streams(queues):
    from paper_2604_05982_amd import gtap
    opts = dict(num_queues=queues, daq_policy=2, daq_bounds=[8, 32, 128]) if queues > 1 else {}
    cases = [(clique_with_tail(n, 3), k) for n in (3, 4, 9, 16, 17, 23, 24) for k in (3, 4, 5)]
    cases += [(clique_with_tail(n, 0), 3) for n in (63, 64, 65, 66, 130)]  # over 1024 children in one iteration
    rng = np.random.default_rng(queues)
    for n, p in ((70, 0.9), (300, 0.2), (65, 0.02)):
        e = [(a, b) for a in range(n) for b in range(a + 1, n) if rng.random() < p]
        cases += [(graphs.oriented_from_edges(n, np.array(e).reshape(-1, 2), order=o, seed=1), k)
                  for o in ("id", "random", "degeneracy") for k in (3, 4)]
    with gtap.Runtime(timeout_ms=60000, num_waves=64, small_frames=1 << 20, big_frames=1 << 17, big_frame_ints=320,
                      **opts) as rt:
        for g, k in cases:
            want = oracle.kclique(g.row_ptr, g.col, k)
            job = rt.submit_kclique(g.row_ptr32, g.col, k, range_leaf=64)
            rt.run()
            st = rt.stats()
            assert rt.result(job) == want.value, (g.n, k)
            assert (st["tasks"], st["conts"]) == (want.tasks, want.conts), (g.n, k)
