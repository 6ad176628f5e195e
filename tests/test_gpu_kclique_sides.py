"""The plain k-clique search's candidate tasks intersect C and N+(u) from the
shorter list: short out-lists next to long candidate lists, the other way
round, and equal ones on the lanes of one wavefront.  Counts and task counts
equal the oracle's, and a hub's time does not grow with the product of its
out-degree and its candidate list."""
import numpy as np
import pytest

import oracle
from synth import graphs

pytestmark = pytest.mark.gpu


def hub(d, tail, fringe=0):
    """Vertex 0 joined to the next d vertices, each of those to the next `tail`;
    of the last vertices some are joined to all after them."""
    e = [(0, i) for i in range(1, d + 1)] + [(i, i + j) for i in range(1, d + 1) for j in range(1, tail + 1)]
    n = d + tail + 2
    e += [(i, j) for i in range(n - fringe, n) for j in range(i + 1, n)]
    return graphs.oriented_from_edges(n, np.array(e), order="id")


@pytest.mark.parametrize("queues", [1, 4])
def test_shorter_side(queues):
    from paper_2604_05982_amd import gtap
    opts = dict(num_queues=queues, daq_policy=2, daq_bounds=[8, 32, 128]) if queues > 1 else {}
    built = [hub(d, tail, fringe) for d, tail, fringe in
             ((1, 1, 0), (2, 1, 0), (63, 1, 5), (64, 3, 20), (65, 7, 30), (300, 2, 30), (257, 4, 20), (40, 60, 12))]
    with gtap.Runtime(timeout_ms=60000, num_waves=64, small_frames=1 << 20, big_frames=1 << 18, big_frame_ints=320,
                      **opts) as rt:
        for g in built:
            for k in (3, 4, 5, 6):
                want = oracle.kclique(g.row_ptr, g.col, k)
                print(f"{queues} queues, {g.n} vertices, k {k}", flush=True)
                job = rt.submit_kclique(g.row_ptr32, g.col, k, range_leaf=64)
                rt.run()
                st = rt.stats()
                assert rt.result(job) == want.value
                assert (st["tasks"], st["conts"]) == (want.tasks, want.conts)


def test_hub_of_short_lists_is_not_quadratic():
    """16 times the out-neighbours, each with one out-neighbour: 24 times the
    comparisons from the shorter side, 256 times from the longer (spread over
    the grid: about 3 and 19 times the time)."""
    from paper_2604_05982_amd import gtap
    with gtap.Runtime(timeout_ms=60000, small_frames=1 << 20, big_frames=1 << 10) as rt:
        def ms(d):
            g = hub(d, 1)
            times = []
            for _ in range(6):
                job = rt.submit_kclique(g.row_ptr32, g.col, 3)
                rt.run()
                assert rt.result(job) == d - 1  # 0, i, i + 1 for 1 <= i < d
                times.append(rt.stats()["kernel_ms"])
            return min(times)

        assert ms(4000) < 8 * ms(250)


@pytest.mark.parametrize("labels", ["ascending", "descending", "random"])
def test_lists_cut_to_their_overlap(labels):
    """Lists of neighbouring ids, which overlap in all, a part or nothing, in
    streams on both sides of the 512 elements from which they are cut, and ids
    that do not ascend along the edges."""
    from paper_2604_05982_amd import gtap
    rng = np.random.default_rng(17)
    with gtap.Runtime(timeout_ms=60000, num_waves=64, small_frames=1 << 20, big_frames=1 << 18, big_frame_ints=320) as rt:
        for n, w in ((20, 7), (60, 8), (70, 9), (200, 8), (300, 30), (150, 64), (170, 70), (140, 130)):
            e = np.array([(i, i + j) for i in range(n) for j in range(1, w + 1) if i + j < n])
            g = graphs.oriented_from_edges(n, e, order="id")
            ids = {"ascending": np.arange(n), "descending": np.arange(n)[::-1], "random": rng.permutation(n)}[labels]
            src = np.repeat(np.arange(n), np.diff(g.row_ptr))
            u, v = ids[src], ids[g.col[: src.size]]
            at = np.lexsort((v, u))
            rp = np.concatenate([[0], np.cumsum(np.bincount(u, minlength=n))]).astype(np.int32)
            col = v[at].astype(np.int32)
            for k in (3, 4, 5) if w < 60 else (3, 4):
                want = oracle.kclique(rp, col, k)
                assert want.value == oracle.kclique(g.row_ptr, g.col, k).value
                print(f"{labels} {n} vertices, {w} next, k {k}", flush=True)
                job = rt.submit_kclique(rp, col, k, range_leaf=64)
                rt.run()
                st = rt.stats()
                assert rt.result(job) == want.value
                assert (st["tasks"], st["conts"]) == (want.tasks, want.conts)
