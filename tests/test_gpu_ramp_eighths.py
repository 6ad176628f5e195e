"""Tasks are exposed in every eighth iteration from the start, also by
wavefronts that still take their early looks: a grid that is never three
quarters idle (two wavefronts per group: more than are resident at once)
exposes as many with early looks as a pool too small for them does without.
Values equal the oracle's."""
import statistics

import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waves", [0, 64])
def test_early_looks_do_not_replace_the_regular_ones(waves):
    from paper_2604_05982_amd import gtap
    want = oracle.nqueens(10)

    def pushed(early):
        opts = dict(waves_per_group=2, num_waves=waves, timeout_ms=60000, big_frames=1 << 10)
        with gtap.Runtime(small_frames=1 << 24, **opts) as rt:  # (for the grid's size)
            rt.submit_fib(1)
            rt.run()
            grid = rt.stats()["num_waves"]
        # early looks need 1024 frames per wavefront
        with gtap.Runtime(small_frames=1 << 24 if early else 1024 * grid - 1, **opts) as rt:
            counts = []
            for _ in range(7):
                job = rt.submit_nqueens(10)
                rt.run()
                st = rt.stats()
                assert rt.result(job) == want.value and st["tasks"] == want.tasks
                counts.append(st["pushed"])
            return statistics.median(counts)

    assert pushed(True) > 0.75 * pushed(False)
