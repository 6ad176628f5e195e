"""Tasks exposed early, while most of the grid is idle: private stacks around
the smallest batch that is exposed (32 tasks) and the largest (64), with a
frame pool that allows it and one that does not (fewer than 1024 frames per
wavefront).  Values and task counts equal the oracle's."""
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("small_frames", [1 << 19, 1 << 21])
@pytest.mark.parametrize("waves", [1, 2, 1024])
def test_early_exposure_counts(small_frames, waves):
    from paper_2604_05982_amd import gtap
    with gtap.Runtime(timeout_ms=60000, num_waves=waves, waves_per_group=min(waves, 4), small_frames=small_frames,
                      big_frames=1 << 10) as rt:
        for n in (1, 5, 6, 7, 8, 9, 10, 11, 12, 16, 20):  # 1 .. 21,891 tasks
            want = oracle.fib(n)
            job = rt.submit_fib(n)
            rt.run()
            st = rt.stats()
            assert rt.result(job) == want.value and (st["tasks"], st["conts"]) == (want.tasks, want.conts), n
        jobs = [(rt.submit_fib(n), oracle.fib(n).value) for n in range(2, 18)]
        rt.run()
        for job, value in jobs:
            assert rt.result(job) == value
