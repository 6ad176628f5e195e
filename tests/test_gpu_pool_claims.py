"""Claims of fresh frames, by an add while the pool has 512 untouched frames
per wavefront left and by compare-and-swap near its end: pools that a job
touches to the last frame give the oracle's values and never report more
frames than they hold; too small ones end in the capacity error."""
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waves,small_frames", [(1, 1024), (1, 2048), (2, 4096), (64, 1 << 15), (64, 1 << 16),
                                                (1024, 1 << 20)])
def test_claims_to_the_end_of_the_pool(waves, small_frames):
    from paper_2604_05982_amd import gtap
    with gtap.Runtime(timeout_ms=60000, num_waves=waves, waves_per_group=min(waves, 4), small_frames=small_frames,
                      big_frames=1 << 10, deque_capacity=1 << 12) as rt:
        for n in (6, 12, 18, 22):
            want = oracle.fib(n)
            job = rt.submit_fib(n)
            try:
                rt.run()
            except gtap.GtapError as e:
                assert e.code == gtap.GTAP_E_CAPACITY and e.report["pool"] in (0, 2)
                assert n > 12  # 465 tasks fit any of these pools
                break
            st = rt.stats()
            assert rt.result(job) == want.value and st["tasks"] == want.tasks
            assert st["small_frames_touched"] <= small_frames
