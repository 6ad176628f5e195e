"""Claims of fresh frames where they change from an add to a compare-and-swap
(512 untouched frames per wavefront left) and where adds pass the end of the
pool: every wavefront claims its share of the roots at once, from the same
value.  A pool of exactly the frames that the claims take in all refuses none
and is touched to its last frame; a larger one is touched no further; in a
smaller one, whose later claims go without spares, a run either gives every
result or ends in the capacity error."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("waves,roots", [(4, 40), (64, 200), (64, 500), (64, 700), (256, 513)])
def test_claims_cross_from_add_to_swap(waves, roots):
    from paper_2604_05982_amd import gtap
    jobs = waves * roots

    def run(small_frames):
        print(f"{waves} wavefronts, {roots} roots each, {small_frames} frames", flush=True)
        with gtap.Runtime(timeout_ms=60000, num_waves=waves, waves_per_group=4, small_frames=small_frames,
                          big_frames=1 << 10, deque_capacity=1 << 12, max_jobs=jobs) as rt:
            ids = [rt.submit_fib(i % 2) for i in range(jobs)]
            rt.run()
            assert [rt.result(i) for i in ids] == [i % 2 for i in range(jobs)]
            st = rt.stats()
            assert st["tasks"] == jobs
            return st["small_frames_touched"]

    need = run(4 * waves * (512 + roots + 512))  # adds only
    assert need >= jobs and need % waves == 0
    for frames in (need, need + 1, need + 256 * waves, need + 512 * waves):
        if frames >= 1024:
            assert run(frames) == need
    for frames in (need - 1, jobs + (need - jobs) // 2, jobs, jobs - 1):
        if frames < 1024:
            continue
        try:
            assert jobs <= run(frames) <= frames
        except gtap.GtapError as e:
            assert e.code == gtap.GTAP_E_CAPACITY and e.report["pool"] == 0
