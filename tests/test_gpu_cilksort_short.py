"""Cilksort with cutoffs so small that several serial sorts or merges share a
register: ranges of up to 8, 16, 32 and 64 keys and one more, few and many of
them at a time.  Keys equal numpy's sort bit for bit; task counts equal the
oracle's."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sort_cutoff,merge_cutoff", [(1, 2), (2, 3), (7, 16), (8, 15), (8, 17), (9, 32), (16, 31),
                                                      (17, 33), (32, 64), (33, 63), (31, 65), (64, 64)])
@pytest.mark.parametrize("queues", [1, 3])
def test_short_ranges(sort_cutoff, merge_cutoff, queues):
    import torch
    from paper_2604_05982_amd import gtap
    opts = dict(num_queues=3, daq_policy=3) if queues > 1 else {}
    rng = np.random.default_rng(100 * sort_cutoff + merge_cutoff)
    arrays = [rng.integers(0, 2**32, size=n, dtype=np.uint32) for n in (1, 2, 3, 8, 9, 17, 64, 65, 500, 9001)]
    arrays += [rng.integers(0, 3, size=777, dtype=np.uint32), np.full(300, 0xFFFFFFFF, dtype=np.uint32),
               np.concatenate([np.arange(150, 300), np.arange(150)]).astype(np.uint32)]
    with gtap.Runtime(timeout_ms=60000, small_frames=1 << 20, big_frames=1 << 10, **opts) as rt:
        keys = [torch.from_numpy(a.view(np.int32).copy()).cuda() for a in arrays]
        for a, t in zip(arrays, keys):
            t2 = t.clone()
            job = rt.submit_cilksort(t2, sort_cutoff=sort_cutoff, merge_cutoff=merge_cutoff)
            rt.run()
            want, w = oracle.cilksort(a, sort_cutoff, merge_cutoff)
            assert np.array_equal(t2.cpu().numpy().view(np.uint32), want), a.size
            st = rt.stats()
            assert (st["tasks"], st["conts"]) == (w.tasks, w.conts) and rt.result(job) == a.size
        for t in keys:  # together: ranges of different jobs and lengths on one wavefront
            rt.submit_cilksort(t, sort_cutoff=sort_cutoff, merge_cutoff=merge_cutoff)
        rt.run()
        for a, t in zip(arrays, keys):
            assert np.array_equal(t.cpu().numpy().view(np.uint32), np.sort(a)), a.size


def test_short_ranges_in_mixed_launches():
    import torch
    from paper_2604_05982_amd import gtap
    rng = np.random.default_rng(5)
    with gtap.Runtime(timeout_ms=60000, waves_per_group=4, small_frames=1 << 20, big_frames=1 << 10) as rt:
        for with_fmm in (False, True):
            arrays = [rng.integers(0, 2**32, size=n, dtype=np.uint32) for n in (70, 3001, 20011)]
            keys = [torch.from_numpy(a.view(np.int32).copy()).cuda() for a in arrays]
            for t, cut in zip(keys, ((8, 16), (64, 256), (32, 64))):
                rt.submit_cilksort(t, sort_cutoff=cut[0], merge_cutoff=cut[1])
            fib = rt.submit_fib(16)
            if with_fmm:
                x, y, z, q = (torch.rand(500, dtype=torch.float64, device="cuda") for _ in range(4))
                phi = torch.empty_like(x)
                rt.submit_fmm(x, y, z, q, phi, traversal=gtap.GTAP_FMM_LISTS)
            rt.run()
            assert rt.result(fib) == 987
            for a, t in zip(arrays, keys):
                assert np.array_equal(t.cpu().numpy().view(np.uint32), np.sort(a)), a.size


def test_small_cutoffs_are_not_much_slower():
    """Four times as many leaves of a fourth the size: 1.6 times the time with
    registers shared, over 3 times with a register or tile to each range."""
    import torch
    from paper_2604_05982_amd import gtap
    keys = torch.from_numpy(np.random.default_rng(9).integers(-2**31, 2**31, size=1000000).astype(np.int32)).cuda()
    with gtap.Runtime(timeout_ms=60000, waves_per_group=4, small_frames=1 << 22, big_frames=1 << 10) as rt:
        def ms(sort_cutoff, merge_cutoff):
            times = []
            for _ in range(5):
                rt.submit_cilksort(keys.clone(), sort_cutoff=sort_cutoff, merge_cutoff=merge_cutoff)
                rt.run()
                times.append(rt.stats()["kernel_ms"])
            return min(times)

        assert ms(8, 16) < 2.4 * ms(64, 256)
