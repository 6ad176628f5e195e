"""Cilksort's wavefront-wide serial sorts and merges at the edges of their
tiles: sorts of 1..64 keys (one wavefront's width), merges of one tile (256
keys), one key more, and many tiles cut at merge-path splits.  Keys equal
numpy's sort bit for bit; task counts equal the oracle's."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sort_cutoff,merge_cutoff", [(64, 255), (64, 256), (63, 257), (33, 1000), (2, 511),
                                                      (64, 1 << 20)])
def test_cilksort_tiles(sort_cutoff, merge_cutoff):
    import torch
    from paper_2604_05982_amd import gtap
    rng = np.random.default_rng(merge_cutoff)
    arrays = [rng.integers(0, 2**32, size=n, dtype=np.uint32) for n in (2, 65, 128, 255, 256, 257, 511, 513, 4099, 70001)]
    arrays += [rng.integers(0, 3, size=5003, dtype=np.uint32),                       # long runs of ties
               np.full(3001, 0xFFFFFFFF, dtype=np.uint32),                           # equal to the pads
               np.concatenate([np.arange(2500, 5000), np.arange(2500)]).astype(np.uint32),  # one side first
               np.concatenate([np.zeros(2000), rng.integers(0, 2**32, 2100)]).astype(np.uint32)]
    with gtap.Runtime(timeout_ms=60000, small_frames=1 << 20, big_frames=1 << 10) as rt:
        keys = [torch.from_numpy(a.view(np.int32).copy()).cuda() for a in arrays]
        for a, t in zip(arrays, keys):  # alone: exact task counts
            t2 = t.clone()
            job = rt.submit_cilksort(t2, sort_cutoff=sort_cutoff, merge_cutoff=merge_cutoff)
            rt.run()
            want, w = oracle.cilksort(a, sort_cutoff, merge_cutoff)
            assert np.array_equal(t2.cpu().numpy().view(np.uint32), want), a.size
            st = rt.stats()
            assert (st["tasks"], st["conts"]) == (w.tasks, w.conts) and rt.result(job) == a.size
        for t in keys:  # together: lanes of one wavefront hold tasks of different jobs
            rt.submit_cilksort(t, sort_cutoff=sort_cutoff, merge_cutoff=merge_cutoff)
        rt.run()
        for a, t in zip(arrays, keys):
            assert np.array_equal(t.cpu().numpy().view(np.uint32), np.sort(a)), a.size
