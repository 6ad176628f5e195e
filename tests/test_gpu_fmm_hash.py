"""The lists' hash and pair counts over list lengths from one entry (one
wavefront, one 1,024-thread workgroup) to past the whole grid (262,144
entries), equal to the block-mode traversal's, which sums the same pairs one
by one."""
import numpy as np
import pytest

from synth import points

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2, 65, 200, 1500, 3000, 20000, 50000])
def test_list_hash_equals_block_mode(n):
    import torch
    from paper_2604_05982_amd import gtap
    pts = [torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).cuda() for a in points.plummer(n, 11)]
    got = []
    for tr, kw in ((gtap.GTAP_FMM_TASKS, dict(mode=gtap.GTAP_MODE_BLOCK, waves_per_group=2, big_frames=0)),
                   (gtap.GTAP_FMM_LISTS, dict(waves_per_group=4, big_frames=1 << 10))):
        with gtap.Runtime(small_frames=1 << 20, timeout_ms=60000, **kw) as rt:
            job = rt.submit_fmm(*pts, torch.zeros_like(pts[0]), leaf_max=16, traversal=tr)
            rt.run()
            res = rt.fmm_result(job)
            got.append([res[k] for k in ("m2l_pairs", "p2p_pairs", "m2l_hash", "p2p_hash")])
    assert got[0] == got[1]
