"""List evaluation of trees around the runs of targets that share an XCD (16
cells, 128 in a round of eight): every cell's locals and every leaf's near field
are there.  Potentials and pair lists against the oracle FMM (1e-12, the bound of
re-ordered double sums)."""
import numpy as np
import pytest

import oracle
from synth import points

pytestmark = pytest.mark.gpu

RTOL = 1e-12


def test_trees_around_the_runs():
    import torch
    from paper_2604_05982_amd import gtap
    seen = set()
    with gtap.Runtime(small_frames=1 << 20, big_frames=1 << 10, timeout_ms=60000, waves_per_group=4) as rt:
        for n in list(range(10, 130, 3)) + list(range(180, 215, 2)):
            pts = list(points.plummer(n, n))
            want = oracle.fmm(*pts, theta=(2, 3), leaf_max=2)
            ts = [torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).cuda() for a in pts]
            phi = torch.full_like(ts[0], float("nan"))
            job = rt.submit_fmm(*ts, phi, leaf_max=2, theta=(2, 3), traversal=gtap.GTAP_FMM_LISTS)
            rt.run()
            res = rt.fmm_result(job)
            for k in ("n_cells", "m2l_pairs", "p2p_pairs", "m2l_hash", "p2p_hash", "p2p_interactions"):
                assert res[k] == want.stats[k], (n, k)
            err = np.abs(phi.cpu().numpy() - want.phi).max()
            assert err <= RTOL * np.abs(want.phi).max(), (n, err)
            seen.add(res["n_cells"] // 16)
    assert {0, 1, 7, 8, 15, 16} <= seen  # below, at and beyond one and two rounds of runs
