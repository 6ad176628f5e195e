"""FMM passes and list evaluation at the sizes where their kernels change:
leaves of 1, 63..65 and more points (a level-21 cell keeps any number of
coincident points), cells with one to eight children, trees of one cell and
of 21 levels; every traversal against the oracle FMM (1e-12, the bound of
re-ordered double sums) and the same pair lists."""
import numpy as np
import pytest

import oracle
from synth import points

pytestmark = pytest.mark.gpu

RTOL = 1e-12


def inputs(name):
    rng = np.random.default_rng(31)
    if name == "one":
        return [np.array([v]) for v in (3.5, -2.0, 0.125, 0.75)], 64
    if name in ("n63", "n64", "n65", "n129"):
        return list(points.plummer(int(name[1:]), 5)), 64
    if name == "leaf1":
        return list(points.plummer(700, 6)), 1
    if name == "deep":  # a pile of 150 coincident points among others: 21 levels, a 150-point leaf
        x, y, z, q = points.plummer(2500, 7)
        at = rng.uniform(-1, 1, 3)
        x, y, z = (np.concatenate([a, np.full(150, v)]) for a, v in zip((x, y, z), at))
        return [x, y, z, np.concatenate([q, rng.uniform(-1, 1, 150)])], 64
    if name == "line":  # cells with one or two children
        t = np.sort(rng.uniform(-100, 100, 3000))
        return [t, np.full(3000, 0.5), np.full(3000, 0.5), rng.uniform(-1, 1, 3000)], 16
    x, y, z, q = points.uniform_cube(20011, 9, half=100.0)  # cells with eight
    return [x, y, z, q], 33


@pytest.mark.parametrize("traversal", ["tasks", "lists", "worklist"])
@pytest.mark.parametrize("name", ["one", "n63", "n64", "n65", "n129", "leaf1", "deep", "line", "cube"])
def test_fmm_against_oracle(traversal, name):
    import torch
    from paper_2604_05982_amd import gtap
    pts, leaf = inputs(name)
    tr = {"tasks": gtap.GTAP_FMM_TASKS, "lists": gtap.GTAP_FMM_LISTS, "worklist": gtap.GTAP_FMM_WORKLIST}[traversal]
    kw = dict(mode=gtap.GTAP_MODE_BLOCK, waves_per_group=2) if traversal == "tasks" else dict(waves_per_group=4)
    with gtap.Runtime(small_frames=1 << 20, big_frames=0 if traversal == "tasks" else 1 << 10, timeout_ms=60000,
                      **kw) as rt:
        ts = [torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).cuda() for a in pts]
        for theta in ((1, 2), (2, 3)):
            phi = torch.full_like(ts[0], float("nan"))
            job = rt.submit_fmm(*ts, phi, leaf_max=leaf, theta=theta, traversal=tr)
            rt.run()
            res, got = rt.fmm_result(job), phi.cpu().numpy()
            want = oracle.fmm(*pts, theta=theta, leaf_max=leaf)
            for k in ("n_cells", "n_leaves", "max_level", "m2l_pairs", "p2p_pairs", "m2l_hash", "p2p_hash",
                      "p2p_interactions", "coincident"):
                assert res[k] == want.stats[k], k
            err = np.abs(got - want.phi).max()
            assert err <= RTOL * max(np.abs(want.phi).max(), 1e-300), (name, theta, err)
