"""Device memory that a context keeps between runs: given back by release(),
allocated again by the next run, kept while jobs wait on it."""
import numpy as np
import pytest

import oracle
from synth import graphs, points

pytestmark = pytest.mark.gpu


def free_bytes():
    import torch
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_release_gives_memory_back():
    import torch
    from paper_2604_05982_amd import gtap
    ts = [torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).cuda() for a in points.plummer(300000, 3)]
    phi = torch.empty_like(ts[0])
    with gtap.Runtime(small_frames=1 << 20, big_frames=1 << 10, waves_per_group=4, timeout_ms=60000) as rt:
        rt.submit_fib(10)
        rt.run()
        before = free_bytes()
        got = []
        for _ in range(2):
            job = rt.submit_fmm(*ts, phi, traversal=gtap.GTAP_FMM_LISTS)
            rt.run()
            got.append((phi.clone(), rt.fmm_result(job)["m2l_pairs"]))
            kept = before - free_bytes()
            assert kept > 100 << 20  # trees and lists of 300,000 points
            rt.release()
            assert before - free_bytes() < 32 << 20
        assert got[0][1] == got[1][1] and torch.allclose(got[0][0], got[1][0], rtol=1e-9)
        rt.release()  # nothing left: no error


def test_release_between_submit_and_run():
    import torch
    from paper_2604_05982_amd import gtap
    g = graphs.chung_lu(3000, 24, 2.3, 1.0, 9)
    rp, col = torch.as_tensor(g.row_ptr32).cuda(), torch.as_tensor(g.col).cuda()
    with gtap.Runtime(waves_per_group=4, small_frames=1 << 20, big_frames=1 << 14, timeout_ms=60000,
                      big_frame_ints=gtap.kclique_split_buffer_ints(1024)) as rt:
        for k in (4, 5):
            job = rt.submit_kclique_split(rp, col, k, max_outdeg=g.max_outdeg)
            rt.release()
            rt.run()
            assert rt.result(job) == oracle.kclique(g.row_ptr, g.col, k).value


def test_release_is_refused_while_serving():
    from paper_2604_05982_amd import gtap
    with gtap.Runtime(waves_per_group=4, small_frames=1 << 20, big_frames=1 << 10, timeout_ms=60000) as rt:
        gtap.gtap_serve_start(rt.ctx, 8, 0, 0)
        try:
            with pytest.raises(gtap.GtapError) as e:
                rt.release()
            assert e.value.code == gtap.GTAP_E_STATE
        finally:
            gtap.gtap_serve_stop(rt.ctx)
        rt.release()
