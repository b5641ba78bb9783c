"""GPU: the contractions of one batch read no weight of the next one.  Two
systems in one plan, one batch each; the first has P points, not a whole
16-point chunk, and the potential of the second is NaN everywhere: the first
system's blocks equal, bit for bit, those of a plan of its own, and are finite."""
import numpy as np
import pytest

import workload as W
from helpers import gpu_available

pytestmark = pytest.mark.gpu


def system(P, seed):
    """Two atoms of 26 functions in all, P random points."""
    r = np.random.default_rng(seed)
    mk = lambda l: (l, np.sort(r.uniform(0.1, 4.0, 3)), r.uniform(0.2, 1.0, 3))
    R = np.array([[0.1, -0.2, 0.3], [2.9, 1.1, -0.7]])
    wl = W.pin_workload([82, 53], R, [[mk(l) for l in ls] for ls in ([2, 1, 0, 0], [3, 1, 1, 0, 0, 0])], nrad=8, ntheta=4,
                        nphi=8, nint=64)
    wl = wl.subset_points(r.permutation(wl.n_points)[:P])
    wl.x, wl.y, wl.z = (r.uniform(-2.0, 4.0, P) for _ in range(3))
    wl.w = r.uniform(0.1, 1.0, P)
    return wl.with_v(r.uniform(-2.0, 1.0, P))


@pytest.mark.parametrize("P", [1, 2, 3, 4, 5, 6, 7, 8, 9, 15, 16, 17, 23, 35])
def test_nan_potential_stays_in_its_system(P):
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2608_00773_amd as q
    import torch
    a, b = system(P, P), system(40, 100 + P)
    both, alone = q.Plan([a, b], p_max=1000), q.Plan(a, p_max=1000)
    assert both.info["n_batches"] == 2 and alone.info["n_batches"] == 1
    s1 = int(both.systems()["store"][1])
    va = torch.from_numpy(a.v).cuda()
    v = torch.cat([va, torch.full((40,), float("nan"), dtype=torch.float64, device="cuda")])
    print("P %d" % P, flush=True)
    for prec in (q.PREC_F64, q.PREC_F64_VALU, q.PREC_F32, q.PREC_SPLIT_F32, q.PREC_BF16X3):
        for parts in (q.PART_ALL, q.PART_V):
            st, ref = q.new_store(both).zero_(), q.new_store(alone).zero_()
            q.q4c_integrate_H(both, v, prec, 0, st, parts=parts)
            q.q4c_integrate_H(alone, va, prec, 0, ref, parts=parts)
            assert bool(torch.isfinite(ref).all())
            assert torch.equal(st[:, :s1], ref), (prec, parts)
    ka, kb = W.with_ket(a, 41), W.with_ket(b, 42)
    both.set_ket_potential([ka, kb])
    alone.set_ket_potential(ka)
    hs, ref = q.new_hs(both), q.new_hs(alone)
    q.q4c_integrate_HS(both, v, 0, hs)
    q.q4c_integrate_HS(alone, va, 0, ref)
    assert bool(torch.isfinite(ref).all())
    assert torch.equal(hs[:, :s1], ref)
