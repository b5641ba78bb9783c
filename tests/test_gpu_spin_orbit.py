"""GPU: the rounding of the FP64 spin-orbit parts of H, which are formed as
M - (D - D) from sums whose products can outweigh Wso's own.

Bar: the RMS error of Wso's elements against the oracle, relative to the
magnitudes of each element's own products, is no larger than that of the nine
products of Wso summed directly on matrix cores, measured once: 6.9e-16 on
points near the axis of two atoms, where grad phi_i and grad phi_j are nearly
parallel and D outweighs Wso most (1.6e-15 without the joins of the sums)."""
import numpy as np
import pytest

import oracle
import workload as W
from helpers import gpu_available, store_to_blocks

pytestmark = pytest.mark.gpu


def rod(seed=5, P=4000):
    """Two atoms on the x axis, points within 0.1 bohr (standard deviation) of it."""
    r = np.random.default_rng(seed)
    mk = lambda l: (l, np.sort(r.uniform(0.1, 4.0, 3)), r.uniform(0.2, 1.0, 3))
    R = np.array([[0.0, 0.0, 0.0], [6.0, 0.1, -0.1]])
    wl = W.pin_workload([82, 53], R, [[mk(l) for l in (0, 0, 1, 1, 2, 3)] for _ in range(2)], nrad=60, ntheta=8, nphi=16,
                        nint=512)
    wl = wl.subset_points(r.permutation(wl.n_points)[:P])
    wl.x, wl.y, wl.z = r.uniform(-2.0, 8.0, P), r.normal(0, 0.1, P), r.normal(0, 0.1, P)
    wl.w = r.uniform(0.1, 1.0, P)
    return wl.with_v(r.uniform(-2.0, 1.0, P))


def test_wso_error_no_larger_than_direct_products():
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2608_00773_amd as q
    import torch
    wl = rod()
    plan = q.Plan(wl)
    pairs, po = plan.pairs()
    nfn = wl.atom_nfn()
    v = torch.from_numpy(np.ascontiguousarray(wl.v)).cuda()
    ref, scale = oracle.pair_blocks(wl, pairs, with_abs=True)
    store = q.new_store(plan)
    q.q4c_integrate_H(plan, v, q.PREC_F64, 0, store)
    got = store_to_blocks(store.cpu().numpy(), pairs, po, nfn)
    e = np.concatenate([((g - r)[2:][s[2:] > 0] / s[2:][s[2:] > 0]) for g, r, s in zip(got, ref, scale)])
    rms = float(np.sqrt(np.mean(e * e)))
    print("Wso RMS error %.2e" % rms, flush=True)
    assert rms <= 6.9e-16
