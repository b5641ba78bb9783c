"""GPU: the operand panels of every precision where shells cross the edges of
the tiles that one wave tabulates (64 functions, 16 on small plans) and points
the edges of its 64 lanes, through H and H/S against the oracle; tables of
values at the same edges.

Bars: the FP64 bar 1e-12 of each value's own scale (the spin-orbit parts with
the D terms of the six-product form, twice the scale of Ws); the stated bounds
of the reduced precisions' W parts."""
import numpy as np
import pytest

import oracle
import workload as W
from helpers import gpu_available, per_point_worst, split_bound_worst, store_to_blocks

pytestmark = pytest.mark.gpu


def workload(ls, P, seed):
    """Shells ls on one atom and ls reversed on another, P random points."""
    r = np.random.default_rng(seed)
    mk = lambda l: (l, np.sort(r.uniform(0.1, 4.0, 3)), r.uniform(0.2, 1.0, 3))
    R = np.array([[0.1, -0.2, 0.3], [2.9, 1.1, -0.7]])
    wl = W.pin_workload([82, 53], R, [[mk(l) for l in ls], [mk(l) for l in ls[::-1]]], nrad=16, ntheta=6, nphi=8, nint=64)
    wl = wl.subset_points(r.permutation(wl.n_points)[:P])
    wl.x, wl.y, wl.z = (r.uniform(-2.0, 4.0, P) for _ in range(3))
    wl.w = r.uniform(0.1, 1.0, P)
    return wl.with_v(r.uniform(-2.0, 1.0, P))


# (points, largest batch): one batch of 65 or 129 points in quarter tiles; 560
# batches of one point, whole tiles
@pytest.mark.parametrize("P, p_max", [(65, 1000), (129, 1000), (560, 1)])
@pytest.mark.parametrize("ls", [[3, 1, 4, 0], [4, 3, 2, 3, 1, 3, 4, 0, 2]], ids=["40", "106"])
def test_panels_against_oracle(P, p_max, ls):
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2608_00773_amd as q
    import torch
    wl = workload(ls, P, P + len(ls))
    plan = q.Plan(wl, p_max=p_max)
    pairs, po = plan.pairs()
    nfn = wl.atom_nfn()
    print("n %d P %d batches %d" % (plan.info["n_fn"], P, plan.info["n_batches"]), flush=True)
    v = torch.from_numpy(wl.v).cuda()
    ref, scale = oracle.pair_blocks(wl, pairs, with_abs=True)
    for prec in (q.PREC_F64, q.PREC_SPLIT_F32, q.PREC_F32, q.PREC_BF16X3):
        store = q.new_store(plan).fill_(float("nan"))
        q.q4c_integrate_H(plan, v, prec, 0, store)
        got = store_to_blocks(store.cpu().numpy(), pairs, po, nfn)
        for g, r, s in zip(got, ref, scale):
            s = s.copy()
            s[2:] += 2.0 * s[1]
            k = 5 if prec == q.PREC_F64 else 1
            assert per_point_worst(g[:k], r[:k], s[:k], 1e-300) <= 1e-12, prec
        if prec != q.PREC_F64:
            assert split_bound_worst(got, ref, scale, prec) <= 1.0, prec
    wk = W.with_ket(wl, 41)
    plan.set_ket_potential(wk)
    hs = q.new_hs(plan).fill_(float("nan"))
    q.q4c_integrate_HS(plan, v, 0, hs)
    rh, sh = oracle.pair_blocks_hs(wk, pairs, with_abs=True)
    for k, (a, b) in enumerate(pairs):
        g = hs.cpu().numpy()[:, po[k]:po[k + 1]].reshape(2, nfn[a], nfn[b])
        assert per_point_worst(g, rh[k], sh[k], 1e-300) <= 1e-12


@pytest.mark.parametrize("P", [1, 64, 65, 130])
@pytest.mark.parametrize("ls", [[0], [3, 1, 4, 0], [4, 3, 2, 3, 1, 3, 4, 0, 2]], ids=["2", "40", "106"])
def test_tabulate_at_tile_edges(P, ls):
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2608_00773_amd as q
    import torch
    wl = workload(ls, P, 7 * P + len(ls))
    plan = q.Plan(wl, p_max=1000)
    _, pidx, _, fidx = plan.batches()
    n = plan.info["n_fn"]
    assert plan.info["n_batches"] == 1 and len(fidx) == n
    print("n %d P %d" % (n, P), flush=True)
    phi, grad, aphi, agrad = oracle.tabulate(wl, wl.x[pidx], wl.y[pidx], wl.z[pidx], with_abs=True)
    ref = np.concatenate([phi[None], np.moveaxis(grad, 2, 0)])[:, :, fidx]
    sref = np.concatenate([aphi[None], np.moveaxis(agrad, 2, 0)])[:, :, fidx]
    for nq in (4, 1):
        out = torch.full((nq * P * n + 1,), -7.0, dtype=torch.float64, device="cuda")
        q.nao_tabulate(plan, 0, 1, int(nq == 4), out[:-1])
        assert float(out[-1]) == -7.0  # nothing past the table
        assert per_point_worst(out[:-1].cpu().numpy().reshape(nq, P, n), ref[:nq], sref[:nq], 1e-300) <= 1e-12
