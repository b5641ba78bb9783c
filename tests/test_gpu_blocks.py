"""GPU: the FP64 matrix-core kernels at the edges of their 16 x 16 blocks,
block pairs, 64-function tiles and point chunks, in one batch of P points and
n functions on two atoms, against the oracle.

Bars: the FP64 bar 1e-12 of each value's own scale.  The spin-orbit parts of
H are formed as M - (D - D) from the products M_x = (a_y - a_z)(b_y + b_z) and
D_m = a_m b_m of the two gradients, so their scale adds the D terms that enter:
twice that of Ws, which sums their magnitudes."""
import numpy as np
import pytest

import oracle
import workload as W
from helpers import blocks_to_store, gpu_available, per_point_worst, store_to_blocks

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2608_00773_amd as q4c
    return q4c


def two_atoms(n, P, seed):
    """n functions (p shells, then s shells) on two atoms, P random points."""
    r = np.random.default_rng(seed)

    def shells(k):
        return [(l, np.sort(r.uniform(0.1, 4.0, 3)), r.uniform(0.2, 1.0, 3)) for l in [1] * (k // 6) + [0] * (k - 3 * (k // 6))]

    na = n // 2 if n < 40 else n // 3  # unequal blocks, an atom boundary off the 16s
    sizes = [na, n - na] if na else [n]
    Z = [82, 53][:len(sizes)]
    R = np.array([[0.1, -0.2, 0.3], [3.9, 1.1, -0.7]])[:len(sizes)]
    wl = W.pin_workload(Z, R, [shells(k) for k in sizes], nrad=8, ntheta=4, nphi=8, nint=64)
    wl = wl.subset_points(r.permutation(wl.n_points)[:P])
    wl.x, wl.y, wl.z = (r.uniform(-2.0, 4.0, P) for _ in range(3))
    wl.w = r.uniform(0.1, 1.0, P)
    return wl.with_v(r.uniform(-2.0, 1.0, P))


@pytest.mark.parametrize("n", [1, 15, 16, 17, 32, 33, 48, 49, 64, 65, 96, 113, 130])
@pytest.mark.parametrize("P", [1, 8, 16, 17, 47])
def test_one_batch_against_oracle(q, n, P):
    import torch
    wl = two_atoms(n, P, 100 * n + P)
    wk = W.with_ket(wl, 41)
    plan = q.Plan(wl, p_max=1000)
    assert plan.info["n_batches"] == 1 and plan.info["n_fn"] == n
    pairs, po = plan.pairs()
    nfn = wl.atom_nfn()
    print("n %d P %d" % (n, P), flush=True)
    v = torch.from_numpy(wl.v).cuda()
    store = q.new_store(plan).fill_(float("nan"))
    q.q4c_integrate_H(plan, v, q.PREC_F64, 0, store)
    ref, scale = oracle.pair_blocks(wl, pairs, with_abs=True)
    for g, r, s in zip(store_to_blocks(store.cpu().numpy(), pairs, po, nfn), ref, scale):
        s = s.copy()
        s[2:] += 2.0 * s[1]
        assert per_point_worst(g, r, s) <= 1e-12
    # the adjoint of the same parts
    rng = np.random.default_rng(n + P)
    coef = [rng.standard_normal((5, nfn[a], nfn[b])) for a, b in pairs]
    cst = torch.from_numpy(blocks_to_store(coef, po)).cuda()
    out = torch.full((P,), float("nan"), dtype=torch.float64, device="cuda")
    q.density_on_grid(plan, cst, q.TERM_ALL, 0, out)
    rd, sd = oracle.density(wl, pairs, coef, idx=np.arange(P), weight_mode=0, with_scale=True)
    assert per_point_worst(out.cpu().numpy(), rd, oracle.density_scale(sd)) <= 1e-12
    # H and S with the ket potential, and the density gradient
    plan.set_ket_potential(wk)
    hs = q.new_hs(plan).fill_(float("nan"))
    q.q4c_integrate_HS(plan, v, 0, hs)
    rh, sh = oracle.pair_blocks_hs(wk, pairs, with_abs=True)
    for k, (a, b) in enumerate(pairs):
        g = hs.cpu().numpy()[:, po[k]:po[k + 1]].reshape(2, nfn[a], nfn[b])
        assert per_point_worst(g, rh[k], sh[k], 1e-300) <= 1e-12
    grad = torch.full((4, P), float("nan"), dtype=torch.float64, device="cuda")
    q.density_gradient_on_grid(plan, cst[0].contiguous(), grad)
    rg, sg = oracle.density_grad(wl, pairs, [c[0] for c in coef], idx=np.arange(P), with_scale=True)
    assert per_point_worst(grad.cpu().numpy(), rg.T, sg.T, 1e-300) <= 1e-12
