"""GPU: calls of more workgroups than one launch takes: panels and tables of a
batch of 4.2 million points (over 65,535 chunks of 64), and a Bloch sum of 16.9
million workgroups (423,660 cell pairs, five parts, 64 k-points).

Bars: the FP64 bar 1e-12 of each value's own scale; the Bloch sum of single
contributions with unit phases repeats the stored values exactly."""
import dataclasses

import numpy as np
import pytest

import oracle
import workload as W
from helpers import gpu_available, per_point_worst, store_to_blocks

pytestmark = pytest.mark.gpu


def s_atoms(R, P, seed):
    """One s function per atom, P random points."""
    r = np.random.default_rng(seed)
    n = len(R)
    one = W.pin_workload([82], np.zeros((1, 3)), [[(0, np.array([0.2, 0.3, 0.5]), np.ones(3))]], nrad=4, ntheta=2, nphi=4,
                         nint=64)
    rep = np.zeros(n, dtype=np.int64)
    return dataclasses.replace(
        one, name="%d s atoms" % n, Z=np.full(n, 82, dtype=np.int32), R=np.asarray(R, dtype=np.float64),
        atom_shell_off=np.arange(n + 1, dtype=np.int32), shell_l=one.shell_l[rep].copy(),
        shell_rcut=one.shell_rcut[rep].copy(), shell_nint=one.shell_nint[rep].copy(),
        shell_coef_off=one.shell_coef_off[rep].copy(), shell_alpha=one.shell_alpha[rep].copy(),
        shell_gcoef=one.shell_gcoef[rep].copy(), x=r.uniform(-2.0, 2.0, P), y=r.uniform(-2.0, 2.0, P),
        z=r.uniform(-2.0, 2.0, P), w=r.uniform(0.1, 1.0, P), pt_atom=np.zeros(P, dtype=np.int32),
        v=r.uniform(-2.0, 1.0, P), molecule=None, shell_u_off=None, u_coef=None, shell_eps=None)


def test_batch_of_four_million_points():
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2608_00773_amd as q
    import torch
    P = 65535 * 64 + 1000
    wl = s_atoms([[0.1, -0.2, 0.3], [1.0, 0.4, -0.6]], P, 3)
    plan = q.Plan(wl, p_max=5000000)
    assert plan.info["n_batches"] == 1 and plan.info["max_batch_points"] == P
    pairs, po = plan.pairs()
    v = torch.from_numpy(wl.v).cuda()
    print("H", flush=True)
    store = q.new_store(plan).fill_(float("nan"))
    q.q4c_integrate_H(plan, v, q.PREC_F64, 0, store)
    ref, scale = oracle.pair_blocks(wl, pairs, with_abs=True)
    for g, r, s in zip(store_to_blocks(store.cpu().numpy(), pairs, po, wl.atom_nfn()), ref, scale):
        s = s.copy()
        s[2:] += 2.0 * s[1]  # the D terms of the six products
        assert per_point_worst(g, r, s) <= 1e-12
    print("tables", flush=True)
    _, pidx, _, fidx = plan.batches()
    out = torch.full((4 * P * 2,), float("nan"), dtype=torch.float64, device="cuda")
    q.nao_tabulate(plan, 0, 1, 1, out)
    idx = np.concatenate([np.arange(100), np.arange(P // 2, P // 2 + 100), np.arange(P - 1100, P)])
    g = out.reshape(4, P, 2)[:, torch.from_numpy(idx).cuda()].cpu().numpy()
    p = pidx[idx]
    phi, grad, aphi, agrad = oracle.tabulate(wl, wl.x[p], wl.y[p], wl.z[p], with_abs=True)
    ref = np.concatenate([phi[None], np.moveaxis(grad, 2, 0)])[:, :, fidx]
    sc = np.concatenate([aphi[None], np.moveaxis(agrad, 2, 0)])[:, :, fidx]
    assert per_point_worst(g, ref, sc, 1e-300) <= 1e-12


def test_bloch_sum_of_many_workgroups():
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2608_00773_amd as q
    import torch
    n, nk = 920, 64
    r = np.random.default_rng(4)
    plan = q.Plan(s_atoms(r.uniform(-1.0, 1.0, (n, 3)), 16, 5), p_max=1000)
    plan.set_cells(n, np.arange(n), np.zeros((n, 3)))
    _, off = plan.cell_pairs()
    ncp = n * (n + 1) // 2
    assert len(off) == ncp + 1 and off[-1] == ncp == plan.info["store_len"]
    store = torch.from_numpy(r.standard_normal((5, ncp))).cuda()
    out = torch.full((nk, 5, ncp, 2), float("nan"), dtype=torch.float64, device="cuda")
    print("Bloch sum", flush=True)
    q.q4c_bloch_sum(plan, 5, store, r.uniform(-1.0, 1.0, (nk, 3)), out)
    pairs, po = plan.pairs()
    cp, _ = plan.cell_pairs()
    assert np.array_equal(pairs, cp) and np.array_equal(po, off)
    for k in range(nk):
        assert torch.equal(out[k, :, :, 0], store) and not bool(out[k, :, :, 1].any()), k
