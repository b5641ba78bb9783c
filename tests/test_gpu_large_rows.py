"""GPU: a batch whose staged block rows exceed 2 GiB, the range of the 32-bit
offsets that the contractions store with: nine atoms of 1,818 functions (the
largest atom pair block a plan takes) in one batch.  The 16 rows that span the
first two atoms take 2.25e9 bytes, the last of them in the pair (1, 8).

Bars: those of each precision, per element of the pairs' own scales."""
import dataclasses

import numpy as np
import pytest

import oracle
import workload as W
from helpers import gpu_available, per_point_worst, split_bound_worst

pytestmark = pytest.mark.gpu

PAIRS = [(0, 1), (1, 1), (1, 8)]


def nine_large_atoms(n_shells=202, P=16):
    """Nine atoms of n_shells shells with l = 4, each with a table of its own, P points."""
    r = np.random.default_rng(9)
    wl = W.config_small(nrad=10, nang=26, nint=64)
    ns, s0, na = 9 * n_shells, int(wl.atom_shell_off[0]), 9
    base = np.asarray(wl.coef[wl.shell_coef_off[s0]:][:4 * 64])
    tab = (base[None, :] * r.uniform(0.2, 1.0, (ns, 1))).reshape(-1)
    pts = np.arange(P)
    return dataclasses.replace(
        wl, name="nine large atoms", Z=np.full(na, 82, dtype=np.int32), R=r.uniform(-1.0, 1.0, (na, 3)),
        atom_shell_off=np.arange(0, ns + 1, n_shells, dtype=np.int32), shell_l=np.full(ns, 4, dtype=np.int32),
        shell_rcut=np.full(ns, wl.shell_rcut[s0]), shell_nint=np.full(ns, 64, dtype=np.int32),
        shell_coef_off=np.arange(0, 4 * 64 * ns, 4 * 64, dtype=np.int64), coef=tab,
        shell_alpha=wl.shell_alpha[np.full(ns, s0)].copy(), shell_gcoef=wl.shell_gcoef[np.full(ns, s0)].copy(),
        x=r.uniform(-2.0, 2.0, P), y=r.uniform(-2.0, 2.0, P), z=r.uniform(-2.0, 2.0, P), w=r.uniform(0.1, 1.0, P),
        pt_atom=np.zeros(P, dtype=np.int32), v=r.uniform(-2.0, 1.0, P), molecule=None,
        shell_u_off=np.arange(0, 4 * 64 * ns, 4 * 64, dtype=np.int64), u_coef=tab * r.uniform(-1.0, 1.0, tab.size),
        shell_eps=None)


def test_rows_beyond_two_gib():
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2608_00773_amd as q
    import torch
    wl = nine_large_atoms()
    plan = q.Plan(wl, p_max=1000)
    nf = 1818
    assert plan.info["n_batches"] == 1 and plan.info["max_batch_fn"] == 9 * nf
    pairs, po = plan.pairs()
    idx = [int(np.nonzero((pairs == p).all(axis=1))[0][0]) for p in PAIRS]
    v = torch.from_numpy(wl.v).cuda()
    ref, scale = oracle.pair_blocks(wl, np.array(PAIRS), with_abs=True)
    store = q.new_store(plan)

    def blocks(st):
        return [st[:, po[i]:po[i + 1]].cpu().numpy().reshape(-1, nf, nf) for i in idx]

    for prec in (q.PREC_F64, q.PREC_F32, q.PREC_SPLIT_F32, q.PREC_BF16X3):
        print("precision", prec, flush=True)
        store.fill_(float("nan"))
        q.q4c_integrate_H(plan, v, prec, 0, store)
        got = blocks(store)
        k = 5 if prec == q.PREC_F64 else 1
        for g, r, s in zip(got, ref, scale):
            s = s.copy()
            s[2:] += 2.0 * s[1]  # the D terms of the six products
            assert per_point_worst(g[:k], r[:k], s[:k], 1e-300) <= 1e-12
        if prec != q.PREC_F64:
            assert split_bound_worst(got, ref, scale, prec) <= 1.0
    print("V alone", flush=True)
    store.fill_(float("nan"))
    q.q4c_integrate_H(plan, v, q.PREC_F64, 0, store, parts=q.PART_V)
    for g, r, s in zip(blocks(store), ref, scale):
        assert per_point_worst(g[:1], r[:1], s[:1], 1e-300) <= 1e-12
    del store
    print("H and S", flush=True)
    plan.set_ket_potential(wl)
    hs = q.new_hs(plan).fill_(float("nan"))
    q.q4c_integrate_HS(plan, v, 0, hs)
    rh, sh = oracle.pair_blocks_hs(wl, np.array(PAIRS), with_abs=True)
    for g, r, s in zip(blocks(hs), rh, sh):
        assert per_point_worst(g, r, s, 1e-300) <= 1e-12
