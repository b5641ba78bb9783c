"""GPU: q4c_bloch_sum and q4c_bloch_density on random blocks of two cell atoms
with 5 and 30 functions (a block of 900 elements does not fit one workgroup's
turned sums) at k-point counts around the sizes of their register groups,
against the oracle.  Each element is a sum of n terms |f| |O| (n_k or the
contributions); bar 1e-14 of the sum of their magnitudes, as for the existing
Bloch tests, n below 100."""
import numpy as np
import pytest

import oracle
import workload as W
from helpers import gpu_available

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2608_00773_amd as q4c
    return q4c


@pytest.fixture(scope="module")
def cell():
    """Two atoms in a 7 bohr cell along x and their images two cells either side."""
    r = np.random.default_rng(9)
    R = np.array([[0.3, 0.1, -0.2], [3.1, 0.9, 0.4]])
    shells = [[(0, np.array([0.3, 0.9, 2.0]), r.uniform(0.2, 1.0, 3)) for _ in range(k)] for k in (5, 30)]
    T = [np.array([7.0 * t, 0.0, 0.0]) for t in (0, -2, -1, 1, 2)]
    atom = np.array([c for _ in T for c in (0, 1)], dtype=np.int32)
    shift = np.array([t for t in T for _ in (0, 1)])
    wl = W.pin_workload([82 if a else 6 for a in atom], R[atom] + shift, [shells[a] for a in atom], nrad=4, ntheta=2,
                        nphi=4, nint=32)
    return wl, atom, shift


@pytest.mark.parametrize("n_k", [1, 2, 3, 5, 8, 9, 10, 19, 65])
@pytest.mark.parametrize("n_parts", [1, 5])
def test_sum_and_density_against_oracle(q, cell, n_k, n_parts):
    import torch
    wl, atom, shift = cell
    plan = q.Plan(wl)
    plan.set_cells(2, atom, shift)
    pairs, po = plan.pairs()
    nfn = wl.atom_nfn()
    rng = np.random.default_rng(10 * n_k + n_parts)
    kp = rng.uniform(-0.4, 0.4, (n_k, 3))
    store = rng.standard_normal((n_parts, plan.info["store_len"]))
    blocks = [store[:, po[p]:po[p + 1]].reshape(n_parts, nfn[a], nfn[b]) for p, (a, b) in enumerate(pairs)]
    cpa, cpo = plan.cell_pairs()
    out = torch.full((n_k, n_parts, int(cpo[-1]), 2), float("nan"), dtype=torch.float64, device="cuda")
    print("n_k %d parts %d" % (n_k, n_parts), flush=True)
    q.q4c_bloch_sum(plan, n_parts, torch.from_numpy(store).cuda(), kp, out)
    got = torch.view_as_complex(out).cpu().numpy()
    ref = oracle.bloch_sum(atom, shift, pairs, blocks, kp)
    nc = [int(nfn[0]), int(nfn[1])]
    for c, (a, b) in enumerate(cpa):
        g = got[:, :, cpo[c]:cpo[c + 1]].reshape(n_k, n_parts, nc[a], nc[b])
        want = ref[(int(a), int(b))]
        m = np.zeros((n_parts, nc[a], nc[b]))
        for p, (A, B) in enumerate(pairs):
            if (atom[A], atom[B]) == (a, b):
                m += np.abs(blocks[p])
            if A != B and (atom[B], atom[A]) == (a, b):
                m += np.abs(blocks[p]).transpose(0, 2, 1)
        assert np.all(np.abs(g - want) <= 1e-14 * m[None])
    if n_parts > 2:
        return
    rho = {(int(a), int(b)): rng.standard_normal((n_k, n_parts, nc[a], nc[b])) +
           1j * rng.standard_normal((n_k, n_parts, nc[a], nc[b])) for a, b in cpa}
    flat = np.concatenate([rho[(int(a), int(b))].reshape(n_k, n_parts, -1) for a, b in cpa], axis=2)
    w = rng.uniform(0.1, 1.0, n_k)
    coef = torch.full((n_parts, plan.info["store_len"]), float("nan"), dtype=torch.float64, device="cuda")
    q.q4c_bloch_density(plan, n_parts, torch.view_as_real(torch.from_numpy(flat)).contiguous().cuda(), kp, w, coef)
    got = coef.cpu().numpy()
    ref = oracle.bloch_density(atom, shift, pairs, rho, kp, w, nfn)
    mag = oracle.bloch_density(atom, 0.0 * shift, pairs, {k: np.abs(x) for k, x in rho.items()}, kp, w, nfn)
    for p in range(len(pairs)):
        g = got[:, po[p]:po[p + 1]].reshape(ref[p].shape)
        assert np.all(np.abs(g - ref[p]) <= 1e-14 * mag[p])
