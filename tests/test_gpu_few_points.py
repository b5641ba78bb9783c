"""GPU: batches of few points, for which tables take a kernel of their own: at
the edges of 8 points and of 64 functions, against the oracle.

Bar: the FP64 bar 1e-12 of each value's own scale."""
import numpy as np
import pytest

import oracle
from helpers import gpu_available, per_point_worst
from test_gpu_blocks import two_atoms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 17, 64, 65, 130])
@pytest.mark.parametrize("P, p_max", [(1, 8), (8, 8), (9, 16), (31, 8), (48, 48), (127, 40)])
def test_tables(n, P, p_max):
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2608_00773_amd as q
    import torch
    wl = two_atoms(n, P, 500 * n + P)
    plan = q.Plan(wl, p_max=p_max)
    po, pidx, fo, fidx = plan.batches()
    nb = plan.info["n_batches"]
    print("n %d P %d batches %d" % (n, P, nb), flush=True)
    out = torch.full((plan.tabulate_size(0, nb, 1) + 1,), -7.0, dtype=torch.float64, device="cuda")
    q.nao_tabulate(plan, 0, nb, 1, out[:-1])
    val = torch.full((plan.tabulate_size(0, nb, 0),), -7.0, dtype=torch.float64, device="cuda")
    q.nao_tabulate(plan, 0, nb, 0, val)
    hl = torch.full((2 * plan.tabulate_size(0, nb, 1),), -7.0, dtype=torch.float32, device="cuda")
    q.nao_tabulate(plan, 0, nb, 1, hl, q.DTYPE_F32_HILO)
    out, val, hl = out.cpu().numpy(), val.cpu().numpy(), hl.cpu().numpy()
    assert out[-1] == -7.0  # nothing past the tables
    phi, grad, aphi, agrad = oracle.tabulate(wl, wl.x[pidx], wl.y[pidx], wl.z[pidx], with_abs=True)
    ref = np.concatenate([phi[None], np.moveaxis(grad, 2, 0)])
    sref = np.concatenate([aphi[None], np.moveaxis(agrad, 2, 0)])
    o = 0
    for b in range(nb):
        p, f = slice(po[b], po[b + 1]), fidx[fo[b]:fo[b + 1]]
        m = (po[b + 1] - po[b]) * len(f)
        got = out[4 * o:4 * (o + m)].reshape(4, -1, len(f))
        assert per_point_worst(got, ref[:, p][:, :, f], sref[:, p][:, :, f], 1e-300) <= 1e-12
        assert np.array_equal(val[o:o + m], got[0].reshape(-1))
        h = hl[8 * o:8 * (o + m)].reshape(4, 2, -1).astype(np.float64)
        hi = got.reshape(4, -1).astype(np.float32)
        assert np.array_equal(h[:, 0], hi)
        assert np.array_equal(h[:, 1], (got.reshape(4, -1) - hi).astype(np.float32))
        o += m
