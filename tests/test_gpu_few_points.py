"""GPU: batches of few points, for which tables and the FP64 adjoint take code of
their own: at the edges of 8 points and of one 16-point chunk, and of the
adjoint's 16-function blocks and 48-row items, against the oracle.

Bars: the FP64 bar 1e-12 of each value's own scale; a batch's values are the
same bits whatever batches surround it."""
import numpy as np
import pytest

import oracle
from helpers import blocks_to_store, gpu_available, per_point_worst
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


@pytest.mark.parametrize("n", [1, 16, 17, 48, 49, 113])
@pytest.mark.parametrize("P", [1, 7, 16])
def test_adjoint(n, P):
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2608_00773_amd as q
    import torch
    wl, other = two_atoms(n, P, 700 * n + P), two_atoms(40, 33, 7)
    plan, both = q.Plan(wl, p_max=1000), q.Plan([wl, other], p_max=1000)
    assert plan.info["n_batches"] == 1
    pairs, po = plan.pairs()
    nfn = wl.atom_nfn()
    rng = np.random.default_rng(n + P)
    coef = [rng.standard_normal((5, nfn[a], nfn[b])) for a, b in pairs]
    cst = torch.from_numpy(blocks_to_store(coef, po)).cuda()
    off = both.systems()
    call = torch.zeros((5, both.info["store_len"]), dtype=torch.float64, device="cuda")
    call[:, off["store"][0]:off["store"][1]] = cst
    _, parts, sd = oracle.density(wl, pairs, coef, idx=np.arange(P), weight_mode=0, with_parts=True, with_scale=True)
    print("n %d P %d" % (n, P), flush=True)
    for terms in (q.TERM_ALL, q.TERM_LL, q.TERM_SO):
        ref = sum(parts[:, k] for k in range(3) if terms >> k & 1)
        first = None
        for shape in ((0, 0), (1, 0), (0, 3), (1, 2)):
            plan.set_launch(q.KERNEL_DENSITY, *shape)
            out = torch.full((P,), float("nan"), dtype=torch.float64, device="cuda")
            q.density_on_grid(plan, cst, terms, 0, out)
            got = out.cpu().numpy()
            assert per_point_worst(got, ref, oracle.density_scale(sd, terms=terms), 1e-300) <= 1e-12
            first = got if first is None else first
            assert np.array_equal(got, first), shape
        out = torch.empty(P + 33, dtype=torch.float64, device="cuda")
        q.density_on_grid(both, call, terms, 0, out)
        assert np.array_equal(out[:P].cpu().numpy(), first)
