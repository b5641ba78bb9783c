"""GPU: density_on_grid with the spin-orbit terms but not the V term, which has
a kernel form of its own (nine products), at the edges of its 16-function
blocks, 48-row items and 16-point chunks, against the oracle; every launch
shape gives the same bits.

Bar: the FP64 bar 1e-12 of each point's own scale over the selected terms."""
import numpy as np
import pytest

import oracle
from helpers import blocks_to_store, gpu_available, per_point_worst
from test_gpu_blocks import two_atoms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 16, 17, 48, 49, 97, 130])
@pytest.mark.parametrize("P", [1, 16, 17, 65, 130])
def test_spin_orbit_without_v(n, P):
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2608_00773_amd as q
    import torch
    wl = two_atoms(n, P, 300 * n + P)
    plan = q.Plan(wl, p_max=1000)
    assert plan.info["n_batches"] == 1 and plan.info["n_fn"] == n
    pairs, po = plan.pairs()
    nfn = wl.atom_nfn()
    rng = np.random.default_rng(n + P)
    coef = [rng.standard_normal((5, nfn[a], nfn[b])) for a, b in pairs]
    cst = torch.from_numpy(blocks_to_store(coef, po)).cuda()
    _, parts, sd = oracle.density(wl, pairs, coef, idx=np.arange(P), weight_mode=0, with_parts=True, with_scale=True)
    print("n %d P %d" % (n, P), flush=True)
    for terms in (q.TERM_SO, q.TERM_SS | q.TERM_SO):
        ref = parts[:, 2] + (parts[:, 1] if terms & q.TERM_SS else 0.0)
        first = None
        for shape in ((0, 0), (1, 0), (0, 3), (1, 2)):
            plan.set_launch(q.KERNEL_DENSITY, *shape)
            out = torch.full((P,), float("nan"), dtype=torch.float64, device="cuda")
            q.density_on_grid(plan, cst, terms, 0, out)
            got = out.cpu().numpy()
            assert per_point_worst(got, ref, oracle.density_scale(sd, terms=terms), 1e-300) <= 1e-12
            first = got if first is None else first
            assert np.array_equal(got, first), shape
