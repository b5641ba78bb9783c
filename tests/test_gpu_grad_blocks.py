"""GPU: the density and its gradient at the edges of the product's items: 1 to
9 blocks of 16 functions against 1 to 9 blocks of 16 points in one batch, i.e.
items of every size from 1 x 1 to 4 x 4 blocks, against the oracle at the FP64
bar, 1e-12 of each value's own scale."""
import numpy as np
import pytest

import oracle
from helpers import blocks_to_store, gpu_available, per_point_worst
from test_gpu_blocks import two_atoms

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [7, 32, 41, 64, 70, 129])
@pytest.mark.parametrize("P", [3, 32, 33, 50, 65, 80, 100, 130])
def test_gradient_items_against_oracle(n, P):
    if not gpu_available():
        pytest.skip("no GPU")
    import paper_2608_00773_amd as q
    import torch
    wl = two_atoms(n, P, 1000 * n + P)
    plan = q.Plan(wl, p_max=1000)
    assert plan.info["n_batches"] == 1 and plan.info["n_fn"] == n
    pairs, po = plan.pairs()
    nfn = wl.atom_nfn()
    print("n %d P %d" % (n, P), flush=True)
    rng = np.random.default_rng(n + P)
    coef = [rng.standard_normal((5, nfn[a], nfn[b])) for a, b in pairs]
    cst = torch.from_numpy(blocks_to_store(coef, po)[0]).cuda()
    grad = torch.full((4, P), float("nan"), dtype=torch.float64, device="cuda")
    q.density_gradient_on_grid(plan, cst, grad)
    ref, scale = oracle.density_grad(wl, pairs, [c[0] for c in coef], idx=np.arange(P), with_scale=True)
    assert per_point_worst(grad.cpu().numpy(), ref.T, scale.T, 1e-300) <= 1e-12
