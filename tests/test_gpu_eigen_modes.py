"""The eigen-truncated A-solve at the edges of its tiles and of the shares
that the waves of a block take of the contraction."""
import numpy as np
import pytest
import torch

from oracle import fields

pytestmark = pytest.mark.gpu


# sides below, at and past the 16 and 32 cells of a tile and the 16 indices of
# a chunk, odd ones (rows not on 16 bytes) and one with part-filled blocks of
# four row tiles; one mode (fewer chunks than waves), several and all
@pytest.mark.parametrize("n", [8, 15, 16, 17, 32, 33, 47, 65, 81])
@pytest.mark.parametrize("eps", [0.9, 1e-3, 1e-300])
def test_eigen_modes_tile_edges_match_oracle(n, eps):
    """1e-10 of the largest |A|, the bound of the full test of this solve."""
    import paper_2205_15000_amd as qs
    print("case n %d eps %g" % (n, eps), flush=True)
    mask = np.ones((n, n), dtype=np.uint8)
    mask[: n // 3, n // 2:] = 0
    sp = dict(nx=n, ny=n, h=0.3, shapes=[{"kind": "mask", "mask": mask, "add": True}], n_theta=4, n_poles=2, t=0.5,
              components=[("s", 1.0)], kappa=2.3, flux_quanta=0.0, gauge="symmetric", charge_sign=-1)
    g = qs.Grain(sp, "fp64")
    j = np.random.default_rng(n).standard_normal((2, n, n))
    g.set_A_solver(eps)
    A, _ = g.solve_A(torch.as_tensor(j).cuda(), B=False)
    ax, ay, nstar = fields.solve_A_eigen(j[0], j[1], mask.astype(bool), sp["h"], sp["kappa"], eps)
    assert g.A_solver()[1] == nstar
    ref = np.stack([ax, ay])
    assert np.max(np.abs(A.cpu().numpy() - ref)) <= 1e-10 * np.max(np.abs(ref))
    g.close()
