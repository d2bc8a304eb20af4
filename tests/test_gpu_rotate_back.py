"""The rotate-back with each number of waves a block, and its zeros off the
grain, against the oracle."""
import numpy as np
import pytest
import torch

from helpers import oracle_grain, rel_err

pytestmark = pytest.mark.gpu


# grain cells in blocks of 64: one block and less, 256 and 257 blocks, 1023
# and 1024 blocks; one and two components; fewer angles than waves, odd count
@pytest.mark.parametrize("side", [(5, 7), (16, 16), (128, 128), (128, 129), (256, 255), (256, 256)])
@pytest.mark.parametrize("comps", [[("s", 1.0)], [("s", 1.0), ("dxy", 0.8)]])
@pytest.mark.parametrize("n_theta", [4, 5])
def test_rotate_back_matches_oracle(side, comps, n_theta):
    """FP64 results against the oracle's within 1e-10, the bound of the
    repository's FP64 sweeps; poisoned output memory is zero off the grain."""
    import paper_2205_15000_amd as qs
    ny, nx = side[1] + 3, side[0] + 2
    mask = np.zeros((ny, nx), dtype=np.uint8)
    mask[2:-1, 1:-1] = 1
    sp = dict(nx=nx, ny=ny, h=0.4, shapes=[{"kind": "mask", "mask": mask, "add": True}], n_theta=n_theta, n_poles=2,
              t=0.5, components=comps, kappa=2.3, flux_quanta=0.4, gauge="symmetric", charge_sign=-1)
    print("case %s components %d angles %d" % (side, len(comps), n_theta), flush=True)
    rng = np.random.default_rng(7)
    m = mask.astype(bool)
    d = 0.5 * (rng.standard_normal((len(comps), ny, nx)) + 1j * rng.standard_normal((len(comps), ny, nx))) * m
    a = 0.1 * rng.standard_normal((2, ny, nx))
    g = qs.Grain(sp, "fp64")
    dd, ad = torch.as_tensor(d).cuda(), torch.as_tensor(a).cuda()
    poison = [torch.full_like(dd, float("nan")), torch.full_like(ad, float("nan"))]
    del poison
    dn, j, om = [x.cpu().numpy() if torch.is_tensor(x) else x for x in g.sweep(dd, ad)]
    ref = oracle_grain(sp).iterate(d, a)
    assert rel_err(dn[:, m], ref["delta_new"][:, m]) <= 1e-10
    assert rel_err(j[:, m], ref["j"][:, m]) <= 1e-10
    assert np.all(dn[:, ~m] == 0.0) and np.all(j[:, ~m] == 0.0)
    g.close()


# partial sums in the rotate-back (up to 256 blocks of 64 grain cells and 256
# of 512 cells of the grid) and in launches of their own beyond either count;
# nodes straight from the fields (up to 9216 cells) and from packed cells
@pytest.mark.parametrize("grid,side", [((9, 8), (6, 5)), ((96, 96), (94, 90)), ((97, 96), (94, 90)),
                                       ((131, 130), (128, 128)), ((132, 132), (128, 129)), ((362, 363), (9, 9))])
@pytest.mark.parametrize("kappa", [0.0, 2.3])
def test_partial_sums_match_oracle(grid, side, kappa):
    """Free energy against the oracle's (1e-10, the bound of the FP64 sweeps),
    and one Picard step of A, which takes the mean current off, against the
    A-solve of the same current (1e-12: sums in another order)."""
    import paper_2205_15000_amd as qs
    nx, ny = grid
    mask = np.zeros((ny, nx), dtype=np.uint8)
    mask[1:1 + side[1], 1:1 + side[0]] = 1
    sp = dict(nx=nx, ny=ny, h=0.4, shapes=[{"kind": "mask", "mask": mask, "add": True}], n_theta=4, n_poles=2, t=0.5,
              components=[("s", 1.0)], kappa=kappa, flux_quanta=0.4, gauge="symmetric", charge_sign=-1)
    print("case grid %s grain %s kappa %g" % (grid, side, kappa), flush=True)
    rng = np.random.default_rng(11)
    y, x = np.mgrid[:ny, :nx]
    d = (1.0 + 0.2 * rng.standard_normal((1, ny, nx)) + 0.3j) * mask
    a = 0.05 * np.stack([np.sin(0.1 * y), np.cos(0.07 * x)]) * (kappa > 0.0)
    g = qs.Grain(sp, "fp64")
    dd, ad = torch.as_tensor(d).cuda(), torch.as_tensor(a).cuda()
    om = g.sweep(dd, ad)[2]
    ref = oracle_grain(sp).iterate(d, a)["omega_total"]
    assert abs(float(om) - ref) <= 1e-10 * abs(ref)
    if kappa > 0.0:
        g.reset_bc()
        want = g.solve_A(g.sweep(dd, 0.0 * ad)[1], B=False)[0].cpu().numpy()
        g.reset_bc()
        d1, a1 = dd.clone(), 0.0 * ad
        g.scf(d1, a1, alpha=1.0, tol=0.0, max_iter=1)
        assert np.max(np.abs(a1.cpu().numpy() - want)) <= 1e-12 * np.max(np.abs(want))
    g.close()
