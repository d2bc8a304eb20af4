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
