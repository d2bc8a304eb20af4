"""The rotate-back where its number of waves a block changes: exactly 256 and
257, 1023 and 1024 blocks of 64 grain cells."""
import numpy as np
import pytest
import torch

from helpers import oracle_grain, rel_err

pytestmark = pytest.mark.gpu


# cells of the last block: one, or all 64
@pytest.mark.parametrize("cells", [255 * 64 + 1, 256 * 64, 256 * 64 + 1, 1022 * 64 + 1, 1023 * 64, 1023 * 64 + 1])
@pytest.mark.parametrize("comps", [[("s", 1.0)], [("s", 1.0), ("dxy", 0.8)]])
def test_block_counts_match_oracle(cells, comps):
    """FP64 results within 1e-10 of the oracle's, the bound of the FP64 sweeps."""
    import paper_2205_15000_amd as qs
    side = 256 if cells > 512 * 64 else 128
    rows, rest = divmod(cells, side)
    mask = np.zeros((rows + 3, side + 2), dtype=np.uint8)
    mask[1:1 + rows, 1:-1] = 1
    mask[1 + rows, 1:1 + rest] = 1
    assert mask.sum() == cells
    ny, nx = mask.shape
    sp = dict(nx=nx, ny=ny, h=0.4, shapes=[{"kind": "mask", "mask": mask, "add": True}], n_theta=4, n_poles=1, t=0.5,
              components=comps, kappa=2.3, flux_quanta=0.4, gauge="symmetric", charge_sign=-1)
    print("case %d cells, %d components" % (cells, len(comps)), flush=True)
    rng = np.random.default_rng(7)
    m = mask.astype(bool)
    d = 0.5 * (rng.standard_normal((len(comps), ny, nx)) + 1j * rng.standard_normal((len(comps), ny, nx))) * m
    a = 0.1 * rng.standard_normal((2, ny, nx))
    g = qs.Grain(sp, "fp64")
    assert g.info["n_grain_cells"] == cells
    dn, j, om = g.sweep(torch.as_tensor(d).cuda(), torch.as_tensor(a).cuda())
    ref = oracle_grain(sp).iterate(d, a)
    assert rel_err(dn.cpu().numpy()[:, m], ref["delta_new"][:, m]) <= 1e-10
    assert rel_err(j.cpu().numpy()[:, m], ref["j"][:, m]) <= 1e-10
    assert abs(om - ref["omega_total"]) <= 1e-10 * abs(ref["omega_total"])
    g.close()
