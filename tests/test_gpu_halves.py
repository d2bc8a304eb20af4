"""The sweep's two half-marches per segment, against the oracle at the sizes
where their bookkeeping can go wrong, and the step's two forms."""
import math

import numpy as np
import pytest
import torch

from helpers import oracle_grain, rel_err
from paper_2205_15000_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _spec(nx, ny, h, n_theta, n_poles, turn):
    return dict(nx=nx, ny=ny, h=h, shapes=[wl._square(0.0, 0.0, 0.93 * min(nx, ny) * h, turn)], n_theta=n_theta,
                n_poles=n_poles, t=0.3, components=[("dx2y2", 1.0)], crystal_rotation=0.06, kappa=3.0, flux_quanta=0.7,
                gauge="symmetric", charge_sign=-1)


def _fields(sp, amp, seed=5):
    rng = np.random.default_rng(seed)
    shape = (sp["ny"], sp["nx"])
    d = 0.25 * (1.0 + 0.2 * rng.standard_normal(shape)) * np.exp(1j * rng.uniform(-1.0, 1.0, shape))
    return d[None], amp * rng.standard_normal((2,) + shape)


# node counts of a segment run from 0 to about the grid's side (odd and even,
# one node included); the poles give every lane layout: padded lanes, two
# segments and one per wave, groups below and above eight lanes; amplitude of
# A: 0.05 keeps |K_y| = h |v.A| / 2 small, 6 takes it across 0.49 from node to
# node, where a wave leaves the step's short form
@pytest.mark.parametrize("amp", [0.05, 6.0])
@pytest.mark.parametrize("nx,ny,n_theta,n_poles,lanes", [
    (3, 3, 8, 1, 0), (4, 3, 7, 3, 1), (5, 7, 12, 5, 2), (9, 8, 16, 8, 2), (8, 9, 12, 17, 3), (11, 10, 16, 33, 4),
    (13, 6, 8, 64, 1), (12, 13, 12, 64, 0), (7, 7, 8, 24, 8)])
def test_half_marches_match_oracle(nx, ny, n_theta, n_poles, lanes, amp):
    import paper_2205_15000_amd as qs
    sp = _spec(nx, ny, 0.4, n_theta, n_poles, 0.07)
    d, a = _fields(sp, amp)
    og = oracle_grain(sp)
    m = og.mask
    for precision, tol in (("fp64", 1e-10), ("mixed", 2e-5)):
        print("case %dx%d %d poles lanes %d amp %g %s" % (nx, ny, n_poles, lanes, amp, precision), flush=True)
        g = qs.Grain(sp, precision)
        g.set_lanes(lanes)
        bc = None
        for it in range(2):  # bulk starts, then specular taps
            dn, j, om, od = g.sweep(torch.as_tensor(d).cuda(), torch.as_tensor(a).cuda(), omega_density=True)
            ref = og.iterate(d, a, bc)
            bc = ref["bc"]
            assert rel_err(dn.cpu().numpy()[:, m], ref["delta_new"][:, m]) <= tol, (precision, it)
            # j and omega may vanish to rounding: measured against the gap's scale
            scale = np.linalg.norm(ref["delta_new"][:, m]) / math.sqrt(m.sum())
            for got, want in ((j.cpu().numpy(), ref["j"]), (od.cpu().numpy(), ref["omega_density"])):
                norm = max(np.linalg.norm(want), scale * math.sqrt(m.sum()))
                assert np.linalg.norm(got - want) <= tol * norm, (precision, it)
        g.close()


def test_half_march_counts_of_these_grids_include_none_one_odd_and_even():
    import paper_2205_15000_amd as qs
    n = set()
    for nx, ny, n_theta in ((3, 3, 8), (4, 3, 7), (5, 7, 12), (9, 8, 16)):
        n |= set(qs.Plan(_spec(nx, ny, 0.4, n_theta, 1, 0.07)).segments()[:, 5].astype(int).tolist())
    assert {0, 1, 2, 3, 5, 6} <= n
