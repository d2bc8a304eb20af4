"""Lane shapes that the caller sets: each runs as it is, alone and with the
longest segments on twice the lanes."""
import numpy as np
import pytest
import torch

from helpers import oracle_grain, rel_err
from paper_2205_15000_amd import workloads as wl

pytestmark = pytest.mark.gpu

NAME = "small_d110_field"


def _case(n_poles):
    sp = dict(wl.spec(NAME), n_poles=n_poles)
    return sp, wl.initial_delta(NAME, sp), wl.initial_A(NAME, sp)


# each number of energies a lane with one, four, eight (the node sums change
# form at 4 and 8 lanes a segment) and more lanes, and with part-filled lanes
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-10), ("mixed", 2e-5)])
@pytest.mark.parametrize("n_poles,lanes", [(1, 1), (8, 1), (2, 2), (8, 2), (15, 2), (3, 3), (7, 3), (24, 3), (4, 4), (13, 4),
                                           (32, 4), (8, 8), (30, 8), (61, 8), (64, 8)])
def test_forced_shape_matches_oracle(n_poles, lanes, precision, tol):
    """Two chained sweeps in one shape (the split is off), at the bounds of
    the repository's sweeps."""
    import paper_2205_15000_amd as qs
    print("case %d poles lanes %d %s" % (n_poles, lanes, precision), flush=True)
    sp, d, a = _case(n_poles)
    og = oracle_grain(sp)
    m = og.mask
    g = qs.Grain(sp, precision)
    g.set_lanes(lanes)
    g.set_split(0.0)
    assert g.lanes()[0] == lanes and g.split()[1] == 0
    bc = None
    for it in range(2):
        dn, j, om = g.sweep(torch.as_tensor(d).cuda(), torch.as_tensor(a).cuda())
        ref = og.iterate(d, a, bc)
        bc = ref["bc"]
        assert rel_err(dn.cpu().numpy()[:, m], ref["delta_new"][:, m]) <= tol, it
        assert rel_err(j.cpu().numpy()[:, m], ref["j"][:, m]) <= 10 * tol, it
        assert abs(om - ref["omega_total"]) <= tol * abs(ref["omega_total"]), it
    g.close()


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-13), ("mixed", 1e-6)])
@pytest.mark.parametrize("n_poles,lanes", [(8, 2), (8, 4), (64, 4), (8, 8), (30, 8)])
def test_split_inside_a_forced_shape(n_poles, lanes, precision, tol):
    """On a grain that leaves wave slots empty a forced shape is kept: only
    the longest segments take twice the lanes, with the results of one shape
    (the order of the pole sums: 1e-13; FP32 terms of another variant: 1e-6)."""
    import paper_2205_15000_amd as qs
    print("case %d poles lanes %d %s" % (n_poles, lanes, precision), flush=True)
    sp, d, a = _case(n_poles)
    d, a = torch.as_tensor(d).cuda(), torch.as_tensor(a).cuda()
    out = []
    for frac in (0.8, 0.0):
        g = qs.Grain(sp, precision)
        g.set_lanes(lanes)
        g.set_split(frac)
        assert g.lanes()[0] == lanes
        n_wide = g.split()[1]
        assert 0 < n_wide < g.info["n_segments"] // 2 if frac > 0.0 else n_wide == 0, n_wide
        x = d
        for _ in range(3):
            x, j, om = g.sweep(x, a)
        out.append((x.cpu().numpy(), j.cpu().numpy(), om))
        g.close()
    for p, f in zip(out[0][:2], out[1][:2]):
        assert np.max(np.abs(p - f)) <= tol * np.max(np.abs(f))
    assert abs(out[0][2] - out[1][2]) <= tol * abs(out[1][2])
