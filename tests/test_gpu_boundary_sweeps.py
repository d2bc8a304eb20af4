"""Boundary-only Matsubara sweeps (the burn-in of the Luttinger-Ward
functional) against whole sweeps."""
import numpy as np
import pytest
import torch

from paper_2205_15000_amd import workloads as wl

pytestmark = pytest.mark.gpu


# paired and unpaired grains, lane shapes with full and part-filled last lanes
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("pair", [True, False])
@pytest.mark.parametrize("lanes", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("name", ["small_d110_field", "small_mask_blob", "small_polygon_landau"])
def test_burn_in_equals_whole_sweeps(name, lanes, pair, precision):
    """With one coupling (0.5) the functional depends on the burn-in only
    through sum Re(conj(Delta) Delta_new[Delta / 2]), so its changes from no
    burn-in to one and to two sweeps are in the ratio that whole sweeps give.
    End values that differ in the last bit of the FP32 marches (6e-8) would
    move the ratio, of changes some 1e-2 of the sum, by 1e-5; the FP64 sums
    leave 1e-11 of it."""
    import paper_2205_15000_amd as qs
    sp = wl.spec(name)
    print("case %s lanes %d pair %s %s" % (name, lanes, pair, precision), flush=True)
    d = torch.as_tensor(wl.initial_delta(name, sp)).cuda()
    a = torch.as_tensor(wl.initial_A(name, sp)).cuda()
    g = qs.Grain(sp, precision)
    if pair and not g.pairing()[0]:
        g.close()
        return
    g.set_pairing(pair)
    g.set_lanes(lanes)
    om = []
    for bc in range(3):
        r = g.free_energy_lw(d, a, 1, bc)
        om.append(float(r[0] if isinstance(r, tuple) else r))
    g.reset_bc()
    s = []
    for _ in range(3):
        dn = g.sweep(0.5 * d, a)[0]
        s.append(float((torch.conj(d) * dn).real.sum()))
    got, ref = (om[2] - om[0]) / (om[1] - om[0]), (s[2] - s[0]) / (s[1] - s[0])
    assert abs(got - ref) <= 1e-8 * abs(ref), (got, ref)
    g.close()
