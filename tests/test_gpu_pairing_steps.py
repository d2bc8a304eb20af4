"""The steps that a grain's paired sweeps march, against the planner's count."""
import pytest

from paper_2205_15000_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["s_disc_32", "small_d110_field", "small_holed_mixed", "small_polygon_landau"])
def test_swept_steps_equal_the_plans(name):
    import paper_2205_15000_amd as qs
    sp = wl.spec(name)
    g, p = qs.Grain(sp, "fp64"), qs.Plan(sp)
    available, enabled, steps = g.pairing()
    assert (available, steps) == (p.pairing()[0], p.pairing()[1]) and enabled == available
    if available:
        g.set_pairing(False)
        assert g.pairing()[1:] == (False, g.steps_per_sweep)
    g.close()
