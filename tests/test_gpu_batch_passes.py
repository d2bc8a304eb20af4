"""The passes of a batch over grains of every kind at once."""
import numpy as np
import pytest
import torch

from paper_2205_15000_amd import workloads as wl

pytestmark = pytest.mark.gpu

NAMES = ["small_d110_field", "small_holed_mixed", "small_mask_blob", "small_polygon_landau", "s_disc_32"]


# one and several components, with and without screening, paired and not, and
# enough grains for blocks of 16, 8 and 4 waves (1, 3 and 30 of each)
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("copies", [1, 3, 30])
@pytest.mark.parametrize("graph", [False, True])
def test_batch_equals_single_grain_picard(precision, copies, graph):
    """Five iterations with a step of one against the single-grain loop from
    the same fields (the same marches; sums in other orders: 1e-11, and 1e-5
    where a last bit of the FP32 marches can turn), and zeros off the grain."""
    import paper_2205_15000_amd as qs
    tol = 1e-11 if precision == "fp64" else 1e-5
    print("case batch %s x%d graph %s" % (precision, copies, graph), flush=True)
    ref = []
    for name in NAMES:
        sp = wl.spec(name)
        g = qs.Grain(sp, precision)
        d = torch.as_tensor(wl.initial_delta(name, sp)).cuda()
        a = torch.as_tensor(wl.initial_A(name, sp)).cuda()
        if sp.get("kappa", 0.0) <= 0.0:
            a = a * 0.0
        start = (d.clone(), a.clone())
        for _ in range(5):
            dn, j, _ = g.sweep(d, a)
            if sp.get("kappa", 0.0) > 0.0:
                a = g.solve_A(j, B=False)[0]
            d = dn
        ref.append((sp, start, d.cpu().numpy(), a.cpu().numpy()))
        g.close()
    grains = [qs.Grain(ref[i % len(NAMES)][0], precision) for i in range(len(NAMES) * copies)]
    b = qs.Batch(grains)
    for i in range(len(grains)):
        b.set_fields(i, *ref[i % len(NAMES)][1])
    b.iterate(5, graph=graph)
    for i, g in enumerate(grains):
        sp, _, dr, ar = ref[i % len(NAMES)]
        d, a = [x.cpu().numpy() for x in b.get_fields(i)]
        assert np.max(np.abs(d - dr)) <= tol * np.max(np.abs(dr)), NAMES[i % len(NAMES)]
        assert np.max(np.abs(a - ar)) <= tol * max(np.max(np.abs(ar)), 1e-30), NAMES[i % len(NAMES)]
        assert np.all(d[:, ~g.mask().astype(bool)] == 0.0)
    b.close()
    for g in grains:
        g.close()
