"""What a batch's captured graph was captured with, and calls between its
replays that change it."""
import numpy as np
import pytest
import torch

from paper_2205_15000_amd import workloads as wl

pytestmark = pytest.mark.gpu

NAMES = ["small_d110_field", "s_disc_32", "small_polygon_landau"]


class _Picard:
    """The single-grain loop that a batch of step one runs."""

    def __init__(self, qs, name):
        sp = wl.spec(name)
        self.g = qs.Grain(sp, "fp64")
        self.d = torch.as_tensor(wl.initial_delta(name, sp)).cuda()
        self.a = torch.as_tensor(wl.initial_A(name, sp)).cuda()
        self.screened = sp.get("kappa", 0.0) > 0.0
        if not self.screened:
            self.a = 0.0 * self.a
        self.start = (self.d.clone(), self.a.clone())

    def iterate(self, n):
        for _ in range(n):
            dn, j, _ = self.g.sweep(self.d, self.a)
            if self.screened:
                self.a = self.g.solve_A(j, B=False)[0]
            self.d = dn


def _batch(qs):
    ref = [_Picard(qs, nm) for nm in NAMES]
    grains = [qs.Grain(wl.spec(nm), "fp64") for nm in NAMES]
    b = qs.Batch(grains)
    for i, r in enumerate(ref):
        b.set_fields(i, *r.start)
    return ref, grains, b


def _check(ref, b):
    """The same marches; sums in other orders: 1e-11."""
    for i, r in enumerate(ref):
        d, a = [x.cpu().numpy() for x in b.get_fields(i)]
        dr, ar = r.d.cpu().numpy(), r.a.cpu().numpy()
        assert np.max(np.abs(d - dr)) <= 1e-11 * np.max(np.abs(dr)), NAMES[i]
        assert np.max(np.abs(a - ar)) <= 1e-11 * max(np.max(np.abs(ar)), 1e-30), NAMES[i]


def _close(ref, grains, b):
    b.close()
    for g in grains + [r.g for r in ref]:
        g.close()


def test_bulk_starts_between_replays():
    """Boundary stores reset twice between replays: the eager sweeps from bulk
    starts bring the stores' parity back to the graph's, whose arguments they
    must not have touched."""
    import paper_2205_15000_amd as qs
    ref, grains, b = _batch(qs)
    for reset, n in ((False, 5), (True, 1), (True, 5), (False, 2), (True, 3), (False, 4)):
        if reset:
            for g in grains + [r.g for r in ref]:
                g.reset_bc()
        b.iterate(n, graph=True)
        torch.zeros(1000, device="cuda").sum().item()  # eager work between replays
        for r in ref:
            r.iterate(n)
        _check(ref, b)
    _close(ref, grains, b)


def test_another_A_solver_between_replays():
    import paper_2205_15000_amd as qs
    ref, grains, b = _batch(qs)
    for eps in (0.0, 1e-6, 1e-2, 0.0, 1e-6):
        print("case eps %g" % eps, flush=True)
        for g in (grains[0], ref[0].g):
            g.set_A_solver(eps)
        n = 5 if eps == 0.0 else 4
        b.iterate(n, graph=True)
        for r in ref:
            r.iterate(n)
        _check(ref, b)
    _close(ref, grains, b)
