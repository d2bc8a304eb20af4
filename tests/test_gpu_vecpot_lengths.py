"""The FFT A-solve at the lengths whose launches need the most LDS."""
import math

import numpy as np
import pytest
import torch

from helpers import rel_err
from oracle import fields

pytestmark = pytest.mark.gpu

H, KAPPA = 0.3, 2.3


def _kernel(m, n, h):
    """The oracle's cell-averaged Green's function, each value by the same
    operations in the same order as the library's table.  The terms, about
    side^2, cancel to a few units, so that two evaluations in FP64 differ by
    1e-11 of A from side 900 on (7e-11 at 2048): that is not measured here."""
    def alpha(a, b):
        return (1 + 2 * a) * (1 + 2 * b) * math.log(0.5 * (1 + 2 * a) * (1 + 2 * a) + 0.5 * (1 + 2 * b) * (1 + 2 * b))

    def beta(a, b):
        return (-2 * a * a + 2 * b * b + 4 * b + 1) * math.atan((1 + 2 * a) / (1 + 2 * b))

    def value(m, n):
        tot = 0.0
        for a in (m, -m):
            for b in (n, -n):
                tot += alpha(a, b) + beta(a, b) + beta(b, a)
        return h * h / (4.0 * math.pi) * (2.0 * math.log(h) - math.log(2.0) - 3.0 + 0.25 * tot)

    m, n = np.broadcast_arrays(m, n)
    return np.reshape([value(float(x), float(y)) for x, y in zip(m.ravel(), n.ravel())], m.shape)


def _grain(qs, nx, ny):
    m = np.ones((ny, nx), dtype=np.uint8)
    m[:, nx // 2:] = np.arange(ny)[:, None] % 3 != 2  # (grooves, so that the mask counts)
    m[0] = 1
    sp = dict(nx=nx, ny=ny, h=H, shapes=[{"kind": "mask", "mask": m, "add": True}], n_theta=4, n_poles=1, t=0.5,
              components=[("s", 1.0)], kappa=KAPPA, flux_quanta=0.0, gauge="symmetric", charge_sign=-1)
    return qs.Grain(sp, "fp64"), m.astype(bool)


def _check(g, m, monkeypatch, seed=3):
    """Within 1e-11 of the oracle's correlation with the same kernel."""
    monkeypatch.setattr(fields, "green_kernel", _kernel)
    ny, nx = m.shape
    j = np.random.default_rng(seed).standard_normal((2, ny, nx))
    A, _ = g.solve_A(torch.as_tensor(j).cuda())
    ref = np.stack(fields.solve_A(j[0], j[1], m, H, KAPPA, method="fft")[:2])
    assert rel_err(A.cpu().numpy(), ref) <= 1e-11


# lengths 1024, 2048 (64 KB and the means), 2560, 3072, 4096 (the largest), as
# rows and as columns
@pytest.mark.parametrize("side", [400, 900, 1025, 1400, 2048])
@pytest.mark.parametrize("rows", [True, False])
def test_long_lengths_match_oracle(side, rows, monkeypatch):
    import paper_2205_15000_amd as qs
    nx, ny = (side, 5) if rows else (5, side)
    print("case %dx%d" % (nx, ny), flush=True)
    g, m = _grain(qs, nx, ny)
    _check(g, m, monkeypatch)
    g.close()


def test_a_smaller_grain_leaves_a_larger_ones_launches_alone(monkeypatch):
    """The largest length in both directions, then grains of smaller ones
    that also need more than 64 KB, then the first again."""
    import paper_2205_15000_amd as qs
    big = [_grain(qs, 2048, 4), _grain(qs, 4, 2048)]
    small = [_grain(qs, 1030, 4), _grain(qs, 4, 1030), _grain(qs, 12, 9)]
    for i, (g, m) in enumerate(big + small + big):
        print("case %d" % i, flush=True)
        _check(g, m, monkeypatch, seed=i)
    for g, _ in big + small:
        g.close()
