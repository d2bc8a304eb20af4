"""Buffers of the reverse mode on grains that come to it by other ways."""
import ctypes

import pytest
import torch

from paper_2205_15000_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _inputs(name):
    sp = wl.spec(name)
    d = torch.as_tensor(wl.initial_delta(name, sp)).cuda()
    a = torch.as_tensor(wl.initial_A(name, sp)).cuda()
    gen = torch.Generator(device="cuda").manual_seed(5)
    gd = torch.randn(d.shape, dtype=d.dtype, device="cuda", generator=gen)
    gj = torch.randn(a.shape, dtype=a.dtype, device="cuda", generator=gen)
    return sp, d, a, gd, gj


def _equal(x, y):
    """The same kernels on the same inputs."""
    for p, q in zip(x, y):
        assert (p - q).abs().max() <= 1e-13 * q.abs().max()


@pytest.mark.parametrize("every", [0, 3])
def test_reverse_mode_after_an_allocation_free_sweep(every):
    """A grain from a batch has no spill of its own, nor does the
    allocation-free sweep give it one."""
    import paper_2205_15000_amd as qs
    print("case checkpoint %d" % every, flush=True)
    sp, d, a, gd, gj = _inputs("small_d110_field")
    ref, g = qs.Grain(sp, "fp64"), qs.Grain(sp, "fp64")
    ref.sweep(d, a)
    ref.set_adjoint_checkpoint(every)
    want = ref.sweep_adjoint(d, a, gd, gj, 0.3)
    qs.Batch([g]).close()
    dn, j = torch.empty_like(d), torch.empty_like(a)
    p = [ctypes.c_void_p(t.data_ptr()) for t in (d, a, dn, j)]
    rc = qs.lib.qc_sweep_static(g._g, p[0], p[1], p[2], p[3], None, None,
                                ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0, qs.lib.qc_last_error()
    g.set_adjoint_checkpoint(every)
    _equal(g.sweep_adjoint(d, a, gd, gj, 0.3), want)
    ref.close()
    g.close()
