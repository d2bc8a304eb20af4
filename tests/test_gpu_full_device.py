"""Calls on a device whose memory is nearly taken up by others."""
import numpy as np
import pytest
import torch

from paper_2205_15000_amd import workloads as wl

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def _fill(leave):
    """Takes the device's memory until about `leave` bytes are free."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    for _ in range(8):
        free = torch.cuda.mem_get_info()[0]
        if free <= leave + 64 * MIB:
            break
        held.append(torch.empty(free - leave, dtype=torch.uint8, device="cuda"))
    print("free: %d MiB" % (torch.cuda.mem_get_info()[0] // MIB), flush=True)
    return held


def test_grain_tables_take_the_place_of_idle_work_memory():
    """The LDOS work memory of an idle grain (about 3 GB) gives way to the
    tables of a new grain (over 1 GB) where about 300 MiB are free."""
    import paper_2205_15000_amd as qs
    sp = wl.spec("d_disc_200")
    d = torch.as_tensor(wl.initial_delta("d_disc_200", sp)).cuda()
    a = torch.as_tensor(wl.initial_A("d_disc_200", sp)).cuda()
    g = qs.Grain(sp, "fp64")
    g.set_pairing(False)
    en = np.linspace(0.01, 0.4, 64)
    before = torch.cuda.mem_get_info()[0]
    out = g.ldos(d, a, en, 0.03, 1)
    torch.cuda.synchronize()
    assert before - torch.cuda.mem_get_info()[0] > 2048 * MIB
    big = wl.spec("d110_square_400")
    full = _fill(300 * MIB)
    try:
        h = qs.Grain(big, "fp64")
        assert h.mask().sum() == h.info["n_grain_cells"]
        h.close()
    finally:
        del full
        torch.cuda.empty_cache()
    # the first grain maps its work memory again
    assert torch.equal(g.ldos(d, a, en, 0.03, 1), out)
    g.close()


def test_batch_after_an_autotune_that_ran_out_of_memory():
    """Three energies per lane need 2.5 GB of spill, more than there is: the
    autotuner fails, and the batch iterates as one that was never tuned."""
    import paper_2205_15000_amd as qs
    sp = wl.spec("d_disc_200")
    d = torch.as_tensor(wl.initial_delta("d_disc_200", sp)).cuda()
    a = torch.as_tensor(wl.initial_A("d_disc_200", sp)).cuda()
    out = []
    for tune in (False, True):
        g = qs.Grain(sp, "fp64")
        b = qs.Batch([g])
        b.set_fields(0, d, a)
        b.iterate(1, graph=False)
        if tune:
            full = _fill(300 * MIB)
            try:
                with pytest.raises(qs.QcError, match="memory"):
                    b.autotune(1)
            finally:
                del full
                torch.cuda.empty_cache()
            assert b.info()["energies_per_lane"] == 0
        b.set_fields(0, d, a)
        g.reset_bc()
        b.iterate(3, graph=True)
        out.append(b.get_fields(0)[0])
        b.close()
        g.close()
    assert torch.equal(out[0], out[1])


def test_reverse_mode_after_calls_that_ran_out_of_memory():
    """Its tables and buffers take about 1 GB. Calls that find less free, from
    nearly nothing on, fail or not; the call with enough memory afterwards
    gives what a grain that never failed gives (the same kernels: 1e-13)."""
    import paper_2205_15000_amd as qs
    sp = wl.spec("d_disc_200")
    d = torch.as_tensor(wl.initial_delta("d_disc_200", sp)).cuda()
    a = torch.as_tensor(wl.initial_A("d_disc_200", sp)).cuda()
    gj = torch.randn(a.shape, dtype=a.dtype, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    ref, g = qs.Grain(sp, "fp64"), qs.Grain(sp, "fp64")
    ref.sweep(d, a)
    want = ref.sweep_adjoint(d, a, d, gj, 0.2)
    ref.close()
    g.sweep(d, a)
    failed = 0
    for mib, every in ((80, 32), (350, 32), (500, 32), (520, 7), (560, 32), (100, 7)):
        full = _fill(mib * MIB)
        g.set_adjoint_checkpoint(every)
        try:
            g.sweep_adjoint(d, a, d, gj, 0.2)
        except qs.QcError as e:
            assert "memory" in str(e)
            failed += 1
        finally:
            torch.cuda.synchronize()
            del full
            torch.cuda.empty_cache()
    assert failed >= 3, failed
    g.set_adjoint_checkpoint(32)
    got = g.sweep_adjoint(d, a, d, gj, 0.2)
    for p, q in zip(got, want):
        assert (p - q).abs().max() <= 1e-13 * q.abs().max()
    g.close()
