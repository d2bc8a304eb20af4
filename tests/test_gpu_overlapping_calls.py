"""Work memory of LDOS calls of one grain that overlap in time."""
import threading

import numpy as np
import pytest
import torch

from paper_2205_15000_amd import workloads as wl

pytestmark = pytest.mark.gpu


def test_overlapping_ldos_calls_keep_their_own_memory():
    """Two threads on one grain with the same fields, one with more energies
    (a larger block) than the other: bit for bit the calls made in turn."""
    import paper_2205_15000_amd as qs
    name = "small_d110_field"
    sp = wl.spec(name)
    d = torch.as_tensor(wl.initial_delta(name, sp)).cuda()
    a = torch.as_tensor(wl.initial_A(name, sp)).cuda()
    g = qs.Grain(sp, "fp64")
    sets = [np.linspace(0.05, 0.45, n) for n in (5, 90)]
    want = [g.ldos(d, a, en, 0.03, 3) for en in sets]
    g.close()
    g = qs.Grain(sp, "fp64")
    g.ldos(d, a, sets[0], 0.03, 0)  # the buffers that every call shares
    torch.cuda.synchronize()
    gate = threading.Barrier(2)
    bad = []

    def work(i):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(20):
                    gate.wait(30)
                    if not torch.equal(g.ldos(d, a, sets[i], 0.03, 3), want[i]):
                        bad.append(i)
        except Exception as e:
            bad.append(e)
            gate.abort()

    ts = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join(60)
    assert not bad, bad
    g.close()
