"""Control words of many contexts at once: more than the 64 that have a slot of
pinned memory, the rest reading theirs without one, and slots handed on when
contexts end, from several threads. Identical boxes give identical results,
and a refused list is reported by its own context only.
"""
import threading

import numpy as np
import pytest

from paper_2406_04210_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ljmd():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2406_04210_amd import ljmd as L
    return L


def box(ljmd, w, n, **kw):
    s = ljmd.System(n, w.box, w.params, precision=1, **kw)
    s.set_state(w.x, w.v, w.species)
    return s


@pytest.mark.parametrize("count", [1, 64, 70])
def test_many_contexts(ljmd, count):
    n = 300
    w = W.thermostat_fluid(n, seed_index=3)
    systems = [box(ljmd, w, n) for _ in range(count)]
    for s in systems:
        s.run(2, observe=False)
    got = [s.observables() for s in systems]
    assert all(g == got[0] for g in got)
    del systems[::2]
    again = box(ljmd, w, n)
    again.run(2, observe=False)
    assert again.observables() == got[0]
    with pytest.raises(ljmd.LJMDError):
        bad = box(ljmd, w, n, nbr_capacity=16)
        bad.sync()
    for s in systems:
        s.run(1, observe=False)
        s.sync()


def test_contexts_of_several_threads(ljmd):
    n = 300
    w = W.thermostat_fluid(n, seed_index=3)
    out = [None] * 8

    def work(k):
        r = []
        for _ in range(4):
            s = box(ljmd, w, n)
            s.run(2, observe=False)
            r.append(s.observables())
        out[k] = r

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(out))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert all(g == out[0][0] for r in out for g in r)
