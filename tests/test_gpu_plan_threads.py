"""Batches of one plan made by several threads at once: the plan's tables for the
matrix-core kernels, which the first of them builds, are built once."""
import threading

import pytest

pytestmark = pytest.mark.gpu


def test_batches_made_by_several_threads():
    import gc

    import paper_1303_4945_amd as sht
    lmax, n = 700, 6
    g = sht.Geometry.gauss(lmax + 1, 2 * lmax + 1)
    grown = []
    for together in (False, True):
        p = sht.Plan(g, lmax)   # one transform: vector kernels, no two-step table yet
        gc.collect()
        before = sht.memory_stats()
        made, gate = [], threading.Barrier(n if together else 1)

        def make():
            gate.wait()
            made.append(sht.Batch([p]))

        if together:
            ts = [threading.Thread(target=make) for _ in range(n)]
            for t in ts:
                t.start()
            for t in ts:
                t.join()
        else:
            for _ in range(n):
                make()
        assert len(made) == n
        after = sht.memory_stats()
        grown.append((after[0] - before[0], after[1] - before[1]))
        made.clear()
        del p
    assert grown[0] == grown[1]
