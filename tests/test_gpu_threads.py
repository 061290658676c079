"""Contexts of several threads, each on a stream of its own: while some capture
graphs, others lay out batches, read, restore and start walks; every call works
and the walks are those of a context alone."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _work(libpsl, torch, stream, graph, rounds, out, i):
    try:
        with libpsl.Context(0, stream=stream) as c:
            states = []
            for r in range(rounds):
                ids = c.init_walks(1021, 1, 3) + c.init_walks(300, 2, 4 + r)
                c.step_batch(ids, 9, graph=graph)
                c.apply_flip(ids[0], 7)
                ck = c.checkpoint(ids[0])
                c.restore(ids[0], ck)
                c.set_option(libpsl.OPT_EVAL_ITEMS, -1)      # drops the layouts
                c.step_batch(ids, 8, graph=graph)
                c.eval_neighbourhood(ids[0], r, 1021)
                states.append([c.read_walk(w) for w in ids])
                c.free_walks(ids)
            out[i] = states
    except Exception as e:                                   # noqa: BLE001 (reported by the test)
        out[i] = e


def test_layouts_and_reads_beside_captures():
    import torch
    from paper_2107_09801_amd import libpsl
    rounds, out = 20, {}
    _work(libpsl, torch, torch.cuda.Stream(), False, rounds, out, "alone")
    assert not isinstance(out["alone"], Exception), out["alone"]
    ts = [threading.Thread(target=_work, args=(libpsl, torch, torch.cuda.Stream(), g, rounds, out, i))
          for i, g in enumerate((True, False, True, False))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for i in range(4):
        assert not isinstance(out[i], Exception), out[i]
        for a, b in zip(out[i], out["alone"]):
            for x, y in zip(a, b):
                assert all(np.array_equal(x[k], y[k]) for k in ("pivot", "C", "best", "local_best"))
                assert x["t"] == y["t"] and x["value_local"] == y["value_local"]
