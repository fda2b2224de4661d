"""Which chains the bodies that draw a block of steps ahead take: those whose
blocks, of 16 steps at the least, can be numbered in 32 bits, the two blocks
ahead of the last step among them.  The rule on the CPU, its use on the GPU."""
import ctypes as C

import numpy as np
import pytest


@pytest.fixture(scope="module")
def P():
    import os
    import paper_1411_4622_amd as P
    if not os.path.exists(P.LIB_PATH):
        from paper_1411_4622_amd import build
        build.build()
    P.load()
    return P


@pytest.mark.parametrize("steps,proposal,want", [(0, "clamp", True), (10**9, "clamp", True), (1 << 34, "clamp", True),
                                                 ((1 << 34) + 1, "clamp", False), (1 << 40, "clamp", False),
                                                 (1000, "redraw", False)])
def test_steps_drawn_ahead(P, steps, proposal, want):
    allowed = P.load()._ZN4pila13ahead_allowedEPK10sat_params
    allowed.restype = C.c_bool
    prm = P.SatParams(n_steps=steps, T0=1e-2, TN=1e-5, proposal=proposal).c()
    assert allowed(C.byref(prm)) is want
    assert not want or (steps + 2 * 64) // 16 < 1 << 31


@pytest.mark.gpu
def test_longer_chains_take_the_general_queue(P):
    """Served, and cancelled as soon as they run (a ticket's low bits name its queue)."""
    import time

    import torch
    import datagen
    N, U, K = 24, 30, 35
    sl = datagen.make_slice(N, U, K, datagen.random_ellipses(4, N, 6), masked=True, I0=1e4, noise_seed=5)
    geom = P.Geometry(N, sl.angles, K, sl.mask, "f32")
    sino = torch.from_numpy(sl.sino).cuda()
    with P.Server(mem_budget=1 << 30) as srv:
        for steps, queue in ((1 << 34, 0), ((1 << 34) + 1, 1), (1 << 40, 1)):
            img = torch.from_numpy(sl.f0.copy()).cuda()
            torch.cuda.synchronize()
            t = srv.submit(geom, sino, img, P.SatParams(n_steps=steps, seed=1, m_cand=4, T0=1e-2, TN=1e-5,
                                                        precision="f32", resync_every=4096))
            assert t & 3 == queue
            srv.cancel(t)
            t0, st = time.time(), None
            while st is None:
                assert time.time() - t0 < 60.0
                st = srv.poll(t)
                time.sleep(0.002)
            assert st["status"] == P._binding.PILA_ECANCELED and np.isfinite(st["sse_final"])
