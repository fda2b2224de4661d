"""Chains of more than 2^30 stages take the general body, whose schedule takes any
number of them (its stages are stepped on the CPU in test_chain_schedule.py): the
rule on the CPU, the route on the GPU."""
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


@pytest.mark.parametrize("stages,want", [(1, True), (1 << 30, True), ((1 << 30) + 1, False), (2**31 - 1, False)])
def test_stages_of_the_other_bodies(P, stages, want):
    allowed = P.load()._ZN4pila13ahead_allowedEPK10sat_params
    allowed.restype = C.c_bool
    assert allowed(C.byref(P.SatParams(n_steps=1000, n_stages=stages, T0=1e-2, TN=1e-5).c())) is want


@pytest.mark.gpu
@pytest.mark.parametrize("M,U", [(3, 12), (32, 900)])
def test_a_chain_of_many_stages(P, M, U):
    """One step (a step passes its stages one by one, so that more would take minutes)."""
    import torch

    import datagen
    import oracle
    N, K, stages = 20, 29, 2**31 - 1
    print("M=%d U=%d, %d stages" % (M, U, stages), flush=True)
    sl = datagen.make_slice(N, U, K, datagen.random_ellipses(4, N, 6), masked=True, I0=1e4, noise_seed=5)
    kw = dict(n_steps=1, seed=3, n_stages=stages, m_cand=M, T0=3e-3, TN=1e-5, delta_max=0.3)
    pl = P.pila_build(P.Geometry(N, sl.angles, K, sl.mask, "f64"))
    img = torch.from_numpy(sl.f0.copy()).cuda()
    st, tr = P.sat_run(pl, torch.from_numpy(sl.sino).cuda(), P.SatParams(**kw), img, trace=True)
    assert st["body"] & 15 == P._binding.BODY_GENERAL
    f, st_o, tr_o = oracle.sat_run(N, U, K, oracle.pila(N, U, K, sl.angles, sl.mask), sl.sino, sl.f0, mask=sl.mask, **kw)
    assert np.array_equal(tr["m_star"].cpu().numpy(), tr_o["m_star"])
    assert np.array_equal(tr["accept"].cpu().numpy(), tr_o["accept"])
    assert np.max(np.abs(img.cpu().numpy() - f)) <= 1e-9
