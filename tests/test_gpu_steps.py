"""GPU: the step loop's bookkeeping at its edges, against the oracle: step
counts around the 64 steps that a trace or a block of draws holds, stages that
do not divide the steps or outnumber them, and estimate counts on either side
of the 16 lanes that the first minimum is taken over (MI355X).

Decisions are compared one by one; Delta C within 1e-12 of its own scale, as
for every FP64 chain here (the GPU adds a row's terms in another order)."""
import numpy as np
import pytest

import datagen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    import paper_1411_4622_amd as P
    P.load()
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return P


def _slice(N, U, K, seed):
    ell = datagen.random_ellipses(seed, N, 6)
    return datagen.make_slice(N, U, K, ell, masked=True, I0=1e4, noise_seed=seed + 1)


@pytest.mark.parametrize("steps,stages,M,U", [
    (1, 1, 1, 12), (63, 7, 2, 12), (64, 64, 16, 12), (65, 100, 17, 12), (129, 1000, 3, 12), (700, 33, 16, 90),
    (700, 701, 17, 90), (321, 5, 64, 40), (200, 13, 4, 300), (130, 130, 8, 420)])
def test_trace_and_schedule_edges(P, steps, stages, M, U):
    N, K = 20, 29
    print("steps=%d stages=%d M=%d U=%d" % (steps, stages, M, U), flush=True)
    sl = _slice(N, U, K, seed=steps)
    prm = P.SatParams(n_steps=steps, seed=9, chain_id=M, n_stages=stages, m_cand=M, T0=2e-2, TN=1e-5, delta_max=0.2)
    img = torch.from_numpy(sl.f0.copy()).cuda()
    pl = P.pila_build(P.Geometry(N, sl.angles, K, sl.mask, "f64"))
    st, tr = P.sat_run(pl, torch.from_numpy(sl.sino).cuda(), prm, img, trace=True)
    csr = oracle.pila(N, U, K, sl.angles, sl.mask)
    f_o, st_o, tr_o = oracle.sat_run(N, U, K, csr, sl.sino, sl.f0, mask=sl.mask, seed=9, chain_id=M, n_steps=steps,
                                     n_stages=stages, m_cand=M, T0=2e-2, TN=1e-5, delta_max=0.2)
    assert np.array_equal(tr["m_star"].cpu().numpy(), tr_o["m_star"])
    assert np.array_equal(tr["accept"].cpu().numpy(), tr_o["accept"])
    err = np.abs(tr["dC"].cpu().numpy() - tr_o["dC"])
    assert np.all(err <= 1e-12 * (np.abs(tr_o["dC"]) + tr_o["scale"]) + 1e-300)
    assert np.max(np.abs(img.cpu().numpy() - f_o)) <= 1e-9
    assert st["accepts"] == st_o["accepts"] and st["accepts_nonzero"] == st_o["accepts_nonzero"]


@pytest.mark.parametrize("resync,M", [(1, 4), (37, 4), (50, 20)])
def test_trace_across_resync_segments(P, resync, M):
    """An FP32 chain that stops for a resync every few steps, with and without
    a trace and on the smallest workspace: the same image, and a trace that
    holds every step."""
    N, U, K, steps = 48, 300, 69, 400
    sl = _slice(N, U, K, seed=resync)
    prm = P.SatParams(n_steps=steps, seed=3, chain_id=1, n_stages=21, m_cand=M, T0=None, q_auto=20, precision="f32",
                      delta_max=0.1, resync_every=resync)
    pl = P.pila_build(P.Geometry(N, sl.angles, K, sl.mask, "f32"))
    sino = torch.from_numpy(sl.sino).cuda()
    images = []
    for trace, minimal in ((True, False), (False, False), (True, True)):
        img = torch.from_numpy(sl.f0.copy()).cuda()
        ws = P.sat_workspace(pl.geom, prm, minimal=minimal)
        st, tr = P.sat_run(pl, sino, prm, img, workspace=ws, trace=trace)
        images.append(img)
        assert st["resyncs"] == st["accepts_nonzero"] // resync
        if trace:
            acc, m, dC = (tr[k].cpu().numpy() for k in ("accept", "m_star", "dC"))
            assert set(np.unique(acc)) <= {0, 1} and int(acc.sum()) == st["accepts"]
            assert m.min() >= 0 and m.max() < M and len(np.unique(m)) > 1
            assert np.all(np.isfinite(dC)) and np.all(acc[dC <= 0] == 1)
    assert torch.equal(images[0], images[1]) and torch.equal(images[0], images[2])


def test_non_finite_sums_are_never_chosen_over_finite_ones(P):
    """Rays measured as infinite or NaN make every sum over them infinite or
    NaN; the oracle's rules (a NaN never wins, Delta C of an infinite total)
    hold step by step."""
    N, U, K, steps = 20, 12, 29, 200
    sl = _slice(N, U, K, seed=5)
    for value in (np.nan, np.inf):
        sino = sl.sino.copy()
        sino[3, 14] = value
        prm = P.SatParams(n_steps=steps, seed=4, chain_id=0, n_stages=10, m_cand=4, T0=1e-2, TN=1e-5, delta_max=0.2)
        img = torch.from_numpy(sl.f0.copy()).cuda()
        pl = P.pila_build(P.Geometry(N, sl.angles, K, sl.mask, "f64"))
        st, tr = P.sat_run(pl, torch.from_numpy(sino).cuda(), prm, img, trace=True)
        acc, dC = tr["accept"].cpu().numpy(), tr["dC"].cpu().numpy()
        # the total is not finite: no Delta C is, so Step 4 accepts nothing but what it calls downhill
        assert np.array_equal(acc == 1, dC <= 0.0), value
        assert int(acc.sum()) == st["accepts"]
