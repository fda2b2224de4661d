"""GPU: the choice among estimates whose sums are infinite or NaN, step by step:
rays measured as infinite, against the oracle; rays measured as NaN, against the
first least of each step's sums that is not NaN (the oracle keeps a first sum that
is; nothing is accepted, so the sums are those of the start); and changes
whose square overflows beside ones whose does not (finite totals, which move);
numbers of estimates on either side of the 16 lanes of the first minimum, in FP64
and FP32, on the pipelined and the general body (MI355X)."""
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


def _both(P, sl, sino, f0, prec, **kw):
    pl = P.pila_build(P.Geometry(sl.N, sl.angles, sl.K, sl.mask, prec))
    img = torch.from_numpy(f0.copy()).cuda()
    st, tr = P.sat_run(pl, torch.from_numpy(sino).cuda(), P.SatParams(precision=prec, **kw), img, trace=True)
    csr = oracle.pila(sl.N, sl.U, sl.K, sl.angles, sl.mask)
    if prec == "f32":
        csr = (csr[0], csr[1], csr[2].astype(np.float32).astype(np.float64))
    f_o, st_o, tr_o = oracle.sat_run(sl.N, sl.U, sl.K, csr, sino, f0, mask=sl.mask, precision=prec, **kw)
    tr = {k: v.cpu().numpy() for k, v in tr.items()}
    first = np.flatnonzero((tr["m_star"] != tr_o["m_star"]) | (tr["accept"] != tr_o["accept"]))
    assert not len(first), "step %d: estimate %d accept %d, oracle %d %d" % (
        first[0], tr["m_star"][first[0]], tr["accept"][first[0]], tr_o["m_star"][first[0]], tr_o["accept"][first[0]])
    assert st["accepts"] == st_o["accepts"]
    return img.cpu().numpy(), f_o, tr, st


def _slice():
    return datagen.make_slice(20, 12, 29, datagen.random_ellipses(5, 20, 6), masked=True, I0=1e4, noise_seed=6)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("M", [3, 16, 17, 40])
@pytest.mark.parametrize("value", [np.inf, -np.inf])
def test_infinite_rays(P, prec, M, value):
    print("%s M=%d %r" % (prec, M, value), flush=True)
    sl = _slice()
    sino = sl.sino.copy()
    sino[3, 14] = sino[7, 12] = value
    f, f_o, tr, st = _both(P, sl, sino, sl.f0, prec, seed=4, chain_id=0, n_steps=300, n_stages=10, m_cand=M, T0=1e-2,
                           TN=1e-5, delta_max=0.2)
    assert np.array_equal(f, f_o)
    assert len(np.unique(tr["m_star"])) > 1


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("M", [3, 16, 17, 40])
def test_nan_rays(P, prec, M):
    print("%s M=%d nan" % (prec, M), flush=True)
    sl, steps, delta = _slice(), 200, 0.2
    sino = sl.sino.copy()
    sino[3, 10:18] = np.nan
    csr = oracle.pila(sl.N, sl.U, sl.K, sl.angles, sl.mask)
    if prec == "f32":
        csr = (csr[0], csr[1], csr[2].astype(np.float32).astype(np.float64))
    r = (oracle.forward(sl.N, sl.U, sl.K, csr, sl.f0).reshape(-1) - sino.reshape(-1))
    support, f0 = np.flatnonzero(sl.mask.reshape(-1)), sl.f0.reshape(-1)
    want, left_out = [], 0
    for s in range(steps):
        sums = []
        for m in range(M):
            w = [int(x) for x in oracle.philox((4, 0), (s, m, 0, 0))]
            p = int(support[(w[0] * len(support)) >> 64])
            fn = min(max(f0[p] + delta * (2.0 * ((w[1] >> 11) * 2.0**-53) - 1.0), 0.0), 1.0)
            S = oracle.delta_sse(csr, r, p, fn - f0[p], prec == "f32")
            sums.append(S if prec == "f32" else S[0])
        finite = [x for x in sums if x == x]
        want.append(sums.index(min(finite)) if finite else 0)
        left_out += len(finite) < M
    assert left_out > steps // 4
    pl = P.pila_build(P.Geometry(sl.N, sl.angles, sl.K, sl.mask, prec))
    img = torch.from_numpy(sl.f0.copy()).cuda()
    st, tr = P.sat_run(pl, torch.from_numpy(sino).cuda(),
                       P.SatParams(n_steps=steps, seed=4, m_cand=M, T0=1e-2, TN=1e-5, delta_max=delta, precision=prec),
                       img, trace=True)
    assert st["accepts"] == 0 and not tr["accept"].any() and np.array_equal(img.cpu().numpy(), sl.f0)
    assert np.array_equal(tr["m_star"].cpu().numpy(), want)


# changes up to 1.5 times the one whose square overflows, so that a third do
@pytest.mark.parametrize("prec,delta", [("f64", 2e154), ("f32", 2.7e19)])
@pytest.mark.parametrize("M,proposal", [(3, "clamp"), (17, "clamp"), (40, "clamp"), (4, "redraw")])
def test_changes_whose_square_overflows(P, prec, delta, M, proposal):
    print("%s M=%d %s" % (prec, M, proposal), flush=True)
    sl = _slice()
    f, f_o, tr, st = _both(P, sl, sl.sino, np.zeros((20, 20)), prec, seed=4, chain_id=0, n_steps=40, n_stages=10,
                           m_cand=M, T0=delta, TN=delta / 10, delta_max=delta, f_min=-2 * delta, f_max=2 * delta,
                           proposal=proposal)
    assert np.max(np.abs(f - f_o)) <= 1e-9 * delta
    assert tr["accept"].any()
