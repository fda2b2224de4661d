"""GPU: the general chain body where its rows' 64 x 8 entries in flight begin and
end, for odd and even numbers of estimates a wavefront, against the oracle
(FP64 lengths) and against the same chain in a batch (one-byte and FP32 lengths),
the residual in LDS and in global memory (MI355X)."""
import numpy as np
import pytest

import datagen
import oracle
from test_gpu_sat import _compare_fp64

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    import paper_1411_4622_amd as P
    P.load()
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return P


def _slice(N, U, K):
    return datagen.make_slice(N, U, K, datagen.random_ellipses(N + U, N, 6), masked=True, I0=1e4, noise_seed=3)


# rows of up to about 1.4 U entries: below 64, around 512, above; 900 x 29 values are in global memory
@pytest.mark.parametrize("N,U,K", [(20, 12, 29), (20, 400, 29), (20, 500, 29), (20, 900, 29)])
@pytest.mark.parametrize("M", [1, 2, 16, 17, 33, 48])
def test_general_body_matches_oracle(P, N, U, K, M):
    print("general body U=%d M=%d" % (U, M), flush=True)
    sl = _slice(N, U, K)
    kw = dict(seed=5, chain_id=M, n_steps=150, n_stages=10, m_cand=M, T0=1e-3, TN=1e-6, delta_max=0.2, proposal="redraw")
    pl = P.pila_build(P.Geometry(N, sl.angles, K, sl.mask, "f64"))
    prm, img = P.SatParams(**kw), torch.from_numpy(sl.f0.copy()).cuda()
    ws = P.sat_workspace(pl.geom, prm, minimal=True)
    st, tr = P.sat_run(pl, torch.from_numpy(sl.sino).cuda(), prm, img, workspace=ws, trace=True)
    assert st["body"] & 15 == P._binding.BODY_GENERAL
    assert bool(st["body"] & P._binding.BODY_GLOBAL_R) == (U * K * 8 > 163840)
    csr = oracle.pila(N, U, K, sl.angles, sl.mask)
    want = oracle.sat_run(N, U, K, csr, sl.sino, sl.f0, mask=sl.mask, **kw)
    _compare_fp64((img.cpu().numpy(), st, {k: v.cpu().numpy() for k, v in tr.items()}), want)


@pytest.mark.parametrize("dtype,prec", [("f32", "f32"), ("u8", "f32"), ("u8", "f64")])
@pytest.mark.parametrize("U,resync", [(12, 0), (500, 40), (1500, 40)])
def test_batch_equals_alone(P, dtype, prec, U, resync):
    N, K, M = 20, 29, 20
    sl = _slice(N, U, K)
    prm = P.SatParams(n_steps=200, seed=2, m_cand=M, T0=1e-3, TN=1e-6, precision=prec, n_stages=9, proposal="redraw",
                      delta_max=0.1, resync_every=resync if prec == "f32" else 0)
    pl = P.pila_build(P.Geometry(N, sl.angles, K, sl.mask, dtype))
    sino = torch.from_numpy(sl.sino).cuda()
    a, b = torch.from_numpy(sl.f0.copy()).cuda(), torch.from_numpy(sl.f0.copy()).cuda()
    st, _ = P.sat_run(pl, sino, prm, a, workspace=P.sat_workspace(pl.geom, prm, minimal=True))  # (not split)
    (sb,) = P.sat_run_batch([P.Job(pl, sino, b, prm)])
    assert st["body"] & 15 == P._binding.BODY_GENERAL
    assert torch.equal(a, b) and st["accepts"] == sb["accepts"] and st["sse_final"] == sb["sse_final"]
    assert not np.array_equal(a.cpu().numpy(), sl.f0)
