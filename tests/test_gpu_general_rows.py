"""GPU: the general chain body where rows without entries meet others, against
the oracle: a detector narrower than the image and angles of one side, so that
the last half of the pixels are met by no ray (their rows begin at the end of
the entry arrays) and are scored beside pixels with rows of hundreds of
entries; the residual in global memory and in LDS (MI355X)."""
import numpy as np
import pytest

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


@pytest.mark.parametrize("U,M,proposal", [(1100, 33, "redraw"), (1100, 20, "clamp"), (1100, 64, "clamp"),
                                          (300, 33, "redraw")])
def test_rows_without_entries_beside_long_ones(P, U, M, proposal):
    N, K, steps = 64, 21, 400
    print("general body U=%d M=%d %s" % (U, M, proposal), flush=True)
    angles = np.linspace(0.0, 5.0, U)
    mask = np.zeros((N, N), np.uint8)
    mask[56:, 32:] = 1
    csr = oracle.pila(N, U, K, angles, mask)
    n = np.diff(csr[0])
    assert np.all(n[-16:] == 0) and n.max() > U  # the last rows begin at the arrays' end
    rng = np.random.default_rng(U + M)
    f0 = rng.uniform(0.2, 0.8, (N, N)) * mask
    sino = oracle.forward(N, U, K, csr, rng.uniform(0.0, 1.0, (N, N))).reshape(U, K)
    kw = dict(seed=5, chain_id=M, n_steps=steps, n_stages=10, m_cand=M, T0=1e-3, TN=1e-6, delta_max=0.2,
              proposal=proposal)
    prm = P.SatParams(**kw)
    pl = P.pila_build(P.Geometry(N, angles, K, mask, "f64"))
    img = torch.from_numpy(f0.copy()).cuda()
    ws = P.sat_workspace(pl.geom, prm, minimal=True)  # (no room for a split chain's copies)
    st, tr = P.sat_run(pl, torch.from_numpy(sino).cuda(), prm, img, workspace=ws, trace=True)
    assert st["body"] & 15 == P._binding.BODY_GENERAL
    assert bool(st["body"] & P._binding.BODY_GLOBAL_R) == (U * K * 8 > 163840)
    got = (img.cpu().numpy(), st, {k: v.cpu().numpy() for k, v in tr.items()})
    _compare_fp64(got, oracle.sat_run(N, U, K, csr, sino, f0, mask=mask, **kw))
