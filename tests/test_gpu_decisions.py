"""GPU: Step 4 beside its threshold at the ends of FP32's range, against the
oracle: one-step chains whose temperature puts -dC / T within 1e-5 to 1e-3 of
ln N1 on either side, for sums of squares below FP32's normal numbers, changes
whose dC is, and ordinary ones (MI355X)."""
import numpy as np
import pytest

import datagen
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N, U, K = 20, 12, 29


@pytest.fixture(scope="module")
def P():
    import paper_1411_4622_amd as P
    P.load()
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return P


# measured value of every ray, largest change, least ln N1
@pytest.mark.parametrize("value,delta,least", [
    (3e-20, 1e-14, -40.0),   # the total is below FP32's normal numbers, the change is not
    (1e-19, 3e-14, -40.0),
    (1e-19, 1e-11, -40.0),
    (3e14, 1e-40, -8e-4),    # dC is (and T not far above them, so ln N1 has to be small)
    (3e14, 1e-39, -8e-3),
    (3e11, 1e-34, -40.0),
    (1e-3, 1e-3, -40.0), (1.0, 0.1, -40.0), (1e-9, 1e-9, -40.0)])
def test_one_step_beside_the_threshold(P, value, delta, least):
    angles = datagen.angles_deg(U)
    csr = oracle.pila(N, U, K, angles)
    sino, f0 = np.full((U, K), -value), np.zeros((N, N))
    pl = P.pila_build(P.Geometry(N, angles, K, None, "f64"))
    d_sino = torch.from_numpy(sino).cuda()
    tried = flipped = 0
    for seed in range(40000):
        n1 = float(oracle.philox((seed, 0), (0, 0, 1, 0))[0] >> np.uint64(11)) * 2.0**-53
        ln = float(np.log(n1))
        if ln < least:
            continue
        kw = dict(seed=seed, chain_id=0, n_steps=1, n_stages=1, m_cand=1, delta_max=delta, f_min=-1.0, f_max=1.0)
        dC = float(oracle.sat_run(N, U, K, csr, sino, f0, T0=1.0, TN=1.0, **kw)[2]["dC"][0])
        if dC <= 0.0:
            continue
        tried += 1
        for off in (1e-5, 3e-5, 1e-4, 1e-3):
            got = []
            for T in (-dC / ln * (1.0 - off), -dC / ln * (1.0 + off)):
                want = oracle.sat_run(N, U, K, csr, sino, f0, T0=T, TN=T, **kw)[2]["accept"][0]
                img = torch.from_numpy(f0.copy()).cuda()
                tr = P.sat_run(pl, d_sino, P.SatParams(T0=T, TN=T, **kw), img, trace=True)[1]
                got.append(int(tr["accept"][0]))
                assert got[-1] == want, "seed %d, T %.17g: dC / T = %.9g ln N1" % (seed, T, -dC / T / ln)
            flipped += got == [0, 1]
        if tried == 6:
            break
    assert tried == 6 and flipped == 24
