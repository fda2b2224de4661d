"""GPU: the lone FP32 chains of several estimates a wavefront that form their slot
words at each step (a workspace without room for them): the image, the counts and
the decisions of the same chain on a full workspace, for step counts around a
block of draws (MI355X)."""
import pytest

import datagen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    import paper_1411_4622_amd as P
    P.load()
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return P


@pytest.mark.parametrize("N,U,M,cpw", [(256, 180, 9, 2), (256, 180, 16, 2), (512, 60, 17, 4), (512, 60, 32, 4)])
@pytest.mark.parametrize("steps,resync", [(1, 0), (33, 0), (1500, 0), (1500, 200)])
def test_as_on_a_full_workspace(P, N, U, M, cpw, steps, resync):
    print("no slot words N=%d U=%d M=%d %d steps" % (N, U, M, steps), flush=True)
    K = datagen.n_bins_for(N)
    sl = datagen.make_slice(N, U, K, datagen.random_ellipses(N + U, N, 6), masked=True, I0=1e4, noise_seed=3)
    pl = P.pila_build(P.Geometry(N, sl.angles, K, sl.mask, "f32"))
    prm = P.SatParams(n_steps=steps, seed=5, chain_id=1, m_cand=M, n_stages=7, precision="f32", resync_every=resync,
                      T0=1e-3, TN=1e-6, delta_max=0.05)
    sino, out = torch.from_numpy(sl.sino).cuda(), []
    for minimal in (False, True):
        img = torch.from_numpy(sl.f0.copy()).cuda()
        st, tr = P.sat_run(pl, sino, prm, img, workspace=P.sat_workspace(pl.geom, prm, minimal=minimal), trace=True)
        assert st["body"] & 15 == P._binding.BODY_PIPED and (st["body"] >> 8) & 255 == cpw
        out.append((img, st["accepts"], st["sse_final"], tr))
    (a, b) = out
    assert torch.equal(a[0], b[0]) and a[1:3] == b[1:3]
    assert all(torch.equal(a[3][k], b[3][k]) for k in a[3])
