"""GPU: a chain's first residual, formed by the whole GPU before the chain
starts, at its edges: ray counts around the 64 of a tile, rays without an
entry, rows around the 128 entries of one round of loads, alone (residual in
LDS and in global memory) and in one batch of mixed precisions, length types
and proposals (MI355X).

A chain of one step leaves the sum of squares of A f - Pm for its final image
f.  The projection kernel's own product is the reference.  FP64: 1e-12
relative (both add the same products).  FP32: a residual is rounded once when
it is formed and once when the step changes it, so the sum of squares is
within 4 roundings of 2^-24 relative per term; the bound is four times that."""
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


# N, U, K, lengths, precision, M, proposal
SHAPES = [(16, 4, 16, "f64", "f64", 2, "clamp"), (40, 7, 90, "f64", "f64", 3, "redraw"),
          (64, 3, 91, "f64", "f64", 1, "clamp"), (30, 260, 172, "f64", "f64", 2, "redraw"),
          (100, 5, 13, "f32", "f32", 4, "clamp"), (130, 1, 63, "f32", "f32", 8, "redraw"),
          (40, 300, 181, "f32", "f32", 4, "clamp"), (16, 5, 13, "u8", "f32", 4, "clamp"),
          (40, 300, 181, "u8", "f32", 2, "clamp"), (20, 9, 29, "u8", "f64", 2, "redraw")]


def _job(P, N, U, K, dtype, precision, M, proposal):
    ell = datagen.random_ellipses(N + U, N, 6)
    sl = datagen.make_slice(N, U, K, ell, masked=True, I0=1e4, noise_seed=U)
    pl = P.pila_build(P.Geometry(N, sl.angles, K, sl.mask, dtype))
    prm = P.SatParams(n_steps=1, seed=K, chain_id=M, n_stages=1, m_cand=M, T0=1e-2, TN=1e-5, delta_max=0.2,
                      precision=precision, proposal=proposal)
    return P.Job(pl, torch.from_numpy(sl.sino).cuda(), torch.from_numpy(sl.f0.copy()).cuda(), prm)


def _check(P, job, st):
    r = P.pila_forward(job.pila, job.image) - job.sino
    want = float((r * r).sum())
    tol = 1e-12 if job.params.precision == "f64" else 16 * 2.0 ** -24
    assert abs(st["sse_final"] - want) <= tol * want, (st["sse_final"], want)


@pytest.mark.parametrize("shape", SHAPES)
def test_first_residual_alone(P, shape):
    print("first residual", shape, flush=True)
    job = _job(P, *shape)
    st, _ = P.sat_run(job.pila, job.sino, job.params, job.image)
    _check(P, job, st)


def test_first_residuals_of_a_mixed_batch(P):
    jobs = [_job(P, *s) for s in SHAPES]
    print("first residuals of a batch of", len(jobs), flush=True)
    for job, st in zip(jobs, P.sat_run_batch(jobs, waves_per_chain=4, chains_per_cu=2)):
        _check(P, job, st)
