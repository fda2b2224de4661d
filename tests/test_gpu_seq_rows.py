"""GPU: pixel-sequential SIRT where its look-ahead can go wrong, against the
oracle: rows of up to 64, 128 and 256 entries and beyond (held in registers,
the rest read in place), projections in LDS and in global memory, a support
of one or two pixels (every update reads what the one or two before it
wrote), and update counts around the 64 that a block of draws holds (MI355X).

The GPU adds a row's terms in another order than the oracle; 1e-10 of the
values is some 1e5 roundings, far above what a few hundred updates of
contracting steps can gather."""
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


@pytest.mark.parametrize("N,U,K,support,iters,m_per", [
    (9, 3, 13, "circle", 2, 1),       # fewer updates than the look-ahead
    (9, 40, 13, "circle", 3, 63),     # rows of up to 64 entries
    (12, 60, 17, "circle", 2, 65),    # ... 128
    (12, 150, 17, "circle", 5, 64),   # ... 256
    (12, 300, 17, "circle", 2, 130),  # longer
    (48, 420, 68, "circle", 1, 200),  # longer, projections in global memory
    (40, 620, 57, "one", 2, 70),      # the same pixel again and again, in global memory
    (12, 60, 17, "one", 2, 70),
    (12, 60, 17, "two", 3, 100),
])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_rows_blocks_and_repeats(P, N, U, K, support, iters, m_per, dtype):
    print("seq N=%d U=%d %s %d x %d %s" % (N, U, support, iters, m_per, dtype), flush=True)
    sl = datagen.make_slice(N, U, K, datagen.random_ellipses(N + U, N, 5), masked=True, I0=1e4, noise_seed=3)
    mask = sl.mask.copy()
    if support != "circle":
        mask[:] = 0
        mask[N // 2, N // 2] = 1
        if support == "two":
            mask[N // 2, N // 2 + 1] = 1
    f0 = np.where(mask != 0, 0.3, 0.0)
    csr = oracle.pila(N, U, K, sl.angles, mask)
    if dtype == "f32":
        csr = (csr[0], csr[1], csr[2].astype(np.float32).astype(np.float64))
    f_o, c_o = oracle.sirt_seq_run(N, U, K, csr, sl.sino, f0, iters, m_per, 1.0, seed=11, mask=mask)
    pl = P.pila_build(P.Geometry(N, sl.angles, K, mask, dtype))
    img = torch.from_numpy(f0.copy()).cuda()
    cost = P.sirt_seq_run(pl, torch.from_numpy(sl.sino).cuda(), iters, m_per, 1.0, img, seed=11)
    tol = 1e-10 if dtype == "f64" else 1e-8  # FP32: the two sides may round a length's last bit apart
    assert np.max(np.abs(img.cpu().numpy() - f_o)) <= tol * max(1.0, np.max(np.abs(f_o)))
    assert np.max(np.abs(cost - c_o) / c_o) <= tol
