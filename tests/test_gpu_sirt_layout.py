"""GPU: SIRT's tile layouts where they can go wrong, against a plain NumPy
iteration on the built PILA: sizes around the 8 x 8 pixel tiles, the 64-ray
tiles and the 32 and 64 steps of a span, rays along the diagonal (two entries
at every step: a span's windows exactly full), along the rows (runs longer
than a window, both slopes), detectors narrower and wider than the image, a
support with holes, images and detectors of a single line, each length type;
and the summation straight from the rows (MI355X).

Each iteration adds a few hundred products per value in another order than
NumPy; 1e-12 of the largest value leaves them three orders of room."""
import numpy as np
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


def _flat(U):  # near-horizontal rays of both slopes, the axes and the diagonals first
    a = [90.0, 0.0, 45.0, 135.0, 89.2, 90.8, 89.9999, 90.0001, 87.0, 93.0, 86.5, 93.5, 80.0, 100.0]
    return np.array((a + list(np.linspace(1.0, 179.0, max(U, len(a)))))[:U])


def _mask(kind, N, rng):
    if kind == "full":
        return None
    if kind == "circle":
        return datagen.circle_mask(N)
    m = rng.integers(0, 2, (N, N)).astype(np.uint8)
    m[N // 3] = 0
    return m


def _reference(pl, U, K, sino, iters, lam, f0, dtype):
    def lengths(t):
        v = t.cpu().numpy()
        return (v.astype(np.float32) / np.float32(180.0)).astype(np.float64) if dtype == "u8" else v.astype(np.float64)

    ptr, col, ln = pl.row_ptr.cpu().numpy(), pl.col.cpu().numpy(), lengths(pl.len)
    pix, G, NP = np.repeat(np.arange(len(ptr) - 1), np.diff(ptr)), U * K, len(ptr) - 1
    W = np.bincount(col, weights=ln * ln, minlength=G)
    f, cost = f0.reshape(-1).copy(), []
    for _ in range(iters):
        res = sino.reshape(-1) - np.bincount(col, weights=ln * f[pix], minlength=G)
        cost.append(np.sqrt(np.sum(res * res) / G))
        y = np.where(W > 0, res / np.where(W > 0, W, 1.0), 0.0)
        f = f + (lam / U) * np.bincount(pix, weights=ln * y[col], minlength=NP)
    return f.reshape(f0.shape), np.array(cost)


@pytest.mark.parametrize("N,U,K,angles,mask", [
    (1, 3, 4, "flat", "full"), (5, 4, 1, "flat", "full"), (2, 14, 2, "flat", "full"), (7, 33, 10, "flat", "circle"),
    (31, 32, 44, "uniform", "full"), (33, 31, 47, "flat", "holes"), (64, 65, 91, "uniform", "full"),
    (65, 14, 93, "flat", "full"), (72, 64, 40, "uniform", "holes"), (70, 20, 200, "flat", "circle"),
    (130, 14, 185, "flat", "full")])
@pytest.mark.parametrize("dtype", ["f64", "f32", "u8"])
@pytest.mark.parametrize("rows", [False, True])
def test_layouts_match_the_rows(P, N, U, K, angles, mask, dtype, rows, monkeypatch):
    if rows and (dtype == "u8" or N > 65):
        pytest.skip("the walk of the rows is covered by the other sizes")
    print("sirt N=%d U=%d K=%d %s %s %s rows=%d" % (N, U, K, angles, mask, dtype, rows), flush=True)
    monkeypatch.setenv("PILA_SIRT_CSR", "1" if rows else "0")
    ang = _flat(U) if angles == "flat" else datagen.angles_deg(U)
    rng = np.random.default_rng(N + U)
    pl = P.pila_build(P.Geometry(N, ang, K, _mask(mask, N, rng), dtype))
    sino, f0 = rng.uniform(0.0, 1.0, (U, K)) * N, rng.uniform(0.0, 1.0, (N, N))
    want, cost = _reference(pl, U, K, sino, 3, 0.5, f0, dtype)
    img = torch.from_numpy(f0.copy()).cuda()
    got = P.sirt_run(pl, torch.from_numpy(sino).cuda(), 3, 0.5, img)
    assert np.max(np.abs(img.cpu().numpy() - want)) <= 1e-12 * max(1.0, np.max(np.abs(want)))
    assert np.max(np.abs(got - cost) / cost) <= 1e-12


def test_values_outside_the_rows_do_not_enter(P):
    """A NaN in the image reaches the rays through its pixel and no others."""
    N, U, K = 40, 30, 57
    mask = np.ones((N, N), np.uint8)
    pl = P.pila_build(P.Geometry(N, datagen.angles_deg(U) + 0.7, K, mask, "f64"))
    f0 = np.full((N, N), 0.25)
    f0[3, 5] = np.nan
    sino = torch.full((U, K), 1.0, dtype=torch.float64, device="cuda")
    img = torch.from_numpy(f0.copy()).cuda()
    P.sirt_run(pl, sino, 1, 0.5, img)
    ptr, col = pl.row_ptr.cpu().numpy(), pl.col.cpu().numpy()
    p = 3 * N + 5
    bad = np.zeros(U * K, bool)
    bad[col[ptr[p]:ptr[p + 1]]] = True
    touched = np.array([bad[col[ptr[q]:ptr[q + 1]]].any() for q in range(N * N)]).reshape(N, N)
    assert np.array_equal(np.isnan(img.cpu().numpy()), touched)
