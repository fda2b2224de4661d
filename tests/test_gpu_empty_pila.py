"""GPU: a support that no ray meets (a detector narrower than the gap to a
corner): the PILA has support pixels and not one entry, so every entry point
leaves the image as it is and the costs are those of the empty projections.
The entry arrays are one element long, as a C caller may allocate them, and
hold an index far outside the PILA, which nothing may use (MI355X)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

FAR = 1 << 29


@pytest.fixture(scope="module")
def P():
    import paper_1411_4622_amd as P
    P.load()
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return P


def _empty_pila(P, dtype, U=3):
    """N = 9, three bins, two support pixels in opposite corners off every ray."""
    N, K = 9, 3
    mask = np.zeros((N, N), np.uint8)
    mask[0, 0] = mask[N - 1, N - 1] = 1
    pl = P.pila_build(P.Geometry(N, np.linspace(100.0, 170.0, U), K, mask, dtype))
    assert pl.nnz == 0 and pl.n_support == 2
    ldt = {"f64": torch.float64, "f32": torch.float32, "u8": torch.uint8}[dtype]
    keep = [torch.full((1,), FAR, dtype=torch.int32, device="cuda") for _ in range(2)]
    keep += [torch.ones(1, dtype=ldt, device="cuda") for _ in range(2)]
    pl.c.col, pl.c.t_col, pl.c.len, pl.c.t_len = (t.data_ptr() for t in keep)
    return pl, keep


@pytest.mark.parametrize("dtype", ["f64", "f32", "u8"])
@pytest.mark.parametrize("max_row", [0, 64, 65, 300])
def test_sequential_sirt_without_entries(P, dtype, max_row):
    print("seq without entries, %s, max_row %d" % (dtype, max_row), flush=True)
    pl, keep = _empty_pila(P, dtype)
    pl.c.max_row = max_row  # each form of the kernel
    U, K, N = pl.geom.n_angles, pl.geom.n_bins, pl.geom.n
    sino = torch.rand(U, K, dtype=torch.float64, device="cuda")
    f0 = torch.rand(N, N, dtype=torch.float64, device="cuda")
    img = f0.clone()
    cost = P.sirt_seq_run(pl, sino, 3, 70, 1.0, img, seed=2)
    assert torch.equal(img, f0)
    want = float(torch.sqrt((sino ** 2).sum() / (U * K)))
    assert np.all(np.abs(cost - want) <= 1e-14 * want)


@pytest.mark.parametrize("dtype", ["f64", "f32", "u8"])
def test_projections_and_sirt_without_entries(P, dtype):
    print("projections without entries, %s" % dtype, flush=True)
    pl, keep = _empty_pila(P, dtype)
    U, K, N = pl.geom.n_angles, pl.geom.n_bins, pl.geom.n
    sino = torch.rand(U, K, dtype=torch.float64, device="cuda")
    f0 = torch.rand(N, N, dtype=torch.float64, device="cuda")
    assert not P.pila_forward(pl, f0).any() and not P.pila_backproject(pl, sino).any()
    img = f0.clone()
    cost = P.sirt_run(pl, sino, 2, 1.0, img)
    assert torch.equal(img, f0)
    want = float(torch.sqrt((sino ** 2).sum() / (U * K)))
    assert np.all(np.abs(cost - want) <= 1e-14 * want)
