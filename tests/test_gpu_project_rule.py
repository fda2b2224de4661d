"""GPU: the projections on either side of each line of the rule for the rows a
wavefront takes at once (rows and how far they reach), against a plain NumPy
product with the built PILA (MI355X).

Both sides add the same products, only the order differs, so a row of n terms
agrees to n roundings of its absolute sum."""
import numpy as np
import pytest

import datagen
from test_gpu_project_rows import _check

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    import paper_1411_4622_amd as P
    P.load()
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return P


# rays U K reaching across N, pixels N N reaching across U
@pytest.mark.parametrize("N,U,K", [
    (128, 3, 180), (129, 3, 180), (130, 1, 1023), (130, 1, 1024), (130, 8, 1024), (150, 1, 8191), (150, 4, 8192 // 4),
    (140, 91, 360), (140, 92, 360), (2047, 1, 2500), (2048, 1, 2047), (2048, 1, 2048),
    (31, 128, 5), (31, 129, 5), (32, 129, 5), (90, 200, 9), (91, 200, 9), (45, 2047, 9), (46, 2048, 9), (3, 5000, 5)])
@pytest.mark.parametrize("dtype", ["f64", "u8"])
def test_both_sides_of_the_rule(P, N, U, K, dtype):
    print("projections N=%d U=%d K=%d %s" % (N, U, K, dtype), flush=True)
    pl = P.pila_build(P.Geometry(N, datagen.angles_deg(U) + 0.3, K, datagen.circle_mask(N), dtype))
    rng = np.random.default_rng(N + U)
    f, y = rng.standard_normal(N * N), rng.standard_normal(U * K)

    def lengths(t):
        v = t.cpu().numpy()
        return (v.astype(np.float32) / np.float32(180.0)).astype(np.float64) if dtype == "u8" else v.astype(np.float64)

    out = P.pila_forward(pl, torch.from_numpy(f.reshape(N, N)).cuda()).cpu().numpy().reshape(-1)
    _check(out, pl.t_row_ptr.cpu().numpy(), pl.t_col.cpu().numpy(), lengths(pl.t_len), f)
    out = P.pila_backproject(pl, torch.from_numpy(y.reshape(U, K)).cuda()).cpu().numpy().reshape(-1)
    _check(out, pl.row_ptr.cpu().numpy(), pl.col.cpu().numpy(), lengths(pl.len), y)
