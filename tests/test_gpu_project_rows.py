"""GPU: the projections' 8-rows-at-a-time gather at its edges, against a plain
NumPy product with the built PILA: row counts around 8 and the 8 XCD chunks,
rows that are empty or shorter than a load, a PILA of fewer entries than one
load, each length type, and entries whose last ones end the arrays (MI355X).

Both sides add the same products (one byte and FP32 lengths widened the same
way); only the order differs, so a row of n terms agrees to n roundings of
its absolute sum."""
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


def _check(got, ptr, idx, ln, x):
    rows = np.repeat(np.arange(len(ptr) - 1), np.diff(ptr))
    terms = ln * x[idx]
    want = np.bincount(rows, weights=terms, minlength=len(ptr) - 1)
    size = np.bincount(rows, weights=np.abs(terms), minlength=len(ptr) - 1)
    n = np.diff(ptr)
    assert np.all(np.abs(got - want) <= 2.2e-16 * (n + 2) * size)
    assert np.all(got[n == 0] == 0.0)


@pytest.mark.parametrize("N,U,K,mask", [(1, 1, 1, "full"), (2, 1, 2, "one"), (3, 2, 9, "full"), (8, 1, 5, "full"),
                                        (9, 3, 13, "one"), (13, 4, 40, "circle"), (16, 7, 23, "full"),
                                        (33, 90, 47, "circle"), (65, 33, 20, "circle"), (100, 50, 143, "circle")])
@pytest.mark.parametrize("dtype", ["f64", "f32", "u8"])
def test_projections_match_the_product(P, N, U, K, mask, dtype):
    print("project N=%d U=%d K=%d %s %s" % (N, U, K, mask, dtype), flush=True)
    m = None
    if mask == "circle":
        m = datagen.circle_mask(N)
    elif mask == "one":
        m = np.zeros((N, N), np.uint8)
        m[N // 2, N // 2] = 1
    pl = P.pila_build(P.Geometry(N, datagen.angles_deg(U) + 0.3, K, m, dtype))
    rng = np.random.default_rng(N + U)
    f, y = rng.standard_normal(N * N), rng.standard_normal(U * K)

    def lengths(t):
        v = t.cpu().numpy()
        return (v.astype(np.float32) / np.float32(180.0)).astype(np.float64) if dtype == "u8" else v.astype(np.float64)

    out = P.pila_forward(pl, torch.from_numpy(f.reshape(N, N)).cuda()).cpu().numpy().reshape(-1)
    _check(out, pl.t_row_ptr.cpu().numpy(), pl.t_col.cpu().numpy(), lengths(pl.t_len), f)
    out = P.pila_backproject(pl, torch.from_numpy(y.reshape(U, K)).cuda()).cpu().numpy().reshape(-1)
    _check(out, pl.row_ptr.cpu().numpy(), pl.col.cpu().numpy(), lengths(pl.len), y)
