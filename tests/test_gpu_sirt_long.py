"""GPU: SIRT where a wavefront walks far through a tile's lengths: bands of ray
steps that cross spans of the layout from any step on (rays of either slope,
flat ones among them), and a tile whose lengths take more than 4 GiB (8 x 8
pixels under 7.2 million angles, FP64); one iteration against the projections
and the factors formed from the PILA's entries (MI355X).

A pixel's update adds n terms, of both sides in another order, so it agrees to n
roundings of their absolute sum."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    import paper_1411_4622_amd as P
    P.load()
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    return P


def _one_iteration(P, pl, lam):
    """sirt_run's image and cost against one formed from the projections."""
    N, U, K = pl.geom.n, pl.geom.n_angles, pl.geom.n_bins
    ln = pl.len.double()
    W = torch.zeros(U * K, dtype=torch.float64, device="cuda")
    W.index_add_(0, pl.col, ln * ln)
    gen = torch.Generator(device="cuda").manual_seed(3)
    sino = torch.rand(U, K, dtype=torch.float64, device="cuda", generator=gen) * N
    f0 = torch.rand(N, N, dtype=torch.float64, device="cuda", generator=gen)
    res = sino - P.pila_forward(pl, f0)
    y = torch.where(W.view(U, K) > 0, res / W.view(U, K).clamp_min(1e-300), 0.0)
    want = f0 + (lam / U) * P.pila_backproject(pl, y)
    # a ray's residual is off by its own roundings, W's and the quotient's
    rows = float((pl.t_row_ptr[1:] - pl.t_row_ptr[:-1]).max())
    part = torch.where(W.view(U, K) > 0, (sino + P.pila_forward(pl, f0)) / W.view(U, K).clamp_min(1e-300), 0.0)
    cost = float(torch.sqrt((res * res).sum() / (U * K)))
    n = float((pl.row_ptr[1:] - pl.row_ptr[:-1]).max())
    bound = 2.2e-16 * ((lam / U) * P.pila_backproject(pl, (n + 4) * y.abs() + 2 * (rows + 4) * part) + f0.abs())
    img = f0.clone()
    got = P.sirt_run(pl, sino, 1, lam, img)
    assert bool(((img - want).abs() <= bound).all())
    assert abs(got[0] - cost) <= 2.2e-16 * (U * K + 2 * rows) * cost


@pytest.mark.parametrize("N,U,K", [(300, 900, 424), (260, 500, 300)])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("lo,hi", [(0.0, 90.0), (90.0, 180.0), (91.0, 95.0)])
def test_bands_across_spans(P, N, U, K, dtype, lo, hi):
    print("sirt N=%d U=%d %s %g..%g" % (N, U, dtype, lo, hi), flush=True)
    _one_iteration(P, P.pila_build(P.Geometry(N, np.linspace(lo, hi, U) + 0.1, K, None, dtype)), 0.6)


def test_lengths_of_a_tile_beyond_4_gib(P):
    N, U, K, lam = 8, 7_200_000, 9, 0.7
    if torch.cuda.mem_get_info()[0] < 120e9:
        pytest.skip("needs 120 GB of device memory")
    pl = P.pila_build(P.Geometry(N, (np.arange(U) + 0.5) * (180.0 / U), K, None, "f64"))
    print("built %d entries" % pl.nnz, flush=True)
    assert pl.nnz * 8 > 1 << 32
    _one_iteration(P, pl, lam)
