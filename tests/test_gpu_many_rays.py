"""GPU: more workgroups than one dimension of a grid takes (2^32 threads): the
PILA of 80 million rays, whose ray-major copy has to hold what the pixel-major
one does, and SIRT's layouts of 17 million ray tiles (MI355X).

Both sums of a ray or a pixel have n terms in another order, so they agree to n
roundings of their absolute sum."""
import numpy as np
import pytest

from test_gpu_sirt_long import _one_iteration

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    import paper_1411_4622_amd as P
    P.load()
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    if torch.cuda.mem_get_info()[0] < 60e9:
        pytest.skip("needs 60 GB of device memory")
    return P


def test_pila_of_80_million_rays(P):
    N, U, K = 8, 6_700_000, 12
    pl = P.pila_build(P.Geometry(N, (np.arange(U) + 0.5) * (180.0 / U), K, None, "f32"))
    print("built %d entries" % pl.nnz, flush=True)
    assert U * K * 64 > 1 << 32  # a wavefront a ray
    f = torch.rand(N, N, dtype=torch.float64, device="cuda")
    got = P.pila_forward(pl, f).view(-1)  # from the ray-major copy
    want = torch.zeros(U * K, dtype=torch.float64, device="cuda")
    pixel = torch.arange(N * N, device="cuda").repeat_interleave(pl.row_ptr[1:] - pl.row_ptr[:-1])
    want.index_add_(0, pl.col, pl.len.double() * f.view(-1)[pixel])
    assert float(((got - want).abs() - 2.2e-16 * 2 * N * want).max()) <= 0.0


def test_sirt_of_17_million_ray_tiles(P):
    N, U, K = 2, 17_000_000, 2
    assert U * 256 > 1 << 32  # four wavefronts a tile
    _one_iteration(P, P.pila_build(P.Geometry(N, (np.arange(U) + 0.5) * (180.0 / U), K, None, "f32")), 0.7)
