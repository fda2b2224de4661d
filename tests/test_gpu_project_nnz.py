"""GPU: the projections take the entries that the row offsets name, whatever
the descriptor's entry count says: a count left at zero or stale gives the
same values, and so do the rows of some of the angles alone, whose offsets do
not begin at zero; as do PILAs of fewer entries than one load (MI355X)."""
import ctypes as C

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


@pytest.mark.parametrize("dtype", ["f64", "f32", "u8"])
@pytest.mark.parametrize("N,U,K", [(20, 12, 29), (60, 33, 87)])
def test_the_entry_count_is_not_read(P, N, U, K, dtype):
    print("projections N=%d U=%d %s" % (N, U, dtype), flush=True)
    pl = P.pila_build(P.Geometry(N, datagen.angles_deg(U) + 0.3, K, datagen.circle_mask(N), dtype))
    f = torch.rand(N, N, dtype=torch.float64, device="cuda")
    y = torch.rand(U, K, dtype=torch.float64, device="cuda")
    fwd, back = P.pila_forward(pl, f), P.pila_backproject(pl, y)
    nnz = pl.nnz
    for count in (0, 1, 5, nnz // 2, nnz - 1, nnz + 100):
        pl.c.nnz = count
        assert torch.equal(P.pila_forward(pl, f), fwd), count
        assert torch.equal(P.pila_backproject(pl, y), back), count


def test_rows_of_some_angles(P):
    """Rays of angles u0 .. u1 - 1 alone, by a pointer into the offsets."""
    N, U, K, u0, u1 = 33, 20, 47, 7, 13
    pl = P.pila_build(P.Geometry(N, datagen.angles_deg(U) + 0.3, K, None, "f64"))
    f = torch.rand(N, N, dtype=torch.float64, device="cuda")
    want = P.pila_forward(pl, f)[u0:u1]
    part = P.Geometry(N, datagen.angles_deg(U)[u0:u1] + 0.3, K, None, "f64")
    csr = type(pl.c).from_buffer_copy(pl.c)
    csr.t_row_ptr = pl.t_row_ptr.data_ptr() + 8 * u0 * K
    csr.nnz = int(pl.t_row_ptr[u1 * K] - pl.t_row_ptr[u0 * K])
    out = torch.zeros(u1 - u0, K, dtype=torch.float64, device="cuda")
    rc = P.load().pila_forward(C.byref(part.c), C.byref(csr), f.data_ptr(), out.data_ptr(),
                               torch.cuda.current_stream().cuda_stream)
    assert rc == 0 and torch.equal(out, want)


@pytest.mark.parametrize("N,U,K", [(1, 1, 1), (1, 2, 1), (1, 3, 1), (1, 4, 1), (2, 1, 1), (400, 1, 2)])
def test_fewer_entries_than_a_load(P, N, U, K):
    """Each row of a PILA of 1 to 5 entries against its own sum (400: one
    pixel of 160000, more rows than the grid's wavefronts take at once)."""
    mask = np.zeros((N, N), np.uint8) if N > 2 else None
    if N > 2:
        mask[N // 2, N // 2] = 1
    pl = P.pila_build(P.Geometry(N, datagen.angles_deg(U) + 0.3, K, mask, "f64"))
    print("projections of %d entries" % pl.nnz, flush=True)
    f, y = np.random.default_rng(U).uniform(0.1, 1.0, N * N), np.random.default_rng(N).uniform(0.1, 1.0, U * K)
    for out, ptr, idx, ln, x in (
            (P.pila_forward(pl, torch.from_numpy(f.reshape(N, N)).cuda()), pl.t_row_ptr, pl.t_col, pl.t_len, f),
            (P.pila_backproject(pl, torch.from_numpy(y.reshape(U, K)).cuda()), pl.row_ptr, pl.col, pl.len, y)):
        p, i, v = ptr.cpu().numpy(), idx.cpu().numpy(), ln.cpu().numpy()
        want = [float(np.sum(v[p[r]:p[r + 1]] * x[i[p[r]:p[r + 1]]])) for r in range(len(p) - 1)]
        assert np.max(np.abs(out.cpu().numpy().reshape(-1) - want)) <= 1e-15 * 8
