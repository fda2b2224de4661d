"""GPU: the PILA build's count, fill and support kernels at the sizes and
angles where they can go wrong, against the oracle's ray traces (MI355X).

Lengths: the oracle traces in extended precision, the kernels evaluate the
chord in FP64 from an offset known to 2^-70; both then round a value of at
most sqrt 2 once or twice, and near an axis the ramp's slope 1 / (hi lo)
multiplies the rounding of cos and sin, which both take as given: 1e-12 holds
with room (FP32: half an ulp, 6e-8, on top)."""
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


def _mask(kind, N, rng):
    if kind == "full":
        return None
    if kind == "circle":
        return datagen.circle_mask(N)
    m = np.zeros((N, N), np.uint8)
    if kind == "gaps":      # rows with holes, empty rows, values other than 1
        m[:] = rng.integers(0, 2, (N, N)) * rng.integers(1, 256, (N, N))
        m[:: 3] = 0
    elif kind == "corner":  # a single pixel in the first and the last place
        m[0, 0] = m[N - 1, N - 1] = 1
    return m


ANGLES = {
    "uniform": lambda U: datagen.angles_deg(U),
    # rays nearly along the rows and columns, both slopes, and the diagonals
    "steep": lambda U: np.array([0.0, 1e-7, -1e-7, 1e-3, 89.999999, 90.0, 90.000001, 179.99, 45.0, 135.0, -45.0,
                                 44.999999, 46.0, 134.0, 181.0, 269.9999][:U]),
}


@pytest.mark.parametrize("N,U,K,angles,mask,dtype", [
    (1, 3, 2, "uniform", "full", "f64"),        # one pixel
    (3, 16, 7, "steep", "gaps", "f64"),
    (31, 16, 47, "steep", "gaps", "f64"),       # one word of mask bits, not full
    (33, 16, 46, "steep", "corner", "f32"),     # two words
    (63, 65, 90, "uniform", "circle", "f32"),   # one angle beyond a wavefront
    (64, 64, 91, "uniform", "full", "f64"),     # whole wavefronts; diagonal rays through the corners
    (65, 16, 93, "steep", "full", "f64"),       # a step beyond a wavefront; runs longer than one
    (130, 16, 20, "steep", "gaps", "f64"),      # a detector narrower than the image
    (130, 3, 400, "uniform", "circle", "f64"),  # and wider
    (257, 37, 364, "uniform", "gaps", "f32"),   # a row beyond a scan chunk
    (8, 16, 4, "steep", "full", "f64"),         # one chunk of pixels and one of rays, both full
    (9, 5, 13, "uniform", "gaps", "f32"),       # a ray beyond a chunk
])
def test_build_matches_the_oracle(P, N, U, K, angles, mask, dtype):
    print("build N=%d U=%d K=%d %s %s %s" % (N, U, K, angles, mask, dtype), flush=True)
    ang = np.asarray(ANGLES[angles](U), dtype=np.float64)
    m = _mask(mask, N, np.random.default_rng(N))
    pl = P.pila_build(P.Geometry(N, ang, K, m, dtype))
    (rp, col, ln), (off, pix, rl) = oracle.pila(N, len(ang), K, ang, m, with_rays=True)
    assert pl.nnz == len(col)
    assert np.array_equal(pl.row_ptr.cpu().numpy(), rp)
    assert np.array_equal(pl.col.cpu().numpy(), col)
    assert np.array_equal(pl.t_row_ptr.cpu().numpy(), off)
    rid = np.repeat(np.arange(len(off) - 1), np.diff(off))
    order = np.lexsort((pix, rid))
    assert np.array_equal(pl.t_col.cpu().numpy(), pix[order])
    tol = 1e-12 if dtype == "f64" else 1e-12 + 6e-8 * np.sqrt(2.0)
    lg, tg = pl.len.cpu().numpy(), pl.t_len.cpu().numpy()
    assert np.max(np.abs(lg - ln), initial=0.0) <= tol
    assert np.max(np.abs(tg - rl[order]), initial=0.0) <= tol
    # both copies hold the same bits: pixel-major entries re-ordered by (ray, pixel)
    p_of = np.repeat(np.arange(N * N), np.diff(rp))
    assert np.array_equal(lg[np.lexsort((p_of, col))], tg)
    sup = np.flatnonzero(np.ones(N * N) if m is None else m.reshape(-1))
    assert np.array_equal(pl.support.cpu().numpy(), sup)
    assert pl.max_row == int(np.max(np.diff(rp)))


def test_empty_support_and_mismatched_sizes(P):
    """An all-zero mask gives an empty PILA; a second phase whose csr does not
    match the offsets or the mask is refused and writes no entry from them."""
    import ctypes as C
    from paper_1411_4622_amd import _binding as B
    N, U, K = 9, 5, 13
    pl = P.pila_build(P.Geometry(N, datagen.angles_deg(U), K, np.zeros((N, N), np.uint8), "f64"))
    assert pl.nnz == 0 and pl.n_support == 0 and pl.max_row == 0 and (pl.k_lo, pl.k_hi) == (0, -1)
    assert not pl.row_ptr.any() and not pl.t_row_ptr.any()
    geom = P.Geometry(N, datagen.angles_deg(U), K, None, "f64")
    pl = P.pila_build(geom)
    scratch = torch.empty(N * N + 256, dtype=torch.uint8, device="cuda")
    ends = torch.zeros_like(pl.t_row_ptr)
    for field, value in (("nnz", pl.nnz - 1), ("n_support", pl.n_support - 1), ("t_row_ptr", ends.data_ptr())):
        csr = B.CCsr.from_buffer_copy(pl.c)
        setattr(csr, field, value)
        pl.len.fill_(-1.0)
        pl.t_len.fill_(-1.0)
        torch.cuda.synchronize()
        rc = B.load().pila_build(C.byref(geom.c), C.byref(csr), scratch.data_ptr(), scratch.numel(), None)
        torch.cuda.synchronize()
        assert rc == -4, (field, rc)
        assert bool((pl.t_len == -1.0).all())
        assert field == "t_row_ptr" or bool((pl.len == -1.0).all())
