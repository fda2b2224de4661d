// SIRT with exact lengths, pixel by pixel (section III-D as the paper
// describes it: a pixel is chosen, Eq. 11 gives its change from its PILA row
// and the factor matrix, Eq. 10 applies it, and the pixel's rays get the new
// calculated projections through the PILA before the next pixel is chosen).
//
// The updates form one sequence, each reading the projections the previous
// one wrote, so one wavefront runs it: per update, the lanes take the
// pixel's row entries, the row sum is added in the canonical 64-partial
// order, lane 0 updates the pixel, the lanes scatter the change to the
// row's rays (distinct rays: no atomics).  The calculated projections live
// in LDS when they fit, else in global memory.  Pixels are drawn by the same
// Philox4x64-10 as the annealing chain (key (seed, 0), counter (update, 0,
// 3, 0)), uniform over the support.
//
// Only the projections (and the pixel's value) tie an update to the one
// before.  Everything else is fetched ahead, so that no memory latency is
// left in the sequence: the draws and row offsets of 64 updates at a time
// (one a lane) a block ahead, a row's entries three updates ahead, its rays'
// factors and measurements and the pixel's value two, the factors'
// reciprocals one.  What remains is an LDS read, the quotient (by the
// reciprocal, exact: see below), the 64-lane sum and an LDS write.
// 64 x 64, 60 angles, FP64, 6456 updates: 14.2 -> 4.4 ms (2.2 -> 0.69 us per
// update, about 200 instructions of one wavefront and 700 clocks of waits).
#include <algorithm>
#include <cmath>
#include <vector>

#include "sat_chain.hpp"
#include "sat_host.hpp"

namespace pila {
namespace {

struct SeqArgs {
    int32_t U, K, P, n_iter;
    int64_t m_per;
    int64_t n_pixels;
    double lambda;
    uint64_t seed;
    const int64_t* row_ptr;
    const int32_t* col;
    const void* len;
    const int32_t* support;
    const double* sino;
    double* W;     // factor matrix (U*K)
    double* pc;    // calculated projections (U*K)
    double* f;     // image (N*N)
    double* cost;  // Eq. 4 after each iteration (n_iter)
};

// Factor matrix W_g = sum of l^2 over the ray's support pixels and the
// projections Pc_g = sum of f_p l, each ray summed in ascending pixel order
// (one thread per ray; products and sums rounded separately).
template <typename LenT>
__global__ __launch_bounds__(256) void seq_setup_kernel(int64_t G, const int64_t* __restrict__ rp,
                                                        const int32_t* __restrict__ ci,
                                                        const LenT* __restrict__ ln, const double* __restrict__ f,
                                                        double* __restrict__ W, double* __restrict__ pc)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < G; g += stride) {
        double w = 0.0, s = 0.0;
        for (int64_t q = rp[g]; q < rp[g + 1]; ++q) {
            const double l = (double)ln[q];
            w = w + l * l;
            s = s + f[ci[q]] * l;
        }
        W[g] = w;
        pc[g] = s;
    }
}

// x / w from inv = 1 / w correctly rounded: two corrections of the quotient
// by its exact (fused) residual, the second from a quotient within an ulp,
// give the correctly rounded quotient (Markstein, IBM J. Res. Dev. 34, 1990)
// wherever nothing on the way under- or overflows; other operands divide.
__device__ __forceinline__ double quotient(double x, double w, double inv)
{
    const double ax = fabs(x);
    if (ax > 0x1p-900 && ax < 0x1p900 && w > 0x1p-100 && w < 0x1p100) {
        double q = x * inv;
        q = fma(fma(-q, w, x), inv, q);
        return fma(fma(-q, w, x), inv, q);
    }
    return x / w;
}

template <int E>
struct SeqRow {  // one update: its pixel, and per lane up to E entries of its row
    int64_t b, n;
    int32_t p;
    int32_t g[E];
    double l[E], w[E], s[E], inv[E];
    double fo;
};

// The wavefront's LDS writes before its LDS reads after this point (one
// wavefront's LDS operations complete in order; this orders the compiler)
__device__ __forceinline__ void wave_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <typename LenT, bool PCLDS, int E>
__global__ __launch_bounds__(64) void sirt_seq_kernel(SeqArgs A)
{
    extern __shared__ __align__(16) char lds[];
    const int lane = threadIdx.x;
    const int64_t G = (int64_t)A.U * A.K;
    double* pc = PCLDS ? (double*)lds : A.pc;
    if (PCLDS) {
        for (int64_t g = lane; g < G; g += kWave) pc[g] = A.pc[g];
        __syncthreads();
    }
    const LenT* len = (const LenT*)A.len;
    const double scale = A.lambda / (double)A.U;
    const int64_t total = (int64_t)A.n_iter * A.m_per;

    // draws of updates base .. base + 63, one a lane
    struct Draws {
        int64_t base, b, n;
        int32_t p;
    };
    auto fill = [&](Draws& D, int64_t base) {
        D.base = base;
        D.p = 0;
        D.b = D.n = 0;
        if (base + lane < total) {
            const Words4 w = philox4x64(A.seed, 0, (uint64_t)(base + lane), 0, 3, 0);
            D.p = A.support[__umul64hi(w.w0, (uint64_t)A.P)];
            D.b = A.row_ptr[D.p];
            D.n = A.row_ptr[D.p + 1] - D.b;
        }
    };
    Draws cur, nxt;
    cur.base = nxt.base = -1;
    // the row of update t: its entries (past the row: the array's first)
    auto fetch_row = [&](SeqRow<E>& R, int64_t t) {
        R.p = 0;
        R.b = R.n = 0;
        if (t < total) {
            const int64_t base = t & ~(int64_t)(kWave - 1);
            const int j = (int)(t - base);
            if (cur.base != base) {
                if (nxt.base == base)
                    cur = nxt;
                else
                    fill(cur, base);
            }
            if (j == kWave / 2 && base + kWave < total) fill(nxt, base + kWave);
            R.p = __builtin_amdgcn_readlane(cur.p, j);
            R.b = readlane_i64(cur.b, j);
            R.n = readlane_i64(cur.n, j);
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int64_t q = lane + e * kWave;
            const int64_t at = q < R.n ? R.b + q : 0;
            R.g[e] = A.col[at];
            R.l[e] = (double)len[at];
        }
    };
    auto fetch_rays = [&](SeqRow<E>& R) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            R.w[e] = A.W[R.g[e]];
            R.s[e] = A.sino[R.g[e]];
        }
        R.fo = A.f[R.p];
    };
    auto reciprocals = [&](SeqRow<E>& R) {
#pragma unroll
        for (int e = 0; e < E; ++e) R.inv[e] = 1.0 / R.w[e];
    };

    // the pixels of the last two updates and their values, which an earlier
    // fetch of f cannot hold
    int32_t p1 = -1, p2 = -1;
    double f1 = 0.0, f2 = 0.0;
    int64_t left = A.m_per;  // updates to the end of the iteration
    int32_t it = 0;
    // update t: X its row, complete; Y, Z, V the rows of t + 1, t + 2, t + 3
    auto step = [&](SeqRow<E>& X, SeqRow<E>& Y, SeqRow<E>& Z, SeqRow<E>& V, int64_t t)
                    __attribute__((always_inline)) {
        double c[E];
#pragma unroll
        for (int e = 0; e < E; ++e) c[e] = pc[X.g[e]];
        fetch_row(V, t + 3);
        fetch_rays(Z);
        double part = 0.0;
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (lane + e * kWave < X.n && X.w[e] > 0.0)
                part = part + quotient(X.l[e] * (X.s[e] - c[e]), X.w[e], X.inv[e]);
        for (int64_t q = X.b + E * kWave + lane; q < X.b + X.n; q += kWave) {  // beyond the registers
            const int32_t g = A.col[q];
            const double wg = A.W[g];
            if (wg > 0.0) part = part + ((double)len[q] * (A.sino[g] - pc[g])) / wg;
        }
        const double df = scale * wave_canon_sum(part);
#pragma unroll
        for (int e = 0; e < E; ++e)
            if (lane + e * kWave < X.n) pc[X.g[e]] = c[e] + df * X.l[e];
        for (int64_t q = X.b + E * kWave + lane; q < X.b + X.n; q += kWave) {
            const int32_t g = A.col[q];
            pc[g] = pc[g] + df * (double)len[q];
        }
        if (PCLDS)
            wave_order();
        else
            __syncthreads();  // this update's projections before the next reads them
        const double fo = X.p == p1 ? f1 : (X.p == p2 ? f2 : X.fo);
        p2 = p1;
        f2 = f1;
        p1 = X.p;
        f1 = fo + df;
        if (lane == 0) A.f[X.p] = f1;
        reciprocals(Y);
        if (--left == 0) {
            left = A.m_per;
            if (A.cost) {
                double sq = 0.0;
#pragma unroll 8
                for (int64_t g = lane; g < G; g += kWave) {
                    const double d = pc[g] - A.sino[g];
                    sq = sq + d * d;
                }
                sq = wave_canon_sum(sq);
                if (lane == 0) A.cost[it] = sqrt(sq / ((double)A.K * (double)A.U));
            }
            ++it;
        }
    };
    // Every iteration has the cost of the start: there are no updates, or the
    // PILA has no entries (no ray meets the support), so that none would
    // change anything; the steps' loads, which read entry 0 in the place of
    // those that a row does not have, would find no entry there.
    if (total == 0 || A.row_ptr[A.n_pixels] == 0) {
        if (A.cost) {
            double sq = 0.0;
            for (int64_t g = lane; g < G; g += kWave) {
                const double d = pc[g] - A.sino[g];
                sq = sq + d * d;
            }
            sq = wave_canon_sum(sq);
            for (int32_t n = lane; n < A.n_iter; n += kWave) A.cost[n] = sqrt(sq / ((double)A.K * (double)A.U));
        }
        return;
    }
    SeqRow<E> R0, R1, R2, R3;
    fetch_row(R0, 0);
    fetch_row(R1, 1);
    fetch_row(R2, 2);
    fetch_rays(R0);
    fetch_rays(R1);
    reciprocals(R0);
    for (int64_t t = 0; t < total;) {
        step(R0, R1, R2, R3, t);
        if (++t >= total) break;
        step(R1, R2, R3, R0, t);
        if (++t >= total) break;
        step(R2, R3, R0, R1, t);
        if (++t >= total) break;
        step(R3, R0, R1, R2, t);
        ++t;
    }
}

template <typename LenT, int E>
int32_t launch_seq(const SeqArgs& A, int64_t lds_bytes, hipStream_t st)
{
    if (lds_bytes > 0) {
        const void* k = (const void*)sirt_seq_kernel<LenT, true, E>;
        PILA_TRY(set_lds(k, (int)lds_bytes));
        SeqArgs args = A;
        void* argv[] = {&args};
        PILA_HIP(hipLaunchKernel(k, dim3(1), dim3(kWave), argv, (size_t)lds_bytes, st));
    } else {
        sirt_seq_kernel<LenT, false, E><<<1, kWave, 0, st>>>(A);
    }
    return PILA_OK;
}

size_t seq_bytes(const pila_geom* g, int32_t n_iter)
{
    const size_t G = (size_t)g->n_angles * g->n_bins;
    return 2 * align256(8 * G) + align256(8 * (size_t)(n_iter > 0 ? n_iter : 1));
}

template <typename LenT>
int32_t seq_impl(const pila_geom* geom, const pila_csr* csr, const double* d_sino, const sirt_seq_params* prm,
                 double* d_image, char* ws, double* h_cost, hipStream_t st)
{
    const int64_t G = (int64_t)geom->n_angles * geom->n_bins;
    SeqArgs A;
    A.U = geom->n_angles;
    A.K = geom->n_bins;
    A.P = csr->n_support;
    A.n_iter = prm->n_iter;
    A.m_per = prm->m_per;
    A.n_pixels = (int64_t)geom->n * geom->n;
    A.lambda = prm->lambda;
    A.seed = prm->seed;
    A.row_ptr = csr->row_ptr;
    A.col = csr->col;
    A.len = csr->len;
    A.support = csr->support;
    A.sino = d_sino;
    A.W = (double*)ws;
    A.pc = (double*)(ws + align256(8 * (size_t)G));
    A.f = d_image;
    A.cost = (double*)(ws + 2 * align256(8 * (size_t)G));
    if (G > 0)
        seq_setup_kernel<LenT><<<(unsigned)std::min<int64_t>((G + 255) / 256, 4096), 256, 0, st>>>(
            G, csr->t_row_ptr, csr->t_col, (const LenT*)csr->t_len, d_image, A.W, A.pc);
    PILA_HIP(hipGetLastError());
    hipDeviceProp_t prop;
    PILA_TRY(device_props(&prop));
    const int64_t budget = (int64_t)prop.sharedMemPerBlock - 1024;
    if (prm->n_iter > 0 && A.P > 0) {
        // entries per lane in registers: the smallest that holds the longest
        // row (rows beyond 256 entries read the rest in place)
        const int64_t lds = G * 8 <= budget ? G * 8 : 0;
        if (csr->max_row <= kWave)
            PILA_TRY((launch_seq<LenT, 1>(A, lds, st)));
        else if (csr->max_row <= 2 * kWave)
            PILA_TRY((launch_seq<LenT, 2>(A, lds, st)));
        else
            PILA_TRY((launch_seq<LenT, 4>(A, lds, st)));
    }
    PILA_HIP(hipGetLastError());
    if (h_cost && prm->n_iter > 0) {
        PILA_HIP(hipMemcpyAsync(h_cost, A.cost, sizeof(double) * (size_t)prm->n_iter, hipMemcpyDeviceToHost, st));
        PILA_HIP(hipStreamSynchronize(st));
    }
    return PILA_OK;
}

}  // namespace
}  // namespace pila

using namespace pila;

extern "C" int32_t sirt_seq_workspace_size(const pila_geom* geom, const sirt_seq_params* params, size_t* bytes)
{
    clear_error();
    PILA_TRY(check_geom(geom));
    if (!params || !bytes) return fail(PILA_EINVAL, "params or bytes is NULL");
    if (params->n_iter < 0 || params->m_per < 0) return fail(PILA_EINVAL, "n_iter and m_per must be >= 0");
    *bytes = seq_bytes(geom, params->n_iter);
    return PILA_OK;
}

extern "C" int32_t sirt_seq_run(const pila_geom* geom, const pila_csr* csr, const double* d_sino,
                                const sirt_seq_params* params, double* d_image, void* d_ws, size_t ws_bytes,
                                double* h_cost, void* stream)
{
    clear_error();
    PILA_TRY(check_geom(geom));
    if (!csr || !params || !d_sino || !d_image) return fail(PILA_EINVAL, "csr, params, sinogram or image is NULL");
    if (!csr->row_ptr || !csr->col || !csr->len || !csr->support || !csr->t_row_ptr || !csr->t_col || !csr->t_len)
        return fail(PILA_EINVAL, "PILA arrays (pixel-major, ray-major and support) are required");
    if (params->n_iter < 0 || params->m_per < 0) return fail(PILA_EINVAL, "n_iter and m_per must be >= 0");
    if (!std::isfinite(params->lambda)) return fail(PILA_EINVAL, "lambda is not finite");
    if (params->m_per > 0 && csr->n_support < 1) return fail(PILA_EINVAL, "empty support");
    const size_t need = seq_bytes(geom, params->n_iter);
    if (!d_ws || ws_bytes < need)
        return fail(PILA_ENOMEM, "workspace of %zu bytes is below the %zu needed", ws_bytes, need);
    hipStream_t st = (hipStream_t)stream;
    if (geom->len_dtype == PILA_F64)
        return seq_impl<double>(geom, csr, d_sino, params, d_image, (char*)d_ws, h_cost, st);
    if (geom->len_dtype == PILA_F32)
        return seq_impl<float>(geom, csr, d_sino, params, d_image, (char*)d_ws, h_cost, st);
    return seq_impl<LenQ>(geom, csr, d_sino, params, d_image, (char*)d_ws, h_cost, st);
}
