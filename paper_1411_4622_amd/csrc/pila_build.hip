// PILA build on gfx950 (section II-B, Eq. 5).
//
// The paper runs Siddon's ray trace for one pixel at a time; here every
// (pixel, angle) and every (ray, image row or column) is independent work,
// evaluated with the closed-form chord.  A pixel's shadow at one angle is
// |c| + |s| <= sqrt 2 bins wide, so it meets at most the two bins next to
// its centre's projection q: floor(q) and floor(q) + 1.  A ray closer to the
// columns (|c| >= |s|) is (|c| + |s|) / |c| <= 2 pixels wide in an image
// row, so there it meets at most the two pixels next to its centre, and
// likewise in a column when it is closer to the rows.  (A pixel a whole
// pitch away is a corner touch, far below the 1e-9 that is kept, whatever
// the rounding of the centre.)
//
// Phase 1 counts, phase 2 writes.  Both are bound by FP64 arithmetic and by
// the writes: the count passes therefore decide on the centre distance alone
// (a dozen operations) and evaluate the length only where that distance is
// within 1e-8 of the shadow's edge, where the 1e-9 threshold and rounding
// could matter; the fill passes share one angle's constants over the pixels
// or the ray they belong to, divide by a precomputed reciprocal with exact
// corrections (the quotient IEEE division gives), and place a wavefront's
// entries by ballots.  Rows come out in ascending ray (pixel-major) or pixel
// (ray-major) order without sorting, and both copies call the same length
// function, so they hold bit-identical lengths.
//
// 1024 x 1024, 720 angles, FP32, circular support (7.6e8 entries, 12 GB
// written; 1.8 ms at the rate of a fill): 6.3 ms, of it counts 1.4, pixel fill
// 2.45, ray fill 2.4 ms.  Counting and filling by evaluating the full chord at
// four candidate bins per (pixel, angle), the rays by a lane per image row,
// and one-workgroup scans took 31.9 ms (4.1 + 6.2, 6.1, 11.5, 1.9 ms);
// 512 x 512 x 360: 4.91 -> 0.97 ms, 64 x 64 x 60: 228 -> 106 us.  The fills
// without their stores take 1.5 ms each (FP64 arithmetic, 1.1 ms of issue).
// Collecting a row's entries in LDS and storing whole cache lines was
// measured (2.2 and 2.6 ms; slower at 512 x 512) and not kept.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "common.hpp"
#include "sat_host.hpp"

namespace pila {

namespace {

constexpr int kWavesPerBlock = 4;
// Rows per count block and scan chunk: one wavefront's, so that the 16
// wavefronts of a count block share a row's angles or steps 16 ways and small
// geometries have a block for more compute units.  Whole builds with 256 and
// with 64: 64 x 64, 60 angles 125 and 114 us; 128 x 128, 90 angles 153 and 140;
// 256 x 256, 180 angles 306 and 258; 512 x 512, 360 angles 1.01 and 0.97 ms.
constexpr int kScanChunk = 64;
constexpr double kEdgeBand = 1e-8;    // centre distances this close to the edge: evaluate the length

// The support as the kernels read it, uploaded by each phase: per image row a
// span word (first support column | last << 15 | gaps << 30; first above last
// where the row has none; N <= 2^15), the number of support pixels before it,
// and one bit per pixel for the rows with gaps.
constexpr uint32_t kSpanGaps = 1u << 30;

struct MaskView {
    const uint32_t* spans;   // NULL: every pixel is in the support
    const int32_t* before;
    const uint32_t* bits;
    int32_t words;  // 32-bit words per row of bits
};

__host__ __device__ __forceinline__ int span_first(uint32_t s) { return (int)(s & 0x7fffu); }
__host__ __device__ __forceinline__ int span_last(uint32_t s) { return (int)(s >> 15 & 0x7fffu); }

__device__ __forceinline__ uint32_t row_span(const MaskView& m, int i, int N)
{
    return m.spans ? m.spans[i] : (uint32_t)(N - 1) << 15;
}

// whether column j (any integer) of image row i, whose span is given, is in
// the support
__device__ __forceinline__ bool in_support(const MaskView& m, uint32_t span, int i, int j)
{
    if (j < span_first(span) || j > span_last(span)) return false;
    if (!(span & kSpanGaps)) return true;
    return (m.bits[(int64_t)i * m.words + (j >> 5)] >> (j & 31)) & 1u;
}

// ---------------------------------------------------------------------------
// intersection length of one ray with one pixel (closed form)
//
// The chord of the line  x c + y s = sk  through a unit square, as a function
// of the offset t of the line from the square's centre (xc, yc), is a
// trapezoid: 1 / max(|c|,|s|) for |t| <= (hi - lo)/2, falling linearly to 0
// at |t| = (hi + lo)/2, with hi/lo = max/min(|c|, |s|).  Near-axis rays make
// the ramp steep (slope 1 / (hi lo)), so t is needed to far below 1e-16.  The
// coordinates are half-integers of at most 16 bits; with c and s cut at 35
// fractional bits, sk - xc c_hi - yc s_hi is exact in FP64 (52 bits), so is
// E - 2 |t_hi|, and the rest, xc c_lo + yc s_lo, is below 2^-20 and rounds
// at 2^-73: a handful of operations where error-free products and sums of
// the whole values take some twenty.
// ---------------------------------------------------------------------------
struct AngleC {
    double c_hi, c_lo, s_hi, s_lo;  // cos and sin, cut at 35 fractional bits, and the rest
    double flat, edge, E, Ee;       // half-widths of the trapezoid; hi + lo as an exact pair
    double hl2, inv2, inv_hi;       // 2 hi lo, its reciprocal, 1 / hi
};

__device__ __forceinline__ double cut35(double x)
{
    constexpr double kBig = 196608.0;  // 1.5 x 2^17: an ulp of 2^-35
    return (x + kBig) - kBig;
}

__device__ __forceinline__ AngleC angle_consts(double c, double s)
{
    AngleC a;
    a.c_hi = cut35(c);
    a.c_lo = c - a.c_hi;
    a.s_hi = cut35(s);
    a.s_lo = s - a.s_hi;
    const double ac = fabs(c), as = fabs(s);
    const double hi = fmax(ac, as), lo = fmin(ac, as);
    a.flat = 0.5 * (hi - lo);
    a.edge = 0.5 * (hi + lo);
    a.E = hi + lo;
    a.Ee = lo - (a.E - hi);
    a.hl2 = 2.0 * (hi * lo);
    a.inv2 = 1.0 / a.hl2;
    a.inv_hi = 1.0 / hi;
    return a;
}

// u / d from inv = 1 / d correctly rounded: two corrections of the quotient
// by its exact (fused) residual; the second starts from a quotient within an
// ulp, which makes the result the correctly rounded one (Markstein, IBM J.
// Res. Dev. 34, 1990).  The operands here are far from under- and overflow.
__device__ __forceinline__ double quotient(double u, double d, double inv)
{
    double q = u * inv;
    q = fma(fma(-q, d, u), inv, q);
    return fma(fma(-q, d, u), inv, q);
}

// length of a ray that is not parallel to an axis at offset th + th_lo; false
// where it is not above the threshold
__device__ __forceinline__ bool chord_at(const AngleC& A, double th, double th_lo, double* l)
{
    const double t = fabs(th + th_lo);
    const double u2 = fma(-2.0, fabs(th), A.E) + fma(th < 0.0 ? 2.0 : -2.0, th_lo, A.Ee);
    const double ramp = quotient(u2, A.hl2, A.inv2);
    const bool top = t <= A.flat;
    *l = top ? A.inv_hi : ramp;
    return top || (t < A.edge && ramp > kTau);
}

__device__ __forceinline__ double offset_lo(const AngleC& A, double xc, double yc)
{
    return fma(-xc, A.c_lo, -(yc * A.s_lo));
}

__device__ __forceinline__ bool chord(const AngleC& A, double xc, double yc, double sk, double* l)
{
    return chord_at(A, fma(-yc, A.s_hi, fma(-xc, A.c_hi, sk)), offset_lo(A, xc, yc), l);
}

// Axis-parallel rays go to the pixel whose half-open interval [left, left + 1)
// or [bottom, bottom + 1) contains them, with length 1.
__device__ __forceinline__ bool axis_hit(double c, double s, double xc, double yc, double sk)
{
    const double at = s == 0.0 ? sk * c : sk * s, low = (s == 0.0 ? xc : yc) - 0.5;
    return at >= low && at < low + 1.0;
}

// any ray
__device__ __forceinline__ bool length_at(const AngleC& A, double c, double s, double xc, double yc, double sk,
                                          double* l)
{
    if (c == 0.0 || s == 0.0) {
        *l = 1.0;
        return axis_hit(c, s, xc, yc, sk);
    }
    return chord(A, xc, yc, sk, l);
}

// Ray (c, s, sk) in steps: image rows when it is closer to the columns
// (cols), else image columns.  At step x its centre is at a0 + x slope on the
// other axis, and it reaches w <= 1 to either side.
struct RayLine {
    double c, s, sk, a0, slope, w;
    int lo, hi;  // steps where it can meet the image
    bool cols;
};

__device__ __forceinline__ RayLine ray_line(int N, double c, double s, double sk, const AngleC& A)
{
    RayLine L;
    L.c = c;
    L.s = s;
    L.sk = sk;
    L.cols = fabs(c) >= fabs(s);
    const double hc = 0.5 * N - 0.5;
    // column j has its centre at x = j - hc, row i at y = hc - i
    const double inv = copysign(A.inv_hi, L.cols ? c : s);
    if (L.cols) {
        L.slope = s * inv;
        L.a0 = fma(fma(-hc, s, sk), inv, hc);
    } else {
        L.slope = c * inv;
        L.a0 = fma(-fma(hc, c, sk), inv, hc);
    }
    L.w = A.edge * A.inv_hi;
    double lo = 0.0, hi = (double)(N - 1);
    if (L.slope != 0.0) {
        // the steps at which the centre is within the image or two pixels of
        // it; 1 / slope = +-(hi / lo) = +-2 hi^2 / (2 hi lo)
        const double big = fmax(fabs(c), fabs(s));
        const double per = copysign(2.0 * (big * big) * A.inv2, L.slope);
        const double e1 = (-2.0 - L.a0) * per, e2 = ((double)N + 1.0 - L.a0) * per;
        lo = fmax(lo, floor(fmin(e1, e2)));
        hi = fmin(hi, ceil(fmax(e1, e2)));
    } else if (L.a0 < -2.0 || L.a0 > (double)N + 1.0) {
        hi = -1.0;
    }
    L.lo = 0;
    L.hi = -1;
    if (lo <= hi) {
        L.lo = (int)lo;
        L.hi = (int)hi;
    }
    return L;
}

// ---------------------------------------------------------------------------
// phase 1: counts, scanned within each block's 64 rows
// ---------------------------------------------------------------------------
constexpr int kCountThreads = 1024;
constexpr int kParts = kCountThreads / kScanChunk;

// entries of pixel (i, j) at the angles u0 .. u1 - 1: lane = pixel, all lanes
// at the same angle
__device__ int count_pixel(int i, int j, int N, int u0, int u1, int K, const double* __restrict__ trig)
{
    const double hc = 0.5 * N - 0.5, cK = 0.5 * (K - 1);
    const double xc = j - hc, yc = hc - i;
    int n = 0;
#pragma unroll 4
    for (int u = u0; u < u1; ++u) {
        const double c = trig[2 * u], s = trig[2 * u + 1];
        const double edge = 0.5 * (fabs(c) + fabs(s));
        const double q = fma(xc, c, fma(yc, s, cK)), f = floor(q);
        const double d0 = q - f, d1 = 1.0 - d0;
        const int k = (int)f;
        const bool in0 = (uint32_t)k < (uint32_t)K, in1 = (uint32_t)(k + 1) < (uint32_t)K;
        bool v0 = d0 < edge, v1 = d1 < edge;
        if (c == 0.0 || s == 0.0) {
            v0 = axis_hit(c, s, xc, yc, f - cK);
            v1 = axis_hit(c, s, xc, yc, f - cK + 1.0);
        } else if (fabs(d0 - edge) < kEdgeBand || fabs(d1 - edge) < kEdgeBand) {
            const AngleC A = angle_consts(c, s);
            double l;
            v0 = chord(A, xc, yc, f - cK, &l);
            v1 = chord(A, xc, yc, f - cK + 1.0, &l);
        }
        n += (in0 && v0 ? 1 : 0) + (in1 && v1 ? 1 : 0);
    }
    return n;
}

// Entries of a lane's ray at the steps x0 .. x1, which its wavefront shares
// (a step's image row or column is then the same in every lane).  COLS: the
// ray's orientation.  A ray that does not meet the image at a step finds its
// pixels outside.
template <bool COLS>
__device__ __forceinline__ int count_steps(const RayLine& L, const AngleC& A, int N, int x0, int x1,
                                           const MaskView& mv)
{
    const double hc = 0.5 * N - 0.5, w1 = 1.0 - L.w;
    const bool axis = L.c == 0.0 || L.s == 0.0;
    int n = 0;
#pragma unroll 4
    for (int x = x0; x <= x1; ++x) {
        const double a = fma((double)x, L.slope, L.a0), f = floor(a);
        const double d0 = a - f;
        const int b = (int)f;
        bool v0 = d0 < L.w, v1 = d0 > w1;
        const int i0 = COLS ? x : min(max(b, 0), N - 1), i1 = COLS ? x : min(max(b + 1, 0), N - 1);
        const uint32_t s0 = row_span(mv, i0, N), s1 = COLS ? s0 : row_span(mv, i1, N);
        if (axis) {
            v0 = axis_hit(L.c, L.s, (COLS ? b : x) - hc, hc - (COLS ? x : b), L.sk);
            v1 = axis_hit(L.c, L.s, (COLS ? b + 1 : x) - hc, hc - (COLS ? x : b + 1), L.sk);
        } else if (fabs(d0 - L.w) < 2.0 * kEdgeBand || fabs(d0 - w1) < 2.0 * kEdgeBand) {
            double l;
            v0 = chord(A, (COLS ? b : x) - hc, hc - (COLS ? x : b), L.sk, &l);
            v1 = chord(A, (COLS ? b + 1 : x) - hc, hc - (COLS ? x : b + 1), L.sk, &l);
        }
        v0 = v0 && (COLS || i0 == b) && in_support(mv, s0, i0, COLS ? b : x);
        v1 = v1 && (COLS || i1 == b + 1) && in_support(mv, s1, i1, COLS ? b + 1 : x);
        n += (v0 ? 1 : 0) + (v1 ? 1 : 0);
    }
    return n;
}

// part w of kParts of the steps of a lane's ray; every lane of the wavefront
// calls it
__device__ int count_ray(bool on, int N, double c, double s, double sk, const MaskView& mv, int w)
{
    const AngleC A = angle_consts(c, s);
    const RayLine L = ray_line(N, c, s, sk, A);
    int n = 0;
#pragma unroll
    for (int cols = 0; cols < 2; ++cols) {  // a wavefront may span two angles
        const bool mine = on && L.cols == (cols != 0) && L.lo <= L.hi;
        int x0 = mine ? L.lo : N, x1 = mine ? L.hi : -1;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            x0 = min(x0, __shfl_xor(x0, o, 64));
            x1 = max(x1, __shfl_xor(x1, o, 64));
        }
        x0 = __builtin_amdgcn_readfirstlane(x0);
        x1 = __builtin_amdgcn_readfirstlane(x1);
        if (x0 > x1) continue;
        const int len = x1 - x0 + 1;
        const int a = x0 + len * w / kParts, b = x0 + len * (w + 1) / kParts - 1;
        const int m = cols ? count_steps<true>(L, A, N, a, b, mv) : count_steps<false>(L, A, N, a, b, mv);
        if (mine) n = m;
    }
    return n;
}

// Blocks [0, pixel_blocks): 64 pixels each, a sixteenth of the angles per
// wavefront; the rest: 64 rays each, a sixteenth of the steps per wavefront.  A
// block leaves its rows' counts scanned within the block (inclusive), so the last row of each
// chunk holds the chunk's total.  max_row: longest pixel row.
__global__ __launch_bounds__(kCountThreads, 8) void count_kernel(int32_t N, int32_t U, int32_t K,
                                                              const double* __restrict__ trig, MaskView mv,
                                                              unsigned pixel_blocks,
                                                              int64_t* __restrict__ row_ptr,
                                                              int64_t* __restrict__ t_row_ptr,
                                                              int64_t* __restrict__ max_row)
{
    __shared__ int part[kParts][kScanChunk];
    const int t = threadIdx.x, lane = t & (kWave - 1);
    const unsigned block = block_of();
    const bool px = block < pixel_blocks;
    const int64_t n = px ? (int64_t)N * N : (int64_t)U * K;
    const int64_t first = (int64_t)(px ? block : block - pixel_blocks) * kScanChunk;
    if (first >= n) return;  // the grid's padding
    const int w = __builtin_amdgcn_readfirstlane(t / kScanChunk);
    const int64_t at = first + t % kScanChunk;
    int mine = 0;
    if (!px) {
        const int64_t g = at < n ? at : n - 1;
        const int u = (int)(g / K), k = (int)(g - (int64_t)u * K);
        mine = count_ray(at < n, N, trig[2 * u], trig[2 * u + 1], k - 0.5 * (K - 1), mv, w);
    } else if (at < n) {
        const int i = (int)(at / N), j = (int)(at - (int64_t)i * N);
        if (in_support(mv, row_span(mv, i, N), i, j))
            mine = count_pixel(i, j, N, (int)((int64_t)U * w / kParts), (int)((int64_t)U * (w + 1) / kParts), K,
                               trig);
    }
    part[w][t % kScanChunk] = mine;
    __syncthreads();
    static_assert(kScanChunk == kWave, "the first wavefront scans the block's rows");
    if (t >= kScanChunk) return;
    int cnt = 0;
    for (int q = 0; q < kParts; ++q) cnt += part[q][t];
    const int sum = wave_excl_scan(cnt, lane) + cnt;
    int64_t* out = px ? row_ptr : t_row_ptr;
    const int64_t x = first + t;
    if (x == 0) out[0] = 0;
    if (x < n) out[x + 1] = sum;
    if (px) {
        int m = cnt;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o, 64));
        if (lane == 0 && m > 0) atomicMax((unsigned long long*)max_row, (unsigned long long)m);
    }
}

// Second level, one workgroup per array: the chunk totals (last row of each
// chunk) become running totals; the grand totals go to totals[0] and [1].
__global__ __launch_bounds__(1024) void chunk_scan_kernel(int64_t* __restrict__ row_ptr, int64_t np,
                                                          int64_t* __restrict__ t_row_ptr, int64_t g,
                                                          int64_t* __restrict__ totals)
{
    constexpr int IT = 8;
    __shared__ int64_t wsum[16];
    int64_t* a = blockIdx.x ? t_row_ptr : row_ptr;
    const int64_t n = blockIdx.x ? g : np;
    const int64_t chunks = (n + kScanChunk - 1) / kScanChunk;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    auto last = [&](int64_t b) { return (b + 1) * kScanChunk < n ? (b + 1) * kScanChunk : n; };
    int64_t carry = 0;
    for (int64_t base = 0; base < chunks; base += 1024 * IT) {
        int64_t v[IT];
        int64_t loc = 0;
#pragma unroll
        for (int q = 0; q < IT; ++q) {
            const int64_t b = base + (int64_t)t * IT + q;
            v[q] = b < chunks ? a[last(b)] : 0;
        }
#pragma unroll
        for (int q = 0; q < IT; ++q) v[q] = loc += v[q];
        int64_t x = loc;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        if (lane == 63) wsum[w] = x;
        __syncthreads();
        int64_t pre = carry, all = 0;
        for (int q = 0; q < 16; ++q) {
            if (q < w) pre += wsum[q];
            all += wsum[q];
        }
        pre += x - loc;
#pragma unroll
        for (int q = 0; q < IT; ++q) {
            const int64_t b = base + (int64_t)t * IT + q;
            if (b < chunks) a[last(b)] = v[q] + pre;
        }
        carry += all;
        __syncthreads();
    }
    if (t == 0) totals[blockIdx.x] = carry;
}

// Third level: every row but a chunk's last gets the total before its chunk.
__global__ __launch_bounds__(kScanChunk) void chunk_add_kernel(int64_t* __restrict__ row_ptr, int64_t np,
                                                               unsigned pixel_blocks,
                                                               int64_t* __restrict__ t_row_ptr, int64_t g)
{
    const bool px = blockIdx.x < pixel_blocks;
    int64_t* a = px ? row_ptr : t_row_ptr;
    const int64_t n = px ? np : g;
    const int64_t b = px ? blockIdx.x : blockIdx.x - pixel_blocks;
    const int64_t x = b * kScanChunk + threadIdx.x + 1;
    if (b > 0 && x < n && threadIdx.x + 1 < kScanChunk) a[x] += a[b * kScanChunk];
}

// ---------------------------------------------------------------------------
// phase 2: entries
// ---------------------------------------------------------------------------
// Writes a wavefront's up to two entries per lane (lane order, first before
// second) from entry q on; returns their number.
template <typename LenT>
__device__ __forceinline__ int put_pairs(bool v0, bool v1, int32_t c0, int32_t c1, double l0, double l1, int64_t q,
                                         int32_t* __restrict__ col, LenT* __restrict__ len)
{
    const unsigned long long b0 = __ballot(v0), b1 = __ballot(v1);
    int at = __builtin_amdgcn_mbcnt_lo((uint32_t)b0, 0);
    at = __builtin_amdgcn_mbcnt_hi((uint32_t)(b0 >> 32), at);
    at = __builtin_amdgcn_mbcnt_lo((uint32_t)b1, at);
    at = __builtin_amdgcn_mbcnt_hi((uint32_t)(b1 >> 32), at);
    col += q;
    len += q;
    if (v0) {
        st32(col, (uint32_t)at, c0);
        st32(len, (uint32_t)at, (LenT)l0);
    }
    if (v1) {
        const uint32_t at1 = (uint32_t)(at + (v0 ? 1 : 0));
        st32(col, at1, c1);
        st32(len, at1, (LenT)l1);
    }
    return __popcll(b0) + __popcll(b1);
}

// A wavefront takes kPix neighbouring pixels of one image row; per 64 angles
// (one a lane) the angle's constants and the row's share of the projection
// are formed once for all of them.
constexpr int kPix = 8;

template <typename LenT>
__global__ __launch_bounds__(256) void pixel_fill_kernel(int32_t N, int32_t U, int32_t K, int64_t nnz,
                                                         const double* __restrict__ trig,
                                                         const int64_t* __restrict__ row_ptr,
                                                         int32_t* __restrict__ col, LenT* __restrict__ len)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int per_row = (N + kPix - 1) / kPix;
    const int64_t grp = (int64_t)block_of() * kWavesPerBlock + wave;
    if (grp >= (int64_t)N * per_row || row_ptr[(int64_t)N * N] != nnz) return;
    const int i = (int)(grp / per_row), j0 = (int)(grp - (int64_t)i * per_row) * kPix;
    const double hc = 0.5 * N - 0.5, cK = 0.5 * (K - 1);
    const double xc0 = j0 - hc, yc = hc - i;
    const int64_t* rp = row_ptr + (int64_t)i * N + j0;
    int64_t at[kPix];
    uint32_t some = 0;
#pragma unroll
    for (int x = 0; x < kPix; ++x) {
        at[x] = 0;
        if (j0 + x < N) {
            at[x] = lane0(rp[x]);
            if (lane0(rp[x + 1]) > at[x]) some |= 1u << x;
        }
    }
    if (!some) return;
    for (int u0 = 0; u0 < U; u0 += kWave) {
        const int u = u0 + lane;
        const bool on = u < U;
        const double c = on ? trig[2 * u] : 1.0, s = on ? trig[2 * u + 1] : 0.0;
        const AngleC A = angle_consts(c, s);
        const bool axis = c == 0.0 || s == 0.0;
        const int32_t g0 = u * K;
        const uint32_t bins = on ? (uint32_t)K : 0u;  // no ray for the lanes past the last angle
        const double row_hi = -(yc * A.s_hi);  // exact
#pragma unroll
        for (int x = 0; x < kPix; ++x) {
            if (!(some >> x & 1)) continue;
            const double xc = xc0 + x;
            // minus the centre's projection; its bin may come from the leading part
            const double at_hi = fma(-xc, A.c_hi, row_hi), at_lo = offset_lo(A, xc, yc);
            const double f = floor(cK - at_hi);
            const double sk = f - cK;
            double l0, l1;
            bool v0 = chord_at(A, sk + at_hi, at_lo, &l0), v1 = chord_at(A, (sk + 1.0) + at_hi, at_lo, &l1);
            if (axis) {
                l0 = l1 = 1.0;
                v0 = axis_hit(c, s, xc, yc, sk);
                v1 = axis_hit(c, s, xc, yc, sk + 1.0);
            }
            const int32_t k = (int32_t)f;
            v0 = v0 && (uint32_t)k < bins;
            v1 = v1 && (uint32_t)(k + 1) < bins;
            at[x] += put_pairs<LenT>(v0, v1, g0 + k, g0 + k + 1, l0, l1, at[x], col, len);
        }
    }
}

// A wavefront per ray.  Where the ray's steps are image rows, or columns that
// rise with the rows, walking the steps (one a lane) gives the entries in
// pixel order.  A ray closer to the rows whose columns fall as its rows rise
// meets a run of columns in each image row, and the runs of successive rows
// go backwards: its lanes first find the runs of 64 image rows, then take
// the runs' pixels one a lane in order.
template <typename LenT>
__global__ __launch_bounds__(256) void ray_fill_kernel(int32_t N, int32_t U, int32_t K, int64_t nnz,
                                                       const double* __restrict__ trig, MaskView mv,
                                                       const int64_t* __restrict__ t_row_ptr,
                                                       int32_t* __restrict__ t_col, LenT* __restrict__ t_len)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t G = (int64_t)U * K;
    const int64_t g = (int64_t)block_of() * kWavesPerBlock + wave;
    if (g >= G || t_row_ptr[G] != nnz) return;
    int64_t q = t_row_ptr[g];
    if (t_row_ptr[g + 1] == q) return;
    const int u = (int)(g / K), k = (int)(g - (int64_t)u * K);
    const double c = trig[2 * u], s = trig[2 * u + 1], sk = k - 0.5 * (K - 1);
    const AngleC A = angle_consts(c, s);
    const RayLine L = ray_line(N, c, s, sk, A);
    const double hc = 0.5 * N - 0.5;
    if (L.cols || c * s >= 0.0) {
        for (int x0 = L.lo; x0 <= L.hi; x0 += kWave) {
            const int x = x0 + lane;
            const bool on = x <= L.hi;
            const int b = (int)floor(fma((double)x, L.slope, L.a0));
            const bool in0 = on && b >= 0 && b < N, in1 = on && b >= -1 && b < N - 1;
            const int i0 = L.cols ? x : b, j0 = L.cols ? b : x;
            const int i1 = L.cols ? x : b + 1, j1 = L.cols ? b + 1 : x;
            double l0, l1;
            bool v0 = length_at(A, c, s, j0 - hc, hc - i0, sk, &l0), v1 = length_at(A, c, s, j1 - hc, hc - i1, sk, &l1);
            v0 = v0 && in0;
            v1 = v1 && in1;
            if (mv.spans) {
                v0 = v0 && in_support(mv, mv.spans[i0], i0, j0);
                v1 = v1 && in_support(mv, mv.spans[i1], i1, j1);
            }
            q += put_pairs<LenT>(v0, v1, i0 * N + j0, i1 * N + j1, l0, l1, q, t_col, t_len);
        }
        return;
    }
    // rows the ray passes: those of its centre at the first and last step,
    // and the neighbours it reaches
    const double ra = fma((double)L.lo, L.slope, L.a0), rb = fma((double)L.hi, L.slope, L.a0);
    const int i_lo = (int)fmax(0.0, floor(fmin(ra, rb)) - 1.0);
    const int i_hi = (int)fmin((double)(N - 1), floor(fmax(ra, rb)) + 2.0);
    const double inv_c = 1.0 / c, half = (A.edge + kEdgeBand) * fabs(inv_c);
    for (int r0 = i_lo; r0 <= i_hi; r0 += kWave) {
        const int i = r0 + lane;
        int jl = 0, n = 0;
        if (i <= i_hi) {
            const uint32_t span = row_span(mv, i, N);
            const double mid = (sk - (hc - i) * s) * inv_c + hc;
            const double lo = fmax((double)span_first(span), ceil(mid - half));
            const double hi = fmin((double)span_last(span), floor(mid + half));
            if (lo <= hi) {
                jl = (int)lo;
                n = (int)hi - jl + 1;
            }
        }
        const int off = wave_excl_scan(n, lane);
        const int total = __shfl(off + n, kWave - 1, kWave);
        for (int w0 = 0; w0 < total; w0 += kWave) {
            const int x = w0 + lane;
            int r = 0;  // the last row of the 64 that begins at or before x
#pragma unroll
            for (int step = 32; step > 0; step >>= 1)
                if (__shfl(off, r + step, kWave) <= x) r += step;
            const int j = __shfl(jl, r, kWave) + (x - __shfl(off, r, kWave)), ii = r0 + r;
            double l;
            bool v = chord(A, j - hc, hc - ii, sk, &l) && x < total;
            if (mv.spans && v) v = in_support(mv, mv.spans[ii], ii, j);
            q += put_pairs<LenT>(v, false, ii * N + j, 0, l, 0.0, q, t_col, t_len);
        }
    }
}

// support pixels in ascending order, a wavefront per image row
// (and the offsets' totals, to totals[0] and [1])
__global__ __launch_bounds__(256) void support_kernel(int32_t N, MaskView mv, int32_t* __restrict__ support,
                                                      const int64_t* __restrict__ row_end,
                                                      const int64_t* __restrict__ t_row_end,
                                                      int64_t* __restrict__ totals)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        totals[0] = *row_end;
        totals[1] = *t_row_end;
    }
    const int lane = threadIdx.x & (kWave - 1);
    const int i = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
    if (i >= N) return;
    const uint32_t span = row_span(mv, i, N);
    int64_t q = mv.spans ? mv.before[i] : (int64_t)i * N;
    for (int j0 = 0; j0 < N; j0 += kWave) {
        const int j = j0 + lane;
        const bool v = j < N && in_support(mv, span, i, j);
        const unsigned long long b = __ballot(v);
        int at = __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0);
        at = __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), at);
        if (v) support[q + at] = i * N + j;
        q += __popcll(b);
    }
}

// ---------------------------------------------------------------------------
// host
// ---------------------------------------------------------------------------
unsigned blocks_of(int64_t items, int64_t per) { return (unsigned)((items + per - 1) / per); }

// The support as it is uploaded: 64 bytes of zeros (device results), the row
// spans and counts, the bits; and its size and largest squared distance from
// the axis.  It never exceeds pila_build's scratch:
// 64 + N (8 + 4 ceil(N / 32)) <= N^2 + 256 for every N >= 1.
struct HostMask {
    std::vector<char> blob;
    int64_t n_support = 0;
    double rmax2 = -1.0;
    size_t spans_at = 64, before_at = 0, bits_at = 0;
    int32_t words = 0;

    HostMask(const uint8_t* mask, int32_t N)
    {
        const double hc = 0.5 * N - 0.5;
        if (!mask) {
            n_support = (int64_t)N * N;
            rmax2 = 2.0 * hc * hc;
            blob.assign(64, 0);
            return;
        }
        words = (N + 31) / 32;
        before_at = spans_at + 4 * (size_t)N;
        bits_at = before_at + 4 * (size_t)N;
        blob.assign(bits_at + 4 * (size_t)N * words, 0);
        uint32_t* spans = (uint32_t*)(blob.data() + spans_at);
        int32_t* before = (int32_t*)(blob.data() + before_at);
        uint32_t* bits = (uint32_t*)(blob.data() + bits_at);
        for (int32_t i = 0; i < N; ++i) {
            const uint8_t* m = mask + (size_t)i * N;
            uint32_t* b = bits + (size_t)i * words;
            int32_t lo = N, hi = -1;
            int64_t count = 0;
            for (int32_t w = 0; w < words; ++w) {
                const int32_t n = N - 32 * w < 32 ? N - 32 * w : 32;
                uint8_t part[32] = {0};
                std::memcpy(part, m + 32 * w, (size_t)n);
                uint32_t v = 0;
                for (int32_t a = 0; a < 4; ++a) {  // eight flags to eight bits
                    uint64_t x;
                    std::memcpy(&x, part + 8 * a, 8);
                    x = ((x & 0x7f7f7f7f7f7f7f7full) + 0x7f7f7f7f7f7f7f7full) | x;
                    x = (x >> 7) & 0x0101010101010101ull;
                    v |= (uint32_t)((x * 0x0102040810204080ull) >> 56) << (8 * a);
                }
                b[w] = v;
                if (v) {
                    count += __builtin_popcount(v);
                    if (lo == N) lo = 32 * w + __builtin_ctz(v);
                    hi = 32 * w + 31 - __builtin_clz(v);
                }
            }
            before[i] = (int32_t)n_support;
            spans[i] = hi < 0 ? 1u : (uint32_t)lo | (uint32_t)hi << 15 | (count == hi - lo + 1 ? 0u : kSpanGaps);
            n_support += count;
            if (hi >= 0) {
                const double y = hc - i, x0 = lo - hc, x1 = hi - hc;
                rmax2 = std::max(rmax2, y * y + std::max(x0 * x0, x1 * x1));
            }
        }
    }

    MaskView view(const void* d_scratch) const
    {
        if (!words) return MaskView{nullptr, nullptr, nullptr, 0};
        const char* d = (const char*)d_scratch;
        return MaskView{(const uint32_t*)(d + spans_at), (const int32_t*)(d + before_at),
                        (const uint32_t*)(d + bits_at), words};
    }
};

template <typename LenT>
void launch_fill(const pila_geom* g, pila_csr* csr, const MaskView& mv, hipStream_t st)
{
    const int64_t groups = (int64_t)g->n * ((g->n + kPix - 1) / kPix), G = (int64_t)g->n_angles * g->n_bins;
    pixel_fill_kernel<LenT><<<grid_of(blocks_of(groups, kWavesPerBlock)), 256, 0, st>>>(
        g->n, g->n_angles, g->n_bins, csr->nnz, csr->trig, csr->row_ptr, csr->col, (LenT*)csr->len);
    ray_fill_kernel<LenT><<<grid_of(blocks_of(G, kWavesPerBlock)), 256, 0, st>>>(
        g->n, g->n_angles, g->n_bins, csr->nnz, csr->trig, mv, csr->t_row_ptr, csr->t_col, (LenT*)csr->t_len);
}

}  // namespace

}  // namespace pila

using namespace pila;

size_t pila::pila_build_scratch(const pila_geom* geom) { return 256 + (size_t)geom->n * (size_t)geom->n; }

extern "C" int32_t pila_build_scratch_size(const pila_geom* geom, size_t* bytes)
{
    clear_error();
    PILA_TRY(check_geom(geom));
    if (!bytes) return fail(PILA_EINVAL, "bytes is NULL");
    *bytes = pila_build_scratch(geom);
    return PILA_OK;
}

extern "C" int32_t pila_build(const pila_geom* geom, pila_csr* csr, void* d_scratch, size_t scratch_bytes,
                              void* stream)
{
    clear_error();
    PILA_TRY(check_geom(geom));
    if (!csr) return fail(PILA_EINVAL, "csr is NULL");
    if (!csr->row_ptr || !csr->trig || !csr->t_row_ptr)
        return fail(PILA_EINVAL, "row_ptr, trig and t_row_ptr must be allocated");
    if (!d_scratch) return fail(PILA_EINVAL, "scratch is NULL");
    if (scratch_bytes < pila_build_scratch(geom))
        return fail(PILA_ENOMEM, "scratch of %zu bytes is below the %zu needed", scratch_bytes,
                    pila_build_scratch(geom));
    return pila_build_with(geom, csr, d_scratch, (hipStream_t)stream);
}

int32_t pila::pila_build_with(const pila_geom* geom, pila_csr* csr, void* d_scratch, hipStream_t st)
{
    PILA_TRY(check_geom(geom));
    if (!csr || !d_scratch) return fail(PILA_EINVAL, "csr or scratch is NULL");
    if (!csr->row_ptr || !csr->trig || !csr->t_row_ptr)
        return fail(PILA_EINVAL, "row_ptr, trig and t_row_ptr must be allocated");
    const int32_t N = geom->n, U = geom->n_angles, K = geom->n_bins;
    const int64_t NP = (int64_t)N * N, G = (int64_t)U * K;
    if (csr->col && (!csr->len || !csr->support || !csr->t_col || !csr->t_len))
        return fail(PILA_EINVAL, "phase 2 needs col, len, support, t_col and t_len");

    const HostMask hm(geom->mask, N);
    if (csr->col && csr->n_support != (int32_t)hm.n_support)
        return fail(PILA_ESIZE, "n_support %d does not match the mask (%lld)", csr->n_support,
                    (long long)hm.n_support);
    const MaskView mv = hm.view(d_scratch);
    if (!csr->col || mv.spans)
        PILA_HIP(hipMemcpyAsync(d_scratch, hm.blob.data(), hm.blob.size(), hipMemcpyHostToDevice, st));

    if (!csr->col) {  // phase 1: trig, offsets, sizes
        std::vector<double> cs(2 * (size_t)U);
        for (int u = 0; u < U; ++u) trig_of(geom->angles_deg[u], &cs[2 * u], &cs[2 * u + 1]);
        PILA_HIP(hipMemcpyAsync(csr->trig, cs.data(), sizeof(double) * cs.size(),
                                hipMemcpyHostToDevice, st));
        const unsigned pb = blocks_of(NP, kScanChunk), rb = blocks_of(G, kScanChunk);
        int64_t* d_res = (int64_t*)d_scratch;  // entries by pixel, entries by ray, longest pixel row
        count_kernel<<<grid_of((int64_t)pb + rb), kCountThreads, 0, st>>>(N, U, K, csr->trig, mv, pb, csr->row_ptr,
                                                                         csr->t_row_ptr, d_res + 2);
        PILA_HIP(hipGetLastError());
        chunk_scan_kernel<<<2, 1024, 0, st>>>(csr->row_ptr, NP, csr->t_row_ptr, G, d_res);
        chunk_add_kernel<<<pb + rb, kScanChunk, 0, st>>>(csr->row_ptr, NP, pb, csr->t_row_ptr, G);
        PILA_HIP(hipGetLastError());
        int64_t tot[3] = {0, 0, 0};
        PILA_HIP(hipMemcpyAsync(tot, d_res, sizeof(tot), hipMemcpyDeviceToHost, st));
        PILA_HIP(hipStreamSynchronize(st));
        if (tot[0] != tot[1])
            return fail(PILA_EHIP, "pixel-major (%lld) and ray-major (%lld) entry counts differ",
                        (long long)tot[0], (long long)tot[1]);
        csr->nnz = tot[0];
        csr->n_support = (int32_t)hm.n_support;
        csr->max_row = (int32_t)tot[2];
        // a ray reaches a pixel only within 0.71 of its centre's projection, so
        // every bin used by the support lies within R + 1 of the detector centre
        if (hm.rmax2 < 0.0) {
            csr->k_lo = 0;
            csr->k_hi = -1;
        } else {
            const double R = std::sqrt(hm.rmax2), cK = 0.5 * (K - 1);
            csr->k_lo = (int32_t)std::max(0.0, std::floor(cK - R - 1.0));
            csr->k_hi = (int32_t)std::min((double)(K - 1), std::ceil(cK + R + 1.0));
        }
        return PILA_OK;
    }

    // phase 2: entries.  The kernels write nothing unless the offsets' total
    // is csr->nnz; the total is read back with the synchronisation at the end.
    if (geom->len_dtype == PILA_F64)
        launch_fill<double>(geom, csr, mv, st);
    else if (geom->len_dtype == PILA_F32)
        launch_fill<float>(geom, csr, mv, st);
    else
        launch_fill<LenQ>(geom, csr, mv, st);
    PILA_HIP(hipGetLastError());
    int64_t* d_res = (int64_t*)d_scratch;
    support_kernel<<<blocks_of(N, kWavesPerBlock), 256, 0, st>>>(N, mv, csr->support, csr->row_ptr + NP,
                                                                 csr->t_row_ptr + G, d_res);
    PILA_HIP(hipGetLastError());
    int64_t tot[2] = {-1, -1};
    PILA_HIP(hipMemcpyAsync(tot, d_res, sizeof(tot), hipMemcpyDeviceToHost, st));
    PILA_HIP(hipStreamSynchronize(st));
    for (int64_t t : tot)
        if (t != csr->nnz)
            return fail(PILA_ESIZE, "the offsets hold %lld entries but csr->nnz is %lld", (long long)t,
                        (long long)csr->nnz);
    return PILA_OK;
}
