// PILA-driven projection (Eq. 1), its transpose, and simultaneous SIRT
// (section III-D, Eq. 10-11) on gfx950.
//
// Both directions are gathers, never scatters: the forward projection walks
// the ray-major copy of the PILA (a wavefront per few neighbouring rays, lanes
// stride over the rays' entries, FP64 accumulation, shuffle reduction), the
// back projection walks the pixel-major copy (a wavefront per few pixels).  Every
// output is produced by exactly one wavefront in a fixed order, so results
// are deterministic and need no atomics.  Both stream the PILA from HBM
// once per call (the image / sinogram being gathered stays in L2 / MALL); what
// bounds them at large sizes is the gathers, the accesses of a compute unit's
// address path, at about half of HBM's rate (row_gather_kernel).
#include <cmath>
#include <cstdlib>
#include <vector>

#include "common.hpp"

namespace pila {

namespace {

constexpr int kGatherBlocks = 4096;  // largest grid of the per-row kernels
constexpr int kWPB = 4;              // wavefronts per block

// Rows [0, n) in 8 contiguous chunks, one per XCD: the dispatcher hands
// workgroups to the 8 XCDs round robin (workgroup b to XCD b mod 8), so the
// workgroups of one XCD take neighbouring rays (or pixels), whose gathers
// touch the same image (or sinogram) lines and hit that XCD's L2.  Within a
// chunk the XCD's wavefronts stride over groups of R rows.  The grid is a
// multiple of 8; each row has exactly one wavefront.
struct XcdRows {
    int64_t first, end, stride;
};

template <int R>
__device__ __forceinline__ XcdRows xcd_rows(int64_t n, int w)
{
    constexpr int kXcd = 8;
    const int x = blockIdx.x % kXcd;
    const int64_t nb = gridDim.x / kXcd;
    const int64_t chunk = ((n + kXcd - 1) / kXcd + R - 1) / R * R;
    const int64_t lo = x * chunk;
    const int64_t hi = lo + chunk < n ? lo + chunk : n;
    return {lo + ((int64_t)(blockIdx.x / kXcd) * kWPB + w) * R, hi, nb * kWPB * R};
}

// out[g] = sum over CSR row g of length times x[index] (FP64, fused
// multiply-add).  A wavefront takes R neighbouring rows, L = 64 / R lanes each,
// and a lane V consecutive entries at a time: lane e of a row the entries
// e V + L V i .. + V - 1 by ascending i; its sum is added to the other
// lanes' by a butterfly.  A row's consecutive entries lie on a line of x
// each (a pixel's on another sinogram row per angle, a steep ray's on another
// image row each), while neighbouring rows' entries lie on the same lines, so
// a gather of 8 rows x 8 entries meets about 10 lines where one row's 64
// entries meet 64, and a line's 8 values come from one access; it is the
// accesses of a CU's address path that bound this kernel.  The next entries
// are loaded while the gathers are in flight.
// 1024 x 1024, 720 angles, FP32 (7.6e8 entries, 6 GB; one access a lane alone
// would be 1.3 ms), R = 8: forward 4.05 -> 2.11 ms, back 4.85 -> 2.66 ms; 256 x
// 256 x 180: 45 -> 31 and 56 -> 31 us.  (Eight rows at once but 64 lanes on
// each: 2.41 and 2.94 ms.)
template <typename LenT, int R>
__global__ __launch_bounds__(256) void row_gather_kernel(int64_t n, const int64_t* __restrict__ rp,
                                                         const int32_t* __restrict__ ci,
                                                         const LenT* __restrict__ ln,
                                                         const double* __restrict__ x, double* __restrict__ out)
{
    constexpr int L = 64 / R, V = 4;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const XcdRows xr = xcd_rows<R>(n, w);
    const int64_t last = rp[n] - V;   // where the last V entries begin
    const bool few = last < rp[0];    // fewer entries than one load
    struct Entries {
        int32_t c[V];
        LenT l[V];
    };
    for (int64_t g = xr.first; g < xr.end; g += xr.stride) {
        const int64_t row = g + lane / L;
        const bool on = row < xr.end;
        const int64_t end = on ? rp[row + 1] : 0;
        int64_t q = (on ? rp[row] : 0) + lane % L * V;
        double acc = 0.0;
        Entries e;
        int64_t at = 0;
        auto load = [&]() {  // V entries in one load each, from q or the last V of the array
            at = q < last ? q : last;
            __builtin_memcpy(e.c, ci + at, sizeof(e.c));
            __builtin_memcpy(e.l, ln + at, sizeof(e.l));
        };
        if (few) {
            for (; lane % L == 0 && q < end; ++q) acc = fma((double)ln[q], x[ci[q]], acc);
            q = end;
        }
        if (q < end) load();
        while (q < end) {
            double f[V];
            LenT k[V];
            bool mine[V];
#pragma unroll
            for (int v = 0; v < V; ++v) {
                mine[v] = at + v >= q && at + v < end;
                f[v] = x[e.c[v]];
                k[v] = e.l[v];
            }
            __builtin_amdgcn_sched_barrier(0);
            q += L * V;
            if (q < end) load();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int v = 0; v < V; ++v) {
                const double sum = fma((double)k[v], f[v], acc);
                acc = mine[v] ? sum : acc;
            }
        }
#pragma unroll
        for (int s = 1; s < L; s <<= 1) acc += __shfl_xor(acc, s, 64);
        if (on && lane % L == 0) out[row] = acc;
    }
}

// The same sum by one wavefront a row, 64 entries at a time and kU of these in
// flight, for a few long rows, where the latency of a row's walk is what counts:
// 64 rows of 5100 entries 10 us (two rows a wavefront 26 to 33).
template <typename LenT>
__global__ __launch_bounds__(256) void row_gather_one_kernel(int64_t n, const int64_t* __restrict__ rp,
                                                             const int32_t* __restrict__ ci,
                                                             const LenT* __restrict__ ln,
                                                             const double* __restrict__ x, double* __restrict__ out)
{
    constexpr int kU = 8;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const XcdRows xr = xcd_rows<1>(n, w);
    for (int64_t g = xr.first; g < xr.end; g += xr.stride) {
        const int64_t b = rp[g], e = rp[g + 1];
        double acc = 0.0;
        for (int64_t q0 = b + lane; q0 < e; q0 += 64 * kU) {
            int32_t c[kU];
            double l[kU], v[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
                const int64_t q = q0 + 64 * u < e ? q0 + 64 * u : b;
                c[u] = ci[q];
                l[u] = (double)ln[q];
            }
#pragma unroll
            for (int u = 0; u < kU; ++u) v[u] = x[c[u]];
#pragma unroll
            for (int u = 0; u < kU; ++u)
                if (q0 + 64 * u < e) acc = fma(l[u], v[u], acc);
        }
        acc = wave_sum(acc);
        if (lane == 0) out[g] = acc;
    }
}

// W[g] = sum of the squared lengths of CSR row g: lane e the entries e + 64 i by
// ascending i, the lanes by a butterfly
template <typename LenT>
__global__ __launch_bounds__(256) void row_squares_kernel(int64_t n, const int64_t* __restrict__ rp,
                                                          const LenT* __restrict__ ln, double* __restrict__ W)
{
    constexpr int kU = 8;  // entries per lane in flight
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const XcdRows xr = xcd_rows<1>(n, w);
    for (int64_t g = xr.first; g < xr.end; g += xr.stride) {
        const int64_t b = rp[g], e = rp[g + 1];
        double acc = 0.0;
        for (int64_t q0 = b + lane; q0 < e; q0 += 64 * kU) {
            double l[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) l[u] = (double)ln[q0 + 64 * u < e ? q0 + 64 * u : b];
#pragma unroll
            for (int u = 0; u < kU; ++u)
                if (q0 + 64 * u < e) acc = fma(l[u], l[u], acc);
        }
        acc = wave_sum(acc);
        if (lane == 0) W[g] = acc;
    }
}

// fT = f transposed (N x N), 32 x 32 tiles through LDS
__global__ __launch_bounds__(256) void transpose_kernel(int N, const double* __restrict__ f,
                                                        double* __restrict__ fT)
{
    __shared__ double tile[32][33];
    const int bx = blockIdx.x * 32, by = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8 threads
    for (int r = ty; r < 32; r += 8) {
        const int i = by + r, j = bx + tx;
        if (i < N && j < N) tile[r][tx] = f[(int64_t)i * N + j];
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
        const int j = bx + r, i = by + tx;
        if (i < N && j < N) fT[(int64_t)j * N + i] = tile[tx][r];
    }
}

// one workgroup: out[0] = sum of partial[0..n) in a fixed order
__device__ __forceinline__ void sum_partials(const double* __restrict__ partial, int n, double* __restrict__ out)
{
    __shared__ double ws[4];
    double s = 0.0;
    for (int q = threadIdx.x; q < n; q += 256) s += partial[q];
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) ws[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = (ws[0] + ws[1]) + (ws[2] + ws[3]);
}

// ---------------------------------------------------------------------------
// Tile layouts for SIRT.  Both projections run one wavefront per tile of 64
// PILA rows (lane = row) and walk the tile's rows in step.
//
// Back projection: tiles of 8 x 8 pixels, steps = angles.  A pixel's shadow
// on the detector is at most sqrt 2 bins wide, so at one angle it meets at
// most the two bins b, b + 1 with b = floor(its centre's projection); the
// tile's 64 pixels meet about 12 bins of one sinogram row.
// Forward projection: tiles of 64 rays of consecutive bins at one angle;
// steps are image rows for rays closer to the columns (|cos| >= |sin|), image
// columns for the others.  There a ray meets at most the two pixels b, b + 1
// next to its centre, and the tile's 64 rays meet about 64-91 pixels of one
// image row (read from the image) or column (read from its transpose).
//
// b follows from the geometry (two or three FP64 operations), so a step
// stores only which lanes have the entry at b and which the one at b + 1 (two
// 64-bit masks) and where its lengths begin; the lengths themselves are
// packed in lane order, a lane's one at b before its one at b + 1.  So a lane
// takes one load for its lengths and one for its values at a step, neither
// waiting for the other, and the wavefront reads the lengths as one run.  Per
// entry that is 4.4 bytes in FP32 (with the headers), where an offset and two
// lengths per (row, step), absent ones among them, took 7.1 (back) and 9.5
// (forward) and five loads: the loads a CU's address path takes bound both.
// Every entry is added in the order of a walk by step, b before b + 1.
//
// The layout is built from the PILA's entries and holds their lengths; a tile
// with an entry that is not at b or b + 1 (or two at one place) is flagged and
// its rows are summed straight from the CSR.
// 1024 x 1024, 720 angles, FP32: forward 1.354 -> 0.940 ms, back 1.323 -> 0.939
// ms an iteration (3.3 GB each, 3.5 TB/s, address path 80% busy).
// ---------------------------------------------------------------------------
constexpr int kTile = 8;
constexpr int kOdd = -2;  // flag of a tile summed from its CSR rows

// A tile's lengths have 128 places a step; those of kChunk steps are packed
// together from the chunk's first place on, so that a position in the chunk and
// its byte offset fit in 32 bits whatever the number of angles (a tile of 8 x 8
// pixels under 7 million angles has more than 4 GiB of lengths).
constexpr int kChunk = 1 << 21;

struct StepHead {
    uint64_t m0, m1;  // lanes with an entry at b, at b + 1
    int32_t pos, pad; // the step's first length among its chunk's
};

__device__ __forceinline__ int64_t tile_pixel(const int32_t* tiles, int t, int lane, int N)
{
    const int tt = tiles[t];
    const int ti = tt >> 16, tj = tt & 0xFFFF;
    const int i = ti * kTile + (lane >> 3), j = tj * kTile + (lane & 7);
    return (i < N && j < N) ? (int64_t)i * N + j : -1;
}

__device__ __forceinline__ bool ray_cols(const double* trig, int u)
{
    return fabs(trig[2 * u]) >= fabs(trig[2 * u + 1]);
}

// b of a row at a step.  The layout's builder and its readers call the same
// functions on the same values, so they agree on b whatever its rounding.
struct PixelRow {  // pixel (xc, yc); step = angle
    double xc, yc, cK;
    __device__ __forceinline__ PixelRow(int N, int K, int64_t p)
    {
        const int i = p >= 0 ? (int)(p / N) : 0, j = p >= 0 ? (int)(p - (int64_t)i * N) : 0;
        xc = j - (0.5 * N - 0.5);
        yc = (0.5 * N - 0.5) - i;
        cK = 0.5 * (K - 1);
    }
    __device__ __forceinline__ int at(const double* trig, int u) const
    {
        return (int)floor(fma(xc, trig[2 * u], fma(yc, trig[2 * u + 1], cK)));
    }
};
struct RayRow {  // ray k of an angle; step = image row or column
    double slope, a0;
    __device__ __forceinline__ RayRow(int N, int K, const double* trig, int u, int k)
    {
        const double c = trig[2 * u], s = trig[2 * u + 1], sk = k - 0.5 * (K - 1), hc = 0.5 * N - 0.5;
        if (ray_cols(trig, u)) {
            slope = s / c;
            a0 = (sk - hc * s) / c + hc;
        } else {
            slope = c / s;
            a0 = hc - (sk + hc * c) / s;
        }
    }
    __device__ __forceinline__ int at(const double*, int x) const { return (int)floor(fma((double)x, slope, a0)); }
};

__device__ __forceinline__ int64_t lane0_i64(int64_t v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}

// a / d for 0 <= a < 2^31 by the reciprocal (corrected)
__device__ __forceinline__ int div_by(int a, int d, double inv)
{
    int q = (int)((double)a * inv);
    const int r = a - q * d;
    return r < 0 ? q - 1 : (r >= d ? q + 1 : q);
}

// Builds the layout of one tile per workgroup, a span of steps at a time.
// The wavefronts take 16 rows each and collect the span's masks in LDS; the
// steps' lengths get their places by a scan; the lengths go to their places
// in LDS and leave in contiguous runs.  (Placed straight in memory, each
// length touches a line of its own that is evicted before the next row's.)
//
// A row's entries are in the order of its steps, at most two a step, so a
// span's are the next 2 kSpan at most: all 16 rows' are loaded at once and
// stay in registers until they are placed.  Rays closer to the rows whose
// columns fall as their rows rise are the exception (kRayDown): they are
// taken from the last step to the first, and as each image row's run of
// columns is stored left to right, a span rereads the run that its end cuts
// and may pass two runs' entries of later spans.  With runs of up to 20
// columns (|sin| <= 19 |cos|) that is at most 60 entries more, one more
// window of 64; flatter rays are walked until no later row can reach the span.
// 1024 x 1024, 720 angles, FP32 (6 GB read, 3.3 written a layout): 12.9 + 6.9
// -> 6.2 + 4.3 ms (rays, pixels).  Placing the lengths straight in memory took
// 21 + 15 ms, one row at a time 10 + 11.
enum { kPixels = 0, kRayUp = 1, kRayDown = 2 };
template <typename LenT>
struct LayoutLds {
    static constexpr int kSpan = sizeof(LenT) == 8 ? 32 : 64;  // steps whose lengths fill 32 KB
    LenT stage[kSpan * 128];
    unsigned long long mask[2][kSpan];
    int64_t row_b[64];  // the tile's rows: first entry and length
    int row_n[64];
    int off[kSpan + 1];
    int taken[2][64];  // per row: entries before its first one not taken, this span's and the next's
    int bad;
    unsigned long long entries;
};

// steps of one entry: the step it belongs to and its index in the step's line
template <bool RAY>
struct EntryKey {
    int line;  // entry index = major line + minor
    bool swap; // the step is the minor part
    double inv;
    __device__ __forceinline__ void operator()(int c, int* st, int* idx) const
    {
        const int major = div_by(c, line, inv), minor = c - major * line;
        *st = RAY && swap ? minor : major;
        *idx = RAY && swap ? major : minor;
    }
};

template <typename LenT>
__device__ __forceinline__ void place(LayoutLds<LenT>& L, int x, int slot, int r, LenT l)
{
    const unsigned long long m0 = L.mask[0][x], m1 = L.mask[1][x], below = (1ull << r) - 1;
    const int mine = slot ? (int)(m0 >> r & 1) : 0;  // b before b + 1
    L.stage[L.off[x] + __popcll(m0 & below) + __popcll(m1 & below) + mine] = l;
}

// after the span's masks: its steps' places and heads; `total` lengths of the
// chunk precede
template <typename LenT>
__device__ __forceinline__ void layout_places(LayoutLds<LenT>& L, StepHead* head, int x0, int steps, int total, int lane,
                                              int w, int* first, int* last)
{
    constexpr int kSpan = LayoutLds<LenT>::kSpan;
    if (w == 0) {
        const int n = lane < kSpan ? __popcll(L.mask[0][lane]) + __popcll(L.mask[1][lane]) : 0;
        const int pre = wave_excl_scan(n, lane);
        if (lane < kSpan) {
            L.off[lane] = pre;
            if (x0 + lane < steps) head[x0 + lane] = StepHead{L.mask[0][lane], L.mask[1][lane], total + pre, 0};
        }
        if (lane == kSpan - 1) L.off[kSpan] = pre + n;
        const unsigned long long some = __ballot(n > 0);
        if (some) {
            *first = min(*first, x0 + __ffsll((long long)some) - 1);
            *last = max(*last, x0 + 63 - __clzll((long long)some));
        }
    }
    __syncthreads();
}

// one span of rays taken from the last step to the first.  (The next image
// row's run ends at most one column right of where this one begins: once an
// entry lies two columns left of the span, no later row reaches into it.)
template <typename LenT>
__device__ __forceinline__ void layout_span_down(LayoutLds<LenT>& L, const EntryKey<true>& key, int N, int K,
                                                 const double* trig, int u, int k0, int x0, int x1, int now, int pass,
                                                 int lane, int w, const int32_t* __restrict__ ci,
                                                 const LenT* __restrict__ ln)
{
#pragma unroll 1
    for (int r = w * 16; r < w * 16 + 16; ++r) {
        const int64_t b = L.row_b[r];
        const int n = L.row_n[r];
        const RayRow ray(N, K, trig, u, k0 + r);
        int next = n;          // first entry left for later spans
        int stop = INT32_MAX;  // the image row after which none reaches the span
        for (int q0 = L.taken[now][r]; q0 < n; q0 += 64) {
            const int q = q0 + lane;
            const bool on = q < n;
            const int c = ci[b + (on ? q : q0)];
            const LenT l = ln[b + (on ? q : q0)];
            int st, idx;
            key(c, &st, &idx);
            const bool in = on && st >= x0 && st < x1;
            const int slot = idx - ray.at(trig, in ? st : x0);
            if (in && slot != 0 && slot != 1) L.bad = 1;
            if (in && (slot == 0 || slot == 1)) {
                if (pass == 0)
                    atomicOr(&L.mask[slot][st - x0], 1ull << r);
                else
                    place(L, st - x0, slot, r, l);
            }
            const unsigned long long later = __ballot(on && st < x0);
            if (later && next == n) next = q0 + __ffsll((long long)later) - 1;
            const unsigned long long past = __ballot(on && st < x0 - 1);
            if (past && stop == INT32_MAX) stop = __builtin_amdgcn_readlane(idx, __ffsll((long long)past) - 1);
            if (__ballot(on && idx > stop)) break;
        }
        if (pass == 0 && lane == 0) L.taken[now ^ 1][r] = next;
    }
}

template <typename LenT, int MODE>
__global__ __launch_bounds__(256) void tile_layout_kernel(int N, int U, int K, int nkt, int n_tiles, int64_t nnz,
                                                         const double* __restrict__ trig,
                                                         const int32_t* __restrict__ tiles,
                                                         const int64_t* __restrict__ rp,
                                                         const int32_t* __restrict__ ci,
                                                         const LenT* __restrict__ ln,
                                                         StepHead* __restrict__ heads, LenT* __restrict__ lens,
                                                         int32_t* __restrict__ flag, bool force_csr)
{
    constexpr int kSpan = LayoutLds<LenT>::kSpan;
    constexpr bool RAY = MODE != kPixels;
    // rows of a wavefront; windows of 64 entries a span
    constexpr int kRows = 16, kW = 2 * kSpan / 64 + (MODE == kRayDown ? 1 : 0);
    __shared__ LayoutLds<LenT> L;
    const int t = (int)block_of(), tid = threadIdx.x, lane = tid & 63;
    if (t >= n_tiles) return;  // the grid's padding
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int steps = RAY ? N : U;
    const int u = RAY ? t / nkt : 0, k0 = RAY ? (t - u * nkt) * 64 : 0;
    const bool cols = RAY && ray_cols(trig, u);
    const bool falls = RAY && !cols && trig[2 * u] * trig[2 * u + 1] < 0.0;
    constexpr bool down = MODE == kRayDown;
    if (RAY && falls != down) return;  // the other kernel's tile
    const bool flat = down && fabs(trig[2 * u + 1]) > 19.0 * fabs(trig[2 * u]);
    const int line = RAY ? N : K;
    const EntryKey<RAY> key{line, RAY && !cols, 1.0 / (double)line};
    StepHead* head = heads + (int64_t)t * steps;
    LenT* out = lens + (int64_t)t * steps * 128;
    const int spans = (steps + kSpan - 1) / kSpan;
    if (tid == 0) {
        L.bad = force_csr ? 1 : 0;
        L.entries = 0;
    }
    __syncthreads();
    if (tid < 64) {
        int64_t row = -1;
        if (RAY)
            row = k0 + tid < K ? (int64_t)u * K + k0 + tid : -1;
        else
            row = tile_pixel(tiles, t, tid, N);
        const int64_t b = row >= 0 ? rp[row] : 0;
        const int n = row >= 0 ? (int)(rp[row + 1] - b) : 0;
        L.row_b[tid] = n > 0 ? b : 0;
        L.row_n[tid] = n;
        L.taken[0][tid] = 0;
        if (n > 0) atomicAdd(&L.entries, (unsigned long long)n);
    }
    int total = 0, first = steps, last = -1;
    unsigned long long placed = 0;  // in earlier chunks
    for (int sp = 0; sp < spans; ++sp) {
        const int x0 = (down ? spans - 1 - sp : sp) * kSpan;
        const int x1 = x0 + kSpan < steps ? x0 + kSpan : steps;
        const int now = sp & 1;
        if (!RAY && x0 > 0 && x0 % kChunk == 0) {  // (an image has fewer rows than a chunk)
            placed += (unsigned)total;
            total = 0;
            out += (int64_t)kChunk * 128;
        }
        if (tid < 2 * kSpan) L.mask[tid / kSpan][tid % kSpan] = 0;
        __syncthreads();
        if constexpr (down) {
            if (flat) {
                for (int pass = 0; pass < 2; ++pass) {
                    layout_span_down<LenT>(L, key, N, K, trig, u, k0, x0, x1, now, pass, lane, w, ci, ln);
                    __syncthreads();
                    if (pass == 0) layout_places(L, head, x0, steps, total, lane, w, &first, &last);
                }
            }
        }
        if (!flat) {
            int c[kRows][kW];  // entry indices, then step and slot
            LenT l[kRows][kW];
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                const int rr = w * kRows + r;
                const int64_t b = lane0_i64(L.row_b[rr]);
                const int n = __builtin_amdgcn_readfirstlane(L.row_n[rr]);
                const int from = __builtin_amdgcn_readfirstlane(L.taken[now][rr]);
#pragma unroll
                for (int h = 0; h < kW; ++h) {
                    const int q = from + 64 * h + lane;
                    const uint32_t at = q < n ? (uint32_t)q : 0u;  // (an empty row: the array's first entry)
                    c[r][h] = nnz > 0 ? ci[b + at] : 0;
                    l[r][h] = nnz > 0 ? ln[b + at] : (LenT)0.0;
                }
            }
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                const int rr = w * kRows + r;
                const int n = __builtin_amdgcn_readfirstlane(L.row_n[rr]);
                const int from = __builtin_amdgcn_readfirstlane(L.taken[now][rr]);
                const RayRow ray(N, K, trig, u, k0 + rr);
                const PixelRow px(N, K, RAY ? 0 : tile_pixel(tiles, t, rr, N));
                const int past = min(n, from + 64 * kW);
                int next = past;  // first entry left for later spans
#pragma unroll
                for (int h = 0; h < kW; ++h) {
                    int st, idx;
                    key(c[r][h], &st, &idx);
                    const bool on = from + 64 * h + lane < n;
                    const bool in = on && st >= x0 && st < x1;
                    const int slot = idx - (RAY ? ray.at(trig, in ? st : x0) : px.at(trig, in ? st : x0));
                    const bool ok = slot == 0 || slot == 1;
                    if (in && !ok) L.bad = 1;
                    if (in && ok) atomicOr(&L.mask[slot][st - x0], 1ull << rr);
                    c[r][h] = in && ok ? (st - x0) * 2 + slot : -1;
                    const unsigned long long later = __ballot(on && (down ? st < x0 : st >= x1));
                    if (later && next == past) next = from + 64 * h + __ffsll((long long)later) - 1;
                }
                if (lane == 0) L.taken[now ^ 1][rr] = next;
            }
            __syncthreads();
            layout_places(L, head, x0, steps, total, lane, w, &first, &last);
#pragma unroll
            for (int r = 0; r < kRows; ++r)
#pragma unroll
                for (int h = 0; h < kW; ++h)
                    if (c[r][h] >= 0) place(L, c[r][h] >> 1, c[r][h] & 1, w * kRows + r, l[r][h]);
            __syncthreads();
        }
        const int n = L.off[kSpan];
        for (int q = tid; q < n; q += 256) out[total + q] = L.stage[q];
        total += n;
        __syncthreads();
    }
    if (tid == 0) {
        const bool odd = L.bad || placed + (unsigned)total != L.entries;
        if (RAY) {
            flag[2 * t] = odd ? 0 : first;
            flag[2 * t + 1] = odd ? kOdd : last;
        } else {
            flag[t] = odd ? kOdd : 0;
        }
    }
}

// two neighbouring values in one load (aligned as one value is)
template <typename T>
struct Pair {
    T x, y;
};
template <typename T>
__device__ __forceinline__ Pair<T> pair_at(const T* base, uint32_t i)
{
    Pair<T> p;
    __builtin_memcpy(&p, (const char*)base + i * (uint32_t)sizeof(T), sizeof(p));
    return p;
}

// The S steps from s0: their heads (uniform) first, then lengths and values
// of all of them in flight at once, one load for a lane's two lengths (which
// are neighbours) and one for its two values; absent entries are left out of
// the sum (not added as zeros: what is read in their place may be anything).
// A line has at least two values.
template <typename LenT, int S, typename Row>
__device__ __forceinline__ double tile_steps(double acc, int s0, int line, const Row& row,
                                             const double* __restrict__ trig, const StepHead* __restrict__ head,
                                             const LenT* __restrict__ lens, const double* __restrict__ src)
{
    uint64_t m0[S], m1[S];
    uint32_t pos[S];
    int b[S], at[S];
#pragma unroll
    for (int a = 0; a < S; ++a) {
        m0[a] = head[s0 + a].m0;
        m1[a] = head[s0 + a].m1;
        pos[a] = (uint32_t)head[s0 + a].pos;
    }
#pragma unroll
    for (int a = 0; a < S; ++a) {
        b[a] = row.at(trig, s0 + a);
        at[a] = min(max(b[a], 0), line - 2);
    }
    Pair<double> v[S];
    Pair<LenT> l[S];
#pragma unroll
    for (int a = 0; a < S; ++a) {
        uint32_t i = __builtin_amdgcn_mbcnt_lo((uint32_t)m0[a], pos[a]);
        i = __builtin_amdgcn_mbcnt_hi((uint32_t)(m0[a] >> 32), i);
        i = __builtin_amdgcn_mbcnt_lo((uint32_t)m1[a], i);
        i = __builtin_amdgcn_mbcnt_hi((uint32_t)(m1[a] >> 32), i);
        l[a] = pair_at(lens, i);
        v[a] = pair_at(src + (int64_t)(s0 + a) * line, (uint32_t)at[a]);
    }
#pragma unroll
    for (int a = 0; a < S; ++a) {
        const bool h0 = __builtin_amdgcn_inverse_ballot_w64(m0[a]), h1 = __builtin_amdgcn_inverse_ballot_w64(m1[a]);
        const bool in = b[a] == at[a];  // else b + 1 is the line's first value, or b its last
        const double x = fma((double)l[a].x, in ? v[a].x : v[a].y, acc);
        acc = h0 ? x : acc;
        const double y = fma((double)(h0 ? l[a].y : l[a].x), in ? v[a].y : v[a].x, acc);
        acc = h1 ? y : acc;
    }
    return acc;
}

// acc plus the sum over the steps lo..hi, of one chunk, of one lane's entries:
// length times src[step line + b (+ 1)], by ascending step, b before b + 1.
template <typename LenT, int S, typename Row>
__device__ __forceinline__ double tile_sum(double acc, int lo, int hi, int line, const Row& row,
                                           const double* __restrict__ trig, const StepHead* __restrict__ head,
                                           const LenT* __restrict__ lens, const double* __restrict__ src)
{
    int s = lo;
    for (; s + S - 1 <= hi; s += S) acc = tile_steps<LenT, S>(acc, s, line, row, trig, head, lens, src);
    for (; s <= hi; ++s) acc = tile_steps<LenT, 1>(acc, s, line, row, trig, head, lens, src);
    return acc;
}

// Workgroup b's tile: workgroups go to the 8 XCDs round robin, so XCD x
// takes the x-th eighth of the tiles (neighbouring tiles, shared L2 lines);
// -1 for the padding of the grid to a multiple of 8.
__device__ __forceinline__ int64_t xcd_tile(int64_t n)
{
    constexpr int kXcd = 8;
    const int64_t chunk = (n + kXcd - 1) / kXcd;
    const int64_t t = (int64_t)(blockIdx.x % kXcd) * chunk + blockIdx.x / kXcd;
    return (int64_t)(blockIdx.x / kXcd) < chunk && t < n ? t : -1;
}

unsigned xcd_grid(int64_t n)
{
    return (unsigned)(8 * ((n + 7) / 8));
}

// The steps lo..hi split in kWPB nearly equal parts, wavefront w taking part w
__device__ __forceinline__ void wave_part(int lo, int hi, int w, int* a, int* b)
{
    const int64_t n = (int64_t)hi - lo + 1;
    *a = lo + (int)(n * w / kWPB);
    *b = lo + (int)(n * (w + 1) / kWPB) - 1;
}

// One workgroup per pixel tile; its 4 wavefronts take a quarter of the
// angles each, and their sums are added in wavefront order.  The new values
// go to the image and to its transpose, which the next iteration's projection
// reads; the workgroup after the last tile adds up the iteration's squared
// residuals.  (Both took a kernel of their own, 5 us each at 256 x 256 where
// this one takes 22.)
template <typename LenT>
__global__ __launch_bounds__(256) void tile_back_kernel(int N, int U, int K, int n_tiles,
                                                       const double* __restrict__ trig,
                                                       const int32_t* __restrict__ tiles,
                                                       const int64_t* __restrict__ rp,
                                                       const int32_t* __restrict__ ci,
                                                       const LenT* __restrict__ ln,
                                                       const int32_t* __restrict__ flag,
                                                       const StepHead* __restrict__ heads,
                                                       const LenT* __restrict__ lens,
                                                       const double* __restrict__ y,
                                                       double* __restrict__ f, double* __restrict__ fT, double scale,
                                                       const double* __restrict__ partial, int n_partial,
                                                       double* __restrict__ sse)
{
    constexpr int kA = 8;  // angles in flight
    if (blockIdx.x == gridDim.x - 1) {
        sum_partials(partial, n_partial, sse);
        return;
    }
    __shared__ double part[kWPB][64];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t t = xcd_tile(n_tiles);
    if (t < 0) return;
    const int64_t p = tile_pixel(tiles, (int)t, lane, N);
    double acc = 0.0;
    if (flag[t] == kOdd) {
        if (w == 0 && p >= 0)
            for (int64_t q = rp[p]; q < rp[p + 1]; ++q) acc = fma((double)ln[q], y[ci[q]], acc);
    } else {
        int a, b;
        wave_part(0, U - 1, w, &a, &b);
        const PixelRow row(N, K, p);
        const LenT* l = lens + t * U * 128;
        for (; a <= b; a = (a | (kChunk - 1)) + 1)
            acc = tile_sum<LenT, kA>(acc, a, min(b, a | (kChunk - 1)), K, row, trig, heads + t * U,
                                     l + (int64_t)(a & ~(kChunk - 1)) * 128, y);
    }
    part[w][lane] = acc;
    __syncthreads();
    if (w == 0) {
        const double sum = ((part[0][lane] + part[1][lane]) + part[2][lane]) + part[3][lane];
        if (p >= 0 && rp[p + 1] > rp[p]) {
            const double v = f[p] + scale * sum;
            f[p] = v;
            fT[(p % N) * N + p / N] = v;
        }
    }
}

// Forward projection by bands: the steps of all ray tiles are cut into bands
// of B image rows (or transposed-image rows), B N doubles of each image about
// a megabyte, and the work items (tile, band) of an XCD run band by band, so
// that the XCD's L2 holds the image lines its gathers need.  An item writes
// its 64 partial sums; ray_tile_res_kernel adds them in band order.
//
// A band also is a wavefront's share of a tile: where the tiles are few (n_rt
// of them) the bands are cut further, to 8 steps at the least, for some 8000
// wavefronts (256 x 256, 180 angles, FP64, where 1080 tiles are one wavefront
// a SIMD: 59 -> 23 us).
int ray_band(int N, int64_t n_rt)
{
    int64_t b = 131072 / (N > 0 ? N : 1);
    b = b < 8 ? 8 : (b > 256 ? 256 : b);
    const int64_t few = (int64_t)N * n_rt / 8192;
    b = b < few ? b : few;
    return b < 8 ? 8 : (int)(b & ~(int64_t)7);
}

template <typename LenT>
__global__ __launch_bounds__(64) void ray_tile_part_kernel(int N, int K, int nkt, int n_tiles, int band,
                                                           int n_bands, const double* __restrict__ trig,
                                                           const StepHead* __restrict__ heads,
                                                           const LenT* __restrict__ lens,
                                                           const int32_t* __restrict__ range,
                                                           const int64_t* __restrict__ rp,
                                                           const int32_t* __restrict__ ci,
                                                           const LenT* __restrict__ ln,
                                                           const double* __restrict__ f,
                                                           const double* __restrict__ fT,
                                                           double* __restrict__ part)
{
    constexpr int kS = 8;  // steps in flight
    const int lane = threadIdx.x;
    // item j of XCD x (workgroups go to the XCDs round robin): band j / chunk
    // of tile x chunk + j mod chunk
    const int64_t chunk = (n_tiles + 7) / 8, j = blockIdx.x / 8;
    const int64_t bnd = j / chunk, t = (int64_t)(blockIdx.x % 8) * chunk + j % chunk;
    if (bnd >= n_bands || t >= n_tiles) return;
    const int u = (int)(t / nkt), k = (int)(t - (int64_t)u * nkt) * 64 + lane;
    const double* img = ray_cols(trig, u) ? f : fT;
    const int lo = range[2 * t], hi = range[2 * t + 1];
    double acc = 0.0;
    if (hi == kOdd) {
        if (bnd == 0 && k < K) {
            const int64_t g = (int64_t)u * K + k;
            for (int64_t q = rp[g]; q < rp[g + 1]; ++q) acc = fma((double)ln[q], f[ci[q]], acc);
        }
    } else {
        const int b0 = (int)bnd * band;
        const int a = lo > b0 ? lo : b0, b = hi < b0 + band - 1 ? hi : b0 + band - 1;
        const RayRow row(N, K, trig, u, k);
        acc = tile_sum<LenT, kS>(0.0, a, b, N, row, trig, heads + t * N, lens + t * N * 128, img);
    }
    part[(bnd * n_tiles + t) * 64 + lane] = acc;
}

// res = Pm - A f per ray (A f the band sums added in band order), q = res / W
// (0 where W = 0), and per ray tile the sum of res^2.  A wavefront per tile.
__global__ __launch_bounds__(256) void ray_tile_res_kernel(int K, int nkt, int n_tiles, int n_bands,
                                                           const double* __restrict__ part,
                                                           const double* __restrict__ sino,
                                                           const double* __restrict__ W,
                                                           double* __restrict__ out,
                                                           double* __restrict__ partial)
{
    const int lane = threadIdx.x & 63;
    const int64_t t = (int64_t)blockIdx.x * kWPB + (threadIdx.x >> 6);
    if (t >= n_tiles) return;
    const int u = (int)(t / nkt), k = (int)(t - (int64_t)u * nkt) * 64 + lane;
    double sum = 0.0;
    for (int b = 0; b < n_bands; ++b) sum += part[((int64_t)b * n_tiles + t) * 64 + lane];
    double sq = 0.0;
    if (k < K) {
        const int64_t g = (int64_t)u * K + k;
        const double res = sino[g] - sum;
        const double wg = W[g];
        out[g] = wg > 0.0 ? res / wg : 0.0;
        sq = res * res;
    }
    sq = wave_sum(sq);
    if (lane == 0) partial[t] = sq;
}

// 8 x 8 tiles holding at least one support pixel, as (tile row << 16 | tile column)
std::vector<int32_t> support_tiles(const pila_geom* g)
{
    const int N = g->n, nt = (N + kTile - 1) / kTile;
    std::vector<int32_t> out;
    for (int ti = 0; ti < nt; ++ti)
        for (int tj = 0; tj < nt; ++tj) {
            bool any = false;
            for (int a = 0; a < kTile && !any; ++a)
                for (int b = 0; b < kTile && !any; ++b) {
                    const int i = ti * kTile + a, j = tj * kTile + b;
                    if (i < N && j < N && (!g->mask || g->mask[(int64_t)i * N + j])) any = true;
                }
            if (any) out.push_back((ti << 16) | tj);
        }
    return out;
}

// SIRT workspace: factor matrix, scaled residual, block partials, costs,
// the transposed image and the tile layout
struct SirtLayout {
    size_t W, q, partial, sse, fT, tiles, flag, heads, lens, rheads, rlens, range, bpart, total;
};

SirtLayout sirt_layout(const pila_geom* g, int32_t n_iter, size_t n_tiles)
{
    const size_t G = (size_t)g->n_angles * g->n_bins, NP = (size_t)g->n * g->n;
    const size_t ls = (size_t)len_bytes(g->len_dtype);
    const size_t cells = n_tiles * (size_t)g->n_angles;
    SirtLayout L;
    size_t at = 0;
    auto take = [&](size_t bytes) {
        const size_t o = at;
        at += (bytes + 255) & ~(size_t)255;
        return o;
    };
    L.W = take(sizeof(double) * G);
    L.q = take(sizeof(double) * G);
    const size_t nrt0 = (size_t)g->n_angles * ((g->n_bins + 63) / 64);
    L.partial = take(sizeof(double) * (nrt0 > (size_t)kGatherBlocks ? nrt0 : (size_t)kGatherBlocks));
    L.fT = take(sizeof(double) * NP);
    L.tiles = take(sizeof(int32_t) * (n_tiles ? n_tiles : 1));
    L.flag = take(sizeof(int32_t) * (n_tiles ? n_tiles : 1));
    L.heads = take(sizeof(StepHead) * cells);
    L.lens = take(ls * 128 * cells);  // at most two lengths per lane and step
    const size_t nrt = (size_t)g->n_angles * ((g->n_bins + 63) / 64);
    const size_t rcells = nrt * (size_t)g->n;
    L.rheads = take(sizeof(StepHead) * rcells);
    L.rlens = take(ls * 128 * rcells);
    L.range = take(sizeof(int32_t) * 2 * nrt);
    const int band = ray_band(g->n, (int64_t)nrt);
    const size_t n_bands = (size_t)((g->n + band - 1) / band);
    L.bpart = take(sizeof(double) * n_bands * nrt * 64);
    // last, so that the layouts above sit at the same offsets for any n_iter
    L.sse = take(sizeof(double) * (size_t)(n_iter > 0 ? n_iter : 1));
    L.total = at;
    return L;
}

unsigned gather_blocks(int64_t groups)
{
    int64_t b = (groups + kWPB - 1) / kWPB;
    b = b < kGatherBlocks ? b : kGatherBlocks;
    return (unsigned)((b + 7) / 8 * 8);  // a multiple of the 8 XCDs, at least 8
}

// Rows a wavefront takes at once.  More rows share more lines of x, fewer have
// more wavefronts and more of a row in flight: with n rows that reach across
// `reach` steps (a ray the image's rows or columns, a pixel the angles), eight
// only where they fill the GPU or the rows are short.  Measured (f32 and f64,
// us, 8 / 4 / 2 / 1 rows): rays of 1024 x 1024, 1 angle 24 / 13 / 9 / 8; 6
// angles 35 / 22 / 27 / 30; 512 x 512, 16 angles 19 / 12 / 14 / 16; 2048 x
// 2048, 1 angle 54 / 26 / 31 / 30; pixels of 64 x 64, 720 angles 18 / 12 / 9 /
// 11; 16 x 16, 5000 angles 86 / 50 / 30 / 13; rays of 128 x 128, 90 angles (16380
// rows of 90 entries) 8 whatever is taken, of 64 x 64, 720 angles 8 / 9 / 12 / 15.
int rows_per_wave(int64_t n, int64_t reach)
{
    if (n >= 32768 || reach <= 128) return 8;
    if (n >= 8192 || (n >= 2048 && reach >= 2048)) return 4;
    return n >= 1024 ? 2 : 1;
}

template <typename LenT>
int32_t gather_rows(int64_t n, int64_t reach, const int64_t* rp, const int32_t* ci, const void* ln, const double* x,
                    double* out, hipStream_t st)
{
    const int R = rows_per_wave(n, reach);
    const unsigned blocks = gather_blocks((n + R - 1) / R);
    const LenT* l = (const LenT*)ln;
    if (R == 8)
        row_gather_kernel<LenT, 8><<<blocks, 256, 0, st>>>(n, rp, ci, l, x, out);
    else if (R == 4)
        row_gather_kernel<LenT, 4><<<blocks, 256, 0, st>>>(n, rp, ci, l, x, out);
    else if (R == 2)
        row_gather_kernel<LenT, 2><<<blocks, 256, 0, st>>>(n, rp, ci, l, x, out);
    else
        row_gather_one_kernel<LenT><<<blocks, 256, 0, st>>>(n, rp, ci, l, x, out);
    PILA_HIP(hipGetLastError());
    return PILA_OK;
}

int32_t gather_rows(int32_t len_dtype, int64_t n, int64_t reach, const int64_t* rp, const int32_t* ci, const void* ln,
                    const double* x, double* out, hipStream_t st)
{
    if (len_dtype == PILA_F64) return gather_rows<double>(n, reach, rp, ci, ln, x, out, st);
    if (len_dtype == PILA_F32) return gather_rows<float>(n, reach, rp, ci, ln, x, out, st);
    return gather_rows<LenQ>(n, reach, rp, ci, ln, x, out, st);
}

int32_t check_csr(const pila_geom* g, const pila_csr* c, bool need_rays, bool need_pixels)
{
    PILA_TRY(check_geom(g));
    if (!c) return fail(PILA_EINVAL, "csr is NULL");
    if (need_pixels && (!c->row_ptr || !c->col || !c->len))
        return fail(PILA_EINVAL, "pixel-major PILA arrays missing");
    if (need_rays && (!c->t_row_ptr || !c->t_col || !c->t_len))
        return fail(PILA_EINVAL, "ray-major PILA arrays missing");
    return PILA_OK;
}

}  // namespace

}  // namespace pila

using namespace pila;

extern "C" int32_t pila_forward(const pila_geom* geom, const pila_csr* csr, const double* d_image,
                                double* d_out, void* stream)
{
    clear_error();
    PILA_TRY(check_csr(geom, csr, true, false));
    if (!d_image || !d_out) return fail(PILA_EINVAL, "image or output is NULL");
    return gather_rows(geom->len_dtype, (int64_t)geom->n_angles * geom->n_bins, geom->n, csr->t_row_ptr, csr->t_col,
                       csr->t_len, d_image, d_out, (hipStream_t)stream);
}

extern "C" int32_t pila_backproject(const pila_geom* geom, const pila_csr* csr, const double* d_sino,
                                    double* d_out, void* stream)
{
    clear_error();
    PILA_TRY(check_csr(geom, csr, false, true));
    if (!d_sino || !d_out) return fail(PILA_EINVAL, "sinogram or output is NULL");
    return gather_rows(geom->len_dtype, (int64_t)geom->n * geom->n, geom->n_angles, csr->row_ptr, csr->col, csr->len,
                       d_sino, d_out, (hipStream_t)stream);
}

extern "C" int32_t sirt_workspace_size(const pila_geom* geom, const sirt_params* params, size_t* bytes)
{
    clear_error();
    PILA_TRY(check_geom(geom));
    if (!params || !bytes) return fail(PILA_EINVAL, "params or bytes is NULL");
    if (params->n_iter < 0) return fail(PILA_EINVAL, "n_iter < 0");
    *bytes = sirt_layout(geom, params->n_iter, support_tiles(geom).size()).total;
    return PILA_OK;
}

template <typename LenT>
static int32_t sirt_impl(const pila_geom* geom, const pila_csr* csr, const double* d_sino,
                         const sirt_params* prm, double* d_image, char* ws, double* h_cost,
                         hipStream_t st)
{
    const int N = geom->n, U = geom->n_angles, K = geom->n_bins;
    const int64_t G = (int64_t)U * K;
    const std::vector<int32_t> tiles = support_tiles(geom);
    const int n_tiles = (int)tiles.size();
    const SirtLayout L = sirt_layout(geom, prm->n_iter, tiles.size());
    double* W = (double*)(ws + L.W);
    double* q = (double*)(ws + L.q);
    double* partial = (double*)(ws + L.partial);
    double* sse = (double*)(ws + L.sse);
    double* fT = (double*)(ws + L.fT);
    int32_t* d_tiles = (int32_t*)(ws + L.tiles);
    int32_t* flag = (int32_t*)(ws + L.flag);
    StepHead* heads = (StepHead*)(ws + L.heads);
    LenT* lens = (LenT*)(ws + L.lens);
    // PILA_SIRT_CSR=1 sums every tile from its CSR rows (the path a tile of
    // irregular shape takes), for tests of that path
    const char* env = std::getenv("PILA_SIRT_CSR");
    const bool force_csr = (env && env[0] == '1') || N < 2 || K < 2;  // (a line of one value: from the rows too)
    const bool reuse = (prm->flags & PILA_SIRT_REUSE_LAYOUT) != 0;
    // factor matrix: W_g = sum of squared lengths of ray g over the support
    if (!reuse)
        row_squares_kernel<LenT><<<gather_blocks(G), 256, 0, st>>>(G, csr->t_row_ptr, (const LenT*)csr->t_len, W);
    if (n_tiles > 0 && !reuse) {
        PILA_HIP(hipMemcpyAsync(d_tiles, tiles.data(), sizeof(int32_t) * tiles.size(),
                                hipMemcpyHostToDevice, st));
        tile_layout_kernel<LenT, kPixels><<<grid_of(n_tiles), 256, 0, st>>>(N, U, K, 0, n_tiles, csr->nnz, csr->trig,
                                                                          d_tiles, csr->row_ptr, csr->col,
                                                                          (const LenT*)csr->len, heads, lens, flag,
                                                                          force_csr);
    }
    const int nkt = (K + 63) / 64, n_rt = U * nkt;
    StepHead* rheads = (StepHead*)(ws + L.rheads);
    LenT* rlens = (LenT*)(ws + L.rlens);
    int32_t* range = (int32_t*)(ws + L.range);
    double* bpart = (double*)(ws + L.bpart);
    const int band = ray_band(N, n_rt), n_bands = (N + band - 1) / band;
    if (!reuse) {
        tile_layout_kernel<LenT, kRayUp><<<grid_of(n_rt), 256, 0, st>>>(N, U, K, nkt, n_rt, csr->nnz, csr->trig, nullptr,
                                                              csr->t_row_ptr, csr->t_col, (const LenT*)csr->t_len,
                                                              rheads, rlens, range, force_csr);
        tile_layout_kernel<LenT, kRayDown><<<grid_of(n_rt), 256, 0, st>>>(N, U, K, nkt, n_rt, csr->nnz, csr->trig, nullptr,
                                                                csr->t_row_ptr, csr->t_col, (const LenT*)csr->t_len,
                                                                rheads, rlens, range, force_csr);
    }

    const double scale = prm->lambda / (double)geom->n_angles;
    const dim3 tgrid((unsigned)((N + 31) / 32), (unsigned)((N + 31) / 32));
    if (prm->n_iter > 0) transpose_kernel<<<tgrid, 256, 0, st>>>(N, d_image, fT);
    for (int32_t it = 0; it < prm->n_iter; ++it) {
        ray_tile_part_kernel<LenT><<<(unsigned)(8 * ((n_rt + 7) / 8) * n_bands), 64, 0, st>>>(
            N, K, nkt, n_rt, band, n_bands, csr->trig, rheads, rlens, range, csr->t_row_ptr, csr->t_col,
            (const LenT*)csr->t_len, d_image, fT, bpart);
        ray_tile_res_kernel<<<(unsigned)((n_rt + kWPB - 1) / kWPB), 256, 0, st>>>(K, nkt, n_rt, n_bands, bpart,
                                                                                d_sino, W, q, partial);
        tile_back_kernel<LenT><<<xcd_grid(n_tiles) + 1, 256, 0, st>>>(
            N, U, K, n_tiles, csr->trig, d_tiles, csr->row_ptr, csr->col, (const LenT*)csr->len, flag, heads, lens, q,
            d_image, fT, scale, partial, n_rt, sse + it);
    }
    PILA_HIP(hipGetLastError());
    if (h_cost && prm->n_iter > 0) {
        std::vector<double> s((size_t)prm->n_iter);
        PILA_HIP(hipMemcpyAsync(s.data(), sse, sizeof(double) * s.size(), hipMemcpyDeviceToHost, st));
        PILA_HIP(hipStreamSynchronize(st));
        const double KU = (double)geom->n_bins * (double)geom->n_angles;
        for (size_t i = 0; i < s.size(); ++i) h_cost[i] = std::sqrt(s[i] / KU);
    }
    return PILA_OK;
}

extern "C" int32_t sirt_run(const pila_geom* geom, const pila_csr* csr, const double* d_sino,
                            const sirt_params* params, double* d_image, void* d_ws, size_t ws_bytes,
                            double* h_cost, void* stream)
{
    clear_error();
    PILA_TRY(check_csr(geom, csr, true, true));
    if (!params || !d_sino || !d_image) return fail(PILA_EINVAL, "params, sinogram or image is NULL");
    if (!csr->trig) return fail(PILA_EINVAL, "trig (from pila_build) is NULL");
    if (!std::isfinite(params->lambda)) return fail(PILA_EINVAL, "lambda is not finite");
    if (params->flags & ~PILA_SIRT_REUSE_LAYOUT) return fail(PILA_EINVAL, "unknown flags %d", params->flags);
    size_t need = 0;
    PILA_TRY(sirt_workspace_size(geom, params, &need));
    if (!d_ws || ws_bytes < need)
        return fail(PILA_ENOMEM, "workspace of %zu bytes is below the %zu needed", ws_bytes, need);
    hipStream_t st = (hipStream_t)stream;
    if (geom->len_dtype == PILA_F64)
        return sirt_impl<double>(geom, csr, d_sino, params, d_image, (char*)d_ws, h_cost, st);
    if (geom->len_dtype == PILA_F32)
        return sirt_impl<float>(geom, csr, d_sino, params, d_image, (char*)d_ws, h_cost, st);
    return sirt_impl<LenQ>(geom, csr, d_sino, params, d_image, (char*)d_ws, h_cost, st);
}
