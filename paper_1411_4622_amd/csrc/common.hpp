// Shared device helpers and host error plumbing for the gfx950 PILA library.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "pila.h"

namespace pila {

// ---------------------------------------------------------------------------
// host-side error reporting (thread-local message, status codes of pila.h)
// ---------------------------------------------------------------------------
int32_t fail(int32_t code, const char* fmt, ...);
int32_t hip_fail(hipError_t e, const char* what, const char* file, int line);
void clear_error();

#define PILA_HIP(call)                                                          \
    do {                                                                        \
        hipError_t e_ = (call);                                                 \
        if (e_ != hipSuccess) return ::pila::hip_fail(e_, #call, __FILE__, __LINE__); \
    } while (0)

#define PILA_TRY(expr)                      \
    do {                                    \
        int32_t rc_ = (expr);               \
        if (rc_ != PILA_OK) return rc_;     \
    } while (0)

constexpr double kTau = 1e-9;  // lengths at or below this (corner touches) are not stored
constexpr int kWave = 64;

// One-byte intersection length (section II-B: the length times 180,
// rounded; halves away from zero).  It stands for the float q / 180,
// correctly rounded, which for every byte value equals q * fl(1/180) with
// one fused multiply-add correction of its residual (three instructions
// instead of a division; the identity is checked exhaustively by the test
// suite).  Kernels templated on the length type read it through this float
// conversion; the PILA build stores it through the constructor.
struct LenQ {
    uint8_t q;
    LenQ() = default;
    __host__ __device__ explicit LenQ(double l) : q((uint8_t)round(180.0 * l)) {}
    __host__ __device__ operator float() const
    {
        const float x = (float)q, c = 1.0f / 180.0f;
        const float r = x * c;
        return fmaf(fmaf(-r, 180.0f, x), c, r);
    }
};
static_assert(sizeof(LenQ) == 1, "one byte per length");

// host: (cos, sin) of degrees, exact at multiples of 90 degrees
void trig_of(double deg, double* c, double* s);
// host: validate a geometry (sizes, finite angles, dtype)
int32_t check_geom(const pila_geom* g);
// host: bytes of one stored length of a len_dtype
inline int len_bytes(int32_t dtype) { return dtype == PILA_F64 ? 8 : dtype == PILA_F32 ? 4 : 1; }

// Launches of more workgroups than one grid dimension takes (2^32 threads; more
// are dropped without an error): the workgroups in rows of kGridRow, the last
// row padded, and a workgroup's number.
constexpr unsigned kGridRow = 1u << 21;
inline dim3 grid_of(int64_t blocks)
{
    return blocks <= (int64_t)kGridRow ? dim3((unsigned)blocks)
                                       : dim3(kGridRow, (unsigned)((blocks + kGridRow - 1) / kGridRow));
}
__device__ __forceinline__ unsigned block_of() { return blockIdx.y * kGridRow + blockIdx.x; }

// ---------------------------------------------------------------------------
// device: Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11)
// ---------------------------------------------------------------------------
struct Words4 {
    uint64_t w0, w1, w2, w3;
};

__device__ __forceinline__ Words4 philox4x64(uint64_t k0, uint64_t k1, uint64_t c0, uint64_t c1,
                                             uint64_t c2, uint64_t c3)
{
    constexpr uint64_t M0 = 0xD2E7470EE14C6C93ULL, M1 = 0xCA5A826395121157ULL;
    constexpr uint64_t W0 = 0x9E3779B97F4A7C15ULL, W1 = 0xBB67AE8584CAA73BULL;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += W0;
            k1 += W1;
        }
        const uint64_t hi0 = __umul64hi(M0, c0), lo0 = M0 * c0;
        const uint64_t hi1 = __umul64hi(M1, c2), lo1 = M1 * c2;
        const uint64_t n0 = hi1 ^ c1 ^ k0, n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
    }
    return {c0, c1, c2, c3};
}

__device__ __forceinline__ double unit53(uint64_t w) { return (double)(w >> 11) * 0x1p-53; }

// ---------------------------------------------------------------------------
// device: wavefront reductions (64 lanes)
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ T wave_sum(T v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
    return v;
}

// exclusive prefix over the lanes of a wave (lane order)
__device__ __forceinline__ int wave_excl_scan(int v, int lane)
{
    int x = v;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        int y = __shfl_up(x, o, kWave);
        if (lane >= o) x += y;
    }
    return x - v;
}

}  // namespace pila
