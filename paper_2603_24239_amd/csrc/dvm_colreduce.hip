// Plain reductions along the penultimate axis ([M, size, N] -> [M, 1, N], Table 1's Sum / Max / Min) outside the interpreter.
//
// A meta-kernel whose body is one streaming record, the combination of the waves and the store (a column sum, a bias
// gradient, either half of a split reduction) has nothing to decode per row.  It is bound by memory, and by how many
// loads are in flight where units of work are few: the interpreter kept 4 to 6 rows in flight per wave in an
// instantiation that spills some 280 vector registers, and its tiles are 64 lanes wide, so that the second half of a split
// bias gradient ([128, 4096] fp32) ran on 16 workgroups.  Here
//   - a wave spreads over 64 / L rows by L lanes of 16 bytes (L = 64 down to 8: a row piece is never below a 128-byte
//     line), L being the widest that leaves enough workgroups,
//   - every lane keeps eight loads in flight, the next one issued as one is used,
//   - L lanes hold one partial result: the segment has `waves` * `partials` of them, number w + j * waves being the j-th partial of
//     wave w in the interpreter's terms.  Partial p adds the rows p, p + waves * partials, .. in order; through LDS the partials of a
//     wave are combined in their order, then the waves in pairs.  The order is the segment's, whatever L is.
// Measured (rotating inputs, whole call): bias gradient bf16 [8192, 4096] in two launches 46 -> 25 us (the launches 46 -> 20 us; the
// rest is host time), fp32 [9238, 8192] in one (no divisor to split by) 317 -> 62 us, [38, 535, 2048] 54 -> 32 us (5.3 TB/s).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dvm_bytecode.h"
#include "dvm_internal.h"

using namespace dvmbc;

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));
#define GLOBAL_AS __attribute__((address_space(1)))

constexpr int U = 8;            // loads in flight per lane

template <uint32_t R> __device__ __forceinline__ float comb(float a, float b) {
    if constexpr (R == R_MAX) return __builtin_elementwise_maximum(a, b);
    else if constexpr (R == R_MIN) return __builtin_elementwise_minimum(a, b);
    else return a + b;
}
template <uint32_t R> __device__ __forceinline__ float ident() {
    if constexpr (R == R_MAX) return -__builtin_inff();
    else if constexpr (R == R_MIN) return __builtin_inff();
    else return 0.0f;
}
// acc = comb(acc, the 16 bytes of one row piece): four fp32 or eight bf16 columns
template <int BF16, uint32_t R> __device__ __forceinline__ void take(float *acc, u32x4 r) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t w = r[i];
        if constexpr (BF16) {
            acc[2 * i] = comb<R>(acc[2 * i], __builtin_bit_cast(float, w << 16));
            acc[2 * i + 1] = comb<R>(acc[2 * i + 1], __builtin_bit_cast(float, w & 0xFFFF0000u));
        } else {
            acc[i] = comb<R>(acc[i], __builtin_bit_cast(float, w));
        }
    }
}
// (no streaming hint: with it bf16 [12577, 8192] takes 52 us instead of 40)
__device__ __forceinline__ u32x4 load16(const char *p) {
    return *(const GLOBAL_AS u32x4_a2 *)p;
}

template <int BF16, uint32_t R>
__global__ void __launch_bounds__(1024) dvm_colreduce(const dvm_colreduce_args a) {
    constexpr int E = BF16 ? 8 : 4;         // columns of a 16-byte piece
    constexpr int ES = BF16 ? 2 : 4;
    extern __shared__ float lds[];          // [partial result][column of the tile]
    const uint32_t tid = threadIdx.x;
    const uint32_t L = 1u << a.log2_lanes, slot = tid & (L - 1u);
    const uint32_t step = a.waves * a.partials, first = tid >> a.log2_lanes;    // this lane's partial result (step and above: none)
    const uint32_t outer = blockIdx.x / a.col_tiles, tile = blockIdx.x - outer * a.col_tiles;
    const uint32_t o2 = a.d2 != 0 ? outer % a.d2 : outer, o3 = a.d2 != 0 ? outer / a.d2 : 0u;
    // The row's last piece slides back to end with the row (the caller made sure that it has a whole one).
    const uint64_t c0 = ((uint64_t)tile * L + slot) * E;
    const uint64_t cmax = a.cols - E;
    const uint64_t c = c0 < cmax ? c0 : cmax;
    const uint32_t n = first < step && first < a.size ? (a.size - first + step - 1) / step : 0u;        // rows of this lane
    // (a lane without rows reads row 0, one with fewer than U its first row again, and takes nothing from it)
    const char *p = (const char *)a.in + ((int64_t)o2 * a.in_s2 + (int64_t)o3 * a.in_s3 + (int64_t)c + (int64_t)(n != 0 ? first : 0u) * a.in_s1) * ES;
    const char *next = p;                   // the row to load next
    const int64_t hop = a.in_s1 * ES * (int64_t)step;
    float acc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = ident<R>();
    u32x4 buf[U];
    const uint32_t n_max = (a.size + step - 1) / step;      // the same for every lane of the launch
#pragma unroll
    for (int u = 0; u < U; ++u) {
        buf[u] = load16((uint32_t)u < n ? next : p);
        next += hop;
    }
    for (uint32_t k = 0; k < n_max; k += U) {
        if (k + 2 * U <= n) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                take<BF16, R>(acc, buf[u]);
                buf[u] = load16(next);
                next += hop;
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (k + (uint32_t)u < n) take<BF16, R>(acc, buf[u]);
                if (k + U + (uint32_t)u < n) buf[u] = load16(next);
                next += hop;
            }
        }
    }
    const uint32_t width = L * E;
    if (first < step) {
#pragma unroll
        for (int e = 0; e < E; ++e) lds[first * width + slot * E + e] = acc[e];
    }
    __syncthreads();
    // partials of a wave in their order (all waves side by side), then the waves in pairs
    if (a.partials > 1) {
        const uint32_t all = a.waves * width;
        for (uint32_t j = tid; j < all; j += blockDim.x) {
            float v = lds[j];
#pragma unroll 4
            for (uint32_t k = 1; k < a.partials; ++k) v = comb<R>(v, lds[k * all + j]);
            lds[j] = v;
        }
        __syncthreads();
    }
    for (uint32_t j = tid; j < width; j += blockDim.x) {
        const uint64_t col = (uint64_t)tile * width + j;
        if (col >= a.cols) break;
        const uint64_t piece = col - j % E;
        const uint32_t at = j + (piece > cmax ? (uint32_t)(piece - cmax) : 0u);     // (where the slid piece holds this column)
        // (four reads in flight; a wave the segment does not have reads the last one's and counts as the neutral value)
        float t[4];
#pragma unroll
        for (uint32_t q = 0; q < 4; ++q) {
            t[q] = ident<R>();
            if (4 * q < a.waves) {
                float x[4];
#pragma unroll
                for (uint32_t w = 0; w < 4; ++w) x[w] = lds[(4 * q + w < a.waves ? 4 * q + w : a.waves - 1u) * width + at];
#pragma unroll
                for (uint32_t w = 0; w < 4; ++w) x[w] = 4 * q + w < a.waves ? x[w] : ident<R>();
                t[q] = comb<R>(comb<R>(x[0], x[1]), comb<R>(x[2], x[3]));
            }
        }
        const float v = comb<R>(comb<R>(t[0], t[1]), comb<R>(t[2], t[3]));
        const int64_t off = (int64_t)o2 * a.out_s2 + (int64_t)o3 * a.out_s3 + (int64_t)col;
        if (a.out_bf16) {
            const __bf16 h = (__bf16)v;
            ((GLOBAL_AS uint16_t *)a.out)[off] = __builtin_bit_cast(uint16_t, h);
        } else {
            ((GLOBAL_AS float *)a.out)[off] = v;
        }
    }
}

}  // namespace

extern "C" int dvm_colreduce_launch(const dvm_colreduce_args *a, unsigned grid, unsigned block, void *stream) {
    const unsigned lds = a->waves * a->partials * ((1u << a->log2_lanes) * (a->in_bf16 ? 8u : 4u)) * 4u;
    const hipStream_t s = (hipStream_t)stream;
#define GO(B, R) hipLaunchKernelGGL((dvm_colreduce<B, R>), dim3(grid), dim3(block), lds, s, *a)
    if (a->in_bf16) {
        if (a->op == R_MAX) GO(1, R_MAX); else if (a->op == R_MIN) GO(1, R_MIN); else GO(1, R_SUM);
    } else {
        if (a->op == R_MAX) GO(0, R_MAX); else if (a->op == R_MIN) GO(0, R_MIN); else GO(0, R_SUM);
    }
#undef GO
    return (int)hipGetLastError();
}
