// Rotation of pairs of tensors (y1 = x1 c - x2 s, y2 = x2 c + x1 s: rotary embeddings) over short rows, outside the interpreter.
//
// RoPE's rows are half a head: 64 bf16 columns, one 128-byte line, under tables that all heads of a token share.  In the interpreter that is 13
// records for 16 elements a lane, and the decoding of them, not memory, is what it takes: bf16 over 8111 tokens of 32 heads 30 us, 4.5 TB/s.  Here
//   - a row is held by as many lanes as it has chunks of 16 bytes, a lane takes the same chunk of four rows 64 / lanes apart, so that a wave
//     covers the 32 heads of a token and reads the token's tables once,
//   - a wave takes one such group, and the dispatcher hands them out in order.
// us, interpreter -> here: bf16 over 8111 tokens of 32 heads 31.9 -> 23.6 (5.8 TB/s); the rotations of a 32-layer step of 512 tokens 86 -> 50.
// The arithmetic is the bytecode's: products are rounded where the records round them (a difference rounds both, a sum fuses the one that its
// record fuses), so the bits are the interpreter's and a launch may run in either.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dvm_bytecode.h"
#include "dvm_internal.h"

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));
#define GLOBAL_AS __attribute__((address_space(1)))
#define DI __device__ __forceinline__

DI uint32_t magic_div(uint32_t n, uint32_t m, uint32_t sh) {
    const uint32_t t = __umulhi(m, n);
    return (t + ((n - t) >> (sh & 0xFF))) >> (sh >> 8);
}
template <bool NT> DI u32x4 load16(uint64_t p) {
    if constexpr (NT) return __builtin_nontemporal_load((const GLOBAL_AS u32x4_a2 *)p);
    else return *(const GLOBAL_AS u32x4_a2 *)p;
}
// V elements from 16 bytes (bf16: 8, fp32: 4) or, of an fp32 tensor beside bf16 ones, from twice as many
template <int V, int BF16, bool NT> DI void request(u32x4 *raw, uint64_t p) {
    raw[0] = load16<NT>(p);
    if constexpr (V == 8 && !BF16) raw[1] = load16<NT>(p + 16);
}
template <int V, int BF16> DI void widen(float *o, const u32x4 *raw) {
#pragma unroll
    for (int i = 0; i < V; ++i) {
        const uint32_t w = BF16 ? raw[0][i / 2] : raw[i / 4][i % 4];        // (copied first: a vector's element bit-cast in place is miscompiled)
        if constexpr (BF16) o[i] = __builtin_bit_cast(float, (i & 1) ? w & 0xFFFF0000u : w << 16);
        else o[i] = __builtin_bit_cast(float, w);
    }
}
template <int V> DI u32x4 narrow(const float *v) {
    u32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (V == 8) {
            typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
            typedef float f2 __attribute__((ext_vector_type(2)));
            const f2 x = {v[2 * i], v[2 * i + 1]};
            r[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf2));
        } else {
            r[i] = __builtin_bit_cast(uint32_t, v[i]);
        }
    }
    return r;
}
DI float prod(float a, float b) {
#pragma clang fp contract(off)
    return a * b;
}
DI float diff(float a, float b) {
#pragma clang fp contract(off)
    return a - b;
}
DI float sum(float a, float b) {
#pragma clang fp contract(off)
    return a + b;
}

// V: elements of a chunk (8: x and y are bf16, 4: fp32).  TBF16: the tables' type.  S: rows of a lane.  SHARED: the S rows of a lane differ in
// the first outer index only, along which the tables do not change.  NT: larger than the last-level cache holds.
template <int V, int TBF16, int S, bool SHARED, bool NT>
__global__ void __launch_bounds__(256) dvm_rotary(const dvm_rotary_args a) {
    constexpr int XBF16 = V == 8 ? 1 : 0, XS = XBF16 ? 2 : 4, TS = TBF16 ? 2 : 4, TR = V == 8 && !TBF16 ? 2 : 1, TN = SHARED ? 1 : S;
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t group = blockIdx.x * 4u + (__builtin_amdgcn_readfirstlane(threadIdx.x) >> 6);     // one wave's rows
    if (group >= a.groups) return;
    uint64_t p[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) p[k] = a.p[k];
    if (a.sets != 0) {
        const uint32_t set = magic_div(group, a.set_m, a.set_sh);
        group -= set * a.set_groups;
        const GLOBAL_AS uint64_t *t = (const GLOBAL_AS uint64_t *)a.sets + (uint64_t)set * a.n_tensors;
#pragma unroll
        for (int k = 0; k < 6; ++k) p[k] = t[a.at[k]];
    }
    const uint32_t RW = 64u >> a.log2_lanes;        // rows of a wave side by side
    const int64_t col = (int64_t)(lane & ((1u << a.log2_lanes) - 1u)) * V;
    const uint32_t first = group * (RW * S), mine = lane >> a.log2_lanes;
    int64_t off[6];             // elements from each tensor's start to the lane's chunk of its first row
    auto place = [&](uint32_t row, int64_t *o) {
        const uint32_t q = magic_div(row, a.m1, a.sh1), i1 = row - q * a.d1;
        const uint32_t i3 = magic_div(q, a.m2, a.sh2), i2 = q - i3 * a.d2;
#pragma unroll
        for (int k = 0; k < 6; ++k) o[k] = (int64_t)i1 * a.s[k][0] + (int64_t)i2 * a.s[k][1] + (int64_t)i3 * a.s[k][2] + col;
    };
    u32x4 x1[S][1], x2[S][1], c[TN][TR], s[TN][TR];
    int64_t y1[S], y2[S];
    bool ok[S];
    if constexpr (SHARED) {
        place(first, off);
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const int64_t r = (int64_t)(mine + j * RW);
            request<V, XBF16, NT>(x1[j], p[0] + (uint64_t)((off[0] + r * a.s[0][0]) * XS));
            request<V, XBF16, NT>(x2[j], p[1] + (uint64_t)((off[1] + r * a.s[1][0]) * XS));
            y1[j] = off[4] + r * a.s[4][0];
            y2[j] = off[5] + r * a.s[5][0];
            ok[j] = true;
        }
        request<V, TBF16, false>(c[0], p[2] + (uint64_t)(off[2] * TS));
        request<V, TBF16, false>(s[0], p[3] + (uint64_t)(off[3] * TS));
    } else {
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const uint32_t row = first + mine + (uint32_t)j * RW;
            ok[j] = row < a.rows;
            place(ok[j] ? row : a.rows - 1u, off);
            request<V, XBF16, NT>(x1[j], p[0] + (uint64_t)(off[0] * XS));
            request<V, XBF16, NT>(x2[j], p[1] + (uint64_t)(off[1] * XS));
            request<V, TBF16, false>(c[j], p[2] + (uint64_t)(off[2] * TS));
            request<V, TBF16, false>(s[j], p[3] + (uint64_t)(off[3] * TS));
            y1[j] = off[4];
            y2[j] = off[5];
        }
    }
    float cv[V], sv[V];
    if constexpr (SHARED) {
        widen<V, TBF16>(cv, c[0]);
        widen<V, TBF16>(sv, s[0]);
    }
#pragma unroll
    for (int j = 0; j < S; ++j) {
        float v1[V], v2[V], o1[V], o2[V];
        widen<V, XBF16>(v1, x1[j]);
        widen<V, XBF16>(v2, x2[j]);
        if constexpr (!SHARED) {
            widen<V, TBF16>(cv, c[j]);
            widen<V, TBF16>(sv, s[j]);
        }
#pragma unroll
        for (int e = 0; e < V; ++e) {
            o1[e] = diff(prod(v1[e], cv[e]), prod(v2[e], sv[e]));
            const float q1 = prod(v2[e], cv[e]), q2 = prod(v1[e], sv[e]);
            o2[e] = a.fused == 0 ? sum(q1, q2) : a.fused == 1 ? __builtin_fmaf(v2[e], cv[e], q2) : __builtin_fmaf(v1[e], sv[e], q1);
        }
        if (ok[j]) {
            __builtin_nontemporal_store(narrow<V>(o1), (GLOBAL_AS u32x4_a2 *)(p[4] + (uint64_t)(y1[j] * XS)));
            __builtin_nontemporal_store(narrow<V>(o2), (GLOBAL_AS u32x4_a2 *)(p[5] + (uint64_t)(y2[j] * XS)));
        }
    }
}

template <int V, int TBF16> int launch(const dvm_rotary_args &a, hipStream_t q) {
    const unsigned grid = (a.groups + 3u) / 4u;
#define GO(S, SHARED, NT) hipLaunchKernelGGL((dvm_rotary<V, TBF16, S, SHARED, NT>), dim3(grid), dim3(256), 0, q, a)
    if (a.rows_per_lane == 4) { if (a.stream) GO(4, true, true); else GO(4, true, false); }
    else { if (a.stream) GO(1, false, true); else GO(1, false, false); }
#undef GO
    return (int)hipGetLastError();
}

}  // namespace

extern "C" int dvm_rotary_launch(const dvm_rotary_args *a, void *stream) {
    const hipStream_t q = (hipStream_t)stream;
    if (a->x_bf16) return a->t_bf16 ? launch<8, 1>(*a, q) : launch<8, 0>(*a, q);
    return launch<4, 0>(*a, q);
}
