// Softmax along the row, plain or of a sum of two tensors (attention scores and their mask), outside the interpreter.
//
// A meta-kernel whose body is load [, load, add], max, exp(. - max), 1 / sum, store times that, over at least DVM_SOFTMAX_MIN_BYTES, leaves
// the interpreter wherever it stands (alone, in a stack, in a batched launch: the same arithmetic, the same bits).  It is bound by
// memory, and what the interpreter lost there was not arithmetic (its vector units are busy 30 % of the time) but the way it meets memory:
//   - Rows that are no whole number of 128-byte lines.  A wave's 1 KiB store then begins and ends inside a line, each such line is
//     written in two parts, and the traffic of writes grows by a tenth.  Here the chunk grid of a row is shifted to the lines of the
//     output: every store but a row's first and last covers whole lines (masked softmax fp32 [96, 1411, 1411] 308 -> 285 us).
//   - Workgroups that walk a long list of tiles drift apart and the memory in use with them.  A workgroup here takes one tile; the
//     dispatcher keeps the front together (softmax bf16 [192224, 751] 112 us in 4 workgroups per compute unit, 99 in one per tile).
//   - Rows longer than a tile were read twice.  Here a workgroup holds one in its registers and LDS (a second tensor is read again in each pass).
// Interpreter and this kernel, rotating inputs, us: masked softmax fp32 [64, 2048, 2048] 420 -> 367 (5.9 TB/s), [96, 1411, 1411] 343 -> 267,
// softmax bf16 [192224, 751] 129 -> 94 (6.1 TB/s), fp32 [31250, 4096] 196 -> 161, fp32 [671, 100003] 141 -> 113 (4.7 TB/s), bf16 [1279, 100003]
// 165 -> 120.  What is left in the last two is one row per compute unit: nothing is loaded while its exponentials are taken.
// A row is T lanes wide (8 to 64 lanes of a wave, or 2 to 16 waves of a workgroup), a lane holds NR chunks of 16 bytes.
//
// The bits of a row do not depend on where it stands, although the shift does: column c is summed in the class (c mod T * V); a class
// is one lane's running sum at any shift, over ascending columns, and the classes are brought into their order through LDS before they are
// combined.  The two chunks that reach over the ends of a row slide back inside (every access stays in the row) and hand each class its
// element by a barrel shift.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "dvm_bytecode.h"
#include "dvm_internal.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));
#define GLOBAL_AS __attribute__((address_space(1)))
#define DI __device__ __forceinline__

constexpr float LOG2E = 1.44269504088896340736f;
constexpr float NEG_INF = -__builtin_inff();

DI float maxp(float a, float b) { return __builtin_elementwise_maximum(a, b); }        // (NaN propagates)
template <int CTRL> DI float dpp(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
DI float lane_of(float v, int l) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l)); }
template <bool MAX> DI float comb(float a, float b) {
    if constexpr (MAX) return maxp(a, b);
    else return a + b;
}
// all lanes of a group of T (8 .. 64, beyond that of a wave)
template <bool MAX, int T> DI float group_all(float v) {
    v = comb<MAX>(v, dpp<0xB1>(v));                     // quad_perm [1,0,3,2]
    v = comb<MAX>(v, dpp<0x4E>(v));                     // quad_perm [2,3,0,1]
    v = comb<MAX>(v, dpp<0x141>(v));                    // row_half_mirror
    if constexpr (T >= 16) v = comb<MAX>(v, dpp<0x140>(v));                     // row_mirror
    if constexpr (T >= 32) v = comb<MAX>(v, __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), 0x401F)));    // lane ^ 16
    if constexpr (T >= 64) v = comb<MAX>(lane_of(v, 0), lane_of(v, 32));
    return v;
}

DI float bf16_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
DI float bf16_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xFFFF0000u); }
DI uint32_t pack_bf16x2(float a, float b) {
    typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    const f2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf2));
}
// chunks of 16 bytes: V elements
template <int BF16> DI void widen(float *o, u32x4 r) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t w = r[i];
        if constexpr (BF16) {
            o[2 * i] = bf16_lo(w);
            o[2 * i + 1] = bf16_hi(w);
        } else {
            o[i] = __builtin_bit_cast(float, w);
        }
    }
}
template <int BF16> DI u32x4 narrow(const float *v, float scale) {
    u32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (BF16) r[i] = pack_bf16x2(v[2 * i] * scale, v[2 * i + 1] * scale);
        else r[i] = __builtin_bit_cast(uint32_t, v[i] * scale);
    }
    return r;
}
// (closes a branch of loads with the streaming hint, which the compiler would otherwise merge with the branch of those without it, dropping
// the hint.  It still asks for the slots that every row has before the branch, without the hint: with it on all of them fp32 [30000, 2048] took
// 79 us instead of 71, bf16 [60000, 2048] 77 instead of 70, under a mask fp32 [1, 32, 3000, 3000] 413 instead of 427.)
#define STREAMING() asm volatile("; streaming" ::: "memory")
template <bool NT> DI u32x4 load16(const char *p) {
    if constexpr (NT) return __builtin_nontemporal_load((const GLOBAL_AS u32x4_a2 *)p);
    else return *(const GLOBAL_AS u32x4_a2 *)p;
}
DI void store16(char *p, u32x4 v) { __builtin_nontemporal_store(v, (GLOBAL_AS u32x4_a2 *)p); }

// A chunk that starts at c0 (below 0: before the row; above cmax: it would end behind the row) holds the columns from
// min(max(c0, 0), cmax) on.  Column c0 + e belongs to class e: put every element there, 0 where the class has none.
template <int V> DI void to_classes(float *h, int c0, int cmax) {
    const uint32_t b = c0 < 0 ? (uint32_t)-c0 : 0u, d = c0 > cmax ? (uint32_t)(c0 - cmax) : 0u;
#pragma unroll
    for (int s = V / 2; s >= 1; s /= 2) {
        const bool down = (d & (uint32_t)s) != 0, up = (b & (uint32_t)s) != 0;
#pragma unroll
        for (int e = 0; e < V; ++e) h[e] = down ? (e + s < V ? h[e + s] : 0.0f) : h[e];
#pragma unroll
        for (int e = V - 1; e >= 0; --e) h[e] = up ? (e >= s ? h[e - s] : 0.0f) : h[e];
    }
    const bool none = b >= (uint32_t)V || d >= (uint32_t)V;
#pragma unroll
    for (int e = 0; e < V; ++e) h[e] = none ? 0.0f : h[e];
}

DI uint32_t magic_div(uint32_t n, uint32_t m, uint32_t sh) {
    const uint32_t t = __umulhi(m, n);
    return (t + ((n - t) >> (sh & 0xFF))) >> (sh >> 8);
}

struct Row {            // where a row starts in the three tensors
    const char *a, *b;
    char *y;
    int shift;          // elements of its first line of the output that belong to what stands before it
    bool ok;            // (blocked order, last block: the row exists; where it does not, the addresses are those of the last one)
};
template <int BF16, bool MASK> DI Row place(const dvm_softmax_args &s, uint32_t set, uint32_t row) {
    constexpr int ES = BF16 ? 2 : 4;
    const uint32_t q = magic_div(row, s.m1, s.sh1);
    uint32_t i1 = row - q * s.d1;
    const uint32_t i3 = magic_div(q, s.m2, s.sh2), i2 = q - i3 * s.d2;
    const bool ok = s.limit == 0 || i1 + i3 * s.d1 < s.limit;
    i1 = ok ? i1 : s.limit - 1u - i3 * s.d1;
    uint64_t pa = (uint64_t)(uintptr_t)s.a, pb = (uint64_t)(uintptr_t)s.b, py = (uint64_t)(uintptr_t)s.y;
    if (s.sets != 0) {
        // (the addresses of a stack's alike parts are in the argument block, which is memory like any other)
        uint64_t table = s.sets;
        if (table == DVM_SOFTMAX_PARTS) table = (uint64_t)(uintptr_t)__builtin_amdgcn_kernarg_segment_ptr() + offsetof(dvm_softmax_alike, parts);
        const GLOBAL_AS uint64_t *t = (const GLOBAL_AS uint64_t *)table + (uint64_t)set * s.n_tensors;
        pa = t[s.ia];
        if constexpr (MASK) pb = t[s.ib];
        py = t[s.iy];
    }
    Row r;
    r.a = (const char *)pa + ((int64_t)i1 * s.a_s[0] + (int64_t)i2 * s.a_s[1] + (int64_t)i3 * s.a_s[2]) * ES;
    r.b = MASK ? (const char *)pb + ((int64_t)i1 * s.b_s[0] + (int64_t)i2 * s.b_s[1] + (int64_t)i3 * s.b_s[2]) * ES : nullptr;
    r.y = (char *)py + ((int64_t)i1 * s.y_s[0] + (int64_t)i2 * s.y_s[1] + (int64_t)i3 * s.y_s[2]) * ES;
    r.shift = (int)(((uint32_t)(uintptr_t)r.y & 127u) / ES);
    r.shift = s.shifted != 0 ? r.shift : 0;
    r.ok = ok;
    return r;
}

template <int V> DI float sum_of(const float *p) {
    float v = (p[0] + p[1]) + (p[2] + p[3]);
    if constexpr (V == 8) v += (p[4] + p[5]) + (p[6] + p[7]);
    return v;
}
// The classes of a row lie `shift` places behind the lanes that summed them.  acc: this lane's sums of its V classes, `at` the first of them;
// returns the lane's part of the row's sum with the classes in their order.  rot: T * V floats of this row's LDS.
template <int V, int T> DI float in_order(const float *acc, int at, int shift, float *rot) {
#pragma unroll
    for (int e = 0; e < V; ++e) rot[(uint32_t)(at + e - shift) & (uint32_t)(T * V - 1)] = acc[e];
    if constexpr (T > 64) {
        __syncthreads();
    } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    float p[V];
#pragma unroll
    for (int e = 0; e < V; ++e) p[e] = rot[at + e];
    if constexpr (T <= 64) {        // (the next row's sums come only after these reads)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    return sum_of<V>(p);
}
// The same through 2 * T floats of LDS, which the whole workgroup shares: one class of every lane at a time.
template <int V, int T> DI float in_order_narrow(float *acc, uint32_t tid, int shift, float *rot) {
    const uint32_t b = (uint32_t)shift & (V - 1), a = (uint32_t)shift / V;
#pragma unroll
    for (uint32_t s = 1; s < (uint32_t)V; s *= 2) {        // acc[e] = acc[(e + b) % V]
        const bool turn = (b & s) != 0;
        float t[V];
#pragma unroll
        for (int e = 0; e < V; ++e) t[e] = acc[(e + (int)s) & (V - 1)];
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] = turn ? t[e] : acc[e];
    }
    float p[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        float *plane = rot + (e & 1) * T;
        plane[(tid - a - ((uint32_t)e + b >= (uint32_t)V ? 1u : 0u)) & (uint32_t)(T - 1)] = acc[e];
        __syncthreads();            // (a plane is written again two barriers after it was)
        p[e] = plane[tid];
    }
    return sum_of<V>(p);
}

// ---- rows of up to NR * T * V columns (less the shift), T lanes on a row --------------------------------------------------
// Tiles `first` to `end`, `step` apart (one alone is written so too: outside a loop the compiler makes one vector of a lane's chunks and waits for
// the first of them before it asks for the next, fp32 [1000, 16384] in 1024 lanes of 4 chunks 28.0 -> 28.8 us).  rot: BLOCK * V floats of LDS, red: two for every wave.  HALF: a launch's rows have more than NR / 2 chunks a lane, so that many are not asked for.
template <int BF16, int T, int NR, bool MASK, bool HALF> DI void rows_of(const dvm_softmax_args &s, uint32_t first, uint32_t end, uint32_t step, float *rot, float *red) {
    constexpr int V = BF16 ? 8 : 4, ES = BF16 ? 2 : 4, W = T * V, BLOCK = T < 256 ? 256 : T, RP = BLOCK / T;
    constexpr int GW = T > 64 ? T / 64 : 1;             // waves on a row
    constexpr int SURE = HALF ? NR / 2 : 0;
    float *red0 = red, *red1 = red + BLOCK / 64;
    const uint32_t tid = threadIdx.x;
    const uint32_t g = tid / T, l = tid % T;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid) >> 6;
    const int cols = (int)s.cols, cmax = cols - V;
    const bool shifted = s.shifted != 0;
    const int at = (int)l * V;
    for (uint32_t tile = first; tile < end; tile += step) {
        const uint32_t set = s.sets != 0 ? magic_div(tile, s.set_m, s.set_sh) : 0u;
        uint32_t row = (tile - set * s.set_tiles) * RP + (T >= 64 ? wave / GW : g);
        const bool in = row < s.rows;
        row = in ? row : s.rows - 1u;
        const Row r = place<BF16, MASK>(s, set, row);
        const bool ok = in && r.ok;
        const int c_first = at - r.shift;
        auto col = [&](int c0) { const int c = c0 < cmax ? c0 : cmax; return c > 0 ? c : 0; };
        u32x4 raw[NR], rawb[MASK ? NR : 1];
        if (s.stream != 0) {        // (the same for every lane)
#pragma unroll
            for (int j = 0; j < NR; ++j)
                if (j < SURE || j < (int)s.slots) raw[j] = load16<true>(r.a + (int64_t)col(c_first + j * W) * ES);
            STREAMING();
        } else {
#pragma unroll
            for (int j = 0; j < NR; ++j)
                if (j < SURE || j < (int)s.slots) raw[j] = load16<false>(r.a + (int64_t)col(c_first + j * W) * ES);
        }
        if constexpr (MASK) {
#pragma unroll
            for (int j = 0; j < NR; ++j)
                if (j < SURE || j < (int)s.slots) rawb[j] = load16<false>(r.b + (int64_t)col(c_first + j * W) * ES);
        }
        float v[NR][V];
        float m = NEG_INF;
#pragma unroll
        for (int j = 0; j < NR; ++j)
            if (j < SURE || j < (int)s.slots) {
                widen<BF16>(v[j], raw[j]);
                if constexpr (MASK) {
                    float b[V];
                    widen<BF16>(b, rawb[j]);
#pragma unroll
                    for (int e = 0; e < V; ++e) v[j][e] += b[e];
                }
#pragma unroll
                for (int e = 0; e < V; ++e) m = maxp(m, v[j][e]);
            }
        m = group_all<true, T>(m);
        if constexpr (T > 64) {
            red0[wave] = m;
            __syncthreads();
            const float *w = red0 + wave / GW * GW;
            m = w[0];
#pragma unroll
            for (int i = 1; i < GW; ++i) m = maxp(m, w[i]);
        }
        float acc[V];
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] = 0.0f;
#pragma unroll
        for (int j = 0; j < NR; ++j)
            if (j < SURE || j < (int)s.slots) {
#pragma unroll
                for (int e = 0; e < V; ++e) v[j][e] = __builtin_amdgcn_exp2f((v[j][e] - m) * LOG2E);
                if ((j == 0 && shifted) || j >= (int)s.tail) {        // (the same for every lane)
                    float h[V];
#pragma unroll
                    for (int e = 0; e < V; ++e) h[e] = v[j][e];
                    to_classes<V>(h, c_first + j * W, cmax);
#pragma unroll
                    for (int e = 0; e < V; ++e) acc[e] += h[e];
                } else {
#pragma unroll
                    for (int e = 0; e < V; ++e) acc[e] += v[j][e];
                }
            }
        float sum;
        if (shifted) sum = in_order<V, T>(acc, at, r.shift, rot + g * W);
        else sum = sum_of<V>(acc);
        sum = group_all<false, T>(sum);
        if constexpr (T > 64) {
            red1[wave] = sum;
            __syncthreads();
            const float *w = red1 + wave / GW * GW;
            sum = w[0];
#pragma unroll
            for (int i = 1; i < GW; ++i) sum += w[i];
        }
        const float scale = __builtin_amdgcn_rcpf(sum);
#pragma unroll
        for (int j = 0; j < NR; ++j)
            if (j < SURE || j < (int)s.slots) {
                const int c0 = c_first + j * W;
                if (ok && c0 > -V && c0 < cols) store16(r.y + (int64_t)col(c0) * ES, narrow<BF16>(v[j], scale));
            }
    }
}
template <int BF16, int T, int NR, bool MASK>
__global__ void __launch_bounds__(T < 256 ? 256 : T) dvm_softmax_rows(const dvm_softmax_alike a) {
    constexpr int V = BF16 ? 8 : 4, BLOCK = T < 256 ? 256 : T;
    __shared__ __align__(16) float rot[BLOCK * V];
    __shared__ float red[2 * (BLOCK / 64)];
    rows_of<BF16, T, NR, MASK, true>(a.s, blockIdx.x, a.s.tiles, gridDim.x, rot, red);
}

// ---- longer rows: a workgroup of T = 512 or 1024 threads holds one --------------------------------------------------------
// The row is read once: NR slots of it stay in registers, the rest (s.slots - NR of T * 16 bytes) in LDS.  The loads of the next row follow the
// stores slot by slot, so that only the exponentials of a row run without memory traffic of its own workgroup.
// (fp32 rows of 33 slots leave LDS for one class of every lane at a time only; more barriers)
constexpr bool long_narrow(bool bf16, int nr) { return !bf16 && nr == 24; }
// Src: the launch's rows, of one softmax or of several.
template <int BF16, int T, int NR, bool MASK, class Src> DI void long_rows(const Src &src, float *lds) {
    constexpr int V = BF16 ? 8 : 4, ES = BF16 ? 2 : 4, W = T * V, NW = T / 64;
    constexpr bool NARROW = long_narrow(BF16, NR);
    constexpr int ROT = NARROW ? 2 * T : W;
    // lds: ROT floats for the classes, 32 for the waves, then the row's slots from NR on
    float *rot = lds, *red = lds + ROT;
    u32x4 *stash = (u32x4 *)(lds + ROT + 32);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid) >> 6;
    const int at = (int)tid * V;
    auto col = [&](int c0, int cmax) { const int c = c0 < cmax ? c0 : cmax; return c > 0 ? c : 0; };
    auto placed = [&](uint32_t part, uint32_t tile) {
        const dvm_softmax_args &s = src.args(part);
        tile -= src.first(part);
        const uint32_t set = s.sets != 0 ? magic_div(tile, s.set_m, s.set_sh) : 0u;
        return place<BF16, MASK>(s, set, tile - set * s.set_tiles);
    };
    // what a lane does with a chunk: its values (of the sum, where there is a second tensor)
    auto values = [&](float *v, u32x4 raw, const Row &r, int c0, int cmax) {
        widen<BF16>(v, raw);
        if constexpr (MASK) {
            float b[V];
            widen<BF16>(b, load16<false>(r.b + (int64_t)col(c0, cmax) * ES));
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] += b[e];
        }
    };
    u32x4 raw[NR];
    uint32_t tile = blockIdx.x;
    if (tile >= src.tiles()) return;
    uint32_t part = src.part_of(tile, 0u);
    Row r = placed(part, tile);
#pragma unroll
    for (int j = 0; j < NR; ++j)
        if (j < (int)src.args(part).slots) raw[j] = load16<true>(r.a + (int64_t)col(at - r.shift + j * W, (int)src.args(part).cols - V) * ES);
    for (;;) {
        const dvm_softmax_args &s = src.args(part);
        const int cols = (int)s.cols, cmax = cols - V, n_slots = (int)s.slots;
        const bool shifted = s.shifted != 0;
        const int c_first = at - r.shift;
        float m = NEG_INF;
        for (int j = NR; j < n_slots; ++j) {
            const u32x4 w = load16<true>(r.a + (int64_t)col(c_first + j * W, cmax) * ES);
            stash[(j - NR) * T + tid] = w;
            float v[V];
            values(v, w, r, c_first + j * W, cmax);
#pragma unroll
            for (int e = 0; e < V; ++e) m = maxp(m, v[e]);
        }
#pragma unroll
        for (int j = 0; j < NR; ++j)
            if (j < n_slots) {
                float v[V];
                values(v, raw[j], r, c_first + j * W, cmax);
#pragma unroll
                for (int e = 0; e < V; ++e) m = maxp(m, v[e]);
            }
        m = group_all<true, 64>(m);
        red[wave] = m;
        __syncthreads();
        m = lane_of(group_all<true, NW>(red[lane & (NW - 1u)]), 0);
        float acc[V];
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] = 0.0f;
        auto take = [&](float *v, int j) {
            if ((j == 0 && shifted) || j >= (int)s.tail) to_classes<V>(v, c_first + j * W, cmax);
#pragma unroll
            for (int e = 0; e < V; ++e) acc[e] += v[e];
        };
        auto exps = [&](float *v) {
#pragma unroll
            for (int e = 0; e < V; ++e) v[e] = __builtin_amdgcn_exp2f((v[e] - m) * LOG2E);
        };
#pragma unroll
        for (int j = 0; j < NR; ++j)
            if (j < n_slots) {
                float v[V];
                values(v, raw[j], r, c_first + j * W, cmax);
                exps(v);
                if constexpr (!BF16) raw[j] = narrow<0>(v, 1.0f);       // (fp32 exponentials are kept, bf16 rows are taken from their inputs again)
                take(v, j);
            }
        for (int j = NR; j < n_slots; ++j) {
            float v[V];
            values(v, stash[(j - NR) * T + tid], r, c_first + j * W, cmax);
            exps(v);
            if constexpr (!BF16) stash[(j - NR) * T + tid] = narrow<0>(v, 1.0f);
            take(v, j);
        }
        float sum;
        if (!shifted) sum = sum_of<V>(acc);
        else if constexpr (NARROW) sum = in_order_narrow<V, T>(acc, tid, r.shift, rot);
        else sum = in_order<V, T>(acc, at, r.shift, rot);
        red[16 + wave] = group_all<false, 64>(sum);
        __syncthreads();
        const float scale = __builtin_amdgcn_rcpf(lane_of(group_all<false, NW>(red[16 + (lane & (NW - 1u))]), 0));
        auto put = [&](u32x4 w, int j) {
            const int c0 = c_first + j * W;
            float v[V];
            if constexpr (BF16) {
                values(v, w, r, c0, cmax);
                exps(v);
            } else {
                widen<0>(v, w);
            }
            if (r.ok && c0 > -V && c0 < cols) store16(r.y + (int64_t)col(c0, cmax) * ES, narrow<BF16>(v, scale));
        };
        for (int j = NR; j < n_slots; ++j) put(stash[(j - NR) * T + tid], j);
        const uint32_t next = tile + gridDim.x;
        const bool last = next >= src.tiles();      // (the same for every lane)
        const uint32_t next_part = last ? part : src.part_of(next, part);
        const Row n = placed(next_part, last ? tile : next);
        const int next_slots = last ? 0 : (int)src.args(next_part).slots, next_cmax = (int)src.args(next_part).cols - V;
#pragma unroll
        for (int j = 0; j < NR; ++j) {
            if (j < n_slots) put(raw[j], j);
            if (j < next_slots) raw[j] = load16<true>(n.a + (int64_t)col(at - n.shift + j * W, next_cmax) * ES);
        }
        if (last) break;
        tile = next;
        part = next_part;
        r = n;
    }
}

struct OneSoftmax {
    const dvm_softmax_args &s;
    DI uint32_t tiles() const { return s.tiles; }
    DI uint32_t part_of(uint32_t, uint32_t) const { return 0; }
    DI uint32_t first(uint32_t) const { return 0; }
    DI const dvm_softmax_args &args(uint32_t) const { return s; }
};
template <int BF16, int T, int NR, bool MASK>
__global__ void __launch_bounds__(T) dvm_softmax_long(const dvm_softmax_alike a) {
    extern __shared__ __align__(16) float lds[];
    long_rows<BF16, T, NR, MASK>(OneSoftmax{a.s}, lds);
}

// ---- several softmaxes in one launch --------------------------------------------------------------------------------------
// Independent parts of a stack.  Few rows leave most of the chip idle, and a launch for each is one after the other: eight unlike ones of fp32
// [16, 100003] 156 us so, 48 in the interpreter and 25 here; bf16 [32, 17000] 43, 18 and 6.7; fp32 [600, 8192] 82, 65 and 55.  A workgroup takes its
// tile's part from the argument block; the arithmetic of a row is that of a launch of its own.  One kernel for all rows of up to 256 lanes, with a lane's
// most chunks (alike ones have the kernel for theirs: eight of bf16 [6000, 751] 24 there and 28 here), one for 512 lanes, and those for long rows.
struct ManySoftmaxes {
    const dvm_softmax_mixed &p;
    DI uint32_t tiles() const { return p.first[p.n]; }
    DI uint32_t part_of(uint32_t tile, uint32_t from) const {
        while (tile >= p.first[from + 1]) ++from;
        return from;
    }
    DI uint32_t first(uint32_t part) const { return p.first[part]; }
    DI const dvm_softmax_args &args(uint32_t part) const { return p.part[part]; }
};
template <int BF16, bool MASK> __global__ void __launch_bounds__(256) dvm_softmax_mixed_rows(const dvm_softmax_mixed p) {
    constexpr int V = BF16 ? 8 : 4, NR = BF16 ? 6 : 8;
    __shared__ __align__(16) float rot[256 * V];
    __shared__ float red[8];
    const uint32_t part = ManySoftmaxes{p}.part_of(blockIdx.x, 0u), tile = blockIdx.x - p.first[part], all = p.first[p.n];
    const dvm_softmax_args &s = p.part[part];
    switch (s.lanes) {
        case 8: rows_of<BF16, 8, NR, MASK, false>(s, tile, s.tiles, all, rot, red); break;
        case 16: rows_of<BF16, 16, NR, MASK, false>(s, tile, s.tiles, all, rot, red); break;
        case 32: rows_of<BF16, 32, NR, MASK, false>(s, tile, s.tiles, all, rot, red); break;
        case 64: rows_of<BF16, 64, NR, MASK, false>(s, tile, s.tiles, all, rot, red); break;
        case 128: rows_of<BF16, 128, NR, MASK, false>(s, tile, s.tiles, all, rot, red); break;
        case 256: rows_of<BF16, 256, NR, MASK, false>(s, tile, s.tiles, all, rot, red); break;
        default: break;
    }
}
template <int BF16, int T, int NR, bool MASK> __global__ void __launch_bounds__(T) dvm_softmax_mixed_long(const dvm_softmax_mixed p) {
    extern __shared__ __align__(16) float lds[];
    long_rows<BF16, T, NR, MASK>(ManySoftmaxes{p}, lds);
}
template <int BF16, bool MASK> __global__ void __launch_bounds__(512) dvm_softmax_mixed_wide(const dvm_softmax_mixed p) {
    constexpr int V = BF16 ? 8 : 4, NR = BF16 ? 6 : 8, T = 512;
    __shared__ __align__(16) float rot[T * V];
    __shared__ float red[2 * (T / 64)];
    const uint32_t part = ManySoftmaxes{p}.part_of(blockIdx.x, 0u), tile = blockIdx.x - p.first[part], all = p.first[p.n];
    const dvm_softmax_args &s = p.part[part];
    rows_of<BF16, T, NR, MASK, false>(s, tile, s.tiles, all, rot, red);
}

// ---- rows as the interpreter lays them out --------------------------------------------------------------------------------
// Smaller programs with a launch to themselves (bf16 [3200, 13] 12.6 -> 11.6 us a call, [32000, 120] 12.6 -> 11.5: less to fetch and no decoding).  The chunks of a row start with the row, G lanes hold it as in the segment's plan, and everything is
// added in the interpreter's order -- a lane's elements one after the other (where the row does not fill the tile: chunk by chunk), then the lanes --
// so that the bits are the interpreter's, whichever of the two a launch runs in.  G: 1 to 64.  PART: rows narrower than a chunk, one lane each.
template <int BF16, int NR, bool MASK, bool PART>
__global__ void __launch_bounds__(256) dvm_softmax_exact(const dvm_softmax_args s) {
    constexpr int V = BF16 ? 8 : 4, ES = BF16 ? 2 : 4;
    const uint32_t G = s.lanes, lg = s.log2_lanes;
    const uint32_t g = threadIdx.x >> lg, l = threadIdx.x & (G - 1u), RP = 256u >> lg;
    const int cols = (int)s.cols, cmax = cols - V, W = (int)G * V;
    auto value = [&](const char *p) {       // one element
        if constexpr (BF16) return bf16_lo(*(const GLOBAL_AS uint16_t *)p);
        else return *(const GLOBAL_AS float *)p;
    };
    auto all = [&]<bool MAX>(float v) {     // over the G lanes of a row
        if (G >= 2) v = comb<MAX>(v, dpp<0xB1>(v));
        if (G >= 4) v = comb<MAX>(v, dpp<0x4E>(v));
        if (G >= 8) v = comb<MAX>(v, dpp<0x141>(v));
        if (G >= 16) v = comb<MAX>(v, dpp<0x140>(v));
        if (G >= 32) v = comb<MAX>(v, __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), 0x401F)));
        if (G >= 64) v = comb<MAX>(lane_of(v, 0), lane_of(v, 32));
        return v;
    };
    for (uint32_t tile = blockIdx.x; tile < s.tiles; tile += gridDim.x) {
        const uint32_t set = s.sets != 0 ? magic_div(tile, s.set_m, s.set_sh) : 0u;
        uint32_t row = (tile - set * s.set_tiles) * RP + g;
        const bool ok = row < s.rows;
        row = ok ? row : s.rows - 1u;
        const Row r = place<BF16, MASK>(s, set, row);
        float v[NR][V];
        if constexpr (PART) {
#pragma unroll
            for (int e = 0; e < V; ++e) v[0][e] = value(r.a + (e < cols ? e : 0) * ES);
            if constexpr (MASK) {
#pragma unroll
                for (int e = 0; e < V; ++e) v[0][e] += value(r.b + (e < cols ? e : 0) * ES);
            }
        } else {
            u32x4 raw[NR], rawb[MASK ? NR : 1];
            auto at = [&](int j) { const int c = (int)l * V + j * W; return (int64_t)(c < cmax ? c : cmax) * ES; };
#pragma unroll
            for (int j = 0; j < NR; ++j)
                if (j < NR / 2 || j < (int)s.slots) raw[j] = load16<false>(r.a + at(j));
            if constexpr (MASK) {
#pragma unroll
                for (int j = 0; j < NR; ++j)
                    if (j < NR / 2 || j < (int)s.slots) rawb[j] = load16<false>(r.b + at(j));
            }
#pragma unroll
            for (int j = 0; j < NR; ++j)
                if (j < NR / 2 || j < (int)s.slots) {
                    widen<BF16>(v[j], raw[j]);
                    if constexpr (MASK) {
                        float b[V];
                        widen<BF16>(b, rawb[j]);
#pragma unroll
                        for (int e = 0; e < V; ++e) v[j][e] += b[e];
                    }
                }
        }
        float m = NEG_INF;
#pragma unroll
        for (int j = 0; j < NR; ++j)
            if (j < NR / 2 || j < (int)s.slots) {
#pragma unroll
                for (int e = 0; e < V; ++e) m = maxp(m, PART && e >= cols ? NEG_INF : v[j][e]);
            }
        m = all.template operator()<true>(m);
        float sum = 0.0f;
#pragma unroll
        for (int j = 0; j < NR; ++j)
            if (j < NR / 2 || j < (int)s.slots) {
#pragma unroll
                for (int e = 0; e < V; ++e) v[j][e] = __builtin_amdgcn_exp2f((v[j][e] - m) * LOG2E);
                if constexpr (PART) {
#pragma unroll
                    for (int e = 0; e < V; ++e) sum += e < cols ? v[j][e] : 0.0f;
                } else if (s.ragged == 0) {         // (the same for every lane)
#pragma unroll
                    for (int e = 0; e < V; ++e) sum += v[j][e];
                } else {
                    const int c0 = (int)l * V + j * W, dup = c0 - cmax;         // elements that a chunk which slid back repeats
                    float c = 0.0f;
                    if (j < (int)s.tail) {          // (a slot that lies inside the row)
#pragma unroll
                        for (int e = 0; e < V; ++e) c += v[j][e];
                    } else {
#pragma unroll
                        for (int e = 0; e < V; ++e) c += e >= dup ? v[j][e] : 0.0f;
                    }
                    sum += c0 < cols ? c : 0.0f;
                }
            }
        const float scale = __builtin_amdgcn_rcpf(all.template operator()<false>(sum));
        if constexpr (PART) {
#pragma unroll
            for (int e = 0; e < V; ++e)
                if (ok && e < cols) {
                    if constexpr (BF16) *(GLOBAL_AS uint16_t *)(r.y + e * ES) = (uint16_t)pack_bf16x2(v[0][e] * scale, 0.0f);
                    else *(GLOBAL_AS float *)(r.y + e * ES) = v[0][e] * scale;
                }
        } else {
#pragma unroll
            for (int j = 0; j < NR; ++j)
                if (j < NR / 2 || j < (int)s.slots) {
                    const int c0 = (int)l * V + j * W;
                    if (ok && c0 < cols) store16(r.y + (int64_t)(c0 < cmax ? c0 : cmax) * ES, narrow<BF16>(v[j], scale));
                }
        }
    }
}
template <int BF16, bool MASK> int launch_exact(const dvm_softmax_args &s, unsigned grid, hipStream_t q) {
#define GO(NR, PART) hipLaunchKernelGGL((dvm_softmax_exact<BF16, NR, MASK, PART>), dim3(grid), dim3(256), 0, q, s)
    if (s.cols < (BF16 ? 8u : 4u)) GO(1, true);
    else if (s.slots <= 1) GO(1, false);
    else if (s.slots <= 2) GO(2, false);
    else if (s.slots <= 4) GO(4, false);
    else GO(8, false);
#undef GO
    return (int)hipGetLastError();
}

template <int BF16, int T, bool MASK> int launch_rows(const dvm_softmax_alike &a, unsigned grid, hipStream_t q) {
    constexpr unsigned BLOCK = T < 256 ? 256 : T;
    const dvm_softmax_args &s = a.s;
    if (s.slots <= 2) hipLaunchKernelGGL((dvm_softmax_rows<BF16, T, 2, MASK>), dim3(grid), dim3(BLOCK), 0, q, a);
    else if (s.slots <= 4) hipLaunchKernelGGL((dvm_softmax_rows<BF16, T, 4, MASK>), dim3(grid), dim3(BLOCK), 0, q, a);
    else hipLaunchKernelGGL((dvm_softmax_rows<BF16, T, BF16 ? 6 : 8, MASK>), dim3(grid), dim3(BLOCK), 0, q, a);
    return (int)hipGetLastError();
}
// LDS of a launch whose longest rows have `slots`, and of the longest rows that its kernel takes
template <int BF16, int T, int NR> constexpr unsigned long_lds(unsigned slots) {
    return ((long_narrow(BF16, NR) ? 2 : BF16 ? 8 : 4) * T + 32) * 4u + (slots > NR ? (slots - NR) * (unsigned)T * 16u : 0u);
}
template <int BF16, int T, int NR> constexpr unsigned long_most() { return long_lds<BF16, T, NR>(BF16 ? NR : T == 512 ? (NR == 16 ? 16 : 24) : NR == 20 ? 28 : 33); }
// (the bound on a kernel's LDS is the process's: always the same, whichever thread launches)
template <unsigned MOST> int raise_lds(const void *kernel) {
    if constexpr (MOST > 65536u) return (int)hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)MOST);
    return 0;
}
template <int BF16, int T, int NR, bool MASK> int launch_long(const dvm_softmax_alike &a, unsigned grid, hipStream_t q) {
    const int e = raise_lds<long_most<BF16, T, NR>()>((const void *)dvm_softmax_long<BF16, T, NR, MASK>);
    if (e != 0) return e;
    hipLaunchKernelGGL((dvm_softmax_long<BF16, T, NR, MASK>), dim3(grid), dim3(T), (long_lds<BF16, T, NR>(a.s.slots)), q, a);
    return (int)hipGetLastError();
}
template <int BF16, int T, int NR, bool MASK> int launch_long(const dvm_softmax_mixed &p, unsigned slots, unsigned grid, hipStream_t q) {
    const int e = raise_lds<long_most<BF16, T, NR>()>((const void *)dvm_softmax_mixed_long<BF16, T, NR, MASK>);
    if (e != 0) return e;
    hipLaunchKernelGGL((dvm_softmax_mixed_long<BF16, T, NR, MASK>), dim3(grid), dim3(T), (long_lds<BF16, T, NR>(slots)), q, p);
    return (int)hipGetLastError();
}
template <int BF16, bool MASK> int launch_any(const dvm_softmax_alike &a, unsigned grid, hipStream_t q) {
    const dvm_softmax_args &s = a.s;
    if (s.lanes == 8) return launch_rows<BF16, 8, MASK>(a, grid, q);
    if (s.lanes == 16) return launch_rows<BF16, 16, MASK>(a, grid, q);
    if (s.lanes == 32) return launch_rows<BF16, 32, MASK>(a, grid, q);
    if (s.lanes == 64) return launch_rows<BF16, 64, MASK>(a, grid, q);
    if (s.lanes == 128) return launch_rows<BF16, 128, MASK>(a, grid, q);
    if (s.lanes == 256) return launch_rows<BF16, 256, MASK>(a, grid, q);
    if (s.in_long == 0) return launch_rows<BF16, 512, MASK>(a, grid, q);
    if (s.lanes == 512) {
        if constexpr (BF16) if (s.slots <= 8) return launch_long<BF16, 512, 8, MASK>(a, grid, q);
        if (s.slots <= 16) return launch_long<BF16, 512, 16, MASK>(a, grid, q);
        if constexpr (!BF16) return launch_long<BF16, 512, 20, MASK>(a, grid, q);
    }
    if (BF16 || s.slots <= 28) return launch_long<BF16, 1024, 20, MASK>(a, grid, q);
    if constexpr (!BF16) return launch_long<BF16, 1024, 24, MASK>(a, grid, q);
    return (int)hipErrorInvalidValue;
}
template <int BF16, bool MASK> int launch_mixed(const dvm_softmax_mixed &p, unsigned grid, hipStream_t q) {
    const dvm_softmax_args &s = p.part[0];
    unsigned slots = 0;
    for (uint32_t i = 0; i < p.n; ++i) slots = p.part[i].slots > slots ? p.part[i].slots : slots;
    if (s.lanes <= 256) hipLaunchKernelGGL((dvm_softmax_mixed_rows<BF16, MASK>), dim3(grid), dim3(256), 0, q, p);
    else if (s.in_long == 0) hipLaunchKernelGGL((dvm_softmax_mixed_wide<BF16, MASK>), dim3(grid), dim3(512), 0, q, p);
    else if (s.lanes == 512) return launch_long<BF16, 512, BF16 ? 16 : 20, MASK>(p, slots, grid, q);
    else if (BF16 || slots <= 28) return launch_long<BF16, 1024, 20, MASK>(p, slots, grid, q);
    else if constexpr (!BF16) return launch_long<BF16, 1024, 24, MASK>(p, slots, grid, q);
    return (int)hipGetLastError();
}

}  // namespace

extern "C" int dvm_softmax_launch(const dvm_softmax_alike *a, unsigned grid, void *stream) {
    const hipStream_t q = (hipStream_t)stream;
    const dvm_softmax_args &s = a->s;
    if (s.exact) {
        if (s.bf16) return s.b ? launch_exact<1, true>(s, grid, q) : launch_exact<1, false>(s, grid, q);
        return s.b ? launch_exact<0, true>(s, grid, q) : launch_exact<0, false>(s, grid, q);
    }
    if (s.bf16) return s.b ? launch_any<1, true>(*a, grid, q) : launch_any<1, false>(*a, grid, q);
    return s.b ? launch_any<0, true>(*a, grid, q) : launch_any<0, false>(*a, grid, q);
}
extern "C" int dvm_softmax_launch_mixed(const dvm_softmax_mixed *p, unsigned grid, void *stream) {
    const hipStream_t q = (hipStream_t)stream;
    const dvm_softmax_args &s = p->part[0];
    if (s.bf16) return s.b ? launch_mixed<1, true>(*p, grid, q) : launch_mixed<1, false>(*p, grid, q);
    return s.b ? launch_mixed<0, true>(*p, grid, q) : launch_mixed<0, false>(*p, grid, q);
}
