// The device side of libdvm: the bytecode interpreter kernel for gfx950 and dvm_run.
//
// One workgroup plays the role of one "AI Core" of Algorithm 2 (Section 4.3): it takes a
// contiguous range of tiles, and for every tile walks the code body from its first record to
// CodeSize, dispatching each record on its instruction id.  Decoding is wave-uniform: the
// bytecode sits in the kernel-argument segment and is read with scalar loads into SGPRs, the
// dispatch is a scalar branch tree, so no vector lane ever spends an issue slot on decoding
// (the GPU analogue of decoding on the NPU's Scalar unit, Section 4.3).
//
// Local memory of the paper's AI Core = the vector register file here.  A tile register is K
// fp32 values per lane; the accumulator ACC and the registers R0..R(NR-1) hold fused
// intermediates, which therefore never touch HBM (Section 5.1, vector-vector fusion).  Every
// register reference in a handler is a compile-time constant: handlers are selected by scalar
// switches on the register ids, because a GPU cannot index vector registers dynamically.
//
// Layout of a tile: RP rows x up to G*nvec*V columns.  Row r of the tile is held by the G
// lanes [r*G, (r+1)*G); lane l of the group owns the chunks of V consecutive elements number
// l, l+G, l+2G, ... so that each load instruction of a wave covers whole contiguous runs of
// 16 bytes per lane.  Loads/stores do all address arithmetic (strides, broadcast, views), so
// compute instructions see one canonical layout (Section 4.1, last paragraph).
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>
#include <atomic>
#include <mutex>
#include <utility>

#include "../../include/dvm.h"
#include "dvm_bytecode.h"
#include "dvm_internal.h"

using namespace dvmbc;

namespace {

constexpr int CODE_WORDS = DVM_CODE_MAX_BYTES / 4;
[[maybe_unused]] constexpr int MAX_SEGMENTS = CODE_WORDS / SH_WORDS;

struct KArgs {
    uint32_t code[CODE_WORDS];          // the segments of this launch (headers + bodies)
    uint64_t tensors[DVM_MAX_TENSORS];  // device addresses
    uint64_t ws;                        // the launch's workspace (0: none)
    uint32_t nseg;
    uint32_t spin_limit;                // polls a workgroup spends at a grid-wide synchronisation point before it gives up
    uint64_t sets;                      // batched launch: device array of n_sets * n_tensors addresses (0: `tensors` above)
    uint32_t n_sets;                    // times the program runs, each time on the next set of tensors (at least 1)
    uint32_t n_tensors;
    uint32_t rotate;                    // not 0: every segment deals its tiles out starting at the workgroup after the one the
                                        // segment before stopped at (short segments then do not all land on the first workgroups);
                                        // 1: all of them round-robin, so that workgroup b runs the tiles b, b + N, b + 2N, .. of the
                                        // whole launch, counted over its segments and sets
    uint32_t set_tiles;                 // rotate = 1: tiles of one set (of this launch's segments), and the multiply-shift constants
    uint32_t set_m, set_sh;             // that divide by it
    uint32_t aliased;                   // 1: some segment's output shares memory with another tensor of that segment
};

#define DI __device__ __forceinline__
#define LI __attribute__((always_inline))

// Compile-time loop: f.operator()<I>() for I = 0..N-1.  Every register-array index in this file
// is a template constant, so that the arrays are split into scalar registers before any other
// optimisation can merge the handlers of different registers into one body with a run-time index.
template <class F, int... I> DI void sfor_impl(F &f, std::integer_sequence<int, I...>) {
    (f.template operator()<I>(), ...);
}
template <int N, class F> DI void sfor(F &&f) { sfor_impl(f, std::make_integer_sequence<int, N>{}); }

// ------------------------------------------------------------------------------------------
// scalar math on fp32 lanes
// ------------------------------------------------------------------------------------------
DI float f_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
DI float f_log2(float x) { return __builtin_amdgcn_logf(x); }
DI float f_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
DI float f_rsq(float x) { return __builtin_amdgcn_rsqf(x); }
DI float f_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
DI float f_fma(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
DI float f_mul_sub(float a, float b, float c) {        // a * b rounded, then - c
#pragma clang fp contract(off)
    const float p = a * b;
    return p - c;
}
DI float f_sub_mul(float c, float a, float b) {        // c - a * b, the product rounded
#pragma clang fp contract(off)
    const float p = a * b;
    return c - p;
}
// Table 1's Max / Min are read as propagating a NaN operand (what NumPy's maximum / minimum and the frameworks
// this VM serves do).  gfx950 has that operation as one instruction (v_maximum3_f32 / v_minimum3_f32), which the
// compiler selects for the IEEE-754-2019 maximum / minimum builtins: element-wise ops and every stage of a
// reduction use it, so a NaN anywhere in a row or column reaches the result.
DI float f_maxp(float a, float b) { return __builtin_elementwise_maximum(a, b); }
DI float f_minp(float a, float b) { return __builtin_elementwise_minimum(a, b); }

constexpr float LOG2E    = 1.44269504088896340736f;
constexpr float LOG2E_LO = 1.92596303e-8f;      // log2(e) - (float)log2(e)
constexpr float LN2      = 0.69314718055994530942f;

// exp(x) = 2^(x*log2e); the rounding error of the product is carried as a first-order correction
// so that the relative error stays near 1 ulp for |x| up to the overflow threshold.
DI float f_exp(float x) {
    float t = x * LOG2E;
    float e = f_fma(x, LOG2E, -t);
    e = f_fma(x, LOG2E_LO, e);
    e = (__builtin_fabsf(x) < __builtin_inff()) ? e : 0.0f;
    float r = f_exp2(t);
    return f_fma(r, e * LN2, r);
}
DI float f_sigmoid(float x) { return f_rcp(1.0f + f_exp2(-LOG2E * x)); }
DI float f_silu(float x) { return x * f_sigmoid(x); }
// 0.5 u (1 + tanh(c (u + 0.044715 u^3)))  ==  u * sigmoid(2 c (u + 0.044715 u^3))
DI float f_gelu_tanh(float u) {
    constexpr float C0 = -2.0f * LOG2E * 0.7978845608028654f;
    constexpr float C1 = -2.0f * LOG2E * 0.7978845608028654f * 0.044715f;
    float p = u * f_fma(u * u, C1, C0);
    return u * f_rcp(1.0f + f_exp2(p));
}
DI float f_tanh(float x) {
    float a = __builtin_fabsf(x);
    float t = f_exp2(-2.0f * LOG2E * a);
    float big = (1.0f - t) * f_rcp(1.0f + t);
    float s = a * a;                               // odd Taylor series below 0.04
    float small = a * f_fma(s, f_fma(s, 0.13333333f, -0.33333333f), 1.0f);
    float r = a < 0.04f ? small : big;
    return __builtin_copysignf(r, x);
}
// erf: odd polynomial in x on |x| <= 1, 1 - exp(q(|x| - 2.5)) on 1 < |x| <= 4, 1 beyond.
// Coefficients: least-squares Chebyshev fits of erf(x)/x in x^2 on [0,1] (degree 6) and of
// log(erfc(a)) in a-2.5 on [1,4] (degree 8), converted to the monomial basis.
DI float f_erf(float x) {
    float a = __builtin_fabsf(x);
    float s = a * a;
    float p = 7.882497448008507e-05f;
    p = f_fma(p, s, -0.0008018855005502701f);
    p = f_fma(p, s, 0.005189312156289816f);
    p = f_fma(p, s, -0.02685432881116867f);
    p = f_fma(p, s, 0.11283597350120544f);
    p = f_fma(p, s, -0.3761262595653534f);
    p = f_fma(p, s, 1.1283791065216064f);
    float lo = a * p;
    float u = __builtin_fminf(a, 4.0f) - 2.5f;
    float q = 1.6140616025950294e-06f;
    q = f_fma(q, u, -1.3309389942151029e-05f);
    q = f_fma(q, u, 7.739442662568763e-05f);
    q = f_fma(q, u, -0.0004201445553917438f);
    q = f_fma(q, u, 0.0021651603747159243f);
    q = f_fma(q, u, -0.01085851714015007f);
    q = f_fma(q, u, -0.9438936114311218f);
    q = f_fma(q, u, -5.352680683135986f);
    q = f_fma(q, u, -7.806815147399902f);
    float hi = 1.0f - f_exp2(q * LOG2E);
    float r = a <= 1.0f ? lo : hi;
    r = (a != a) ? a : r;
    return __builtin_copysignf(r, x);
}
DI float f_gelu_erf(float u) { return 0.5f * u * (1.0f + f_erf(u * 0.70710678118654752f)); }
// pow(a, b) = 2^(b log2 |a|) with the sign and the special cases of the C library's pow: a finite negative base
// is defined for integer exponents only (odd ones keep the sign), pow(x, 0) = pow(1, y) = 1 for every x and y,
// pow(-1, +-inf) = 1; zeros and infinities fall out of log2 and exp2.
DI float f_pow(float a, float b) {
    // (conditions are combined with integer and / or: a logical && would become a branch that differs between lanes)
    const float aa = __builtin_fabsf(a), ab = __builtin_fabsf(b);
    float r = f_exp2(b * f_log2(aa));
    const int b_int = __builtin_truncf(b) == b;
    const float half = 0.5f * b;
    const int b_odd = b_int & (int)(__builtin_truncf(half) != half) & (int)(ab < 16777216.0f);
    const int neg_base = (__builtin_bit_cast(uint32_t, a) >> 31) != 0;
    const int no_real_power = (int)(a < 0.0f) & (int)(aa < __builtin_inff()) & (b_int ^ 1);
    r = no_real_power ? __builtin_nanf("") : r;
    r = (neg_base & b_odd) ? -r : r;
    r = ((int)(aa == 1.0f) & (int)(ab == __builtin_inff())) ? 1.0f : r;
    r = ((int)(b == 0.0f) | (int)(a == 1.0f)) ? 1.0f : r;
    return r;
}
DI float f_bf16_round(float x) {
    __bf16 h = (__bf16)x;
    return (float)h;
}

template <uint32_t U> DI float un_op(float x) {
    if constexpr (U == U_SQRT) return f_sqrt(x);
    else if constexpr (U == U_ABS) return __builtin_fabsf(x);
    else if constexpr (U == U_LOG) return f_log2(x) * LN2;
    else if constexpr (U == U_EXP) return f_exp(x);
    else if constexpr (U == U_ROUND) return __builtin_rintf(x);
    else if constexpr (U == U_FLOOR) return __builtin_floorf(x);
    else if constexpr (U == U_ISFINITE) return (__builtin_fabsf(x) < __builtin_inff()) ? 1.0f : 0.0f;
    else if constexpr (U == U_NEG) return -x;
    else if constexpr (U == U_RSQRT) return f_rsq(x);
    else if constexpr (U == U_RCP) return f_rcp(x);
    else if constexpr (U == U_TANH) return f_tanh(x);
    else if constexpr (U == U_ERF) return f_erf(x);
    else if constexpr (U == U_SIGMOID) return f_sigmoid(x);
    else if constexpr (U == U_SQUARE) return x * x;
    else if constexpr (U == U_GELU_TANH) return f_gelu_tanh(x);
    else if constexpr (U == U_GELU_ERF) return f_gelu_erf(x);
    else if constexpr (U == U_SILU) return f_silu(x);
    else if constexpr (U == U_CAST_BF16) return f_bf16_round(x);
    else return x;
}

template <uint32_t B> DI float bin_op(float a, float b) {
    if constexpr (B == B_NONE) return b;
    else if constexpr (B == B_ADD) return a + b;
    else if constexpr (B == B_SUB) return a - b;
    else if constexpr (B == B_RSUB) return b - a;
    else if constexpr (B == B_MUL) return a * b;
    else if constexpr (B == B_DIV) return a * f_rcp(b);
    else if constexpr (B == B_RDIV) return b * f_rcp(a);
    else if constexpr (B == B_MIN) return f_minp(a, b);
    else if constexpr (B == B_MAX) return f_maxp(a, b);
    else if constexpr (B == B_POW) return f_pow(a, b);
    else if constexpr (B == B_RPOW) return f_pow(b, a);
    else if constexpr (B == B_EQ) return a == b ? 1.0f : 0.0f;
    else if constexpr (B == B_NE) return a != b ? 1.0f : 0.0f;
    else if constexpr (B == B_LT) return a < b ? 1.0f : 0.0f;
    else if constexpr (B == B_LE) return a <= b ? 1.0f : 0.0f;
    else if constexpr (B == B_GT) return a > b ? 1.0f : 0.0f;
    else if constexpr (B == B_GE) return a >= b ? 1.0f : 0.0f;
    // exp of a difference: the difference is exact to one rounding, so the plain product with
    // log2(e) keeps the relative error below |a - b| * 2^-24 (5e-6 at the overflow threshold)
    else if constexpr (B == B_EXPSUB) return f_exp2((a - b) * LOG2E);
    else if constexpr (B == B_REXPSUB) return f_exp2((b - a) * LOG2E);
    else return a;
}

// scalar (one value) versions selected at run time; used for the row-scalar registers
DI float un_dyn(uint32_t u, float x) {
    switch (u) {
#define C(U) case U: return un_op<U>(x);
        C(U_SQRT) C(U_ABS) C(U_LOG) C(U_EXP) C(U_ROUND) C(U_FLOOR) C(U_ISFINITE) C(U_NEG) C(U_RSQRT)
        C(U_RCP) C(U_TANH) C(U_ERF) C(U_SIGMOID) C(U_SQUARE) C(U_GELU_TANH) C(U_GELU_ERF) C(U_SILU)
        C(U_CAST_BF16)
#undef C
        default: return x;
    }
}
DI float bin_dyn(uint32_t b, float x, float y) {
    switch (b) {
#define C(B) case B: return bin_op<B>(x, y);
        C(B_NONE) C(B_ADD) C(B_SUB) C(B_RSUB) C(B_MUL) C(B_DIV) C(B_RDIV) C(B_MIN) C(B_MAX) C(B_POW)
        C(B_RPOW) C(B_EQ) C(B_NE) C(B_LT) C(B_LE) C(B_GT) C(B_GE) C(B_EXPSUB) C(B_REXPSUB)
#undef C
        default: return x;
    }
}

// ------------------------------------------------------------------------------------------
// A tile register is a struct of K fp32 per lane.  Helpers below touch it only through constant
// element indices and never choose between two registers at run time (the interpreter's switch
// does that, in the kernel body), so every register is split into K independent scalar VGPRs and
// an instruction updates its destination in place.
// ------------------------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));
// (held as groups of four consecutive registers: a 16-byte load or store moves a whole group without copies)
template <int K> struct Tile { f32x4 q[K / 4]; };
#define TV(T, I) ((T).q[(I) >> 2][(I) & 3])
template <int K> DI void tile_zero(Tile<K> &t) { sfor<K / 4>([&]<int Q>() LI { t.q[Q] = f32x4{0.0f, 0.0f, 0.0f, 0.0f}; }); }

template <int K, uint32_t U> DI void tile_un(Tile<K> &a) {
    sfor<K>([&]<int I>() LI { TV(a, I) = un_op<U>(TV(a, I)); });
}
template <int K, uint32_t B> DI void tile_bin(Tile<K> &a, const Tile<K> &b) {
    sfor<K>([&]<int I>() LI { TV(a, I) = bin_op<B>(TV(a, I), TV(b, I)); });
}
template <int K, uint32_t B> DI void tile_bins(Tile<K> &a, float s) {
    sfor<K>([&]<int I>() LI { TV(a, I) = bin_op<B>(TV(a, I), s); });
}

template <int K> DI void tile_un_dispatch(Tile<K> &a, uint32_t u) {
    switch (u) {
#define C(U) case U: tile_un<K, U>(a); break;
        C(U_SQRT) C(U_ABS) C(U_LOG) C(U_EXP) C(U_ROUND) C(U_FLOOR) C(U_ISFINITE) C(U_NEG) C(U_RSQRT)
        C(U_RCP) C(U_TANH) C(U_ERF) C(U_SIGMOID) C(U_SQUARE) C(U_GELU_TANH) C(U_GELU_ERF) C(U_SILU)
        C(U_CAST_BF16)
#undef C
        default: break;
    }
}
template <int K> DI void tile_bin_dispatch(Tile<K> &a, const Tile<K> &b, uint32_t op) {
    switch (op) {
#define C(B) case B: tile_bin<K, B>(a, b); break;
        C(B_NONE) C(B_ADD) C(B_SUB) C(B_RSUB) C(B_MUL) C(B_DIV) C(B_RDIV) C(B_MIN) C(B_MAX) C(B_POW)
        C(B_RPOW) C(B_EQ) C(B_NE) C(B_LT) C(B_LE) C(B_GT) C(B_GE) C(B_EXPSUB) C(B_REXPSUB)
#undef C
        default: break;
    }
}
template <int K> DI void tile_bins_dispatch(Tile<K> &a, float s, uint32_t op) {
    switch (op) {
#define C(B) case B: tile_bins<K, B>(a, s); break;
        C(B_NONE) C(B_ADD) C(B_SUB) C(B_RSUB) C(B_MUL) C(B_DIV) C(B_RDIV) C(B_MIN) C(B_MAX) C(B_POW)
        C(B_RPOW) C(B_EQ) C(B_NE) C(B_LT) C(B_LE) C(B_GT) C(B_GE) C(B_EXPSUB) C(B_REXPSUB)
#undef C
        default: break;
    }
}

// ------------------------------------------------------------------------------------------
// cross-lane reduction inside a wave with DPP / ds_swizzle / readlane; `width` (lanes per
// row, a power of two up to 64) is wave-uniform.  The combination order is fixed, so results
// are bitwise reproducible.
// ------------------------------------------------------------------------------------------
template <uint32_t R> DI float red_comb(float a, float b) {
    if constexpr (R == R_MAX) return f_maxp(a, b);
    else if constexpr (R == R_MIN) return f_minp(a, b);
    else return a + b;
}
template <uint32_t R> DI float red_ident() {
    if constexpr (R == R_MAX) return -__builtin_inff();
    else if constexpr (R == R_MIN) return __builtin_inff();
    else return 0.0f;
}
template <int CTRL> DI float dpp_mov(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
}
template <uint32_t R> DI float swap16(float v) {   // combine with lane ^ 16
    return red_comb<R>(v, __builtin_bit_cast(float, __builtin_amdgcn_ds_swizzle(__builtin_bit_cast(int, v), 0x401F)));
}
template <uint32_t R> DI float wave_allreduce(float v, uint32_t width) {
    if (width == 64) {          // the common case, free of branches: the row spans the whole wave
        v = red_comb<R>(v, dpp_mov<0xB1>(v));                             // quad_perm [1,0,3,2]
        v = red_comb<R>(v, dpp_mov<0x4E>(v));                             // quad_perm [2,3,0,1]
        v = red_comb<R>(v, dpp_mov<0x141>(v));                            // row_half_mirror
        v = red_comb<R>(v, dpp_mov<0x140>(v));                            // row_mirror
        v = swap16<R>(v);
        float lo = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 0));
        float hi = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 32));
        return red_comb<R>(lo, hi);
    }
    if (width >= 2) v = red_comb<R>(v, dpp_mov<0xB1>(v));
    if (width >= 4) v = red_comb<R>(v, dpp_mov<0x4E>(v));
    if (width >= 8) v = red_comb<R>(v, dpp_mov<0x141>(v));
    if (width >= 16) v = red_comb<R>(v, dpp_mov<0x140>(v));
    if (width >= 32) v = swap16<R>(v);
    return v;
}

// ------------------------------------------------------------------------------------------
// per-tile geometry
// ------------------------------------------------------------------------------------------
// (The instantiation for any launch, and the one for reductions along the penultimate axis, handle a last chunk element
// by element where it may not slide back; the others are launched only where no tile asks for it.)
#if defined(DVM_VARIANT_K) && !defined(DVM_VARIANT_CRED) && !defined(DVM_VARIANT_ANY)
constexpr bool HAVE_PART = false;
#else
constexpr bool HAVE_PART = true;
#endif
// Passing over the sets and segments that hold none of a workgroup's tiles (rotate = 1) is left out of the instantiations for
// launches of few segments and sets for their size: two more values across the record loop cost the 12-op chain 12 %, masked softmax
// 6-15 % and a stack of eight large RMSNorms 15 %.  (Their loops over segments and sets stay: without them the compiler reloads the segment header inside the record
// loop, and the chain is 5 % slower, masked softmax 3 %.)
#if defined(DVM_VARIANT_VISIT)
constexpr bool SKIP = false;
#else
constexpr bool SKIP = true;
#endif
// The wave-uniform part lives across the interpreter loop, whose scalar registers are scarce (a value more there is
// spilled and costs every record): it holds what cannot be derived in a few scalar instructions where it is used.
struct Geo {
    // wave-uniform
    uint64_t colbase;     // first column of the tile
    uint32_t cend;        // chunk slots that start before this column (relative to colbase) are read, reduced and stored whole: the
                          // tile's width, less the elements of a last chunk that is handled element by element
    uint32_t GV;          // G * V: column distance between two chunks of one lane
    uint32_t nact;        // chunks per lane * V
    uint32_t pk;          // packed: PK_* below
    static constexpr uint32_t PK_N = 0xF;           // elements of the last chunk a row ends inside of (0: rows of whole chunks)
    static constexpr uint32_t PK_RAGGED = 0x40;     // some lane has invalid columns inside live chunks: reductions must mask
    static constexpr uint32_t PK_SLIDE = 0x80;      // the last chunk slides back to end with the row (see tile_cols)
    static constexpr uint32_t PK_PART = 0x100;      // the last chunk is handled element by element, by ...
    static constexpr int PK_SLOT = 12, PK_LANE = 20;        // ... the lane (within the row group) PK_LANE in its chunk slot PK_SLOT
    DI uint32_t ragged() const { return pk & PK_RAGGED; }
    DI uint32_t slide() const { return pk & PK_SLIDE; }
    DI uint32_t part() const { return HAVE_PART ? pk & PK_PART : 0u; }
    DI bool chunks() const { return !HAVE_PART || cend != 0; }         // the tile has at least one whole chunk
    DI uint32_t part_n() const { return pk & PK_N; }
    DI uint32_t part_slot() const { return (pk >> PK_SLOT) & 0xFF; }
    DI uint32_t part_lane() const { return pk >> PK_LANE; }
    // per lane
    uint32_t i1, i2, i3;  // decomposition of the lane's row index over the outer dims
    uint32_t lanecol;     // first column of the lane's chunk 0, relative to colbase: V times the lane's index within the row group
    uint32_t rowok;       // 1 when the lane's row lies inside the tensor
};

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 u32x4_a4 __attribute__((aligned(4)));
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));
typedef f32x4 f32x4_a4 __attribute__((aligned(4)));
#define GLOBAL_AS __attribute__((address_space(1)))
typedef const GLOBAL_AS char *gcptr;   // global memory, read
typedef GLOBAL_AS char *gptr;          // global memory, write

DI float bf16_lo(uint32_t w) { return __builtin_bit_cast(float, w << 16); }
DI float bf16_hi(uint32_t w) { return __builtin_bit_cast(float, w & 0xFFFF0000u); }
DI uint32_t pack_bf16x2(float a, float b) {
    typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    f2 v = {a, b};
    bf2 h = __builtin_convertvector(v, bf2);
    return __builtin_bit_cast(uint32_t, h);
}
DI uint16_t pack_bf16(float a) {
    __bf16 h = (__bf16)a;
    return __builtin_bit_cast(uint16_t, h);
}

// element offset of the lane's row for a tensor with outer strides s1..s3
DI int64_t row_offset(const Geo &g, int64_t s1, int64_t s2, int64_t s3) {
    return (int64_t)g.i1 * s1 + (int64_t)g.i2 * s2 + (int64_t)g.i3 * s3;
}

// Predicated stores.  The interpreter loop must not contain a branch that differs between the
// lanes of a wave: with only wave-uniform branches the compiler keeps the dispatch as plain scalar
// jumps and updates registers in place.  Loads therefore clamp the address of an invalid lane to
// a valid one (its data is never used), and stores switch the invalid lanes off in EXEC inside
// one assembly statement.  (The compiler does not look inside the statement, so the wait state that this
// chip wants between a store of more than 8 bytes and an instruction that overwrites the stored registers is
// written out: the s_nop after the restored EXEC mask.)
DI void st_b128(gptr p, f32x4 v, bool ok) {
    const uint64_t m = __builtin_amdgcn_ballot_w64(ok);
    uint64_t sv;
    asm volatile("s_and_saveexec_b64 %0, %1\n\tglobal_store_dwordx4 %2, %3, off nt\n\ts_mov_b64 exec, %0\n\ts_nop 0"
                 : "=&s"(sv) : "s"(m), "v"(p), "v"(v) : "memory", "scc");
}
DI void st_b32(gptr p, float v, bool ok) {
    const uint64_t m = __builtin_amdgcn_ballot_w64(ok);
    uint64_t sv;
    asm volatile("s_and_saveexec_b64 %0, %1\n\tglobal_store_dword %2, %3, off nt\n\ts_mov_b64 exec, %0\n\ts_nop 0"
                 : "=&s"(sv) : "s"(m), "v"(p), "v"(v) : "memory", "scc");
}
DI void st_b16(gptr p, uint32_t v, bool ok) {
    const uint64_t m = __builtin_amdgcn_ballot_w64(ok);
    uint64_t sv;
    asm volatile("s_and_saveexec_b64 %0, %1\n\tglobal_store_short %2, %3, off nt\n\ts_mov_b64 exec, %0\n\ts_nop 0"
                 : "=&s"(sv) : "s"(m), "v"(p), "v"(v) : "memory", "scc");
}

// Loading the lane's part of a tile has two halves, so that the loads of several tensors are in flight
// together: request_inplace issues every whole chunk straight into the destination tile register (no staging
// registers: fp32 chunks land where their elements live, a bf16 chunk of 8 elements = 16 bytes lands in the
// upper half of the register), and finish_tile, called once all loads of a group of load records have been
// issued, widens the bf16 bits in place and fetches the chunk a ragged row ends in.
// DT: 0 = fp32, 1 = bf16.  V = chunk width.  `rowp` points at column `colbase` of the lane's row in this tensor
// (row 0 for a lane whose row is outside the tensor).  A chunk that lies beyond the tile's columns reads the
// tile's last chunk instead: the value is never stored and reductions mask it.  Dtype, chunk width and cache hint
// are fixed at compile time, so the request needs no per-piece scalar arithmetic.  NT: the data is read once,
// hint the caches accordingly.
// DVM_STREAMING closes a branch of loads with the streaming hint: the compiler would merge it with the branch of the same loads without
// the hint and drop the hint (all of them in the general instantiation, those of fp32 tensors in the wide one): fp32 add over 45M elements 104 us so merged, 97 apart.
#define DVM_STREAMING() asm volatile("; streaming" ::: "memory")
typedef f32x4 f32x4_a2 __attribute__((aligned(2)));
template <bool NT> DI f32x4 ld_b128(gcptr q) {
    const GLOBAL_AS f32x4_a2 *src = (const GLOBAL_AS f32x4_a2 *)q;
    if constexpr (NT) return __builtin_nontemporal_load(src);
    else return *src;
}

// First column (relative to the tile's) that the lane's chunk slot J reads and writes.
template <int V> DI uint32_t chunk_col(const Geo &g, int J) {
    const uint32_t c0 = g.lanecol + (uint32_t)J * g.GV;
    const uint32_t cmax = g.cend - V;
    return c0 < cmax ? c0 : cmax;
}
template <int K, int DT, int V, bool NT> DI void request_inplace(Tile<K> &t, gcptr rowp, const Geo &g) {
    constexpr int ES = DT == 0 ? 4 : 2;
    if constexpr (K >= V) {
        constexpr int NJ = K / V;
        if (g.chunks()) {       // wave-uniform: the tile has at least one whole chunk
            sfor<NJ>([&]<int J>() LI {
                gcptr q = rowp + (uint64_t)chunk_col<V>(g, J) * ES;
                if constexpr (DT == 0) {
                    sfor<V / 4>([&]<int H>() LI { t.q[J * (V / 4) + H] = ld_b128<NT>(q + 16 * H); });
                } else {
                    t.q[K / 8 + J] = ld_b128<NT>(q);        // raw bits, widened by finish_tile
                }
            });
            if constexpr (NT) DVM_STREAMING();
        }
    }
}
template <int K> DI void request_dispatch(Tile<K> &t, uint32_t dt, uint32_t V, bool nt, gcptr rowp, const Geo &g) {
    if (nt) {
        if (dt == 0) {
            if (V == 4) request_inplace<K, 0, 4, true>(t, rowp, g);
            else request_inplace<K, 0, 8, true>(t, rowp, g);
        } else {
            request_inplace<K, 1, 8, true>(t, rowp, g);
        }
    } else {
        if (dt == 0) {
            if (V == 4) request_inplace<K, 0, 4, false>(t, rowp, g);
            else request_inplace<K, 0, 8, false>(t, rowp, g);
        } else {
            request_inplace<K, 1, 8, false>(t, rowp, g);
        }
    }
}

// The second half.  bf16: chunk J sits as raw bits in group K/8 + J and becomes the eight values of groups
// 2J and 2J + 1; going through the chunks in ascending order never overwrites bits that are still to be read
// (2J + 1 <= K/8 + J for every J < K/8, and the last chunk is read before its own group is written).
template <int K, int DT, int V> DI void finish_tile(Tile<K> &t, gcptr rowp, const Geo &g) {
    constexpr int ES = DT == 0 ? 4 : 2;
    if constexpr (K < V) tile_zero<K>(t);
    if constexpr (K >= V) {
        constexpr int NJ = K / V;
        if (!g.chunks()) {        // narrower than one chunk: only the ragged part below
            tile_zero<K>(t);
        } else if constexpr (DT == 1) {
            sfor<NJ>([&]<int J>() LI {
                const u32x4 r = __builtin_bit_cast(u32x4, t.q[K / 8 + J]);
                const uint32_t w0 = r.x, w1 = r.y, w2 = r.z, w3 = r.w;
                t.q[2 * J] = f32x4{bf16_lo(w0), bf16_hi(w0), bf16_lo(w1), bf16_hi(w1)};
                t.q[2 * J + 1] = f32x4{bf16_lo(w2), bf16_hi(w2), bf16_lo(w3), bf16_hi(w3)};
            });
        }
        if (g.part() != 0) {   // wave-uniform: this tile ends inside a chunk
            // its elements are read one by one by every lane of the row (one of them keeps them); an element
            // beyond the row reads element 0 again
            const bool own = g.lanecol == g.part_lane() * (uint32_t)V;
            float pv[V];
            sfor<V>([&]<int E>() LI {
                const uint32_t e = (uint32_t)E < g.part_n() ? (uint32_t)E : 0u;       // wave-uniform
                gcptr q = rowp + (uint64_t)(g.cend + e) * ES;
                if constexpr (DT == 0) pv[E] = *(const GLOBAL_AS float *)q;
                else pv[E] = bf16_lo(*(const GLOBAL_AS uint16_t *)q);
            });
            sfor<NJ>([&]<int J>() LI {
                if ((uint32_t)J == g.part_slot()) {       // wave-uniform
                    sfor<V>([&]<int E>() LI {
                        const bool ok = own && (uint32_t)E < g.part_n();
                        // (the empty statement keeps this a select between two values: a select between
                        // two register-array elements would be turned into a select of their addresses,
                        // which forces both arrays into memory)
                        float x = pv[E];
                        asm volatile("" : "+v"(x));
                        TV(t, J * V + E) = ok ? x : TV(t, J * V + E);
                    });
                }
            });
        }
    }
}
template <int K> DI void finish_dispatch(Tile<K> &t, uint32_t dt, uint32_t V, gcptr rowp, const Geo &g) {
    if (dt == 0) {
        if (V == 4) finish_tile<K, 0, 4>(t, rowp, g);
        else finish_tile<K, 0, 8>(t, rowp, g);
    } else {
        finish_tile<K, 1, 8>(t, rowp, g);
    }
}

// The streaming reduction along the penultimate axis keeps several rows of one tensor in flight per wave and
// combines them into an accumulating register: it stages a row's raw bits in registers of its own (only the
// variants with at most 8 elements per lane run it).
template <int K> struct Raw {
    f32x4 q[K / 4];     // the whole chunks, 16 bytes per piece
    uint32_t pv[8];     // the elements of the chunk the row ends in (raw bits), requested alongside
};
template <int K, int DT, int V, bool NT> DI void request_staged(Raw<K> &raw, gcptr rowp, const Geo &g) {
    constexpr int ES = DT == 0 ? 4 : 2;
    if constexpr (K >= V) {
        constexpr int NJ = K / V;
        if (g.chunks()) {
            sfor<NJ>([&]<int J>() LI {
                gcptr q = rowp + (uint64_t)chunk_col<V>(g, J) * ES;
                constexpr int PIECES = DT == 0 ? V / 4 : 1;
                sfor<PIECES>([&]<int H>() LI { raw.q[J * PIECES + H] = ld_b128<NT>(q + 16 * H); });
            });
        }
        if (g.part() != 0) {
            sfor<V>([&]<int E>() LI {
                const uint32_t e = (uint32_t)E < g.part_n() ? (uint32_t)E : 0u;
                gcptr q = rowp + (uint64_t)(g.cend + e) * ES;
                if constexpr (DT == 0) raw.pv[E] = *(const GLOBAL_AS uint32_t *)q;
                else raw.pv[E] = *(const GLOBAL_AS uint16_t *)q;
            });
        }
    }
}
template <int K> DI void request_staged_dispatch(Raw<K> &raw, uint32_t dt, uint32_t V, bool nt, gcptr rowp, const Geo &g) {
    if (nt) {
        if (dt == 0) {
            if (V == 4) request_staged<K, 0, 4, true>(raw, rowp, g);
            else request_staged<K, 0, 8, true>(raw, rowp, g);
        } else {
            request_staged<K, 1, 8, true>(raw, rowp, g);
        }
    } else {
        if (dt == 0) {
            if (V == 4) request_staged<K, 0, 4, false>(raw, rowp, g);
            else request_staged<K, 0, 8, false>(raw, rowp, g);
        } else {
            request_staged<K, 1, 8, false>(raw, rowp, g);
        }
    }
}
// t = B(t, staged row), element by element as the pieces are widened; elements outside the row keep their value
template <int K, int DT, int V, uint32_t B> DI void combine_staged(Tile<K> &t, const Raw<K> &raw, const Geo &g) {
    if constexpr (K >= V) {
        constexpr int NJ = K / V;
        if (g.chunks()) {
            const bool masked = g.ragged() != 0;       // wave-uniform
            auto chunk = [&]<int J>(bool whole) LI {
                float x[V];
                if constexpr (DT == 0) {
                    sfor<V / 4>([&]<int H>() LI {
                        const f32x4 r = raw.q[J * (V / 4) + H];
                        x[4 * H + 0] = r.x; x[4 * H + 1] = r.y; x[4 * H + 2] = r.z; x[4 * H + 3] = r.w;
                    });
                } else {
                    const u32x4 r = __builtin_bit_cast(u32x4, raw.q[J]);
                    const uint32_t w0 = r.x, w1 = r.y, w2 = r.z, w3 = r.w;
                    x[0] = bf16_lo(w0); x[1] = bf16_hi(w0); x[2] = bf16_lo(w1); x[3] = bf16_hi(w1);
                    x[4] = bf16_lo(w2); x[5] = bf16_hi(w2); x[6] = bf16_lo(w3); x[7] = bf16_hi(w3);
                }
                sfor<V>([&]<int E>() LI {
                    const float y = bin_op<B>(TV(t, J * V + E), x[E]);
                    TV(t, J * V + E) = whole ? y : TV(t, J * V + E);
                });
            };
            if (!masked) {
                sfor<NJ>([&]<int J>() LI { chunk.template operator()<J>(true); });
            } else {
                sfor<NJ>([&]<int J>() LI { chunk.template operator()<J>(g.lanecol + (uint32_t)J * g.GV < g.cend); });
            }
        }
        if (g.part() != 0) {
            const bool own = g.lanecol == g.part_lane() * (uint32_t)V;
            float pv[V];
            sfor<V>([&]<int E>() LI {
                const uint32_t bits = raw.pv[E];
                if constexpr (DT == 0) pv[E] = __builtin_bit_cast(float, bits);
                else pv[E] = bf16_lo(bits);
            });
            sfor<NJ>([&]<int J>() LI {
                if ((uint32_t)J == g.part_slot()) {
                    sfor<V>([&]<int E>() LI {
                        const bool ok = own && (uint32_t)E < g.part_n();
                        float x = pv[E];
                        asm volatile("" : "+v"(x));
                        x = bin_op<B>(TV(t, J * V + E), x);
                        TV(t, J * V + E) = ok ? x : TV(t, J * V + E);
                    });
                }
            });
        }
    }
}
template <int K, uint32_t B> DI void combine_staged_dispatch(Tile<K> &t, const Raw<K> &raw, uint32_t dt, uint32_t V, const Geo &g) {
    if (dt == 0) {
        if (V == 4) combine_staged<K, 0, 4, B>(t, raw, g);
        else combine_staged<K, 0, 8, B>(t, raw, g);
    } else {
        combine_staged<K, 1, 8, B>(t, raw, g);
    }
}

template <int K, int DT, int V> DI void store_tile(const Tile<K> &t, gptr rowp, const Geo &g) {
    constexpr int ES = DT == 0 ? 4 : 2;
    if constexpr (K >= V) {
        constexpr int NJ = K / V;
        if (g.chunks()) {
            sfor<NJ>([&]<int J>() LI {
                const bool ok = g.rowok && g.lanecol + (uint32_t)J * g.GV < g.cend;
                gptr q = rowp + (uint64_t)chunk_col<V>(g, J) * ES;
                if constexpr (DT == 0) {
                    sfor<V / 4>([&]<int H>() LI { st_b128(q + 16 * H, t.q[J * (V / 4) + H], ok); });
                } else {
                    const f32x4 lo = t.q[2 * J], hi = t.q[2 * J + 1];
                    const u32x4 r = {pack_bf16x2(lo.x, lo.y), pack_bf16x2(lo.z, lo.w), pack_bf16x2(hi.x, hi.y), pack_bf16x2(hi.z, hi.w)};
                    st_b128(q, __builtin_bit_cast(f32x4, r), ok);
                }
            });
        }
        if (g.part() != 0) {
            const bool own = g.rowok && g.lanecol == g.part_lane() * (uint32_t)V;
            sfor<NJ>([&]<int J>() LI {
                if ((uint32_t)J == g.part_slot()) {
                    sfor<V>([&]<int E>() LI {
                        if ((uint32_t)E < g.part_n()) {       // wave-uniform
                            gptr q = rowp + (uint64_t)(g.cend + E) * ES;
                            if constexpr (DT == 0) st_b32(q, TV(t, J * V + E), own);
                            else st_b16(q, (uint32_t)pack_bf16(TV(t, J * V + E)), own);
                        }
                    });
                }
            });
        }
    }
}
template <int K> DI void store_dispatch(const Tile<K> &t, uint32_t dt, uint32_t V, gptr rowp, const Geo &g) {
    if (dt == 0) {
        if (V == 4) store_tile<K, 0, 4>(t, rowp, g);
        else store_tile<K, 0, 8>(t, rowp, g);
    } else {
        store_tile<K, 1, 8>(t, rowp, g);
    }
}

// ---- wide rows ------------------------------------------------------------------------------------
// When a row is held by at least one whole wave (G >= 64), everything about the row is the same for all lanes
// of a wave: its index, its offsets in every tensor, whether it exists.  The wide instantiation of the kernel
// does that arithmetic once per wave on the scalar unit and addresses memory as a scalar row base plus a 32-bit
// lane offset (the form of the load / store instruction that takes a scalar base), so that a memory record
// costs a handful of scalar instructions and one vector instruction per chunk for the offset.
typedef const GLOBAL_AS char *gcptr_u;      // (a wave-uniform pointer)
struct Wide {
    uint32_t i1, i2, i3;    // the wave's row, decomposed over the outer dims (wave-uniform)
    uint32_t rowok;         // the wave's row lies inside the tensor
};

template <int K, int DT, int V, bool NT> DI void issue_wide(Tile<K> &t, const char *rowbase, const uint32_t (&vo)[K / V]) {
    constexpr int NJ = K / V;
    sfor<NJ>([&]<int J>() LI {
        gcptr q = (gcptr)(rowbase + (uint64_t)vo[J]);
        if constexpr (DT == 0) {
            sfor<V / 4>([&]<int H>() LI { t.q[J * (V / 4) + H] = ld_b128<NT>(q + 16 * H); });
        } else {
            t.q[K / 8 + J] = ld_b128<NT>(q);
        }
    });
    if constexpr (NT) DVM_STREAMING();
}
// The offsets are computed before the destination register is selected: inside the selected case nothing but
// the load instructions may write a register, or the compiler would compute addresses in the registers the
// load is about to overwrite, which costs a wait for every load still in flight into them.
#define DVM_ISSUE_WIDE(DT, V, NT)                                                                   \
    {                                                                                               \
        uint32_t vo[K / V];                                                                         \
        sfor<K / V>([&]<int J>() LI { vo[J] = chunk_col<V>(g, J) * (DT == 0 ? 4 : 2); }); \
        _Pragma("unroll") for (int j_ = 0; j_ < K / V; ++j_) asm volatile("" : "+v"(vo[j_]));       \
        if (ra == SRC_ACC) {                                                                        \
            issue_wide<K, DT, V, NT>(acc, rowbase, vo);                                             \
        } else {                                                                                    \
            DVM_WITH_R(ra, rr, (issue_wide<K, DT, V, NT>(rr, rowbase, vo)))                         \
        }                                                                                           \
    }

// A row that consists of chunks alone (none handled element by element), row inside the tensor: 16-byte stores from
// the scalar row base.  FULL: every chunk slot the tile uses lies inside the row.  Otherwise the slots the row ends in
// switch the lanes behind its end off.
DI void st_b128_off(char *base, uint32_t off, f32x4 v, bool ok) {
    const uint64_t m = __builtin_amdgcn_ballot_w64(ok);
    uint64_t sv;
    asm volatile("s_and_saveexec_b64 %0, %1\n\tglobal_store_dwordx4 %2, %3, %4 nt\n\ts_mov_b64 exec, %0\n\ts_nop 0"
                 : "=&s"(sv) : "s"(m), "v"(off), "v"(v), "s"(base) : "memory", "scc");
}
template <int K, int DT, int V, bool FULL> DI void store_wide(const Tile<K> &t, char *rowbase, const Geo &g) {
    constexpr int ES = DT == 0 ? 4 : 2;
    constexpr int NJ = K / V;
    sfor<NJ>([&]<int J>() LI {
        if (J == 0 || (uint32_t)(J * V) < g.nact) {        // wave-uniform: chunk slots the tile uses
            const uint32_t c0 = g.lanecol + (uint32_t)J * g.GV;
            const uint32_t vo = (FULL ? c0 : chunk_col<V>(g, J)) * ES;
            const bool whole = FULL || (uint32_t)(J + 1) * g.GV <= g.cend;      // wave-uniform
            auto put = [&](f32x4 v, uint32_t at) LI {
                if (whole) __builtin_nontemporal_store(v, (GLOBAL_AS f32x4 *)(rowbase + (uint64_t)vo + at));
                else st_b128_off(rowbase, vo + at, v, c0 < g.cend);
            };
            if constexpr (DT == 0) {
                sfor<V / 4>([&]<int H>() LI { put(t.q[J * (V / 4) + H], 16 * H); });
            } else {
                const f32x4 lo = t.q[2 * J], hi = t.q[2 * J + 1];
                const u32x4 r = {pack_bf16x2(lo.x, lo.y), pack_bf16x2(lo.z, lo.w), pack_bf16x2(hi.x, hi.y), pack_bf16x2(hi.z, hi.w)};
                put(__builtin_bit_cast(f32x4, r), 0);
            }
        }
    });
}
template <int K, bool FULL> DI void store_wide_dispatch(const Tile<K> &t, uint32_t dt, uint32_t V, char *rowbase, const Geo &g) {
    if (dt == 0) {
        if (V == 4) store_wide<K, 0, 4, FULL>(t, rowbase, g);
        else if constexpr (K >= 8) store_wide<K, 0, 8, FULL>(t, rowbase, g);
    } else {
        if constexpr (K >= 8) store_wide<K, 1, 8, FULL>(t, rowbase, g);
    }
}

// in-lane part of a row reduction over the accumulator.  When the tile is ragged, a chunk of a lane
// is either wholly inside the row, wholly outside, or the one chunk the row ends in: whole chunks
// are reduced unmasked and selected per chunk.  A last chunk that slid back repeats elements of the chunk before it:
// a maximum or minimum may take them twice, a sum leaves them out (its first elements, as many as it slid by).  A last chunk
// handled element by element is masked element by element.
template <int K, uint32_t R, int V> DI float lane_reduce_ragged(const Tile<K> &a, const Geo &g) {
    float v = red_ident<R>();
    if constexpr (K >= V) {
        constexpr int NJ = K / V;
        constexpr uint32_t RC = R == R_SUMSQ ? R_SUM : R;      // how partial results combine
        sfor<NJ>([&]<int J>() LI {
            if (J == 0 || (uint32_t)(J * V) < g.nact) {        // wave-uniform
                const uint32_t c0 = g.lanecol + (uint32_t)J * g.GV;
                float c = red_ident<R>();
                if (R == R_MAX || R == R_MIN || g.slide() == 0 || (uint32_t)(J + 1) * g.GV <= g.cend) {      // wave-uniform
                    sfor<V>([&]<int E>() LI {
                        if constexpr (R == R_SUMSQ) c = f_fma(TV(a, J * V + E), TV(a, J * V + E), c);
                        else c = red_comb<R>(c, TV(a, J * V + E));
                    });
                } else {
                    const uint32_t dup = c0 - chunk_col<V>(g, J);
                    sfor<V>([&]<int E>() LI {
                        const float x = (uint32_t)E >= dup ? TV(a, J * V + E) : 0.0f;
                        if constexpr (R == R_SUMSQ) c = f_fma(x, x, c);
                        else c = red_comb<R>(c, x);
                    });
                }
                v = red_comb<RC>(v, c0 < g.cend ? c : red_ident<R>());
            }
        });
        if (g.part() != 0) {
            const bool own = g.lanecol == g.part_lane() * (uint32_t)V;
            sfor<NJ>([&]<int J>() LI {
                if ((uint32_t)J == g.part_slot()) {              // wave-uniform
                    sfor<V>([&]<int E>() LI {
                        const bool ok = own && (uint32_t)E < g.part_n();
                        if constexpr (R == R_SUMSQ) {
                            const float x = ok ? TV(a, J * V + E) : 0.0f;
                            v = f_fma(x, x, v);
                        } else {
                            v = red_comb<R>(v, ok ? TV(a, J * V + E) : red_ident<R>());
                        }
                    });
                }
            });
        }
    }
    return v;
}
template <int K, uint32_t R> DI float lane_reduce(const Tile<K> &a, const Geo &g, uint32_t V) {
    float v = red_ident<R>();
    if (g.ragged() == 0) {
        sfor<K / 4>([&]<int Q>() LI {
            if (Q == 0 || (uint32_t)(Q * 4) < g.nact) {
                sfor<4>([&]<int E>() LI {
                    if constexpr (R == R_SUMSQ) v = f_fma(TV(a, Q * 4 + E), TV(a, Q * 4 + E), v);
                    else v = red_comb<R>(v, TV(a, Q * 4 + E));
                });
            }
        });
    } else if (V == 8) {
        v = lane_reduce_ragged<K, R, 8>(a, g);
    } else {
        v = lane_reduce_ragged<K, R, 4>(a, g);
    }
    return v;
}

// the two halves apart (a row longer than a tile is reduced tile after tile within the lane, then once across the lanes)
template <int K> DI float lane_reduce_dispatch(const Tile<K> &a, const Geo &g, uint32_t V, uint32_t kind) {
    switch (kind) {
        case R_MAX: return lane_reduce<K, R_MAX>(a, g, V);
        case R_MIN: return lane_reduce<K, R_MIN>(a, g, V);
        case R_SUMSQ: return lane_reduce<K, R_SUMSQ>(a, g, V);
        default: return lane_reduce<K, R_SUM>(a, g, V);
    }
}
DI float wave_allreduce_dispatch(float v, uint32_t kind, uint32_t width) {
    switch (kind) {
        case R_MAX: return wave_allreduce<R_MAX>(v, width);
        case R_MIN: return wave_allreduce<R_MIN>(v, width);
        default: return wave_allreduce<R_SUM>(v, width);
    }
}
template <int K> DI float reduce_dispatch(const Tile<K> &a, const Geo &g, uint32_t V, uint32_t kind, uint32_t width) {
    switch (kind) {
        case R_MAX: return wave_allreduce<R_MAX>(lane_reduce<K, R_MAX>(a, g, V), width);
        case R_MIN: return wave_allreduce<R_MIN>(lane_reduce<K, R_MIN>(a, g, V), width);
        case R_SUMSQ: return wave_allreduce<R_SUM>(lane_reduce<K, R_SUMSQ>(a, g, V), width);
        default: return wave_allreduce<R_SUM>(lane_reduce<K, R_SUM>(a, g, V), width);
    }
}

// Every record starts on a 16-byte boundary and is 4 or 8 words long, so one scalar 128-bit load
// fetches a whole record (the view forms take a second one).  The record after the current one is
// requested before the current handler runs, so that the scalar-cache latency of decoding overlaps
// the vector work (the pipelining of decode and execute of Section 4.3).  The prefetch may reach
// past the code body: it stays inside the kernel-argument struct.
typedef uint32_t u32x4s __attribute__((ext_vector_type(4)));
DI u32x4s fetch4(const uint32_t *code, uint32_t pc) {
    return *(const u32x4s *)__builtin_assume_aligned(code + pc, 16);
}
// the same with a byte offset: one scalar load with a register offset, no 64-bit address arithmetic
DI u32x4s fetch4b(const uint32_t *code, uint32_t byte_off) {
    return *(const u32x4s *)__builtin_assume_aligned((const char *)code + (uint64_t)byte_off, 16);
}

DI float pick_s(float s0, float s1, float s2, float s3, uint32_t i) {
    float v = s0;
    v = i == 1 ? s1 : v;
    v = i == 2 ? s2 : v;
    v = i == 3 ? s3 : v;
    return v;
}

// unsigned division by an invariant divisor with a precomputed multiplier and two shifts
// (Granlund & Montgomery, "Division by invariant integers using multiplication", 32-bit case)
DI uint32_t magic_div(uint32_t n, uint32_t m, uint32_t sh) {
    uint32_t t = __umulhi(m, n);
    return (t + ((n - t) >> (sh & 0xFF))) >> (sh >> 8);
}
DI uint32_t sdiv_u(uint32_t n, uint32_t m, uint32_t sh) {   // the same on wave-uniform values
    uint32_t t = (uint32_t)(((uint64_t)m * n) >> 32);
    return (t + ((n - t) >> (sh & 0xFF))) >> (sh >> 8);
}

// Where a tile of a segment sits.  Columns (wave-uniform): first column and width of column tile
// `tile_c`, and which chunk the row ends in.  Rows: the lane's row decomposed over the outer
// iteration dims; `rp` is the row of the tile this lane holds.
DI void tile_cols(Geo &gt, const uint32_t *sh, uint32_t tile_c, uint32_t G, uint32_t V, uint32_t aliased) {
    const uint32_t TC = sh[S_TC];
    const uint64_t D0 = (uint64_t)sh[S_D0LO] | ((uint64_t)sh[S_D0HI] << 32);
    gt.colbase = (uint64_t)tile_c * TC;
    const uint64_t rem = D0 - gt.colbase;
    const uint32_t ncols = rem < TC ? (uint32_t)rem : TC;
    // A row that ends inside a chunk: that chunk slides back so that it ends with the row and repeats elements of the
    // chunk before it.  Every operand of the tile is read at the slid columns, so element-wise results are computed
    // twice alike and stored twice alike, and the row costs whole 16-byte accesses only: reading its last elements one
    // by one, behind the wait for the chunks, made a second wait for memory per tile (softmax over bf16 rows of 751
    // columns 188 us that way and 131 us this way).  A program may write its own input: then the chunk before must belong
    // to the same wave, which reads both before it stores either.  Where it does not, and in rows narrower than a chunk, the
    // last elements are handled one by one (part_*).
    const uint32_t full_chunks = V == 8 ? ncols >> 3 : ncols >> 2;      // V is 4 or 8
    const uint32_t n = ncols - full_chunks * V;
    gt.cend = full_chunks * V;
    // rows never mix in a reduction, so only invalid columns inside live chunks need a mask
    gt.pk = n | (ncols != gt.nact * G ? Geo::PK_RAGGED : 0u);
    if (n != 0) {
        const uint32_t slot = __builtin_amdgcn_readfirstlane(full_chunks / G);
        const uint32_t lane = full_chunks - slot * G;
        if (!HAVE_PART || (full_chunks != 0 && (G <= 64 || (lane & 63u) != 0 || aliased == 0))) {
            gt.pk |= Geo::PK_SLIDE;
            gt.cend = ncols;
        } else {
            gt.pk |= Geo::PK_PART | (slot << Geo::PK_SLOT) | (lane << Geo::PK_LANE);
        }
    }
}
DI void tile_rows_at(Geo &gt, const uint32_t *sh, uint32_t row, bool ok) {
    gt.rowok = ok;
    const uint32_t rowc = gt.rowok ? row : 0;
    gt.i1 = rowc; gt.i2 = 0; gt.i3 = 0;
    const uint32_t D1 = sh[S_D1];
    if (D1 != 0) {
        const uint32_t q = magic_div(rowc, sh[S_M1], sh[S_SH1]);
        gt.i1 = rowc - q * D1;
        gt.i2 = q;
        const uint32_t D2 = sh[S_D2];
        if (D2 != 0) {
            const uint32_t q2 = magic_div(q, sh[S_M2], sh[S_SH2]);
            gt.i2 = q - q2 * D2;
            gt.i3 = q2;
        }
    }
}
DI void tile_rows(Geo &gt, const uint32_t *sh, uint32_t tile_r, uint32_t rp, uint32_t tid, uint32_t RP, uint32_t seg_threads) {
    const uint32_t row = tile_r * RP + rp;
    tile_rows_at(gt, sh, row, (row < sh[S_NROWS]) && (rp < RP) && (tid < seg_threads));
}

// ------------------------------------------------------------------------------------------
// row-invariant operands kept in LDS
// ------------------------------------------------------------------------------------------
#define LDS_AS __attribute__((address_space(3)))
// Copy the first `d0` elements of the tensor at `src` (dtype dt) into an LDS image of n16 16-byte pieces, zero behind
// the row's end.  All `nthreads` threads of the workgroup take part; every branch is wave-uniform (a thread
// past the last piece copies the last piece once more).
// `full` and `back`: elements from `full` on (a last chunk that slides back, see tile_cols) are read `back` elements
// before their place; full = d0 and back = 0 where nothing slides.
DI void lds_copy_row(LDS_AS char *dst, uint32_t n16, gcptr src, uint64_t d0, uint32_t full, uint32_t back, uint32_t dt, uint32_t tid, uint32_t nthreads) {
    const uint32_t es = dt == 0 ? 4u : 2u;
    const uint32_t epp = 16u / es;                        // elements per piece
    const bool aligned = (((uint64_t)(uintptr_t)src) & 15u) == 0;
    for (uint32_t base = 0; base < n16; base += nthreads) {
        const uint32_t want = base + tid;
        const uint32_t i = want < n16 ? want : n16 - 1;
        const uint64_t e0 = (uint64_t)i * epp;
        const bool whole = aligned && e0 + epp <= full;
        u32x4 v;
        if (__builtin_amdgcn_ballot_w64(!whole) == 0) {     // the usual case: this wave's pieces all lie inside the row
            v = *(const GLOBAL_AS u32x4 *)(src + (uint64_t)i * 16u);
        } else {
            uint32_t wds[4] = {0u, 0u, 0u, 0u};
            if (dt == 0) {
                sfor<4>([&]<int E>() LI {
                    const uint64_t p = e0 + E;
                    const uint64_t e = p < full ? p : p - back;
                    const uint32_t x = *(const GLOBAL_AS uint32_t *)(src + (e < d0 ? e : 0) * 4u);
                    wds[E] = e < d0 ? x : 0u;
                });
            } else {
                sfor<8>([&]<int E>() LI {
                    const uint64_t p = e0 + E;
                    const uint64_t e = p < full ? p : p - back;
                    const uint32_t x = *(const GLOBAL_AS uint16_t *)(src + (e < d0 ? e : 0) * 2u);
                    wds[E / 2] |= (e < d0 ? x : 0u) << (16 * (E & 1));
                });
            }
            v = u32x4{wds[0], wds[1], wds[2], wds[3]};
        }
        *(LDS_AS u32x4 *)(dst + (size_t)i * 16u) = v;
    }
}
// Element E (0..V-1) of a chunk of an LDS image held as raw 16-byte pieces: r0 (and r1 for fp32 chunks of eight).
template <int E> DI float lds_elem(const u32x4 &r0, const u32x4 &r1, bool bf16) {
    if (bf16) {
        const uint32_t w = r0[E / 2];
        return (E & 1) ? bf16_hi(w) : bf16_lo(w);
    }
    return __builtin_bit_cast(float, E < 4 ? r0[E & 3] : r1[E & 3]);
}
// acc = acc * s [* A] [+ B] chunk by chunk, A and B read from their LDS images (V = 4: fp32 images; V = 8: bf16 or
// fp32, per image).  A chunk of this lane that lies beyond the image (the lane holds fewer live chunks than
// others) reads the image's first chunk: its result is never stored and reductions mask it.
template <int K, int V, bool HASA, bool HASB>
DI void lds_fma(Tile<K> &acc, float s, const LDS_AS char *pa, const LDS_AS char *pb, bool a_bf16, bool b_bf16, uint32_t lanecol, const Geo &g) {
    if constexpr (K >= V) {
        constexpr int NJ = K / V;
        const uint32_t ncols_pad = g.slide() != 0 ? (g.cend + (uint32_t)V - 1u) / (uint32_t)V * (uint32_t)V : g.cend + (g.part() != 0 ? (uint32_t)V : 0u);
        const uint32_t esa = (V == 8 && a_bf16) ? 2u : 4u, esb = (V == 8 && b_bf16) ? 2u : 4u;
        sfor<NJ>([&]<int J>() LI {
            if ((uint32_t)(J * V) < g.nact) {         // wave-uniform
                const uint32_t c0 = lanecol + (uint32_t)J * g.GV;
                const uint32_t cc = c0 + V <= ncols_pad ? c0 : 0u;
                u32x4 a0 = {0u, 0u, 0u, 0u}, a1 = a0, b0 = a0, b1 = a0;
                if constexpr (HASA) {
                    a0 = *(const LDS_AS u32x4 *)(pa + cc * esa);
                    if (V == 8 && !a_bf16) a1 = *(const LDS_AS u32x4 *)(pa + cc * esa + 16u);
                }
                if constexpr (HASB) {
                    b0 = *(const LDS_AS u32x4 *)(pb + cc * esb);
                    if (V == 8 && !b_bf16) b1 = *(const LDS_AS u32x4 *)(pb + cc * esb + 16u);
                }
                sfor<V>([&]<int E>() LI {
                    const float t = TV(acc, J * V + E) * s;
                    if constexpr (HASA && HASB) TV(acc, J * V + E) = f_fma(t, lds_elem<E>(a0, a1, V == 8 && a_bf16), lds_elem<E>(b0, b1, V == 8 && b_bf16));
                    else if constexpr (HASA) TV(acc, J * V + E) = t * lds_elem<E>(a0, a1, V == 8 && a_bf16);
                    else TV(acc, J * V + E) = t + lds_elem<E>(b0, b1, V == 8 && b_bf16);
                });
            }
        });
    }
}

// ------------------------------------------------------------------------------------------
// the interpreter
// ------------------------------------------------------------------------------------------
// Run STMT with `RR` naming tile register number IDX (a wave-uniform value): one switch case per
// register, so that every case references its register statically.
#define DVM_WITH_R(IDX, RR, STMT)                                        \
    switch (IDX) {                                                       \
        case 0: { Tile<K> &RR = r0; STMT; } break;                         \
        case 1: if constexpr (NR > 1) { Tile<K> &RR = r1; STMT; } break;   \
        case 2: if constexpr (NR > 2) { Tile<K> &RR = r2; STMT; } break;   \
        case 3: if constexpr (NR > 3) { Tile<K> &RR = r3; STMT; } break;   \
        case 4: if constexpr (NR > 4) { Tile<K> &RR = r4; STMT; } break;   \
        case 5: if constexpr (NR > 5) { Tile<K> &RR = r5; STMT; } break;   \
        default: break;                                                  \
    }
#define DVM_WITH_R2(IDX, RR, STMT)                                       \
    switch (IDX) {                                                       \
        case 0: { Tile<K> &RR = r0; STMT; } break;                         \
        case 1: if constexpr (NR > 1) { Tile<K> &RR = r1; STMT; } break;   \
        case 2: if constexpr (NR > 2) { Tile<K> &RR = r2; STMT; } break;   \
        case 3: if constexpr (NR > 3) { Tile<K> &RR = r3; STMT; } break;   \
        case 4: if constexpr (NR > 4) { Tile<K> &RR = r4; STMT; } break;   \
        case 5: if constexpr (NR > 5) { Tile<K> &RR = r5; STMT; } break;   \
        default: break;                                                  \
    }
#define DVM_GET_S(I) pick_s(s0, s1, s2, s3, (I))
#define DVM_SET_S(I, VAL)                   \
    do {                                    \
        const uint32_t si_ = (I);           \
        const float sv_ = (VAL);            \
        s0 = si_ == 0 ? sv_ : s0;           \
        s1 = si_ == 1 ? sv_ : s1;           \
        s2 = si_ == 2 ? sv_ : s2;           \
        s3 = si_ == 3 ? sv_ : s3;           \
    } while (0)
#define DVM_I64(LO, HI) ((int64_t)((uint64_t)(LO) | ((uint64_t)(HI) << 32)))

// The handlers that use the tile geometry must see it through values the optimiser cannot trace
// back across iterations; otherwise it hoists their address arithmetic and lane masks into the
// tile prologue and executes them for every tile, used or not.  The empty assembly statements pin
// each value to its register at no cost.  Handlers that work on registers only skip all of this.
#define DVM_GEO()                                                                                             \
    asm volatile("" : "+v"(gt.i1), "+v"(gt.i2), "+v"(gt.i3), "+v"(gt.lanecol), "+v"(gt.rowok));   \
    Geo g = gt;                                                                                               \
    {                                                                                                         \
        uint32_t cb_lo = __builtin_amdgcn_readfirstlane((uint32_t)gt.colbase);                                \
        uint32_t cb_hi = __builtin_amdgcn_readfirstlane((uint32_t)(gt.colbase >> 32));                        \
        g.cend = __builtin_amdgcn_readfirstlane(gt.cend);                                                     \
        g.GV = __builtin_amdgcn_readfirstlane(gt.GV);                                                         \
        g.nact = __builtin_amdgcn_readfirstlane(gt.nact);                                                     \
        g.pk = __builtin_amdgcn_readfirstlane(gt.pk);                                                         \
        asm volatile("" : "+s"(cb_lo), "+s"(cb_hi), "+s"(g.cend), "+s"(g.GV), "+s"(g.nact), "+s"(g.pk));      \
        g.colbase = (uint64_t)cb_lo | ((uint64_t)cb_hi << 32);                                                \
    }

// CRED: the instantiation that also runs segments which reduce along the penultimate axis (unit loop,
// accumulate and combine records).  Programs without such a segment run the plain instantiation, whose
// tile loop carries none of that bookkeeping (it costs scalar registers the interpreter loop has none
// to spare of: 5-10 % on short tiles).
// WIDE: the instantiation for launches in which every segment spreads a row over at least one whole wave (see
// "wide rows" above); the other instantiations take any geometry.
// LONG: the instantiations that also run segments over rows longer than a tile (column tiles, passes); the others carry none
// of it (its values across the record loop cost softmax over bf16 rows of 751 columns 12 %, RMSNorm 4 %).  The general one
// with LONG runs any launch without a reduction along the penultimate axis: it also handles last chunks element by element.
template <int K, int NR, int MAXT, int WAVES, bool CRED, bool WIDE, bool LONG>
__global__ void __launch_bounds__(MAXT) __attribute__((amdgpu_waves_per_eu(WAVES))) dvm_vm_kernel(const KArgs args) {
    static_assert(!(CRED && LONG), "a launch holds reductions along the penultimate axis or rows longer than a tile");
    static_assert(!(CRED && WIDE), "the instantiation for reductions along the penultimate axis is the general one");
    __shared__ float red_lds[2][16];
    // (sized by the launch: 1 KiB per wave of the widest segment that reduces along the penultimate axis, else nothing)
    extern __shared__ __align__(16) float comb_lds[];

    // the register file of one lane: accumulator, tile registers, row-scalar registers
    Tile<K> acc, r0, r1, r2, r3, r4, r5;
    tile_zero<K>(acc); tile_zero<K>(r0); tile_zero<K>(r1); tile_zero<K>(r2);
    tile_zero<K>(r3); tile_zero<K>(r4); tile_zero<K>(r5);
    float s0 = 0.0f, s1 = 0.0f, s2 = 0.0f, s3 = 0.0f;

    const uint32_t tid = threadIdx.x;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid) >> 6;
    const uint32_t bid = blockIdx.x;
    const uint32_t ngrid = gridDim.x;
    uint32_t red_par = 0;
    uint32_t n_sync = 0;                    // grid-wide synchronisation points passed so far
    uint32_t rot = 0;                       // rotate = 2: first workgroup of the next segment's tiles
    uint32_t gbase = 0, gnext = bid;        // rotate = 1: tiles of the launch before this segment; this workgroup's next tile
    const uint32_t *code = args.code;
    // the launch's tensor addresses, one per lane: a memory record reads the one it needs with a single lane read
    // (the index is wave-uniform) instead of a scalar load whose latency it would have to wait for
    uint32_t tp_lo, tp_hi;
    {
        const uint64_t mine = args.tensors[tid & (DVM_MAX_TENSORS - 1)];
        tp_lo = (uint32_t)mine;
        tp_hi = (uint32_t)(mine >> 32);
    }
    // A batched launch runs the whole program once per set of tensors, the sets one after the other; the workgroups
    // pass from one set to the next without waiting for each other (the sets are independent).
    // A set or segment that holds none of a workgroup's tiles is passed over at once: going through it (its addresses, its
    // header, the divisions of its geometry) took 1.1 us, 173 us of a 32-layer step whatever its size (a step of 11 tokens 221 us
    // that way and 64 now, of 107 tokens 280 and 132, of 512 tokens 639 and 604).  The set of a workgroup's next tile is
    // found by a division: looking at every set before it took 4 us of the larger launch of a step of 5 tokens (21.6 us, 17.6 now).
    for (uint32_t set = 0;; ++set) {
    if (SKIP && args.rotate == 1) {
        set = sdiv_u(gnext, args.set_m, args.set_sh);
        gbase = set * args.set_tiles;
    }
    if (set >= args.n_sets) break;
    if (args.sets != 0) {
        const uint32_t slot = tid & (DVM_MAX_TENSORS - 1);
        const uint32_t idx = set * args.n_tensors + (slot < args.n_tensors ? slot : 0u);
        const uint64_t mine = ((const GLOBAL_AS uint64_t *)args.sets)[idx];
        tp_lo = (uint32_t)mine;
        tp_hi = (uint32_t)(mine >> 32);
    }
#define DVM_TENSOR(IDX)                                                                                  \
    ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)tp_lo, (int)(IDX)) |                             \
     ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)tp_hi, (int)(IDX)) << 32))

    uint32_t seg = 0;                       // word offset of the current segment
    for (uint32_t si = 0; si < args.nseg; ++si) {
        const uint32_t *sh = &code[seg];
        const uint32_t seg_words = sh[S_WORDS];
        const uint32_t M = sh[S_NTILES];
        if (SKIP && args.rotate == 1 && gnext - gbase >= M) {
            gbase += M;
            seg += seg_words;
            continue;
        }
        const uint32_t code_size = sh[S_CODESIZE];
        const uint32_t geom = sh[S_GEOM];
        const uint32_t G = geom & 0xFFFF, V = (geom >> 16) & 0xFF, nvec = geom >> 24;
        const uint32_t RP = sh[S_RP] & 0xFFFF, seg_threads = sh[S_RP] >> 16;
        const uint32_t tbase = sh[S_TBASE];
        const uint32_t body = seg + SH_WORDS;
        const uint32_t body_end = body + code_size;

        Geo gt;
        gt.GV = G * V;
        gt.nact = nvec * V;
        const uint32_t rp = tid / G;            // row of the tile held by this lane
        gt.lanecol = (tid - rp * G) * V;
        const uint32_t gw = G >> 6;             // waves per row when a row spans waves
        const uint32_t width = G < 64 ? G : 64;
        const uint32_t w0i = gw > 1 ? (wave / gw) * gw : wave;   // first wave of this lane's row

        // The prologue of this segment overwrites the LDS images the previous one may still be reading
        if (sh[S_FLAGS] & SF_LDS) __syncthreads();

        // A segment that depends on earlier ones of this launch waits here (Section 5.1, temporal stacking of
        // dependent operators).  Release: this workgroup's stores are complete and visible to the device.
        if (sh[S_FLAGS] & (SF_SYNC_WG | SF_SYNC_GRID)) {
            // every wave: its own stores have left the wave (they sit in this compute unit's caches or beyond)
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __syncthreads();
            if (sh[S_FLAGS] & SF_SYNC_GRID) {
                // every workgroup of the launch arrives once per such point; the grid was sized to be resident as a
                // whole, so all arrive; should the machine be shared and some never start, the bounded wait ends
                // with the status word set and this workgroup leaves the kernel.  One wave per workgroup makes
                // the workgroup's stores visible to the device (the caches it has to write back and, afterwards,
                // invalidate are shared by all its waves) and waits.
                ++n_sync;
                if (wave == 0) {
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                    uint32_t ok = 1;
                    if (tid == 0) {
                        GLOBAL_AS uint32_t *wsp = (GLOBAL_AS uint32_t *)args.ws;
                        __hip_atomic_fetch_add(&wsp[WS_ARRIVED], 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
                        const uint32_t target = n_sync * ngrid;
                        for (uint32_t spins = 0; __hip_atomic_load(&wsp[WS_ARRIVED], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) < target; ++spins) {
                            if (spins >= args.spin_limit || __hip_atomic_load(&wsp[WS_STATUS], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) {
                                __hip_atomic_store(&wsp[WS_STATUS], WS_STATUS_GAVE_UP, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                                ok = 0;
                                break;
                            }
                            __builtin_amdgcn_s_sleep(8);
                        }
                        red_lds[0][0] = __builtin_bit_cast(float, ok);
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                }
                __syncthreads();
                const uint32_t go = __builtin_bit_cast(uint32_t, red_lds[0][0]);
                __syncthreads();
                if (go == 0) return;
            } else {
                // (lines of the buffer that this compute unit cached before the producer wrote them must go)
                if (wave == 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                __syncthreads();
            }
        }

        // Algorithm 2: m = ceil(M / N); this workgroup runs tiles [m*id, min(M, m*(id+1))).  In a
        // spatially stacked launch N and id count the workgroups of this segment's share only.
        uint32_t sbid = bid, sgrid = ngrid;
        if (SKIP && args.rotate == 1) sbid = gnext - gbase;     // (below M: the first of its tiles here)
        if (args.rotate == 2) {
            sbid = bid >= rot ? bid - rot : bid + ngrid - rot;
            rot += M % ngrid;
            if (rot >= ngrid) rot -= ngrid;
        }
        if (sh[S_NWG] != 0) {
            sbid = bid - sh[S_WG0];
            sgrid = sh[S_NWG];
            if (sbid >= sgrid) {        // (unsigned: also true for workgroups below the share)
                seg += seg_words;
                continue;
            }
        }
        // Interleaved assignment: workgroup id runs tiles id, id + N, id + 2N, ...  At any moment the resident
        // workgroups then work on one contiguous stretch of the tensors, which the memory system of this
        // machine serves measurably faster than N streams that are far apart (the blocked ranges).
        uint32_t t_lo, t_hi, t_step;
        if (sh[S_FLAGS] & SF_INTERLEAVED) {
            t_lo = sbid < M ? sbid : M;
            t_hi = M;
            t_step = sgrid;
        } else {
            const uint32_t m = (M + sgrid - 1) / sgrid;
            const uint64_t t_lo64 = (uint64_t)m * sbid;
            t_lo = t_lo64 < M ? (uint32_t)t_lo64 : M;
            t_hi = (M - t_lo) < m ? M : t_lo + m;
            t_step = 1;
        }

        const uint32_t nct = sh[S_NCT];
        if (nct <= 1) tile_cols(gt, sh, 0, G, V, args.aliased);
        // A segment that reduces along the penultimate axis counts units (outer index, column tile) in M;
        // the workgroup walks the `inner` rows of a unit RP at a time, one row per wave and step (rin),
        // accumulating in tile registers, and runs the epilogue records after the last step.  Other
        // segments: one step per tile.
        // A segment over rows longer than a tile (SF_LONGROW) counts rows in M; the workgroup passes over a row once per
        // reduction and once more for the rest (lr_phase), each pass column tile after column tile (lr_c): a pass runs
        // the records from the start of the body up to its reduction, skipping the reductions whose value is final and
        // every store; the last pass runs to the end and stores.  Every pass over a row runs the other way round than the one
        // before (each row's first from its start, so that a row's bits do not depend on where in the launch it stands): the
        // rows in flight together are about as large as the last-level cache, and a pass that starts where the one before
        // ended finds part of its row there (RMSNorm bf16 [671, 100000] 85.4 us with all passes from the start, 81.5 so; softmax fp32
        // [671, 100003] 145.6 and 142.4).
        const bool longrow = LONG && (sh[S_FLAGS] & SF_LONGROW) != 0;
        const uint32_t n_red = longrow ? sh[S_NCTSH] : 0u;
        uint32_t lr_phase = 0, lr_c = 0;
        uint32_t lr_back = 0;               // 1: this pass runs from the row's last column tile to its first
        float racc = 0.0f, racc2 = 0.0f;    // the lane's part of the reduction of the current pass (R_ONLINE: maximum and sum)
        uint32_t rin = 0;
        for (uint32_t tile = t_lo; tile < t_hi;) {
            const uint32_t *shl = sh;
            uint32_t this_end = body_end;
            if constexpr (CRED) {
                const uint32_t inner = shl[S_INNER];
                uint32_t tile_r0 = tile;
                if (nct > 1) {          // (a single column tile was placed once, before the loop)
                    tile_r0 = sdiv_u(tile, shl[S_NCTM], shl[S_NCTSH]);
                    if (rin == 0) tile_cols(gt, shl, tile - tile_r0 * nct, G, V, args.aliased);      // the steps of a unit share its columns
                }
                if (inner != 0) {
                    const uint32_t r = rin * RP + rp;
                    tile_rows_at(gt, shl, tile_r0 * inner + r, (r < inner) && (rp < RP) && (tid < seg_threads));
                    if ((rin + 1) * RP < inner && !(shl[S_FLAGS] & SF_CSTREAM)) this_end = body + shl[S_EPILOG];
                } else {
                    tile_rows(gt, shl, tile_r0, rp, tid, RP, seg_threads);
                }
            } else {
                // tile prologue: where this tile sits, which of its lanes and chunks are valid
                uint32_t tile_r = tile;
                if (longrow) {
                    tile_cols(gt, sh, lr_back != 0 ? nct - 1 - lr_c : lr_c, G, V, args.aliased);
                } else if (nct > 1) {   // (a single column tile was placed once, before the loop)
                    tile_r = sdiv_u(tile, sh[S_NCTM], sh[S_NCTSH]);
                    tile_cols(gt, sh, tile - tile_r * nct, G, V, args.aliased);
                }
                tile_rows(gt, sh, tile_r, rp, tid, RP, seg_threads);
            }
            Wide wd;
            if constexpr (WIDE) {       // all lanes of a wave hold the same row: its place as wave-uniform values
                wd.i1 = __builtin_amdgcn_readfirstlane(gt.i1);
                wd.i2 = __builtin_amdgcn_readfirstlane(gt.i2);
                wd.i3 = __builtin_amdgcn_readfirstlane(gt.i3);
                wd.rowok = __builtin_amdgcn_readfirstlane(gt.rowok);
            }

            // the first tile of this workgroup also runs the prologue records (pinned operands)
            // (its second part runs again when the second outer index of the tile's first or last row
            // differs from that of the previous tile: an operand pinned there varies with that index only)
            uint32_t first = body;
            uint32_t red_idx = 0;           // reductions met so far in this pass over the records
            if (tile != t_lo || rin != 0) {
                first = body + shl[S_PROLOG];
                if (shl[S_PROLOGA] != shl[S_PROLOG]) {
                    const uint32_t m1 = shl[S_M1], sh1 = shl[S_SH1];
                    const uint32_t ra = tile * RP;          // prologues exist in row mode only: tile = row tile
                    const uint32_t rb = ra - t_step * RP;   // first row of the tile this workgroup ran before
                    const bool crossed = sdiv_u(ra, m1, sh1) != sdiv_u(rb, m1, sh1) ||
                                         sdiv_u(ra + RP - 1, m1, sh1) != sdiv_u(rb + RP - 1, m1, sh1);
                    if (crossed) first = body + shl[S_PROLOGA];
                }
            }
            // (the program counter is a byte offset into the code)
            u32x4s nw = fetch4b(code, first * 4);
            for (uint32_t pcb = first * 4; pcb < this_end * 4;) {
                const u32x4s cw = nw;
                // (elements are copied to scalars first: bit-casting a vector element directly is miscompiled)
                const uint32_t w = cw.x, cw1 = cw.y, cw2 = cw.z, cw3 = cw.w;
                const uint32_t op = w & 0xFF, a = (w >> 16) & 0xFF, b = w >> 24;
                const uint32_t cur = pcb >> 2;
                pcb += (w >> 6) & 0x3FCu;       // record length in words, times four
                nw = fetch4b(code, pcb);
                switch (op) {
                    case I_LOAD:
                    case I_VLOAD: {
                        // A run of consecutive load records is one group: first every record of the run issues its
                        // requests (all of them are then in flight together, each into its own destination
                        // register), then a second walk over the same records finishes them (bf16 widening in
                        // place, the chunk a ragged row ends in).
                        if constexpr (WIDE) {
                            Geo g = gt;
                            uint32_t gp = cur;
                            u32x4s rw = cw;
                            uint32_t widen = 0;             // bit r + 1: register r (bit 0: ACC) holds raw bf16 bits
                            for (;;) {
                                asm volatile("" : "+v"(g.lanecol), "+s"(g.pk), "+s"(g.cend));
                                const uint32_t r0w = rw.x, w1 = rw.y, r2w = rw.z, r3w = rw.w;
                                const uint32_t rop = r0w & 0xFF, ra = (r0w >> 16) & 0xFF;
                                const uint32_t ti = w1 & 0xFF, dt = (w1 >> 8) & 0xFF;
                                int64_t off = (int64_t)wd.i1 * DVM_I64(r2w, r3w) + (int64_t)g.colbase;
                                if (rop == I_VLOAD) {
                                    const u32x4s hw = fetch4(code, gp + 4);
                                    const uint32_t h0 = hw.x, h1 = hw.y, h2 = hw.z, h3 = hw.w;
                                    off += (int64_t)wd.i2 * DVM_I64(h0, h1) + (int64_t)wd.i3 * DVM_I64(h2, h3);
                                }
                                const char *rowbase = (const char *)DVM_TENSOR(tbase + ti) + off * (dt == 0 ? 4 : 2);
                                if (g.chunks()) {
                                    if (!LONG && ((w1 >> 16) & MF_STREAM)) {      // (long rows are read once per pass: no hint)
                                        if (dt != 0) { if constexpr (K >= 8) DVM_ISSUE_WIDE(1, 8, true) }
                                        else if (V == 4) DVM_ISSUE_WIDE(0, 4, true)
                                        else { if constexpr (K >= 8) DVM_ISSUE_WIDE(0, 8, true) }
                                    } else {
                                        if (dt != 0) { if constexpr (K >= 8) DVM_ISSUE_WIDE(1, 8, false) }
                                        else if (V == 4) DVM_ISSUE_WIDE(0, 4, false)
                                        else { if constexpr (K >= 8) DVM_ISSUE_WIDE(0, 8, false) }
                                    }
                                }
                                if (dt != 0) widen |= ra == SRC_ACC ? 1u : 2u << ra;
                                gp += (r0w >> 8) & 0xFF;
                                if (gp >= this_end) break;
                                rw = fetch4(code, gp);
                                const uint32_t nop = rw.x & 0xFF;
                                if (nop != I_LOAD && nop != I_VLOAD) break;
                            }
                            if (widen != 0) {           // the bf16 registers need their second half
                                if constexpr (K >= 8) {
                                    if (widen & 1u) finish_tile<K, 1, 8>(acc, nullptr, g);
                                    if (widen & 2u) finish_tile<K, 1, 8>(r0, nullptr, g);
                                    if constexpr (NR > 1) if (widen & 4u) finish_tile<K, 1, 8>(r1, nullptr, g);
                                    if constexpr (NR > 2) if (widen & 8u) finish_tile<K, 1, 8>(r2, nullptr, g);
                                    if constexpr (NR > 3) if (widen & 16u) finish_tile<K, 1, 8>(r3, nullptr, g);
                                    if constexpr (NR > 4) if (widen & 32u) finish_tile<K, 1, 8>(r4, nullptr, g);
                                    if constexpr (NR > 5) if (widen & 64u) finish_tile<K, 1, 8>(r5, nullptr, g);
                                }
                            }
                            pcb = gp * 4;
                            nw = fetch4b(code, pcb);
                            break;
                        }
                        DVM_GEO()
                        uint32_t gp = cur;              // word offset of the record being issued
                        u32x4s rw = cw;
                        bool finish = g.part() != 0;
                        for (;;) {
                            // (the lane's column is made opaque once per record: otherwise the chunk addresses of every
                            // dtype and chunk width are computed ahead of the loop and held in registers throughout)
                            asm volatile("" : "+v"(g.lanecol), "+s"(g.pk), "+s"(g.cend));
                            const uint32_t r0w = rw.x, w1 = rw.y, r2w = rw.z, r3w = rw.w;
                            const uint32_t rop = r0w & 0xFF, ra = (r0w >> 16) & 0xFF;
                            const uint32_t ti = w1 & 0xFF, dt = (w1 >> 8) & 0xFF;
                            int64_t off = (int64_t)g.i1 * DVM_I64(r2w, r3w) + (int64_t)g.colbase;
                            if (rop == I_VLOAD) {
                                const u32x4s hw = fetch4(code, gp + 4);
                                const uint32_t h0 = hw.x, h1 = hw.y, h2 = hw.z, h3 = hw.w;
                                off += (int64_t)g.i2 * DVM_I64(h0, h1) + (int64_t)g.i3 * DVM_I64(h2, h3);
                            }
                            const uint32_t es = dt == 0 ? 4 : 2;
                            gcptr rowp = (gcptr)DVM_TENSOR(tbase + ti) + off * es;
                            const bool nt = ((w1 >> 16) & MF_STREAM) != 0;
                            if (ra == SRC_ACC) {
                                request_dispatch<K>(acc, dt, V, nt, rowp, g);
                            } else {
                                DVM_WITH_R(ra, rr, (request_dispatch<K>(rr, dt, V, nt, rowp, g)))
                            }
                            finish |= dt != 0;
                            gp += (r0w >> 8) & 0xFF;
                            if (gp >= this_end) break;
                            rw = fetch4(code, gp);
                            const uint32_t nop = rw.x & 0xFF;
                            if (nop != I_LOAD && nop != I_VLOAD) break;
                        }
                        if (finish) {
                            for (uint32_t fp = cur; fp < gp;) {
                                asm volatile("" : "+v"(g.lanecol), "+s"(g.pk), "+s"(g.cend));
                                const u32x4s fw = fetch4(code, fp);
                                const uint32_t r0w = fw.x, w1 = fw.y, r2w = fw.z, r3w = fw.w;
                                const uint32_t rop = r0w & 0xFF, ra = (r0w >> 16) & 0xFF;
                                const uint32_t ti = w1 & 0xFF, dt = (w1 >> 8) & 0xFF;
                                gcptr rowp = nullptr;
                                if (g.part() != 0) {       // (only the ragged chunk needs the address again)
                                    int64_t off = (int64_t)g.i1 * DVM_I64(r2w, r3w) + (int64_t)g.colbase;
                                    if (rop == I_VLOAD) {
                                        const u32x4s hw = fetch4(code, fp + 4);
                                        const uint32_t h0 = hw.x, h1 = hw.y, h2 = hw.z, h3 = hw.w;
                                        off += (int64_t)g.i2 * DVM_I64(h0, h1) + (int64_t)g.i3 * DVM_I64(h2, h3);
                                    }
                                    rowp = (gcptr)DVM_TENSOR(tbase + ti) + off * (dt == 0 ? 4 : 2);
                                }
                                if (ra == SRC_ACC) {
                                    finish_dispatch<K>(acc, dt, V, rowp, g);
                                } else {
                                    DVM_WITH_R(ra, rr, (finish_dispatch<K>(rr, dt, V, rowp, g)))
                                }
                                fp += (r0w >> 8) & 0xFF;
                            }
                        }
                        pcb = gp * 4;                   // resume behind the group
                        nw = fetch4b(code, pcb);
                        break;
                    }
                    case I_STORE:
                    case I_VSTORE: {
                        if (longrow && lr_phase != n_red) break;    // (only the last pass over a long row stores)
                        if constexpr (WIDE) {       // (rows consist of chunks in this instantiation)
                            if (wd.rowok) {
                                Geo g = gt;
                                asm volatile("" : "+v"(g.lanecol), "+s"(g.pk), "+s"(g.cend));
                                const uint32_t w1 = cw1;
                                const uint32_t ti = w1 & 0xFF, dt = (w1 >> 8) & 0xFF;
                                int64_t off = (int64_t)wd.i1 * DVM_I64(cw2, cw3) + (int64_t)g.colbase;
                                if (op == I_VSTORE) {
                                    const u32x4s hw = fetch4(code, cur + 4);
                                    const uint32_t h0 = hw.x, h1 = hw.y, h2 = hw.z, h3 = hw.w;
                                    off += (int64_t)wd.i2 * DVM_I64(h0, h1) + (int64_t)wd.i3 * DVM_I64(h2, h3);
                                }
                                char *rowbase = (char *)DVM_TENSOR(tbase + ti) + off * (dt == 0 ? 4 : 2);
                                if (a == SRC_ACC) {
                                    if (b != 0) tile_bins<K, B_MUL>(acc, DVM_GET_S(b - 1));
                                    if (g.ragged() == 0) store_wide_dispatch<K, true>(acc, dt, V, rowbase, g);
                                    else store_wide_dispatch<K, false>(acc, dt, V, rowbase, g);
                                } else if (g.ragged() == 0) {
                                    DVM_WITH_R(a, rr, (store_wide_dispatch<K, true>(rr, dt, V, rowbase, g)))
                                } else {
                                    DVM_WITH_R(a, rr, (store_wide_dispatch<K, false>(rr, dt, V, rowbase, g)))
                                }
                            }
                            break;
                        }
                        DVM_GEO()
                        const uint32_t w1 = cw1;
                        const uint32_t ti = w1 & 0xFF, dt = (w1 >> 8) & 0xFF;
                        int64_t off = (int64_t)g.i1 * DVM_I64(cw2, cw3) + (int64_t)g.colbase;
                        if (op == I_VSTORE) {
                            const u32x4s hw = fetch4(code, cur + 4);
                            const uint32_t h0 = hw.x, h1 = hw.y, h2 = hw.z, h3 = hw.w;
                            off += (int64_t)g.i2 * DVM_I64(h0, h1) + (int64_t)g.i3 * DVM_I64(h2, h3);
                        }
                        const uint32_t es = dt == 0 ? 4 : 2;
                        gptr base = (gptr)DVM_TENSOR(tbase + ti);
                        gptr rowp = base + off * es;
                        if (a == SRC_ACC) {
                            // (b: a row scalar to multiply by first; the accumulator's value is dead afterwards)
                            if (b != 0) tile_bins<K, B_MUL>(acc, DVM_GET_S(b - 1));
                            store_dispatch<K>(acc, dt, V, rowp, g);
                        } else {
                            DVM_WITH_R(a, rr, store_dispatch<K>(rr, dt, V, rowp, g))
                        }
                        break;
                    }
                    case I_LOADS: {
                        DVM_GEO()
                        const uint32_t w1 = cw1;
                        const uint32_t ti = w1 & 0xFF, dt = (w1 >> 8) & 0xFF;
                        const u32x4s hw = fetch4(code, cur + 4);
                        const uint32_t h0 = hw.x, h1 = hw.y, h2 = hw.z, h3 = hw.w;
                        const int64_t off = row_offset(g, DVM_I64(cw2, cw3), DVM_I64(h0, h1), DVM_I64(h2, h3));
                        gcptr base = (gcptr)DVM_TENSOR(tbase + ti);
                        float v;       // a lane outside the tensor reads row 0: valid memory, value unused
                        if (dt == 0) v = *(const GLOBAL_AS float *)(base + off * 4);
                        else v = bf16_lo(*(const GLOBAL_AS uint16_t *)(base + off * 2));
                        DVM_SET_S(a, v);
                        break;
                    }
                    case I_STORES: {
                        if (longrow && (lr_phase != n_red || gt.colbase != 0)) break;     // (once per row, in its last pass)
                        DVM_GEO()
                        const uint32_t w1 = cw1;
                        const uint32_t ti = w1 & 0xFF, dt = (w1 >> 8) & 0xFF;
                        const u32x4s hw = fetch4(code, cur + 4);
                        const uint32_t h0 = hw.x, h1 = hw.y, h2 = hw.z, h3 = hw.w;
                        const int64_t off = row_offset(g, DVM_I64(cw2, cw3), DVM_I64(h0, h1), DVM_I64(h2, h3));
                        gptr base = (gptr)DVM_TENSOR(tbase + ti);
                        const float v = DVM_GET_S(a);
                        const bool ok = g.rowok && g.lanecol == 0 && g.colbase == 0;
                        if (dt == 0) st_b32(base + off * 4, v, ok);
                        else st_b16(base + off * 2, (uint32_t)pack_bf16(v), ok);
                        break;
                    }
                    case I_MOVRA:
                        DVM_WITH_R(a, rr, rr = acc)
                        break;
                    case I_MOVAR:
                        DVM_WITH_R(a, rr, acc = rr)
                        break;
                    case I_UN:
                        tile_un_dispatch<K>(acc, b);
                        break;
                    case I_BIN:
                        if (a < SRC_S0) {
                            DVM_WITH_R(a, rr, tile_bin_dispatch<K>(acc, rr, b))
                        } else if (a == SRC_ACC) {
                            const Tile<K> t = acc;
                            tile_bin_dispatch<K>(acc, t, b);
                        } else {
                            const float s = a == SRC_IMM ? __builtin_bit_cast(float, cw1) : DVM_GET_S(a - SRC_S0);
                            tile_bins_dispatch<K>(acc, s, b);
                        }
                        break;
                    case I_CACC: if constexpr (CRED) {      // the first step of a unit starts the accumulator, the others combine into it
                        // (a wave whose row lies past the end of the unit contributes nothing)
                        const bool ok = gt.rowok;
                        if (rin == 0) {
                            const float ident = b == R_SUM ? 0.0f : (b == R_MAX ? -__builtin_inff() : __builtin_inff());
                            DVM_WITH_R(a, rr, sfor<K>([&]<int I>() LI { TV(rr, I) = ok ? TV(acc, I) : ident; }))
                        } else if (b == R_SUM) {
                            DVM_WITH_R(a, rr, sfor<K>([&]<int I>() LI { TV(rr, I) = ok ? TV(rr, I) + TV(acc, I) : TV(rr, I); }))
                        } else if (b == R_MAX) {
                            DVM_WITH_R(a, rr, sfor<K>([&]<int I>() LI { TV(rr, I) = ok ? f_maxp(TV(rr, I), TV(acc, I)) : TV(rr, I); }))
                        } else {
                            DVM_WITH_R(a, rr, sfor<K>([&]<int I>() LI { TV(rr, I) = ok ? f_minp(TV(rr, I), TV(acc, I)) : TV(rr, I); }))
                        }
                    }
                        break;
                    case I_CSTREAM: if constexpr (CRED && K <= 8) {      // (the encoder emits it for these variants only)
                        // this wave's share of the unit's rows (every RP-th, starting at its own), U rows in flight:
                        // all their loads are issued before the first is combined into the accumulator
                        DVM_GEO()
                        const uint32_t w1 = cw1;
                        const uint32_t ti = w1 & 0xFF, dt = (w1 >> 8) & 0xFF;
                        const bool nt = ((w1 >> 16) & MF_STREAM) != 0;
                        const int64_t st1 = DVM_I64(cw2, cw3);
                        const u32x4s hw = fetch4(code, cur + 4);
                        const uint32_t h0 = hw.x, h1 = hw.y, h2 = hw.z, h3 = hw.w;
                        const uint32_t es = dt == 0 ? 4 : 2;
                        // (a wave without a valid first row decomposed row 0: in bounds, and it combines nothing)
                        const int64_t off0 = (int64_t)g.i2 * DVM_I64(h0, h1) + (int64_t)g.i3 * DVM_I64(h2, h3) + (int64_t)g.colbase;
                        gcptr base = (gcptr)DVM_TENSOR(tbase + ti);
                        const uint32_t inner_n = sh[S_INNER];
                        const float ident = b == R_SUM ? 0.0f : (b == R_MAX ? -__builtin_inff() : __builtin_inff());
                        constexpr int U = K <= 4 ? 6 : 4;       // (as many as the registers hold)
                        // (the order of the rows is the one dvm_colreduce takes for the same segment as a launch of its own)
                        const uint32_t q = (w1 >> 24) > 1 ? w1 >> 24 : 1u, step = RP * q;
                        Tile<K> sum;
                        sfor<K>([&]<int I>() LI { TV(sum, I) = ident; });
                        for (uint32_t first_r = wave, j = 0; wave < RP && j < q; ++j, first_r += RP) {
                            Tile<K> part;
                            sfor<K>([&]<int I>() LI { TV(part, I) = ident; });
                            for (uint32_t r = first_r; r < inner_n; r += step * U) {
                                Raw<K> raw[U];
                                sfor<U>([&]<int J>() LI {
                                    const uint32_t ru = r + (uint32_t)J * step;
                                    const uint32_t rc = ru < inner_n ? ru : r;      // past the end: read row r again, unused
                                    request_staged_dispatch<K>(raw[J], dt, V, nt, base + (off0 + (int64_t)rc * st1) * es, g);
                                });
                                sfor<U>([&]<int J>() LI {
                                    if (r + (uint32_t)J * step < inner_n) {
                                        if (b == R_SUM) combine_staged_dispatch<K, B_ADD>(part, raw[J], dt, V, g);
                                        else if (b == R_MAX) combine_staged_dispatch<K, B_MAX>(part, raw[J], dt, V, g);
                                        else combine_staged_dispatch<K, B_MIN>(part, raw[J], dt, V, g);
                                    }
                                });
                            }
                            if (j == 0) sum = part;
                            else if (b == R_SUM) tile_bin<K, B_ADD>(sum, part);
                            else if (b == R_MAX) tile_bin<K, B_MAX>(sum, part);
                            else tile_bin<K, B_MIN>(sum, part);
                        }
                        DVM_WITH_R(a, rr, rr = sum)
                    }
                        break;
                    case I_CCOMB:       // every wave ends up with the combination, taken in wave order; the first wave stores
                        if constexpr (CRED) if (sh[S_INNER] != 0 && RP > 1) {
                            uint32_t lane = tid & 63u;
                            asm volatile("" : "+v"(lane));      // (keeps the LDS addresses out of the registers that live across the loop)
                            DVM_WITH_R(a, rr, sfor<K / 4>([&]<int Q>() LI {
                                if (wave < RP) {
                                    float *mine = &comb_lds[(wave * 64u + lane) * 4u];
                                    mine[0] = TV(rr, 4 * Q); mine[1] = TV(rr, 4 * Q + 1); mine[2] = TV(rr, 4 * Q + 2); mine[3] = TV(rr, 4 * Q + 3);
                                }
                                __syncthreads();
                                // (in pairs: a wave writes its own slot in the steps in which no other wave reads it)
                                if (cw1 != 0) {
                                    for (uint32_t s = 1; s < RP; s <<= 1) {
                                        if (wave < RP && (wave & (2u * s - 1u)) == 0 && wave + s < RP) {
                                            float *mine = &comb_lds[(wave * 64u + lane) * 4u];
                                            const float *p = mine + s * 256u;
                                            if (b == R_SUM) { mine[0] += p[0]; mine[1] += p[1]; mine[2] += p[2]; mine[3] += p[3]; }
                                            else if (b == R_MAX) { mine[0] = f_maxp(mine[0], p[0]); mine[1] = f_maxp(mine[1], p[1]); mine[2] = f_maxp(mine[2], p[2]); mine[3] = f_maxp(mine[3], p[3]); }
                                            else { mine[0] = f_minp(mine[0], p[0]); mine[1] = f_minp(mine[1], p[1]); mine[2] = f_minp(mine[2], p[2]); mine[3] = f_minp(mine[3], p[3]); }
                                        }
                                        __syncthreads();
                                    }
                                }
                                float c0 = comb_lds[lane * 4u], c1 = comb_lds[lane * 4u + 1], c2 = comb_lds[lane * 4u + 2], c3 = comb_lds[lane * 4u + 3];
                                for (uint32_t o = 1; cw1 == 0 && o < RP; ++o) {
                                    const float *p = &comb_lds[(o * 64u + lane) * 4u];
                                    if (b == R_SUM) { c0 += p[0]; c1 += p[1]; c2 += p[2]; c3 += p[3]; }
                                    else if (b == R_MAX) { c0 = f_maxp(c0, p[0]); c1 = f_maxp(c1, p[1]); c2 = f_maxp(c2, p[2]); c3 = f_maxp(c3, p[3]); }
                                    else { c0 = f_minp(c0, p[0]); c1 = f_minp(c1, p[1]); c2 = f_minp(c2, p[2]); c3 = f_minp(c3, p[3]); }
                                }
                                __syncthreads();
                                TV(rr, 4 * Q) = c0; TV(rr, 4 * Q + 1) = c1; TV(rr, 4 * Q + 2) = c2; TV(rr, 4 * Q + 3) = c3;
                            }))
                            gt.rowok = (rp == 0) && (tid < seg_threads);
                        }
                        break;
                    case I_SEL:         // every pair of registers gets its own copy of the loop: no tile is copied
                        DVM_WITH_R(a, xa, DVM_WITH_R2(b, xb, sfor<K>([&]<int I>() LI { TV(acc, I) = TV(acc, I) != 0.0f ? TV(xa, I) : TV(xb, I); })))
                        break;
                    case I_FMA: {
                        const float s = cw1 != 0 ? DVM_GET_S(cw1 - 1) : 1.0f;
                        if constexpr (NR <= 4) {        // one loop per (multiplier, addend) pair of registers
                            if (cw1 == 0) {
                                DVM_WITH_R(a, xa, DVM_WITH_R2(b, xb, sfor<K>([&]<int I>() LI { TV(acc, I) = f_fma(TV(acc, I), TV(xa, I), TV(xb, I)); })))
                            } else if (b == FMA_NO_ADDEND) {
                                DVM_WITH_R(a, xa, sfor<K>([&]<int I>() LI { TV(acc, I) = TV(acc, I) * s * TV(xa, I); }))
                            } else {
                                DVM_WITH_R(a, xa, DVM_WITH_R2(b, xb, sfor<K>([&]<int I>() LI { TV(acc, I) = f_fma(TV(acc, I) * s, TV(xa, I), TV(xb, I)); })))
                            }
                        } else {                        // many registers: the pairs would multiply the code size
                            if (cw1 != 0) tile_bins<K, B_MUL>(acc, s);
                            DVM_WITH_R(a, xa, (tile_bin<K, B_MUL>(acc, xa)))
                            if (b != FMA_NO_ADDEND) {
                                DVM_WITH_R(b, xb, (tile_bin<K, B_ADD>(acc, xb)))
                            }
                        }
                        break;
                    }
                    // (the sum rounds once and the differences twice, as the records do that a program without I_MAC has: see the encoder)
                    case I_MAC: if constexpr (!(LONG && WIDE)) {       // (long rows with such a record run in the instantiation for any launch)
                        if (cw1 == MAC_ADD) {
                            DVM_WITH_R(a, xa, DVM_WITH_R2(b, xb, sfor<K>([&]<int I>() LI { TV(acc, I) = f_fma(TV(xa, I), TV(xb, I), TV(acc, I)); })))
                        } else if (cw1 == MAC_SUB) {
                            DVM_WITH_R(a, xa, DVM_WITH_R2(b, xb, sfor<K>([&]<int I>() LI { TV(acc, I) = f_sub_mul(TV(acc, I), TV(xa, I), TV(xb, I)); })))
                        } else {
                            DVM_WITH_R(a, xa, DVM_WITH_R2(b, xb, sfor<K>([&]<int I>() LI { TV(acc, I) = f_mul_sub(TV(xa, I), TV(xb, I), TV(acc, I)); })))
                        }
                    }
                        break;
                    case I_LDSCOPY: {
                        // every thread of the workgroup copies 16-byte pieces of the tensor's only row into the image;
                        // pieces that reach beyond the row's end are put together element by element, zero-filled
                        const uint32_t ti = cw1 & 0xFF, dt = (cw1 >> 8) & 0xFF;
                        gcptr src = (gcptr)DVM_TENSOR(tbase + ti);
                        // (a program with LDS images has one column tile: the tile's columns are the row's)
                        const uint32_t n = gt.part_n();
                        const uint32_t d0 = gt.slide() != 0 ? gt.cend : gt.cend + n;
                        const uint32_t full = gt.slide() != 0 ? d0 - n : d0, back = gt.slide() != 0 ? V - n : 0u;
                        lds_copy_row((LDS_AS char *)comb_lds + cw2, cw3 >> 4, src, d0, full, back, dt, tid, blockDim.x);
                        if (b != 0) __syncthreads();
                        break;
                    }
                    case I_LFMA: {
                        const float s = cw1 != 0 ? DVM_GET_S(cw1 - 1) : 1.0f;
                        const uint32_t la = a & 0xF, lb = a >> 4;
                        const LDS_AS char *pa = (const LDS_AS char *)comb_lds + cw2;
                        const LDS_AS char *pb = (const LDS_AS char *)comb_lds + cw3;
                        const uint32_t lc = gt.lanecol;
                        if (V == 4) {
                            if (la != LFMA_NONE && lb != LFMA_NONE) lds_fma<K, 4, true, true>(acc, s, pa, pb, false, false, lc, gt);
                            else if (la != LFMA_NONE) lds_fma<K, 4, true, false>(acc, s, pa, pb, false, false, lc, gt);
                            else lds_fma<K, 4, false, true>(acc, s, pa, pb, false, false, lc, gt);
                        } else {
                            if constexpr (K >= 8) {
                                if (la != LFMA_NONE && lb != LFMA_NONE) lds_fma<K, 8, true, true>(acc, s, pa, pb, (b & 1u) != 0, (b & 2u) != 0, lc, gt);
                                else if (la != LFMA_NONE) lds_fma<K, 8, true, false>(acc, s, pa, pb, (b & 1u) != 0, false, lc, gt);
                                else lds_fma<K, 8, false, true>(acc, s, pa, pb, false, (b & 2u) != 0, lc, gt);
                            }
                        }
                        break;
                    }
                    case I_RED: {
                        if (longrow) {
                            const uint32_t mine = red_idx++;
                            if (mine < lr_phase) break;         // its value is final: S[a] holds it
                        }
                        DVM_GEO()
                        // A row that spans gw waves: exchange the per-wave results through LDS.  Two buffers alternate, so
                        // one barrier per reduction is enough.
                        auto exchange = [&](float x, uint32_t kind) LI {
                            if (gw > 1) {
                                red_lds[red_par][wave & 15] = x;     // every lane of the wave holds the same value
                                __syncthreads();
                                x = red_lds[red_par][w0i & 15];
                                for (uint32_t i = 1; i < gw; ++i) {
                                    const float o = red_lds[red_par][(w0i + i) & 15];
                                    x = kind == R_MAX ? f_maxp(x, o) : (kind == R_MIN ? f_minp(x, o) : x + o);
                                }
                                red_par ^= 1;
                            }
                            return x;
                        };
                        float v;
                        if (longrow) {
                            // this pass's reduction: the lane's part of this column tile joins those of the tiles before;
                            // after the row's last tile the lanes (and waves) are combined as for a short row
                            const uint32_t kind = b & R_KIND;
                            const float part = lane_reduce_dispatch<K>(acc, g, V, kind);
                            const float before = racc;
                            racc = lr_c == 0 ? part : (kind == R_MAX ? f_maxp(racc, part) : (kind == R_MIN ? f_minp(racc, part) : racc + part));
                            pcb = this_end * 4;                 // the pass ends here
                            if (b & R_ONLINE) {
                                // The sum of exp(x - maximum) in the pass of the maximum: the lane sums against its own maximum
                                // so far and rescales the sum when that grows, which saves one of the three passes of a softmax
                                // over the row.  (Nothing but -inf so far: the exponentials are taken against 0 and are 0.)
                                const float neg = -__builtin_inff();
                                const float ms = racc == neg ? 0.0f : racc;
                                tile_bins<K, B_EXPSUB>(acc, ms);
                                const float add = lane_reduce<K, R_SUM>(acc, g, V);
                                racc2 = lr_c == 0 ? add : f_fma(racc2, f_exp2((before - ms) * LOG2E), add);
                                if (lr_c + 1 < nct) break;
                                v = exchange(wave_allreduce<R_MAX>(racc, width), R_MAX);
                                const float vs = v == neg ? 0.0f : v;
                                float sum = exchange(wave_allreduce<R_SUM>(racc2 * f_exp2((racc - vs) * LOG2E), width), R_SUM);
                                sum = v == neg ? __builtin_nanf("") : sum;      // (a row of -inf alone: -inf - -inf)
                                DVM_SET_S(a, v);
                                const u32x4s sr = fetch4(code, cur + 2 * LEN_REC);      // the record of the sum
                                const uint32_t sw = sr.x, sw1 = sr.y, sw2 = sr.z, sw3 = sr.w;
                                sum = f_fma(sum, __builtin_bit_cast(float, sw2), __builtin_bit_cast(float, sw3));
                                if (sw1 != U_NONE) sum = un_dyn(sw1, sum);
                                DVM_SET_S((sw >> 16) & 0xFF, sum);
                                ++lr_phase;                     // both reductions are final
                                break;
                            }
                            if (lr_c + 1 < nct) break;
                            v = wave_allreduce_dispatch(racc, kind, width);
                            v = exchange(v, kind);
                        } else {
                            v = reduce_dispatch<K>(acc, g, V, b, width);
                            v = exchange(v, b);
                        }
                        // the row-scalar ops folded into this record: U(v * scale + shift)
                        v = f_fma(v, __builtin_bit_cast(float, cw2), __builtin_bit_cast(float, cw3));
                        if (cw1 != U_NONE) v = un_dyn(cw1, v);
                        DVM_SET_S(a, v);
                        break;
                    }
                    case I_SOP: {
                        const uint32_t w1 = cw1;
                        const uint32_t kind = w1 & 0xFF, srck = (w1 >> 8) & 0xFF, c = (w1 >> 16) & 0xFF;
                        const float x = DVM_GET_S(b);
                        float r;
                        if (kind >= SOP_UNARY) {
                            r = un_dyn(kind - SOP_UNARY, x);
                        } else {
                            const float y = srck == 1 ? __builtin_bit_cast(float, cw2) : DVM_GET_S(c);
                            r = bin_dyn(kind, x, y);
                        }
                        DVM_SET_S(a, r);
                        break;
                    }
                    default:
                        break;
                }
            }
            if constexpr (CRED) {   // next step of this unit, or the next tile
                const uint32_t inner = sh[S_INNER];
                if (inner == 0 || (rin + 1) * RP >= inner || (sh[S_FLAGS] & SF_CSTREAM)) { rin = 0; tile += t_step; } else { ++rin; }
            } else if (longrow) {
                if (++lr_c == nct) {
                    lr_c = 0;
                    lr_back ^= 1;
                    if (++lr_phase > n_red) { lr_phase = 0; lr_back = 0; tile += t_step; }      // (nothing of the next row is cached)
                }
            } else {
                tile += t_step;
            }
        }
        if (SKIP && args.rotate == 1) {         // (one past the last tile this workgroup ran here, in steps of the grid)
            gnext += (M - sbid + ngrid - 1) / ngrid * ngrid;
            gbase += M;
        }
        seg += seg_words;
    }
    }   // (sets)
}

// ------------------------------------------------------------------------------------------
// interpreter variants and host side
// ------------------------------------------------------------------------------------------
// X(K, NR, largest workgroup, resident waves per SIMD the register allocation aims for).  Every
// variant is compiled in a translation unit of its own (this file with -DDVM_VARIANT_K=.. etc.),
// which defines the kernel and a launcher; the translation unit without those macros holds the
// host side.  The build script reads this list.
#define DVM_VARIANT_LIST(X) \
    X(4, 2, 1024, 8) X(4, 6, 1024, 8) X(8, 2, 1024, 7) X(8, 6, 512, 4) \
    X(16, 2, 1024, 6) X(16, 4, 512, 4) X(16, 6, 512, 3) X(32, 2, 256, 4) X(32, 4, 256, 2) X(64, 1, 256, 3)

// (the variants also built as the instantiation that runs reductions along the penultimate axis)
#define DVM_CRED_VARIANT_LIST(X) \
    X(4, 2, 1024, 4) X(4, 6, 1024, 4) X(8, 2, 1024, 4) X(8, 6, 512, 4) X(16, 6, 512, 3) X(32, 2, 256, 3) X(32, 4, 256, 2)

#define DVM_LAUNCHER_NAME_(K, NR) dvm_vm_launch_##K##_##NR
#define DVM_LAUNCHER_NAME(K, NR) DVM_LAUNCHER_NAME_(K, NR)
#define DVM_CRED_LAUNCHER_NAME_(K, NR) dvm_vm_launch_c_##K##_##NR
#define DVM_CRED_LAUNCHER_NAME(K, NR) DVM_CRED_LAUNCHER_NAME_(K, NR)
#define DVM_WIDE_LAUNCHER_NAME_(K, NR) dvm_vm_launch_w_##K##_##NR
#define DVM_WIDE_LAUNCHER_NAME(K, NR) DVM_WIDE_LAUNCHER_NAME_(K, NR)
#define DVM_ANY_LAUNCHER_NAME_(K, NR) dvm_vm_launch_a_##K##_##NR
#define DVM_ANY_LAUNCHER_NAME(K, NR) DVM_ANY_LAUNCHER_NAME_(K, NR)
#define DVM_VISIT_LAUNCHER_NAME_(K, NR) dvm_vm_launch_v_##K##_##NR
#define DVM_VISIT_LAUNCHER_NAME(K, NR) DVM_VISIT_LAUNCHER_NAME_(K, NR)
#define DVM_VISIT_WIDE_LAUNCHER_NAME_(K, NR) dvm_vm_launch_vw_##K##_##NR
#define DVM_VISIT_WIDE_LAUNCHER_NAME(K, NR) DVM_VISIT_WIDE_LAUNCHER_NAME_(K, NR)
#define DVM_LONG_WIDE_LAUNCHER_NAME_(K, NR) dvm_vm_launch_lw_##K##_##NR
#define DVM_LONG_WIDE_LAUNCHER_NAME(K, NR) DVM_LONG_WIDE_LAUNCHER_NAME_(K, NR)

}  // namespace

#ifdef DVM_VARIANT_K
// ---- one interpreter variant: kernel instantiation + launcher ---------------------------------
// launcher(grid, block, lds_bytes, stream, kargs, blocks_per_cu): blocks_per_cu null: launch; else only report how
// many workgroups of this size one compute unit holds at a time.  Returns the hipError_t of the calls it made.
#if defined(DVM_VARIANT_CRED)
#define DVM_THIS_LAUNCHER DVM_CRED_LAUNCHER_NAME(DVM_VARIANT_K, DVM_VARIANT_NR)
#define DVM_THIS_KERNEL dvm_vm_kernel<DVM_VARIANT_K, DVM_VARIANT_NR, DVM_VARIANT_MAXT, DVM_VARIANT_WAVES, true, false, false>
#elif defined(DVM_VARIANT_LONG) && defined(DVM_VARIANT_WIDE)
#define DVM_THIS_LAUNCHER DVM_LONG_WIDE_LAUNCHER_NAME(DVM_VARIANT_K, DVM_VARIANT_NR)
#define DVM_THIS_KERNEL dvm_vm_kernel<DVM_VARIANT_K, DVM_VARIANT_NR, DVM_VARIANT_MAXT, DVM_VARIANT_WAVES, false, true, true>
#elif defined(DVM_VARIANT_ANY)
#define DVM_THIS_LAUNCHER DVM_ANY_LAUNCHER_NAME(DVM_VARIANT_K, DVM_VARIANT_NR)
#define DVM_THIS_KERNEL dvm_vm_kernel<DVM_VARIANT_K, DVM_VARIANT_NR, DVM_VARIANT_MAXT, DVM_VARIANT_WAVES, false, false, true>
#elif defined(DVM_VARIANT_WIDE) && defined(DVM_VARIANT_VISIT)
#define DVM_THIS_LAUNCHER DVM_VISIT_WIDE_LAUNCHER_NAME(DVM_VARIANT_K, DVM_VARIANT_NR)
#define DVM_THIS_KERNEL dvm_vm_kernel<DVM_VARIANT_K, DVM_VARIANT_NR, DVM_VARIANT_MAXT, DVM_VARIANT_WAVES, false, true, false>
#elif defined(DVM_VARIANT_VISIT)
#define DVM_THIS_LAUNCHER DVM_VISIT_LAUNCHER_NAME(DVM_VARIANT_K, DVM_VARIANT_NR)
#define DVM_THIS_KERNEL dvm_vm_kernel<DVM_VARIANT_K, DVM_VARIANT_NR, DVM_VARIANT_MAXT, DVM_VARIANT_WAVES, false, false, false>
#elif defined(DVM_VARIANT_WIDE)
#define DVM_THIS_LAUNCHER DVM_WIDE_LAUNCHER_NAME(DVM_VARIANT_K, DVM_VARIANT_NR)
#define DVM_THIS_KERNEL dvm_vm_kernel<DVM_VARIANT_K, DVM_VARIANT_NR, DVM_VARIANT_MAXT, DVM_VARIANT_WAVES, false, true, false>
#else
#define DVM_THIS_LAUNCHER DVM_LAUNCHER_NAME(DVM_VARIANT_K, DVM_VARIANT_NR)
#define DVM_THIS_KERNEL dvm_vm_kernel<DVM_VARIANT_K, DVM_VARIANT_NR, DVM_VARIANT_MAXT, DVM_VARIANT_WAVES, false, false, false>
#endif
extern "C" int DVM_THIS_LAUNCHER(unsigned grid, unsigned block, unsigned lds_bytes, void *stream, const void *kargs, int *blocks_per_cu) {
    if (blocks_per_cu) return (int)hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, DVM_THIS_KERNEL, (int)block, lds_bytes);
    hipLaunchKernelGGL((DVM_THIS_KERNEL), dim3(grid), dim3(block), lds_bytes, (hipStream_t)stream, *(const KArgs *)kargs);
    return (int)hipGetLastError();
}
#else
// ---- host side: dvm_run ---------------------------------------------------------------------
#define X(K, NR, MAXT, W) extern "C" int DVM_LAUNCHER_NAME(K, NR)(unsigned, unsigned, unsigned, void *, const void *, int *);
DVM_VARIANT_LIST(X)
#undef X
#define X(K, NR, MAXT, W) extern "C" int DVM_WIDE_LAUNCHER_NAME(K, NR)(unsigned, unsigned, unsigned, void *, const void *, int *);
DVM_VARIANT_LIST(X)
#undef X
#define X(K, NR, MAXT, W) extern "C" int DVM_ANY_LAUNCHER_NAME(K, NR)(unsigned, unsigned, unsigned, void *, const void *, int *);
DVM_VARIANT_LIST(X)
#undef X
#define X(K, NR, MAXT, W) extern "C" int DVM_LONG_WIDE_LAUNCHER_NAME(K, NR)(unsigned, unsigned, unsigned, void *, const void *, int *);
DVM_VARIANT_LIST(X)
#undef X
#define X(K, NR, MAXT, W) extern "C" int DVM_VISIT_LAUNCHER_NAME(K, NR)(unsigned, unsigned, unsigned, void *, const void *, int *);
DVM_VARIANT_LIST(X)
#undef X
#define X(K, NR, MAXT, W) extern "C" int DVM_VISIT_WIDE_LAUNCHER_NAME(K, NR)(unsigned, unsigned, unsigned, void *, const void *, int *);
DVM_VARIANT_LIST(X)
#undef X
#define X(K, NR, MAXT, W) extern "C" int DVM_CRED_LAUNCHER_NAME(K, NR)(unsigned, unsigned, unsigned, void *, const void *, int *);
DVM_CRED_VARIANT_LIST(X)
#undef X

// The workspace of dvm_run_static: one array per device, in the library's own image, so that the entry point
// needs no allocation.  In host code the array's name is only a handle for hipGetSymbolAddress; the device
// address it yields (per device) is what kernels and fills get.
static __device__ __align__(256) unsigned char scratch[DVM_STATIC_WORKSPACE_BYTES];

namespace {

typedef int (*vm_launch_t)(unsigned, unsigned, unsigned, void *, const void *, int *);
struct VariantEntry { int K, NR; vm_launch_t launch; };
#define X(K, NR, MAXT, W) {K, NR, DVM_LAUNCHER_NAME(K, NR)},
const VariantEntry g_variants[] = {DVM_VARIANT_LIST(X)};
#undef X
#define X(K, NR, MAXT, W) {K, NR, DVM_WIDE_LAUNCHER_NAME(K, NR)},
const VariantEntry g_wide_variants[] = {DVM_VARIANT_LIST(X)};
#undef X
#define X(K, NR, MAXT, W) {K, NR, DVM_ANY_LAUNCHER_NAME(K, NR)},
const VariantEntry g_any_variants[] = {DVM_VARIANT_LIST(X)};
#undef X
#define X(K, NR, MAXT, W) {K, NR, DVM_LONG_WIDE_LAUNCHER_NAME(K, NR)},
const VariantEntry g_long_wide_variants[] = {DVM_VARIANT_LIST(X)};
#undef X
#define X(K, NR, MAXT, W) {K, NR, DVM_VISIT_LAUNCHER_NAME(K, NR)},
const VariantEntry g_visit_variants[] = {DVM_VARIANT_LIST(X)};
#undef X
#define X(K, NR, MAXT, W) {K, NR, DVM_VISIT_WIDE_LAUNCHER_NAME(K, NR)},
const VariantEntry g_visit_wide_variants[] = {DVM_VARIANT_LIST(X)};
#undef X
#define X(K, NR, MAXT, W) {K, NR, DVM_CRED_LAUNCHER_NAME(K, NR)},
const VariantEntry g_cred_variants[] = {DVM_CRED_VARIANT_LIST(X)};
#undef X

thread_local int t_last_hip_error = 0;

constexpr int MAX_DEVICES = 64;
std::atomic<void *> g_scratch_ptr[MAX_DEVICES];

// Look up this device's copy of `scratch` (once per device; the device must be current for the lookup).
int scratch_setup(int device) {
    if (device < 0 || device >= MAX_DEVICES) return dvm_set_error(DVM_E_ARGS, "device index out of range");
    if (g_scratch_ptr[device].load(std::memory_order_acquire)) return DVM_OK;
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e == hipSuccess && cur != device) e = hipSetDevice(device);
    void *ptr = nullptr;
    if (e == hipSuccess) e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch));
    if (cur >= 0 && cur != device) {
        const hipError_t e2 = hipSetDevice(cur);
        if (e == hipSuccess) e = e2;
    }
    if (e != hipSuccess || !ptr) {
        t_last_hip_error = (int)e;
        return dvm_set_error(DVM_E_HIP, e != hipSuccess ? hipGetErrorString(e) : "hipGetSymbolAddress returned no address");
    }
    g_scratch_ptr[device].store(ptr, std::memory_order_release);
    return DVM_OK;
}

// clears the first words of the synchronisation area of a launch's workspace (a kernel rather than a memset node, so that
// the clearing may be captured into a HIP graph with the launch it precedes)
__global__ void dvm_ws_clear(uint32_t *ws, uint32_t words) {
    if (threadIdx.x < words) ws[threadIdx.x] = 0;
}

// The address table of a batched launch, written by a kernel that carries the addresses in its arguments: a copy from the caller's
// array (ordinary host memory) is staged and waited for by the host (a 32-layer step of 100 tokens, two launches, 145 us with copies, 141 so; of
// 20 tokens, bound by the host, 65 and 62).  A table of many pieces is copied after all.
constexpr uint32_t TABLE_PIECE = 496, TABLE_PIECES = 4;     // (4 KiB of arguments)
struct TableArgs { uint64_t dst; uint32_t n, pad; uint64_t addr[TABLE_PIECE]; };
__global__ void __launch_bounds__(512) dvm_table_write(const TableArgs a) {
    if (threadIdx.x < a.n) ((GLOBAL_AS uint64_t *)a.dst)[threadIdx.x] = a.addr[threadIdx.x];
}
hipError_t write_table(void *table, void *const *tensors, size_t n, hipStream_t stream) {
    if (n > (size_t)TABLE_PIECE * TABLE_PIECES) return hipMemcpyAsync(table, tensors, n * 8, hipMemcpyHostToDevice, stream);
    TableArgs a;
    a.pad = 0;
    for (size_t at = 0; at < n; at += TABLE_PIECE) {
        a.n = (uint32_t)(n - at < TABLE_PIECE ? n - at : TABLE_PIECE);
        a.dst = (uint64_t)(uintptr_t)table + at * 8;
        memcpy(a.addr, tensors + at, (size_t)a.n * 8);
        hipLaunchKernelGGL(dvm_table_write, dim3(1), dim3(512), 0, stream, a);
    }
    return hipGetLastError();
}

}  // namespace

extern "C" int dvm_last_hip_error(void) { return t_last_hip_error; }

extern "C" int dvm_ctx_query_device(int hip_device, int *n_cu) {
    hipDeviceProp_t prop;
    hipError_t e = hipGetDeviceProperties(&prop, hip_device);
    if (e != hipSuccess) {
        t_last_hip_error = (int)e;
        return DVM_E_HIP;
    }
    *n_cu = prop.multiProcessorCount;
    return scratch_setup(hip_device);
}

namespace {

// Workgroups of `block` threads and `lds_bytes` that one compute unit holds at a time, per launcher; asked of the
// runtime once and remembered (a handful of combinations occur).
struct OccEntry { vm_launch_t launch; uint32_t block, lds_bytes; int per_cu; };
constexpr int OCC_SLOTS = 64;
OccEntry g_occ[OCC_SLOTS];
std::atomic<int> g_occ_n{0};
std::mutex g_occ_mu;

int resident_per_cu(vm_launch_t launch, uint32_t block, uint32_t lds_bytes, int *per_cu) {
    const int n = g_occ_n.load(std::memory_order_acquire);
    for (int i = 0; i < n; ++i)
        if (g_occ[i].launch == launch && g_occ[i].block == block && g_occ[i].lds_bytes == lds_bytes) { *per_cu = g_occ[i].per_cu; return 0; }
    int v = 0;
    const int e = launch(0, block, lds_bytes, nullptr, nullptr, &v);
    if (e != 0) return e;
    std::lock_guard<std::mutex> lock(g_occ_mu);
    const int m = g_occ_n.load(std::memory_order_relaxed);
    if (m < OCC_SLOTS) {
        g_occ[m] = OccEntry{launch, block, lds_bytes, v};
        g_occ_n.store(m + 1, std::memory_order_release);
    }
    *per_cu = v;
    return 0;
}

struct Batch { int n_sets; void *table; size_t table_bytes; };     // device memory for the sets' address table
int run_impl(const dvm_ctx *ctx, const void *bytecode, size_t len, void *const *tensors_in, int n_tensors, void *hip_stream, bool static_ws,
             const Batch *batch);

}  // namespace

extern "C" int dvm_run(const dvm_ctx *ctx, const void *bytecode, size_t len, void *const *tensors, int n_tensors,
                       void *hip_stream) {
    return run_impl(ctx, bytecode, len, tensors, n_tensors, hip_stream, false, nullptr);
}

extern "C" int dvm_run_static(const dvm_ctx *ctx, const void *bytecode, size_t len, void *const *tensors, int n_tensors,
                              void *hip_stream) {
    return run_impl(ctx, bytecode, len, tensors, n_tensors, hip_stream, true, nullptr);
}

extern "C" int dvm_run_batched(const dvm_ctx *ctx, const void *bytecode, size_t len, void *const *tensor_sets, int n_tensors, int n_sets,
                               void *table, size_t table_bytes, void *hip_stream) {
    if (n_sets < 1 || n_tensors < 1 || !table) return dvm_set_error(DVM_E_ARGS, "dvm_run_batched: at least one set of at least one tensor, and a table buffer");
    if (((uintptr_t)table & 7) || table_bytes < (size_t)n_sets * (size_t)n_tensors * 8)
        return dvm_set_error(DVM_E_ARGS, "dvm_run_batched: the table buffer holds n_sets * n_tensors addresses of 8 bytes, 8-byte aligned");
    const Batch b{n_sets, table, table_bytes};
    return run_impl(ctx, bytecode, len, tensor_sets, n_tensors, hip_stream, false, &b);
}

namespace {

// One set of tensors against the bytecode's tensor table: no null pointer, the alignment the bytecode was encoded
// for, equal pointers where it names two entries as the same buffer, and no overlap between a buffer one segment
// writes and a buffer of another segment unless the bytecode orders them.
// *aliased is set where an output shares memory with another tensor of its own segment.
int check_tensor_set(const uint32_t *w, const uint8_t *seg_of, void *const *tensors, uint32_t *aliased) {
    const uint32_t ntens = w[PH_NTENS];
    uint64_t addr_of[DVM_MAX_TENSORS], size_of[DVM_MAX_TENSORS];
    for (uint32_t i = 0; i < ntens; ++i) {
        const uint32_t *te = w + PH_WORDS_N + i * TT_WORDS;
        const uint32_t info = te[TT_INFO];
        const uint64_t align = 1ull << ((info >> 16) & 0xFF);
        const uint64_t addr = (uint64_t)(uintptr_t)tensors[i];
        if (addr == 0) return dvm_set_error(DVM_E_ARGS, "dvm_run: null tensor pointer");
        if (addr & (align - 1)) return dvm_set_error(DVM_E_ALIGN, "dvm_run: tensor pointer below the alignment the bytecode was encoded for");
        if ((info >> 24) != 0 && addr != (uint64_t)(uintptr_t)tensors[(info >> 24) - 1])
            return dvm_set_error(DVM_E_ARGS, "dvm_run: two entries the bytecode names as the same buffer got different pointers");
        addr_of[i] = addr;
        size_of[i] = (uint64_t)te[TT_BYTES_LO] | ((uint64_t)te[TT_BYTES_HI] << 32);
    }
    for (uint32_t i = 0; i < ntens; ++i) {
        if (!(w[PH_WORDS_N + i * TT_WORDS + TT_INFO] & TI_OUTPUT)) continue;
        for (uint32_t j = 0; j < ntens; ++j)
            if (i != j && seg_of[i] == seg_of[j] && addr_of[i] < addr_of[j] + size_of[j] && addr_of[j] < addr_of[i] + size_of[i]) *aliased = 1;
    }
    if (w[PH_NSEG] > 1) {
        for (uint32_t i = 0; i < ntens; ++i) {
            const uint32_t ii = w[PH_WORDS_N + i * TT_WORDS + TT_INFO];
            if (ii & TI_WORKSPACE) continue;
            uint32_t root_i = i;
            while (w[PH_WORDS_N + root_i * TT_WORDS + TT_INFO] >> 24) root_i = (w[PH_WORDS_N + root_i * TT_WORDS + TT_INFO] >> 24) - 1;
            for (uint32_t j = 0; j < i; ++j) {
                const uint32_t ij = w[PH_WORDS_N + j * TT_WORDS + TT_INFO];
                if (seg_of[i] == seg_of[j] || !((ii | ij) & TI_OUTPUT)) continue;
                if (addr_of[i] >= addr_of[j] + size_of[j] || addr_of[j] >= addr_of[i] + size_of[i]) continue;
                uint32_t root_j = j;
                while (w[PH_WORDS_N + root_j * TT_WORDS + TT_INFO] >> 24) root_j = (w[PH_WORDS_N + root_j * TT_WORDS + TT_INFO] >> 24) - 1;
                if (root_i != root_j)
                    return dvm_set_error(DVM_E_ARGS, "dvm_run: a buffer one stacked part writes overlaps a buffer of another part "
                                                     "and the bytecode does not order them (dvm_stack_dependent)");
            }
        }
    }
    return DVM_OK;
}

// A segment that is a plain reduction along the penultimate axis -- one streaming record, the combination of the waves, the
// store, over rows of one 16-byte piece at least -- as the arguments of the kernel for those.  Which rows are added to which
// partial result, and in which order those are combined, is the segment's (its waves and their partial results): the bits are
// the interpreter's for the same segment in a stack or a batched launch.  Only the lanes that share a row are chosen here: as many
// as leave two workgroups per compute unit (down to a 128-byte line) and a workgroup of 1024 threads at most, 256 where a lane has
// few rows ([256, 64, 1024] fp32 in 8 partials 17.6 us in workgroups of 512 threads, 11.8 in 256; over longer columns no difference).
// An output written over a row of the input stays with the interpreter where a row's last piece slides back into columns that another
// workgroup stores.
bool plain_colreduce(const dvm_ctx *ctx, const uint32_t *sh, const uint64_t *tensors, bool aliased, dvm_colreduce_args *a, uint32_t *grid, uint32_t *block) {
    if (!(sh[S_FLAGS] & SF_CSTREAM) || sh[S_PROLOG] != 0 || sh[S_NWG] != 0 || (sh[S_FLAGS] & (SF_SYNC_WG | SF_SYNC_GRID))) return false;
    const uint32_t *r = sh + SH_WORDS;
    if ((r[0] & 0xFF) != I_CSTREAM || sh[S_EPILOG] != LEN_VLOAD) return false;
    const uint32_t *cc = r + LEN_VLOAD, *st = cc + LEN_REC;
    if (sh[S_CODESIZE] < LEN_VLOAD + LEN_REC + LEN_LOAD || (cc[0] & 0xFF) != I_CCOMB || cc[1] == 0 || (cc[0] >> 16) != (r[0] >> 16)) return false;
    const uint32_t sop = st[0] & 0xFF;
    if (sop != I_STORE && sop != I_VSTORE) return false;
    if (sh[S_CODESIZE] != LEN_VLOAD + LEN_REC + ((st[0] >> 8) & 0xFF) || ((st[0] >> 16) & 0xFF) != ((r[0] >> 16) & 0xFF) || (st[0] >> 24) != 0) return false;
    const uint64_t D0 = (uint64_t)sh[S_D0LO] | ((uint64_t)sh[S_D0HI] << 32);
    auto i64 = [](const uint32_t *w) { return (int64_t)((uint64_t)w[0] | ((uint64_t)w[1] << 32)); };
    a->in_bf16 = (r[1] >> 8) & 0xFF;
    a->out_bf16 = (st[1] >> 8) & 0xFF;
    const uint32_t piece = a->in_bf16 ? 8u : 4u;
    if (D0 < piece || i64(st + 2) != 0) return false;
    a->in = (const void *)(uintptr_t)tensors[sh[S_TBASE] + (r[1] & 0xFF)];
    a->out = (void *)(uintptr_t)tensors[sh[S_TBASE] + (st[1] & 0xFF)];
    a->in_s1 = i64(r + 2); a->in_s2 = i64(r + 4); a->in_s3 = i64(r + 6);
    a->out_s2 = sop == I_VSTORE ? i64(st + 4) : 0;
    a->out_s3 = sop == I_VSTORE ? i64(st + 6) : 0;
    a->cols = D0;
    a->size = sh[S_INNER];
    a->d2 = sh[S_D2];
    a->op = r[0] >> 24;
    int n_cu = 256;
    dvm_ctx_planner_get(ctx, &n_cu, nullptr);
    const uint64_t outer = sh[S_NROWS] / sh[S_INNER];
    uint32_t lg = 6;
    auto tiles = [&](uint32_t l) { return (D0 + ((uint64_t)piece << l) - 1) / ((uint64_t)piece << l); };
    a->waves = sh[S_RP] & 0xFFFF;
    a->partials = (r[1] >> 24) > 1 ? r[1] >> 24 : 1u;
    const uint32_t parts = a->waves * a->partials;
    while (lg > 3 && (outer * tiles(lg) < 2ull * (uint64_t)n_cu || parts << lg > 1024u)) --lg;
    while (lg > 4 && a->size < 32u * parts && parts << lg > 256u) --lg;
    const uint64_t units = outer * tiles(lg);
    if (units == 0 || units >= (1ull << 31) || parts << lg > 1024u) return false;
    if (aliased && D0 % piece != 0 && ((D0 / piece) & ((1u << lg) - 1u)) == 0) return false;
    a->log2_lanes = lg;
    a->col_tiles = (uint32_t)tiles(lg);
    *grid = (uint32_t)units;
    *block = ((parts << lg) + 63u) / 64u * 64u;
    return true;
}

// Multiply-shift constants of magic_div (Granlund & Montgomery): n / d for every 32-bit n.
void magic_of(uint32_t d, uint32_t *m, uint32_t *sh) {
    uint32_t l = 0;
    while (l < 32 && (1ull << l) < d) ++l;
    *m = (uint32_t)(((1ull << 32) * ((1ull << l) - d)) / d + 1);
    *sh = (l < 1 ? l : 1u) | (l > 1 ? l - 1 : 0u) << 8;
}

// A segment that is a softmax along the row, of one tensor or of the sum of two, as the arguments of the kernel for those: load [, load,
// add], max, exp of the difference, reciprocal of the sum, store of the product.  It takes segments that read and write at least
// DVM_SOFTMAX_MIN_BYTES in a layout of its own (rows longer than a tile, which the interpreter reads twice: an eighth of that): below, a launch
// is bound by its own cost, and in a stack an extra one (2 us) would cost more than it gives.  Rows of less than a line and smaller segments
// go to the kernel with the interpreter's bits where they are the whole program (fp32 [400000, 9] 12.4 us in the interpreter and 18.0 in the
// layout here).  The rule looks at the segment alone, so that its bits are the same alone, in a stack and in a batched launch (apart from outputs that
// overlap an operand, see below; in a spatial stack, whose parts share one launch, it stays with the interpreter).
// Lanes on a row: those that leave the fewest idle, lanes * chunks being what a row costs, over up to 8 chunks of 16 bytes a lane (bf16: 6,
// for the registers).  More than 4 cost an eighth for the waves they displace (not in fp32 rows of one wave), a row of several waves a
// sixteenth for its barriers: bf16 [64000, 2000] 141 us in 256 lanes of 2 chunks, 99 in 128 of 3, 82 in 64 of 5; fp32 [31250, 4096] 169 in 128 of
// 8, 161 in 256 of 4.  512 at most: 1024 leave one or two workgroups to a compute unit and were slower than 512 of twice the chunks, and than the
// interpreter (fp32 [1000, 16384] 27.7 and 24.6 us, interpreter 27.0; [1100, 15000] from the cache 28.4, 21.3 and 25.7; bf16 [1500, 24500] 41.2 and 30.3).
// Longer rows go to the kernel that keeps one per workgroup.
bool plain_softmax(const uint32_t *sh, const uint32_t *table, void *const *tensors, int n_sets, uint32_t n_tensors, bool may_exact,
                   dvm_softmax_args *a) {
    if (sh[S_INNER] != 0 || sh[S_NWG] != 0 || (sh[S_FLAGS] & (SF_LDS | SF_CSTREAM)) || sh[S_NROWS] == 0) return false;
    const uint32_t *r = sh + SH_WORDS, *end = r + sh[S_CODESIZE];
    auto op_of = [&]() { return r < end ? r[0] & 0xFF : (uint32_t)I_COUNT; };
    auto ra = [&]() { return (r[0] >> 16) & 0xFF; };
    auto rb = [&]() { return r[0] >> 24; };
    auto next = [&]() { r += (r[0] >> 8) & 0xFF; };
    auto is_load = [&]() { return op_of() == I_LOAD || op_of() == I_VLOAD; };
    constexpr uint32_t ONE = 0x3F800000u;
    const uint32_t *la = nullptr, *lb = nullptr, *st;
    uint32_t reg = 0;
    for (int i = 0; i < 2 && is_load(); ++i, next()) {
        if (ra() == SRC_ACC && !la) la = r;
        else if (ra() != SRC_ACC && !lb) { lb = r; reg = ra(); }
        else return false;
    }
    if (!la) return false;
    if (lb) {
        if (op_of() != I_BIN || ra() != reg || rb() != B_ADD) return false;
        next();
    }
    if (op_of() != I_RED || (rb() & R_KIND) != R_MAX || r[1] != U_NONE || r[2] != ONE || r[3] != 0) return false;
    const uint32_t smax = ra();
    next();
    if (op_of() != I_BIN || ra() != SRC_S0 + smax || rb() != B_EXPSUB) return false;
    next();
    if (op_of() != I_RED || rb() != R_SUM || r[1] != U_RCP || r[2] != ONE || r[3] != 0) return false;
    const uint32_t ssum = ra();
    next();
    if ((op_of() != I_STORE && op_of() != I_VSTORE) || ra() != SRC_ACC || rb() != ssum + 1) return false;
    st = r;
    next();
    if (r != end) return false;
    const uint32_t dt = (la[1] >> 8) & 0xFF;
    if (((st[1] >> 8) & 0xFF) != dt || (lb && ((lb[1] >> 8) & 0xFF) != dt)) return false;
    const uint32_t es = dt ? 2 : 4, V = 16 / es, line = 128 / es;
    const uint64_t cols = (uint64_t)sh[S_D0LO] | ((uint64_t)sh[S_D0HI] << 32);
    const uint64_t rows = sh[S_NROWS];
    if (cols > (1u << 24)) return false;
    const int64_t bytes = (int64_t)(rows * cols * es * 2);
    a->exact = cols < line || bytes < (sh[S_FLAGS] & SF_LONGROW ? DVM_SOFTMAX_MIN_BYTES / 8 : DVM_SOFTMAX_MIN_BYTES);
    if (a->exact) {         // the interpreter's order: a choice of speed alone
        const uint32_t G = sh[S_GEOM] & 0xFFFF, nvec = sh[S_GEOM] >> 24;
        if (!may_exact || (sh[S_FLAGS] & SF_LONGROW) || sh[S_NCT] != 1 || ((sh[S_GEOM] >> 16) & 0xFF) != V || G > 64 || (G & (G - 1)) != 0 ||
            nvec > 8 || (cols < V && G != 1)) return false;
        a->lanes = G;
        a->slots = nvec;
        a->log2_lanes = 0;
        while ((1u << a->log2_lanes) < G) ++a->log2_lanes;
        a->ragged = cols != (uint64_t)G * nvec * V;
    }
    // the outer dims and the strides along them, in the order of the output's strides: rows that follow each other in memory do so in the grid
    uint32_t ext[3] = {(uint32_t)rows, 1, 1};
    if (sh[S_D1] != 0) {
        ext[0] = sh[S_D1];
        ext[1] = (uint32_t)(rows / sh[S_D1]);
        if (sh[S_D2] != 0) {
            ext[2] = ext[1] / sh[S_D2];
            ext[1] = sh[S_D2];
        }
    }
    auto stride = [&](const uint32_t *rec, int k) {
        const bool view = (rec[0] & 0xFF) == I_VLOAD || (rec[0] & 0xFF) == I_VSTORE;
        return k == 0 || view ? (int64_t)((uint64_t)rec[2 + 2 * k] | ((uint64_t)rec[3 + 2 * k] << 32)) : (int64_t)0;
    };
    int dim[3] = {0, 1, 2};
    auto weight = [&](int k) { return ext[k] == 1 ? INT64_MAX : (stride(st, k) < 0 ? -stride(st, k) : stride(st, k)); };
    for (int i = 1; i < 3; ++i)
        for (int j = i; j > 0 && weight(dim[j]) < weight(dim[j - 1]); --j) { const int t = dim[j]; dim[j] = dim[j - 1]; dim[j - 1] = t; }
    bool even = true;               // every row starts where the first does in its line
    for (int k = 0; k < 3; ++k) {
        a->a_s[k] = stride(la, dim[k]);
        a->b_s[k] = lb ? stride(lb, dim[k]) : 0;
        a->y_s[k] = stride(st, dim[k]);
        even &= ext[dim[k]] == 1 || a->y_s[k] % (int64_t)line == 0;
    }
    // (masked softmax fp32 [96, 1411, 1411] 293 -> 267 us by the filling up; [64, 1800, 1800] 344 us in rows as they come, 315 in
    // blocks, 283 filled up; the blocks pay beyond 24 MB of mask: [32, 2500, 2500] 280 and 282, [32, 3500, 3500] 560 and 651)
    // A second tensor that all indices of the second dim share (a mask under batch * heads) is read again from the cache of the die that
    // read it before, if the same rows go to the same die every time: workgroups are dealt to the eight dies in turn, so the rows
    // of an index are filled up to a multiple of eight workgroups.  A mask larger than the dies' caches hold is taken in blocks of rows, each for
    // all indices before the next block.
    a->limit = 0;
    uint64_t all = rows;
    uint32_t block = ext[dim[0]];
    if (!a->exact && lb && ext[dim[2]] == 1 && ext[dim[1]] > 1 && block > 256 && a->b_s[1] == 0 && a->b_s[0] != 0) {
        a->limit = block;
        block = (uint64_t)block * cols * es <= (24u << 20) ? (block + 31) / 32 * 32 : 256 * cols * es < (4u << 20) ? 256 : 64;
        all = (uint64_t)((a->limit + block - 1) / block) * block * ext[dim[1]];
        a->a_s[2] = a->a_s[0] * block;
        a->b_s[2] = a->b_s[0] * block;
        a->y_s[2] = a->y_s[0] * block;
    }
    a->d1 = block;
    a->d2 = ext[dim[1]];
    magic_of(a->d1, &a->m1, &a->sh1);
    magic_of(a->d2, &a->m2, &a->sh2);
    a->ia = sh[S_TBASE] + (la[1] & 0xFF);
    a->ib = lb ? sh[S_TBASE] + (lb[1] & 0xFF) : 0;
    a->iy = sh[S_TBASE] + (st[1] & 0xFF);
    // An output may be an input, element for element: a row is read before it is stored.  Any other overlap stays with the interpreter, and so
    // does a long bf16 row written over the second tensor, which that kernel reads once more beside its stores (the last chunk of a row slides back over
    // columns that another wave stores).
    bool over_b = false;
    uint32_t shift = 0;
    for (int k = 0; k < n_sets; ++k) {
        void *const *t = tensors + (size_t)k * n_tensors;
        auto span = [&](uint32_t i, uint64_t *lo, uint64_t *hi) {
            const uint32_t *te = table + i * TT_WORDS;
            *lo = (uint64_t)(uintptr_t)t[i];
            *hi = *lo + ((uint64_t)te[TT_BYTES_LO] | ((uint64_t)te[TT_BYTES_HI] << 32));
        };
        uint64_t ylo, yhi, lo, hi;
        span(a->iy, &ylo, &yhi);
        if (ylo % es != 0) return false;
        for (int i = 0; i < (lb ? 2 : 1); ++i) {
            span(i ? a->ib : a->ia, &lo, &hi);
            if (lo % es != 0) return false;
            if (lo >= yhi || ylo >= hi) continue;
            for (int d = 0; d < 3; ++d)
                if (lo != ylo || (ext[d] > 1 && stride(i ? lb : la, d) != stride(st, d))) return false;
            over_b |= i == 1;
        }
        const uint32_t at = (uint32_t)(ylo % 128) / es;
        if (at > shift) shift = at;
    }
    // Lanes and kernel follow from the strides alone, never from an address: the sums of a row depend on them, and a set of a batch keeps its bits
    // whatever the others' addresses are.  Rows of whole lines in an output that starts inside one take the slots that the shift needs where their
    // kernel has them, and stay where they are otherwise (the classes of columns, and with them the bits, are the same).
    auto need = [&](uint32_t lanes, uint32_t by) { return (uint32_t)((cols + by + (uint64_t)lanes * V - 1) / ((uint64_t)lanes * V)); };
    const uint32_t planned = even ? 0 : line - 1;
    if (!a->exact) a->lanes = 0;
    uint64_t best = a->exact ? 0 : UINT64_MAX;
    for (uint32_t lanes = 8; lanes <= 512; lanes *= 2) {
        const uint32_t n = need(lanes, planned);
        if (n > (dt ? 6u : 8u)) continue;
        const uint64_t cost = (uint64_t)lanes * n * (n > 4 && (dt || lanes != 64) ? 18 : 16) * (lanes > 64 ? 17 : 16);
        if (cost < best) {
            best = cost;
            a->lanes = lanes;
        }
    }
    a->in_long = a->lanes == 0;
    if (a->in_long != 0 && dt && over_b) return false;
    if (a->in_long != 0) a->lanes = need(512, planned) <= (dt ? 16u : 24u) ? 512 : 1024;
    a->shifted = 0;
    if (!a->exact) {
        const uint32_t most = a->in_long != 0 ? (a->lanes == 512 ? (dt ? 16u : 24u) : dt ? 20u : 33u) : dt ? 6u : 8u;
        a->slots = need(a->lanes, planned);
        if (a->slots > most) return false;
        if (!even) shift = planned;
        if (need(a->lanes, shift) <= most) {
            a->slots = need(a->lanes, shift);
            a->shifted = shift != 0;
        }
    }
    a->tail = (uint32_t)(cols / ((uint64_t)a->lanes * V));
    const uint64_t rp = a->lanes >= 256 ? 1 : 256 / a->lanes, tiles = (all + rp - 1) / rp;
    if (all >= (1ull << 32) || tiles * (uint64_t)n_sets >= (1ull << 31)) return false;
    a->rows = (uint32_t)all;
    a->cols = (uint32_t)cols;
    a->bf16 = dt;
    a->set_tiles = (uint32_t)tiles;
    magic_of(a->set_tiles, &a->set_m, &a->set_sh);
    a->tiles = (uint32_t)(tiles * (uint64_t)n_sets);
    a->a = tensors ? tensors[a->ia] : nullptr;
    a->b = lb ? (tensors ? tensors[a->ib] : sh) : nullptr;         // (where only the launches are counted: there is one)
    a->y = tensors ? tensors[a->iy] : nullptr;
    return true;
}

// A segment that is a rotation of pairs, y1 = x1 c - x2 s and y2 = x2 c + x1 s, over rows of a power of two of 16-byte chunks (64 at most), as
// the arguments of the kernel for those.  The records may come in many forms (registers, products that ride along, inputs loaded twice), so
// they are evaluated on symbols first; the kernel rounds where the form does, and its bits are the interpreter's.
bool plain_rotary(const uint32_t *sh, int nr, const uint32_t *table, void *const *tensors, int n_sets, uint32_t n_tensors, dvm_rotary_args *a) {
    if (sh[S_INNER] != 0 || sh[S_NWG] != 0 || (sh[S_FLAGS] & (SF_LDS | SF_CSTREAM | SF_LONGROW)) || sh[S_NTENS] != 6 || sh[S_NCT] != 1) return false;
    const uint64_t cols = (uint64_t)sh[S_D0LO] | ((uint64_t)sh[S_D0HI] << 32);
    if (cols > 512 || cols == 0) return false;
    struct Expr { uint8_t kind, a, b, c; };         // kind: 0 nothing, 1 tensor a, 2 a * b, 3 a - b, 4 a + b, 5 fma(a, b, c)
    Expr e[64] = {};
    uint32_t n_e = 1, reg[8] = {};                  // (value 0: nothing known); registers 0 .. 5 and, last, the accumulator
    constexpr uint32_t ACC = 7;
    const uint32_t *rec_of[6] = {};                 // a record that loads or stores each tensor
    uint32_t out_expr[2] = {}, out_tensor[2] = {}, n_out = 0;
    auto make = [&](uint8_t k, uint32_t x, uint32_t y, uint32_t z) { e[n_e] = Expr{k, (uint8_t)x, (uint8_t)y, (uint8_t)z}; return n_e++; };
    auto slot = [&](uint32_t r) { return r == SRC_ACC ? ACC : r; };
    for (const uint32_t *r = sh + SH_WORDS, *end = r + sh[S_CODESIZE]; r < end; r += (r[0] >> 8) & 0xFF) {
        const uint32_t op = r[0] & 0xFF, ra = (r[0] >> 16) & 0xFF, rb = r[0] >> 24;
        if (n_e + 2 > 64) return false;
        if (op == I_LOAD || op == I_VLOAD) {
            const uint32_t t = r[1] & 0xFF;
            if (t >= 6 || (ra != SRC_ACC && ra > 5)) return false;
            if (rec_of[t] && memcmp(rec_of[t] + 2, r + 2, ((r[0] >> 8) & 0xFF) * 4 - 8) != 0) return false;
            rec_of[t] = r;
            reg[slot(ra)] = make(1, t, 0, 0);
        } else if (op == I_STORE || op == I_VSTORE) {
            if (n_out == 2 || rb != 0 || (ra != SRC_ACC && ra > 5)) return false;
            rec_of[r[1] & 0xFF] = r;
            out_tensor[n_out] = r[1] & 0xFF;
            out_expr[n_out++] = reg[slot(ra)];
        } else if (op == I_MOVRA && ra < 6) {
            reg[ra] = reg[ACC];
        } else if (op == I_MOVAR && ra < 6) {
            reg[ACC] = reg[ra];
        } else if (op == I_BIN && ra < 6 && (rb == B_MUL || rb == B_SUB || rb == B_RSUB || rb == B_ADD)) {
            reg[ACC] = rb == B_RSUB ? make(3, reg[ra], reg[ACC], 0) : make(rb == B_MUL ? 2 : rb == B_SUB ? 3 : 4, reg[ACC], reg[ra], 0);
        } else if (op == I_MAC && ra < 6 && rb < 6) {
            if (r[1] == MAC_ADD) {
                reg[ACC] = make(5, reg[ra], reg[rb], reg[ACC]);
            } else {
                const uint32_t p = make(2, reg[ra], reg[rb], 0);
                reg[ACC] = r[1] == MAC_SUB ? make(3, reg[ACC], p, 0) : make(3, p, reg[ACC], 0);
            }
        } else if (op == I_FMA && ra < 6 && r[1] == 0 && rb < 6 && rb != FMA_NO_ADDEND) {
            reg[ACC] = nr <= 4 ? make(5, reg[ACC], reg[ra], reg[rb]) : make(4, make(2, reg[ACC], reg[ra], 0), reg[rb], 0);     // (as the variants take it)
        } else {
            return false;
        }
    }
    if (n_out != 2 || out_tensor[0] == out_tensor[1]) return false;
    for (int k = 0; k < 6; ++k)
        if (!rec_of[k]) return false;
    // the two products of a sum or difference, as pairs of tensors
    auto product = [&](uint32_t x, uint32_t *p) {
        if (e[x].kind != 2 || e[e[x].a].kind != 1 || e[e[x].b].kind != 1) return false;
        p[0] = e[e[x].a].a;
        p[1] = e[e[x].b].a;
        return true;
    };
    int one = e[out_expr[0]].kind == 3 ? 0 : 1;
    const Expr d = e[out_expr[one]], s = e[out_expr[1 - one]];
    uint32_t p[2], q[2], u[2], w[2];
    if (d.kind != 3 || !product(d.a, p) || !product(d.b, q)) return false;
    uint32_t fused = 0;
    if (s.kind == 4) {
        if (!product(s.a, u) || !product(s.b, w)) return false;
    } else if (s.kind == 5) {
        if (e[s.a].kind != 1 || e[s.b].kind != 1 || !product(s.c, w)) return false;
        u[0] = e[s.a].a;
        u[1] = e[s.b].a;
        fused = 1;
    } else {
        return false;
    }
    auto is = [](const uint32_t *x, uint32_t y, uint32_t z) { return (x[0] == y && x[1] == z) || (x[0] == z && x[1] == y); };
    bool found = false;
    uint32_t x1 = 0, x2 = 0, c = 0, sn = 0;
    for (int k = 0; k < 4 && !found; ++k) {
        x1 = p[k & 1]; c = p[1 - (k & 1)]; x2 = q[k >> 1]; sn = q[1 - (k >> 1)];
        if (is(u, x2, c) && is(w, x1, sn)) found = true;
        else if (is(u, x1, sn) && is(w, x2, c)) { found = true; fused *= 2; }
    }
    if (!found || x1 == x2 || c == sn || x1 == sn || x2 == c) return false;
    const uint32_t t[6] = {x1, x2, c, sn, out_tensor[one], out_tensor[1 - one]};
    auto dtype = [&](int k) { return (rec_of[t[k]][1] >> 8) & 0xFF; };
    a->x_bf16 = dtype(0);
    a->t_bf16 = dtype(2);
    if (dtype(1) != a->x_bf16 || dtype(4) != a->x_bf16 || dtype(5) != a->x_bf16 || dtype(3) != a->t_bf16 || (a->t_bf16 && !a->x_bf16)) return false;
    const uint32_t V = a->x_bf16 ? 8 : 4, es = a->x_bf16 ? 2 : 4;
    if (cols % V != 0 || (cols / V & (cols / V - 1)) != 0 || cols / V > 64) return false;
    a->log2_lanes = 0;
    while ((V << a->log2_lanes) < cols) ++a->log2_lanes;
    const uint64_t rows = sh[S_NROWS];
    uint32_t ext[3] = {(uint32_t)rows, 1, 1};
    if (sh[S_D1] != 0) {
        ext[0] = sh[S_D1];
        ext[1] = (uint32_t)(rows / sh[S_D1]);
        if (sh[S_D2] != 0) {
            ext[2] = ext[1] / sh[S_D2];
            ext[1] = sh[S_D2];
        }
    }
    if (rows == 0) return false;
    for (int k = 0; k < 6; ++k) {
        const uint32_t *r = rec_of[t[k]];
        const bool view = (r[0] & 0xFF) == I_VLOAD || (r[0] & 0xFF) == I_VSTORE;
        for (int i = 0; i < 3; ++i) a->s[k][i] = i == 0 || view ? (int64_t)((uint64_t)r[2 + 2 * i] | ((uint64_t)r[3 + 2 * i] << 32)) : 0;
        a->at[k] = sh[S_TBASE] + t[k];
        a->p[k] = (uint64_t)(uintptr_t)tensors[a->at[k]];
    }
    // Outputs apart from the inputs, and from each other (two halves of the same rows are)
    for (int k = 0; k < n_sets; ++k) {
        uint64_t lo[6], hi[6];
        for (int i = 0; i < 6; ++i) {
            const uint32_t *te = table + a->at[i] * TT_WORDS;
            lo[i] = (uint64_t)(uintptr_t)tensors[(size_t)k * n_tensors + a->at[i]];
            hi[i] = lo[i] + ((uint64_t)te[TT_BYTES_LO] | ((uint64_t)te[TT_BYTES_HI] << 32));
            if (lo[i] % (dtype(i) ? 2 : 4) != 0) return false;
        }
        for (int o = 4; o < 6; ++o)
            for (int i = 0; i < 4; ++i)
                if (lo[i] < hi[o] && lo[o] < hi[i]) return false;
        if (lo[4] < hi[5] && lo[5] < hi[4]) {
            const uint64_t apart = lo[4] < lo[5] ? lo[5] - lo[4] : lo[4] - lo[5];
            if (apart < cols * es) return false;
            for (int i = 0; i < 3; ++i)
                if (a->s[4][i] != a->s[5][i] || (ext[i] > 1 && (a->s[4][i] < 0 || (uint64_t)a->s[4][i] * es < apart + cols * es))) return false;
        }
    }
    a->d1 = ext[0];
    a->d2 = ext[1];
    magic_of(a->d1, &a->m1, &a->sh1);
    magic_of(a->d2, &a->m2, &a->sh2);
    const uint32_t rw = 64u >> a->log2_lanes;
    a->rows_per_lane = ext[0] % (4 * rw) == 0 && a->s[2][0] == 0 && a->s[3][0] == 0 ? 4 : 1;
    const uint64_t per = (uint64_t)rw * a->rows_per_lane, groups = (rows + per - 1) / per;
    if (groups * (uint64_t)n_sets >= (1ull << 26)) return false;       // (a wave each, and a launch has fewer than 2^32 threads)
    a->rows = (uint32_t)rows;
    a->set_groups = (uint32_t)groups;
    magic_of(a->set_groups, &a->set_m, &a->set_sh);
    a->groups = (uint32_t)(groups * (uint64_t)n_sets);
    a->fused = fused;
    a->n_tensors = n_tensors;
    return true;
}

// Loads take the streaming hint in launches that read more than this.  Less may still be in the last-level cache (256 MB) from the program that
// wrote it or the one that read it last, beside what others use; the hint then costs (RMSNorm bf16 [11000, 4096], 90 MB read, 30.8 us
// without and 36.5 with it, RoPE over 8111 tokens, 66 MB, 31.6 and 38.1), and pays beyond (fp32 add, 128 MB, 34.0 and 31.5, the 12-op chain over
// 2245 rows of 8192, 110 MB, 40.1 and 36.7), where the inputs are in memory: RMSNorm reading 128 MB 51.8 and 48.6 us, from the cache 42.4 and 47.1.
constexpr uint64_t STREAM_MIN_READS = 96ull << 20;
// A bf16 program that reads several tensors so gains earlier: us without and with the hint, inputs in memory (in the cache), the chain (three tensors)
// reading 16 MB 15.4 14.6 (11.6 13.0), 24 MB 18.8 16.1 (12.7 14.3), 48 MB 24.2 20.4 (20.1 19.4), add (two) 16 MB 8.8 8.4 (6.0 7.4), 32 MB 13.1 12.0 (9.2 9.9),
// 64 MB 21.4 19.6 (18.5 17.6); but RMSNorm (one) 48 MB
// 22.2 20.8 (18.5 19.1), 80 MB 33.9 31.7 (27.7 30.0).  In fp32 what the hint drops from a cache that is nearly full costs more than it gives: an addition
// beside a softmax of its size, 34 MB read by each, 19.8 and 24.4, alone 64 MB 21.4 19.7 (17.9 17.7).
constexpr uint64_t STREAM_MIN_READS_OF_SEVERAL = 32ull << 20;
constexpr uint64_t LARGE_MIN_BYTES = 256ull << 20;      // launches larger than the last-level cache
constexpr uint64_t FLAT_MIN_BYTES = 64ull << 20;        // the same for rows cut into column tiles

// Bytes of a launch of some segments, over one set of tensors
struct LaunchBytes {
    uint64_t spans = 0, touched = 0, reads = 0;     // the last two: without what lies between the rows of views
    uint32_t streams = 0;                           // of a segment alone, all of bf16: tensors that it reads past the caches if it may
    bool stream(int n_sets) const {
        return reads * (uint64_t)n_sets >= (streams > 1 ? STREAM_MIN_READS_OF_SEVERAL : STREAM_MIN_READS);
    }
};
LaunchBytes launch_bytes(const uint32_t *w, const uint32_t *seg_at, const uint32_t *segs, uint32_t n_segs) {
    LaunchBytes b;
    for (uint32_t i = 0; i < n_segs; ++i) {
        const uint32_t *sh = w + seg_at[segs[i]];
        for (uint32_t t = 0; t < sh[S_NTENS]; ++t) {
            const uint32_t *te = w + PH_WORDS_N + (sh[S_TBASE] + t) * TT_WORDS;
            const uint64_t span = (uint64_t)te[TT_BYTES_LO] | ((uint64_t)te[TT_BYTES_HI] << 32);
            const uint64_t whole = (uint64_t)sh[S_NROWS] * ((uint64_t)sh[S_D0LO] | ((uint64_t)sh[S_D0HI] << 32)) * ((te[TT_INFO] & 0xFF) == DVM_BF16 ? 2u : 4u);
            b.spans += span;
            b.touched += whole < span ? whole : span;
            if (!(te[TT_INFO] & TI_OUTPUT)) b.reads += whole < span ? whole : span;
        }
        bool bf16 = n_segs == 1;
        for (uint32_t pc = SH_WORDS; pc < sh[S_WORDS]; pc += (sh[pc] >> 8) & 0xFF) {
            if (((sh[pc] & 0xFF) != I_LOAD && (sh[pc] & 0xFF) != I_VLOAD) || !((sh[pc + 1] >> 16) & MF_STREAM)) continue;
            bf16 &= ((sh[pc + 1] >> 8) & 0xFF) == DVM_BF16;
            ++b.streams;
        }
        if (!bf16) b.streams = 0;
    }
    return b;
}

// A softmax that runs apart (plain_softmax): the segment at word `at`.  A smaller one, whose bits are the interpreter's, only where it is the whole
// program: in a batched stack its arithmetic hides behind the traffic of the other parts (a 32-layer step of 200 tokens 213 us, 219 with it apart).
bool runs_apart(const uint32_t *w, uint32_t at, void *const *tensors, int n_sets, dvm_softmax_args *sm) {
    return plain_softmax(w + at, w + PH_WORDS_N, tensors, n_sets, w[PH_NTENS], w[PH_NSEG] == 1, sm);
}
// Threads of a workgroup, and workgroups of its launch.  The kernel for long rows loads a workgroup's next row while it stores the one before: as many
// as are resident.  The others take a tile each, as far as a launch may have that many threads (below 2^32), and the rest in turn.
uint32_t softmax_block(const dvm_softmax_args &sm) { return sm.exact || sm.lanes < 256 ? 256 : sm.lanes; }
uint32_t softmax_grid(const dvm_softmax_args &sm, uint32_t tiles, int n_cu) {
    const uint32_t most = sm.in_long != 0 ? (uint32_t)n_cu * (sm.lanes == 1024 ? 1u : 2u) : UINT32_MAX / softmax_block(sm);
    return tiles > most ? most : tiles;
}

// The kernel launches: segments in a run share one.  A segment starts a run of its own where it asks for one, and a softmax that runs apart is
// one.  Segments that are independent of each other go first, all but those, in one launch.  Of independent softmaxes those alike in all but their addresses
// share a launch of the kernel that each has alone, wherever they stand, as long as such a group fills the chip or there is no other to join; those of
// smaller groups share one of the kernel for several shapes, since few rows leave most of the chip idle and launches follow each other (eight of fp32
// [16, 100003], of two widths in turn: 25 us, each in its own launch 156, in the interpreter 48; bf16 [32, 17000] 6.6, 43 and 18; [6000, 751], where both
// groups fill the chip, 29, 51 and 43).  A softmax that is alone among other programs pays its launch, 1 to 2 us: with an addition of its size, launch and
// interpreter, bf16 [6000, 751] 13.9 and 12.3, fp32 [2100, 2049] 19.8 and 17.7, but bf16 [50000, 128] 14.5 and 27.6, fp32 [16, 100003] 28 and 49.
enum : uint8_t { RUN_VM = 0, RUN_SOFTMAX, RUN_MIXED };
struct Runs {
    uint32_t n = 0, n_list = 0;
    uint32_t list[MAX_SEGMENTS], at[MAX_SEGMENTS + 1];      // segments, run after run, and where the runs start
    uint8_t kind[MAX_SEGMENTS];
    void push(uint32_t s, bool fresh, uint8_t k) {
        if (fresh || n == 0) { kind[n] = k; at[n++] = n_list; }
        list[n_list++] = s;
    }
};
void plan_runs(const uint32_t *w, void *const *tensors, int n_sets, bool ordered, Runs *runs) {
    uint32_t seg_at[MAX_SEGMENTS];
    uint8_t which[MAX_SEGMENTS];            // 1 + a softmax that runs apart, 0: any other segment
    static_assert(DVM_SOFTMAX_MAX_PARTS >= DVM_MAX_TENSORS / 2, "softmaxes of a launch");
    dvm_softmax_args soft[DVM_MAX_TENSORS / 2];
    uint32_t seg_of[DVM_MAX_TENSORS / 2], n_soft = 0;
    for (uint32_t s = 0, at = PH_WORDS_N + w[PH_NTENS] * TT_WORDS; s < w[PH_NSEG]; at += w[at + S_WORDS], ++s) {
        seg_at[s] = at;
        which[s] = 0;
        if (n_soft == DVM_MAX_TENSORS / 2) continue;
        dvm_softmax_args &sm = soft[n_soft];
        memset(&sm, 0, sizeof sm);
        if (!runs_apart(w, at, tensors, n_sets, &sm)) continue;
        seg_of[n_soft] = s;
        which[s] = (uint8_t)++n_soft;
    }
    if (ordered || n_soft < 2) {
        if (!ordered) for (uint32_t s = 0; s < w[PH_NSEG]; ++s) if (!which[s]) runs->push(s, false, RUN_VM);
        for (uint32_t s = 0; s < w[PH_NSEG]; ++s)
            if (ordered || which[s])
                runs->push(s, which[s] || (s > 0 && which[s - 1]) || (w[seg_at[s] + S_FLAGS] & SF_NEW_LAUNCH), which[s] ? RUN_SOFTMAX : RUN_VM);
        runs->at[runs->n] = runs->n_list;
        return;
    }
    for (uint32_t s = 0; s < w[PH_NSEG]; ++s) if (!which[s]) runs->push(s, false, RUN_VM);
    // groups of alike ones (alike[i]: the first that i is like), and the kernels they could share with others
    uint32_t alike[DVM_MAX_TENSORS / 2], size[DVM_MAX_TENSORS / 2], kernel[DVM_MAX_TENSORS / 2];
    for (uint32_t i = 0; i < n_soft; ++i) {
        dvm_softmax_args &sm = soft[i];
        kernel[i] = sm.bf16 | (sm.b ? 2u : 0u) | sm.in_long << 2 | (sm.lanes > 256 ? sm.lanes << 3 : 0u);
        sm.a = sm.y = nullptr;
        if (sm.b) sm.b = w;         // (there is one)
        sm.ia = sm.ib = sm.iy = 0;
        alike[i] = i;
        size[i] = 1;
        for (uint32_t j = 0; j < i && n_sets <= 1; ++j)
            if (alike[j] == j && memcmp(&sm, &soft[j], sizeof sm) == 0 && (uint64_t)sm.tiles * (size[j] + 1) < (1ull << 31)) {
                alike[i] = j;
                ++size[j];
                break;
            }
    }
    auto fills = [&](uint32_t i) { return (uint64_t)soft[i].tiles * size[i] >= (soft[i].lanes <= 256 ? 2048u : 1024u * 512u / soft[i].lanes); };
    bool done[DVM_MAX_TENSORS / 2] = {};
    for (uint32_t i = 0; i < n_soft; ++i) {
        if (done[i]) continue;
        // (i stands first in its group: the others of it are done with it)
        auto joins = [&](uint32_t j) { return !done[j] && !fills(alike[j]) && kernel[j] == kernel[i]; };
        bool mixed = false;
        for (uint32_t j = i + 1; j < n_soft && !fills(i); ++j) mixed |= joins(j) && alike[j] != i;
        uint32_t n = 0;
        for (uint32_t j = i; j < n_soft; ++j) {
            if (done[j] || !(mixed ? joins(j) : alike[j] == i)) continue;
            runs->push(seg_of[j], n++ == 0, mixed ? RUN_MIXED : RUN_SOFTMAX);
            done[j] = true;
        }
    }
    runs->at[runs->n] = runs->n_list;
}
// The arguments of a run's launch; its tiles
uint32_t softmax_args(const uint32_t *w, const uint32_t *seg_at, const uint32_t *segs, uint32_t n, void *const *tensors, int n_sets, uint64_t sets, dvm_softmax_alike *a) {
    dvm_softmax_args &sm = a->s;
    if (n > 1) {
        for (uint32_t i = 0; i < n; ++i) {
            runs_apart(w, seg_at[segs[i]], tensors, n_sets, &sm);
            a->parts[3 * i] = (uint64_t)(uintptr_t)sm.a;
            a->parts[3 * i + 1] = (uint64_t)(uintptr_t)sm.b;
            a->parts[3 * i + 2] = (uint64_t)(uintptr_t)sm.y;
        }
        sm.sets = DVM_SOFTMAX_PARTS;
        sm.n_tensors = 3;
        sm.ia = 0, sm.ib = 1, sm.iy = 2;
        sm.tiles *= n;
    } else {
        runs_apart(w, seg_at[segs[0]], tensors, n_sets, &sm);
        sm.sets = sets;
        sm.n_tensors = w[PH_NTENS];
    }
    sm.stream = (uint64_t)sm.rows * sm.cols * (sm.bf16 ? 2u : 4u) * (uint64_t)n_sets * n >= STREAM_MIN_READS;
    return sm.tiles;
}
uint32_t softmax_args(const uint32_t *w, const uint32_t *seg_at, const uint32_t *segs, uint32_t n, void *const *tensors, int n_sets, uint64_t sets, dvm_softmax_mixed *p) {
    uint64_t bytes = 0;
    p->n = n;
    p->first[0] = 0;
    for (uint32_t i = 0; i < n; ++i) {
        dvm_softmax_args &sm = p->part[i];
        runs_apart(w, seg_at[segs[i]], tensors, n_sets, &sm);
        sm.sets = sets;
        sm.n_tensors = w[PH_NTENS];
        p->first[i + 1] = p->first[i] + sm.tiles;
        bytes += (uint64_t)sm.rows * sm.cols * (sm.bf16 ? 2u : 4u) * (uint64_t)n_sets;
    }
    for (uint32_t i = 0; i < n; ++i) p->part[i].stream = bytes >= STREAM_MIN_READS;
    return p->first[n];
}

// Segments that may depend on each other
bool is_ordered(const uint32_t *w) {
    bool r = (w[PH_TYPE] & 0xFFFF) == KT_STACK_SPATIAL;
    for (uint32_t i = 0; i < w[PH_NTENS]; ++i) r |= (w[PH_WORDS_N + i * TT_WORDS + TT_INFO] & TI_WORKSPACE) != 0 || (w[PH_WORDS_N + i * TT_WORDS + TT_INFO] >> 24) != 0;
    for (uint32_t s = 0, at = PH_WORDS_N + w[PH_NTENS] * TT_WORDS; s < w[PH_NSEG]; at += w[at + S_WORDS], ++s)
        r |= (w[at + S_FLAGS] & (SF_SYNC_WG | SF_SYNC_GRID | SF_NEW_LAUNCH)) != 0;
    return r;
}

int run_impl(const dvm_ctx *ctx, const void *bytecode, size_t len, void *const *tensors_in, int n_tensors, void *hip_stream, bool static_ws,
             const Batch *batch) {
    if (!ctx || !bytecode || (!tensors_in && n_tensors > 0)) return dvm_set_error(DVM_E_ARGS, "dvm_run: null argument");
    if (dvm_ctx_device(ctx) < 0) return dvm_set_error(DVM_E_ARGS, "dvm_run: context was created without a device");
    int st = dvm_validate(bytecode, len);
    if (st != DVM_OK) return st;
    const uint32_t *w = (const uint32_t *)bytecode;
    const uint32_t ntens = w[PH_NTENS];
    // dvm_run_static: the library's own array stands in for the workspace entry, which the caller leaves out
    void *tensors_full[DVM_MAX_TENSORS];
    void *const *tensors = tensors_in;
    if (static_ws && ntens > 0 && (w[PH_WORDS_N + (ntens - 1) * TT_WORDS + TT_INFO] & TI_WORKSPACE)) {
        if ((uint32_t)n_tensors + 1 != ntens) return dvm_set_error(DVM_E_ARGS, "dvm_run_static: pass the bytecode's tensors without its workspace");
        const uint32_t *te = w + PH_WORDS_N + (ntens - 1) * TT_WORDS;
        if (te[TT_BYTES_HI] != 0 || te[TT_BYTES_LO] > DVM_STATIC_WORKSPACE_BYTES)
            return dvm_set_error(DVM_E_LIMIT, "dvm_run_static: the launch needs a workspace beyond DVM_STATIC_WORKSPACE_BYTES; use dvm_run with a workspace of the caller's");
        st = scratch_setup(dvm_ctx_device(ctx));
        if (st != DVM_OK) return st;
        for (int i = 0; i < n_tensors; ++i) tensors_full[i] = tensors_in[i];
        tensors_full[n_tensors] = g_scratch_ptr[dvm_ctx_device(ctx)].load(std::memory_order_acquire);
        tensors = tensors_full;
        ++n_tensors;
    }
    if ((uint32_t)n_tensors != ntens) return dvm_set_error(DVM_E_ARGS, "dvm_run: tensor count does not match the bytecode");
    const uint32_t segs_off = PH_WORDS_N + ntens * TT_WORDS;
    const uint32_t seg_words = w[PH_WORDS] - segs_off;
    if (seg_words > (uint32_t)CODE_WORDS) return dvm_set_error(DVM_E_LIMIT, "dvm_run: bytecode exceeds the kernel-argument budget");

    if (w[PH_GRID] == 0) return DVM_OK;   // an empty iteration space: nothing to launch, pointers may be null

    KArgs ka;
    ka.ws = 0;
    for (uint32_t i = 0; i < ntens; ++i) {
        ka.tensors[i] = (uint64_t)(uintptr_t)tensors[i];
        if (w[PH_WORDS_N + i * TT_WORDS + TT_INFO] & TI_WORKSPACE) {
            ka.ws = ka.tensors[i];                      // the synchronisation area
            ka.tensors[i] += DVM_WORKSPACE_BYTES;       // segments that name the workspace as a tensor see its data area
        }
    }
    ka.sets = 0;
    ka.n_sets = 1;
    ka.n_tensors = ntens;
    ka.rotate = 0;
    ka.set_tiles = 0;
    ka.set_m = ka.set_sh = 0;
    ka.aliased = 0;
    ka.nseg = w[PH_NSEG];
    ka.spin_limit = (uint32_t)dvm_ctx_sync_limit(ctx);

    const int K = (int)(w[PH_VARIANT] & 0xFF), NR = (int)((w[PH_VARIANT] >> 8) & 0xFF);
    const uint32_t block = w[PH_BLOCK];
    // What decides which instantiation a launch of some of the segments takes
    struct Needs {
        uint32_t lds_bytes = 0;         // the combination across waves of a reduction along the penultimate axis: four floats per lane of
                                        // every participating wave; the images that prologues copy into LDS
        bool longrow = false, mac = false, part = false;
    };
    bool wide = true;                   // every segment of the program spreads a row over whole waves
    bool cred = false;                  // a segment that reduces along the penultimate axis needs the instantiation that runs such segments
    bool grid_sync = false, wg_sync = false, longrow = false;
    uint32_t seg_at[MAX_SEGMENTS];      // where the segments start
    uint8_t seg_of[DVM_MAX_TENSORS];    // the segment a tensor belongs to
    memset(seg_of, 0xFF, sizeof(seg_of));
    if (w[PH_NSEG] > (uint32_t)MAX_SEGMENTS) return dvm_set_error(DVM_E_LIMIT, "dvm_run: bytecode exceeds the kernel-argument budget");
    for (uint32_t s = 0, at = segs_off; s < w[PH_NSEG]; ++s) {
        const uint32_t *sh = w + at;
        seg_at[s] = at;
        wide &= (sh[S_GEOM] & 0xFFFF) >= 64;
        cred |= sh[S_INNER] != 0;
        grid_sync |= (sh[S_FLAGS] & SF_SYNC_GRID) != 0;
        wg_sync |= (sh[S_FLAGS] & SF_SYNC_WG) != 0;
        longrow |= (sh[S_FLAGS] & SF_LONGROW) != 0;
        for (uint32_t t = 0; t < sh[S_NTENS]; ++t) seg_of[sh[S_TBASE] + t] = (uint8_t)s;
        at += sh[S_WORDS];
    }
    // Segments of one launch run without order between them unless the bytecode says otherwise: see check_tensor_set
    const int n_sets = batch ? batch->n_sets : 1;
    for (int k = 0; k < n_sets; ++k) {
        st = check_tensor_set(w, seg_of, tensors + (size_t)k * ntens, &ka.aliased);
        if (st != DVM_OK) return st;
    }
    if (batch) {
        if (grid_sync || ka.ws != 0) return dvm_set_error(DVM_E_UNSUPPORTED, "dvm_run_batched: bytecode with a workspace runs one set at a time");
        // the sets' addresses travel through the caller's table buffer (written on the launch's stream)
        const hipError_t ce = write_table(batch->table, tensors, (size_t)n_sets * ntens, (hipStream_t)hip_stream);
        if (ce != hipSuccess) {
            t_last_hip_error = (int)ce;
            return dvm_set_error(DVM_E_HIP, hipGetErrorString(ce));
        }
        ka.sets = (uint64_t)(uintptr_t)batch->table;
        ka.n_sets = (uint32_t)n_sets;
    }
    auto add_needs = [&](const uint32_t *sh, Needs *n) {
        const uint32_t rp = sh[S_RP] & 0xFFFF, G = sh[S_GEOM] & 0xFFFF, V = (sh[S_GEOM] >> 16) & 0xFF;
        n->longrow |= (sh[S_FLAGS] & SF_LONGROW) != 0;
        if (sh[S_FLAGS] & SF_LONGROW)
            for (uint32_t pc = SH_WORDS; pc < sh[S_WORDS]; pc += (sh[pc] >> 8) & 0xFF) n->mac |= (sh[pc] & 0xFF) == I_MAC;
        if (sh[S_INNER] != 0 && rp > 1 && rp * 64u * 16u > n->lds_bytes) n->lds_bytes = rp * 64u * 16u;
        if (sh[S_FLAGS] & SF_LDS)
            for (uint32_t pc = SH_WORDS; pc < SH_WORDS + sh[S_PROLOGA]; pc += (sh[pc] >> 8) & 0xFF)
                if ((sh[pc] & 0xFF) == I_LDSCOPY && sh[pc + 2] + sh[pc + 3] > n->lds_bytes) n->lds_bytes = sh[pc + 2] + sh[pc + 3];
        // A last chunk that is handled element by element (see tile_cols) needs the instantiation that runs any launch.
        if (sh[S_NTILES] == 0) return;
        const uint64_t D0 = (uint64_t)sh[S_D0LO] | ((uint64_t)sh[S_D0HI] << 32), ncols = D0 - (uint64_t)(sh[S_NCT] - 1) * sh[S_TC], full = ncols / V;
        n->part |= ncols % V != 0 && (full == 0 || (G > 64 && ka.aliased != 0 && (full % G) % 64 == 0));
    };
    if (cred && longrow)
        return dvm_set_error(DVM_E_UNSUPPORTED, "dvm_run: a launch holds both a reduction along the penultimate axis and rows longer than a tile");
    // Segments planned for 32 elements per lane or fewer that have a launch to themselves in a program of the 64-element variant
    // (dvm_stack sets large ones apart) run in the one of 32: more resident waves, and no idle half of every tile register.
    bool apart = false;
    for (uint32_t s = 0, at = segs_off, k_max = 64; s < w[PH_NSEG]; at += w[at + S_WORDS], ++s) {
        const uint32_t k = (w[at + S_GEOM] >> 24) * ((w[at + S_GEOM] >> 16) & 0xFF);
        k_max = w[at + S_FLAGS] & SF_NEW_LAUNCH ? k : (k > k_max ? k : k_max);
        const bool last = s + 1 == w[PH_NSEG] || (w[at + w[at + S_WORDS] + S_FLAGS] & SF_NEW_LAUNCH);
        apart |= last && k_max <= 32 && K == 64 && NR <= 2 && block <= 256 && !cred;
    }
    const bool rotates = (w[PH_NSEG] > 1 || n_sets > 1) && !wg_sync && (w[PH_TYPE] & 0xFFFF) != KT_STACK_SPATIAL;
    if (grid_sync) hipLaunchKernelGGL(dvm_ws_clear, dim3(1), dim3(64), 0, (hipStream_t)hip_stream, (uint32_t *)(uintptr_t)ka.ws, (uint32_t)WS_SYNC_WORDS);
    hipError_t e;
    dvm_rotary_args ra;
    if (w[PH_NSEG] == 1 && plain_rotary(w + segs_off, NR, w + PH_WORDS_N, tensors, n_sets, ntens, &ra)) {
        ra.sets = ka.sets;
        ra.stream = (uint64_t)ra.rows * (uint64_t)(((uint64_t)w[segs_off + S_D0LO]) * (ra.x_bf16 ? 4u : 8u)) * (uint64_t)n_sets >= STREAM_MIN_READS;
        e = (hipError_t)dvm_rotary_launch(&ra, hip_stream);
        if (e != hipSuccess) {
            t_last_hip_error = (int)e;
            return dvm_set_error(DVM_E_HIP, hipGetErrorString(e));
        }
        return DVM_OK;
    }
    Runs runs;
    plan_runs(w, tensors, n_sets, is_ordered(w), &runs);
    uint32_t vm_runs = 0;
    for (uint32_t run = 0; run < runs.n; ++run) {
        const uint32_t *segs = runs.list + runs.at[run];
        const uint32_t n_segs = runs.at[run + 1] - runs.at[run];
        if (runs.kind[run] != RUN_VM) {     // (the launch boundaries are what orders it behind the parts it depends on, and those behind it)
            int n_cu = 256;
            dvm_ctx_planner_get(ctx, &n_cu, nullptr);
            if (runs.kind[run] == RUN_MIXED) {
                dvm_softmax_mixed sm;
                const uint32_t tiles = softmax_args(w, seg_at, segs, n_segs, tensors, n_sets, ka.sets, &sm);
                e = (hipError_t)dvm_softmax_launch_mixed(&sm, softmax_grid(sm.part[0], tiles, n_cu), hip_stream);
            } else {
                dvm_softmax_alike sm;
                const uint32_t tiles = softmax_args(w, seg_at, segs, n_segs, tensors, n_sets, ka.sets, &sm);
                e = (hipError_t)dvm_softmax_launch(&sm, softmax_grid(sm.s, tiles, n_cu), hip_stream);
            }
            if (e != hipSuccess) {
                t_last_hip_error = (int)e;
                return dvm_set_error(DVM_E_HIP, hipGetErrorString(e));
            }
            continue;
        }
        ka.nseg = n_segs;
        ka.set_tiles = 0;
        Needs need;
        uint64_t total = 0;                 // tiles of this launch
        uint32_t k_need = 0;                // elements per lane its segments use
        bool round_robin = true;
        for (uint32_t i = 0; i < n_segs; ++i) {
            const uint32_t *sh = w + seg_at[segs[i]];
            add_needs(sh, &need);
            total += sh[S_NTILES];
            round_robin &= (sh[S_FLAGS] & SF_INTERLEAVED) != 0;
            const uint32_t k = (sh[S_GEOM] >> 24) * ((sh[S_GEOM] >> 16) & 0xFF);
            if (k > k_need) k_need = k;
        }
        // (streaming loads go past the last-level cache)
        const LaunchBytes bytes = launch_bytes(w, seg_at, segs, n_segs);
        const bool stream = bytes.stream(n_sets);
        for (uint32_t i = 0, to = 0; i < n_segs; ++i) {
            const uint32_t *sh = w + seg_at[segs[i]];
            memcpy(ka.code + to, sh, (size_t)sh[S_WORDS] * 4);
            for (uint32_t pc = SH_WORDS; !stream && pc < sh[S_WORDS]; pc += (sh[pc] >> 8) & 0xFF)
                if ((sh[pc] & 0xFF) == I_LOAD || (sh[pc] & 0xFF) == I_VLOAD) ka.code[to + pc + 1] &= ~(MF_STREAM << 16);
            to += sh[S_WORDS];
        }
        ka.set_tiles = (uint32_t)total;
        if (total == 0) continue;       // (its segments are empty)
        if (total < (1ull << 31)) magic_of(ka.set_tiles, &ka.set_m, &ka.set_sh);
        total *= (uint64_t)n_sets;
        // Several segments, or several sets: the tiles of each are dealt out from where the one before stopped.  (Not
        // when a segment relies on its producer's assignment of tiles to workgroups, nor when the segments own shares
        // of the workgroups.)
        ka.rotate = !rotates ? 0u : round_robin && !grid_sync && total < (1ull << 31) ? 1u : 2u;        // (every workgroup arrives at a grid-wide wait)
        // The instantiations that pass over foreign sets and segments are some 8 % slower per tile; the others spend 1.1 us on each.
        // They pay where that is more than 8 % of the time the launch's bytes take at 5 TB/s, i.e. below 69 MB per segment and set
        // (32 layers of five programs at 512 tokens, 18 MB each: 604 us against 639; eight RMSNorms of 285 MB: the other way round).
        const bool skip = ka.rotate == 1 && bytes.spans < (uint64_t)n_segs * (69ull << 20);
        const bool narrow = apart && k_need <= 32;
        const int K_l = narrow ? 32 : K, NR_l = narrow ? 2 : NR;
        vm_launch_t launch = nullptr;
        if (cred) {
            for (const VariantEntry &v : g_cred_variants)
                if (v.K == K && v.NR == NR) launch = v.launch;
        } else {
            const bool one = n_segs == 1 && n_sets == 1;
            const bool any = need.part || (need.longrow && (!wide || need.mac || !one));
            if (!any && !skip && ka.rotate == 1) ka.rotate = 2;         // (they know the other way of counting only)
            const VariantEntry *list = any ? g_any_variants : need.longrow ? g_long_wide_variants
                                       : skip ? (wide ? g_wide_variants : g_variants) : (wide ? g_visit_wide_variants : g_visit_variants);
            for (int i = 0; i < N_VARIANTS; ++i)
                if (list[i].K == K_l && list[i].NR == NR_l) launch = list[i].launch;
        }
        if (!launch) return dvm_set_error(DVM_E_BADCODE, "dvm_run: no interpreter variant for this bytecode");
        uint32_t grid = w[PH_GRID];
        if (grid_sync || (ka.rotate != 0 && (total > grid || apart))) {
            int per_cu = 0, n_cu = 0;
            e = (hipError_t)resident_per_cu(launch, block, need.lds_bytes, &per_cu);
            if (e != hipSuccess) {
                t_last_hip_error = (int)e;
                return dvm_set_error(DVM_E_HIP, hipGetErrorString(e));
            }
            dvm_ctx_planner_get(ctx, &n_cu, nullptr);
            if (grid_sync) {
                // every workgroup waits for all the others: the whole grid has to be resident at once
                // (the parts were planned one by one, some for interpreter variants that hold more waves than the
                // launch's common one: the interpreter deals the tiles out over whatever grid it finds itself in)
                if (per_cu < 1 || n_cu < 1)
                    return dvm_set_error(DVM_E_UNSUPPORTED, "dvm_run: the device holds no workgroup of this launch's size");
                if ((uint64_t)grid > (uint64_t)per_cu * (uint64_t)n_cu) grid = (uint32_t)per_cu * (uint32_t)n_cu;
            } else {
                // A launch whose segments (and sets) deal their tiles out in rotation keeps as many workgroups busy as it has
                // tiles in all: the grid grows from what the largest segment alone asked for to that, up to what the device holds
                // at once (short segments of many sets then run side by side instead of one after the other on a few workgroups).
                // Where launches differ in variant, each gets the grid of its own.
                const uint64_t cap = (uint64_t)(per_cu > 0 ? per_cu : 1) * (uint64_t)(n_cu > 0 ? n_cu : 1);
                const uint64_t want = total < cap ? total : cap;
                if (want > grid || (apart && want > 0)) grid = (uint32_t)want;
            }
        }
        // (every launch counts its arrivals at grid-wide waits from zero; the status word stays)
        if (grid_sync && vm_runs++ != 0) hipLaunchKernelGGL(dvm_ws_clear, dim3(1), dim3(64), 0, (hipStream_t)hip_stream, (uint32_t *)(uintptr_t)ka.ws, 1u);
        dvm_colreduce_args ca;
        uint32_t cgrid = 0, cblock = 0;
        const uint32_t *first_sh = w + seg_at[segs[0]];
        // A large launch of one segment spreads its tiles over eight times the workgroups that are resident: those that walk many tiles
        // drift apart, and the memory in use with them, while the dispatcher starts the next ones in order (fp32 add over 45M elements 93.6 -> 87.2 us,
        // RMSNorm bf16 [42648, 4096] 127 -> 119).  A prologue (pinned operands) runs in every workgroup: each of its records wants two and a
        // half tiles behind it (LayerNorm bf16 [163840, 2048] 250 -> 241, but [81920, 1024], with one tile behind two, 63 -> 68).  Flat programs, whose tiles
        // cost the same, gain from 64 MB on, where their last round is not full (fp32 add over 15M elements 34.0 -> 31.9, over 10M 23.1 -> 23.3).
        if (w[PH_NSEG] == 1 && n_sets == 1 && !cred && !longrow && bytes.touched >= (first_sh[S_NCT] > 1 ? FLAT_MIN_BYTES : LARGE_MIN_BYTES) && (first_sh[S_FLAGS] & SF_INTERLEAVED) && !(first_sh[S_FLAGS] & SF_LDS)) {
            uint32_t records = 0;
            for (uint32_t pc = SH_WORDS; pc < SH_WORDS + first_sh[S_PROLOG]; pc += (first_sh[pc] >> 8) & 0xFF) ++records;
            if (records == 0 || 2 * total >= 5ull * records * 8u * grid) grid = total < 8ull * grid ? (uint32_t)total : 8u * grid;
        }
        if (cred && n_segs == 1 && !batch && plain_colreduce(ctx, first_sh, ka.tensors, ka.aliased != 0, &ca, &cgrid, &cblock))
            e = (hipError_t)dvm_colreduce_launch(&ca, cgrid, cblock, hip_stream);
        else
            e = (hipError_t)launch(grid, block, need.lds_bytes, hip_stream, &ka, nullptr);
        if (e != hipSuccess) {
            t_last_hip_error = (int)e;
            return dvm_set_error(DVM_E_HIP, hipGetErrorString(e));
        }
    }
    return DVM_OK;
}

}  // namespace

// The number of kernel launches that a run of valid bytecode makes over tensors that start on a line and apart from each other (no HIP call).
extern "C" int dvm_launch_count(const uint32_t *w) {
    if (w[PH_NSEG] > (uint32_t)MAX_SEGMENTS) return 1;      // (none: dvm_run refuses it)
    Runs runs;
    plan_runs(w, nullptr, 0, is_ordered(w), &runs);
    return runs.n > 1 ? (int)runs.n : 1;
}

// The kernel launches that a run of `bytecode` over these tensors makes, without making them (for tests; no HIP call).
extern "C" int dvm_launch_plan(const void *bytecode, size_t len, void *const *tensors, int n_sets, int n_cu, dvm_launch *out, int cap, int *n) {
    if (!bytecode || !tensors || n_sets < 1 || !out || !n) return dvm_set_error(DVM_E_ARGS, "dvm_launch_plan: null argument");
    const int st = dvm_validate(bytecode, len);
    if (st != DVM_OK) return st;
    const uint32_t *w = (const uint32_t *)bytecode;
    if (w[PH_NSEG] > (uint32_t)MAX_SEGMENTS) return dvm_set_error(DVM_E_LIMIT, "dvm_launch_plan: bytecode exceeds the kernel-argument budget");
    uint32_t seg_at[MAX_SEGMENTS];
    for (uint32_t s = 0, at = PH_WORDS_N + w[PH_NTENS] * TT_WORDS; s < w[PH_NSEG]; at += w[at + S_WORDS], ++s) seg_at[s] = at;
    Runs runs;
    plan_runs(w, tensors, n_sets, is_ordered(w), &runs);
    dvm_rotary_args ra;
    const bool rotary = w[PH_NSEG] == 1 && plain_rotary(w + seg_at[0], (int)((w[PH_VARIANT] >> 8) & 0xFF), w + PH_WORDS_N, tensors, n_sets, w[PH_NTENS], &ra);
    *n = (int)runs.n;
    for (uint32_t r = 0; r < runs.n && (int)r < cap; ++r) {
        dvm_launch &l = out[r];
        l = dvm_launch{};
        l.first_segment = runs.list[runs.at[r]];
        l.n_segments = runs.at[r + 1] - runs.at[r];
        if (runs.kind[r] != RUN_VM) {
            dvm_softmax_alike sa;
            dvm_softmax_mixed sx;
            const bool mixed = runs.kind[r] == RUN_MIXED;
            const uint32_t *segs = runs.list + runs.at[r];
            const uint32_t tiles = mixed ? softmax_args(w, seg_at, segs, l.n_segments, tensors, n_sets, 0, &sx) : softmax_args(w, seg_at, segs, l.n_segments, tensors, n_sets, 0, &sa);
            const dvm_softmax_args &sm = mixed ? sx.part[0] : sa.s;
            l.mixed = mixed;
            l.kind = sm.exact ? DVM_LAUNCH_SOFTMAX_EXACT : sm.in_long ? DVM_LAUNCH_SOFTMAX_LONG : DVM_LAUNCH_SOFTMAX;
            l.grid = softmax_grid(sm, tiles, n_cu);
            l.block = softmax_block(sm);
            l.lanes = sm.lanes;
            l.slots = sm.slots;
        } else if (!rotary) {
            l.stream = launch_bytes(w, seg_at, runs.list + runs.at[r], l.n_segments).stream(n_sets);
        } else {
            l.kind = DVM_LAUNCH_ROTARY;
            l.grid = (ra.groups + 3) / 4;
            l.block = 256;
        }
    }
    return DVM_OK;
}

extern "C" int dvm_workspace_status(const void *workspace, void *hip_stream, int *gave_up) {
    if (!workspace || !gave_up) return dvm_set_error(DVM_E_ARGS, "dvm_workspace_status: null argument");
    uint32_t word = 0;
    hipError_t e = hipMemcpyAsync(&word, (const uint32_t *)workspace + WS_STATUS, 4, hipMemcpyDeviceToHost, (hipStream_t)hip_stream);
    if (e == hipSuccess) e = hipStreamSynchronize((hipStream_t)hip_stream);
    if (e != hipSuccess) {
        t_last_hip_error = (int)e;
        return dvm_set_error(DVM_E_HIP, hipGetErrorString(e));
    }
    *gave_up = word != 0;
    return DVM_OK;
}
#endif  // host side
