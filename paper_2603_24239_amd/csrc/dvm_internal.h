// Declarations shared by the host encoder (dvm_encode.cpp) and the device file (dvm_vm.hip).
#ifndef DVM_INTERNAL_H
#define DVM_INTERNAL_H

#include "../../include/dvm.h"

#ifdef __cplusplus
extern "C" {
#endif

// Record an error detail for dvm_last_error_detail() on this thread and return `status`.
int dvm_set_error(int status, const char *detail);
// HIP device the context was created for, or -1.
int dvm_ctx_device(const dvm_ctx *ctx);
// Planner inputs of the context (either pointer may be null).
void dvm_ctx_planner_get(const dvm_ctx *ctx, int *n_cu, int *overhead);
// Bound on the polls of a grid-wide synchronisation point (dvm_ctx_set_sync_limit).
int64_t dvm_ctx_sync_limit(const dvm_ctx *ctx);
// A plain reduction along the penultimate axis as its own kernel takes it (dvm_colreduce.hip): sizes and strides in elements.
typedef struct dvm_colreduce_args {
    const void *in;
    void *out;
    int64_t in_s1, in_s2, in_s3;    // strides of the reduced axis and of the two outer dims
    int64_t out_s2, out_s3;
    uint64_t cols;                  // N: at least one 16-byte piece of the input
    uint32_t size;                  // rows reduced
    uint32_t d2;                    // extent of the first outer dim (0: the only one)
    uint32_t col_tiles, log2_lanes; // column tiles of a row; lanes (of 16 bytes) that share a row
    uint32_t waves, partials;       // the segment's waves per unit and partial results per wave: they fix the order of the rows
    uint32_t op;                    // R_SUM, R_MAX or R_MIN
    uint32_t in_bf16, out_bf16;
} dvm_colreduce_args;
int dvm_colreduce_launch(const dvm_colreduce_args *a, unsigned grid, unsigned block, void *stream);
// A softmax along the row, of one tensor or of the sum of two, as its own kernel takes it (dvm_softmax.hip): sizes and strides in elements.
typedef struct dvm_softmax_args {
    const void *a, *b;              // b: the second tensor of the sum (null: none)
    void *y;
    uint64_t sets;                  // batched launch: device array of n_sets * n_tensors addresses (0: the three above)
    uint32_t n_tensors, ia, ib, iy; // and where the three stand in a set
    uint32_t bf16;                  // the dtype of all three: bf16 or fp32
    int64_t a_s[3], b_s[3], y_s[3]; // strides of the outer dims, the first of them varying fastest from row to row
    uint32_t d1, m1, sh1, d2, m2, sh2;      // extents of the first two and the multiply-shift constants that divide by them
    uint32_t limit;                 // blocked order (0: none): the third index counts blocks of d1 along one dim, of this extent
    uint32_t rows, cols;            // rows of a set (blocked order: with those that the last block has too many), columns
    uint32_t tiles;                 // of all sets
    uint32_t set_tiles, set_m, set_sh;      // of one set
    uint32_t exact;                 // 1: rows laid out and added up as the interpreter does
    uint32_t ragged;                // exact: the row does not fill the tile
    uint32_t lanes, log2_lanes;     // lanes on a row: a power of two from 8 to 512, in long rows 512 or 1024 (exact: from 1 to 64, log2 given)
    uint32_t in_long;               // 1: the kernel for long rows (lanes: 512 or 1024)
    uint32_t slots;                 // 16-byte chunks of a lane
    uint32_t tail;                  // a row may end in this slot of chunks or behind it
    uint32_t stream;                // 1: larger than the last-level cache holds, read past it
    uint32_t shifted;               // 1: a row's chunks are laid on the 128-byte lines of the output, 0: they start with the row
} dvm_softmax_args;
// What a launch takes: one of them, or (sets = DVM_SOFTMAX_PARTS, n_tensors 3, in the order 0, 1, 2) several alike in all but their addresses
constexpr uint32_t DVM_SOFTMAX_MAX_PARTS = 16;
constexpr uint64_t DVM_SOFTMAX_PARTS = 1;
typedef struct dvm_softmax_alike {
    dvm_softmax_args s;
    uint64_t parts[3 * DVM_SOFTMAX_MAX_PARTS];
} dvm_softmax_alike;
// or several alike in type, second tensor or none, and kernel (lanes up to 256; or the same lanes and in_long) only
typedef struct dvm_softmax_mixed {
    uint32_t n;
    uint32_t first[DVM_SOFTMAX_MAX_PARTS + 1];          // tiles of the parts before each, and of all
    dvm_softmax_args part[DVM_SOFTMAX_MAX_PARTS];
} dvm_softmax_mixed;
static_assert(sizeof(dvm_softmax_mixed) <= 4096, "a kernel's arguments");
constexpr int64_t DVM_SOFTMAX_MIN_BYTES = 16 << 20;
int dvm_softmax_launch(const dvm_softmax_alike *a, unsigned grid, void *stream);
int dvm_softmax_launch_mixed(const dvm_softmax_mixed *p, unsigned grid, void *stream);
// A rotation of pairs over short rows as its own kernel takes it (dvm_rotary.hip): tensors in the order x1, x2, c, s, y1, y2; strides in elements.
typedef struct dvm_rotary_args {
    uint64_t p[6];                  // addresses
    uint64_t sets;                  // batched launch: device array of n_sets * n_tensors addresses (0: `p`)
    int64_t s[6][3];                // strides of the outer dims, the first of them varying fastest from row to row
    uint32_t at[6], n_tensors;      // where the six stand in a set
    uint32_t d1, m1, sh1, d2, m2, sh2;      // extents of the first two outer dims and the multiply-shift constants that divide by them
    uint32_t rows;                  // of a set
    uint32_t groups;                // waves' shares of rows, of all sets
    uint32_t set_groups, set_m, set_sh;     // of one set
    uint32_t log2_lanes;            // lanes on a row, of 16 bytes of x each
    uint32_t rows_per_lane;         // 4: rows of one index of the dims behind the first, along which the tables do not change; else 1
    uint32_t fused;                 // y2: 0: both products rounded, 1: x2 c fused into the sum, 2: x1 s
    uint32_t x_bf16, t_bf16;        // x1, x2, y1, y2; c, s
    uint32_t stream;                // 1: larger than the last-level cache holds, read past it
} dvm_rotary_args;
int dvm_rotary_launch(const dvm_rotary_args *a, void *stream);
// One kernel launch of a run, as far as it is known without the device (the interpreter's grid is not).
typedef struct dvm_launch {
    uint32_t kind;                  // DVM_LAUNCH_*
    uint32_t first_segment, n_segments;
    uint32_t grid, block;
    uint32_t lanes, slots;          // a softmax: lanes on a row, 16-byte chunks of a lane (mixed: of the first part)
    uint32_t mixed;                 // softmaxes of several shapes
    uint32_t stream;                // the interpreter: loads take the streaming hint
} dvm_launch;
enum { DVM_LAUNCH_INTERPRETER = 0, DVM_LAUNCH_SOFTMAX, DVM_LAUNCH_SOFTMAX_LONG, DVM_LAUNCH_SOFTMAX_EXACT, DVM_LAUNCH_ROTARY };
int dvm_launch_count(const uint32_t *program);
int dvm_launch_plan(const void *bytecode, size_t len, void *const *tensors, int n_sets, int n_cu, dvm_launch *out, int cap, int *n);
// Implemented in the device file so that the encoder object stays free of HIP calls.
int dvm_ctx_query_device(int hip_device, int *n_cu);

#ifdef __cplusplus
}
#endif
#endif
