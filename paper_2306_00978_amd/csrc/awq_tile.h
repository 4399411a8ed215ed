// Host interface of the K-split tile kernel (awq_tile.hip): one linear, 4-, 3- or 2-bit weights.
#pragma once

#include "awq_common.h"

struct TilePlan {
    int mt, nt;          // 16-row token tiles and 16-row weight tiles per workgroup
    double us;           // estimated time of the launch
};

// The workgroup shape with the smallest estimated time, for `points` products of this shape in one launch.
TilePlan awq_tile_plan(int M, int N, int K, int points = 1);

// A tie between its estimate and the prefill kernel's is the tile kernel's: it applies the steps in fp32, the prefill kernel
// rounds the dequantized weights to fp16 (errors against 64 bits 2.1e-4 and 2.9e-4).  The estimates are 5 % off.
constexpr double AWQ_TILE_TIE = 1.05;

// The tuning build can force the shape (AWQ_TILE_PLAN = 10 * mt + nt, at every token count above 16) or, with 0, the
// kernels that run where this one does not.
inline int awq_tile_override() { return awq_knob("AWQ_TILE_PLAN", -1); }
inline bool awq_tile_forced() { return awq_tile_override() > 0; }
int64_t awq_tile_count(const TilePlan &plan, int M, int N);          // workgroups

// bits is 4, 3 (group 128) or 2 (group 64); M >= 16; other arguments were validated by the caller.
int awq_tile_launch(int bits, const TilePlan &plan, const void *x, const void *qweight, const void *scales,
                    const void *zeros, void *y, int M, int N, int K, hipStream_t stream);

// 4-bit, group 128: stores nothing; loss[workgroup] = sum of (output - y_ref)^2 over the workgroup's tile.  The next one of
// `points` grid points has its operands `step` bytes and its sums loss_step further.
int awq_tile_launch_loss(const TilePlan &plan, const void *x, const void *qweight, const void *scales, const void *zeros,
                         const void *y_ref, int M, int N, int K, double *loss, int points, size_t step, size_t loss_step,
                         hipStream_t stream);
