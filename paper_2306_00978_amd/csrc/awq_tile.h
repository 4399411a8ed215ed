// Host interface of the K-split tile kernel (awq_tile.hip): one linear, 4-, 3- or 2-bit weights.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

struct TilePlan {
    int mt, nt;          // 16-row token tiles and 16-row weight tiles per workgroup
    double us;           // estimated time of the launch
};

// The workgroup shape with the smallest estimated time.
TilePlan awq_tile_plan(int M, int N, int K);
int64_t awq_tile_count(const TilePlan &plan, int M, int N);          // workgroups

// bits is 4, 3 (group 128) or 2 (group 64); M >= 16; other arguments were validated by the caller.
int awq_tile_launch(int bits, const TilePlan &plan, const void *x, const void *qweight, const void *scales,
                    const void *zeros, void *y, int M, int N, int K, hipStream_t stream);

// 4-bit, group 128: stores nothing; loss[workgroup] = sum of (output - y_ref)^2 over the workgroup's tile.
int awq_tile_launch_loss(const TilePlan &plan, const void *x, const void *qweight, const void *scales, const void *zeros,
                         const void *y_ref, int M, int N, int K, double *loss, hipStream_t stream);
