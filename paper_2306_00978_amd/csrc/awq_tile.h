// Host interface of the K-split tile kernel (awq_tile.hip): one linear, 4-, 3- or 2-bit weights.
#pragma once

#include <hip/hip_runtime.h>

struct TilePlan {
    int mt, nt;          // 16-row token tiles and 16-row weight tiles per workgroup
    double us;           // estimated time of the launch
};

// The workgroup shape with the smallest estimated time.
TilePlan awq_tile_plan(int M, int N, int K);

// bits is 4, 3 (group 128) or 2 (group 64); M >= 16; other arguments were validated by the caller.
int awq_tile_launch(int bits, const TilePlan &plan, const void *x, const void *qweight, const void *scales,
                    const void *zeros, void *y, int M, int N, int K, hipStream_t stream);
