// The end of a 128 x 256 output tile computed by eight waves in pairs (wave w and w + 4 hold partial sums of
// the same 128 x 64 sub-tile, 8 x 4 tiles of 16x16 accumulators): shared by the W4A16 prefill kernel and the dense
// fp16 product of the scale search.
#pragma once

#include "awq_common.h"

// Wave kh (0, 1) of a pair keeps the token tiles 4 kh .. 4 kh + 3 and hands the other four to its partner
// through LDS: 64 accumulators per lane, stored as [wave][accumulator][lane] (consecutive lanes in consecutive
// words; 128 KB).  own receives the sums of the four it keeps.  (No reference is selected: that puts the accumulators into
// scratch memory.)  3.1 thousand cycles, 5.2 with a selection per value; as 16 bytes per lane 5.4.
// Nobody may use the LDS for anything else: every wave has passed a barrier.
__device__ __forceinline__ void gemm_pair_sum(const floatx4 (&acc)[8][4], floatx4 (&own)[4][4], unsigned char *smem,
                                              int wave, int lane, int kh)
{
    float *xch = reinterpret_cast<float *>(smem);
    float *mine = xch + (size_t)wave * (64 * 64);
    const float *theirs = xch + (size_t)(wave ^ 4) * (64 * 64);
    // the tiles this wave gives away: kh = 0 gives 4 .. 7; kh = 1 gives 0 .. 3
    auto divide = [&](const floatx4 (*keep)[4], const floatx4 (*give)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int n = 0; n < 4; ++n)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    mine[((i * 4 + n) * 4 + v) * 64 + lane] = give[i][n][v];
                    own[i][n][v] = keep[i][n][v];
                }
    };
    // (the comments differ so that the compiler keeps two branches: as one with a selection per value it costs 128 more
    // vector instructions)
    if (kh) {
        divide(acc + 4, acc);
        asm volatile("; keeps 4 .. 7");
    } else {
        divide(acc, acc + 4);
        asm volatile("; keeps 0 .. 3");
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int n = 0; n < 4; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v) own[i][n][v] += theirs[((i * 4 + n) * 4 + v) * 64 + lane];
    __syncthreads();
}

// Lane (r, c) = (l % 16, l / 16): accumulator v of tile (i, n) is y[m0 + 16 i + 4 c + v][16 nt0 + 16 n + r]: a lane
// holds single columns, which would leave as 2-byte stores.  Each wave turns its 64 x 64 part around, rounded to fp16,
// through its own 9 KB of LDS (rows of 128 + 16 bytes: the padding spreads the banks); afterwards lane l reads
// row 8 it + l / 8, columns 8 (l % 8) .. + 8 with gemm_row16.
constexpr int GEMM_ROWB = 144;
__device__ __forceinline__ unsigned char *gemm_turn(const floatx4 (&own)[4][4], unsigned char *smem, int wave, int lane)
{
    unsigned char *mine = smem + (size_t)wave * (64 * GEMM_ROWB);
    const int r = lane & 15, c = lane >> 4;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int n = 0; n < 4; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                *reinterpret_cast<half_t *>(mine + (16 * i + 4 * c + v) * GEMM_ROWB + (16 * n + r) * 2) = (half_t)own[i][n][v];
    // wave-private area: the compiler orders the LDS reads after the writes above
    return mine;
}
__device__ __forceinline__ uint4 gemm_row16(const unsigned char *mine, int it, int lane)
{
    return *reinterpret_cast<const uint4 *>(mine + (it * 8 + (lane >> 3)) * GEMM_ROWB + (lane & 7) * 16);
}

// The wave's 64 x 64 part to y: 16 bytes per lane, 8 rows x 128 contiguous bytes per instruction.
__device__ __forceinline__ void gemm_store(const unsigned char *mine, half_t *y, int m_first, int n_first, int M, int N,
                                           int lane)
{
    const int n = n_first + (lane & 7) * 8;
#pragma unroll
    for (int it = 0; it < 8; ++it) {
        const uint4 v = gemm_row16(mine, it, lane);
        const int m = m_first + it * 8 + (lane >> 3);
        if (m < M && n < N) *reinterpret_cast<uint4 *>(y + (size_t)m * N + n) = v;
    }
}
