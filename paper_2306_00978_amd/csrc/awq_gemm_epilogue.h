// The end of a 128 x 256 output tile computed by eight waves in pairs (wave w and w + 4 hold partial sums of
// the same 128 x 64 sub-tile, 4 x 2 tiles of 32x32 accumulators): shared by the W4A16 prefill kernel and the dense
// fp16 product of the scale search.
#pragma once

#include "awq_common.h"

// Wave kh (0, 1) of a pair keeps token blocks 2 kh, 2 kh + 1 and hands the other two to its partner
// through LDS: 64 accumulators per lane, stored as [wave][accumulator][lane] (consecutive lanes in consecutive
// words; 128 KB).  own receives the sums of the two it keeps.  (Values are selected, not references: a selected
// reference puts the accumulators into scratch memory.)  Nobody may use the LDS for anything else: every wave has passed a barrier.
__device__ __forceinline__ void gemm_pair_sum(const floatx16 (&acc)[4][2], floatx16 (&own)[2][2], unsigned char *smem,
                                              int wave, int lane, int kh)
{
    float *xch = reinterpret_cast<float *>(smem);
    float *mine = xch + (size_t)wave * (64 * 64);
    const float *theirs = xch + (size_t)(wave ^ 4) * (64 * 64);
#pragma unroll
    for (int ii = 0; ii < 2; ++ii)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                // the block this wave gives away: kh = 0 gives 2, 3; kh = 1 gives 0, 1
                const float first = acc[ii][b][v], second = acc[2 + ii][b][v];
                const float give = kh ? first : second;
                own[ii][b][v] = kh ? second : first;
                mine[((ii * 2 + b) * 16 + v) * 64 + lane] = give;
            }
    __syncthreads();
#pragma unroll
    for (int ii = 0; ii < 2; ++ii)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                own[ii][b][v] += theirs[((ii * 2 + b) * 16 + v) * 64 + lane];
            }
    __syncthreads();
}

// Accumulator v of tile (i, b) is y[m0 + 32 i + 8 (v/4) + 4 hi + v%4][16 nt0 + 32 b + l32]: a lane holds
// single columns, which would leave as 2-byte stores.  Each wave turns its 64 x 64 part around, rounded to fp16,
// through its own 9 KB of LDS (rows of 128 + 16 bytes: the padding spreads the banks); afterwards lane l reads
// row 8 it + l / 8, columns 8 (l % 8) .. + 8 with gemm_row16.
constexpr int GEMM_ROWB = 144;
__device__ __forceinline__ unsigned char *gemm_turn(const floatx16 (&own)[2][2], unsigned char *smem, int wave, int l32,
                                                    int hi)
{
    unsigned char *mine = smem + (size_t)wave * (64 * GEMM_ROWB);
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int ii = 0; ii < 2; ++ii)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int row = 32 * ii + 8 * (v >> 2) + 4 * hi + (v & 3);
                *reinterpret_cast<half_t *>(mine + row * GEMM_ROWB + (32 * b + l32) * 2) = (half_t)own[ii][b][v];
            }
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
