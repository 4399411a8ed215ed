// Decode path of awq_w4a16_linear (M <= 16) for gfx950.
//
// AWQ Sec. 4.2: generation is memory-bound and weight traffic dominates, so the
// 4-bit weights are streamed once and dequantized on the fly inside the
// matrix-vector kernel; nothing dequantized is written back to memory.  The same
// passage warns that dequantization (shift, AND, FMA per weight) costs more ALU
// work than the product it feeds; the scheme below brings it to 5 vector
// instructions per 8 weights.
//
// Mapping.  A workgroup owns one 16-row block of W (its tiles are contiguous along
// K); its waves split the K/128 groups between them.  Per tile a lane issues one
// 16-byte load (the wave reads the 1 KB tile fully coalesced) and receives, in
// word j, eight codes that are its B-operand fragment of the j-th
// v_mfma_f32_16x16x32_f16 step (n = lane%16, k = 32j + 8*(lane/16) + 0..7).  The
// activations are the A operand (m = lane%16), so one MFMA chain handles up to 16
// tokens at the cost of one, and the k-reduction across lanes happens inside the
// matrix core instead of through shuffles.
//
// Dequantization.  The nibble order of a word makes
//   (w >> {0,8}) & 0x000F000F | 0x64006400  the half pair (1024+q, 1024+q')  and
//   (w >> {0,8}) & 0x00F000F0 | 0x54005400  the half pair (  64+q,   64+q'),
// one v_and_or_b32 each.  These biased halves go to the matrix core as they are, and
// a second MFMA with the constant fragment -(1024+z), -(64+z) takes the bias and the
// zero point out again:  sum_k x_k (1024 + q_k) - sum_k x_k (1024 + z) = sum_k x_k (q_k - z).
// All products are exact in fp32; the two chains alternate so the running sum stays
// small.  The group's step is applied once per group in fp32.
//
// The partial sums of the waves are combined through LDS in a fixed order
// (deterministic output), rounded once to fp16 and stored.
#include "awq_common.h"
#include "awq_gemv_stream.h"

#include <stdlib.h>

#include <algorithm>

namespace {

// The four constants of the expansion, held in registers.  They are made opaque to the
// optimizer so that (w & mask) | bits is selected as ONE v_and_or_b32 (mask in an SGPR,
// bits in a VGPR) instead of a v_and_b32 and a v_or_b32 with literal operands.
struct ExpandConsts {
    uint32_t mask_lo, mask_hi;   // 0x000F000F, 0x00F000F0  (SGPR)
    uint32_t magA, magB;         // 0x64006400, 0x54005400  (VGPR)
};

__device__ __forceinline__ ExpandConsts expand_consts()
{
    ExpandConsts k = {0x000F000Fu, 0x00F000F0u, 0x64006400u, 0x54005400u};
    asm("" : "+s"(k.mask_lo));
    asm("" : "+s"(k.mask_hi));
    asm("" : "+v"(k.magA));
    asm("" : "+v"(k.magB));
    return k;
}

// Eight codes of one packed word -> eight biased halves, in k order.
__device__ __forceinline__ half8_t biased_halves(uint32_t w, const ExpandConsts &k)
{
    const uint32_t w8 = w >> 8;
    uint4 t;
    t.x = (w & k.mask_lo) | k.magA;    // 1024 + (e0, e1)
    t.y = (w & k.mask_hi) | k.magB;    //   64 + (e2, e3)
    t.z = (w8 & k.mask_lo) | k.magA;   // 1024 + (e4, e5)
    t.w = (w8 & k.mask_hi) | k.magB;   //   64 + (e6, e7)
    return __builtin_bit_cast(half8_t, t);
}

// One batch of U consecutive tiles (groups) of a wave, as loaded from global memory.  The
// tiles of a row block are contiguous along K, so the U loads differ by a constant 1 KB.
// The step and zero point are fetched with ONE 2-byte and ONE 1-byte load per lane for the
// whole batch: lane (r, c) fetches those of row r of group base + min(c, U-1), turns them
// into the three per-tile constants, and tile u later takes them from lane r + 16u with
// cross-lane permutes.
// BITS = 4: a tile is 64 slots of 16 bytes; BITS = 3 (the INT3-g128 variant of Sec. 5): 64 slots
// of 12 bytes, three words per lane.
template <int BITS, int U>
struct TileBatch {
    uint32_t q[U][BITS];
    uint32_t s_raw, z_raw;
};

template <int BITS, int U>
__device__ __forceinline__ void load_batch(TileBatch<BITS, U> &b, const uint32_t *qt, const uint16_t *sc,
                                           const uint8_t *zp, int base)
{
    // the two small loads go first: loads return in order, and the first tile can only be
    // consumed once its step and zero point are there
    b.s_raw = sc[base * 16];
    b.z_raw = zp[base * 8];
    const uint32_t *p = qt + base * (64 * BITS);          // qt already points at this lane's slot
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (BITS == 4) {
            const uint4 v = *reinterpret_cast<const uint4 *>(p + u * 256);
            b.q[u][0] = v.x; b.q[u][1] = v.y; b.q[u][2] = v.z; b.q[u][BITS - 1] = v.w;
        } else {
#pragma unroll
            for (int i = 0; i < BITS; ++i) b.q[u][i] = p[u * 192 + i];
        }
    }
}

// INT3 slot: pair p = 0..14 of the 16 code pairs sits in word p/5 at bits [3f, 3f+3), f = p%5,
// of both halves; pair 15 in the top bits of the six halves.  (word >> 3f) & 0x00070007 is the
// pair as two fp16 subnormals q * 2^-24, exactly (raised_halves below: what the matrix core makes of them).
__device__ __forceinline__ half8_t w3_halves(const uint32_t (&w)[3], uint32_t last_pair, int j)
{
    uint32_t t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int p = 4 * j + i;
        t[i] = p < 15 ? ((w[p / 5] >> (3 * (p % 5))) & 0x00070007u) : last_pair;
    }
    return __builtin_bit_cast(half8_t, make_uint4(t[0], t[1], t[2], t[3]));
}

// Decode kernel.
// U     = tiles (groups) per batch, a divisor of G: 1 or 2.  A wave owns whole batches.
// PIPE  = double-buffer the batches (only worth its registers when a wave has several).
// MS (M <= MS <= 16, a multiple of the 4 / U rows that a load covers): each wave copies the slice of x that its batch needs
//   (MS rows x U*128 halves; rows >= M repeat row M-1) into a private LDS area with one coalesced
//   16-byte load per lane for every 4 / U rows, issued before the weight loads so that it returns first,
//   and then reads its A fragments from LDS.  No workgroup barrier is involved, so a wave
//   starts computing as soon as its own weights arrive.  With few rows most lanes of an A
//   fragment are duplicates, which is why this is cheaper than loading fragments from
//   global memory.
//
// The workgroup has W = 2^logW waves; wave w owns batches [NB*w/W, NB*(w+1)/W), NB = G/U.
// Dynamic LDS: [W][MS rows x (U*256 + 16) bytes], then 16*M outputs x 16 wave slots of
// fp32 for the cross-wave reduction.
template <int BITS, int U, int MS, bool PIPE>
__global__ __launch_bounds__(1024, MS >= 8 ? 4 : 6) void gemv_kernel(
    const half_t *__restrict__ x, const uint32_t *__restrict__ qweight,
    const uint16_t *__restrict__ scales, const uint8_t *__restrict__ zeros,
    half_t *y, int M, int N, int K, int G, int logW, const half_t *res)
{
    extern __shared__ __align__(16) unsigned char smem[];
    // all arguments are fetched in one round, before the first branch: left to itself the
    // compiler sinks the pointer loads below it, a second scalar-cache miss in front of the
    // first request of a kernel that lives for a few microseconds
    asm volatile("" ::"s"(x), "s"(qweight), "s"(scales), "s"(zeros), "s"(y), "s"(M), "s"(N), "s"(K), "s"(G),
                 "s"(logW), "s"(res));
    const ExpandConsts kc = expand_consts();
    // staging: a row of the batch is U*16 lanes wide, so one 16-byte load per lane covers
    // RPP = 64 / (U*16) rows; NS passes cover the MS rows
    constexpr int LPR = U * 16, RPP = 64 / LPR;
    constexpr int NS = MS / RPP;
    static_assert(MS % RPP == 0, "whole loads");
    constexpr int ROW_BYTES = U * 256 + 16;           // +16: rows land on different banks
    constexpr int WAVE_BYTES = MS * ROW_BYTES;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform
    const int W = 1 << logW;
    const int rb = blockIdx.x;
    const int r = lane & 15, c = lane >> 4;
    const int cu = c < U ? c : U - 1;                 // group of the batch this lane fetches meta for

    const int NB = G / U;
    const int g0 = ((NB * wave) >> logW) * U, g1 = ((NB * (wave + 1)) >> logW) * U;
    const uint32_t *qt = qweight + ((int64_t)rb * G * 64 + lane) * BITS;
    const uint16_t *sc = scales + (int64_t)rb * G * 16 + cu * 16 + r;
    const uint8_t *zp = zeros + (int64_t)rb * G * 8 + cu * 8 + (r >> 1);
    const int zshift = (r & 1) * 4;

    // A-operand row m = lane%16.  Rows >= M use row M-1 instead of zeros: row m of the MFMA
    // result depends on row m of A only, and rows >= M are never stored.
    const int mrow = r < M ? r : M - 1;
    unsigned char *xw = smem + (size_t)wave * WAVE_BYTES;                 // this wave's x slice
    const uint4 *xl = reinterpret_cast<const uint4 *>(xw + mrow * ROW_BYTES) + c;
    // staging source of this lane in pass i: row i*RPP + lane/LPR (clamped to M-1 for the load),
    // 16-byte chunk lane%LPR of the batch
    const int srow = lane / LPR, schunk = lane % LPR;
    const uint4 *xstage = reinterpret_cast<const uint4 *>(x) + schunk;
    const int64_t K8 = (int64_t)K >> 3;
    auto stage_src = [&](int i, int g) -> const uint4 & {
        const int m = i * RPP + srow;
        return xstage[(int64_t)(m < M ? m : M - 1) * K8 + g * 16];
    };
    auto stage_store = [&](int i, const uint4 &v) {
        const int m = i * RPP + srow;
        reinterpret_cast<uint4 *>(xw + m * ROW_BYTES)[schunk] = v;
    };

    TileBatch<BITS, U> cur;
    uint4 xs[NS];
#pragma unroll
    for (int m = 0; m < NS; ++m) xs[m] = make_uint4(0, 0, 0, 0);
    if (g0 < g1) {
        // first: it must not wait for the weights
#pragma unroll
        for (int m = 0; m < NS; ++m) xs[m] = stage_src(m, g0);
        load_batch<BITS, U>(cur, qt, sc, zp, g0);
    }

    floatx4 total = {0.f, 0.f, 0.f, 0.f};
    for (int base = g0; base < g1; base += U) {
        // LDS ops of one wave execute in order
#pragma unroll
        for (int m = 0; m < NS; ++m) stage_store(m, xs[m]);
        // PIPE: the next batch is requested before this one is consumed
        TileBatch<BITS, U> nxt;
        const bool more = base + U < g1;
        if (PIPE && more) {
#pragma unroll
            for (int m = 0; m < NS; ++m) xs[m] = stage_src(m, base + U);
            load_batch<BITS, U>(nxt, qt, sc, zp, base + U);
        }
        // constants of (group base + cu, row r), computed once per batch by their owner lane
        const uint32_t z = (cur.z_raw >> zshift) & 0xFu;
        const uint32_t own_nzA = 0xE400E400u | (z * 0x00010001u);      // -(1024 + z) twice
        const uint32_t own_nzB = 0xD400D400u | (z * 0x00100010u);      // -(  64 + z) twice
        const float own_sv = (float)__builtin_bit_cast(half_t, (uint16_t)cur.s_raw);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            uint4 xa[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // k = 128g + 32j + 8c + 0..7 -> 16-byte chunk 16g + 4j (+c folded into xl)
                xa[j] = xl[u * 16 + 4 * j];
            }
            const int src = r + 16 * u;
            const uint32_t nzA = __shfl(own_nzA, src);
            const uint32_t nzB = __shfl(own_nzB, src);
            const float sv = __shfl(own_sv, src);
            if (BITS == 4) {
                const half8_t nb = __builtin_bit_cast(half8_t, make_uint4(nzA, nzB, nzA, nzB));
                floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const half8_t a = __builtin_bit_cast(half8_t, xa[j]);
                    const half8_t b = biased_halves(cur.q[u][j & (BITS - 1)], kc);
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, nb, acc, 0, 0, 0);
                }
#pragma unroll
                for (int v = 0; v < 4; ++v) total[v] += sv * acc[v];
            } else {
                // codes as subnormals q * 2^-24; the zero point leaves in fp32 through
                // S = 2^-24 * sum_k x_k (a second chain against the constant code 1)
                const uint32_t w3[3] = {cur.q[u][0], cur.q[u][1], cur.q[u][2]};
                const uint32_t last = ((w3[0] >> 15) & 0x00010001u) | ((w3[1] >> 14) & 0x00020002u) |
                                      ((w3[2] >> 13) & 0x00040004u);
                const half8_t ones = __builtin_bit_cast(half8_t, make_uint4(0x00010001u, 0x00010001u, 0x00010001u, 0x00010001u));
                floatx4 acc = {0.f, 0.f, 0.f, 0.f}, xsum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const half8_t a = __builtin_bit_cast(half8_t, xa[j]);
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, w3_halves(w3, last, j), acc, 0, 0, 0);
                    xsum = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, ones, xsum, 0, 0, 0);
                }
                const float zf = __shfl((float)z, src);
                const float s24 = sv * 16777216.f;
#pragma unroll
                for (int v = 0; v < 4; ++v) total[v] += s24 * (acc[v] - zf * xsum[v]);
            }
        }
        if (PIPE) {
            if (more) cur = nxt;
        } else if (more) {
#pragma unroll
            for (int m = 0; m < NS; ++m) xs[m] = stage_src(m, base + U);
            load_batch<BITS, U>(cur, qt, sc, zp, base + U);
        }
    }

    // lane holds the partial y[m = 4c + v][n = 16 rb + r]; combine the waves in fixed order.
    // red[t][w], t = 16 m + n: the 16 partials of one output are contiguous.
    float *red = reinterpret_cast<float *>(smem + (size_t)W * WAVE_BYTES);
    if (4 * c < M) {
#pragma unroll
        for (int v = 0; v < 4; ++v) red[((4 * c + v) * 16 + r) * 16 + wave] = total[v];
    }
    __syncthreads();
    for (int t = threadIdx.x; t < 16 * M; t += blockDim.x) {
        const float4 *p = reinterpret_cast<const float4 *>(red + t * 16);
        const float4 a0 = p[0], a1 = p[1], a2 = p[2], a3 = p[3];
        const float part[16] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w,
                                a2.x, a2.y, a2.z, a2.w, a3.x, a3.y, a3.z, a3.w};
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < 16; ++w) sum += (w < W) ? part[w] : 0.f;
        // `res` (may be y itself): a residual added in fp32 before the one rounding
        const int64_t at = (int64_t)(t >> 4) * N + rb * 16 + (t & 15);
        y[at] = (half_t)(res ? sum + (float)res[at] : sum);
    }
}

// The eight codes of step j as subnormals with their top bit at bit 9 of the halves, the place below the exponent: q 2^-18 in 4 bits,
// q 2^-17 in 3 (`last`: pair 15 of a 3-bit slot, in place).  The matrix core aligns a product by the exponents that its
// operands are written with, that of a subnormal always 2^-14, and cuts it off some 23 bits below: codes at the bottom (q 2^-24)
// lose six bits.  Error of the outputs of a layer of hidden size 1024 to 2048 against fp64, 2-norm: 2.13e-4 to 2.23e-4 with codes at the bottom,
// 2.07e-4 with these, which is the rounding to fp16 alone (0.04 to 0.08 % of the outputs rounded otherwise, 14 to 26 % then); one shift more for
// eight codes, the same times (5.5 us at hidden size 1024 and 4 tokens, 7.5 at 1536).
template <int BITS>
__device__ __forceinline__ half8_t raised_halves(const uint32_t *w, uint32_t last, int j)
{
    uint32_t t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int p = 4 * j + i;
        if (BITS == 4) {
            const uint32_t v = w[j & (BITS - 1)];
            t[i] = (i < 2 ? v << (6 - 4 * i) : v >> (4 * i - 6)) & 0x03C003C0u;
        } else if (p < 15) {
            const uint32_t v = w[p / 5], at = 3 * (p % 5);
            t[i] = (at <= 7 ? v << (7 - at) : v >> (at - 7)) & 0x03800380u;
        } else t[i] = last;
    }
    return __builtin_bit_cast(half8_t, make_uint4(t[0], t[1], t[2], t[3]));
}

// Several linears in one launch: the same kernel with eight waves to a row block, which divide the groups of a row evenly,
// whatever their number, and take them two at a time.  A group past the end of a wave's range repeats its last one (loads that
// hit the cache) and is skipped by a wave-uniform branch.  It starts sooner than the streaming kernel (no plan to read, no
// activations to stage for a whole row, everything of a wave requested at once) and spends more instructions per weight, so it
// takes the small launches (awq_linear.hip).  A layer of seven linears at 1 / 4 / 8 tokens, us, before and now: hidden size 1024 (2816)
// 6.3 / 7.9 / 8.5 and 4.7 / 4.7 / 5.6, 1536 (4608) 7.0 / 8.8 / 10.8 and 5.8 / 5.9 / 7.0, 2048 (5632) 8.6 / 10.9 / 13.1 and 8.0 / 8.2 / 10.0.
// (Four groups at a time: 4.9 to 6.9, 6.3 to 9.2, 9.3 to 12.5.)
struct GemvGroupArgs {
    GemvProblem p[GEMV_GROUP_MAX];
    int first[GEMV_GROUP_MAX];                     // workgroup of each
    int count, M;
};
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr int GROUP_LOGW = 3, GROUP_U = 2;

template <int BITS, int MS>
__global__ __launch_bounds__(64 << GROUP_LOGW, MS >= 8 ? 4 : 6) void gemv_group_kernel(const GemvGroupArgs A)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int W = 1 << GROUP_LOGW, U = GROUP_U;
    constexpr int LPR = U * 16, RPP = 64 / LPR, NS = (MS + RPP - 1) / RPP;
    constexpr int ROW_BYTES = U * 256 + 16, WAVE_BYTES = MS * ROW_BYTES;
    int pi = 0;
#pragma unroll
    for (int n = 1; n < GEMV_GROUP_MAX; ++n)
        if (n < A.count && (int)blockIdx.x >= A.first[n]) pi = n;
    const GemvProblem &P = A.p[pi];
    const half_t *__restrict__ x = P.x;
    const uint32_t *__restrict__ qweight = reinterpret_cast<const uint32_t *>(P.q);
    const int N = P.N, G = P.K / AWQ_GROUP, M = A.M;
    half_t *y = P.y;
    asm volatile("" ::"s"(x), "s"(qweight), "s"(P.sc), "s"(P.zp), "s"(y), "s"(N), "s"(G), "s"(M));
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rb = (int)blockIdx.x - A.first[pi];
    const int r = lane & 15, c = lane >> 4;
    const int cu = c < U ? c : U - 1;
    const int g0 = (G * wave) >> GROUP_LOGW, g1 = (G * (wave + 1)) >> GROUP_LOGW;
    const uint32_t *qt = qweight + ((int64_t)rb * G * 64 + lane) * BITS;
    const uint16_t *sc = P.sc + (int64_t)rb * G * 16 + r;
    const uint8_t *zp = P.zp + (int64_t)rb * G * 8 + (r >> 1);
    const int zshift = (r & 1) * 4;
    const int mrow = r < M ? r : M - 1;
    unsigned char *xw = smem + (size_t)wave * WAVE_BYTES;
    const uint4 *xl = reinterpret_cast<const uint4 *>(xw + mrow * ROW_BYTES) + c;
    const int srow = lane / LPR, schunk = lane % LPR;
    const int64_t K8 = (int64_t)G * 16;

    uint32_t q[U][BITS], s_raw = 0, z_raw = 0;
    u32x4 xs[NS];
    auto request = [&](int base) {
        const int last = g1 - 1;
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const int m = i * RPP + srow;
            xs[i] = reinterpret_cast<const u32x4 *>(x)[(int64_t)(m < M ? m : M - 1) * K8 + min(base + (schunk >> 4), last) * 16 + (schunk & 15)];
        }
        const int gm = min(base + cu, last);
        s_raw = sc[gm * 16];
        z_raw = zp[gm * 8];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t *at = qt + min(base + u, last) * (64 * BITS);
            if (BITS == 4) {
                const u32x4 v = *reinterpret_cast<const u32x4 *>(at);
                q[u][0] = v[0]; q[u][1] = v[1]; q[u][2] = v[2]; q[u][BITS - 1] = v[3];
            } else {
#pragma unroll
                for (int i = 0; i < BITS; ++i) q[u][i] = at[i];
            }
        }
    };
    floatx4 total = {0.f, 0.f, 0.f, 0.f};
    if (g0 < g1) request(g0);
    for (int base = g0; base < g1; base += U) {
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const int m = i * RPP + srow;
            reinterpret_cast<u32x4 *>(xw + m * ROW_BYTES)[schunk] = xs[i];
        }
        uint32_t qc[U][BITS];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < BITS; ++i) qc[u][i] = q[u][i];
        // the zero point leaves in fp32 through sum_k x_k (a second chain against the constant 1)
        constexpr float UNIT = BITS == 4 ? 262144.f : 131072.f;        // 1 over a code's step
        const float own_zf = (float)((z_raw >> zshift) & 0xFu) * (1.f / UNIT);
        const float own_sv = (float)__builtin_bit_cast(half_t, (uint16_t)s_raw) * UNIT;
        if (base + U < g1) request(base + U);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (base + u >= g1) continue;                              // wave-uniform
            uint4 xa[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) xa[j] = xl[u * 16 + 4 * j];
            const int src = r + 16 * u;
            const float sv = __shfl(own_sv, src), zf = __shfl(own_zf, src);
            const half8_t ones = __builtin_bit_cast(half8_t, make_uint4(0x3C003C00u, 0x3C003C00u, 0x3C003C00u, 0x3C003C00u));
            floatx4 acc = {0.f, 0.f, 0.f, 0.f}, xsum = {0.f, 0.f, 0.f, 0.f};
            const uint32_t *w = qc[u];
            const uint32_t last = BITS == 3 ? ((w[0] >> 8) & 0x00800080u) | ((w[1] >> 7) & 0x01000100u) | ((w[2] >> 6) & 0x02000200u) : 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const half8_t a = __builtin_bit_cast(half8_t, xa[j]);
                acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, raised_halves<BITS>(w, last, j), acc, 0, 0, 0);
                xsum = __builtin_amdgcn_mfma_f32_16x16x32_f16(a, ones, xsum, 0, 0, 0);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) total[v] += sv * (acc[v] - zf * xsum[v]);
        }
    }
    // the partials of one output are contiguous: red[16 m + n][wave]
    float *red = reinterpret_cast<float *>(smem + (size_t)W * WAVE_BYTES);
    if (4 * c < M) {
#pragma unroll
        for (int v = 0; v < 4; ++v) red[((4 * c + v) * 16 + r) * W + wave] = total[v];
    }
    __syncthreads();
    for (int t = threadIdx.x; t < 16 * M; t += 64 * W) {
        const float4 *p = reinterpret_cast<const float4 *>(red + t * W);
        const float4 a0 = p[0], a1 = p[1];
        const float sum = ((((((a0.x + a0.y) + a0.z) + a0.w) + a1.x) + a1.y) + a1.z) + a1.w;
        y[(int64_t)(t >> 4) * N + rb * 16 + (t & 15)] = (half_t)sum;
    }
}

template <int BITS, int MS>
int gemv_group_one(const GemvGroupArgs &A, int total, hipStream_t stream)
{
    const size_t lds = (size_t)(8 * MS * (GROUP_U * 256 + 16)) + (size_t)((A.M + 3) / 4 * 4) * 16 * 8 * 4;
    static AwqOncePerDevice once;
    std::atomic<bool> &raised = once.here();
    if (lds > 64 * 1024 && !raised.load(std::memory_order_relaxed)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(gemv_group_kernel<BITS, MS>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
            return AWQ_ERR_HIP;
        raised.store(true, std::memory_order_relaxed);
    }
    gemv_group_kernel<BITS, MS><<<dim3((unsigned)total), dim3(64 << GROUP_LOGW), lds, stream>>>(A);
    return awq_launch_status();
}

template <int BITS>
int gemv_group_bits(const GemvGroupArgs &A, int total, hipStream_t stream)
{
    const int M = A.M;
    return M <= 2 ? gemv_group_one<BITS, 2>(A, total, stream)
         : M <= 4 ? gemv_group_one<BITS, 4>(A, total, stream) : M <= 8 ? gemv_group_one<BITS, 8>(A, total, stream)
                                                                       : gemv_group_one<BITS, 16>(A, total, stream);
}

// Waves that share a row block (a power of two) and groups per batch.  Few row blocks: sixteen waves each, so that a CU, which then has
// one of them, has work for all its SIMDs; many: fewer waves with more groups each.  One group per batch from three tokens (two rows staged
// by a load would be a second load), else two where a wave has more than one; four are faster at single shapes only (sixteen waves with four groups
// each, 3392 x 8192 at one token 5.3 us and 5.6).  Over 4900 launches of 16 to
// 1792 row blocks and 8 to 224 groups, against four, eight and sixteen waves from 8, 24 and 64 groups and the largest batch of 4, 2 and 1 that
// divides them: 1.08 times faster at 1 and 2 tokens, 1.10 at 4, 1.07 at 8, 1.07 at 9 and 1.14 at 16 in 4 bits, as much in 3; 1 % of
// the launches are more than 3 % slower.  us, 1 token: 4096 x 4096 4.3 and 4.2, 3584 x 9216 7.1 and 6.4, 9216 x 3584 6.4 and 6.2;
// 4 tokens 3584 x 9216 7.4 and 6.4.
struct GemvShape {
    int waves, unroll;
};
GemvShape gemv_shape(int M, int row_blocks, int G)
{
    GemvShape s;
    if (M > 12) s.waves = row_blocks <= 256 ? 8 : 4;
    else s.waves = row_blocks <= 256 ? 16 : row_blocks <= (M == 3 || M == 4 ? 800 : 512) ? 8 : 4;
    while (s.waves > 4 && G < s.waves) s.waves /= 2;
    s.unroll = M <= 2 && G % 2 == 0 && 5 * G >= 6 * s.waves ? 2 : 1;
    const int waves = awq_knob("AWQ_GEMV_WAVES", 0), unroll = awq_knob("AWQ_GEMV_UNROLL", 0);
    if (waves == 1 || waves == 2 || waves == 4 || waves == 8 || waves == 16) s.waves = waves;
    if (unroll == 1 || (unroll == 2 && G % 2 == 0 && M <= 2)) s.unroll = unroll;
    return s;
}

}  // namespace

namespace {

// one instantiation: raises its dynamic-LDS limit once if the launch needs more than 64 KB
template <int BITS, int U, int MS, bool PIPE>
int gemv_launch_one(dim3 grid, dim3 block, size_t lds, hipStream_t stream, const half_t *x,
                    const uint32_t *qweight, const uint16_t *scales, const uint8_t *zeros, half_t *y, int M,
                    int N, int K, int G, int logW, const half_t *res)
{
    static AwqOncePerDevice once;
    std::atomic<bool> &raised = once.here();
    if (lds > 64 * 1024 && !raised.load(std::memory_order_relaxed)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(gemv_kernel<BITS, U, MS, PIPE>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
            return AWQ_ERR_HIP;
        raised.store(true, std::memory_order_relaxed);
    }
    gemv_kernel<BITS, U, MS, PIPE><<<grid, block, lds, stream>>>(x, qweight, scales, zeros, y, M, N, K, G, logW, res);
    return awq_launch_status();
}

template <int BITS>
int gemv_launch_bits(const void *x, const void *qweight, const void *scales, const void *zeros,
                     void *y, int M, int N, int K, hipStream_t stream, const void *res = nullptr)
{
    const int G = K / AWQ_GROUP;
    const GemvShape shape = gemv_shape(M, N / 16, G);
    const int W = shape.waves, U = shape.unroll, logW = __builtin_ctz(W);
    // every decode M stages its activations through LDS: 2, 4, 8 or 16 rows per wave.  A load covers 4 / U rows: fewer staged rows
    // than that would be a store under a mask, and the compiler then moves the load down to it, behind the weights (1 token, 3584 x
    // 9216, two groups per batch: 7.4 us, with two rows 6.4)
    const int MS = U == 2 ? 2 : M <= 4 ? 4 : M <= 8 ? 8 : 16;
    const dim3 grid(N / 16), block(W * 64);
    const bool pipe = (G / U + W - 1) / W > 1;      // some wave has more than one batch
    // reduction area: 16*M outputs x 16 wave slots x 4 bytes, after the staging areas
    // (a lane parks four token rows at once: the area covers M rounded up to a multiple of 4)
    const size_t lds = (size_t)((M + 3) / 4 * 4) * 1024 + (size_t)W * MS * (U * 256 + 16);
    if (lds > (size_t)160 * 1024) return AWQ_ERR_BAD_SHAPE;
#define AWQ_GEMV_LAUNCH(UU, MM, PP)                                                                   \
    return gemv_launch_one<BITS, UU, MM, PP>(grid, block, lds, stream, (const half_t *)x,             \
                                             (const uint32_t *)qweight, (const uint16_t *)scales,     \
                                             (const uint8_t *)zeros, (half_t *)y, M, N, K, G, logW,   \
                                             (const half_t *)res)
    if (U == 2 && pipe) AWQ_GEMV_LAUNCH(2, 2, true);
    if (U == 2) AWQ_GEMV_LAUNCH(2, 2, false);
    switch (MS) {
    case 4: if (pipe) AWQ_GEMV_LAUNCH(1, 4, true); AWQ_GEMV_LAUNCH(1, 4, false);
    case 8: if (pipe) AWQ_GEMV_LAUNCH(1, 8, true); AWQ_GEMV_LAUNCH(1, 8, false);
    default: if (pipe) AWQ_GEMV_LAUNCH(1, 16, true); AWQ_GEMV_LAUNCH(1, 16, false);
    }
#undef AWQ_GEMV_LAUNCH
}

}  // namespace

// Host side of the decode path; arguments were validated by awq_w4a16_linear / awq_w3a16_linear.
int awq_gemv_launch(const void *x, const void *qweight, const void *scales, const void *zeros,
                    void *y, int M, int N, int K, hipStream_t stream)
{
    return gemv_launch_bits<4>(x, qweight, scales, zeros, y, M, N, K, stream);
}

int awq_gemv_launch_w3(const void *x, const void *qweight, const void *scales, const void *zeros,
                       void *y, int M, int N, int K, hipStream_t stream)
{
    return gemv_launch_bits<3>(x, qweight, scales, zeros, y, M, N, K, stream);
}

// the 4-bit decode launch with a residual [M,N] (may be y) added to the output
int awq_gemv_launch_residual(const void *x, const void *qweight, const void *scales, const void *zeros,
                             void *y, const void *res, int M, int N, int K, hipStream_t stream)
{
    return gemv_launch_bits<4>(x, qweight, scales, zeros, y, M, N, K, stream, res);
}

// Linears with the longest rows first: their workgroups run longest.
int awq_gemv_group_launch(int bits, const GemvProblem *p, int count, int M, hipStream_t stream)
{
    if (count < 1 || count > GEMV_GROUP_MAX) return AWQ_ERR_BAD_ARGUMENT;
    GemvGroupArgs A = {};
    int order[GEMV_GROUP_MAX];
    for (int i = 0; i < count; ++i) order[i] = i;
    std::stable_sort(order, order + count, [&](int a, int b) { return p[a].K > p[b].K; });
    int64_t total = 0;
    for (int i = 0; i < count; ++i) {
        A.p[i] = p[order[i]];
        A.first[i] = (int)total;
        total += A.p[i].N / 16;
    }
    if (total > (1 << 30)) return AWQ_ERR_BAD_SHAPE;
    A.count = count;
    A.M = M;
    return bits == 4 ? gemv_group_bits<4>(A, (int)total, stream) : gemv_group_bits<3>(A, (int)total, stream);
}

// us, from the row blocks, the weight tiles (16 x 128) and the batches of the longest row and of all rows.  Fitted to 16000 launches of one
// to seven linears of 256 to 32768 features and 256 to 28672 columns: 6 to 7 % rms.
double awq_gemv_group_us(int bits, const GemvProblem *p, int count, int M)
{
    double blocks = 0.0, tiles = 0.0, batches = 0.0, longest = 0.0;
    for (int i = 0; i < count; ++i) {
        const int rb = p[i].N / 16, G = p[i].K / AWQ_GROUP, per = ((G + 7) / 8 + GROUP_U - 1) / GROUP_U;
        blocks += rb;
        tiles += (double)rb * G;
        batches += (double)rb * per;
        longest = std::max(longest, (double)per);
    }
    static const double fit[2][3][5] = {{{2.116, 0.064, 0.162, 0.443, 0.608}, {2.173, 0.300, 0.209, 0.468, 0.409}, {2.207, 0.446, 0.257, 0.657, 0.373}},
                                        {{2.111, 0.058, 0.168, 0.434, 0.772}, {2.203, 0.272, 0.225, 0.456, 0.506}, {2.311, 0.450, 0.282, 0.666, 0.402}}};
    const double *c = fit[bits == 4][M <= 4 ? 0 : M <= 8 ? 1 : 2];
    return c[0] + c[1] * blocks / 256.0 + c[2] * tiles / 1000.0 + c[3] * longest + c[4] * batches / 1000.0;
}

// us of the launch of one linear at five tokens and more: tiles that a wave walks (rounds of workgroups, as the LDS admits them), and all
// tiles.  2900 launches in 4 bits, 2100 in 3: 5 to 9 % rms.
double awq_gemv_us(int bits, int M, int N, int K)
{
    const int G = K / AWQ_GROUP;
    const GemvShape shape = gemv_shape(M, N / 16, G);
    const int W = shape.waves, MS = M <= 8 ? 8 : 16;
    const int lds = (M + 3) / 4 * 4 * 1024 + W * MS * 272;
    const int resident = std::max(1, std::min(160 * 1024 / lds, 16 / W));
    const double rounds = (double)((N / 16 + 256 * resident - 1) / (256 * resident)), walk = rounds * ((G + W - 1) / W);
    const double tiles = (double)(N / 16) * G / 1000.0;
    if (M <= 8) return bits == 4 ? 2.42 + 0.338 * walk + 0.201 * tiles : 2.44 + 0.343 * walk + 0.166 * tiles;
    if (M <= 12) return bits == 4 ? 2.45 + 0.492 * walk + 0.232 * tiles : 2.54 + 0.468 * walk + 0.198 * tiles;
    return bits == 4 ? 0.23 + 2.27 * rounds + 0.358 * walk + 0.244 * tiles : 0.48 + 2.04 * rounds + 0.366 * walk + 0.207 * tiles;
}
