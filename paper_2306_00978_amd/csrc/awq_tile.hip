// K-split tile kernel for gfx950: one linear at more than 16 tokens, 4- or 3-bit (group 128) or 2-bit
// (group 64) weights.
//
// AWQ Sec. 4.2: dequantization fused into the matrix kernel.
//
// Mapping.  A workgroup of eight waves computes a tile of 16 MT tokens x 16 NT out-features; its
// waves divide K (whole runs of 128 columns) and add their tiles through LDS at the end, in a fixed order.
// Every wave thus needs its own columns of x and its own weight tiles only: nothing is shared
// during the loop, there is no barrier in it, each weight is fetched and expanded once per
// 16 MT tokens, and both operands go from memory to registers in the layout of
// v_mfma_f32_16x16x32_f16 -- the packed weight tile is the B operand, and lane (r, c) of the A operand of step
// j takes the 16 bytes at row r, column 32 j + 8 c of the run.
//
// Arithmetic.  A code becomes (q - z) 2^-9 in fp16, exactly (the masked codes are fp16 subnormals; one fused multiply-add
// scales them and subtracts the zero point); the products of a group are summed in fp32 by the matrix core and the group's
// step, times 2^9, is applied to the sum, in fp32, with one FMA per output.  No dequantized weight is rounded.
// The vector instructions are chosen by what they cost with two waves to a SIMD (measured): 2.3 cycles for and, or, shift,
// add and fp32 multiply-adds, 4.4 for v_and_or, packed fp16 and mixed-precision ones.  So a pair of codes costs 6.7 cycles where
// v_and_or and a packed subtraction cost 9.1, and the steps are converted to fp32 once instead of 20 times.
//
// Pipeline.  Per run of 128 columns a wave expands NT weight tiles (4 steps x NT fragments in
// registers), then walks its MT token tiles: 4 NT MFMAs and 4 NT FMAs (8 NT for two groups of 64) per
// token tile.  Memory -> LDS loads (no staging registers) bring the next three token tiles and the
// packed words, steps and zero points of the next run into areas that belong to the wave; one load
// instruction takes four rows of 256 contiguous bytes of x, the 16-byte chunk k of row i landing at place
// k ^ i, so that the fragment reads of 16 rows hit 16 different bank groups.  (Fragments
// loaded from memory directly -- 64 pieces of 16 bytes per instruction -- ran at 14 B/clk per CU: 4 us per
// token tile at K = 4096.)  The loads complete in order and are counted by hand.
//
// What bounds it (11008 x 4096 at 77 tokens, time stamps, 25 thousand cycles): the token tiles, 11 thousand, where the two waves
// of a SIMD share its matrix pipe; the expansions, 4.7 thousand, which both do at the same time; 4.6 thousand until the first
// words are there; waiting for the last wave and the exchange, 4.9 thousand.  Loading alone (62 B/clk per CU) would take
// 12 thousand.  Started later, or with a raised priority throughout, one wave of a SIMD does not leave the other's
// step; expanding the next run beside the MFMAs of this one takes 32 more registers per weight tile and was slower at every
// shape (13.0 -> 14.8 us for 8192 x 4096 at 77 tokens).
#include "awq_common.h"
#include "awq_gemv_stream.h"
#include "awq_tile.h"

#include <algorithm>

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int TILE_WAVES = 8;
constexpr int RUN = 128;                        // columns per step of the loop

constexpr int TILE_RING = 3;                    // token tiles of x a wave has in LDS
constexpr int UNIT_BYTES = 16 * RUN * 2;
// a wave's LDS: the ring, then packed words, steps and zero points (a dword per row and tile) of one run
constexpr int RAW_OFS = TILE_RING * UNIT_BYTES;
constexpr int sc_ofs(int nt) { return RAW_OFS + nt * 1024; }
constexpr int zp_ofs(int nt) { return sc_ofs(nt) + 256; }
constexpr int wave_lds(int nt) { return zp_ofs(nt) + 256; }
// The final exchange: a 16 x 16 tile takes 320 floats, row 4 c + v at 80 c + 16 v (the rows of a write fall 16 banks
// apart); token tiles whose partial sums are in LDS at once
constexpr int EXCHANGE_TILE = 320;
constexpr int tile_pass(int mt, int nt)
{
    const int fit = 16 / nt, passes = (mt + fit - 1) / fit;
    return (mt + passes - 1) / passes;
}
constexpr int tile_lds(int mt, int nt)
{
    const int exchange = TILE_WAVES * tile_pass(mt, nt) * nt * EXCHANGE_TILE * 4, loop = TILE_WAVES * wave_lds(nt);
    return exchange > loop ? exchange : loop;
}

typedef __attribute__((address_space(3))) void lds_void_t;
typedef const __attribute__((address_space(1))) void gbl_void_t;

template <int BYTES>
__device__ __forceinline__ void dma(const unsigned char *g, uint32_t lds_addr)
{
    gbl_void_t *src = (gbl_void_t *)(uintptr_t)g;
    lds_void_t *dst = (lds_void_t *)(uintptr_t)lds_addr;       // + 16 (4 for the small ones) x lane
    if constexpr (BYTES == 16) __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 0);
    else if constexpr (BYTES == 4) __builtin_amdgcn_global_load_lds(src, dst, 4, 0, 0);
    else if constexpr (BYTES == 2) __builtin_amdgcn_global_load_lds(src, dst, 2, 0, 0);
    else __builtin_amdgcn_global_load_lds(src, dst, 1, 0, 0);
}

// LDS reads as asm, so that the compiler does not tie them to the loads in flight; each is waited for
// by an lgkmcnt wait that names its result
__device__ __forceinline__ u32x4 lds_read16(uint32_t addr)
{
    u32x4 v;
    asm volatile("ds_read_b128 %0, %1" : "=v"(v) : "v"(addr));
    return v;
}
__device__ __forceinline__ uint32_t lds_read4(uint32_t addr)
{
    uint32_t v;
    asm volatile("ds_read_b32 %0, %1" : "=v"(v) : "v"(addr));
    return v;
}
template <int N>
__device__ __forceinline__ void wait_loads()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Codes of up to four bits in bits 0 .. 9 of the halves of a dword are fp16 subnormals, multiples of 2^-24.  With f a power of
// two that brings them to multiples of 2^-9 and nz = -z 2^-9 in both halves, (q - z) 2^-9, exactly.
__device__ __forceinline__ uint32_t centred(uint32_t codes, uint32_t f, uint32_t nz)
{
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(__builtin_bit_cast(half2_t, codes), __builtin_bit_cast(half2_t, f),
                                                                  __builtin_bit_cast(half2_t, nz)));
}
__device__ __forceinline__ constexpr uint32_t half_pair(int exponent) { return (uint32_t)(exponent + 15) * 0x04000400u; }   // 2^exponent twice
// -z 2^-9 in both halves, z in the low bits (up to four) of a dword
__device__ __forceinline__ uint32_t negated_zero(uint32_t z)
{
    const half2_t minus = __builtin_bit_cast(half2_t, half_pair(15) | 0x80008000u);
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, z * 0x00010001u) * minus);
}

// a / b by the inverse floor((2^32 - 1) / b), which gives one too little at most: a division by an argument is 150 cycles in
// front of the first load
__device__ __forceinline__ int quotient(int a, int b, uint32_t inverse)
{
    const int q = (int)(((uint64_t)(uint32_t)a * inverse) >> 32);
    return a - q * b >= b ? q + 1 : q;
}

// TILE_LOSS (the scale search, 4-bit): the tiles of several grid points follow each other; point i has its operands i `step` bytes
// and its sums loss_step further.  TILE_FEW: several linears at up to 16 tokens.  (Forms, not arguments: with `loss` tested at
// run time a 4-bit prompt's workgroup of 80 x 48 has 1268 instructions, 228 in front of its first request, without 1067 and 185; 77 tokens
// through 11008 x 4096 0.3 to 0.7 %.)
enum TileForm { TILE_PLAIN, TILE_LOSS, TILE_FEW };
template <TileForm FORM>
struct TilePoints {};
template <>
struct TilePoints<TILE_LOSS> {
    double *loss;
    int tiles;                     // of a point
    uint32_t tiles_inverse;
    int64_t step, loss_step;
};

// The tile (tile_m, tile_n) of one product; `unit` is the workgroup's number among those that read the same x.
template <int BITS, int MT, int NT, TileForm FORM>
__device__ __forceinline__ void tile_work(
    const unsigned char *__restrict__ x, const unsigned char *__restrict__ qweight,
    const unsigned char *__restrict__ scales, const unsigned char *__restrict__ zeros,
    half_t *__restrict__ y, int M, int N, int K, int tile_m, int tile_n, int unit, uint32_t runs_inverse,
    uint32_t runs_inverse_long, double *__restrict__ loss, unsigned char *smem)
{
    const uint32_t lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t r = lane & 15, c = lane >> 4;
    const int G = K / RUN;
    // The wave's runs: wave, wave + 8, ..., walked in cyclic order from a start of the workgroup's own, one run after its
    // neighbour's (unit % cnt): the workgroups of a token tile then read a run of x one step after the other, while the L2
    // has it.  Spread over all of K they read it at any time, and where the token tiles of an XCD are more than its 4 MB
    // each brings it in again (1024 x 28672 at 700 tokens 95 us, so 69; 256 x 28672 at 960 58 and 37).
    const int cnt = (G - wave + TILE_WAVES - 1) / TILE_WAVES;
    const int rot = cnt > 0 ? unit - cnt * quotient(unit, cnt, wave < G % TILE_WAVES ? runs_inverse_long : runs_inverse) : 0;
    auto run_at = [&](int i) {                             // i-th run; past the end: a harmless repeat
        i = min(i, cnt - 1) + rot;
        return wave + TILE_WAVES * (i < cnt ? i : i - cnt);
    };
    const int m0 = tile_m * (16 * MT), nt0 = tile_n * NT;

    // A token tile that would reach past M is moved back to end there (more than one: M >= 16); the rows it shares with
    // its neighbour are computed twice, bit for bit alike, and stored once.
    // (TILE_FEW, one token tile: rows past the end repeat the last one in LDS, and are not stored)
    auto first_row = [&](int m) { return FORM == TILE_FEW ? 0 : min(m0 + 16 * m, M - 16); };
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem) + wave * wave_lds(NT);
    // packed words: tile n of the workgroup, wave-uniform; steps and zero points: one load for all tiles, lane
    // (r, c) fetching those of row r of tile c.  Ragged N repeats the last tile.  Counted in runs: K % 256 == 0
    // for the 2-bit layout, so G is even and a tile's first run starts a block.
    size_t trun[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) trun[n] = (size_t)min(nt0 + n, (N >> 4) - 1) * G;
    const size_t lrun = (size_t)min(nt0 + min((int)c, NT - 1), (N >> 4) - 1) * G;

    floatx4 tot[MT][NT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int n = 0; n < NT; ++n) tot[m][n] = floatx4{0.f, 0.f, 0.f, 0.f};

    // x: load i (0..3) of a token tile takes its rows 4 i + c, lane r the chunk that belongs at place r
    uint32_t xofs[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
        xofs[i] = (FORM == TILE_FEW ? min(4 * i + c, (uint32_t)(M - 1)) : 4 * i + c) * (uint32_t)(K * 2) + 16 * (r ^ (4 * i + c));
    auto issue_x = [&](int run, int m, uint32_t slot) {
        const unsigned char *p = x + ((size_t)first_row(m) * K + (size_t)run * RUN) * 2;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            asm volatile("" : "+v"(xofs[i]));              // a 32-bit offset beside a wave-uniform base, not a 64-bit address
            dma<16>(p + xofs[i], lds0 + slot + i * 1024);
        }
    };
    constexpr int RAW_LOADS = NT + 2;
    auto issue_raw = [&](int run) {
        if (BITS != 2) {                                   // a run is a group: 1 KB (768 bytes), 16 steps, 8 bytes of zero points
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                if (BITS == 4) dma<16>(qweight + (trun[n] + run) * 1024 + lane * 16, lds0 + RAW_OFS + n * 1024);
                else if (lane < 48) dma<16>(qweight + (trun[n] + run) * 768 + lane * 16, lds0 + RAW_OFS + n * 1024);
            }
            dma<2>(scales + (lrun + run) * 32 + r * 2, lds0 + sc_ofs(NT));
            dma<1>(zeros + (lrun + run) * 8 + (r >> 1), lds0 + zp_ofs(NT));
        } else {                                           // half a block of 256 columns: groups 2 (run % 2), + 1
#pragma unroll
            for (int n = 0; n < NT; ++n)
                dma<16>(qweight + ((trun[n] + run) >> 1) * 1024 + lane * 16, lds0 + RAW_OFS + n * 1024);
            dma<4>(scales + ((lrun + run) >> 1) * 128 + (run & 1) * 4 + r * 8, lds0 + sc_ofs(NT));
            dma<1>(zeros + ((lrun + run) >> 1) * 16 + r, lds0 + zp_ofs(NT));
        }
    };
    uint32_t frag[4];                                      // of this lane inside a token tile
#pragma unroll
    for (int j = 0; j < 4; ++j) frag[j] = lds0 + r * 256 + (((4 * j + c) ^ r) * 16);

    if (cnt > 0) {
        issue_raw(run_at(0));
        issue_x(run_at(0), 0, 0);
        issue_x(run_at(1 / MT), 1 % MT, UNIT_BYTES);
        issue_x(run_at(2 / MT), 2 % MT, 2 * UNIT_BYTES);
        uint32_t slot = 0;                                 // of the token tile being multiplied
        uint32_t a[4][4];
        // Counting: behind a token tile that is waited for, the two after it have been requested (8 loads)
        // and, if it was itself requested before the run's weights, those as well.  A smaller count only waits longer.
        for (int i = 0; i < cnt; ++i) {
            wait_loads<(MT >= 2 ? 8 : 4)>();               // this run's packed words: 4 MT loads behind them
            u32x4 q[NT];
            uint32_t sraw[NT], zraw[NT], q3[NT][3];
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                if (BITS != 3) {
                    q[n] = lds_read16(lds0 + RAW_OFS + n * 1024 + lane * 16);
                } else {                                   // 12-byte slots
#pragma unroll
                    for (int i = 0; i < 3; ++i) q3[n][i] = lds_read4(lds0 + RAW_OFS + n * 1024 + lane * 12 + 4 * i);
                }
                sraw[n] = lds_read4(lds0 + sc_ofs(NT) + (16 * n + r) * 4);
                zraw[n] = lds_read4(lds0 + zp_ofs(NT) + (16 * n + r) * 4);
            }
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                if (BITS != 3) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(q[n]), "+v"(sraw[n]), "+v"(zraw[n]));
                else asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(q3[n][0]), "+v"(q3[n][1]), "+v"(q3[n][2]), "+v"(sraw[n]), "+v"(zraw[n]));
            }
            issue_raw(run_at(i + 1));
            if (i == 0) {
                wait_loads<8 + RAW_LOADS>();
                u32x4 a0[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) a0[j] = lds_read16(frag[j]);
                asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a0[0]), "+v"(a0[1]), "+v"(a0[2]), "+v"(a0[3]));
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[j][e] = a0[j][e];
            }
            half8_t bf[NT][4];
            float s0[NT], s1[NT];
            __builtin_amdgcn_s_setprio(1);                 // (1 to 4 %: a wave that expands lets the other's MFMAs wait, not itself)
            const int hb = run_at(i) & 1;
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                if (BITS == 3) {
                    // pair 5 i + f of word i at bits 3 f; pair 15 in the top bits of the three words
                    const uint32_t nz = negated_zero((zraw[n] >> ((r & 1) * 4)) & 0xFu);
                    s0[n] = s1[n] = (float)__builtin_bit_cast(half_t, (uint16_t)sraw[n]) * 512.0f;
                    uint32_t pr[16];
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const uint32_t w = q3[n][i], w9 = w >> 9;
#pragma unroll
                        for (int f = 0; f < 5; ++f)
                            pr[5 * i + f] = centred((f < 3 ? w : w9) & (0x00070007u << (3 * (f % 3))), half_pair(15 - 3 * (f % 3)), nz);
                    }
                    const uint32_t top = ((q3[n][0] >> 15) & 0x00010001u) | ((q3[n][1] >> 14) & 0x00020002u) |
                                         ((q3[n][2] >> 13) & 0x00040004u);
                    pr[15] = centred(top, half_pair(15), nz);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        bf[n][j] = __builtin_bit_cast(half8_t, u32x4{pr[4 * j], pr[4 * j + 1], pr[4 * j + 2], pr[4 * j + 3]});
                } else if (BITS == 4) {
                    const uint32_t nz = negated_zero((zraw[n] >> ((r & 1) * 4)) & 0xFu);
                    s0[n] = s1[n] = (float)__builtin_bit_cast(half_t, (uint16_t)sraw[n]) * 512.0f;
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const uint32_t w = q[n][j], w8 = w >> 8;
                        bf[n][j] = __builtin_bit_cast(half8_t, u32x4{
                            centred(w & 0x000F000Fu, half_pair(15), nz), centred(w & 0x00F000F0u, half_pair(11), nz),
                            centred(w8 & 0x000F000Fu, half_pair(15), nz), centred(w8 & 0x00F000F0u, half_pair(11), nz)});
                    }
                } else {
                    // groups t = 2 hb, 2 hb + 1 of the block: codes at bits 2t of a half
                    const half2_t ss = __builtin_bit_cast(half2_t, sraw[n]);
                    s0[n] = (float)ss[0] * 512.0f;
                    s1[n] = (float)ss[1] * 512.0f;
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const uint32_t mk = 0x00030003u << (4 * hb + 2 * t), f = half_pair(15 - 4 * hb - 2 * t);
                        const uint32_t nz = negated_zero((zraw[n] >> (4 * hb + 2 * t)) & 3u);
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            bf[n][2 * t + j] = __builtin_bit_cast(half8_t, u32x4{
                                centred((q[n][0] >> (8 * j)) & mk, f, nz), centred((q[n][1] >> (8 * j)) & mk, f, nz),
                                centred((q[n][2] >> (8 * j)) & mk, f, nz), centred((q[n][3] >> (8 * j)) & mk, f, nz)});
                    }
                }
                // (steps in fp32 registers: left to itself the compiler multiplies with the fp16 step, at half the rate)
                asm("" : "+v"(s0[n]), "+v"(s1[n]));
            }
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                // the token tile in registers frees its place in the ring: request the third after it
                issue_x(run_at(i + (m + 3) / MT), (m + 3) % MT, slot);
                const uint32_t next = slot == 2 * UNIT_BYTES ? 0 : slot + UNIT_BYTES;
                if (m < 2) wait_loads<8 + RAW_LOADS>();
                else wait_loads<8>();
                u32x4 an[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) an[j] = lds_read16(frag[j] + next);
                __builtin_amdgcn_sched_barrier(0);
                floatx4 acc[NT];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const half8_t av = __builtin_bit_cast(half8_t, u32x4{a[j][0], a[j][1], a[j][2], a[j][3]});
#pragma unroll
                    for (int n = 0; n < NT; ++n) {
                        if (j == 0 || (BITS == 2 && j == 2)) acc[n] = floatx4{0.f, 0.f, 0.f, 0.f};
                        acc[n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, bf[n][j], acc[n], 0, 0, 0);
                    }
                    if (j == 3 || (BITS == 2 && j == 1)) {
#pragma unroll
                        for (int n = 0; n < NT; ++n)
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                tot[m][n][v] = __builtin_fmaf(acc[n][v], j == 3 ? s1[n] : s0[n], tot[m][n][v]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);         // the wait stays behind the multiplications
                asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(an[0]), "+v"(an[1]), "+v"(an[2]), "+v"(an[3]));
                // (dwords, not vectors: those the compiler copies with v_mov_b64, which one token tile cannot hide: 43 tokens through
                // 1616 x 9472 8.9 us and 9.4 so)
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) a[j][e] = an[j][e];
                slot = next;
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        wait_loads<0>();                                   // the harmless repeats
    }
    __syncthreads();                                       // the exchange below reuses every wave's LDS

    // Sum over the waves.  Lane (r, c) holds rows 4 c + v, column r of each 16 x 16 tile.  All tiles that fit at once: in passes
    // of three token tiles, each with a nearly empty second round of lanes, this took 3.8 thousand cycles at (5, 3), now 2.8.
    constexpr int MC = tile_pass(MT, NT), TILES = MC * NT;
    // TILE_LOSS: nothing is stored, y holds the layer's reference outputs, and loss[workgroup] becomes the sum of the squared
    // differences of the outputs, rounded to fp16, to them: four squared and added in fp32, the rest in fp64, in a fixed order.
    float *lds = reinterpret_cast<float *>(smem);
    double diff = 0.0;
    float *mine = lds + wave * (TILES * EXCHANGE_TILE) + 80 * c + r;
#pragma unroll
    for (int p = 0; p < MT; p += MC) {
        if (p > 0) __syncthreads();
#pragma unroll
        for (int i = 0; i < MC; ++i)
            if (p + i < MT) {
#pragma unroll
                for (int n = 0; n < NT; ++n)
#pragma unroll
                    for (int v = 0; v < 4; ++v)
                        mine[(i * NT + n) * EXCHANGE_TILE + 16 * v] = tot[p + i < MT ? p + i : 0][n][v];
            }
        __syncthreads();
        // a wave adds whole tiles, a lane four columns of a row
#pragma unroll
        for (int t0 = 0; t0 < TILES; t0 += TILE_WAVES) {
            const int t = t0 + wave, i = t / NT;
            const int row = lane >> 2, col = ((t - i * NT) * 4 + (lane & 3)) * 4;
            const int mt = p + i, m = first_row(mt) + row, n = nt0 * 16 + col;
            if (t >= TILES || mt >= MT || m < m0 + 16 * mt || m >= M || n >= N) continue;
            const float *src = lds + t * EXCHANGE_TILE + 80 * (row >> 2) + 16 * (row & 3) + 4 * (lane & 3);
            float4 s = *reinterpret_cast<const float4 *>(src);
#pragma unroll
            for (int w = 1; w < TILE_WAVES; ++w) {
                const float4 b = *reinterpret_cast<const float4 *>(src + w * (TILES * EXCHANGE_TILE));
                s.x += b.x; s.y += b.y; s.z += b.z; s.w += b.w;
            }
            const half2_t lo = {(half_t)s.x, (half_t)s.y}, hi = {(half_t)s.z, (half_t)s.w};
            if constexpr (FORM == TILE_LOSS) {
                const uint2 ref = *reinterpret_cast<const uint2 *>(y + (size_t)m * N + n);
                const half2_t rlo = __builtin_bit_cast(half2_t, ref.x), rhi = __builtin_bit_cast(half2_t, ref.y);
                const float d0 = (float)lo[0] - (float)rlo[0], d1 = (float)lo[1] - (float)rlo[1];
                const float d2 = (float)hi[0] - (float)rhi[0], d3 = (float)hi[1] - (float)rhi[1];
                diff += (double)(d0 * d0 + d1 * d1 + d2 * d2 + d3 * d3);
            } else {
                *reinterpret_cast<uint2 *>(y + (size_t)m * N + n) =
                    make_uint2(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi));
            }
        }
    }
    if constexpr (FORM == TILE_LOSS) {
#pragma unroll
        for (int d = 1; d <= 32; d <<= 1) diff += __shfl_xor(diff, d);
        __syncthreads();                                   // the last pass has been read
        double *red = reinterpret_cast<double *>(smem);
        if (lane == 0) red[wave] = diff;
        __syncthreads();
        if (threadIdx.x == 0) {
            double sum = red[0];
            for (int w = 1; w < TILE_WAVES; ++w) sum += red[w];
            loss[unit] = sum;
        }
    }
}

struct TileGroupArgs {
    GemvProblem p[GEMV_GROUP_MAX];
    int first[GEMV_GROUP_MAX];                     // workgroup of each
    uint32_t inverse[GEMV_GROUP_MAX][2];
    int count, M;
};

template <int BITS, int MT, int NT, TileForm FORM>
__global__ __launch_bounds__(64 * TILE_WAVES, 1) void tile_kernel(
    const unsigned char *__restrict__ x, const unsigned char *__restrict__ qweight,
    const unsigned char *__restrict__ scales, const unsigned char *__restrict__ zeros,
    half_t *__restrict__ y, int M, int N, int K, int tiles_n, uint32_t tiles_n_inverse, uint32_t runs_inverse,
    uint32_t runs_inverse_long, int tiles_total, const TilePoints<FORM> points)
{
    extern __shared__ __align__(16) unsigned char smem[];
    asm volatile("" ::"s"(x), "s"(qweight), "s"(scales), "s"(zeros), "s"(y), "s"(M), "s"(N), "s"(K), "s"(tiles_n),
                 "s"(tiles_n_inverse), "s"(runs_inverse), "s"(runs_inverse_long), "s"(tiles_total));   // arguments in one round
    // contiguous ranges of tiles, token-tile-major, per XCD (own L2): see gemm_kernel
    const int per_xcd = (tiles_total + 7) >> 3;
    int unit = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    if (unit >= tiles_total || ((int)blockIdx.x >> 3) >= per_xcd) return;
    double *loss = nullptr;
    if constexpr (FORM == TILE_LOSS) {
        const int point = quotient(unit, points.tiles, points.tiles_inverse);
        unit -= point * points.tiles;
        x += point * points.step;
        qweight += point * points.step;
        scales += point * points.step;
        zeros += point * points.step;
        loss = points.loss + point * points.loss_step;
    }
    const int tile_m = quotient(unit, tiles_n, tiles_n_inverse), tile_n = unit - tile_m * tiles_n;
    tile_work<BITS, MT, NT, FORM>(x, qweight, scales, zeros, y, M, N, K, tile_m, tile_n, unit, runs_inverse, runs_inverse_long, loss, smem);
}

// Several linears at up to 16 tokens in one launch: workgroup b of a linear takes its weight tiles NT b .. + NT - 1.  A token tile
// costs the same whether it has five rows or sixteen, and a weight is expanded once for all of them, so this takes what lies between the small
// launches of the batch kernel and the large ones that stream at the memory's rate (awq_linear.hip).  A layer of seven linears at 9 / 16
// tokens, us, before and now: hidden size 1536 (4608) in 4 bits 11.3 / 11.5 and 7.8 / 8.1, 2304 (7680) 16.6 / 16.9 and 13.1 / 15.1; 4096 (11008) in
// 3 bits 30.0 / 32.5 and 25.6 / 27.8, in 2 bits 28.2 / 32.6 and 23.8 / 25.8.  One linear of 11008 x 4096 in 4 bits 10.9 / 15.8 and 8.1 / 9.0.
template <int BITS, int NT>
__global__ __launch_bounds__(64 * TILE_WAVES, 1) void tile_group_kernel(const TileGroupArgs A)
{
    extern __shared__ __align__(16) unsigned char smem[];
    int i = 0;
#pragma unroll
    for (int n = 1; n < GEMV_GROUP_MAX; ++n)
        if (n < A.count && (int)blockIdx.x >= A.first[n]) i = n;
    const GemvProblem &P = A.p[i];
    const int tile_n = (int)blockIdx.x - A.first[i];
    tile_work<BITS, 1, NT, TILE_FEW>((const unsigned char *)P.x, (const unsigned char *)P.q, (const unsigned char *)P.sc, (const unsigned char *)P.zp,
                           (half_t *)P.y, A.M, P.N, P.K, 0, tile_n, tile_n, A.inverse[i][0], A.inverse[i][1], nullptr, smem);
}

template <int BITS, int NT>
int launch_group(const TileGroupArgs &A, int total, hipStream_t stream)
{
    constexpr int lds = tile_lds(1, NT);
    static AwqOncePerDevice once;
    std::atomic<bool> &attr_set = once.here();
    if (lds > 64 * 1024 && !attr_set.load(std::memory_order_relaxed)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(tile_group_kernel<BITS, NT>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
            return AWQ_ERR_HIP;
        attr_set.store(true, std::memory_order_relaxed);
    }
    tile_group_kernel<BITS, NT><<<dim3((unsigned)total), dim3(64 * TILE_WAVES), lds, stream>>>(A);
    return awq_launch_status();
}

// (loss, count, step, loss_step: TILE_LOSS)
template <int BITS, int MT, int NT, TileForm FORM>
int launch_one(const void *x, const void *qweight, const void *scales, const void *zeros, void *y, int M, int N,
               int K, double *loss, int count, size_t step, size_t loss_step, hipStream_t stream)
{
    const int tiles_n = (N / 16 + NT - 1) / NT;
    const int64_t tiles = awq_tile_count({MT, NT, 0.0}, M, N), total = tiles * count;
    if (total > (1 << 30)) return AWQ_ERR_BAD_SHAPE;
    constexpr int lds = tile_lds(MT, NT);
    static_assert(lds <= 160 * 1024, "LDS of a CU");
    static AwqOncePerDevice once;
    std::atomic<bool> &attr_set = once.here();
    if (lds > 64 * 1024 && !attr_set.load(std::memory_order_relaxed)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(tile_kernel<BITS, MT, NT, FORM>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, lds) != hipSuccess)
            return AWQ_ERR_HIP;
        attr_set.store(true, std::memory_order_relaxed);
    }
    // a wave has G / 8 runs, or one more
    const uint32_t runs = (uint32_t)(K / RUN / TILE_WAVES);
    TilePoints<FORM> points = {};
    if constexpr (FORM == TILE_LOSS) points = {loss, (int)tiles, 0xFFFFFFFFu / (uint32_t)tiles, (int64_t)step, (int64_t)loss_step};
    tile_kernel<BITS, MT, NT, FORM><<<dim3((unsigned)((total + 7) / 8 * 8)), dim3(64 * TILE_WAVES), lds, stream>>>(
        (const unsigned char *)x, (const unsigned char *)qweight, (const unsigned char *)scales,
        (const unsigned char *)zeros, (half_t *)y, M, N, K, tiles_n, 0xFFFFFFFFu / (uint32_t)tiles_n,
        0xFFFFFFFFu / (runs > 0 ? runs : 1u), 0xFFFFFFFFu / (runs + 1), (int)total, points);
    return awq_launch_status();
}

typedef int (*TileFn)(const void *, const void *, const void *, const void *, void *, int, int, int, double *, int, size_t, size_t,
                      hipStream_t);

constexpr int MTS[] = {1, 2, 3, 4, 5, 6, 8};
// 128 x 64 does not fit the registers
constexpr bool tile_built(int mt, int nt) { return !(mt == 8 && nt == 4); }

template <int BITS, int NT, TileForm FORM>
TileFn pick_mt(int mt)
{
    switch (mt) {
    case 1: return launch_one<BITS, 1, NT, FORM>;
    case 2: return launch_one<BITS, 2, NT, FORM>;
    case 3: return launch_one<BITS, 3, NT, FORM>;
    case 4: return launch_one<BITS, 4, NT, FORM>;
    case 5: return launch_one<BITS, 5, NT, FORM>;
    case 6: return launch_one<BITS, 6, NT, FORM>;
    default: return launch_one<BITS, 8, NT == 4 ? 3 : NT, FORM>;      // (8, 4) is never planned
    }
}

template <int BITS, TileForm FORM = TILE_PLAIN>
TileFn pick(int mt, int nt)
{
    return nt == 1 ? pick_mt<BITS, 1, FORM>(mt) : nt == 2 ? pick_mt<BITS, 2, FORM>(mt) : nt == 3 ? pick_mt<BITS, 3, FORM>(mt)
                                                                                                 : pick_mt<BITS, 4, FORM>(mt);
}

}  // namespace

// The estimate, in us, of a launch from a graph, the weights of which no cache holds: 2.9 and, per round of 256 workgroups (one per
// CU: the LDS), 0.75, for every 1024 columns of K (a run of each wave) 0.24 per token tile (32 KB of x per CU: 62 B/clk) and 0.185
// per weight tile (7 % more with four of them: measured, not explained), and 0.113 per pair for the exchange; up to a quarter more
// as the round fills the chip.
// Long K: x comes from the L2 as long as it fits.  Where the rows of one token tile are more than 0.4 of its 4 MB, or those of all
// token tiles that an XCD works on more than 0.75, its part takes longer.
// Fitted to 12300 launches of 2036 shapes (256 to 128256 features, 128 to 32768 columns, 17 to 1600 tokens; of each the shapes of a
// workgroup within a quarter of the fastest): 6 % rms, 9 % above 24576 columns (where it is 32 % off in one of twenty without the
// last two terms).  The shape it picks takes 0.8 % longer than the fastest one on average.
TilePlan awq_tile_plan(int M, int N, int K, int points)
{
    const int forced = awq_tile_override();
    if (forced > 0) return {forced / 10, forced % 10, 0.0};
    TilePlan best = {1, 1, -1.0};
    for (const int mt : MTS)
        for (int nt = 1; nt <= 4; ++nt) {
            if (!tile_built(mt, nt)) continue;
            const int tiles_n = (N / 16 + nt - 1) / nt, tiles_m = (int)(((unsigned)M + 16 * mt - 1) / (16u * mt));
            const int64_t wgs = (int64_t)tiles_n * tiles_m * points;
            const double rounds = (double)((wgs + 255) / 256), full = (double)wgs / (256.0 * rounds);
            const double l2 = mt * (double)K / 131072.0;                            // a token tile's rows, of 4 MB
            double longer = 1.0;
            if (l2 * tiles_m > 0.4) {
                const int xcd = ((int)std::min<int64_t>(wgs, 256) + 7) / 8;         // workgroups of an XCD at a time
                const double l2_all = l2 * std::min((double)tiles_m, 1.0 + (xcd - 1) / (double)tiles_n);
                longer += 0.4 * std::max(l2 - 0.4, 0.0) + 0.25 * std::min(std::max(l2_all - 0.75, 0.0), 1.0);
            }
            const double loop = K / 1024.0 * (0.24 * mt * longer + 0.185 * nt) * (nt == 4 ? 1.07 : 1.0);
            const double us = 2.9 + rounds * (0.75 + loop + 0.113 * mt * nt) * (1.0 + 0.24 * full * full);
            if (best.us < 0.0 || us < best.us) best = {mt, nt, us};
        }
    return best;
}

int64_t awq_tile_count(const TilePlan &plan, int M, int N)
{
    return (int64_t)((N / 16 + plan.nt - 1) / plan.nt) * ((M + 16 * plan.mt - 1) / (16 * plan.mt));
}

int awq_tile_launch(int bits, const TilePlan &plan, const void *x, const void *qweight, const void *scales,
                    const void *zeros, void *y, int M, int N, int K, hipStream_t stream)
{
    const TileFn fn = bits == 4 ? pick<4>(plan.mt, plan.nt) : bits == 3 ? pick<3>(plan.mt, plan.nt) : pick<2>(plan.mt, plan.nt);
    return fn(x, qweight, scales, zeros, y, M, N, K, nullptr, 1, 0, 0, stream);
}

int awq_tile_launch_loss(const TilePlan &plan, const void *x, const void *qweight, const void *scales, const void *zeros,
                         const void *y_ref, int M, int N, int K, double *loss, int points, size_t step, size_t loss_step,
                         hipStream_t stream)
{
    return pick<4, TILE_LOSS>(plan.mt, plan.nt)(x, qweight, scales, zeros, const_cast<void *>(y_ref), M, N, K, loss, points, step,
                                                loss_step, stream);
}

// Linears with the longest rows first: their workgroups run longest.
int awq_tile_group_launch(int bits, int nt, const GemvProblem *p, int count, int M, hipStream_t stream)
{
    if (count < 1 || count > GEMV_GROUP_MAX) return AWQ_ERR_BAD_ARGUMENT;
    TileGroupArgs A = {};
    int order[GEMV_GROUP_MAX];
    for (int i = 0; i < count; ++i) order[i] = i;
    std::stable_sort(order, order + count, [&](int a, int b) { return p[a].K > p[b].K; });
    int64_t total = 0;
    for (int i = 0; i < count; ++i) {
        A.p[i] = p[order[i]];
        A.first[i] = (int)total;
        total += (A.p[i].N / 16 + nt - 1) / nt;
        const uint32_t runs = (uint32_t)(A.p[i].K / RUN / TILE_WAVES);
        A.inverse[i][0] = 0xFFFFFFFFu / (runs > 0 ? runs : 1u);
        A.inverse[i][1] = 0xFFFFFFFFu / (runs + 1);
    }
    if (total > (1 << 30)) return AWQ_ERR_BAD_SHAPE;
    A.count = count;
    A.M = M;
    typedef int (*Fn)(const TileGroupArgs &, int, hipStream_t);
    static const Fn fn[3][4] = {{launch_group<2, 1>, launch_group<2, 2>, launch_group<2, 3>, launch_group<2, 4>},
                                {launch_group<3, 1>, launch_group<3, 2>, launch_group<3, 3>, launch_group<3, 4>},
                                {launch_group<4, 1>, launch_group<4, 2>, launch_group<4, 3>, launch_group<4, 4>}};
    return fn[bits - 2][nt - 1](A, (int)total, stream);
}

// us of that launch, and the weight tiles per workgroup that make it shortest: a workgroup takes 1.15 us, 0.18 for each weight tile and,
// for every run of its waves, 0.30 and 0.145 a weight tile, up to 12 % more as the chip fills; one to a CU, in rounds where all rows are
// alike, else the longest first with half of a short one's time lost at the end.  40000 launches of one to seven linears, as in awq_gemv_group_us: 7 %
// rms; its choice takes 0.4 % longer than the best one on average.
double awq_tile_group_us(int bits, const GemvProblem *p, int count, int M, int *nt)
{
    double tiles = 0.0;
    for (int i = 0; i < count; ++i) tiles += (double)(p[i].N / 16) * (p[i].K / RUN);
    const double memory = 1e-4 * tiles * (bits == 4 ? 0.75 : bits == 3 ? 0.5 : 0.4) * (M > 8 ? 1.25 : 1.0);
    double best = 0.0;
    for (int n = 1; n <= 4; ++n) {
        double total = 0.0, longest = 0.0, shortest = 1e30;
        int wgs = 0;
        for (int i = 0; i < count; ++i) {
            const int w = (p[i].N / 16 + n - 1) / n;
            const double d = 1.15 + 0.18 * n + (p[i].K / RUN + TILE_WAVES - 1) / TILE_WAVES * (0.30 + 0.145 * n);
            wgs += w;
            total += w * d;
            longest = std::max(longest, d);
            shortest = std::min(shortest, d);
        }
        const double span = longest == shortest ? (wgs + 255) / 256 * longest : std::max(longest, total / 256.0 + 0.53 * shortest);
        const double us = 1.27 + span * (1.0 + 0.12 * std::min(1.0, wgs / 256.0)) + memory;
        if (n == 1 || us < best) {
            best = us;
            *nt = n;
        }
    }
    return best;
}
