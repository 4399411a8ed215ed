// Prefill path of awq_w4a16_linear (M > 16) for gfx950.
//
// AWQ Sec. 4.2: with 4-bit storage and 16-bit compute the dequantization has to
// sit inside the main loop of the matrix-matrix kernel (it cannot be moved to the
// epilogue as with W8A8), and dequantized weights are never written to memory.
//
// Mapping.  A workgroup computes a 128 (tokens) x 256 (out-features) tile of y with
// eight waves: four side by side along N (128 x 64 = 8 x 4 tiles of
// v_mfma_f32_16x16x32_f16, 128 fp32 accumulators per lane), each of them twice, the two
// copies sharing a SIMD and splitting K between them: of a quantization group (128 columns) each takes half of the
// slots of every packed tile, two MFMA steps of 32 columns, and
// the two partial tiles are added through LDS at the end.  A single wave per SIMD cannot keep
// the matrix pipe busy (loop overhead, waits, the change of group all stall it); with two,
// one computes while the other does that work, and no weight is dequantized twice.
//
// What bounds it is power, then issue: on activations and 4-bit weights a loop of nothing but MFMAs runs at 2000
// TFLOP/s with the 16x16x32 shape and at 1740 with 32x32x16 (the clock falls; on zeros both reach 2400), and every
// vector instruction beside them costs about as much energy as a thirtieth of an MFMA.  Hence the small shape, 126 vector
// instructions to 64 MFMAs (offsets that stay in their registers, constants by one multiply-add each), fragment reads
// without bank conflicts, and consecutive MFMAs that share their weight fragment and then their token fragment.  Against
// the 32x32x16 form of the same tile, at first: 2048 x 11008 x 4096 176 -> 160 us, 2048 x 4096 x 4096 62 -> 56.5, 2048 x 4096 x 11008
// 156 -> 138, on zeros 138 -> 127, 48 -> 44, 118 -> 104; with the shorter start and exchange (GemmUnits, gemm_pair_sum) the first
// takes 152 to 161 from box to box (1150 to 1215 TFLOP/s).
//
// Operands.  Nothing is staged through registers on the way in: both operands are
// fetched with global_load_lds (memory -> LDS, 16 bytes per lane landing in lane order),
// two groups ahead of the one being computed, into a ring of three stages.
//   * x: one load instruction fetches 8 rows x 128 contiguous bytes (whole cache lines) and
//     lands as 8 LDS rows of 128 bytes.  Which 16-byte chunk of the row a lane fetches is
//     XOR-swizzled with the row index, so that a fragment (16 rows, a chunk each) is read back with one conflict-free
//     ds_read_b128.  All waves share the x tile (wave (n-quarter q, k-half h) loads row block
//     q, column half h of every group); one barrier per group.
//   * weights: the packed layout is already the B-operand layout.  A wave loads and reads only its own half of a tile,
//     the slots 2 h and 2 h + 1 of every row (512 contiguous bytes), and its own steps and zero points.  Lane (r, c) takes
//     words 2 (c/2) and 2 (c/2) + 1 of slot 2 h + c%2, one in each of the wave's steps; the columns that they hold are
//     chunk 4 step + 2 h + c%2 of column half c/2 of the group, which is what the token fragment reads.  (A pair of
//     adjacent words: with words c/2 and 2 + c/2, which would make the columns of a step contiguous, the reads had two-way
//     bank conflicts, 4 % on 2048 x 11008 x 4096.)
//   Each fragment word is expanded in registers to fp16 (q - z) * scale and feeds eight
//   MFMAs (the token tiles).
// fp32 accumulation, one rounding to fp16 at the end.
#include "awq_common.h"
#include "awq_gemm_epilogue.h"

#include <type_traits>
#include <utility>

namespace {

typedef __attribute__((address_space(3))) void lds_void_t;
typedef const __attribute__((address_space(1))) void gbl_void_t;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr int BM = 128, BN = 256;
constexpr int NSTAGE = 3;
constexpr int A_STAGE = 32 * 1024;               // 4 row blocks x 2 column halves x (32 rows x 128 B)
constexpr int B_STAGE = 2048 + 256 + 256;        // of a wave: half of four tiles, 64 steps, 64 zero bytes (a dword each)
constexpr int B_SC = 2048, B_ZP = 2304;
constexpr int LDS_BYTES = NSTAGE * A_STAGE + 8 * NSTAGE * B_STAGE;
constexpr int LOADS_PER_GROUP = 4 + 2 + 2;       // per wave
constexpr int PART_ROW = 68;                     // floats per row of a partial tile on its way out
static_assert(8 * 64 * PART_ROW * 4 <= LDS_BYTES && LDS_BYTES <= 160 * 1024, "LDS");

__device__ __forceinline__ void dma16(const void *g, uint32_t lds_addr)
{
    __builtin_amdgcn_global_load_lds((gbl_void_t *)(uintptr_t)g, (lds_void_t *)(uintptr_t)lds_addr,
                                     16, 0, 0);
}
__device__ __forceinline__ void dma2(const void *g, uint32_t lds_addr)
{
    __builtin_amdgcn_global_load_lds((gbl_void_t *)(uintptr_t)g, (lds_void_t *)(uintptr_t)lds_addr,
                                     2, 0, 0);
}
__device__ __forceinline__ void dma1(const void *g, uint32_t lds_addr)
{
    __builtin_amdgcn_global_load_lds((gbl_void_t *)(uintptr_t)g, (lds_void_t *)(uintptr_t)lds_addr,
                                     1, 0, 0);
}

// LDS reads are written as asm so that the compiler does not tie them to the outstanding
// memory->LDS loads of later groups; the waits are placed by hand.
template <int OFF>
__device__ __forceinline__ u32x4 lds_read16_off(uint32_t addr)
{
    u32x4 v;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
template <int OFF>
__device__ __forceinline__ u32x2 lds_read8(uint32_t addr)
{
    u32x2 v;
    asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
    return v;
}
// the dwords at addr + 4 O0 and addr + 4 O1
template <int O0, int O1>
__device__ __forceinline__ u32x2 lds_read2(uint32_t addr)
{
    u32x2 v;
    asm volatile("ds_read2_b32 %0, %1 offset0:%2 offset1:%3" : "=v"(v) : "v"(addr), "n"(O0), "n"(O1));
    return v;
}
__device__ __forceinline__ void lds_wait(u32x4 &a, u32x4 &b, u32x4 &c, u32x4 &d)
{
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d));
}

// f(integral_constant 0), f(1), ... in order
template <int... I, class F>
__device__ __forceinline__ void in_order(std::integer_sequence<int, I...>, F f)
{
    (f(std::integral_constant<int, I>{}), ...);
}

struct DqConsts {
    uint32_t mask_lo, mask_hi;   // SGPR
    uint32_t magA, magB;         // VGPR
};

__device__ __forceinline__ DqConsts dq_consts()
{
    DqConsts k = {0x000F000Fu, 0x00F000F0u, 0x64006400u, 0x54005400u};
    asm("" : "+s"(k.mask_lo));
    asm("" : "+s"(k.mask_hi));
    asm("" : "+v"(k.magA));
    asm("" : "+v"(k.magB));
    return k;
}

// Dequantization of one packed word (eight codes) to fp16 (q - z) * scale, k order, cut into
// 13 single-instruction steps so that the main loop can place them one by one in the issue
// shadow of the MFMAs:  (w & mask) | magic is 1024+q or 64+q as a half pair; subtracting
// 1024+z / 64+z is exact; one rounding in the multiplication by the step.
struct DqWord {
    uint32_t w, w8;
    uint32_t t[4];
};

template <int OP>
__device__ __forceinline__ void dq_step(DqWord &d, const DqConsts &k, half2_t zA, half2_t zB,
                                        half2_t s2)
{
    if (OP == 0) d.w8 = d.w >> 8;
    if (OP == 1) d.t[0] = (d.w & k.mask_lo) | k.magA;
    if (OP == 2) d.t[1] = (d.w & k.mask_hi) | k.magB;
    if (OP == 3) d.t[2] = (d.w8 & k.mask_lo) | k.magA;
    if (OP == 4) d.t[3] = (d.w8 & k.mask_hi) | k.magB;
    if (OP >= 5 && OP <= 8) {
        const int i = OP - 5;
        d.t[i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, d.t[i]) - ((i & 1) ? zB : zA));
    }
    if (OP >= 9 && OP <= 12) {
        const int i = OP - 9;
        d.t[i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, d.t[i]) * s2);
    }
}

// part SLOT of SLOTS of the 52 steps that dequantize the four words of an MFMA step
template <int SLOT, int SLOTS>
__device__ __forceinline__ void dq_slice(DqWord (&d)[4], const DqConsts &k, const half2_t (&zA)[4],
                                         const half2_t (&zB)[4], const half2_t (&s2)[4])
{
    in_order(std::make_integer_sequence<int, 52>{}, [&](auto step) {
        constexpr int I = decltype(step)::value, n = I / 13, op = I % 13;
        if constexpr (I >= 52 * SLOT / SLOTS && I < 52 * (SLOT + 1) / SLOTS) dq_step<op>(d[n], k, zA[n], zB[n], s2[n]);
    });
}

__device__ __forceinline__ half8_t dq_result(const DqWord &d)
{
    return __builtin_bit_cast(half8_t, make_uint4(d.t[0], d.t[1], d.t[2], d.t[3]));
}

// SPLIT: K is cut into `ksplit` ranges of whole groups, one workgroup per (tile, range); each
// writes its partial tile in fp32 to part[range][M][N] and a second kernel adds the ranges.  For
// a few hundred tokens there are far fewer tiles than CUs (ceil(M/128) * N/256), and a workgroup
// per tile would leave most of the chip idle while a handful of CUs walk all of K.
// GEMM_LOSS (the scale search): nothing is stored; y holds the layer's reference outputs, and the workgroup
// leaves the sum over its tile of the squared differences to them in loss[tile] -- of the outputs
// rounded to fp16, eight differences squared and added in fp32, the rest in fp64, in a fixed order, as the
// separate pass over two stored outputs does it.
// How the units of a launch are numbered, without a division in the kernel (two by arguments and one in 64 bits are 0.4 us
// in front of the first load): a / b is the high half of a times floor((2^32 - 1) / b), one too small at most.
struct GemmUnits {
    int tiles_n, ksplit, units_total, group_base, group_rem;      // G = ksplit * group_base + group_rem
    uint32_t tiles_n_inverse, ksplit_inverse;
};
__device__ __forceinline__ int quotient(int a, int b, uint32_t inverse)
{
    const int q = (int)(((uint64_t)(uint32_t)a * inverse) >> 32);
    return a - q * b >= b ? q + 1 : q;
}

enum { GEMM_PLAIN, GEMM_SPLIT, GEMM_LOSS };
// GEMM_LOSS: the units of several grid points follow each other; point i reads x, weights, steps and zero points i `step` bytes
// further and leaves its sums loss_step further.
template <int MODE>
struct GemmPoints {};
template <>
struct GemmPoints<GEMM_LOSS> {
    int tiles;                     // of a point
    uint32_t tiles_inverse;
    int64_t step, loss_step;
};
template <int MODE>
__global__ __launch_bounds__(512, 1) void gemm_kernel(
    const half_t *__restrict__ x, const unsigned char *__restrict__ qweight,
    const unsigned char *__restrict__ scales, const unsigned char *__restrict__ zeros,
    half_t *__restrict__ y, int M, int N, int K, int G, const GemmUnits U, float *__restrict__ part,
    double *__restrict__ loss, const GemmPoints<MODE> points)
{
    constexpr bool SPLIT = MODE == GEMM_SPLIT;
    extern __shared__ __align__(16) unsigned char smem[];
    // all arguments fetched in one round (otherwise one scalar-cache miss per first use)
    asm volatile("" ::"s"(x), "s"(qweight), "s"(scales), "s"(zeros), "s"(y), "s"(M), "s"(N), "s"(K), "s"(G),
                 "s"(U.tiles_n), "s"(U.ksplit), "s"(U.units_total), "s"(U.group_base), "s"(U.group_rem), "s"(U.tiles_n_inverse),
                 "s"(U.ksplit_inverse), "s"(part), "s"(loss));
    // Workgroups are handed to the eight XCDs round-robin by their linear id, and each XCD has
    // its own L2.  The tile a workgroup computes is therefore chosen so that an XCD gets a
    // contiguous range of tiles in token-block-major order: its workgroups then share a few x
    // row blocks and sweep the same weight groups at about the same time, which keeps the
    // operand traffic inside that L2.
    const int per_xcd = (U.units_total + 7) >> 3;            // units: (tile, K range) pairs
    const int unit = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    if (unit >= U.units_total) return;
    int tile = SPLIT ? quotient(unit, U.ksplit, U.ksplit_inverse) : unit;
    if constexpr (MODE == GEMM_LOSS) {
        const int point = quotient(unit, points.tiles, points.tiles_inverse);
        tile = unit - point * points.tiles;
        x = reinterpret_cast<const half_t *>(reinterpret_cast<const unsigned char *>(x) + point * points.step);
        qweight += point * points.step;
        scales += point * points.step;
        zeros += point * points.step;
        loss += point * points.loss_step;
    }
    const int ks = SPLIT ? unit - tile * U.ksplit : 0;
    // groups [gofs, gofs + GL) of the G of a row: the first ranges are one longer where the count does not divide G
    const int gofs = SPLIT ? ks * U.group_base + min(ks, U.group_rem) : 0;
    const int GL = SPLIT ? U.group_base + (ks < U.group_rem ? 1 : 0) : G;
    const int tile_m = quotient(tile, U.tiles_n, U.tiles_n_inverse), tile_n = tile - tile_m * U.tiles_n;
    const DqConsts kc = dq_consts();
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // waves w and w+4 run on the same SIMD: they form a pair on the same 128 x 64 sub-tile
    const int nq = wave & 3;                                 // which 64 out-features
    const int kh = wave >> 2;                                // which MFMA steps: 2 t + kh
    const int r = lane & 15, c = lane >> 4;
    const int m0 = tile_m * BM;
    const int NT = N >> 4;                                   // 16-row weight tiles in the matrix
    const int nt0 = tile_n * (BN / 16) + nq * 4;            // first of the pair's four tiles

    // ---- sources of this lane's memory->LDS loads: 32-bit offsets beside wave-uniform bases (group 0)
    // x: the wave fetches rows 32 nq .. +32, columns 64 kh .. +64 of the group; load q (0..3)
    // covers rows 8 q .. +8 of them; lane l takes row 8 q + l/8 (rows >= M repeat row M-1) and
    // chunk (l%8) ^ f, f = ((row in block)/2)%8, and lands at chunk l%8: sixteen consecutive
    // rows then hold any given chunk in sixteen different bank groups
    const unsigned char *xbase = reinterpret_cast<const unsigned char *>(x) + (size_t)m0 * K * 2 + kh * 128 + (size_t)gofs * 256;
    uint32_t xofs[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int row = min(32 * nq + 8 * q + (lane >> 3), M - 1 - m0);
        const int chunk = (lane & 7) ^ (((8 * q + (lane >> 3)) >> 1) & 7);
        xofs[q] = (uint32_t)row * (uint32_t)(K * 2) + 16 * chunk;
    }
    // weights: half kh of the tiles, two tiles (2 b, 2 b + 1) per load: lane l takes slot (l%16) + 16 (2 kh + l/32)
    // of tile 2 b + l/16 % 2.  Ragged N: repeats the last tile.
    const unsigned char *qbase[2];
    uint32_t qofs[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int t0 = min(nt0 + 2 * b, NT - 1), t1 = min(nt0 + 2 * b + 1, NT - 1);
        qbase[b] = qweight + (size_t)t0 * G * 1024 + kh * 512 + (size_t)gofs * 1024;
        qofs[b] = (c & 1) * (uint32_t)((t1 - t0) * G * 1024) + (r + 16 * (c >> 1)) * 16;
    }
    // steps and zero points: lane (r, c) those of row r of tile c
    const int mt0 = min(nt0, NT - 1);
    const uint32_t mrun = (uint32_t)((min(nt0 + c, NT - 1) - mt0) * G);
    const unsigned char *sbase = scales + ((size_t)mt0 * G + gofs) * 32, *zbase = zeros + ((size_t)mt0 * G + gofs) * 8;
    uint32_t sofs = mrun * 32 + r * 2, zofs = mrun * 8 + (r >> 1);

    const uint32_t a_ring = lds0;
    const uint32_t b_ring = lds0 + NSTAGE * A_STAGE + (uint32_t)wave * (NSTAGE * B_STAGE);

    // One of the 8 loads of a group (PIECE 0..3: x, 4..5: weights, 6: steps, 7: zero points).
    // They are issued one at a time from the issue shadow of the MFMAs.
    auto issue_piece = [&](auto piece_tag, int g, int stage) {
        constexpr int PIECE = decltype(piece_tag)::value;
        g = g < GL ? g : GL - 1;                             // past the end: a harmless repeat
        uint32_t &at = PIECE < 4 ? xofs[PIECE & 3] : PIECE < 6 ? qofs[PIECE & 1] : PIECE == 6 ? sofs : zofs;
        asm volatile("" : "+v"(at));                         // an offset, not part of a 64-bit address
        if constexpr (PIECE < 4) {
            // LDS: [row block 4][column half 2][32 rows x 128 B]
            const uint32_t adst = a_ring + (uint32_t)stage * A_STAGE + (uint32_t)nq * 8192 + (uint32_t)kh * 4096;
            dma16(xbase + (size_t)g * 256 + at, adst + PIECE * 1024);
        } else {
            const uint32_t bdst = b_ring + (uint32_t)stage * B_STAGE;
            if constexpr (PIECE < 6) dma16(qbase[PIECE & 1] + (size_t)g * 1024 + at, bdst + (PIECE & 1) * 1024);
            else if constexpr (PIECE == 6) dma2(sbase + (size_t)g * 32 + at, bdst + B_SC);
            else dma1(zbase + (size_t)g * 8 + at, bdst + B_ZP);
        }
    };
    auto issue_group = [&](int g, int stage) {
        in_order(std::make_integer_sequence<int, LOADS_PER_GROUP>{}, [&](auto piece) { issue_piece(piece, g, stage); });
    };

    floatx4 acc[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int n = 0; n < 4; ++n) acc[i][n] = floatx4{0.f, 0.f, 0.f, 0.f};

    issue_group(0, 0);
    issue_group(1, 1);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS_PER_GROUP) : "memory");
    __builtin_amdgcn_s_barrier();

    // This lane's words of a tile: those of slot 2 kh + c%2 at 2 (c/2) + step, a pair of dwords.  So its A fragment of a
    // step is, of row r of a token tile, chunk 4 step + 2 kh + c%2 of column half c/2.
    const uint32_t boff = (uint32_t)(c & 1) * 512 + (uint32_t)r * 16 + (uint32_t)(c >> 1) * 8;
    const uint32_t aoff[2] = {(uint32_t)(c >> 1) * 4096 + (uint32_t)r * 128 + (uint32_t)(((2 * kh + (c & 1)) ^ ((r >> 1) & 7)) * 16),
                              (uint32_t)(c >> 1) * 4096 + (uint32_t)r * 128 + (uint32_t)(((4 + 2 * kh + (c & 1)) ^ ((r >> 1) & 7)) * 16)};
    const uint32_t moff = (uint32_t)r * 4;
    const int zshift = (r & 1) * 4;

    // ---- what a wave holds in registers for the group it is computing
    u32x2 braw[4];                        // packed words: [tile][step]
    u32x2 sraw[2], zraw[2];               // steps and zero points as read: [tile / 2][tile % 2]
    half2_t s2[4], zA[4], zB[4];          // per tile: step, 1024 + z, 64 + z (as half pairs)
    u32x4 a[4];                           // A fragments: half of the token tiles
    DqWord dq[4];                         // dequantization in flight (next step)
    half8_t bf[4];                        // B fragments of the current step

    auto read_weights = [&](int st) {
        const uint32_t bb = b_ring + (uint32_t)st * B_STAGE;
        braw[0] = lds_read8<0>(bb + boff);
        braw[1] = lds_read8<256>(bb + boff);
        braw[2] = lds_read8<1024>(bb + boff);
        braw[3] = lds_read8<1280>(bb + boff);
        sraw[0] = lds_read2<0, 16>(bb + B_SC + moff);
        sraw[1] = lds_read2<32, 48>(bb + B_SC + moff);
        zraw[0] = lds_read2<0, 16>(bb + B_ZP + moff);
        zraw[1] = lds_read2<32, 48>(bb + B_ZP + moff);
    };
    auto wait_weights = [&]() {
        asm volatile("s_waitcnt lgkmcnt(0)"
                     : "+v"(braw[0]), "+v"(braw[1]), "+v"(braw[2]), "+v"(braw[3]), "+v"(sraw[0]), "+v"(sraw[1]),
                       "+v"(zraw[0]), "+v"(zraw[1]));
    };
    // a tile's constants from what was read, and its first step's word set up
    auto tile_consts = [&](int n) {
        const uint32_t sw = sraw[n >> 1][n & 1], zw = zraw[n >> 1][n & 1];
        const half_t sh = __builtin_bit_cast(half_t, (uint16_t)sw);
        s2[n] = half2_t{sh, sh};
        const uint32_t z = (zw >> zshift) & 0xFu;
        zA[n] = __builtin_bit_cast(half2_t, kc.magA + z * 0x00010001u);
        zB[n] = __builtin_bit_cast(half2_t, kc.magB + z * 0x00100010u);
        dq[n].w = braw[n][0];
    };
    // fragments of token tiles 4 HALF .. + 3 for step S (0, 1) of the wave: one at a time
    auto read_a = [&](auto which, uint32_t stage_base, auto step, auto half) {
        constexpr int I = 4 * decltype(half)::value + decltype(which)::value;
        return lds_read16_off<(I >> 1) * 8192 + (I & 1) * 2048>(stage_base + aoff[decltype(step)::value]);
    };
    typedef std::integral_constant<int, 0> C0;
    typedef std::integral_constant<int, 1> C1;

    // group 0: nothing to overlap with yet
    read_weights(0);
    wait_weights();
#pragma unroll
    for (int n = 0; n < 4; ++n) tile_consts(n);
    in_order(std::make_integer_sequence<int, 4>{}, [&](auto i) { a[i] = read_a(i, a_ring, C0{}, C0{}); });
    dq_slice<0, 1>(dq, kc, zA, zB, s2);
    lds_wait(a[0], a[1], a[2], a[3]);

    int stage = 0;
    for (int g = 0; g < GL; ++g) {
        const int nstage = stage + 1 == NSTAGE ? 0 : stage + 1;    // stage of group g+1
        const int fstage = nstage + 1 == NSTAGE ? 0 : nstage + 1;  // stage to fill with group g+2; it was
                                                                   // last read in group g-1, which every
                                                                   // wave left before the previous barrier
        const uint32_t abase = a_ring + (uint32_t)stage * A_STAGE, nbase = a_ring + (uint32_t)nstage * A_STAGE;
        // Four quarters: step 0 on token tiles 0..3 and 4..7, then step 1.  A quarter is 16 MFMAs, each with
        // something in its issue shadow (the scheduling barriers pin the interleaving): the fragment reads of the
        // next quarter, the loads of group g+2 (quarters 0 and 1), the dequantization of step 1 (0 and 1) or of
        // step 0 of group g+1 (2 and 3).
        in_order(std::make_integer_sequence<int, 4>{}, [&](auto quarter) {
            constexpr int t = decltype(quarter)::value;
            if constexpr ((t & 1) == 0) {
#pragma unroll
                for (int n = 0; n < 4; ++n) bf[n] = dq_result(dq[n]);
            }
            if constexpr (t == 0) {
#pragma unroll
                for (int n = 0; n < 4; ++n) dq[n].w = braw[n][1];
            }
            // this wave's loads of group g+1 have landed once only those of group g+2 are outstanding; behind the
            // barrier that holds for every wave, and nobody reads this group's stage any more
            if constexpr (t == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS_PER_GROUP) : "memory");
            if constexpr (t == 3) __builtin_amdgcn_s_barrier();
            u32x4 an[4];
            __builtin_amdgcn_sched_barrier(0);
            in_order(std::make_integer_sequence<int, 16>{}, [&](auto slot) {
                constexpr int s = decltype(slot)::value, n = s >> 2, i = (n & 1) ? 3 - (s & 3) : s & 3;
                acc[4 * (t & 1) + i][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a[i]), bf[n],
                                                                                 acc[4 * (t & 1) + i][n], 0, 0, 0);
                if constexpr (s < 4) {
                    if constexpr (t == 0) an[s] = read_a(slot, abase, C0{}, C1{});
                    if constexpr (t == 1) an[s] = read_a(slot, abase, C1{}, C0{});
                    if constexpr (t == 2) an[s] = read_a(slot, abase, C1{}, C1{});
                    if constexpr (t == 3) an[s] = read_a(slot, nbase, C0{}, C0{});
                }
                if constexpr (t < 2) {
                    if constexpr (s >= 4 && s < 12 && (s & 1) == 0)
                        issue_piece(std::integral_constant<int, 4 * t + (s - 4) / 2>{}, g + 2, fstage);
                    dq_slice<16 * t + s, 32>(dq, kc, zA, zB, s2);
                }
                if constexpr (t == 2 && s == 4) read_weights(nstage);
                if constexpr (t == 2 && s == 9) wait_weights();
                if constexpr (t == 2 && s >= 9 && s < 13) tile_consts(s - 9);
                if constexpr (t == 2 && s >= 13) dq_slice<s - 13, 19>(dq, kc, zA, zB, s2);
                if constexpr (t == 3) dq_slice<3 + s, 19>(dq, kc, zA, zB, s2);
                __builtin_amdgcn_sched_barrier(0);
            });
            lds_wait(an[0], an[1], an[2], an[3]);
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = an[i];
        });
        stage = nstage;
    }
    // drain the two harmless repeats; after the barrier nobody reads the rings any more
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();

    floatx4 own[4][4];
    gemm_pair_sum(acc, own, smem, wave, lane, kh);

    if (SPLIT) {
        // partial sums leave in fp32, turned around through the wave's own LDS: 16 bytes per lane, four rows of
        // 256 contiguous bytes per instruction
        float *turn = reinterpret_cast<float *>(smem) + wave * (64 * PART_ROW);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int n = 0; n < 4; ++n)
#pragma unroll
                for (int v = 0; v < 4; ++v) turn[(16 * i + 4 * c + v) * PART_ROW + 16 * n + r] = own[i][n][v];
        float *dst = part + (size_t)ks * M * N;
#pragma unroll
        for (int it = 0; it < 16; ++it) {
            const int m = m0 + 64 * kh + 4 * it + c, n = nt0 * 16 + 4 * r;
            const float4 v = *reinterpret_cast<const float4 *>(turn + (4 * it + c) * PART_ROW + 4 * r);
            if (m < M && n < N) *reinterpret_cast<float4 *>(dst + (size_t)m * N + n) = v;
        }
        return;
    }
    const unsigned char *mine = gemm_turn(own, smem, wave, lane);
    if (MODE == GEMM_PLAIN) {
        gemm_store(mine, y, m0 + 64 * kh, nt0 * 16, M, N, lane);
        return;
    }
    const int n = nt0 * 16 + (lane & 7) * 8;
    uint4 ref[8];
#pragma unroll
    for (int it = 0; it < 8; ++it) {
        const int m = m0 + 64 * kh + it * 8 + (lane >> 3);
        // a place outside the matrix re-reads its end and is not counted
        ref[it] = *reinterpret_cast<const uint4 *>(y + (size_t)min(m, M - 1) * N + min(n, N - 8));
    }
    double sum = 0.0;
#pragma unroll
    for (int it = 0; it < 8; ++it) {
        const uint4 v = gemm_row16(mine, it, lane);
        const half_t *ha = reinterpret_cast<const half_t *>(&v), *hb = reinterpret_cast<const half_t *>(&ref[it]);
        float c = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float d = (float)ha[e] - (float)hb[e];
            c += d * d;
        }
        if (m0 + 64 * kh + it * 8 + (lane >> 3) < M && n < N) sum += (double)c;
    }
#pragma unroll
    for (int d = 1; d <= 32; d <<= 1) sum += __shfl_xor(sum, d);
    __syncthreads();                                         // every wave has read its rows
    double *sums = reinterpret_cast<double *>(smem);
    if (lane == 0) sums[wave] = sum;
    __syncthreads();
    if (tid == 0) {
        double total = sums[0];
#pragma unroll
        for (int w = 1; w < 8; ++w) total += sums[w];
        loss[tile] = total;
    }
}

// y = fp16(sum over the KS ranges of the fp32 partial tiles), four outputs per thread, all ranges requested at once (one by
// one they are a chain of KS round trips)
template <int KS>
__global__ __launch_bounds__(256) void gemm_reduce_kernel(const float4 *__restrict__ part, uint2 *__restrict__ y, int64_t quads)
{
    asm volatile("" ::"s"(part), "s"(y), "s"(quads));        // arguments in one round
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= quads) return;
    float4 v[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) v[k] = part[(int64_t)k * quads + i];
    float4 a = v[0];
#pragma unroll
    for (int k = 1; k < KS; ++k) {
        a.x += v[k].x; a.y += v[k].y; a.z += v[k].z; a.w += v[k].w;
    }
    const half2_t lo = {(half_t)a.x, (half_t)a.y}, hi = {(half_t)a.z, (half_t)a.w};
    y[i] = make_uint2(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi));
}

}  // namespace

// How many K ranges the prefill launch of this shape is cut into when a workspace is given: the
// count (1..8, at least four groups per range) with the smallest estimated time.  A workgroup
// taken at 4 us + 1.4 us per group, workgroups in rounds of 256 (one per CU), and the
// second kernel at (ranges + 1/2) * M * N * 4 bytes at 3.5 TB/s after a launch of
// 2.5 us -- figures of an earlier form of the kernel on the three Llama-2-7B shapes at 160..2048 tokens.  They stay because the
// size of the workspace, which callers know, follows from the count: by the estimates below two shapes of 2000 would gain more
// than 5 % from another one, 6 % at most.  Cutting K pays
// while the tiles (ceil(M/128) * N/256) are fewer than the CUs, or just over a multiple of them.
int awq_gemm_ksplit(int M, int N, int K, double *estimate_us)
{
    const int G = K / AWQ_GROUP;
    const int64_t tiles = (int64_t)((N + BN - 1) / BN) * ((M + BM - 1) / BM);
    int best = 1;
    double best_us = 0.0;
    for (int ks = 1; ks <= 8 && (ks == 1 || G / ks >= 4); ++ks) {
        const double rounds = (double)((tiles * ks + 255) / 256);
        const double gl = (double)((G + ks - 1) / ks);
        double us = rounds * (4.0 + 1.4 * gl);
        if (ks > 1) us += 2.5 + (ks + 0.5) * (double)M * (double)N * 4.0 / 3.5e6;
        if (ks == 1 || us < 0.95 * best_us) {       // a split has to win by a margin
            best = ks;
            best_us = us;
        }
    }
    if (estimate_us) *estimate_us = best_us;
    return best;
}

// The time of the launch that does not cut K: rounds of 256 workgroups, 5 us + 1.08 us a group each, and up to half as
// much again as the chip fills, where the power limit lowers the clock.  186 measured launches (16 x 256 to 128256 x 4096 and
// 28672 x 8192, 40 to 1500 tokens): 2.7 % rms, at most 9 % off; 736 others of up to 28672 columns 3.4 %.
double awq_gemm_unsplit_us(int M, int N, int K)
{
    const int64_t tiles = (int64_t)((N + BN - 1) / BN) * ((M + BM - 1) / BM);
    const double rounds = (double)((tiles + 255) / 256), full = (double)tiles / (256.0 * rounds);
    return 1.56 + rounds * (5.0 + 1.083 * (K / AWQ_GROUP)) * (1.0 + 0.46 * full * full);
}

// The time with K cut into awq_gemm_ksplit() ranges: the same with the groups of a range, and the second kernel, which moves
// (ranges + 1/2) * M * N * 4 bytes at 4 TB/s after 7 us of launch, run-out and the first kernel's own stores.  122 launches: 4 % rms, 482 others too.
// (The estimate above is 0.92 to 1.36 of the time.)
double awq_gemm_ranges_us(int M, int N, int K)
{
    const int G = K / AWQ_GROUP, ks = awq_gemm_ksplit(M, N, K, nullptr);
    const int64_t units = (int64_t)((N + BN - 1) / BN) * ((M + BM - 1) / BM) * ks;
    const double rounds = (double)((units + 255) / 256), full = (double)units / (256.0 * rounds);
    return 7.19 + rounds * (2.185 + 1.088 * ((G + ks - 1) / ks)) * (1.0 + 0.342 * full * full) +
           0.25 * (ks + 0.5) * (double)M * (double)N * 4.0e-6;
}

namespace {

template <int MODE>
int gemm_launch_any(const void *x, const void *qweight, const void *scales, const void *zeros,
                    void *y, int M, int N, int K, float *part, int ksplit, double *loss, hipStream_t stream, int count = 1,
                    size_t step = 0, size_t loss_step = 0)
{
    const int G = K / AWQ_GROUP;
    const int tiles_n = (N + BN - 1) / BN;
    const int64_t tiles = (int64_t)tiles_n * ((M + BM - 1) / BM), tiles_total = tiles * count;
    if (tiles_total * ksplit > (1 << 30)) return AWQ_ERR_BAD_SHAPE;
    const dim3 grid((unsigned)((tiles_total * ksplit + 7) / 8 * 8)), block(512);
    const GemmUnits units = {tiles_n, ksplit, (int)(tiles_total * ksplit), G / ksplit, G % ksplit, 0xFFFFFFFFu / (uint32_t)tiles_n,
                             0xFFFFFFFFu / (uint32_t)ksplit};
    static AwqOncePerDevice once;
    std::atomic<bool> &attr_set = once.here();
    if (!attr_set.load(std::memory_order_relaxed)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(gemm_kernel<MODE>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES) != hipSuccess)
            return AWQ_ERR_HIP;
        attr_set.store(true, std::memory_order_relaxed);
    }
    GemmPoints<MODE> points = {};
    if constexpr (MODE == GEMM_LOSS) points = {(int)tiles, 0xFFFFFFFFu / (uint32_t)tiles, (int64_t)step, (int64_t)loss_step};
    gemm_kernel<MODE><<<grid, block, LDS_BYTES, stream>>>(
        (const half_t *)x, (const unsigned char *)qweight, (const unsigned char *)scales,
        (const unsigned char *)zeros, (half_t *)y, M, N, K, G, units, part, loss, points);
    return awq_launch_status();
}

}  // namespace

// Host side of the prefill path; arguments were validated by awq_w4a16_linear.
int awq_gemm_launch(const void *x, const void *qweight, const void *scales, const void *zeros,
                    void *y, int M, int N, int K, hipStream_t stream)
{
    return gemm_launch_any<GEMM_PLAIN>(x, qweight, scales, zeros, y, M, N, K, nullptr, 1, nullptr, stream);
}

// The same with K cut into awq_gemm_ksplit() ranges; part: ksplit * M * N floats, 16-byte aligned.
int awq_gemm_launch_split(const void *x, const void *qweight, const void *scales, const void *zeros,
                          void *y, int M, int N, int K, void *part, int ksplit, hipStream_t stream)
{
    int st = gemm_launch_any<GEMM_SPLIT>(x, qweight, scales, zeros, y, M, N, K, (float *)part, ksplit, nullptr, stream);
    if (st != AWQ_OK) return st;
    const int64_t quads = (int64_t)M * N / 4;
    const dim3 grid((unsigned)((quads + 255) / 256)), block(256);
    const float4 *p = (const float4 *)part;
    uint2 *out = (uint2 *)y;
    switch (ksplit) {
    case 2: gemm_reduce_kernel<2><<<grid, block, 0, stream>>>(p, out, quads); break;
    case 3: gemm_reduce_kernel<3><<<grid, block, 0, stream>>>(p, out, quads); break;
    case 4: gemm_reduce_kernel<4><<<grid, block, 0, stream>>>(p, out, quads); break;
    case 5: gemm_reduce_kernel<5><<<grid, block, 0, stream>>>(p, out, quads); break;
    case 6: gemm_reduce_kernel<6><<<grid, block, 0, stream>>>(p, out, quads); break;
    case 7: gemm_reduce_kernel<7><<<grid, block, 0, stream>>>(p, out, quads); break;
    case 8: gemm_reduce_kernel<8><<<grid, block, 0, stream>>>(p, out, quads); break;
    default: return AWQ_ERR_BAD_SHAPE;                       // awq_gemm_ksplit gives 2 to 8 where there is a workspace
    }
    return awq_launch_status();
}

// The loss form: y_ref [M,N] fp16 is read, loss receives one partial sum for each of awq_gemm_tiles() tiles; the next one of
// `points` grid points has its operands `step` bytes and its sums loss_step further.
int64_t awq_gemm_tiles(int M, int N) { return (int64_t)((N + BN - 1) / BN) * ((M + BM - 1) / BM); }

int awq_gemm_launch_loss(const void *x, const void *qweight, const void *scales, const void *zeros, const void *y_ref,
                         int M, int N, int K, double *loss, int points, size_t step, size_t loss_step, hipStream_t stream)
{
    return gemm_launch_any<GEMM_LOSS>(x, qweight, scales, zeros, const_cast<void *>(y_ref), M, N, K, nullptr, 1, loss,
                                      stream, points, step, loss_step);
}
