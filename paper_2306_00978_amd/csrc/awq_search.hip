// awq_search_scale for gfx950: the grid search for the activation-aware scale.
//
// AWQ Sec. 3.2, the search for the scale.  Eq. 4 asks for the per-input-channel scale s that
// minimises the output difference of one layer after quantization,
//     L(s) = || Q(W diag(s)) (diag(s)^-1 X) - W X ||,
// on calibration rows X cached for that layer; Eq. 5 restricts s to s_X^alpha (s_X = mean |X|
// per channel) and picks alpha on a grid over [0, 1].
//
// Every candidate is evaluated with the kernels that serve the layer afterwards, so the loss is
// the loss of the deployed arithmetic: quantize_pack(W, s_X^alpha) -> x' = X / s ->
// awq_w4a16_linear(x') -> sum of squared differences to the fp16 layer X W^T (one dense fp16
// MFMA product, computed once).  Sums of squares are kept in fp64 and reduced in a fixed order;
// the argmin and s* = s_X^alpha* are taken on the device, so the call neither synchronises nor
// copies to the host.
#include "awq_common.h"
#include "awq_gemm_epilogue.h"
#include "awq_tile.h"

#include <algorithm>
#include <type_traits>

int awq_act_mean_launch(const void *X_f16, int64_t T, int64_t K, float *mean, hipStream_t stream);
int awq_quantize_inv_launch(const void *W, const float *s, int64_t N, int64_t K, void *qweight, void *scales, void *zeros,
                            const void *x, int64_t M, void *xs, int points, size_t step, hipStream_t stream);
bool awq_linear_takes_prefill(int M, int N, int K);
int64_t awq_gemm_tiles(int M, int N);
int awq_gemm_launch_loss(const void *x, const void *qweight, const void *scales, const void *zeros, const void *y_ref,
                         int M, int N, int K, double *loss, int points, size_t step, size_t loss_step, hipStream_t stream);

namespace {

constexpr int LOSS_BLOCKS = 1024;
constexpr int MAX_ALPHAS = 64;

struct AlphaList {
    float a[MAX_ALPHAS];
};

// s_X^alpha for the grid points [first, first + gridDim.y)
__global__ __launch_bounds__(256) void pow_kernel(const float *__restrict__ mean, AlphaList alphas, int first, int K,
                                                  float *__restrict__ s)
{
    asm volatile("" ::"s"(mean), "s"(K), "s"(s));                       // arguments in one round
    const int k = blockIdx.x * 256 + threadIdx.x;
    if (k < K) s[(size_t)blockIdx.y * K + k] = powf(mean[k], alphas.a[first + blockIdx.y]);
}

typedef __attribute__((address_space(3))) void lds_void_t;
typedef const __attribute__((address_space(1))) void gbl_void_t;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void dma16(const unsigned char *g, uint32_t lds_addr)
{
    __builtin_amdgcn_global_load_lds((gbl_void_t *)(uintptr_t)g, (lds_void_t *)(uintptr_t)lds_addr, 16, 0, 0);
}

// Y[T,N] = X[T,K] W[N,K]^T, fp16 operands, fp32 accumulation, fp16 result: the unquantized layer of Eq. 4.
// The geometry of the W4A16 prefill kernel: 128 x 256 tile, eight waves, four side by side along N (128 x 64
// each, 8 x 4 tiles of v_mfma_f32_16x16x32_f16), the two waves of a SIMD taking a half of a stage's columns
// each.  A stage is 64 columns of K: 128 rows of X and 256 of W, 128 bytes each, memory -> LDS in whole
// cache lines, 16-byte chunk k of row i at place k ^ (i / 2 % 8), so that the fragment reads (16 rows) are free
// of bank conflicts; a ring of three stages (144 KB), one barrier per stage.  The second half of a wave's token tiles
// runs behind the barrier: its MFMAs cover the first fragment reads of the next stage.
// (128 x 128 tiles staged through registers with two barriers per 64 columns: 296 us = 232 TFLOP/s at
// 2048 x 4096 x 4096; this form 71 us = 970; with 32x32x16 MFMAs 75.)
constexpr int DM = 128, DN = 256, DSTAGES = 3;
constexpr int D_A = DM * 128, D_STAGE = (DM + DN) * 128;
constexpr int D_LDS = DSTAGES * D_STAGE;

__global__ __launch_bounds__(512, 1) void dense_gemm_kernel(const half_t *__restrict__ X, const half_t *__restrict__ W,
                                                            half_t *__restrict__ Y, int T, int N, int K, int tiles_n,
                                                            int tiles_total)
{
    extern __shared__ __align__(16) unsigned char smem[];
    asm volatile("" ::"s"(X), "s"(W), "s"(Y), "s"(T), "s"(N), "s"(K), "s"(tiles_n), "s"(tiles_total));
    const int per_xcd = (tiles_total + 7) >> 3;              // contiguous ranges of tiles per XCD
    const int tile = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    if (tile >= tiles_total || ((int)blockIdx.x >> 3) >= per_xcd) return;
    const int tile_m = tile / tiles_n, tile_n = tile - tile_m * tiles_n;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nq = wave & 3, kh = wave >> 2, r = lane & 15, c = lane >> 4;
    const int m0 = tile_m * DM, n0 = tile_n * DN;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem);

    // the wave fetches rows 16 w .. + 16 of X and 32 w .. + 32 of W, eight rows per load; rows past the end
    // repeat the last one
    const unsigned char *src[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const int row = (i < 2 ? 16 * wave + 8 * i : 32 * wave + 8 * (i - 2)) + (lane >> 3);
        const int chunk = (lane & 7) ^ ((row >> 1) & 7);
        src[i] = i < 2 ? reinterpret_cast<const unsigned char *>(X + (size_t)min(m0 + row, T - 1) * K) + 16 * chunk
                       : reinterpret_cast<const unsigned char *>(W + (size_t)min(n0 + row, N - 1) * K) + 16 * chunk;
    }
    const int stages = K / 64;
    auto request = [&](int st, int slot) {
        const size_t at = (size_t)min(st, stages - 1) * 128;             // past the end: a harmless repeat
        const uint32_t dst = lds0 + slot * D_STAGE;
#pragma unroll
        for (int i = 0; i < 6; ++i)
            dma16(src[i] + at, dst + (i < 2 ? wave * 2048 + i * 1024 : D_A + wave * 4096 + (i - 2) * 1024));
    };
    // fragments of the wave's step, columns 32 kh .. + 32 of the stage: rows 16 i + r, chunk 4 kh + c
    const uint32_t place = (uint32_t)(((4 * kh + c) ^ ((r >> 1) & 7)) * 16);
    const uint32_t aofs = lds0 + r * 128 + place, bofs = lds0 + D_A + (64 * nq + r) * 128 + place;
    u32x4 a[4], b[4], an[4], bn[4];
#define AWQ_READ_A(HALF_, SLOT_)                                                                              \
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(an[0]) : "v"(aofs + (SLOT_) * D_STAGE), "n"((HALF_) * 8192));        \
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(an[1]) : "v"(aofs + (SLOT_) * D_STAGE), "n"((HALF_) * 8192 + 2048)); \
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(an[2]) : "v"(aofs + (SLOT_) * D_STAGE), "n"((HALF_) * 8192 + 4096)); \
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(an[3]) : "v"(aofs + (SLOT_) * D_STAGE), "n"((HALF_) * 8192 + 6144));
#define AWQ_READ_B(SLOT_)                                                                                     \
    asm volatile("ds_read_b128 %0, %1" : "=v"(bn[0]) : "v"(bofs + (SLOT_) * D_STAGE));                        \
    asm volatile("ds_read_b128 %0, %1 offset:2048" : "=v"(bn[1]) : "v"(bofs + (SLOT_) * D_STAGE));            \
    asm volatile("ds_read_b128 %0, %1 offset:4096" : "=v"(bn[2]) : "v"(bofs + (SLOT_) * D_STAGE));            \
    asm volatile("ds_read_b128 %0, %1 offset:6144" : "=v"(bn[3]) : "v"(bofs + (SLOT_) * D_STAGE));
#define AWQ_ADOPT_A()                                                                                         \
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(an[0]), "+v"(an[1]), "+v"(an[2]), "+v"(an[3]));                \
    a[0] = an[0]; a[1] = an[1]; a[2] = an[2]; a[3] = an[3];
#define AWQ_ADOPT_B()                                                                                         \
    asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(bn[0]), "+v"(bn[1]), "+v"(bn[2]), "+v"(bn[3]));                \
    b[0] = bn[0]; b[1] = bn[1]; b[2] = bn[2]; b[3] = bn[3];
    floatx4 acc[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](auto half) {
        constexpr int H = decltype(half)::value;
#pragma unroll
        for (int s = 0; s < 16; ++s) {
            // back and forth along the tokens: see the W4A16 prefill kernel
            const int j = s >> 2, i = (j & 1) ? 3 - (s & 3) : s & 3;
            acc[4 * H + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a[i]),
                                                                       __builtin_bit_cast(half8_t, b[j]),
                                                                       acc[4 * H + i][j], 0, 0, 0);
        }
    };

    request(0, 0);
    request(1, 1);
    request(2, 2);
    asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    AWQ_READ_A(0, 0)
    AWQ_READ_B(0)
    AWQ_ADOPT_A()
    AWQ_ADOPT_B()
    int slot = 0;
    for (int st = 0; st < stages; ++st) {
        AWQ_READ_A(1, slot)
        __builtin_amdgcn_sched_barrier(0);
        multiply(std::integral_constant<int, 0>{});
        __builtin_amdgcn_sched_barrier(0);
        AWQ_ADOPT_A()
        // this wave has read all it needs of the stage; the next one has landed when only the six loads of
        // the stage after it are outstanding, and behind the barrier that holds for every wave
        asm volatile("s_waitcnt vmcnt(6)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        request(st + 3, slot);
        slot = slot + 1 == DSTAGES ? 0 : slot + 1;
        AWQ_READ_A(0, slot)
        AWQ_READ_B(slot)
        __builtin_amdgcn_sched_barrier(0);
        multiply(std::integral_constant<int, 1>{});
        __builtin_amdgcn_sched_barrier(0);
        AWQ_ADOPT_A()
        AWQ_ADOPT_B()
    }
#undef AWQ_READ_A
#undef AWQ_READ_B
#undef AWQ_ADOPT_A
#undef AWQ_ADOPT_B
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // the harmless repeats
    __syncthreads();
    floatx4 own[4][4];
    gemm_pair_sum(acc, own, smem, wave, lane, kh);
    gemm_store(gemm_turn(own, smem, wave, lane), Y, m0 + 64 * kh, n0 + 64 * nq, T, N, lane);
}

int dense_gemm_launch(const half_t *X, const half_t *W, half_t *Y, int T, int N, int K, hipStream_t stream)
{
    const int tiles_n = (N + DN - 1) / DN;
    const int64_t total = (int64_t)tiles_n * ((T + DM - 1) / DM);
    if (total > (1 << 30)) return AWQ_ERR_BAD_SHAPE;
    static AwqOncePerDevice once;
    std::atomic<bool> &attr_set = once.here();
    if (!attr_set.load(std::memory_order_relaxed)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(dense_gemm_kernel),
                                hipFuncAttributeMaxDynamicSharedMemorySize, D_LDS) != hipSuccess)
            return AWQ_ERR_HIP;
        attr_set.store(true, std::memory_order_relaxed);
    }
    dense_gemm_kernel<<<dim3((unsigned)((total + 7) / 8 * 8)), dim3(512), D_LDS, stream>>>(X, W, Y, T, N, K, tiles_n,
                                                                                           (int)total);
    return awq_launch_status();
}

// partial[b] = sum over the 16-byte chunks of workgroup b of (Yq - Y)^2: eight differences are
// squared and added in fp32, the chunk sums are added in fp64; the workgroup's 256 sums are
// folded in a fixed tree, so the result does not depend on timing.
__global__ __launch_bounds__(256) void loss_kernel(const uint4 *__restrict__ Yq,
                                                   const uint4 *__restrict__ Y, int64_t chunks,
                                                   double *__restrict__ partial)
{
    asm volatile("" ::"s"(Yq), "s"(Y), "s"(chunks), "s"(partial));     // arguments in one round
    __shared__ double red[256];
    double acc = 0.0;
    // four chunk pairs requested together (a chunk past the end re-reads the last one and is not
    // counted); the order of the additions is the order of the chunks either way
    const int64_t stride = (int64_t)LOSS_BLOCKS * 256;
    for (int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x; i0 < chunks; i0 += 4 * stride) {
        uint4 a[4], b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t i = i0 + u * stride, ic = i < chunks ? i : chunks - 1;
            a[u] = Yq[ic];
            b[u] = Y[ic];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const half_t *ha = reinterpret_cast<const half_t *>(&a[u]);
            const half_t *hb = reinterpret_cast<const half_t *>(&b[u]);
            float c = 0.f;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float d = (float)ha[e] - (float)hb[e];
                c += d * d;
            }
            if (i0 + u * stride < chunks) acc += (double)c;
        }
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int half = 128; half >= 1; half >>= 1) {
        if ((int)threadIdx.x < half) red[threadIdx.x] += red[threadIdx.x + half];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// losses[i] = sum of the `count` partial sums of grid point i (a wave per grid point, fixed order); best = first
// index of the smallest loss (a loss that is not a number never wins); s_best = s_X^alpha[best].
__global__ __launch_bounds__(1024) void finalize_kernel(const double *__restrict__ partial, int count, int n_alpha,
                                                        AlphaList alphas, const float *__restrict__ mean,
                                                        int K, double *__restrict__ losses,
                                                        int32_t *__restrict__ best, float *__restrict__ s_best)
{
    __shared__ double total[MAX_ALPHAS];
    __shared__ int chosen;
    const int tid = threadIdx.x, lane = tid & 63;
    for (int i = tid >> 6; i < n_alpha; i += 16) {
        double v[LOSS_BLOCKS / 64];                 // requested together
#pragma unroll
        for (int k = 0; k < LOSS_BLOCKS / 64; ++k)
            v[k] = lane + 64 * k < count ? partial[(size_t)i * LOSS_BLOCKS + lane + 64 * k] : 0.0;
        double sum = v[0];
#pragma unroll
        for (int k = 1; k < LOSS_BLOCKS / 64; ++k) sum += v[k];
#pragma unroll
        for (int d = 1; d <= 32; d <<= 1) sum += __shfl_xor(sum, d);
        if (lane == 0) total[i] = sum;
    }
    __syncthreads();
    if (tid == 0) {
        int b = 0;
        double lb = total[0] == total[0] ? total[0] : __builtin_inf();
        for (int i = 1; i < n_alpha; ++i) {
            const double li = total[i] == total[i] ? total[i] : __builtin_inf();
            if (li < lb) { lb = li; b = i; }
        }
        chosen = b;
        *best = b;
    }
    if (tid < n_alpha) losses[tid] = total[tid];
    __syncthreads();
    const float alpha = alphas.a[chosen];
    for (int k = tid; k < K; k += 1024) s_best[k] = powf(mean[k], alpha);
}

struct SearchLayout {
    size_t mean, s, xs, q, sc, zp, step, y, yq, partial, powers, total;
};

inline size_t up256(size_t v) { return (v + 255) & ~(size_t)255; }

// `points` candidates, `step` bytes apart
SearchLayout search_layout(int64_t T, int64_t N, int64_t K, int n_alpha, int points)
{
    SearchLayout L;
    const int64_t G = K / AWQ_GROUP;
    size_t o = 0;
    L.mean = o; o = up256(o + (size_t)K * 4);
    L.s = o; o = up256(o + (size_t)K * 4);
    L.xs = o; o = up256(o + (size_t)T * K * 2);
    L.q = o; o = up256(o + (size_t)N * K / 2);
    L.sc = o; o = up256(o + (size_t)N * G * 2);
    L.zp = o; o = up256(o + (size_t)N * G / 2);
    L.step = o - L.xs;
    o += (size_t)(points - 1) * L.step;
    L.y = o; o = up256(o + (size_t)T * N * 2);
    L.yq = o; o = up256(o + (size_t)T * N * 2);
    L.partial = o; o = up256(o + (size_t)n_alpha * LOSS_BLOCKS * 8);
    // the powers of all grid points: in the place of the candidate's outputs, where that is large enough (several candidates at a time
    // are evaluated without it)
    L.powers = (int64_t)n_alpha * K * 4 <= T * N * 2 ? L.yq : o;
    if (points > 1 && L.powers == o) o = up256(o + (size_t)n_alpha * K * 4);
    L.total = o;
    return L;
}

// How a grid point's product and loss are computed.
struct SearchProduct {
    bool fused, prefill;           // the loss in the product's epilogue; by the prefill kernel
    TilePlan plan;                 // otherwise by the tile kernel
    int64_t tiles;                 // partial sums of a point
};

SearchProduct search_product(int64_t T, int64_t N, int64_t K, int points)
{
    // Above 16 tokens the kernel that the layer runs, prefill or tile, has a loss form that takes the differences
    // in the product's epilogue (2048 x 4096 x 4096: the product 59 us either way, without the 7 us pass over both
    // outputs; 159 x 1120 x 2944: 21.2 us a grid point before, 16.5 then); its tiles have to fit the
    // partial sums of a grid point
    SearchProduct P = {false, false, {1, 1, 0.0}, 0};
    if (T <= 16) return P;
    P.prefill = awq_linear_takes_prefill((int)T, (int)N, (int)K);
    if (!P.prefill) P.plan = awq_tile_plan((int)T, (int)N, (int)K, points);
    P.tiles = P.prefill ? awq_gemm_tiles((int)T, (int)N) : awq_tile_count(P.plan, (int)T, (int)N);
    P.fused = P.tiles <= LOSS_BLOCKS;
    return P;
}

// Candidates at a time, given the workspace for it.  One by one a search is a chain of launches: quantizing and dividing (17 us at 4096 x
// 4096 and 2048 rows, a third of it start and run-out) and a product that fills the chip only where the layer is large.  Together W and X
// are read, and the launches made, once for all of them, and their products fill the chip together.  As many as 128 MB hold, so
// that the memory-side cache still has them for the product (60 / 128 / 180 / 600 MB: 4096 x 4096 at 2048 rows 1389 / 1360 / 1373 /
// 1407 us, at 200 rows 497 / 488 / 489 / 476).  us, one by one and together, 20 points: 2048 x 4096 x 4096 1483 / 1360,
// 1722 x 3472 x 2304 846 / 654, 537 x 1328 x 1920 349 / 188, 95 x 1456 x 1792 273 / 91, 64 x 1024 x 1024 195 / 60.
int search_points(int64_t T, int64_t N, int64_t K, int n_alpha)
{
    static const int64_t megabytes = awq_knob("AWQ_SEARCH_MB", 128);
    const SearchLayout L = search_layout(T, N, K, n_alpha, 1);
    const int64_t most = std::min<int64_t>(n_alpha, (megabytes << 20) / (int64_t)L.step);
    if (most < 2) return 1;
    const int launches = (int)((n_alpha + most - 1) / most), points = (n_alpha + launches - 1) / launches;
    return search_product(T, N, K, points).fused ? points : 1;
}

int check_search_shape(int64_t T, int64_t N, int64_t K, int n_alpha, int group)
{
    int st = awq_check_weight_shape(N, K, group);
    if (st != AWQ_OK) return st;
    if (T <= 0 || T > (int64_t)1 << 22) return AWQ_ERR_BAD_SHAPE;
    if (n_alpha < 1 || n_alpha > MAX_ALPHAS) return AWQ_ERR_BAD_ARGUMENT;
    return AWQ_OK;
}

}  // namespace

extern "C" size_t awq_search_scale_workspace_bytes(int64_t T, int64_t N, int64_t K, int n_alpha,
                                                   int group)
{
    if (check_search_shape(T, N, K, n_alpha, group) != AWQ_OK) return 0;
    return search_layout(T, N, K, n_alpha, 1).total;
}

extern "C" size_t awq_search_scale_batch_workspace_bytes(int64_t T, int64_t N, int64_t K, int n_alpha, int group)
{
    if (check_search_shape(T, N, K, n_alpha, group) != AWQ_OK) return 0;
    return search_layout(T, N, K, n_alpha, search_points(T, N, K, n_alpha)).total;
}

extern "C" int awq_search_scale(const void *W_f16, const void *X_f16, int64_t T, int64_t N, int64_t K,
                                const float *alphas, int n_alpha, int group, void *workspace,
                                size_t workspace_bytes, double *losses, int32_t *best, float *s_best,
                                void *stream)
{
    if (!W_f16 || !X_f16 || !alphas || !workspace || !losses || !best || !s_best)
        return AWQ_ERR_NULL_POINTER;
    int st = check_search_shape(T, N, K, n_alpha, group);
    if (st != AWQ_OK) return st;
    AlphaList al = {};
    for (int i = 0; i < n_alpha; ++i) {
        if (!(alphas[i] >= 0.0f && alphas[i] <= 1.0f)) return AWQ_ERR_BAD_ARGUMENT;
        al.a[i] = alphas[i];
    }
    if (!awq_aligned16(W_f16) || !awq_aligned16(X_f16) || !awq_aligned16(s_best) ||
        (reinterpret_cast<uintptr_t>(workspace) & 255u) != 0 ||
        (reinterpret_cast<uintptr_t>(losses) & 7u) != 0 || (reinterpret_cast<uintptr_t>(best) & 3u) != 0)
        return AWQ_ERR_MISALIGNED;
    if (workspace_bytes < search_layout(T, N, K, n_alpha, 1).total) return AWQ_ERR_WORKSPACE_TOO_SMALL;
    int points = search_points(T, N, K, n_alpha);
    // (fewer at a time: as many as fit and whose plan has room for its partial sums, as search_points() asks of its own number)
    if (points > 1 && workspace_bytes < search_layout(T, N, K, n_alpha, points).total) {
        do --points;
        while (points > 1 && (workspace_bytes < search_layout(T, N, K, n_alpha, points).total || !search_product(T, N, K, points).fused));
    }
    const SearchLayout L = search_layout(T, N, K, n_alpha, points);
    unsigned char *ws = static_cast<unsigned char *>(workspace);
    float *mean = reinterpret_cast<float *>(ws + L.mean);
    float *s = reinterpret_cast<float *>(ws + L.s);
    void *xs = ws + L.xs, *q = ws + L.q, *sc = ws + L.sc, *zp = ws + L.zp;
    half_t *Y = reinterpret_cast<half_t *>(ws + L.y);
    half_t *Yq = reinterpret_cast<half_t *>(ws + L.yq);
    double *partial = reinterpret_cast<double *>(ws + L.partial);
    hipStream_t hs = (hipStream_t)stream;

    st = awq_act_mean_launch(X_f16, T, K, mean, hs);
    if (st != AWQ_OK) return st;
    st = dense_gemm_launch((const half_t *)X_f16, (const half_t *)W_f16, Y, (int)T, (int)N, (int)K, hs);
    if (st != AWQ_OK) return st;
    const SearchProduct P = search_product(T, N, K, points);
    const int64_t chunks = T * N / 8;                    // N % 16 == 0
    // the powers of all grid points in one launch, where their place is not used for outputs
    const bool table = P.fused && L.powers < L.total;
    float *powers = table ? reinterpret_cast<float *>(ws + L.powers) : s;
    for (int i = 0; i < n_alpha; i += points) {
        const int count = std::min(points, n_alpha - i);
        if (!table || i == 0) {
            pow_kernel<<<dim3((unsigned)((K + 255) / 256), table ? (unsigned)n_alpha : 1u), dim3(256), 0, hs>>>(
                mean, al, i, (int)K, powers);
            st = awq_launch_status();
            if (st != AWQ_OK) return st;
        }
        st = awq_quantize_inv_launch(W_f16, table ? powers + (size_t)i * K : s, N, K, q, sc, zp, X_f16, T, xs, count, L.step, hs);
        if (st != AWQ_OK) return st;
        double *part = partial + (size_t)i * LOSS_BLOCKS;
        if (P.fused) {
            st = P.prefill ? awq_gemm_launch_loss(xs, q, sc, zp, Y, (int)T, (int)N, (int)K, part, count, L.step, LOSS_BLOCKS, hs)
                           : awq_tile_launch_loss(P.plan, xs, q, sc, zp, Y, (int)T, (int)N, (int)K, part, count, L.step, LOSS_BLOCKS, hs);
            if (st != AWQ_OK) return st;
            continue;
        }
        st = awq_w4a16_linear(xs, q, sc, zp, Yq, T, N, K, group, nullptr, 0, stream);
        if (st != AWQ_OK) return st;
        loss_kernel<<<dim3(LOSS_BLOCKS), dim3(256), 0, hs>>>((const uint4 *)Yq, (const uint4 *)Y, chunks, part);
        st = awq_launch_status();
        if (st != AWQ_OK) return st;
    }
    finalize_kernel<<<dim3(1), dim3(1024), 0, hs>>>(partial, P.fused ? (int)P.tiles : LOSS_BLOCKS, n_alpha, al, mean, (int)K, losses, best, s_best);
    return awq_launch_status();
}
