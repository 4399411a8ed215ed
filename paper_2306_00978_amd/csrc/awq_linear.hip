// awq_w4a16_linear: validation and dispatch between the decode kernels (M <= 16), the K-split tile kernel
// (a few dozen to a few hundred tokens) and the prefill kernel.  AWQ Sec. 4.2: the same fused dequantization is used
// by the matrix-vector and the matrix-matrix kernel.
#include "awq_common.h"
#include "awq_gemv_stream.h"
#include "awq_tile.h"

#include <stdlib.h>
#include <algorithm>
#include <atomic>
#include <string>

int awq_gemv_launch_residual(const void *x, const void *qweight, const void *scales, const void *zeros,
                             void *y, const void *res, int M, int N, int K, hipStream_t stream);
int awq_gemv_launch(const void *x, const void *qweight, const void *scales, const void *zeros,
                    void *y, int M, int N, int K, hipStream_t stream);
int awq_gemm_launch(const void *x, const void *qweight, const void *scales, const void *zeros,
                    void *y, int M, int N, int K, hipStream_t stream);

int awq_gemm_launch_split(const void *x, const void *qweight, const void *scales, const void *zeros,
                          void *y, int M, int N, int K, void *part, int ksplit, hipStream_t stream);
int awq_gemm_ksplit(int M, int N, int K, double *estimate_us);
double awq_gemm_unsplit_us(int M, int N, int K);
double awq_gemm_ranges_us(int M, int N, int K);

// Only the prefill kernel at a few hundred tokens uses scratch: fp32 partial tiles of its K ranges.  (The
// tile kernel has taken over part of these shapes and needs none; the figure stays what callers size
// their buffers by, and what decides which shapes the static entry point refuses.)
extern "C" size_t awq_linear_workspace_bytes(int64_t M, int64_t N, int64_t K, int group)
{
    if (awq_check_weight_shape(N, K, group) != AWQ_OK || M <= 48 || M > (int64_t)1 << 22) return 0;
    double split_us = 0.0;
    const int ks = awq_gemm_ksplit((int)M, (int)N, (int)K, &split_us);
    // 49..128 tokens are the tile kernel's, but for large matrices with a workspace.  The figure is the one that
    // callers know: nothing where blocks of 16 tokens through the decode kernels would do (7 us + blocks * packed
    // bytes at 6 TB/s) and the shape fits one launch of them
    if (M <= 128 && awq_gemv_stream_fits((int)N, (int)K, 16)) {
        const double blocked_us = 7.0 + (double)((M + 15) / 16) * ((double)N * (double)K * 0.53125) / 6.0e6;
        if (ks < 2 || split_us > 0.85 * blocked_us) return 0;
    }
    return ks > 1 ? (size_t)ks * (size_t)M * (size_t)N * sizeof(float) : 0;
}

namespace {

// The prefill kernel's tiles are 128 x 256: at a few hundred tokens there are few of them, each
// walking a long K, and cutting K over workgroups costs a second pass over fp32 partial tiles.  The tile
// kernel cuts K over the waves of a workgroup and pays with more reads of x (a tile is at most 128 x 48
// or 96 x 64), so it wins until the prefill kernel fills the chip.
//
// By the estimates; a tie is the tile kernel's (awq_tile.h).  us, tile kernel and K whole: 4096 x 4096 at 300 / 512 / 1000 tokens
// 18 / 29 / 50 and 43 / 44 / 48, 4096 x 14336 at 960 127 and 140; tile kernel and ranges: 4096 x 4096 at 400 / 700 / 1000 25 / 36 /
// 51 and 29 / 38 / 43, 4096 x 11008 at 129 / 200 / 256 / 448 25 / 32 / 32 / 57 and 32 / 34 / 36 / 50, 1024 x 28672 at 256 33 and 43,
// 28672 x 8192 at 96 / 128 58 / 87 and 60 / 63.
// Without a workspace up to 128 tokens always the tile kernel: the faster one but where features are many (128 tokens: 28672 x 512
// 18.3 and 12.2, 128256 x 4096 201 and 115; 160 tokens 28672 x 512 21.5 and 14.1, 57344 x 512 36.1 and 24.9).
bool takes_tile_kernel(const TilePlan &plan, int M, int N, int K, bool split)
{
    if (awq_tile_override() >= 0) return awq_tile_forced();
    if (split) return plan.us < AWQ_TILE_TIE * awq_gemm_ranges_us(M, N, K);
    return M <= 128 || plan.us < AWQ_TILE_TIE * awq_gemm_unsplit_us(M, N, K);
}

}  // namespace

// Which kernel takes the linears of a decode call: the estimated times of the batch kernel (several linears, 4 and 3 bits) and of the
// tile kernel against one of the kernels that would run otherwise -- for several linears a fit to what those took, of the weight
// tiles in thousands, the longest row in thousands of columns and the row blocks in 256: the streaming kernel up to four tokens, from five (3 bits:
// nine) the one that takes the activations through LDS, or several launches; 7 to 14 % rms.  8 % in favour of those, and 15 % from 32
// thousand tiles (a layer of hidden size 2304), where the estimates' errors are larger than what is to be gained.  Over 1900 calls of two to
// seven linears in 4 bits and 1800 in 3 (graph replays, eight token counts each) the choice is 1.16, 1.24, 1.35, 1.25, 1.38 and 1.37 times faster at 1, 2, 4,
// 5, 8 and 9 to 16 tokens -- 1.3 to 1.6 times below 16 thousand tiles -- and more than 3 % slower in one call of a hundred.
// One linear: from five tokens, 1.03 times faster at 5 to 8 and 1.1 from 9.  2 bits: from nine tokens, 1.07.
int awq_few_launch(int bits, const GemvProblem *p, int count, int M, hipStream_t stream)
{
    // (the tuning build: 0 the kernels that would run otherwise, 1 to 4 the tile kernel, 5 the batch kernel)
    // (and an override of another decode kernel's plan asks for that kernel)
    int forced = awq_knob("AWQ_FEW", -1);
#ifdef AWQ_TUNING_KNOBS
    for (const char *plan : {"STAGES", "SLOTS", "KSL", "ITERS", "JOBS", "WAVES", "STREAM_SINGLE"})
        if (getenv((std::string("AWQ_GEMV_") + plan).c_str())) forced = 0;
#endif
    if (forced == 0 || !awq_few_considered(bits, count, M, count == 1 ? (int64_t)p[0].N * p[0].K : 0)) return AWQ_GEMV_STREAM_UNFIT;
    if (forced > 0 && forced < 5) return awq_tile_group_launch(bits, forced, p, count, M, stream);
    if (forced == 5) return bits == 2 ? AWQ_GEMV_STREAM_UNFIT : awq_gemv_group_launch(bits, p, count, M, stream);
    double tiles = 0.0, blocks = 0.0, longest = 0.0, shortest = 1e30;
    for (int i = 0; i < count; ++i) {
        blocks += p[i].N / 16 / 256.0;
        tiles += (double)(p[i].N / 16) * (p[i].K / AWQ_GROUP) / 1000.0;
        longest = std::max(longest, p[i].K / 1024.0);
        shortest = std::min(shortest, p[i].K / 1024.0);
    }
    // 2 bits: the estimates of short launches are half a microsecond off; below 4 thousand tiles nothing is gained (23 groups at 9 to 16 tokens 0.89 to 1.04 times
    // as fast: 1024 x 1024 with two of 128 x 1024 3.0 us and 3.4), nor by a lone linear of up to 2048 columns (10 of 5728 to 27616 features 0.93 to 1.02: 9952 x
    // 1024 4.2 and 4.5).  A lone linear has 4 thousand tiles in any case.
    if (bits == 2 && (tiles < 4.0 || (count == 1 && longest <= 2.0))) return AWQ_GEMV_STREAM_UNFIT;
    // Rows of 2048 columns beside longer ones of 4096 and more, all of which the streaming kernel takes, fill its batches at five and six tokens
    // (3 bits: to eight), and it is up to a quarter faster than the fit below says: from 18 thousand tiles, in 4 bits up to its 32 MB, such a
    // call is left to it.  us, streaming and as chosen otherwise, 5 tokens: a layer of hidden size 2048 (7936) in 4 bits 10.6 / 14.1, 2048 (5120) 9.6 /
    // 11.1, in 3 bits 9.8 / 11.5 and, 2048 (7680), 10.2 / 14.3.  (Calls of two to seven linears: 80 above the line 0.91 times as fast on average by the
    // estimates, 0.72 to 1.22, 36 below 1.29, at least 1.09; all rows 4096 and longer, above, 1.06.)
    if (count > 1 && bits != 2 && M > 4 && M <= (bits == 4 ? 6 : 8) && tiles > 18.0 && (bits == 3 || tiles <= 32.8)) {
        bool whole = shortest == 2.0 && longest > 2.0;
        for (int i = 0; i < count; ++i)
            whole = whole && (p[i].K == 2048 || p[i].K >= 4096) && awq_gemv_stream_fits(p[i].N, p[i].K, M);
        if (whole) return AWQ_GEMV_STREAM_UNFIT;
    }
    static const double fit[2][6][4] = {{{3.75, 0.137, 0.239, 0.255}, {4.11, 0.130, 0.282, 0.236}, {4.74, 0.141, 0.333, 0.284},
                                         {3.76, 0.179, 0.507, 0.174}, {4.26, 0.173, 0.595, 0.280}, {3.75, 0.112, 1.072, 0.431}},
                                        {{3.60, 0.165, 0.206, 0.194}, {4.03, 0.163, 0.228, 0.167}, {4.64, 0.156, 0.326, 0.289},
                                         {3.68, 0.174, 0.681, 0.064}, {4.10, 0.122, 1.091, 0.161}, {4.65, 0.121, 1.150, 0.134}}};
    double present;
    if (bits == 2) present = 2.9 + (0.165 + 0.0062 * M) * tiles + 0.37 * longest + 0.09 * blocks;
    else if (count == 1) present = awq_gemv_us(bits, M, p[0].N, p[0].K);
    else {
        const double *c = fit[bits == 4][M <= 2 ? M - 1 : M <= 4 ? 2 : M <= 6 ? 3 : M <= 8 ? 4 : 5];
        present = c[0] + c[1] * tiles + c[2] * longest + c[3] * blocks;
        if (M == 3) present = 0.5 * (present + fit[bits == 4][1][0] + fit[bits == 4][1][1] * tiles + fit[bits == 4][1][2] * longest +
                                     fit[bits == 4][1][3] * blocks);
    }
    int nt = 1;
    const double tile = awq_tile_group_us(bits, p, count, M, &nt);
    const double batch = bits != 2 && count > 1 ? awq_gemv_group_us(bits, p, count, M) : 1e30;
    // (2 bits, rows of different lengths: 16 %.  Of 44 such calls between the two lines 12 were slower by the tile kernel, a layer of hidden size 2048
    // (7168) at 16 tokens 11.5 us and 14.5, of 72 beyond none.)
    const double margin = bits == 2 && longest != shortest ? 1.16 : tiles < 32.8 ? 1.08 : 1.15;
    if (std::min(tile, batch) * margin > present) return AWQ_GEMV_STREAM_UNFIT;
    if (count > 1) awq_note_plain_plan();
    return batch < tile ? awq_gemv_group_launch(bits, p, count, M, stream) : awq_tile_group_launch(bits, nt, p, count, M, stream);
}

// Whether awq_w4a16_linear without a workspace runs the prefill kernel (whose loss form the scale search uses).
bool awq_linear_takes_prefill(int M, int N, int K)
{
    return M > 16 && !takes_tile_kernel(awq_tile_plan(M, N, K), M, N, K, false);
}

extern "C" int awq_w4a16_linear(const void *x_f16, const void *qweight, const void *scales,
                                const void *zeros, void *y_f16, int64_t M, int64_t N,
                                int64_t K, int group, void *workspace, size_t workspace_bytes,
                                void *stream)
{
    if (!x_f16 || !qweight || !scales || !zeros || !y_f16) return AWQ_ERR_NULL_POINTER;
    int st = awq_check_weight_shape(N, K, group);
    if (st != AWQ_OK) return st;
    if (M <= 0 || M > (int64_t)1 << 22) return AWQ_ERR_BAD_SHAPE;
    if (!awq_aligned16(x_f16) || !awq_aligned16(qweight) || !awq_aligned16(scales) ||
        !awq_aligned16(zeros) || !awq_aligned16(y_f16))
        return AWQ_ERR_MISALIGNED;
    // the workspace is optional: with NULL, K is not split
    const size_t need = awq_linear_workspace_bytes(M, N, K, group);
    const bool split = need > 0 && workspace;
    if (split && workspace_bytes < need) return AWQ_ERR_WORKSPACE_TOO_SMALL;
    if (split && !awq_aligned16(workspace)) return AWQ_ERR_MISALIGNED;
    if (M <= 16) {
        // a single linear is a short kernel dominated by one memory round trip: the batch
        // kernel (everything requested at once) is the faster one; the streaming kernel is
        // for grouped launches.  (The tuning build can force it: AWQ_GEMV_STREAM_SINGLE.)
        static const bool stream_single = awq_knob("AWQ_GEMV_STREAM_SINGLE", 0) != 0;
        if (stream_single) {
            GemvProblem p = {};
            p.x = (const half_t *)x_f16;
            p.q = (const uint4 *)qweight;
            p.sc = (const uint16_t *)scales;
            p.zp = (const uint8_t *)zeros;
            p.y = (half_t *)y_f16;
            p.N = (int)N;
            p.K = (int)K;
            st = awq_gemv_stream_launch(&p, 1, (int)M, (hipStream_t)stream);
            if (st != AWQ_GEMV_STREAM_UNFIT) return st;
        }
        if (awq_few_considered(4, 1, (int)M, N * K)) {
            GemvProblem p = {};
            p.x = (const half_t *)x_f16;
            p.q = (const uint4 *)qweight;
            p.sc = (const uint16_t *)scales;
            p.zp = (const uint8_t *)zeros;
            p.y = (half_t *)y_f16;
            p.N = (int)N;
            p.K = (int)K;
            st = awq_few_launch(4, &p, 1, (int)M, (hipStream_t)stream);
            if (st != AWQ_GEMV_STREAM_UNFIT) return st;
        }
        return awq_gemv_launch(x_f16, qweight, scales, zeros, y_f16, (int)M, (int)N, (int)K,
                               (hipStream_t)stream);
    }
    const TilePlan plan = awq_tile_plan((int)M, (int)N, (int)K);
    if (takes_tile_kernel(plan, (int)M, (int)N, (int)K, split))
        return awq_tile_launch(4, plan, x_f16, qweight, scales, zeros, y_f16, (int)M, (int)N, (int)K,
                               (hipStream_t)stream);
    if (split)
        return awq_gemm_launch_split(x_f16, qweight, scales, zeros, y_f16, (int)M, (int)N, (int)K, workspace,
                                     awq_gemm_ksplit((int)M, (int)N, (int)K, nullptr), (hipStream_t)stream);
    return awq_gemm_launch(x_f16, qweight, scales, zeros, y_f16, (int)M, (int)N, (int)K,
                           (hipStream_t)stream);
}

// ---- the entry point that allocates nothing ---------------------------------------------------
// The K-range form of the prefill kernel needs room for its fp32 partial tiles.  Callers that cannot
// allocate (code under graph capture, serving loops, harnesses that forbid it) get that room from
// this array: one copy per GPU the library runs on, held until the process ends.  In host code the
// name `scratch` is only a handle for hipGetSymbolAddress; kernels receive the device address.
static __device__ __align__(256) unsigned char scratch[AWQ_STATIC_SCRATCH_BYTES];

namespace {

// Device address of `scratch` on the current device, looked up once per device.
int static_scratch(void **out)
{
    static std::atomic<void *> address[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return AWQ_ERR_HIP;
    void *p = address[dev].load(std::memory_order_acquire);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return AWQ_ERR_HIP;
        }
        address[dev].store(p, std::memory_order_release);      // every thread finds the same address
    }
    *out = p;
    return AWQ_OK;
}

}  // namespace

extern "C" size_t awq_static_scratch_bytes(void) { return AWQ_STATIC_SCRATCH_BYTES; }

extern "C" int awq_w4a16_linear_static(const void *x_f16, const void *qweight, const void *scales,
                                       const void *zeros, void *y_f16, int64_t M, int64_t N, int64_t K,
                                       int group, void *stream)
{
    // same validation order as awq_w4a16_linear, so that a bad argument reads the same from both
    if (!x_f16 || !qweight || !scales || !zeros || !y_f16) return AWQ_ERR_NULL_POINTER;
    int st = awq_check_weight_shape(N, K, group);
    if (st != AWQ_OK) return st;
    if (M <= 0 || M > (int64_t)1 << 22) return AWQ_ERR_BAD_SHAPE;
    const size_t need = awq_linear_workspace_bytes(M, N, K, group);
    if (need > AWQ_STATIC_SCRATCH_BYTES) return AWQ_ERR_SCRATCH_LIMIT;
    void *ws = nullptr;
    if (need > 0) {
        st = static_scratch(&ws);
        if (st != AWQ_OK) return st;
    }
    return awq_w4a16_linear(x_f16, qweight, scales, zeros, y_f16, M, N, K, group, ws, need, stream);
}

extern "C" int awq_w4a16_linear_multi(const awq_linear_desc *descs, int count, int64_t M, int group,
                                      void *workspace, size_t workspace_bytes, void *stream)
{
    (void)workspace; (void)workspace_bytes;
    if (!descs) return AWQ_ERR_NULL_POINTER;
    if (count < 1 || count > AWQ_MULTI_MAX) return AWQ_ERR_BAD_ARGUMENT;
    if (M <= 0 || M > 16) return AWQ_ERR_BAD_SHAPE;
    GemvProblem p[GEMV_MAX_PROBLEMS] = {};
    for (int i = 0; i < count; ++i) {
        const awq_linear_desc &d = descs[i];
        if (!d.x_f16 || !d.qweight || !d.scales || !d.zeros || !d.y_f16) return AWQ_ERR_NULL_POINTER;
        int st = awq_check_weight_shape(d.N, d.K, group);
        if (st != AWQ_OK) return st;
        if (!awq_aligned16(d.x_f16) || !awq_aligned16(d.qweight) || !awq_aligned16(d.scales) ||
            !awq_aligned16(d.zeros) || !awq_aligned16(d.y_f16))
            return AWQ_ERR_MISALIGNED;
        p[i].x = (const half_t *)d.x_f16;
        p[i].q = (const uint4 *)d.qweight;
        p[i].sc = (const uint16_t *)d.scales;
        p[i].zp = (const uint8_t *)d.zeros;
        p[i].y = (half_t *)d.y_f16;
        p[i].N = (int)d.N;
        p[i].K = (int)d.K;
    }
    // More than four tokens: the kernel that takes the activations through LDS (any K) runs all
    // linears of the call in one launch.  A lone linear goes there only when it has row blocks
    // enough for every CU; a smaller one stays with the batch kernel, where everything requested at once is the faster way
    // through a small matrix (N = 4096, K = 11008: 10 us against 20 us), or goes to the tile kernel.  Where a row of workgroups of
    // the tile kernel, four weight tiles each, is more than one round of 256, N > 16384, a lone linear is not looked at: over 107 shapes up to
    // 152064 features at 5 to 16 tokens the tile kernel takes 0.95 to 2.4 times as long, 1.22 on average (us, through LDS and by tiles, 16 tokens: 32000 x 4096 18.2 / 19.1,
    // 50304 x 2048 15.6 / 22.5, 128256 x 4096 50.1 / 66.3; 5 tokens, 128256 x 8192 89.9 / 107.7), and at 16384 the faster one
    // (16384 x 4096 14.3 / 10.9).
    if (count > 1 || M <= 4 || p[0].N <= 16384) {
        const int st_few = awq_few_launch(4, p, count, (int)M, (hipStream_t)stream);
        if (st_few != AWQ_GEMV_STREAM_UNFIT) return st_few;
    }
    static const int rows_min_count = awq_knob("AWQ_ROWS_MIN_COUNT", 2);
    // At five and six tokens a small launch is the streaming kernel's still, whose waves request all of it at
    // once (a layer of hidden size 1280 / 3840 at five tokens, 9.4 MB: 7.5 us and 10.1 through LDS; 2048 / 5632, 22 MB: 9.8
    // and 13.3; at eight tokens even).  How small: a wave holds two batches of 512 columns of K at these M, and where K is no
    // multiple of the waves' share some have two and some one.  Groups of two and three linears over 4 to 31 MiB, streaming over rows kernel:
    // K of 2048, 4096 and more 1.03 to 1.9 throughout; other K 1.07 to 1.6 at 4 MiB and 0.80 to 1.3 from 8 on.  Layers of
    // seven linears, hidden sizes 1024 to 2304: 1.05 to 1.4 up to 25 MiB, 0.92 to 1.2 from there.
    bool small = M <= 6 && count > 1, even = true;
    int64_t packed = 0;
    for (int i = 0; i < count; ++i) {
        packed += (int64_t)p[i].N * p[i].K / 2;
        even = even && (p[i].K == 2048 || p[i].K >= 4096);
        small = small && awq_gemv_stream_fits(p[i].N, p[i].K, (int)M);
    }
    small = small && packed <= (int64_t)(even ? 32 : count >= 4 ? 24 : 4) << 20;
    if (M > 4 && !small && (count >= rows_min_count || p[0].N >= 16384))
        return awq_gemv_rows_launch(p, count, (int)M, (hipStream_t)stream);
    // The linears whose K fits the register-resident activations of the streaming kernel at
    // this M go out in one launch; the others (and a lone linear) take one launch of the batch
    // kernel each.
    GemvProblem fit[GEMV_MAX_PROBLEMS];
    int nfit = 0;
    bool grouped[GEMV_MAX_PROBLEMS] = {};
    if (count > 1) {
        for (int i = 0; i < count; ++i)
            if (awq_gemv_stream_fits(p[i].N, p[i].K, (int)M)) {
                fit[nfit++] = p[i];
                grouped[i] = true;
            }
        if (nfit < 2) {
            nfit = 0;
            for (int i = 0; i < count; ++i) grouped[i] = false;
        }
    }
    if (nfit > 0) {
        int st = awq_gemv_stream_launch(fit, nfit, (int)M, (hipStream_t)stream);
        if (st == AWQ_GEMV_STREAM_UNFIT) {
            for (int i = 0; i < count; ++i) grouped[i] = false;
        } else if (st != AWQ_OK) {
            return st;
        }
    }
    for (int i = 0; i < count; ++i) {
        if (grouped[i]) continue;
        int st = awq_gemv_launch(p[i].x, p[i].q, p[i].sc, p[i].zp, p[i].y, (int)M, p[i].N, p[i].K,
                                 (hipStream_t)stream);
        if (st != AWQ_OK) return st;
    }
    return AWQ_OK;
}

namespace {

// validation of the linears of a fused / chained call and their translation for the launcher
int fused_problems(const awq_fused_desc *descs, int count, int group, GemvProblem *p, GemvFusedExtra *e)
{
    for (int i = 0; i < count; ++i) {
        const awq_linear_desc &d = descs[i].linear;
        if (!d.x_f16 || !d.qweight || !d.scales || !d.zeros || !d.y_f16) return AWQ_ERR_NULL_POINTER;
        int st = awq_check_weight_shape(d.N, d.K, group);
        if (st != AWQ_OK) return st;
        if (!awq_aligned16(d.x_f16) || !awq_aligned16(d.qweight) || !awq_aligned16(d.scales) ||
            !awq_aligned16(d.zeros) || !awq_aligned16(d.y_f16))
            return AWQ_ERR_MISALIGNED;
        if (descs[i].pre_op == AWQ_PRE_RMSNORM || descs[i].pre_op == AWQ_PRE_SCALE) {
            if (!descs[i].pre_f16) return AWQ_ERR_NULL_POINTER;
            if (!awq_aligned16(descs[i].pre_f16)) return AWQ_ERR_MISALIGNED;
            if (descs[i].pre_op == AWQ_PRE_RMSNORM && !(descs[i].eps >= 0.0f)) return AWQ_ERR_BAD_ARGUMENT;
        } else if (descs[i].pre_op != AWQ_PRE_NONE) {
            return AWQ_ERR_BAD_ARGUMENT;
        }
        p[i] = GemvProblem{};
        p[i].x = (const half_t *)d.x_f16;
        p[i].q = (const uint4 *)d.qweight;
        p[i].sc = (const uint16_t *)d.scales;
        p[i].zp = (const uint8_t *)d.zeros;
        p[i].y = (half_t *)d.y_f16;
        p[i].N = (int)d.N;
        p[i].K = (int)d.K;
        e[i].pre = (const half_t *)descs[i].pre_f16;
        e[i].res = (const half_t *)descs[i].residual_f16;
        e[i].eps = descs[i].eps;
        e[i].pre_op = descs[i].pre_op == AWQ_PRE_RMSNORM ? GEMV_PRE_RMSNORM
                      : descs[i].pre_op == AWQ_PRE_SCALE ? GEMV_PRE_SCALE : GEMV_PRE_NONE;
    }
    return AWQ_OK;
}

}  // namespace

extern "C" int awq_w4a16_linear_chain(const awq_chain_stage *stages, int n_stages, int64_t M, int group, void *sync,
                                      int spin_limit, void *stream)
{
    if (!stages || !sync) return AWQ_ERR_NULL_POINTER;
    if (n_stages < 1 || n_stages > AWQ_CHAIN_MAX_STAGES || spin_limit < 0) return AWQ_ERR_BAD_ARGUMENT;
    if (M <= 0 || M > 16) return AWQ_ERR_BAD_SHAPE;
    if (!awq_aligned16(sync)) return AWQ_ERR_MISALIGNED;
    GemvProblem p[AWQ_CHAIN_MAX_STAGES][AWQ_CHAIN_MAX_LINEARS];
    GemvFusedExtra e[AWQ_CHAIN_MAX_STAGES][AWQ_CHAIN_MAX_LINEARS];
    const GemvProblem *pp[AWQ_CHAIN_MAX_STAGES];
    const GemvFusedExtra *ee[AWQ_CHAIN_MAX_STAGES];
    int counts[AWQ_CHAIN_MAX_STAGES];
    static_assert(AWQ_CHAIN_MAX_STAGES == CHAIN_MAX_STAGES && AWQ_CHAIN_MAX_LINEARS == CHAIN_MAX_ENTRIES &&
                  AWQ_CHAIN_SYNC_BYTES >= CHAIN_SYNC_BYTES, "limits");
    for (int s = 0; s < n_stages; ++s) {
        if (!stages[s].descs) return AWQ_ERR_NULL_POINTER;
        if (stages[s].count < 1 || stages[s].count > AWQ_CHAIN_MAX_LINEARS) return AWQ_ERR_BAD_ARGUMENT;
        const int st = fused_problems(stages[s].descs, stages[s].count, group, p[s], e[s]);
        if (st != AWQ_OK) return st;
        for (int i = 0; i < stages[s].count; ++i)
            if (!awq_gemv_stream_fits(p[s][i].N, p[s][i].K, (int)M)) return AWQ_ERR_BAD_SHAPE;
        pp[s] = p[s];
        ee[s] = e[s];
        counts[s] = stages[s].count;
    }
    const int st = awq_gemv_chain_launch(pp, ee, counts, n_stages, (int)M, (uint32_t *)sync, spin_limit,
                                         (hipStream_t)stream);
    return st == AWQ_GEMV_STREAM_UNFIT ? AWQ_ERR_BAD_SHAPE : st;
}

extern "C" int awq_w4a16_linear_fused_multi(const awq_fused_desc *descs, int count, int64_t M, int group,
                                            void *stream)
{
    if (!descs) return AWQ_ERR_NULL_POINTER;
    if (count < 1 || count > AWQ_FUSED_MAX) return AWQ_ERR_BAD_ARGUMENT;
    if (M <= 0 || M > 16) return AWQ_ERR_BAD_SHAPE;
    GemvProblem p[GEMV_MAX_FUSED] = {};
    GemvFusedExtra e[GEMV_MAX_FUSED] = {};
    {
        const int st = fused_problems(descs, count, group, p, e);
        if (st != AWQ_OK) return st;
    }
    // a lone linear without a normalisation: the batch kernel (every shape, and the faster one
    // for a single small matrix)
    if (count == 1 && e[0].pre_op == GEMV_PRE_NONE)
        return awq_gemv_launch_residual(p[0].x, p[0].q, p[0].sc, p[0].zp, p[0].y, e[0].res, (int)M, p[0].N,
                                        p[0].K, (hipStream_t)stream);
    for (int i = 0; i < count; ++i)
        if (!awq_gemv_stream_fits(p[i].N, p[i].K, (int)M)) return AWQ_ERR_BAD_SHAPE;
    int st = awq_gemv_stream_launch_fused(p, e, count, (int)M, (hipStream_t)stream);
    return st == AWQ_GEMV_STREAM_UNFIT ? AWQ_ERR_BAD_SHAPE : st;
}

extern "C" int awq_w4a16_linear_fused_fits(int64_t N, int64_t K, int64_t M, int group)
{
    if (M <= 0 || M > 16 || awq_check_weight_shape(N, K, group) != AWQ_OK) return 0;
    return awq_gemv_stream_fits((int)N, (int)K, (int)M) ? 1 : 0;
}
