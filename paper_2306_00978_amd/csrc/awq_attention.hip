// awq_decode_attention for gfx950: one decode step of the attention layer.
//
// Sec. 4.2, kernel fusion: the attention kernel evaluates the position embedding itself and
// writes the new key and value into caches that were allocated ahead.  One call
// takes the q, k, v rows the (fused) QKV projection produced for the current token, rotates q
// and k by the rotary embedding of the token's position, stores the rotated key and the value
// in the caches, and returns softmax(q K^T / sqrt(D)) V over all positions so far.
//
// The step is bound by reading the caches once (2 * L * Hkv * D * 2 bytes).  They are laid out
// [kv head][position][D], so the keys of a head are one contiguous stream.  A workgroup handles
// one query head and one slice of the positions; a wave takes 16 positions at a time: lane
// l = 16 g + u holds dimensions 8 u .. 8 u + 7 (one 16-byte load) of positions 4 i + g for four i.  The partial
// dot products of the four are folded over the 16 lanes of a group by rotations within the row, one after the other without
// waiting, and each group keeps a running (max, sum, weighted values) of its own positions, brought up to date once for the
// four; merged at the end (groups by shuffles, waves through LDS).  (A position at a time, four xor-shuffles and an update
// each: a chain of some 300 cycles per position, 7.0 us a call and 6.4 with the batches at 8 heads and 200 positions, 8.7 and 8.1 at 32 heads and
// 400; 12.2 and 12.4 at 2000, where the loads bound it.)  Slices are merged by a second, tiny kernel; a short context is one slice.
// The current token's key and value are taken from the inputs, not from the cache row that is
// written in the same launch, so no workgroup depends on another one's stores.
#include "awq_common.h"

#include <cmath>
#include <cstddef>
#include <type_traits>

namespace {

constexpr int AD = 128;                 // head dimension
constexpr int ATT_WAVES = 4, ATT_WHOLE_WAVES = 16;

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// theta^(-2 i / 128), i = 0..63, computed once per call on the host in fp64
struct RopeTable {
    double inv_freq[AD / 2];
};

// q (or k) of one head, rotated: pairs (i, i + 64), angle pos * theta^(-2 i / 128).  The angle (a
// few thousand radians at long contexts) is formed and reduced to [-pi, pi] in fp64, sine and
// cosine of the reduced angle in fp32.  (a, b) are elements t and t + 64, inv_freq is entry t.
__device__ __forceinline__ void rope_pair(float a, float b, double inv_freq, int pos, float &lo, float &hi)
{
    const double ang = (double)pos * inv_freq;
    const double turns = __builtin_rint(ang * 0.15915494309189535);        // 1 / (2 pi)
    const float red = (float)(ang - turns * 6.283185307179586);
    const float sn = sinf(red), cs = cosf(red);
    lo = a * cs - b * sn;
    hi = b * cs + a * sn;
}

struct Running {
    float m, l;          // running maximum of the scores and sum of exp(score - m)
    float acc[8];        // sum of exp(score - m) * value, this lane's eight dimensions
};

// The sum over the 16 lanes of a group, in every one of them: four rotations within the row.
__device__ __forceinline__ float row_sum(float s)
{
    auto turned = [](float v, auto by) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + decltype(by)::value, 0xF, 0xF, false));
    };
    s += turned(s, std::integral_constant<int, 8>{});
    s += turned(s, std::integral_constant<int, 4>{});
    s += turned(s, std::integral_constant<int, 2>{});
    return s + turned(s, std::integral_constant<int, 1>{});
}

__device__ __forceinline__ void merge(Running &r, float m2, float l2, const float (&acc2)[8])
{
    const float m_new = fmaxf(r.m, m2);
    // an empty side has m = -inf and l = 0: exp(-inf - finite) = 0, and two empty sides stay empty
    const float k1 = r.m == m_new ? 1.0f : __expf(r.m - m_new), k2 = m2 == m_new ? 1.0f : __expf(m2 - m_new);
    r.l = r.l * k1 + l2 * k2;
#pragma unroll
    for (int e = 0; e < 8; ++e) r.acc[e] = r.acc[e] * k1 + acc2[e] * k2;
    r.m = m_new;
}

// grid (H, splits); 64 WAVES threads.  partial: [H][splits][AD + 2] floats = (acc[128], m, l).  WHOLE: one slice, finished here (out
// is [H][AD] halves): a second launch costs more than a short context's rows.
template <int WAVES, bool WHOLE>
__global__ __launch_bounds__(64 * WAVES) void attention_partial_kernel(
    const half_t *__restrict__ q, const half_t *__restrict__ k, const half_t *__restrict__ v,
    half_t *__restrict__ k_cache, half_t *__restrict__ v_cache, int H, int Hkv, int Lmax, int pos,
    RopeTable tab, int chunk, std::conditional_t<WHOLE, half_t, float> *__restrict__ partial)
{
    __shared__ float qs[AD];                         // rotated query times 1/sqrt(D)
    __shared__ float ks[AD];                         // rotated key of the current token (fp32)
    __shared__ float wave_state[WAVES][AD + 2];
    // all pointer arguments fetched in one round (the compiler would otherwise fetch each where
    // it is first needed, one scalar-cache miss after the other)
    asm volatile("" ::"s"(q), "s"(k), "s"(v), "s"(k_cache), "s"(v_cache), "s"(partial), "s"(H), "s"(Hkv),
                 "s"(Lmax), "s"(pos), "s"(chunk));
    const int h = blockIdx.x, split = blockIdx.y;
    const int g_kv = h / (H / Hkv);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = lane >> 4, u = lane & 15;
    // what the rotary prologue needs (wave 0: the query, wave 1: the key; elements lane and
    // lane + 64), requested before the cache rows so that it is not waited for behind them
    const half_t *rsrc = wave == 1 ? k + (size_t)g_kv * AD : q + (size_t)h * AD;
    const half_t ra_h = rsrc[lane], rb_h = rsrc[lane + 64];
    const double rfreq = tab.inv_freq[lane];
    const int p0 = split * chunk, p1 = min(pos, p0 + chunk);             // rows of the caches
    const u32x4 *kbase = reinterpret_cast<const u32x4 *>(k_cache + (size_t)g_kv * Lmax * AD) + u;
    const u32x4 *vbase = reinterpret_cast<const u32x4 *>(v_cache + (size_t)g_kv * Lmax * AD) + u;
    const u32x4 vnow = reinterpret_cast<const u32x4 *>(v + (size_t)g_kv * AD)[u];
    // A wave takes BATCH x 4 positions at a time, STEP apart; one batch is folded in while the next one travels.  The first ones go
    // out before anything else: they do not depend on the query, and the rotary prologue below runs meanwhile.  WHOLE: one batch of
    // up to 512 positions.  A wave leaves out what is not there of its last batch, by a branch in front of a form without any for whole
    // batches; keys travel in front of the values, so that the scores are under way while the values come.  (Slices of 80 to 144 positions with the last batch
    // made up, keys and values in turn, and now, us: 24 / 24 heads at 1500 10.3 and 9.7, 40 / 40 at 1000 12.4 and 11.8, 48 / 24 at 1500 13.1 and 12.7; one
    // position at a time before the batches 9.7, 11.8 and 12.5, which 32 / 32 at 511 and 3000 took 8.1 and 15.3 for, now 7.4 and 14.5.)
    constexpr int BATCH = WHOLE ? 8 : 4, BUFFERS = WHOLE ? 1 : 2, STEP = 4 * WAVES;
    u32x4 kq[BUFFERS][BATCH], vq[BUFFERS][BATCH];
    const int first = p0 + 4 * wave;                                     // wave-uniform; lane group: + grp
    auto request_some = [&](u32x4 (&kr)[BATCH], u32x4 (&vr)[BATCH], int p, auto all) {
        // a row past the end reads the slice's first one and is ignored: a predicated load would be waited for on the spot
#pragma unroll
        for (int a = 0; a < BATCH; ++a) {
            if (!all && p + STEP * a >= p1) break;
            const int pa = p + STEP * a + grp;
            kr[a] = kbase[(size_t)(pa < p1 ? pa : p0) * (AD / 8)];
        }
#pragma unroll
        for (int a = 0; a < BATCH; ++a) {
            if (!all && p + STEP * a >= p1) break;
            const int pa = p + STEP * a + grp;
            vr[a] = vbase[(size_t)(pa < p1 ? pa : p0) * (AD / 8)];
        }
    };
    auto request = [&](u32x4 (&kr)[BATCH], u32x4 (&vr)[BATCH], int p) {
        if (p >= p1) return;                                             // wave-uniform
        if (!WHOLE && p + STEP * (BATCH - 1) < p1) request_some(kr, vr, p, std::true_type{});
        else request_some(kr, vr, p, std::false_type{});
    };
    request(kq[0], vq[0], first);
    if constexpr (!WHOLE) request(kq[BUFFERS - 1], vq[BUFFERS - 1], first + STEP * BATCH);

    {
        // every wave rotates what it fetched (all but the first two discard the result): a rotation
        // only some waves need would have its loads moved down behind the cache rows
        float lo, hi;
        rope_pair((float)ra_h, (float)rb_h, rfreq, pos, lo, hi);
        if (wave == 0) {
            qs[lane] = lo * 0.08838834764831845f;    // 1 / sqrt(128)
            qs[lane + 64] = hi * 0.08838834764831845f;
        } else if (wave == 1) {
            ks[lane] = lo;
            ks[lane + 64] = hi;
            // the first query head of a kv group (first slice) files the token into the caches
            if (split == 0 && h % (H / Hkv) == 0) {
                half_t *kd = k_cache + ((size_t)g_kv * Lmax + pos) * AD;
                half_t *vd = v_cache + ((size_t)g_kv * Lmax + pos) * AD;
                kd[lane] = (half_t)lo;
                kd[lane + 64] = (half_t)hi;
                vd[lane] = v[(size_t)g_kv * AD + lane];
                vd[lane + 64] = v[(size_t)g_kv * AD + lane + 64];
            }
        }
    }
    __syncthreads();

    float qf[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) qf[e] = qs[8 * u + e];
    Running r;
    r.m = -__builtin_inff();
    r.l = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) r.acc[e] = 0.f;

    auto dot = [&](const u32x4 &row) {
        const half8_t kh = __builtin_bit_cast(half8_t, row);
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) s = __builtin_fmaf(qf[e], (float)kh[e], s);
        return s;
    };
    // the token of this call, from the inputs, with its key in fp32: the initial state of one lane group.  (A score of -inf has the
    // weight 0; +inf gives NaN, as inf - inf does.)
    {
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) s = __builtin_fmaf(qf[e], ks[8 * u + e], s);
        s = row_sum(s);
        if (split == pos / chunk && wave == 0 && grp == 0 && s != -__builtin_inff()) {
            const half8_t vh = __builtin_bit_cast(half8_t, vnow);
            r.m = s;
            r.l = 1.f + (s - s);
#pragma unroll
            for (int e = 0; e < 8; ++e) r.acc[e] = (float)vh[e];
        }
    }
    auto fold_some = [&](const u32x4 (&kr)[BATCH], u32x4 (&vr)[BATCH], int p, auto all) {
        float s[BATCH], top = r.m;
#pragma unroll
        for (int a = 0; a < BATCH; ++a) {
            if (!all && p + STEP * a >= p1) break;
            s[a] = row_sum(dot(kr[a]));
        }
#pragma unroll
        for (int a = 0; a < BATCH; ++a) {
            if (!all && p + STEP * a >= p1) break;
            // a row past the end: weight 0, and values 0, because an infinity times 0 is NaN
            if (p + STEP * a + grp >= p1) {
                s[a] = -__builtin_inff();
                vr[a] = u32x4{0, 0, 0, 0};
            }
            top = fmaxf(top, s[a]);
        }
        const float zero = top == -__builtin_inff() ? 0.f : top;         // all scores so far -inf: all weights 0
        const float keep = __expf(r.m - zero);
        r.m = top;
        r.l *= keep;
#pragma unroll
        for (int e = 0; e < 8; ++e) r.acc[e] *= keep;
#pragma unroll
        for (int a = 0; a < BATCH; ++a) {
            if (!all && p + STEP * a >= p1) break;
            const float w = __expf(s[a] - zero);
            const half8_t vh = __builtin_bit_cast(half8_t, vr[a]);
            r.l += w;
#pragma unroll
            for (int e = 0; e < 8; ++e) r.acc[e] = __builtin_fmaf(w, (float)vh[e], r.acc[e]);
        }
    };
    auto fold = [&](const u32x4 (&kr)[BATCH], u32x4 (&vr)[BATCH], int p) {
        if (!WHOLE && p + STEP * (BATCH - 1) < p1) fold_some(kr, vr, p, std::true_type{});
        else fold_some(kr, vr, p, std::false_type{});
    };
    for (int p = first; p < p1; p += BUFFERS * STEP * BATCH) {
        fold(kq[0], vq[0], p);
        request(kq[0], vq[0], p + BUFFERS * STEP * BATCH);
        if constexpr (!WHOLE) {
            if (p + STEP * BATCH >= p1) break;
            fold(kq[BUFFERS - 1], vq[BUFFERS - 1], p + STEP * BATCH);
            request(kq[BUFFERS - 1], vq[BUFFERS - 1], p + 3 * STEP * BATCH);
        }
    }
    // the four groups of the wave (lanes u, u+16, u+32, u+48 hold the same dimensions)
#pragma unroll
    for (int d = 16; d <= 32; d <<= 1) {
        const float m2 = __shfl_xor(r.m, d), l2 = __shfl_xor(r.l, d);
        float a2[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) a2[e] = __shfl_xor(r.acc[e], d);
        merge(r, m2, l2, a2);
    }
    if (grp == 0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) wave_state[wave][8 * u + e] = r.acc[e];
        if (u == 0) {
            wave_state[wave][AD] = r.m;
            wave_state[wave][AD + 1] = r.l;
        }
    }
    __syncthreads();
    if (tid < AD) {
        float m = wave_state[0][AD];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) m = fmaxf(m, wave_state[w][AD]);
        float l = 0.f, a = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            const float mw = wave_state[w][AD];
            const float kf = mw == m ? 1.0f : __expf(mw - m);
            l += wave_state[w][AD + 1] * kf;
            a += wave_state[w][tid] * kf;
        }
        if constexpr (WHOLE) {
            partial[(size_t)h * AD + tid] = (half_t)(a / l);
        } else {
            float *dst = partial + ((size_t)h * gridDim.y + split) * (AD + 2);
            dst[tid] = a;
            if (tid == 0) {
                dst[AD] = m;
                dst[AD + 1] = l;
            }
        }
    }
}

// ---- grouped query heads ----------------------------------------------------------------------
// With G = H / Hkv > 2 query heads to a key/value head the kernel above reads every key and value G
// times (from L2) and spends G times the vector work on it: 26.8 us a call at 64 / 8 heads, 4000
// positions, for 16 MB of caches.  Here a workgroup serves up to 16 query heads of one kv head at once
// and both products run on the matrix cores:
//   scores   v_mfma_f32_16x16x32_f16, A = 16 keys from the cache, B = the rotated queries as the sum of three
//            halves (of the fp32 value times a power of two of the head's own; the third is what is left of it times
//            2^20): all 24 bits of every element down to 2^-31 of the head's largest, 2^-55 of that beyond;
//   values   v_mfma_f32_16x16x4_f32, fp32 probabilities and fp32 values: nothing is rounded to 16 bits.
// A score tile has lane (r, c) holding head r, positions 4 c + v: with step v of the value product
// taken over positions {v, 4 + v, 8 + v, 12 + v} that is its A operand as it stands, and its B operand
// is a contiguous piece of row 4 c + v if output column r of value tile t is dimension T r + t.
// Memory -> LDS loads bring blocks of 16 positions into a ring of the wave's own, up to three ahead; no
// barrier until the waves are merged.  The workspace has room for attention_splits() slices only,
// which at 64 heads are eight, 64 workgroups: so F workgroups of a slice (on one XCD, sharing its L2) take
// the same scores and 128 / F dimensions of the values each.  The current token enters as the initial state of
// one wave, with its key in fp32.  64 / 8 heads, 4000 positions:
// 26.8 -> 13.3 us a call with the merge (12.8 with two halves to a query, which left small elements beside a large
// one with fewer bits than fp32 has); what is left is a chain of latencies (arguments, small inputs 2 us,
// rotation 1 us, two rounds of cache rows, two merges), not the 16 MB.
typedef __attribute__((address_space(3))) void lds_void_t;
typedef const __attribute__((address_space(1))) void gbl_void_t;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ void dma16(const unsigned char *g, uint32_t lds_addr)
{
    __builtin_amdgcn_global_load_lds((gbl_void_t *)(uintptr_t)g, (lds_void_t *)(uintptr_t)lds_addr, 16, 0, 0);
}

constexpr int GQ_BLOCK = 16;                    // positions per step of a wave: one score tile (32: same time)
constexpr int GQ_WAVES = 8;                     // two to a SIMD: one's chain of dependent steps hides the other's
template <int F> struct GqShape {
    static constexpr int T = 8 / F;             // value tiles of 16 dimensions
    static constexpr int VROW = 256 / F;        // bytes of a value row this workgroup takes
    static constexpr int STAGE = GQ_BLOCK * (256 + VROW);
    static constexpr int STAGES = F == 1 ? 2 : 3;
    static constexpr int LOADS = 4 + 4 / F;     // per stage
    // 16 query rows (then their high halves), the token's key and value, the rotary table, the low halves, the
    // third ones, two numbers per head
    static constexpr int SHARED = 13 * 1024 + 128;
    static constexpr int LDS = SHARED + GQ_WAVES * STAGES * STAGE;
};

// one struct, so that the rotary table can be fetched from the kernel arguments by address
struct GroupedArgs {
    const half_t *q, *k, *v;
    half_t *k_cache, *v_cache;
    float *partial;
    int H, Hkv, qgroups, Lmax, pos, chunk, splits, pad;
    RopeTable tab;
};

// lane's piece of a value row: T halves
template <int F> struct GqValue;
template <> struct GqValue<1> { u32x4 d; };
template <> struct GqValue<2> { u32x2 d; };
template <> struct GqValue<4> { uint32_t d; };

template <int F>
__global__ __launch_bounds__(64 * GQ_WAVES, 1) void attention_grouped_kernel(const GroupedArgs A)
{
    extern __shared__ __align__(16) unsigned char smem[];
    typedef GqShape<F> Sh;
    constexpr int T = Sh::T;
    const int H = A.H, Hkv = A.Hkv, qgroups = A.qgroups, Lmax = A.Lmax, pos = A.pos, chunk = A.chunk, splits = A.splits;
    const half_t *__restrict__ q = A.q, *__restrict__ k = A.k, *__restrict__ v = A.v;
    half_t *__restrict__ k_cache = A.k_cache, *__restrict__ v_cache = A.v_cache;
    float *__restrict__ partial = A.partial;
    asm volatile("" ::"s"(q), "s"(k), "s"(v), "s"(k_cache), "s"(v_cache), "s"(partial), "s"(H), "s"(Hkv),
                 "s"(qgroups), "s"(Lmax), "s"(pos), "s"(chunk), "s"(splits));
    // block -> (XCD, place): the F workgroups of a slice are neighbours on one XCD
    const int place = (int)blockIdx.x >> 3;
    const int item = (place / F) * 8 + ((int)blockIdx.x & 7), f = place % F;
    if (item >= Hkv * qgroups * splits) return;
    const int split = item % splits, gq = item / splits;
    const int g_kv = gq / qgroups, G = H / Hkv, h0 = g_kv * G + (gq % qgroups) * 16;
    const int heads = min(16, G - (gq % qgroups) * 16);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, c = lane >> 4;

    const int p0 = split * chunk, p1 = min(pos, p0 + chunk);             // rows of the caches
    const int blocks = p1 > p0 ? (p1 - p0 + GQ_BLOCK - 1) / GQ_BLOCK : 0;
    const int mine = blocks > wave ? (blocks - wave + GQ_WAVES - 1) / GQ_WAVES : 0;
    const unsigned char *kb = reinterpret_cast<const unsigned char *>(k_cache + (size_t)g_kv * Lmax * AD);
    const unsigned char *vb = reinterpret_cast<const unsigned char *>(v_cache + (size_t)g_kv * Lmax * AD) + f * Sh::VROW;
    const uint32_t shared = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)smem);
    const uint32_t lds0 = shared + Sh::SHARED + wave * (Sh::STAGES * Sh::STAGE);

    // Block b of this wave.  Keys: rows of 256 bytes, the 16-byte chunk k of row i at place k ^ (i % 16) (the 16
    // rows a fragment read touches fall into 16 bank groups); values: rows of VROW bytes as they are.
    // Rows past the end repeat the last one and are masked; a wave without blocks fetches rows it never uses.
    const int last_row = max(p1 - 1, 0);
    auto request = [&](int b, int stage) {
        b = max(min(b, mine - 1), 0);                                    // past the end: a harmless repeat
        const int first = p0 + (wave + GQ_WAVES * b) * GQ_BLOCK;
        const uint32_t dst = lds0 + stage * Sh::STAGE;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 4 * i + c;
            dma16(kb + (size_t)min(first + row, last_row) * 256 + 16 * (r ^ row), dst + i * 1024);
        }
#pragma unroll
        for (int i = 0; i < 4 / F; ++i) {
            constexpr int per_row = Sh::VROW / 16;
            const int row = i * (64 / per_row) + lane / per_row;
            dma16(vb + (size_t)min(first + row, last_row) * 256 + 16 * (lane % per_row), dst + GQ_BLOCK * 256 + i * 1024);
        }
    };

    // The small inputs come the same way, first: a register load between the requests would be waited for
    // behind all of them.  Each wave fetches four query rows (a missing head repeats the last one; chunks
    // placed as the keys'), and all of them, alike: the token's key and value and the rotary table.
    {
        const int row = 4 * (wave & 3) + c;
        dma16(reinterpret_cast<const unsigned char *>(q + (size_t)(h0 + min(row, heads - 1)) * AD) + 16 * (r ^ row),
              shared + (wave & 3) * 1024);
        const unsigned char *args = (const unsigned char *)__builtin_amdgcn_kernarg_segment_ptr();
        const unsigned char *src = lane < 16 ? reinterpret_cast<const unsigned char *>(k + (size_t)g_kv * AD) + 16 * lane
                                 : lane < 32 ? reinterpret_cast<const unsigned char *>(v + (size_t)g_kv * AD) + 16 * (lane - 16)
                                             : args + offsetof(GroupedArgs, tab) + 16 * (lane - 32);
        dma16(src, shared + 4096);
    }
#pragma unroll
    for (int st = 0; st < Sh::STAGES; ++st) request(st, st);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(Sh::STAGES * Sh::LOADS) : "memory");
    __builtin_amdgcn_s_barrier();
    // Rotation: wave w takes heads 2 w and 2 w + 1, lane i the dimensions i and i + 64 (frequency i, as in
    // rope_pair), of the key as well.  The queries become three halves of q 2^-ex, ex from the head's largest
    // element (score = accumulators * unscale).
    const uint32_t qa = shared + 8 * wave * 64 + 2 * (lane & 7), sw = lane >> 3;     // element i of row 2 w: chunk i / 8
    uint32_t qe[2][2], ke[2], vraw;
    double rfreq;
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t row = 2 * wave + n;
            asm volatile("ds_read_u16 %0, %1" : "=v"(qe[n][h]) : "v"(qa + 256 * n + (((sw + 8 * h) ^ row) * 16)));
        }
#pragma unroll
    for (int h = 0; h < 2; ++h) asm volatile("ds_read_u16 %0, %1" : "=v"(ke[h]) : "v"(shared + 4096 + 2 * lane + 128 * h));
    asm volatile("ds_read_b32 %0, %1" : "=v"(vraw) : "v"(shared + 4352 + 4 * lane));
    asm volatile("ds_read_b64 %0, %1" : "=v"(rfreq) : "v"(shared + 4608 + 8 * lane));
    GqValue<F> vnow;                                                     // of the current token, this lane's columns
    {
        const uint32_t at = shared + 4352 + f * Sh::VROW + r * (2 * T);
        if constexpr (F == 1) asm volatile("ds_read_b128 %0, %1" : "=v"(vnow.d) : "v"(at));
        else if constexpr (F == 2) asm volatile("ds_read_b64 %0, %1" : "=v"(vnow.d) : "v"(at));
        else asm volatile("ds_read_b32 %0, %1" : "=v"(vnow.d) : "v"(at));
    }
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(qe[0][0]), "+v"(qe[0][1]), "+v"(qe[1][0]), "+v"(qe[1][1]), "+v"(ke[0]), "+v"(ke[1]), "+v"(vraw),
                   "+v"(rfreq), "+v"(vnow.d));
    auto half_of = [](const GqValue<F> &g, int t) {
        uint32_t w;
        if constexpr (F == 4) w = g.d;
        else w = g.d[t / 2];
        return (float)__builtin_bit_cast(half2_t, w)[t & 1];
    };
    auto f32 = [](uint32_t h) { return (float)__builtin_bit_cast(half_t, (uint16_t)h); };
    float sn, cs;
    {
        const double ang = (double)pos * rfreq;
        const double turns = __builtin_rint(ang * 0.15915494309189535);
        const float red = (float)(ang - turns * 6.283185307179586);
        sn = sinf(red);
        cs = cosf(red);
    }
    const float ka = f32(ke[0]), kz = f32(ke[1]);
    const float klo = ka * cs - kz * sn, khi = kz * cs + ka * sn;
    if (split == 0 && f == 0 && gq % qgroups == 0 && wave == 0) {        // files the token into the caches
        half_t *kd = k_cache + ((size_t)g_kv * Lmax + pos) * AD;
        kd[lane] = (half_t)klo;
        kd[lane + 64] = (half_t)khi;
        reinterpret_cast<uint32_t *>(v_cache + ((size_t)g_kv * Lmax + pos) * AD)[lane] = vraw;
    }
    float qlo_f[2], qhi_f[2], big[2], dot[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const float a = f32(qe[n][0]), z = f32(qe[n][1]);
        qlo_f[n] = a * cs - z * sn;
        qhi_f[n] = z * cs + a * sn;
        big[n] = fmaxf(__builtin_fabsf(qlo_f[n]), __builtin_fabsf(qhi_f[n]));
        dot[n] = qlo_f[n] * klo + qhi_f[n] * khi;
    }
#pragma unroll
    for (int d = 1; d <= 32; d <<= 1)
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            big[n] = fmaxf(big[n], __shfl_xor(big[n], d));
            dot[n] += __shfl_xor(dot[n], d);
        }
    // the raw query rows have been read by their wave: rows 2 w, 2 w + 1 of the high halves take their place,
    // the low and third halves follow at QLO and QREST, then (unscale, score) per head
    constexpr uint32_t QLO = 5 * 1024, QREST = 9 * 1024, HEAD = 13 * 1024;
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        int ex = 0;
        if (big[n] > 0.f && big[n] < __builtin_inff()) ex = ilogbf(big[n]) - 10;     // largest element in [2^10, 2^11)
        const uint32_t row = 2 * wave + n;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const float a = ldexpf(h ? qhi_f[n] : qlo_f[n], -ex);
            half_t top = (half_t)a, low = (half_t)(a - (float)top);
            const half_t rest = (half_t)((a - (float)top - (float)low) * 0x1p20f);
            // an element too small for the high half keeps its sign there, for keys that hold an infinity
            if (a != 0.f && top == (half_t)0.f) {
                top = (half_t)__builtin_copysignf(0x1p-24f, a);
                low = -top;
            }
            const uint32_t at = qa + 256 * n + (((sw + 8 * h) ^ row) * 16);
            asm volatile("ds_write_b16 %0, %1" ::"v"(at), "v"((uint32_t)__builtin_bit_cast(uint16_t, top)) : "memory");
            asm volatile("ds_write_b16 %0, %1" ::"v"(at + QLO), "v"((uint32_t)__builtin_bit_cast(uint16_t, low)) : "memory");
            asm volatile("ds_write_b16 %0, %1" ::"v"(at + QREST), "v"((uint32_t)__builtin_bit_cast(uint16_t, rest)) : "memory");
        }
        if (lane == 0) {
            const float unscale = ldexpf(0.08838834764831845f, ex), score = dot[n] * 0.08838834764831845f;   // 1 / sqrt(128)
            asm volatile("ds_write_b64 %0, %1" ::"v"(shared + HEAD + 8 * row),
                         "v"(u32x2{__builtin_bit_cast(uint32_t, unscale), __builtin_bit_cast(uint32_t, score)}) : "memory");
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    half8_t qhi[4], qlo[4], qrest[4];
    u32x2 head;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t at = shared + r * 256 + (((4 * j + c) ^ r) * 16);
        asm volatile("ds_read_b128 %0, %1" : "=v"(qhi[j]) : "v"(at));
        asm volatile("ds_read_b128 %0, %1" : "=v"(qlo[j]) : "v"(at + QLO));
        asm volatile("ds_read_b128 %0, %1" : "=v"(qrest[j]) : "v"(at + QREST));
    }
    asm volatile("ds_read_b64 %0, %1" : "=v"(head) : "v"(shared + HEAD + 8 * r));
    asm volatile("s_waitcnt lgkmcnt(0)"
                 : "+v"(qhi[0]), "+v"(qhi[1]), "+v"(qhi[2]), "+v"(qhi[3]), "+v"(qlo[0]), "+v"(qlo[1]), "+v"(qlo[2]),
                   "+v"(qlo[3]), "+v"(qrest[0]), "+v"(qrest[1]), "+v"(qrest[2]), "+v"(qrest[3]), "+v"(head));
    // (values, not elements: a bit_cast of a vector element reads element 0)
    const uint32_t head_unscale = head[0], head_score = head[1];
    const float unscale = __builtin_bit_cast(float, head_unscale), now = __builtin_bit_cast(float, head_score);

    // state of head r (m and l; l per lane, added over c at the end) and sums of heads 4 c + v, dimension T r + t
    float m = -__builtin_inff(), l = 0.f;
    floatx4 acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    // (a score of -inf has the weight 0: the state stays empty; +inf gives NaN, as inf - inf does)
    if (wave == 0 && split == pos / chunk && now != -__builtin_inff()) {
        m = now;
        l = c == 0 ? 1.f + (now - now) : 0.f;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const float vt = half_of(vnow, t);
            acc[t] = floatx4{vt, vt, vt, vt};
        }
    }

    uint32_t kofs[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) kofs[j] = r * 256 + (((4 * j + c) ^ r) * 16);
    int stage = 0;
    for (int b = 0; b < mine; ++b) {
        // loads complete in order: this block is there when only the later stages' are outstanding (other loads
        // of this wave that were issued in between only make the wait longer)
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((Sh::STAGES - 1) * Sh::LOADS) : "memory");
        const uint32_t base = lds0 + stage * Sh::STAGE;
        u32x4 kf[4];
        GqValue<F> vv[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) asm volatile("ds_read_b128 %0, %1" : "=v"(kf[j]) : "v"(base + kofs[j]));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t at = base + GQ_BLOCK * 256 + (4 * c + i) * Sh::VROW + r * (2 * T);
            if constexpr (F == 1) asm volatile("ds_read_b128 %0, %1" : "=v"(vv[i].d) : "v"(at));
            else if constexpr (F == 2) asm volatile("ds_read_b64 %0, %1" : "=v"(vv[i].d) : "v"(at));
            else asm volatile("ds_read_b32 %0, %1" : "=v"(vv[i].d) : "v"(at));
        }
        asm volatile("s_waitcnt lgkmcnt(0)"
                     : "+v"(kf[0]), "+v"(kf[1]), "+v"(kf[2]), "+v"(kf[3]), "+v"(vv[0].d), "+v"(vv[1].d), "+v"(vv[2].d),
                       "+v"(vv[3].d));
        request(b + Sh::STAGES, stage);                                  // the stage has been read
        stage = stage + 1 == Sh::STAGES ? 0 : stage + 1;

        const int first = p0 + (wave + GQ_WAVES * b) * GQ_BLOCK + 4 * c;
        // rows past the end have the weight 0, and an infinity times 0 is NaN: their values become 0
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (first + i >= p1) vv[i].d = decltype(vv[i].d){};
        floatx4 hi = {0.f, 0.f, 0.f, 0.f}, lo = {0.f, 0.f, 0.f, 0.f}, rest = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const half8_t kv = __builtin_bit_cast(half8_t, kf[j]);
            rest = __builtin_amdgcn_mfma_f32_16x16x32_f16(kv, qrest[j], rest, 0, 0, 0);
            lo = __builtin_amdgcn_mfma_f32_16x16x32_f16(kv, qlo[j], lo, 0, 0, 0);
            hi = __builtin_amdgcn_mfma_f32_16x16x32_f16(kv, qhi[j], hi, 0, 0, 0);
        }
        float s[4], top = -__builtin_inff();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // a key with an infinity: the high halves alone have the sign; Inf times a low half of 0 or of the other
            // sign would make it NaN
            const float all = __builtin_fabsf(hi[i]) < __builtin_inff() ? hi[i] + (lo[i] + rest[i] * 0x1p-20f) : hi[i];
            s[i] = first + i < p1 ? all * unscale : -__builtin_inff();
            top = fmaxf(top, s[i]);
        }
        top = fmaxf(top, __shfl_xor(top, 16));
        top = fmaxf(top, __shfl_xor(top, 32));
        const float m_new = fmaxf(m, top);
        const float zero = m_new == -__builtin_inff() ? 0.f : m_new;     // all scores so far -inf: all weights 0
        const float keep = __expf(m - zero);
        m = m_new;
        l *= keep;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            s[i] = __expf(s[i] - zero);
            l += s[i];
        }
        if (__any(keep != 1.0f)) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float ki = __shfl(keep, 4 * c + i);
#pragma unroll
                for (int t = 0; t < T; ++t) acc[t][i] *= ki;
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int t = 0; t < T; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(s[i], half_of(vv[i], t), acc[t], 0, 0, 0);
    }
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);

    // merge the waves: [wave][head][dimensions, m, l]
    constexpr int DW = AD / F, ROW = DW + 2;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    float *state = reinterpret_cast<float *>(smem);
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) state[(wave * 16 + 4 * c + i) * ROW + T * r + t] = acc[t][i];
    if (c == 0) {
        state[(wave * 16 + r) * ROW + DW] = m;
        state[(wave * 16 + r) * ROW + DW + 1] = l;
    }
    __syncthreads();
    for (int e = tid; e < heads * DW; e += 64 * GQ_WAVES) {
        const int h = e / DW, d = e - h * DW;
        float mm = state[h * ROW + DW];
#pragma unroll
        for (int w = 1; w < GQ_WAVES; ++w) mm = fmaxf(mm, state[(w * 16 + h) * ROW + DW]);
        float ll = 0.f, a = 0.f;
#pragma unroll
        for (int w = 0; w < GQ_WAVES; ++w) {
            const float mw = state[(w * 16 + h) * ROW + DW];
            const float kf = mw == mm ? 1.0f : __expf(mw - mm);
            ll += state[(w * 16 + h) * ROW + DW + 1] * kf;
            a += state[(w * 16 + h) * ROW + d] * kf;
        }
        float *dst = partial + ((size_t)(h0 + h) * splits + split) * (AD + 2);
        dst[f * DW + d] = a;
        if (f == 0 && d == 0) {
            dst[AD] = mm;
            dst[AD + 1] = ll;
        }
    }
}

template <int F>
int attention_grouped_launch(const GroupedArgs &A, hipStream_t stream)
{
    static_assert(GqShape<F>::LDS <= 160 * 1024 && GQ_WAVES * 16 * (AD / F + 2) * 4 <= GqShape<F>::LDS, "LDS");
    static AwqOncePerDevice once;
    std::atomic<bool> &attr_set = once.here();
    if (!attr_set.load(std::memory_order_relaxed)) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(attention_grouped_kernel<F>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, GqShape<F>::LDS) != hipSuccess)
            return AWQ_ERR_HIP;
        attr_set.store(true, std::memory_order_relaxed);
    }
    const int64_t items = (int64_t)A.Hkv * A.qgroups * A.splits;
    attention_grouped_kernel<F><<<dim3((unsigned)((items + 7) / 8 * 8 * F)), dim3(64 * GQ_WAVES), GqShape<F>::LDS, stream>>>(A);
    return awq_launch_status();
}

// grid H, 256 threads: merge up to 16 slices of a head in a fixed order.  The head's partial results
// (at most 16 x 130 floats) are first copied to LDS with coalesced loads: read one by one from
// memory they would be a chain of dependent round trips.
constexpr int MERGE_LOOP_SLICES = 16, MERGE_LOOP_LOADS = 9;
static_assert(MERGE_LOOP_SLICES * (AD + 2) <= 256 * MERGE_LOOP_LOADS, "one round of loads");
__global__ __launch_bounds__(256) void attention_merge_kernel(const float *__restrict__ partial,
                                                              int splits, half_t *__restrict__ out)
{
    __shared__ float ps[MERGE_LOOP_SLICES * (AD + 2)];
    const int h = blockIdx.x, t = threadIdx.x;
    const float *p = partial + (size_t)h * splits * (AD + 2);
    asm volatile("" ::"s"(partial), "s"(splits), "s"(out));       // arguments in one round
    const int n = splits * (AD + 2);
    float tmp[MERGE_LOOP_LOADS];                                  // in flight together
#pragma unroll
    for (int e = 0; e < MERGE_LOOP_LOADS; ++e) {
        const int i = 256 * e + t;
        tmp[e] = p[i < n ? i : n - 1];
    }
#pragma unroll
    for (int e = 0; e < MERGE_LOOP_LOADS; ++e) {
        const int i = 256 * e + t;
        if (i < n) ps[i] = tmp[e];
    }
    __syncthreads();
    if (t >= AD) return;
    float m = -__builtin_inff();
    for (int s = 0; s < splits; ++s) m = fmaxf(m, ps[s * (AD + 2) + AD]);
    float l = 0.f, a = 0.f;
    for (int s = 0; s < splits; ++s) {
        const float ms = ps[s * (AD + 2) + AD];
        const float kf = ms == m ? 1.0f : __expf(ms - m);
        l += ps[s * (AD + 2) + AD + 1] * kf;
        a += ps[s * (AD + 2) + t] * kf;
    }
    out[(size_t)h * AD + t] = (half_t)(a / l);
}

// The same for more than 16 slices, where the loops above are what takes the time.  Wave w takes slices w, w + 4, ..., a pair of
// dimensions per lane, and every wave the maxima and sums of all slices, one per lane, everything requested in one round.
// Maximum and sum are shuffles, the weight of a slice is one lane's exponential, and the four waves meet in LDS once.  us a call from
// a graph, above and here: 8 heads at 17, 21, 32, 47 and 63 slices 7.3 / 7.2, 8.6 / 7.6, 8.7 / 7.8, 11.0 / 8.8, 12.2 / 9.2; 30 heads
// at 17 and 18 9.3 / 9.1, 10.3 / 9.5.  (Only rows that are there are requested: with the last one again in the place of the others
// it was slower than above by up to 11 % where heads are no multiple of 8, whose slices lie in other L2s.)  At 8 and 16
// slices the twelve dependent shuffles cost more than the loops (measured with those repeats: 13.3 -> 13.8 and 12.0 -> 12.8 us; by
// DPP instead 13.5 and 12.6), so those stay with the kernel above.
constexpr int MERGE_WAVES = 4, MERGE_ROWS = 16;
__global__ __launch_bounds__(64 * MERGE_WAVES) void attention_merge_many_kernel(const float *__restrict__ partial,
                                                                                int splits, half_t *__restrict__ out)
{
    __shared__ float2 sums[MERGE_WAVES][64];
    asm volatile("" ::"s"(partial), "s"(splits), "s"(out));       // arguments in one round
    const int h = blockIdx.x, lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float *p = partial + (size_t)h * splits * (AD + 2);
    const float2 state = *reinterpret_cast<const float2 *>(p + min(lane, splits - 1) * (AD + 2) + AD);
    float2 row[MERGE_ROWS];
#pragma unroll
    for (int i = 0; i < MERGE_ROWS; ++i)
        if (wave + MERGE_WAVES * i < splits)
            row[i] = *reinterpret_cast<const float2 *>(p + (wave + MERGE_WAVES * i) * (AD + 2) + 2 * lane);
    float m = state.x;
#pragma unroll
    for (int d = 1; d <= 32; d <<= 1) m = fmaxf(m, __shfl_xor(m, d));
    const float weight = state.x == m ? 1.0f : __expf(state.x - m);
    float l = lane < splits ? state.y * weight : 0.f;
#pragma unroll
    for (int d = 1; d <= 32; d <<= 1) l += __shfl_xor(l, d);
    float2 a = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < MERGE_ROWS; ++i) {
        const int s = wave + MERGE_WAVES * i;
        if (s < splits) {
            const float w = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, weight), s));
            a.x += row[i].x * w;
            a.y += row[i].y * w;
        }
    }
    sums[wave][lane] = a;
    __syncthreads();
    if (wave != 0) return;
#pragma unroll
    for (int w = 1; w < MERGE_WAVES; ++w) {
        const float2 b = sums[w][lane];
        a.x += b.x;
        a.y += b.y;
    }
    reinterpret_cast<half2_t *>(out + (size_t)h * AD)[lane] = half2_t{(half_t)(a.x / l), (half_t)(a.y / l)};
}

int attention_splits(int64_t H, int64_t L)
{
    // about two workgroups per CU (the best of 256, 512 and 1024 at 32 heads x 2048 positions),
    // at least 64 positions each
    int64_t s = (512 + H - 1) / H;
    const int64_t most = (L + 63) / 64;
    if (s > most) s = most;
    if (s < 1) s = 1;
    if (s > 64) s = 64;
    return (int)s;
}

// Which kernel takes G = H / Hkv > 2 query heads to a kv head.  The grouped one starts slower (1.3 to 2 us: twice the
// threads, its inputs through LDS, two barriers) and then reads every cache row for up to 16 heads at once; the
// other one's time grows with the rows that all heads read.  The line is where the two met over 17 pairs of
// H and Hkv, 3 <= G <= 48, at 0 to 16000 positions (graph replays): H * L of 17 to 20 thousand for G of 5 to 9, 30 to 42 for 4
// and for 16 and more, 67 to 110 for 3, whose tiles are mostly empty.  us, vector and grouped: 64 / 8 heads at 100 positions 7.2 / 8.4, 300
// 9.1 / 8.7, 1000 11.7 / 9.3; 128 / 32 at 300 10.0 / 10.1, 500 11.8 / 10.4; 24 / 8 at 1500 10.9 / 12.8, 6000 18.5 / 16.9.
bool attention_grouped(int64_t H, int64_t Hkv, int64_t L)
{
    const int64_t G = H / Hkv;
    return H * L >= (G < 4 ? 110000 : G > 4 && G < 10 ? 20000 : 42000);
}

// Whether one workgroup takes a head's whole context, in one launch: up to 320 positions.  us a call from a graph, two launches and one, 8 / 8,
// 32 / 32 and 64 / 8 heads: 100 positions 6.2 / 6.5 / 6.6 and 5.3 / 5.5 / 5.4, 200 6.6 / 6.6 / 8.2 and 6.0 / 6.2 / 7.1, 300 6.7 / 7.5 / 8.9 and
// 6.7 / 7.4 / 8.1, 400 6.8 / 8.2 / 9.0 and 7.4 / 8.3 / 9.2 (an eager caller saves a launch besides).  Such a workgroup fills a CU: more than 256 heads
// are a second round (272 / 17 heads at 100 and 300 positions 8.7 / 9.4 and 10.2 / 13.9, 1024 / 64 9.1 / 11.3 and 19.0 / 31.0; 256 / 256
// 9.6 / 13.4 and 7.7 / 12.0).  Each reads its kv head's rows for itself: with nearly as many heads and 16 kv heads and more, shared by more than two heads
// each, the grouped kernel is even from 210 positions (256 / 32 at 190 / 210 / 300 8.9 / 8.9 / 9.9 and 8.8 / 9.1 / 11.2, 192 / 16 at 255 / 319 even).
bool attention_whole(int64_t H, int64_t Hkv, int64_t L)
{
    return L <= 320 && H <= 256 && (H <= 192 || Hkv < 16 || H / Hkv <= 2 || L <= 200);
}

}  // namespace

extern "C" size_t awq_decode_attention_workspace_bytes(int64_t H, int64_t D, int64_t L)
{
    if (H <= 0 || D != AD || L <= 0) return 0;
    return (size_t)H * attention_splits(H, L) * (AD + 2) * sizeof(float);
}

extern "C" int awq_decode_attention(const void *q_f16, const void *k_f16, const void *v_f16,
                                    void *k_cache_f16, void *v_cache_f16, int64_t H, int64_t Hkv,
                                    int64_t D, int64_t Lmax, int64_t pos, float rope_theta,
                                    void *out_f16, void *workspace, size_t workspace_bytes,
                                    void *stream)
{
    if (!q_f16 || !k_f16 || !v_f16 || !k_cache_f16 || !v_cache_f16 || !out_f16 || !workspace)
        return AWQ_ERR_NULL_POINTER;
    if (D != AD || H <= 0 || Hkv <= 0 || H % Hkv != 0 || H > 65535 || Lmax <= 0 || Lmax > (int64_t)1 << 24 ||
        pos < 0 || pos >= Lmax)
        return AWQ_ERR_BAD_SHAPE;
    if (!(rope_theta > 1.0f)) return AWQ_ERR_BAD_ARGUMENT;
    if (!awq_aligned16(q_f16) || !awq_aligned16(k_f16) || !awq_aligned16(v_f16) ||
        !awq_aligned16(k_cache_f16) || !awq_aligned16(v_cache_f16) || !awq_aligned16(out_f16) ||
        !awq_aligned16(workspace))
        return AWQ_ERR_MISALIGNED;
    const int64_t L = pos + 1;
    if (workspace_bytes < awq_decode_attention_workspace_bytes(H, D, L)) return AWQ_ERR_WORKSPACE_TOO_SMALL;
    const int splits = attention_splits(H, L);
    int chunk = (int)((L + splits - 1) / splits);
    chunk = (chunk + 15) / 16 * 16;                  // whole steps of the four waves
    RopeTable tab;
    // products of 16 powers (one rounding of 2^-53 more) instead of 64: 1.1 us of the host's 6.6 for a call of two launches
    double coarse[8], fine[8];
    for (int i = 0; i < 8; ++i) {
        coarse[i] = pow((double)rope_theta, -16.0 * i / AD);
        fine[i] = pow((double)rope_theta, -2.0 * i / AD);
    }
    for (int i = 0; i < AD / 2; ++i) tab.inv_freq[i] = coarse[i / 8] * fine[i % 8];
    const half_t *qp = (const half_t *)q_f16, *kp = (const half_t *)k_f16, *vp = (const half_t *)v_f16;
    half_t *kc = (half_t *)k_cache_f16, *vc = (half_t *)v_cache_f16;
    float *partial = (float *)workspace;
    int st;
    const int forced = awq_knob("AWQ_ATTENTION_F", -1);      // (the tuning build: the kernel below, 0, or the number of workgroups to a slice)
    const int whole = awq_knob("AWQ_ATTENTION_WHOLE", -1);   // (the largest L of one launch)
    if (forced < 0 && (whole < 0 ? attention_whole(H, Hkv, L) : L <= whole)) {
        attention_partial_kernel<ATT_WHOLE_WAVES, true><<<dim3((unsigned)H, 1), dim3(64 * ATT_WHOLE_WAVES), 0, (hipStream_t)stream>>>(
            qp, kp, vp, kc, vc, (int)H, (int)Hkv, (int)Lmax, (int)pos, tab, (int)L, (half_t *)out_f16);
        return awq_launch_status();
    }
    if (H / Hkv > 2 && (forced < 0 ? attention_grouped(H, Hkv, L) : forced > 0)) {
        GroupedArgs A = {qp, kp, vp, kc, vc, partial, (int)H, (int)Hkv, (int)((H / Hkv + 15) / 16), (int)Lmax, (int)pos,
                         chunk, splits, 0, tab};
        // One workgroup per CU (the LDS): the values are divided as long as all workgroups run at once.  24 / 8 heads, 1500
        // positions, 176 items: 12.8 us undivided, 16.5 in two, 19.9 in four; 128 / 32, 700, 128 items: 12.8, 11.6, 15.9
        const int64_t items = Hkv * A.qgroups * splits;
        const int F = forced > 0 ? forced : items <= 64 ? 4 : items <= 128 ? 2 : 1;
        st = F == 1 ? attention_grouped_launch<1>(A, (hipStream_t)stream)
             : F == 2 ? attention_grouped_launch<2>(A, (hipStream_t)stream)
                      : attention_grouped_launch<4>(A, (hipStream_t)stream);
    } else {
        attention_partial_kernel<ATT_WAVES, false><<<dim3((unsigned)H, (unsigned)splits), dim3(64 * ATT_WAVES), 0, (hipStream_t)stream>>>(
            qp, kp, vp, kc, vc, (int)H, (int)Hkv, (int)Lmax, (int)pos, tab, chunk, partial);
        st = awq_launch_status();
    }
    if (st != AWQ_OK) return st;
    if (splits > MERGE_LOOP_SLICES)                  // (at most 64: attention_splits)
        attention_merge_many_kernel<<<dim3((unsigned)H), dim3(64 * MERGE_WAVES), 0, (hipStream_t)stream>>>(
            (const float *)workspace, splits, (half_t *)out_f16);
    else
        attention_merge_kernel<<<dim3((unsigned)H), dim3(256), 0, (hipStream_t)stream>>>(
            (const float *)workspace, splits, (half_t *)out_f16);
    return awq_launch_status();
}
