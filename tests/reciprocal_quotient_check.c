/* Exhaustive check of the claim behind the scale search's division of activations: with y = fl(1 / s), the correctly rounded
 * reciprocal,
 *     q0 = fl(x y),  e = fma(-q0, s, x),  q = fma(e, y, q0)
 * is fl(x / s) for every fp16 significand x and every binary32 significand s.  (Scaling either by a power of two scales every
 * step exactly as long as nothing underflows or overflows; e, the smallest number that occurs, is at least 2^-48 |x|.)
 * Prints the number of pairs checked and of mismatches; argv: threads, and a step through the significands of s (1: all;
 * without fused multiply-adds in hardware every 257th).  NO_CORRECTION leaves the last two operations out. */
#include <math.h>
#include <pthread.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

static int threads;
static uint32_t step;

static void *part(void *arg)
{
    const int t = (int)(intptr_t)arg;
    uint64_t bad = 0;
    for (uint32_t m = (uint32_t)t * step; m < 1u << 23; m += step * (uint32_t)threads) {
        const uint32_t bits = 0x3F800000u | m;
        float s;
        memcpy(&s, &bits, 4);
        const float y = 1.0f / s;
        uint32_t wrong = 0;
        for (int a = 1024; a < 2048; ++a) {
            const float x = (float)a;
            const float q0 = x * y;
            const float e = fmaf(-q0, s, x);
#ifdef NO_CORRECTION
            const float q = q0 + 0.0f * e;
#else
            const float q = fmaf(e, y, q0);
#endif
            wrong += q != x / s;
        }
        bad += wrong;
    }
    return (void *)(uintptr_t)bad;
}

int main(int argc, char **argv)
{
    threads = argc > 1 ? atoi(argv[1]) : 1;
    step = argc > 2 ? (uint32_t)atoi(argv[2]) : 1u;
#ifndef __FP_FAST_FMAF
    if (step == 1) step = 257;
#endif
    if (threads < 1 || threads > 64 || step < 1) return 2;
    pthread_t id[64];
    uint64_t bad = 0;
    for (int t = 0; t < threads; ++t)
        if (pthread_create(&id[t], NULL, part, (void *)(intptr_t)t)) return 2;
    for (int t = 0; t < threads; ++t) {
        void *r;
        pthread_join(id[t], &r);
        bad += (uint64_t)(uintptr_t)r;
    }
    printf("%llu pairs, %llu mismatches\n", (unsigned long long)(((1u << 23) + step - 1) / step) * 1024ull, (unsigned long long)bad);
    return bad != 0;
}
