/*
 * Readback and upload (wkv_state, wkv_load) as a C caller sees them that stands between libwkv and the HIP runtime: this
 * program's own hipHostMalloc, hipMalloc and hipEventSynchronize are the ones the library calls (the symbols of an executable come first).
 *   - All pinned memory is asked for as coherent: the host rewrites a slot, and reads one, while kernels of the same call still run.
 *   - A call that finds the kept memory lent to another thread's call gets memory of its own, of the same kind.
 *   - Without pinned memory both calls work all the same; without device memory either they say so, and the cache is what it was.
 * Prints "pinned ok" and exits 0 on success.
 */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>
#include <pthread.h>
#include <semaphore.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include "../../include/wkv.h"

#define HIP(x) do { hipError_t e_ = (x); if (e_ != hipSuccess) { printf("hip: %s (line %d)\n", hipGetErrorString(e_), __LINE__); exit(2); } } while (0)
#define WKV(x) do { int r_ = (x); if (r_ != WKV_OK) { printf("wkv: %d %s (line %d)\n", r_, wkv_last_error(), __LINE__); exit(3); } } while (0)
#define CHECK(c) do { if (!(c)) { printf("check failed: %s (line %d)\n", #c, __LINE__); exit(4); } } while (0)

static int host_calls, host_flags_differ, refuse_host, refuse_device;
hipError_t hipHostMalloc(void** p, size_t n, unsigned flags)
{
    static hipError_t (*next)(void**, size_t, unsigned);
    if (!next) next = (hipError_t (*)(void**, size_t, unsigned))dlsym(RTLD_NEXT, "hipHostMalloc");
    ++host_calls;
    if (refuse_host) return hipErrorOutOfMemory;
    if (flags != (hipHostMallocPortable | hipHostMallocCoherent)) { ++host_flags_differ; printf("hipHostMalloc with flags 0x%x\n", flags); }
    return next(p, n, flags);
}

hipError_t hipMalloc(void** p, size_t n)
{
    static hipError_t (*next)(void**, size_t);
    if (!next) next = (hipError_t (*)(void**, size_t))dlsym(RTLD_NEXT, "hipMalloc");
    return refuse_device ? hipErrorOutOfMemory : next(p, n);
}

/* A thread that has `held` set stops in its first wait for an event until it is let go. */
static __thread int held;
static sem_t inside, go;
hipError_t hipEventSynchronize(hipEvent_t e)
{
    static hipError_t (*next)(hipEvent_t);
    if (!next) next = (hipError_t (*)(hipEvent_t))dlsym(RTLD_NEXT, "hipEventSynchronize");
    if (held) { held = 0; sem_post(&inside); sem_wait(&go); }
    return next(e);
}

/* 16 units x 700 slots of 256 bytes: several chunks a matrix, more than there are slots for; `seed` makes it another state */
#define UNITS 16
#define D 64
#define M 700
#define TOKENS 2000
static float K[2][UNITS * M * D], V[2][UNITS * M * D], back[2][UNITS * M * D];
static double A[2][UNITS * M];
static int32_t P[2][UNITS * M];

static void make(int i, unsigned seed)
{
    for (size_t j = 0; j < (size_t)UNITS * M * D; ++j) {
        seed = seed * 1664525u + 1013904223u;
        K[i][j] = (float)(int)seed;
        V[i][j] = (float)(int)(seed ^ 0x5bd1e995u);
    }
    for (int u = 0; u < UNITS; ++u)
        for (int l = 0; l < M; ++l) {
            P[i][u * M + l] = l < M - 1 ? 2 * l + (u + l + i) % 2 : TOKENS - 1;
            A[i][u * M + l] = 1.0 + l + 1000.0 * u + i;
        }
}

static void expect(wkv_handle* h, int i)
{
    static double a[2][UNITS * M];
    static int32_t p[2][UNITS * M];
    int64_t tokens = 0;
    WKV(wkv_state(h, WKV_STEP, &tokens, sizeof tokens));
    CHECK(tokens == TOKENS);
    WKV(wkv_state(h, WKV_K, back[i], sizeof back[i]));
    CHECK(memcmp(back[i], K[i], sizeof K[i]) == 0);
    WKV(wkv_state(h, WKV_V, back[i], sizeof back[i]));
    CHECK(memcmp(back[i], V[i], sizeof V[i]) == 0);
    WKV(wkv_state(h, WKV_SCORE_SUM, a[i], sizeof a[i]));
    CHECK(memcmp(a[i], A[i], sizeof A[i]) == 0);
    WKV(wkv_state(h, WKV_POS, p[i], sizeof p[i]));
    CHECK(memcmp(p[i], P[i], sizeof P[i]) == 0);
}

static void* hold(void* handle)
{
    held = 1;
    expect((wkv_handle*)handle, 0);
    return NULL;
}

int main(void)
{
    wkv_handle *h = NULL, *other = NULL;
    make(0, 1u);
    make(1, 2u);
    HIP(hipSetDevice(0));

    /* no pinned memory: nothing is kept from these calls */
    refuse_host = 1;
    WKV(wkv_create(&h, 1, UNITS, D, M, 9, WKV_FP32));
    WKV(wkv_load(h, TOKENS, M, K[0], V[0], A[0], P[0]));
    expect(h, 0);
    CHECK(host_calls > 0);
    refuse_device = 1;
    CHECK(wkv_load(h, TOKENS, M, K[1], V[1], A[1], P[1]) == WKV_ENOMEM);
    CHECK(wkv_state(h, WKV_K, back[0], sizeof back[0]) == WKV_ENOMEM);
    refuse_host = refuse_device = 0;
    host_calls = 0;
    expect(h, 0);
    WKV(wkv_destroy(h));
    host_calls = 0;

    WKV(wkv_create(&h, 1, UNITS, D, M, 9, WKV_FP32));
    WKV(wkv_create(&other, 1, UNITS, D, M, 9, WKV_FP32));
    WKV(wkv_load(h, TOKENS, M, K[0], V[0], A[0], P[0]));
    WKV(wkv_load(other, TOKENS, M, K[1], V[1], A[1], P[1]));
    expect(h, 0);
    expect(other, 1);
    CHECK(host_calls == 1);                                 /* kept from the first call on */

    /* one thread inside a readback, another one with a load and readbacks of its own meanwhile */
    pthread_t thread;
    sem_init(&inside, 0, 0);
    sem_init(&go, 0, 0);
    CHECK(pthread_create(&thread, NULL, hold, h) == 0);
    sem_wait(&inside);
    make(1, 3u);
    WKV(wkv_load(other, TOKENS, M, K[1], V[1], A[1], P[1]));
    expect(other, 1);
    CHECK(host_calls > 1);
    sem_post(&go);
    pthread_join(thread, NULL);
    CHECK(host_flags_differ == 0);

    WKV(wkv_destroy(h));
    WKV(wkv_destroy(other));
    printf("pinned ok\n");
    return 0;
}
