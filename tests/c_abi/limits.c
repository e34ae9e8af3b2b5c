/*
 * A kernel's limit of dynamic workgroup memory belongs to the process, not to a handle: creating a handle must not lower it for one
 * that was there before.  This program's own hipFuncSetAttribute is the one libwkv calls (the symbols of an executable come first).
 * Prints "limits ok" and exits 0 on success.
 */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>
#include <stdio.h>
#include <string.h>

#include "../../include/wkv.h"

static struct { const void* f; int bytes; } seen[256];
static int kernels, lowered;
hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute what, int value)
{
    static hipError_t (*next)(const void*, hipFuncAttribute, int);
    if (!next) next = (hipError_t (*)(const void*, hipFuncAttribute, int))dlsym(RTLD_NEXT, "hipFuncSetAttribute");
    if (what == hipFuncAttributeMaxDynamicSharedMemorySize) {
        int i = 0;
        while (i < kernels && seen[i].f != f) ++i;
        if (i < kernels && value < seen[i].bytes) { ++lowered; printf("a limit of %d bytes is lowered to %d\n", seen[i].bytes, value); }
        if (i == kernels && kernels < 256) seen[kernels++].f = f;
        if (i < kernels) seen[i].bytes = value;
    }
    return next(f, what, value);
}

int main(void)
{
    const int budgets[] = { 4095, 3000, 300, 2500 }, splits[] = { 1, 4 };
    for (int s = 0; s < 2; ++s) {
        wkv_handle* h[4] = { 0 };
        for (int i = 0; i < 4; ++i) {
            wkv_options o;
            memset(&o, 0, sizeof o);
            o.batch = 1; o.heads = 2; o.head_dim = 128; o.budget = budgets[i]; o.recent_window = 8; o.dtype = WKV_FP16; o.split = splits[s];
            if (wkv_create_ex(&h[i], &o) != WKV_OK) { printf("wkv: %s\n", wkv_last_error()); return 3; }
        }
        for (int i = 0; i < 4; ++i) wkv_destroy(h[i]);
    }
    if (kernels == 0) { printf("no limit was set\n"); return 4; }
    if (lowered) return 5;
    printf("limits ok\n");
    return 0;
}
