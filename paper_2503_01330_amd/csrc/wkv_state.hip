// Readback and upload of a cache, gfx950: slots in token order to and from memory that host and GPU share.
//
// A slot's place in token order is the number of live slots of its unit with an older token.  That is counted, not
// sorted: a workgroup has the unit's token indices in LDS, and a wave counts for 16 rows at once (one LDS read, 16 compares a
// lane and 64 slots), which is nothing beside moving the rows over the host link, needs no scratch, and holds for any order of slots.  The rows
// go straight into pinned host memory, and from there into the caller's arrays while the next units' are on their way.
// Measured (16 units x 700 slots of 512 bytes, 5.7 MB a matrix): reading K 600 -> 232 us, score sums 70 -> 24, loading 565 -> 380;
// before, pageable copies, a sort of every unit for every item and a gather on the host.  What bounds reading is what kernels write over the host link, 27 GB/s
// whatever the launch (16 to 64 rows a workgroup, non-temporal stores: 231-246 us).  The copy engine does 53, but a gather into device memory and chunked copies
// from there took 284 to 395 us: each hand-over from a kernel or copy to the next costs more than the chunk gains.
#include "../../include/wkv.h"
#include "wkv_internal.h"
#include "wkv_device.h"

namespace {

constexpr int ROWS = 64, NT = 256;        // rows a workgroup moves, its threads

__device__ __forceinline__ void load_positions(const int32_t* pos, int len, int32_t* lds) {
    for (int i = threadIdx.x; i < len; i += NT) lds[i] = pos[i];
    __syncthreads();
}

// The places of PER slots from `first` on, which a wave counts together: lane r < PER ends with that of slot first + r, and with the newest
// older token (-1: none) if that is asked for.
constexpr int PER = ROWS / (NT / 64);
template <bool BEFORE>
__device__ __forceinline__ int count_places(const int32_t* position, int first, int len, int lane, int* newest_older) {
    int mine[PER], older[PER], before[PER], place = 0;
#pragma unroll
    for (int r = 0; r < PER; ++r) { mine[r] = position[min(first + r, len - 1)]; older[r] = 0; before[r] = -1; }
    for (int j = lane; j < len; j += 64) {
        const int p = position[j];
#pragma unroll
        for (int r = 0; r < PER; ++r) {
            older[r] += p < mine[r] ? 1 : 0;
            if (BEFORE) before[r] = max(before[r], p < mine[r] ? p : -1);
        }
    }
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int n = wave_sum(older[r]);
        if (lane == r) place = n;
        if constexpr (BEFORE) {
            int m = before[r];
            for (int off = 32; off > 0; off >>= 1) m = max(m, __shfl_xor(m, off));
            if (lane == r) *newest_older = m;
        }
    }
    return place;
}

// Rows of the live slots 0 .. len - 1 of units unit0 .., in token order: dst [unit - unit0][place][row_bytes].
__global__ __launch_bounds__(NT)
void wkv_gather_rows_kernel(WkvCache c, const char* __restrict__ src, int row_bytes, int unit0, int blocks, int len, char* __restrict__ dst)
{
    extern __shared__ int32_t position[];
    __shared__ int place[ROWS];
    const int u = unit0 + (int)(blockIdx.x / blocks), s0 = (int)(blockIdx.x % blocks) * ROWS;
    load_positions(c.pos + (size_t)u * c.m, len, position);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int n = count_places<false>(position, s0 + wid * PER, len, lane, nullptr);
    if (lane < PER) place[wid * PER + lane] = n;
    __syncthreads();
    const int shift = __ffs(row_bytes) - 1 - 4, here = min(ROWS, len - s0);        // rows are 128, 256 or 512 bytes
    const char* from = src + ((size_t)u * c.m + s0) * row_bytes;
    char* to = dst + (size_t)(u - unit0) * len * row_bytes;
    for (int i = threadIdx.x; i < here << shift; i += NT) {
        const int row = i >> shift, at = (i & ((1 << shift) - 1)) * 16;
        *reinterpret_cast<u32x4_t*>(to + (size_t)place[row] * row_bytes + at) = *reinterpret_cast<const u32x4_t*>(from + (size_t)row * row_bytes + at);
    }
}

// One number a live slot, in token order: dst [unit - unit0][place] (fp64 for the score sums, else int32).  WAVE: a wave counts for 16 slots at once, else a
// thread for its own slot, one look after the other.  The latter is level or ahead for short units (us, thread | wave, score sums and merge counts:
// 256 units x 64 23 | 25, 20 | 22; 2048 x 128 116 | 114, 77 | 95; 256 x 410 64 | 62, 42 | 48), and what a long unit waits for (1 x 819 32 | 21, 31 | 22;
// 32 x 819 41 | 30, 37 | 28; 1 x 4095 89 | 31, 88 | 32, where copies and a sort on the host took 53 and 41).
constexpr int WAVE_FROM = 512;
template <bool WAVE>
__global__ __launch_bounds__(NT)
void wkv_gather_item_kernel(WkvCache c, int what, int unit0, int blocks, int len, int tokens, void* __restrict__ dst)
{
    extern __shared__ int32_t position[];
    const int u = unit0 + (int)(blockIdx.x / blocks), block = (int)(blockIdx.x % blocks);
    load_positions(c.pos + (size_t)u * c.m, len, position);
    int s, older = 0, before = -1;
    if constexpr (WAVE) {
        const int lane = threadIdx.x & 63, first = block * ROWS + (threadIdx.x >> 6) * PER;
        if (what == WKV_NMERGED) older = count_places<true>(position, first, len, lane, &before);
        else older = count_places<false>(position, first, len, lane, nullptr);
        s = lane < PER ? first + lane : len;
        if (s >= len) return;
    } else {
        s = block * NT + threadIdx.x;
        if (s >= len) return;
        const int mine = position[s];
        for (int j = 0; j < len; ++j) {
            const int p = position[j];
            if (p < mine) { ++older; before = max(before, p); }
        }
    }
    const int mine = position[s];
    const size_t at = (size_t)(u - unit0) * len + older;
    if (what == WKV_SCORE_SUM) static_cast<double*>(dst)[at] = c.a[(size_t)u * c.m + s];
    else static_cast<int32_t*>(dst)[at] = what == WKV_POS ? mine
                                        : what == WKV_COUNT ? tokens - mine          // attended once in every step since
                                        : c.merge_mode == WKV_MERGE_CONVEX ? mine - before : 1;   // a slot holds the run of tokens that ends at its own
}

// Rows in token order into slots 0, 1, ...: src [unit - unit0][len][row_bytes].
__global__ __launch_bounds__(NT)
void wkv_place_rows_kernel(WkvCache c, char* __restrict__ dst, int row_bytes, int unit0, int blocks, int len, const char* __restrict__ src)
{
    const int u = unit0 + (int)(blockIdx.x / blocks), s0 = (int)(blockIdx.x % blocks) * ROWS, here = min(ROWS, len - s0);
    const char* from = src + ((size_t)(u - unit0) * len + s0) * row_bytes;
    char* to = dst + ((size_t)u * c.m + s0) * row_bytes;
    for (int i = threadIdx.x; i < here * (row_bytes / 16); i += NT)
        reinterpret_cast<u32x4_t*>(to)[i] = reinterpret_cast<const u32x4_t*>(from)[i];
}

// Score sums, token indices and links of slots 0 .. len - 1 (the others are an empty cache's already).
__global__ __launch_bounds__(NT)
void wkv_place_items_kernel(WkvCache c, int unit0, int blocks, int len, const double* __restrict__ sums, const int32_t* __restrict__ pos)
{
    const int u = unit0 + (int)(blockIdx.x / blocks), l = (int)(blockIdx.x % blocks) * NT + threadIdx.x;
    if (l >= len) return;
    const size_t from = (size_t)(u - unit0) * len + l, to = (size_t)u * c.m + l;
    c.a[to] = sums[from];
    c.pos[to] = pos[from];
    c.nxt[to] = l + 1 < len ? l + 1 : -1;
}

hipError_t launch(const void* kernel, long long workgroups, size_t lds, void** args, hipStream_t stream)
{
    if (workgroups * NT >= (1ll << 32)) return hipErrorInvalidConfiguration;          // (a chunk is a few megabytes: never)
    return hipLaunchKernel(kernel, dim3((unsigned)workgroups), dim3(NT), args, lds, stream);
}

}  // namespace

hipError_t wkv_launch_gather(const WkvCache& c, int what, int row_bytes, int unit0, int units, int len, int64_t tokens, void* dst,
                             hipStream_t stream)
{
    WkvCache cache = c;
    const size_t lds = (size_t)len * sizeof(int32_t);
    if (what == WKV_K || what == WKV_V) {
        const char* src = static_cast<const char*>(what == WKV_K ? c.K : c.V);
        char* to = static_cast<char*>(dst);
        int blocks = (len + ROWS - 1) / ROWS;
        void* args[] = { &cache, &src, &row_bytes, &unit0, &blocks, &len, &to };
        return launch(reinterpret_cast<const void*>(&wkv_gather_rows_kernel), (long long)units * blocks, lds, args, stream);
    }
    const bool wave = len > WAVE_FROM;
    const int slots = wave ? ROWS : NT;                       // of a workgroup
    int blocks = (len + slots - 1) / slots, t = (int)tokens;
    void* args[] = { &cache, &what, &unit0, &blocks, &len, &t, &dst };
    return launch(wave ? reinterpret_cast<const void*>(&wkv_gather_item_kernel<true>) : reinterpret_cast<const void*>(&wkv_gather_item_kernel<false>),
                  (long long)units * blocks, lds, args, stream);
}

hipError_t wkv_launch_place_rows(const WkvCache& c, int what, int row_bytes, int unit0, int units, int len, const void* src,
                                 hipStream_t stream)
{
    WkvCache cache = c;
    char* to = static_cast<char*>(what == WKV_K ? c.K : c.V);
    const char* from = static_cast<const char*>(src);
    int blocks = (len + ROWS - 1) / ROWS;
    void* args[] = { &cache, &to, &row_bytes, &unit0, &blocks, &len, &from };
    return launch(reinterpret_cast<const void*>(&wkv_place_rows_kernel), (long long)units * blocks, 0, args, stream);
}

hipError_t wkv_launch_place_items(const WkvCache& c, int unit0, int units, int len, const double* sums, const int32_t* pos, hipStream_t stream)
{
    WkvCache cache = c;
    int blocks = (len + NT - 1) / NT;
    void* args[] = { &cache, &unit0, &blocks, &len, &sums, &pos };
    return launch(reinterpret_cast<const void*>(&wkv_place_items_kernel), (long long)units * blocks, 0, args, stream);
}
