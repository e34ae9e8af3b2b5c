// Bulk prefill of an empty WeightedKV cache with a prompt of P tokens, gfx950.
//
// The paper streams tokens one by one (Algorithm 1) and gives no procedure for a prompt that
// arrives at once.  What is computed here: row t of the prompt is softmax attention of q_t over
// tokens 0..t of the UNcompressed prompt (Section III-A, scale of Section III-B); the score list
// is what Algorithm 1's bookkeeping accumulates over these rows, a_i = sum_t A_t[i], with
// n_i = P - i; then, while more than m entries remain, Algorithm 1's selection and merge are
// repeated with these (now fixed) scores.  For P <= m + 1 this is exactly Algorithm 1 fed token
// by token; beyond that it is a different function (streamed tokens attend to an already
// compressed cache).
//
// Four kernels (three for a prompt that fits the cache, one more behind the second in large launches of rows of 256 bytes):
//   1. wkv_prefill_rows: causal attention in tiles of 16 queries x 16 keys.  A wave takes one tile of queries, two in large launches of
//      long prompts, or shares one with another wave in small launches (the rules stand at run()).
//      The logits are a dense contraction of 16-bit numbers, formed exactly: every row becomes 8-bit
//      digits (once per workgroup, in LDS), the digits go through the int8 matrix instruction, the
//      integer sums are put together in fp64 (what makes the later selection reproduce an fp64
//      reference exactly, as in the decode kernels).  Rows that digits do not hold take the fp64 matrix instruction.  Online softmax in
//      fp64; P.V with v_mfma_f32_16x16x16_f16 / _bf16 (fp32 accumulation): the weights go in as
//      two or three 16-bit parts straight from the registers the logits arrive in, the values as the raw
//      cache words.  Writes o_t and the log-sum-exp of every row.
//   2. wkv_prefill_scores: the column sums a_i = sum_{t >= i} exp(s_ti - lse_t): tiles of 16 keys, one a wave or
//      shared by two in small launches, looping over the query tiles below the diagonal, the same contraction
//      again (recomputing the logits costs less than storing P^2/2 of them);
//      sums stay in registers, no atomics.  Large launches leave keys of rows that digits do not hold to wkv_prefill_scores_marked.  The order of a sum is fixed for a launch form, so a result is the same from call to
//      call, and from one number of units to another as long as the form is.
//   3. wkv_prefill_compress (prompts longer than the budget): one workgroup per unit: rank of every candidate by (score, token),
//      the P - m lowest are removed; survivors get slots in token order; the weight with which every raw row
//      enters the survivor on its right, as the sequence of pairwise merges in ascending score order gives it.
//   4. wkv_prefill_fold: 16 survivors a workgroup: key rows copied, value rows summed with those weights.
//
// MFMA operand layouts (one wave; g = lane / 16, x = lane % 16), as measured on gfx950:
//   both: A operand = A[row x][k = g], B operand = B[k = g][column x];
//   f64 16x16x4: result register r holds D[row g + 4r][column x];
//   f32 16x16x16 (16-bit inputs): A operand = A[row x][k = 4g .. 4g+3], B operand = B[k = 4g .. 4g+3][column x],
//   result register r holds D[row 4g + r][column x];
//   i32 16x16x64 (8-bit inputs): A[row x][k = 16g .. 16g+15], B[k = 16g .. 16g+15][column x], result as f32.
// The reduction index of a contraction may be permuted at will as long as A and B agree, so a lane
// simply takes a contiguous quarter of its row (or of 64 elements of it).
#include "../../include/wkv.h"
#include "wkv_internal.h"
#include <mutex>
#include <type_traits>
#include "wkv_device.h"

namespace {

typedef double double4_t __attribute__((ext_vector_type(4)));
typedef float  float4_t  __attribute__((ext_vector_type(4)));

typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef short    short4_t __attribute__((ext_vector_type(4)));
typedef uint32_t uint2_t  __attribute__((ext_vector_type(2)));

constexpr int TILE = 16;
constexpr int WKV_PREFILL_MAX_TOKENS = WKV_MAX_PROMPT;   // prompt length the compression stages in LDS

// element e of a row fragment held as raw 32-bit words (two 16-bit elements per word)
template <class TT> __device__ __forceinline__ float frag_elem(const uint32_t* w, int e) {
    const uint32_t x = w[e >> 1];
    if constexpr (__is_same(TT, TF16)) {
        const half2_t h = __builtin_bit_cast(half2_t, x);
        return (e & 1) ? (float)h.y : (float)h.x;
    } else {
        return __builtin_bit_cast(float, (e & 1) ? (x & 0xFFFF0000u) : (x << 16));
    }
}

// Workgroups are dealt to the chip's eight partitions (each with its own L2) round-robin by index.
// All workgroups of a unit re-read that unit's 1-2 MB of Q, K and V, so a unit is given to ONE
// partition: workgroup b belongs to partition b % 8, and there to unit 8 * ((b / 8) / groups) + b % 8.
// (With units dealt across the partitions instead, every L2 sees the ~10 units in flight at once,
// more than it holds, and the operands come from the memory-side cache.)
constexpr int XCDS = 8;
__device__ __forceinline__ int xcd_unit(unsigned b, int groups) { return (int)((b >> 3) / groups) * XCDS + (int)(b & 7); }
inline int xcd_grid(int units, int groups) { return (units + XCDS - 1) / XCDS * XCDS * groups; }

// Units of a launch.  A grid of 2^32 threads and more is not refused: the count wraps, without an error (2796203 units x 3 workgroups of
// 512 threads: one ran).  So a launch has at most 2^31, in whole rounds of the partitions.
constexpr int units_of_a_launch(int workgroups, int threads) { return (int)((1ll << 31) / threads / workgroups) / XCDS * XCDS; }
static_assert(units_of_a_launch(1, 1024) == 1 << 21 && units_of_a_launch(256, 1024) >= XCDS && units_of_a_launch(3, 512) * 3ll * 512 <= 1ll << 31,
              "every kernel of a prompt has launches of some units");
// launch(u0, n) for the units u0 .. u0 + n - 1, until all have been launched
template <class F> inline void launches(int units, int workgroups, int threads, F&& launch) {
    const int most = units_of_a_launch(workgroups, threads);
    for (int u0 = 0; u0 < units; u0 += most) launch(u0, units - u0 < most ? units - u0 : most);
}

// Four softmax weights p >= 0, each as a sum of 16-bit numbers of the cache format, packed as MFMA
// operands, so that P.V can run on the 16-bit matrix instruction without costing accuracy against
// an fp32 P.V.  Every part but the last is the running remainder cut to the format's significand
// (a mask: exact in the format, and the next remainder is exact in fp32).
//   fp16: two parts, 11 + 11 bits, the last one cut (2^-22; weights below 2^-14 lose bits below
//         2^-24 absolute);
//   bf16: three parts, 8 + 8 + 8 bits, the last one rounded to nearest.  Two parts (2^-17) were not
//         enough: in entries that cancel to 1e-4 of their row's scale the error of the weights
//         showed, about one element in 1e8 beyond the test's bound.
// No conversion of a double to 16 bits appears here: the compiler expands that one into some
// thirty integer instructions.
typedef _Float16 half2v_t __attribute__((ext_vector_type(2)));
typedef float    float2v_t __attribute__((ext_vector_type(2)));
typedef __bf16   bf16x2_t  __attribute__((ext_vector_type(2)));
template <class TT> constexpr int weight_parts() { return __is_same(TT, TF16) ? 2 : 3; }
template <class TT> __device__ __forceinline__ void split16x4(const float (&p)[4], uint2_t (&part)[weight_parts<TT>()]) {
    if constexpr (__is_same(TT, TF16)) {
        auto cut2 = [](float a, float b) { return __builtin_bit_cast(half2v_t, __builtin_amdgcn_cvt_pkrtz(a, b)); };
        const half2v_t h01 = cut2(p[0], p[1]), h23 = cut2(p[2], p[3]);
        float l[4];
        l[0] = p[0] - (float)h01.x; l[1] = p[1] - (float)h01.y; l[2] = p[2] - (float)h23.x; l[3] = p[3] - (float)h23.y;
        part[0] = uint2_t{ __builtin_bit_cast(uint32_t, h01), __builtin_bit_cast(uint32_t, h23) };
        part[1] = uint2_t{ __builtin_bit_cast(uint32_t, cut2(l[0], l[1])), __builtin_bit_cast(uint32_t, cut2(l[2], l[3])) };
    } else {
        auto cut = [](float x) { return __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, x) & 0xFFFF0000u); };
        auto pack = [](float a, float b) {                   // the upper halves of two words: exact for cut values
            return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, b), __builtin_bit_cast(uint32_t, a), 0x07060302u);
        };
        auto round2 = [](float a, float b) {                 // v_cvt_pk_bf16_f32: to nearest even
            return __builtin_bit_cast(uint32_t, __builtin_convertvector(float2v_t{a, b}, bf16x2_t));
        };
        float h[4], m[4], l[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) { h[r] = cut(p[r]); const float rem = p[r] - h[r]; m[r] = cut(rem); l[r] = rem - m[r]; }
        part[0] = uint2_t{ pack(h[0], h[1]), pack(h[2], h[3]) };
        part[1] = uint2_t{ pack(m[0], m[1]), pack(m[2], m[3]) };
        part[2] = uint2_t{ round2(l[0], l[1]), round2(l[2], l[3]) };
    }
}

// D += A.B with 16-bit operands (four per lane, packed in two words) and fp32 accumulation
template <class TT> __device__ __forceinline__ float4_t mfma16(uint2_t a, uint2_t b, float4_t c) {
    if constexpr (__is_same(TT, TF16))
        return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(half4_t, a), __builtin_bit_cast(half4_t, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4_t, a), __builtin_bit_cast(short4_t, b), c, 0, 0, 0);
}

// exp(x) for the arguments a softmax produces, x <= 0 or a little above:
// x = (256 n + j + f) ln2 / 256 with integers n, 0 <= j < 256 and |f| <= 1/2, and
// exp(x) = 2^n . 2^(j/256) . exp(f ln2 / 256); the middle factor comes from a table in LDS, the last one from the Taylor
// quartic (remainder below r^5 / 120 < 4e-17 for |r| <= ln2 / 512), the
// first is applied by ldexp, which also takes care of gradual underflow.  Relative error a few roundings, at ten double-precision
// instructions against the library routine's two dozen: the exponentials are a good part of what bounds both kernels.  256 entries,
// and not 64: the entry's place is one byte of n, which the shift that makes its address selects by itself, and the same quartic is 1000 times closer.
// Score sums of 16 units, 77 to 1024 tokens, against 64 bits: 1.6e-16 to 1.4e-15 rms, 9.5e-15 at most (64 entries: 2.2e-15 to 8.8e-15, 5.5e-14; a cubic,
// which saves 1 % of the prompt's time, 2.0e-15 to 1.1e-14).
constexpr int EXP_STEPS = 256;
// unit: a power of two that every result is a multiple of (exactly: it only moves the exponent).
__device__ __forceinline__ void exp_table_init(double* tab, double unit) {
    static_assert(EXP_STEPS == 256, "one entry a thread of a workgroup");
    tab[threadIdx.x & 255] = unit * exp2((double)(threadIdx.x & 255) * (1.0 / EXP_STEPS));
    __syncthreads();
}
// ------------------------------------------------------------------ logits from 8-bit digits
// A row of 16-bit numbers is, up to a power of two, a row of integers: n = x * 2^s with the row's own s,
// chosen so that its largest magnitude has 31 bits.  n is written in four balanced base-256
// digits (d0..d2 in [-128, 127], d3 in [-127, 127]), and q.k becomes sixteen dot products of digits,
// which v_mfma_i32_16x16x64_i8 forms without any rounding: seven sums S_w over the pairs of weight
// w = i + j, then A = S0 + 2^8 S1, B = S2 + 2^8 S3, C = S4 + 2^8 S5 + 2^16 S6, and
// q.k = (A + 2^16 B + 2^32 C) 2^-(s_q + s_k) with the rounding of two fp64 additions: closer to the
// exact logit than a chain of D fp64 additions.  For 128 elements A, B and S4 + 2^8 S5 stay below 2^31 (the largest is B: S3 <= 128 (2 127 128 + 2 128^2)
// and S2 <= 3 128^3 make 2145386496 at most); S6 joins in fp64, exactly.
// Why: the fp64 matrix instruction takes 64 cycles for 16x16x4 on this part and shares its pipe
// with the fp64 vector instructions of the softmax; the sixteen digit products take 512 cycles per
// 16x16x128 tile against 2048.
// The lowest digit is seldom used: only by an element more than 2^-12 (fp16) or 2^-15 (bf16) below its row's largest, of normal numbers
// by a row in 31 (d 128) and one in 240.  Where no row of a tile uses it, its seven products and A are left out: one tile of
// normal numbers in three (fp16) or seven in eight (bf16).  256 units x 4096, d 128: scores 4.15 -> 3.85 ms in fp16, 4.57 -> 3.54 in bf16 (with the launch form
// below); where every tile uses it (keys with one channel at 20, fp16) what is left is the test for it.
// What bounds both kernels: the instructions of a SIMD in turn.  A vector instruction takes 4 cycles, one of these matrix instructions 8 of its 16 (alone and beside each
// other, measured in loops of both); waves on one SIMD overlap the rest, two of them badly (rows with two tiles a wave: 1560 cycles a tile
// where the instructions add up to 1010), four well (scores: 1050 of 860).  So scores keeps to 128 registers, rows to 168 (three waves) where a wave has one tile, and
// the fp64 tile among others is a function of its own (128 units x 2048, bf16: rows 1.03 -> 0.94 ms, scores 0.71 -> 0.62).
// The 32x32 matrix instructions would need half the issue cycles and were slower: the chip lowers its clock (2.2 -> 1.95 GHz).
// A row whose elements are not all integers at its scale (an element more than 2^-23 below the
// largest that uses its last bits; possible for bf16, and for fp16 rows that reach 128) or that holds
// an infinity or a NaN is marked, and a tile that touches a marked row takes the fp64 instruction.
constexpr int DIGITS = 4;
// Bits of a row's integers.  A wave whose own rows are marked is slow for its whole loop, and its workgroup waits for it, so
// what counts is how many 16 x 128 tiles hold an element too small.  Of normal numbers, 27 | 30 bits: bf16 0.6 % | 0.08 %; fp16
// none, but with one channel at 20, as keys with rotary embeddings have them, 22 % | none (no fp16 element has a bit below 2^-24:
// every row below 8 | 64 fits, and below 128 with 31 bits, which mark 0.02 % of bf16 tiles).  Measured, that channel in a prompt of 256 units x 4096 (d 128, fp16): 22.6 | 11.5 ms.
constexpr int INT_BITS = 31;

typedef int int4v_t __attribute__((ext_vector_type(4)));

// Logits are kept in units of ln 2 / 256: the exponential below then starts with a rounding, not a product.
constexpr double LOGIT_UNIT = 369.3299304675746;                           // 256 / ln 2
template <int D> __device__ __forceinline__ double logit_scale() { return LOGIT_UNIT / sqrt((double)D); }

// exp(x ln 2 / 256), times the table's unit: method above the table.  -inf would give NaN, so where a
// logit may be -inf (a masked one, a row with infinities) the argument goes through no_infinity first.  NaN stays NaN.
// Finite arguments go far beyond int (logits of fp16 rows reach 1e12 units): the cast, undefined there in C++, is the one
// instruction v_cvt_i32_f64, which saturates, and with any k that low ldexp gives 0.  (That instruction written out costs 2 % of a
// 128 x 2048 prompt, a clamp before it more; a test with logits of 3e10 units holds the result.)
// COLD: in a seldom path; its constants are not held in registers across the loop.
template <bool COLD = false> __device__ __forceinline__ double exp_units(double x, const double* tab) {
    const double kd = __builtin_rint(x);
    const double r = x - kd;
    const int k = (int)kd;
    const double tj = tab[k & 255];
    // ln2/256 = c: c, c^2/2, c^3/6, c^4/24
    double c1 = 0.0027076061740622863, c2 = 3.665565596910106e-06, c3 = 3.308302680541371e-09;
    if constexpr (COLD) asm volatile("" : "+s"(c1), "+s"(c2), "+s"(c3));
    double p = fma(r, 2.239395190875157e-12, c3);
    p = fma(p, r, c2);
    p = fma(p, r, c1);
    p = fma(p, r, 1.0);
    return ldexp(tj * p, k >> 8);
}
__device__ __forceinline__ double no_infinity(double x) { return (x < -1e6) ? -1e6 : x; }

// What the scale of a row is found from, over packed 16-bit words: the largest |x| and, for bf16, the
// smallest nonzero one (less one unit, so that zero wraps to the top).
typedef unsigned short ushort2v_t __attribute__((ext_vector_type(2)));
template <class TT> struct RowSpan {
    ushort2v_t mx = {0, 0}, mn = {0xFFFF, 0xFFFF};
    __device__ __forceinline__ void add(uint32_t w) {
        const ushort2v_t a = __builtin_bit_cast(ushort2v_t, w & 0x7FFF7FFFu);
        mx = __builtin_elementwise_max(mx, a);
        if constexpr (!__is_same(TT, TF16)) mn = __builtin_elementwise_min(mn, (ushort2v_t)(a - ushort2v_t{1, 1}));
    }
    __device__ __forceinline__ uint32_t largest() const { return max((uint32_t)mx.x, (uint32_t)mx.y); }
    __device__ __forceinline__ uint32_t smallest_exponent() const { return (min((uint32_t)mn.x, (uint32_t)mn.y) + 1u) >> 7; }
};

// Scale 2^s of a row whose largest |x| has the 16 bits `top`: the largest integer gets INT_BITS bits, or one fewer where its upper digit
// would be rounded up to 128 (from 1.9922 times a power of two on).
// bad: the row must not be sliced.  e: biased fp32 exponent of the largest element (that one up in the second case).
template <class TT> __device__ __forceinline__ int digit_shift(uint32_t top, int& e, bool& bad) {
    const uint32_t one[1] = { top + (__is_same(TT, TF16) ? 8u : 1u) };
    e = (int)(__builtin_bit_cast(uint32_t, frag_elem<TT>(one, 0)) >> 23);
    bad = e >= 255 || (e < 36 && top != 0u);             // (beyond 255: the format's last NaNs, which the addition takes into the sign)
    return (top == 0u || bad) ? 0 : INT_BITS - 1 + 127 - e;
}
// Whether this lane's elements are no integers at that scale.  fp16 has no bit below 2^-24, so a row that
// stays below 128 (s >= 24) fits; beyond, the elements are looked at.  bf16: 8 significant bits,
// the last one 7 below the exponent.
template <class TT, int NWORDS> __device__ __forceinline__ bool no_integers(const uint32_t (&w)[NWORDS], const RowSpan<TT>& span, int e, float mul) {
    if constexpr (__is_same(TT, TF16)) {
        float frac = 0.f;
        if (__any(e > 133))
#pragma unroll
            for (int i = 0; i < NWORDS; ++i) {
                uint32_t x[1] = { w[i] };
                asm("" : "+v"(x[0]));                         // (or the conversions made for this are used for the digits, which need none)
                frac = fmaxf(frac, fmaxf(__builtin_amdgcn_fractf(frag_elem<TT>(x, 0) * mul), __builtin_amdgcn_fractf(frag_elem<TT>(x, 1) * mul)));
            }
        return frac != 0.f;
    } else {
        return (int)span.smallest_exponent() + INT_BITS - 8 < e;
    }
}

// Four elements -> the words of the four digit planes (byte i of plane b = digit b of element i)
__device__ __forceinline__ void digits4(const float (&x)[4], float mul, uint32_t (&w)[DIGITS]) {
    uint32_t t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = (uint32_t)(int)fmaf(x[i], mul, 0.f) + 0x00808080u;   // the low bytes become digits + 128
    const uint32_t l01 = __builtin_amdgcn_perm(t[1], t[0], 0x05010400u), h01 = __builtin_amdgcn_perm(t[1], t[0], 0x07030602u);
    const uint32_t l23 = __builtin_amdgcn_perm(t[3], t[2], 0x05010400u), h23 = __builtin_amdgcn_perm(t[3], t[2], 0x07030602u);
    w[0] = __builtin_amdgcn_perm(l23, l01, 0x05040100u) ^ 0x80808080u;
    w[1] = __builtin_amdgcn_perm(l23, l01, 0x07060302u) ^ 0x80808080u;
    w[2] = __builtin_amdgcn_perm(h23, h01, 0x05040100u) ^ 0x80808080u;
    w[3] = __builtin_amdgcn_perm(h23, h01, 0x07060302u);
}

// Operands of one wave's own 16 rows, in registers: lane (g, x) holds elements 64 c + 16 g .. + 15 of row x.
// scale: unit * 2^-s of row x.  Returns whether a row is marked (uniform).
template <class TT, int D>
__device__ __forceinline__ bool own_digits(const char* base, int row0, int P, size_t tok, int g, int x,
                                           int4v_t (&dg)[D / 64][DIGITS], double& scale, double unit, bool& low)
{
    constexpr int KS = D / 64;
    const char* src = base + (size_t)min(row0 + x, P - 1) * tok;
    uint32_t w[KS][8];
    RowSpan<TT> span;
#pragma unroll
    for (int c = 0; c < KS; ++c) {
        load_words<8>(src + (64 * c + 16 * g) * TT::BYTES, w[c]);
#pragma unroll
        for (int i = 0; i < 8; ++i) span.add(w[c][i]);
    }
    uint32_t top = span.largest();
    top = max(top, (uint32_t)__shfl_xor((int)top, 16));
    top = max(top, (uint32_t)__shfl_xor((int)top, 32));
    bool bad;
    int ex;
    const int s = digit_shift<TT>(top, ex, bad);
    const float mul = __builtin_bit_cast(float, (uint32_t)(127 + s) << 23);
    uint32_t lowest = 0;
#pragma unroll
    for (int c = 0; c < KS; ++c) {
        bad |= no_integers<TT>(w[c], span, ex, mul);
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
            float f[4];
            uint32_t pl[DIGITS];
#pragma unroll
            for (int i = 0; i < 4; ++i) f[i] = frag_elem<TT>(w[c], 4 * e4 + i);
            digits4(f, mul, pl);
#pragma unroll
            for (int b = 0; b < DIGITS; ++b) dg[c][b][e4] = (int)pl[b];
            lowest |= pl[0];
        }
    }
    low = __any(lowest != 0);
    scale = ldexp(unit, 16 - s);
    return __any(bad);
}

// Operands of the rows that a workgroup's waves share, in LDS: CHUNK rows (two tiles), double-buffered.  Sixteen elements
// of one digit of a row are 16 bytes; those of a chunk's rows follow each other (what 16 lanes read is contiguous); HALF is the
// step to the next sixteen elements, PLANE to the next digit, STEP to the next 32 elements, so that the lanes that write
// a row, sixteen elements each, fall into different banks.
constexpr int CTILES = 2, CHUNK = CTILES * TILE;
constexpr int HALF = CHUNK * 16 + 32, PLANE = 2 * HALF, STEP = DIGITS * PLANE + 64;
__device__ __forceinline__ int digit_place(int sixteen) { return (sixteen >> 1) * STEP + (sixteen & 1) * HALF; }
constexpr int MARKED = 1, LOW = 2;       // of a row: not to be sliced; uses the lowest digit
template <int D> struct SharedRows {
    alignas(16) unsigned char dg[2][D / 32 * STEP];
    double scale[2][CHUNK];
    double lse[2][CHUNK];
    int flags[2][CHUNK];
};

// The share of a chunk of one of the workgroup's NT threads: EPT consecutive elements of a row; TPR threads a row.  (Sixteen
// elements where the row is long enough: what is paid once a thread and row, the maximum over the row's lanes, its scale, its mark, is as
// many instructions as six elements are.)
template <class TT, int D, int NT> struct ChunkLoad {
    static constexpr int EPT = CHUNK * D / NT, TPR = D / EPT, W = EPT / 2;
    static_assert((EPT == 8 || EPT == 16) && NT == CHUNK * TPR, "a thread takes half a block of a digit plane, or a whole one");
    uint32_t w[W];
    double lse;
    __device__ __forceinline__ void request(const char* base, const double* lsep, int row0, int P, size_t tok) {
        const int j = threadIdx.x % TPR, row = min(row0 + (int)threadIdx.x / TPR, P - 1);
        load_words<W>(base + (size_t)row * tok + j * EPT * TT::BYTES, w);
        if (lsep != nullptr && j == 0) lse = lsep[row];
    }
    __device__ __forceinline__ void store(SharedRows<D>& sh, int buf, bool with_lse, double unit) const {
        const int j = threadIdx.x % TPR, row = threadIdx.x / TPR;
        RowSpan<TT> span;
#pragma unroll
        for (int e = 0; e < W; ++e) span.add(w[e]);
        uint32_t top = span.largest();                            // over the row's lanes
        top = max(top, dpp_in<0xB1>(top));        // quad_perm [1,0,3,2]
        top = max(top, dpp_in<0x4E>(top));        // quad_perm [2,3,0,1]
        top = max(top, dpp_in<0x141>(top));       // row_half_mirror
        if constexpr (TPR == 16) top = max(top, dpp_in<0x140>(top));      // row_mirror
        static_assert(TPR == 8 || TPR == 16, "a row's lanes are half a DPP row, or one");
        bool bad;
        int ex;
        const int s = digit_shift<TT>(top, ex, bad);
        const float mul = __builtin_bit_cast(float, (uint32_t)(127 + s) << 23);
        bad |= no_integers<TT>(w, span, ex, mul);
        unsigned char* dst = &sh.dg[buf][digit_place(j * EPT >> 4) + row * 16 + (j * EPT & 15)];
        uint32_t pl[EPT / 4][DIGITS];
#pragma unroll
        for (int e4 = 0; e4 < EPT / 4; ++e4) {
            float f[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) f[e] = frag_elem<TT>(w, 4 * e4 + e);
            digits4(f, mul, pl[e4]);
        }
#pragma unroll
        for (int b = 0; b < DIGITS; ++b) {
            if constexpr (EPT == 16) *reinterpret_cast<u32x4_t*>(dst + b * PLANE) = u32x4_t{ pl[0][b], pl[1][b], pl[2][b], pl[3][b] };
            else *reinterpret_cast<uint2_t*>(dst + b * PLANE) = uint2_t{ pl[0][b], pl[1][b] };
        }
        uint32_t lowest = 0;
#pragma unroll
        for (int e4 = 0; e4 < EPT / 4; ++e4) lowest |= pl[e4][0];
        const unsigned long long fm = __ballot(bad), fl = __ballot(lowest != 0);
        if (j == 0) {
            constexpr unsigned long long mask = (1ull << TPR) - 1;
            int lane = threadIdx.x & 63;
            if constexpr (D == 128) asm volatile("" : "+v"(lane));    // (not a 64-bit mask held across the loop)
            sh.scale[buf][row] = ldexp(unit, -s);
            bool mark = ((fm >> lane) & mask) != 0;
            if (with_lse) {
                sh.lse[buf][row] = lse;
                mark |= !(fabs(lse) < INFINITY);
            }
            sh.flags[buf][row] = (mark ? MARKED : 0) | (((fl >> lane) & mask) != 0 ? LOW : 0);
        }
    }
};

// Products of a tile in units of 2^16, unscaled (rows = keys, columns = queries): register r of lane (g, x) = key 4g + r, query x.
// SHARED_KEYS: the shared rows are the keys and the own rows the queries, or the other way round.  low (uniform): whether any of the rows
// uses the lowest digit.  parked: the lane's own lowest digits, where they are kept in LDS and not in own.
template <class TT, int D, bool SHARED_KEYS, bool PARKED = false>
__device__ __forceinline__ void digit_tile(const unsigned char* pl, const int4v_t (&own)[D / 64][DIGITS], bool low,
                                           int g, int x, double (&s)[4], const int4v_t* parked = nullptr)
{
    auto mm = [](int4v_t a, int4v_t o, int4v_t c) __attribute__((always_inline)) {
        return SHARED_KEYS ? __builtin_amdgcn_mfma_i32_16x16x64_i8(a, o, c, 0, 0, 0) : __builtin_amdgcn_mfma_i32_16x16x64_i8(o, a, c, 0, 0, 0);
    };
    const int place = digit_place(g) + x * 16;
    auto plane = [&](int c, int i) __attribute__((always_inline)) {
        return *reinterpret_cast<const int4v_t*>(pl + place + c * 2 * STEP + i * PLANE);
    };
    const int4v_t zero = {0, 0, 0, 0};
    auto sums = [&](auto from_c) __attribute__((always_inline)) {
        constexpr int from = decltype(from_c)::value;
        int4v_t S[2 * DIGITS - 1];
#pragma unroll
        for (int w = 0; w < 2 * DIGITS - 1; ++w) S[w] = zero;
#pragma unroll
        for (int c = 0; c < D / 64; ++c)
#pragma unroll
            for (int i = from; i < DIGITS; ++i) {
                const int4v_t a = plane(c, i);
#pragma unroll
                for (int j = from; j < DIGITS; ++j) S[i + j] = mm(a, PARKED && j == 0 ? parked[c * 64] : own[c][j], S[i + j]);
            }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int B = S[2][r] + (S[3][r] << 8);
            const double C = fma((double)S[6][r], 65536.0, (double)(S[4][r] + (S[5][r] << 8)));
            s[r] = fma(C, 65536.0, (double)B);
            if constexpr (from == 0) s[r] = fma((double)(S[0][r] + (S[1][r] << 8)), 1.0 / 65536.0, s[r]);
        }
    };
    if (low) sums(std::integral_constant<int, 0>{});
    else sums(std::integral_constant<int, 1>{});
}

// A tile that touches a marked row, scaled, with the fp64 matrix instruction.  Its result register r of lane (g, x) is row g + 4r: row i is given key 4 (i % 4) + i / 4, so that the layout is digit_tile's.
// All words are requested ahead of the first product: these tiles wait for memory, not for the instruction (256 units x 4096,
// d 128, fp16, every key marked, two requests a tile against one: 34.3 against 30.9 ms).
// A function of its own (not inlined): its registers are then not the kernel's, which saves what it needs of its own only around the call.  It needs
// no stack, and neither does any kernel here: the runtime gives every queue stack memory for the whole chip when a kernel first wants some (396 bytes a lane:
// 200 MB a queue), behind the back of a caller who was promised that nothing is allocated.
template <class TT, int D, bool SHARED_KEYS>
__device__ __attribute__((noinline)) double4_t exact_tile(const char* shared, const char* own, int shared0, int own0, int P, size_t tok, int lane)
{
    constexpr int NWORDS = D / 8;
    const int g = lane >> 4, x = lane & 15;
    const int kx = 4 * (x & 3) + (x >> 2), col = g * (D / 4) * TT::BYTES;
    uint32_t sw[NWORDS], ow[NWORDS];
    load_words<NWORDS>(shared + (size_t)min(shared0 + (SHARED_KEYS ? kx : x), P - 1) * tok + col, sw);
    load_words<NWORDS>(own + (size_t)min(own0 + (SHARED_KEYS ? x : kx), P - 1) * tok + col, ow);
    double4_t s0 = {0.0, 0.0, 0.0, 0.0}, s1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int e = 0; e < 2 * NWORDS; e += 2) {
        const double a0 = (double)frag_elem<TT>(sw, e), a1 = (double)frag_elem<TT>(sw, e + 1);
        const double b0 = (double)frag_elem<TT>(ow, e), b1 = (double)frag_elem<TT>(ow, e + 1);
        s0 = SHARED_KEYS ? __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, s0, 0, 0, 0) : __builtin_amdgcn_mfma_f64_16x16x4f64(b0, a0, s0, 0, 0, 0);
        s1 = SHARED_KEYS ? __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b1, s1, 0, 0, 0) : __builtin_amdgcn_mfma_f64_16x16x4f64(b1, a1, s1, 0, 0, 0);
    }
    return (s0 + s1) * logit_scale<D>();
}

// Whether a workgroup takes the fp64 instruction for all it does: every wave holds a marked row of its own, or four of the 32 rows of the first
// shared chunk are marked (at that rate two tiles in three hold one; a row or two at a prompt's beginning say nothing about the rest).  (Uniform over the workgroup; the chunk is visible afterwards.)  Tile by tile, with the digits made beside it and
// nothing requested ahead, a prompt of marked rows only is slower than the fp64 instruction alone was before there were digits; in
// loops of its own it is not.  Rows + scores, every key marked, tile by tile | in loops of its own | before: 256 units x 4096, d 128,
// fp16 16.4 + 14.1 | 13.6 + 10.2 | 13.0 + 10.5 ms; 128 x 2048 2.51 + 2.07 | 1.93 + 1.77 | 1.85 + 1.48 ms.
// Without marked rows the test costs nothing that shows (11.32 | 11.32 ms, 1.91 | 1.92 ms for the whole prompts); with __syncthreads_and
// instead of one barrier and two ballots 11.40 ms.
template <int NW> __device__ __forceinline__ bool mostly_marked(bool own, const int (&flags)[CHUNK]) {
    static_assert(CHUNK == 32 && NW <= 32, "half a wave");
    __shared__ int waves[NW];
    if ((threadIdx.x & 63) == 0) waves[threadIdx.x >> 6] = own;
    __syncthreads();
    const unsigned m = (unsigned)__ballot(flags[threadIdx.x & (CHUNK - 1)] & MARKED);      // (both halves of the wave look at the same rows)
    return __all(waves[threadIdx.x & (NW - 1)]) || __popc(m) >= 4;
}

// ------------------------------------------------------------------ 1. rows
// Softmax and output accumulators of N consecutive tiles of 16 queries.
template <class TT, int D, int N> struct Rows {
    static constexpr double AHEAD = 8.0 * EXP_STEPS;
    static constexpr double UNIT = __is_same(TT, TBF16) ? 1.0 / 256 : 1.0;     // of the weights: the kernel's table has it
    static constexpr int NE = D / 16;         // output column sets: lane (g, x) owns columns NE*x .. NE*x+NE-1
    double m[N], l[N];                        // reference of query x (same in the 4 lanes x, x+16, ...); this lane's share of the sum
    float4_t o[N][NE];
    __device__ __forceinline__ void clear() {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            m[i] = -INFINITY;
            l[i] = 0.0;
#pragma unroll
            for (int e = 0; e < NE; ++e) o[i][e] = float4_t{0.f, 0.f, 0.f, 0.f};
        }
    }
    // Sixteen more keys.  s: their logits, register r of lane (g, x) = key 4g + r, query x; vfrag: columns NE*x .. of the values of
    // keys 4g + r.  infinities: whether a logit may be -inf (uniform).  lone: see below.
    __device__ __forceinline__ void add(double (&s)[N][4], const uint32_t (&vfrag)[4][NE / 2], bool infinities, bool lone, const double* etab, int g) {
        // Weights are relative to a reference m, the row's maximum when it was last looked for; that is when a logit exceeds it by
        // more than AHEAD units, so weights stay below 2^8 (and one of them is 1 or more: the 16-bit parts that P.V takes lose no more
        // than with the running maximum itself).  bf16 values reach 2^128, where a weight above 1 would take a product out of fp32: there all
        // weights are times 2^-8 (UNIT), and what is added up is never more than with the running maximum.  Following the maximum costs a rescaling of the sum and all output
        // accumulators in every tile in which any of the wave's rows has a new one, 16 / k of the k-th tiles with random logits:
        // half the tiles of a prompt of 4096 where a wave has 32 rows.
        double tmax[N];
        bool moved = false;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            tmax[i] = fmax(fmax(s[i][0], s[i][1]), fmax(s[i][2], s[i][3]));
            moved |= tmax[i] > m[i] + AHEAD;
        }
        if (__any(moved)) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const double top = pair_max<32>(pair_max<16>(tmax[i]));        // all 16 keys of the tile
                const double mnew = fmax(m[i], top);          // finite: key 16 kt + 0 <= every query of a later tile,
                                                              // and on the diagonal key x is attended by query x
                const double resc = exp_units<D == 128>(no_infinity(m[i] - mnew), etab) * (1.0 / UNIT);  // 0 on the first tile (m = -inf), 1 where nothing moved
                l[i] *= resc;
                m[i] = mnew;
                const float rf = (float)resc;                 // the output rows this lane holds (queries 4g + r') by their own factor
                int row = 4 * g;
                if constexpr (D == 128) asm volatile("" : "+v"(row));     // (not four lane numbers held across the loop)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float f = __shfl(rf, row + r);
#pragma unroll
                    for (int e = 0; e < NE; ++e) o[i][e][r] *= f;
                }
            }
        }
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int r = 0; r < 4; ++r) s[i][r] -= m[i];
        if (infinities) {
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) s[i][r] = no_infinity(s[i][r]);
        }
        // O[query][column] += sum over keys P[query][key] V[key][column] with the 16-bit matrix
        // instruction (k = 16 keys at once): lane (g, x) supplies k-slots 4g + r: as A operand
        // P[query x][key 4g + r], as B operand V[key 4g + r][column NE*x + e], the raw cache values.
        // P goes in as a sum of 16-bit parts.
        uint2_t pa[N][weight_parts<TT>()];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            float p[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) { const double e = exp_units(s[i][r], etab); l[i] += e; p[r] = (float)e; }
            split16x4<TT>(p, pa[i]);
        }
        // lone (uniform over the wave): the keys are the last tile's of several, newer than every query of the others, which leave
        // the product out: their weights are 0, but 0 times an infinity among the values is NaN.
        auto values = [&](auto first) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;      // high / low halves of two words
                const uint2_t vb2 = { __builtin_amdgcn_perm(vfrag[1][e >> 1], vfrag[0][e >> 1], sel),
                                      __builtin_amdgcn_perm(vfrag[3][e >> 1], vfrag[2][e >> 1], sel) };
#pragma unroll
                for (int i = decltype(first)::value; i < N; ++i)
#pragma unroll
                    for (int w = 0; w < weight_parts<TT>(); ++w) o[i][e] = mfma16<TT>(pa[i][w], vb2, o[i][e]);
            }
        };
        if (lone) values(std::integral_constant<int, N - 1>{});
        else values(std::integral_constant<int, 0>{});
    }
    // o_t = O / l and the log-sum-exp m + log l of the queries from q0 on
    __device__ __forceinline__ void finish(int q0, int P, char* out, size_t tok, double* lse, int g, int x) const {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const double sum = rows_sum(l[i]);
            const float linv = (float)(1.0 / sum);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int t = q0 + i * TILE + 4 * g + r;
                const float f = __shfl(linv, 4 * g + r);
                if (t < P && out != nullptr) {
                    char* dst = out + (size_t)t * tok + x * NE * TT::BYTES;
#pragma unroll
                    for (int e = 0; e < NE; ++e) store_elem<TT>(dst, e, o[i][e][r] * f);
                }
            }
            const int tq = q0 + i * TILE + x;
            if (g == 0 && tq < P) lse[tq] = m[i] + log(sum * (1.0 / UNIT)) * LOGIT_UNIT;
        }
    }
};

// The tile of queries qt against all its keys with the fp64 matrix instruction, for workgroups of marked rows: the queries stay in
// fp64, the next tile's keys and values are requested before this one's are used (two sets of registers take turns).  LEAN: the queries
// are converted anew for every tile and nothing is requested ahead, for a kernel that has no registers for more (and three waves a SIMD to wait with:
// 128 units x 2048, every key marked, the prompt 3.86 -> 3.74 ms, against a call of a function with the other form and a stack).
template <class TT, int D, bool LEAN>
__device__ __forceinline__ void exact_rows(const char* qb, const char* kb, const char* vb, char* ob, double* lse, int qt, int P, size_t tok,
                                           const double* etab, int g, int x)
{
    constexpr int NWORDS = D / 8, NE = D / 16;
    const int kx = 4 * (x & 3) + (x >> 2), col = g * (D / 4) * TT::BYTES;     // keys: see exact_tile
    uint32_t qw[NWORDS];
    double qd[2 * NWORDS];
    load_words<NWORDS>(qb + (size_t)min(qt * TILE + x, P - 1) * tok + col, qw);
    auto convert = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 2 * NWORDS; ++e) qd[e] = (double)frag_elem<TT>(qw, e);
    };
    if constexpr (!LEAN) convert();
    Rows<TT, D, 1> rows;
    rows.clear();
    auto request = [&](int kt, uint32_t (&kf)[NWORDS], uint32_t (&vf)[4][NE / 2]) __attribute__((always_inline)) {
        load_words<NWORDS>(kb + (size_t)min(kt * TILE + kx, P - 1) * tok + col, kf);
#pragma unroll
        for (int r = 0; r < 4; ++r) load_words<NE / 2>(vb + (size_t)min(kt * TILE + 4 * g + r, P - 1) * tok + x * NE * TT::BYTES, vf[r]);
    };
    auto tile = [&](int kt, const uint32_t (&kf)[NWORDS], const uint32_t (&vf)[4][NE / 2]) __attribute__((always_inline)) {
        if constexpr (LEAN) {
#pragma unroll
            for (int i = 0; i < NWORDS; ++i) asm volatile("" : "+v"(qw[i]));
            convert();
        }
        double4_t s0 = {0.0, 0.0, 0.0, 0.0}, s1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < 2 * NWORDS; e += 2) {
            s0 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)frag_elem<TT>(kf, e), qd[e], s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f64_16x16x4f64((double)frag_elem<TT>(kf, e + 1), qd[e + 1], s1, 0, 0, 0);
        }
        double s[1][4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s[0][r] = (s0[r] + s1[r]) * logit_scale<D>();
            if (kt == qt && 4 * g + r > x) s[0][r] = -INFINITY;
        }
        rows.add(s, vf, true, false, etab, g);
    };
    uint32_t kf0[NWORDS], vf0[4][NE / 2];
    if constexpr (LEAN) {
#pragma unroll 1
        for (int kt = 0; kt <= qt; ++kt) {
            request(kt, kf0, vf0);
            tile(kt, kf0, vf0);
        }
    } else {
        uint32_t kf1[NWORDS], vf1[4][NE / 2];
        request(0, kf0, vf0);
        for (int kt = 0; kt <= qt; kt += 2) {
            request(min(kt + 1, qt), kf1, vf1);               // past the last tile: a repeat, unused
            tile(kt, kf0, vf0);
            if (kt + 1 > qt) break;
            request(min(kt + 2, qt), kf0, vf0);
            tile(kt + 1, kf1, vf1);
        }
    }
    rows.finish(qt * TILE, P, ob, tok, lse, g, x);
}

// q, k, v, out: [P][units][D] (token-major, as a decode step sees them one token at a time).
// lse: [units][P], in units of ln 2 / 256.  One workgroup = NW waves of QT consecutive query tiles of one unit;
// the keys are sliced into digits once per workgroup and read by every wave from LDS.  What bounds
// this kernel and the next is vector instructions (slicing, recombining the digit sums, the
// exponentials), so a wave takes two tiles where that pays: slicing, value loads and their
// permutes are then paid once for both (d 128: 250 registers of two waves a SIMD).  One tile, d 128: three waves a SIMD, 167 registers.
// To that end (rows of 128 bytes have no need) a lane's own lowest digits, which are seldom used, wait in LDS, the base of a tile of values is kept scalar (the compiler
// makes a 64-bit address a lane of each of its rows otherwise, 16 registers for a chunk), and what only seldom paths need is made there.
// Before, 23 and 11 registers were spilled: 128 units x 2048 1.82 -> 1.76 ms (fp16), 1.77 -> 1.67 (bf16), 256 x 4096 10.2 -> 9.9, 10.1 -> 9.7.
// In small launches SPLIT waves share a tile instead, each taking every SPLIT-th tile of keys.
template <class TT, int D, int NW, int QT, int SPLIT>
__global__ __launch_bounds__(64 * NW, D == 128 && SPLIT == 1 && QT == 1 ? 3 : 2)
void wkv_prefill_rows(const void* __restrict__ q_, const void* __restrict__ k_, const void* __restrict__ v_,
                      void* __restrict__ out_, double* __restrict__ lse, int P, int units, int unit0)
{
    constexpr int ROWB = D * TT::BYTES;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int g = lane >> 4, x = lane & 15;
    const int ntiles = (P + TILE - 1) / TILE;
    constexpr int TPG = NW / SPLIT * QT;                                         // tiles of a workgroup
    const int groups = (ntiles + TPG - 1) / TPG;
    const int u = unit0 + xcd_unit(blockIdx.x, groups);
    const int qt0 = (groups - 1 - (int)((blockIdx.x >> 3) % groups)) * TPG;      // long rows are scheduled first
    if (u >= units) return;                                                      // the whole workgroup
    const int qt = qt0 + wid / SPLIT * QT, part = wid % SPLIT;                   // first tile of the wave; its share of the keys
    const bool active = qt < ntiles;                                             // an idle wave still slices keys
    const int mine = min(qt + QT, ntiles) - 1;                                   // its last key tile, and the workgroup's
    const int last = min(qt0 + TPG, ntiles) - 1;
    __shared__ double etab[EXP_STEPS];
    __shared__ SharedRows<D> sh;
    exp_table_init(etab, Rows<TT, D, QT>::UNIT);
    const size_t tok = (size_t)units * ROWB;                              // bytes from one token to the next
    const char* qb = reinterpret_cast<const char*>(q_) + (size_t)u * ROWB;
    const char* kb = reinterpret_cast<const char*>(k_) + (size_t)u * ROWB;
    const char* vb = reinterpret_cast<const char*>(v_) + (size_t)u * ROWB;
    char* ob = out_ == nullptr ? nullptr : reinterpret_cast<char*>(out_) + (size_t)u * ROWB;

    ChunkLoad<TT, D, 64 * NW> next;
    next.request(kb, nullptr, 0, P, tok);
    int4v_t qdg[QT][D / 64][DIGITS];
    double qscale[QT];
    bool qmarked = false, qlow[QT];
#pragma unroll
    for (int i = 0; i < QT; ++i) qmarked |= own_digits<TT, D>(qb, (qt + i) * TILE, P, tok, g, x, qdg[i], qscale[i], 1.0, qlow[i]);
    next.store(sh, 0, false, logit_scale<D>());
    constexpr bool PARK = D == 128 && SPLIT == 1;
    __shared__ int4v_t parked[PARK ? NW * QT * (D / 64) * 64 : 1];
    int4v_t* park = parked + (PARK ? wid * QT * (D / 64) * 64 + lane : 0);
    if constexpr (PARK)
#pragma unroll
        for (int i = 0; i < QT; ++i)
#pragma unroll
            for (int c = 0; c < D / 64; ++c) park[(i * (D / 64) + c) * 64] = qdg[i][c][0];         // (read by the same lane)

    if constexpr (SPLIT == 1) {
        if (mostly_marked<NW>(qmarked || !active, sh.flags[0])) {
            if (active)
#pragma unroll 1
                for (int t = qt; t <= mine; ++t)
                    exact_rows<TT, D, D == 128 && QT == 1>(qb, kb, vb, ob, lse + (size_t)u * P, t, P, tok, etab, g, x);
            return;
        }
    }
    Rows<TT, D, QT> rows;
    rows.clear();
    constexpr int NE = rows.NE;
    // a lane's place in a tile of values; the four rows are a uniform stride apart (four offsets held ready take six registers more)
    const size_t voff = (size_t)(4 * g) * tok + x * NE * TT::BYTES;
    auto tile = [&](int kt, int buf) __attribute__((always_inline)) {
        // V fragments: keys 16 kt + 4g + r, columns NE*x .. NE*x+NE-1; requested here, used after the softmax
        // (a lane's offsets in a tile never change; only a tile that reaches past the prompt clamps its rows)
        uint32_t vfrag[4][NE / 2];
        if (kt * TILE + TILE <= P) {                          // uniform
            const char* vt = vb + (size_t)(kt * TILE) * tok;
            if constexpr (PARK) asm volatile("" : "+s"(vt));      // (see above; with parts, kt is not known to be scalar)
#pragma unroll
            for (int r = 0; r < 4; ++r) load_words<NE / 2>(vt + r * tok + voff, vfrag[r]);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r)
                load_words<NE / 2>(vb + (size_t)min(kt * TILE + 4 * g + r, P - 1) * tok + x * NE * TT::BYTES, vfrag[r]);
        }
        const int t = kt % CTILES;
        double s[QT][4];
        const int flags = sh.flags[buf][t * TILE + x];
        const bool special = __any(flags & MARKED) || qmarked, low = __any(flags & LOW);       // uniform
        if (special) {
#pragma unroll
            for (int i = 0; i < QT; ++i) {
                const double4_t e = exact_tile<TT, D, true>(kb, qb, kt * TILE, (qt + i) * TILE, P, tok, lane);
#pragma unroll
                for (int r = 0; r < 4; ++r) s[i][r] = e[r];
            }
        } else {
#pragma unroll
            for (int i = 0; i < QT; ++i) {
                if (QT > 1) __builtin_amdgcn_sched_barrier(0);       // one tile's sums at a time: the registers do not hold two
                digit_tile<TT, D, true, PARK>(&sh.dg[buf][t * TILE * 16], qdg[i], low || qlow[i], g, x, s[i], park + i * (D / 64) * 64);
#pragma unroll
                for (int r = 0; r < 4; ++r) s[i][r] *= sh.scale[buf][t * TILE + 4 * g + r] * qscale[i];
            }
        }
        const bool edge = kt >= qt;           // a diagonal tile: key 4g + r may be attended by query x only if not newer
        if (edge) {
#pragma unroll
            for (int i = 0; i < QT; ++i)
#pragma unroll
                for (int r = 0; r < 4; ++r) if ((kt - qt - i) * TILE + 4 * g + r > x) s[i][r] = -INFINITY;
        }
        rows.add(s, vfrag, special || edge, QT > 1 && kt > qt, etab, g);
    };
    // A chunk is worked on from one buffer while the next one is on its way from memory; it is sliced into
    // the other buffer at the end of the round, which every wave left before the barrier at its start.
    for (int kt = 0, buf = 0; kt <= last; kt += CTILES, buf ^= 1) {
        __syncthreads();
        const bool more = kt + CTILES <= last;
        if (more) next.request(kb, nullptr, (kt + CTILES) * TILE, P, tok);
        if (active)
            for (int t = part; t < CTILES && kt + t <= mine; t += SPLIT) tile(kt + t, buf);
        if (more) next.store(sh, buf ^ 1, false, logit_scale<D>());
    }
    // The parts of a split row: maxima, sums and accumulators go through LDS (the digits have been used) and are put
    // together by the first part's wave, in order.  A part that saw no key has maximum -inf and adds nothing.
    if constexpr (SPLIT > 1) {
        constexpr int PS = (NW - NW / SPLIT) * 64;                         // lanes that hand something over
        static_assert(QT == 1 && sizeof(sh.dg) >= PS * (NE * 16 + 16), "the parts fit the digits' place");
        double* dm = reinterpret_cast<double*>(&sh.dg);                    // [2][PS] maximum, sum
        float* po = reinterpret_cast<float*>(dm + 2 * PS);                // [NE * 4][PS]
        const int me = (wid - wid / SPLIT - 1) * 64 + lane;                // of a later part; of the first: one row of lanes before
        __syncthreads();
        if (part != 0) {
            dm[me] = rows.m[0];
            dm[PS + me] = rows.l[0];
#pragma unroll
            for (int e = 0; e < NE; ++e)
#pragma unroll
                for (int r = 0; r < 4; ++r) po[(e * 4 + r) * PS + me] = rows.o[0][e][r];
        }
        __syncthreads();
        if (part != 0 || !active) return;
        for (int w = 1; w < SPLIT; ++w) {
            const double m2 = dm[me + w * 64], l2 = dm[PS + me + w * 64];
            if (__all(l2 == 0.0)) continue;                                // uniform: no key of this part (a NaN goes on)
            const double mnew = fmax(rows.m[0], m2);
            const double f1 = exp_units(no_infinity(rows.m[0] - mnew), etab) * (1.0 / rows.UNIT);
            const double f2 = exp_units(no_infinity(m2 - mnew), etab) * (1.0 / rows.UNIT);
            rows.l[0] = rows.l[0] * f1 + l2 * f2;
            rows.m[0] = mnew;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float g1 = __shfl((float)f1, 4 * g + r), g2 = __shfl((float)f2, 4 * g + r);
#pragma unroll
                for (int e = 0; e < NE; ++e) rows.o[0][e][r] = rows.o[0][e][r] * g1 + po[(e * 4 + r) * PS + me + w * 64] * g2;
            }
        }
    }
    if (!active) return;

    rows.finish(qt * TILE, P, ob, tok, lse + (size_t)u * P, g, x);
}

// ------------------------------------------------------------------ 2. scores
// The tile of keys kt against all its queries with the fp64 matrix instruction, for workgroups of marked rows: the next tile of
// queries is requested before this one is used.  LEAN: the keys are converted anew each round, which keeps the kernel within 128 registers (four waves;
// d 64, 256 units x 4096, every key marked: the prompt 15.5 -> 13.9 ms, 14.7 before there were digits).  With d 128 and long loops they
// stay in fp64 (see wkv_prefill_scores_marked).
template <class TT, int D, bool LEAN>
__device__ __forceinline__ void exact_scores(const char* qb, const char* kb, const double* lse, double* a, int kt, int ntiles, int P, size_t tok,
                                             const double* etab, int g, int x)
{
    constexpr int NWORDS = D / 8;
    const int kx = 4 * (x & 3) + (x >> 2), col = g * (D / 4) * TT::BYTES;     // keys: see exact_tile
    uint32_t kw[NWORDS], next[NWORDS];
    double kd[2 * NWORDS], next_l, acc[4] = {0.0, 0.0, 0.0, 0.0};
    load_words<NWORDS>(kb + (size_t)min(kt * TILE + kx, P - 1) * tok + col, kw);
    auto convert = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 2 * NWORDS; ++e) kd[e] = (double)frag_elem<TT>(kw, e);
    };
    auto request = [&](int qt) __attribute__((always_inline)) {
        const int t = min(min(qt, ntiles - 1) * TILE + x, P - 1);          // past the last tile: a repeat, unused
        load_words<NWORDS>(qb + (size_t)t * tok + col, next);
        next_l = *reinterpret_cast<const double*>(reinterpret_cast<const char*>(lse) + (unsigned)t * 8u);     // (t < 4096: a 32-bit offset)
    };
    request(kt);
    if constexpr (!LEAN) {
        convert();
#pragma unroll
        for (int e = 0; e < 2 * NWORDS; ++e) asm volatile("" : "+v"(kd[e]));      // (held, and not converted in the loop all the same)
    }
    for (int qt = kt; qt < ntiles; ++qt) {
        uint32_t w[NWORDS];
#pragma unroll
        for (int i = 0; i < NWORDS; ++i) w[i] = next[i];
        const double l = next_l;
        request(qt + 1);
        constexpr bool TIED = LEAN && D == 128;               // converted four words at a time, when the products before are done
        if constexpr (LEAN && !TIED) {
#pragma unroll
            for (int i = 0; i < NWORDS; ++i) asm volatile("" : "+v"(kw[i]));
            convert();
        }
        double4_t s0 = {0.0, 0.0, 0.0, 0.0}, s1 = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int e = 0; e < 2 * NWORDS; e += 2) {
            if constexpr (TIED) {
                asm volatile("" : "+v"(kw[e >> 1]), "+v"(w[e >> 1]));
                if (e % 8 == 0) asm volatile("" : "+v"(s0));
                kd[e] = (double)frag_elem<TT>(kw, e);
                kd[e + 1] = (double)frag_elem<TT>(kw, e + 1);
            }
            s0 = __builtin_amdgcn_mfma_f64_16x16x4f64(kd[e], (double)frag_elem<TT>(w, e), s0, 0, 0, 0);
            s1 = __builtin_amdgcn_mfma_f64_16x16x4f64(kd[e + 1], (double)frag_elem<TT>(w, e + 1), s1, 0, 0, 0);
        }
        const int tq = qt * TILE + x;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const bool on = tq < P && kt * TILE + 4 * g + r <= tq;         // causal, and inside the prompt
            acc[r] += exp_units<LEAN && D == 128>(no_infinity(on ? (s0[r] + s1[r]) * logit_scale<D>() - l : -INFINITY), etab);
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const double c = row_allsum(acc[r]);                               // over the 16 queries x
        const int key = kt * TILE + 4 * g + r;
        if (x == 0 && key < P) a[key] = c;
    }
}
constexpr double LATER = -1.0;        // in place of a tile's first column sum, which is never negative: left to wkv_prefill_scores_marked

// a[u][i] = sum over rows t >= i of exp(s_ti - lse_t).  A wave has one tile of keys, or shares it with SPLIT - 1 others; NW waves, a workgroup,
// share the sliced queries.
template <class TT, int D, int NW, int SPLIT>
__global__ __launch_bounds__(64 * NW, D == 128 && SPLIT == 1 ? 4 : 2)
void wkv_prefill_scores(const void* __restrict__ q_, const void* __restrict__ k_, const double* __restrict__ lse,
                        double* __restrict__ a, int P, int units, int unit0)
{
    constexpr int ROWB = D * TT::BYTES;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int g = lane >> 4, x = lane & 15;
    const int ntiles = (P + TILE - 1) / TILE;
    constexpr int TPG = NW / SPLIT;                                       // tiles of a workgroup
    const int groups = (ntiles + TPG - 1) / TPG;
    const int u = unit0 + xcd_unit(blockIdx.x, groups);
    const int kt0 = (int)((blockIdx.x >> 3) % groups) * TPG;              // low key tiles have the most rows: first
    if (u >= units) return;                                               // the whole workgroup
    const int kt = kt0 + wid / SPLIT, part = wid % SPLIT;
    const bool active = kt < ntiles;
    __shared__ double etab[EXP_STEPS];
    __shared__ SharedRows<D> sh;
    exp_table_init(etab, 1.0);
    const size_t tok = (size_t)units * ROWB;
    const char* qb = reinterpret_cast<const char*>(q_) + (size_t)u * ROWB;
    const char* kb = reinterpret_cast<const char*>(k_) + (size_t)u * ROWB;
    const double* lseu = lse + (size_t)u * P;

    ChunkLoad<TT, D, 64 * NW> next;
    next.request(qb, lseu, kt0 * TILE, P, tok);
    int4v_t kdg[D / 64][DIGITS];
    double kx, kscale[4], acc[4];
    bool klow;
    const bool kmarked = own_digits<TT, D>(kb, kt * TILE, P, tok, g, x, kdg, kx, logit_scale<D>(), klow);
#pragma unroll
    for (int r = 0; r < 4; ++r) { kscale[r] = __shfl(kx, 4 * g + r); acc[r] = 0.0; }
    next.store(sh, 0, true, 1.0);

    if constexpr (SPLIT == 1) {
        if (mostly_marked<NW>(kmarked || !active, sh.flags[0])) {
            if (active) {
                if constexpr (NW == 8) {
                    if (lane == 0) a[(size_t)u * P + kt * TILE] = LATER;
                } else {
                    int tid = threadIdx.x;
                    asm volatile("" : "+v"(tid));                         // (what the two paths share would be held, or spilled, across the other one)
                    exact_scores<TT, D, true>(qb, kb, lseu, a + (size_t)u * P, kt, ntiles, P, tok, etab, tid >> 4 & 3, tid & 15);
                }
            }
            return;
        }
    }
    for (int q0 = kt0, buf = 0; q0 < ntiles; q0 += CTILES, buf ^= 1) {
        __syncthreads();
        const bool more = q0 + CTILES < ntiles;
        if (more) next.request(qb, lseu, (q0 + CTILES) * TILE, P, tok);
        if (active)
            for (int qt = q0 + part; qt < min(q0 + CTILES, ntiles); qt += SPLIT) {
                if (qt < kt) continue;
                const int t = qt - q0;
                const double l = sh.lse[buf][t * TILE + x];
                double s[4];
                const int flags = sh.flags[buf][t * TILE + x];
                const bool special = __any(flags & MARKED) || kmarked, low = __any(flags & LOW);   // uniform
                if (special) {
                    const double4_t e = exact_tile<TT, D, false>(qb, kb, qt * TILE, kt * TILE, P, tok, lane);
#pragma unroll
                    for (int r = 0; r < 4; ++r) s[r] = e[r];
                } else {
                    const double qs = sh.scale[buf][t * TILE + x];
                    digit_tile<TT, D, false>(&sh.dg[buf][t * TILE * 16], kdg, low || klow, g, x, s);
#pragma unroll
                    for (int r = 0; r < 4; ++r) s[r] *= kscale[r] * qs;
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) s[r] -= l;
                if (special || qt == kt || qt == ntiles - 1) {             // causal, and inside the prompt
                    const int tq = qt * TILE + x;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const bool on = tq < P && kt * TILE + 4 * g + r <= tq;
                        s[r] = no_infinity(on ? s[r] : -INFINITY);         // exp gives 0; no branch
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[r] += exp_units(s[r], etab);
            }
        if (more) next.store(sh, buf ^ 1, true, 1.0);
    }
    if constexpr (SPLIT > 1) {                                            // the parts' sums, added in order by the first part's wave
        double* ps = reinterpret_cast<double*>(&sh.dg);                   // [4][NW * 64]
        const int me = threadIdx.x;
        __syncthreads();
        if (part != 0)
#pragma unroll
            for (int r = 0; r < 4; ++r) ps[r * NW * 64 + me] = acc[r];
        __syncthreads();
        if (part != 0) return;
        for (int w = 1; w < SPLIT; ++w)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] += ps[r * NW * 64 + me + w * 64];
    }
    if (!active) return;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));                                         // (as above)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const double c = row_allsum(acc[r]);                               // over the 16 queries x
        const int key = kt * TILE + 4 * (tid >> 4 & 3) + r;
        if ((tid & 15) == 0 && key < P) a[(size_t)u * P + key] = c;
    }
}

// The tiles of keys that the launch before left out, as its workgroups had marked rows.  A kernel of its own, where the keys stay in fp64: the registers
// for that would cost the kernel above two of its four waves a SIMD.  Only after launches with eight waves a workgroup, which take milliseconds: where nothing is
// marked all it does is look, 12 us.  A wave has a long tile and a short one, so that all have the same work: half as many workgroups look (a tile each
// 19.5 us), and the chip empties at once.  256 units x 4096, every key marked, fp16: scores 12.8 -> 10.2 ms (a tile a wave 10.4; two or four next to each
// other 11.8, 13.6; the same tile of four units 11.8), the prompt 26.4 -> 23.9.
constexpr int MARKED_WAVES = 4;
template <class TT, int D>
__global__ __launch_bounds__(64 * MARKED_WAVES, 2)
void wkv_prefill_scores_marked(const void* __restrict__ q_, const void* __restrict__ k_, const double* __restrict__ lse,
                               double* __restrict__ a, int P, int units, int unit0)
{
    constexpr int ROWB = D * TT::BYTES;
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int ntiles = (P + TILE - 1) / TILE, pairs = (ntiles + 1) / 2, groups = (pairs + MARKED_WAVES - 1) / MARKED_WAVES;
    const int u = unit0 + xcd_unit(blockIdx.x, groups);
    const int kt = (int)((blockIdx.x >> 3) % groups) * MARKED_WAVES + wid, other = ntiles - 1 - kt;   // a wave's tiles (the middle one alone)
    if (u >= units) return;                                               // the whole workgroup
    double* au = a + (size_t)u * P;
    const bool left = kt < pairs && (lane == 0 || (lane == 1 && other != kt)) && au[(lane == 0 ? kt : other) * TILE] == LATER;
    if (!__syncthreads_or(left)) return;
    __shared__ double etab[EXP_STEPS];
    exp_table_init(etab, 1.0);
    const char* qb = reinterpret_cast<const char*>(q_) + (size_t)u * ROWB;
    const char* kb = reinterpret_cast<const char*>(k_) + (size_t)u * ROWB;
    unsigned long long todo = __ballot(left);                             // uniform over the wave
#pragma unroll 1
    for (; todo != 0; todo &= todo - 1)
        exact_scores<TT, D, false>(qb, kb, lse + (size_t)u * P, au, (todo & 1) ? kt : other, ntiles, P, (size_t)units * ROWB, etab, lane >> 4, lane & 15);
}

// ------------------------------------------------------------------ 3. compress
// One workgroup per unit, for prompts longer than the budget.  Scores are fixed during the compression, so the P - L tokens that
// the repeated selection removes are the candidates of lowest (score, token), in that order.
//
// Values.  A removed token j folds into the nearest token on its right that is still present
// when its turn comes, i.e. the nearest one with a higher rank (survivors rank above everything):
// its parent.  The merges therefore form a forest whose roots are the survivors, and a node
// receives its children in ascending rank.  With s the scores, a child c of p contributes
//     g_c * prod_{children c' of p ranked after c} f_c',   f_c' = s_p / (s_c' + s_p),  g_c = s_c / (s_c + s_p)
// of its accumulated value to p's, and p's own raw value keeps prod_{children} f_c'.  The weight
// of a raw token in its survivor's row is the product of these coefficients up the tree, and the
// row is the weighted sum of the raw rows of the run -- the same numbers as the sequence of pairwise
// merges (Algorithm 1) in fp64, with no dependent chain of row updates.  Rows are rounded to the
// cache format once, when they are written.
//
// What bounds it is LDS: the sort's traffic and the dependent looks of the two searches.  us, 24 units x 1237 | 128 x 2048 | 256 x 4096: pairs a step and
// searches entry by entry, then 64 at a time 52 | 74 | 148 (of it sort 20 | 21 | 43, searches 15 | 30 | 62); four elements through two steps
// at a time, groups of 8 in between 36 | 45 | 90.
//
// What is left is a weight per token, written to global memory; the rows themselves are moved by
// wkv_prefill_fold, which has the whole chip where this kernel has a workgroup per unit.
//
// LDS: sc[P] score, then list products, finally weight | ae[P] f, then edge coefficient | a0[P] g, then
//      own coefficient | slot[P] | wcnt[NT] (one per wave is used) | rk[P] rank (16 bit) | par[P] parent (16 bit) |
//      ptr[P] list successor (16 bit) | bmax[64]; gmax[512] takes wcnt's place.  The sort keys borrow ae[], a0[] and slot[].
__global__ __launch_bounds__(1024)
void wkv_prefill_compress(WkvCache c, const double* __restrict__ a, double* __restrict__ weight, int P, int unit0)
{
    const int tid = threadIdx.x, NT = blockDim.x, lane = tid & 63, wid = tid >> 6, NW = NT >> 6;
    const int u = unit0 + blockIdx.x, m = c.m;
    double*  au = c.a + (size_t)u * m;
    int32_t* pu = c.pos + (size_t)u * m;
    int32_t* nu = c.nxt + (size_t)u * m;
    const double* ap = a + (size_t)u * P;
    double* wu = weight + (size_t)u * P;

    extern __shared__ double lds[];
    double*   sc   = lds;
    double*   ae   = sc + P;
    double*   a0   = ae + P;
    int32_t*  slot = reinterpret_cast<int32_t*>(a0 + P);      // slot of a survivor, -1 for a removed token
    int32_t*  wcnt = slot + P;
    uint16_t* rk   = reinterpret_cast<uint16_t*>(wcnt + NT);
    uint16_t* par  = rk + P;
    uint16_t* ptr  = par + P;                                 // successor in the list a product runs along
    uint16_t* bmax = ptr + P;                                 // [64] highest rank in a block of 64 tokens
    const int L = m, nrem = P - m;                            // tokens that stay, tokens to remove: P > m
    const int lo = c.n_sink, hi = P - c.R;                    // candidates: lo <= token < hi

    for (int i = tid; i < P; i += NT) {
        const double ai = ap[i];
        double s = (c.score_mode == 0) ? ai / (double)(P - i) : ai;       // abar = a / n, n_i = P - i
        if (!(s == s) || s == INFINITY) { s = INFINITY; atomicAdd(&c.status[1], 1); }
        sc[i] = s;
    }
    __syncthreads();
    // rank among the candidates by (score, token); the nrem lowest are removed.  A bitonic sort of
    // (score bits, token) in LDS (the key arrays borrow ae[], a0[] and slot[], not yet in use).
    for (int i = tid; i < P; i += NT) rk[i] = 0xFFFF;
    {
        unsigned long long* key = reinterpret_cast<unsigned long long*>(ae);   // [N2]
        uint16_t* kid = reinterpret_cast<uint16_t*>(slot);                     // [N2]
        int N2 = 1;
        while (N2 < P) N2 <<= 1;
        for (int i = tid; i < N2; i += NT) {
            unsigned long long kb64 = ~0ull;                                   // not a candidate, or padding: sorts last
            if (i >= lo && i < hi) {
                const unsigned long long bits = (unsigned long long)__double_as_longlong(sc[i]);
                kb64 = (bits >> 63) ? ~bits : (bits | 0x8000000000000000ull);  // order of the doubles as order of integers
                if (kb64 == ~0ull) kb64 = ~0ull - 1;                           // (no score maps there; keep the sentinel unique)
            }
            key[i] = kb64;
            kid[i] = (uint16_t)i;
        }
        __syncthreads();
        // What takes the time is LDS traffic, so a thread takes four elements through two steps at a time (distances j and j / 2).
        // Steps of distance 128 and less stay within the 256 elements that a wave's quadruples (or pairs, two a lane) span:
        // LDS operations of a wave complete in order, so those need no workgroup barrier.
        auto order = [](unsigned long long& ka, uint16_t& ia, unsigned long long& kb, uint16_t& ib, bool up) __attribute__((always_inline)) {
            const bool gt = ka > kb || (ka == kb && ia > ib), swap = gt == up;
            const unsigned long long k0 = swap ? kb : ka, k1 = swap ? ka : kb;
            const uint16_t i0 = swap ? ib : ia, i1 = swap ? ia : ib;
            ka = k0; kb = k1; ia = i0; ib = i1;
        };
        auto one_step = [&](int j, int k) __attribute__((always_inline)) {
            for (int half = 0; half < 2; ++half) {
                const int t = wid * 128 + half * 64 + lane;
                if (t >= (N2 >> 1)) break;
                const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1)), l = i | j;
                unsigned long long ki = key[i], kl = key[l];
                uint16_t di = kid[i], dl = kid[l];
                order(ki, di, kl, dl, (i & k) == 0);
                key[i] = ki; key[l] = kl; kid[i] = di; kid[l] = dl;
            }
        };
        auto two_steps = [&](int j, int k) __attribute__((always_inline)) {
            const int h = j >> 1;
            if (tid < (N2 >> 2)) {
                const int i = ((tid & ~(h - 1)) << 2) | (tid & (h - 1));
                const bool up = (i & k) == 0;
                unsigned long long q[4];
                uint16_t d[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) { q[e] = key[i + e * h]; d[e] = kid[i + e * h]; }
                order(q[0], d[0], q[2], d[2], up);
                order(q[1], d[1], q[3], d[3], up);
                order(q[0], d[0], q[1], d[1], up);
                order(q[2], d[2], q[3], d[3], up);
#pragma unroll
                for (int e = 0; e < 4; ++e) { key[i + e * h] = q[e]; kid[i + e * h] = d[e]; }
            }
        };
        auto settle = [&](int j) __attribute__((always_inline)) {
            if (j > 128) {
                __syncthreads();
            } else {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        };
        for (int k = 2, steps = 1; k <= N2; k <<= 1, ++steps) {
            int j = k >> 1;
            if (steps & 1) { one_step(j, k); settle(j); j >>= 1; }
            for (; j >= 2; j >>= 2) { two_steps(j, k); settle(j); }
            if (k >= 256) __syncthreads();                    // the next k starts with a distance of 256 or more
        }
        __syncthreads();
        for (int r = tid; r < nrem; r += NT) rk[kid[r]] = (uint16_t)r;         // the nrem lowest keys are candidates
        __syncthreads();
    }
    for (int i = tid; i < P; i += NT) slot[i] = (rk[i] != 0xFFFF) ? -1 : 0;
    __syncthreads();
    // survivors get consecutive slots in token order: exclusive scan over the keep flags
    const int per = (P + NT - 1) / NT;
    const int b0 = min(tid * per, P), b1 = min(b0 + per, P);
    int mine = 0;
    for (int i = b0; i < b1; ++i) mine += (slot[i] == 0) ? 1 : 0;
    int upto = mine;                                          // inclusive scan: over the wave, then over the waves' totals
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) { const int t = __shfl_up(upto, off); if (lane >= off) upto += t; }
    if (lane == 63) wcnt[wid] = upto;
    __syncthreads();
    {
        int sidx = upto - mine;
        for (int w = 0; w < wid; ++w) sidx += wcnt[w];
        for (int i = b0; i < b1; ++i) if (slot[i] == 0) slot[i] = sidx++;
    }
    __syncthreads();
    // score sums, token indices and links of the survivors
    for (int i = tid; i < P; i += NT) {
        const int sidx = slot[i];
        if (sidx >= 0) { au[sidx] = ap[i]; pu[sidx] = i; nu[sidx] = (sidx + 1 < L) ? sidx + 1 : -1; }
    }
    const bool merging = c.merge_mode == 0;
    if (merging) {
        // Parent of a removed token: the nearest token to its right that outranks it (survivors
        // outrank everything: rank 0xFFFF); also the nearest one to its LEFT that outranks it.  Both by
        // a search that skips whole groups of 8 and blocks of 64 tokens whose highest rank is too low: each look waits for LDS, and a
        // wave for the lane with the most of them, so each of a token's two searches looks at no more than 100 entries however long the runs are.
        constexpr int NIL = 0xFFFF;
        const int nblk = (P + 63) >> 6;
        uint16_t* gmax = reinterpret_cast<uint16_t*>(wcnt);   // [512] highest rank in a group of 8 (the counts have been used)
        for (int b = wid; b < nblk; b += NW) {
            const int i = b * 64 + lane;
            int r = (i < P) ? (int)rk[i] : 0;
#pragma unroll
            for (int off = 1; off < 8; off <<= 1) r = max(r, __shfl_xor(r, off));
            if ((lane & 7) == 0) gmax[b * 8 + (lane >> 3)] = (uint16_t)r;
#pragma unroll
            for (int off = 8; off < 64; off <<= 1) r = max(r, __shfl_xor(r, off));
            if (lane == 0) bmax[b] = (uint16_t)r;
        }
        __syncthreads();
        for (int i = tid; i < P; i += NT) {
            int right = i, left = NIL;                        // a survivor is its own parent
            if (slot[i] < 0) {
                const int ri = rk[i];
                {                                             // a survivor lies to the right (the newest tokens are never removed): every search ends
                    const int e = (i | 7) + 1;
                    int k = i + 1;
                    while (k < e && rk[k] <= ri) ++k;
                    if (k == e) {
                        const int ge = ((i >> 6) + 1) * 8;
                        int n = (i >> 3) + 1;
                        while (n < ge && gmax[n] <= ri) ++n;
                        if (n == ge) {
                            int b = (i >> 6) + 1;
                            while (bmax[b] <= ri) ++b;
                            n = b * 8;
                            while (gmax[n] <= ri) ++n;
                        }
                        k = n * 8;
                        while (rk[k] <= ri) ++k;
                    }
                    right = k;
                }
                {
                    const int e = (i & ~7) - 1;
                    int k = i - 1;
                    while (k > e && rk[k] <= ri) --k;
                    if (k == e) {
                        const int ge = (i >> 6) * 8 - 1;
                        int n = (i >> 3) - 1;
                        while (n > ge && gmax[n] <= ri) --n;
                        if (n == ge) {
                            int b = (i >> 6) - 1;
                            while (b >= 0 && bmax[b] <= ri) --b;
                            n = -1;
                            if (b >= 0) { n = b * 8 + 7; while (gmax[n] <= ri) --n; }      // bmax[b] > ri: ends inside block b
                        }
                        k = -1;
                        if (n >= 0) { k = n * 8 + 7; while (rk[k] <= ri) --k; }
                    }
                    left = (k >= 0) ? k : NIL;
                }
            }
            par[i] = (uint16_t)right;
            ptr[i] = (uint16_t)left;
        }
        __syncthreads();
        // f and g of every removed token with respect to its parent (one division each): f -> ae[], g -> a0[]
        for (int i = tid; i < P; i += NT) {
            if (slot[i] >= 0) continue;
            const double sp = sc[par[i]], si = sc[i], den = si + sp;
            ae[i] = (den > 0.0) ? sp / den : 0.5;
            a0[i] = (den > 0.0) ? si / den : 0.5;
            if (!(den > 0.0)) atomicAdd(&c.status[0], 1);
        }
        __syncthreads();
        // Products along lists by pointer jumping: every removed token i has a successor (held in
        // ptr[i], NIL at the end); on return sc[i] = product of val[] over all tokens after i in its
        // list.  log2(list length) rounds, each token's update held in registers across a barrier.
        // sc[] (the scores) is free from here on.
        constexpr int MAXTOK = (WKV_PREFILL_MAX_TOKENS + 1023) / 1024;   // tokens per thread
        auto list_products = [&](const double* val) {
            for (int i = tid; i < P; i += NT) {
                const int j = (slot[i] < 0) ? (int)ptr[i] : NIL;
                sc[i] = (j != NIL) ? val[j] : 1.0;
            }
            __syncthreads();
            for (;;) {
                double wn[MAXTOK];
                int jn[MAXTOK];
                int pending = 0;
#pragma unroll
                for (int kk = 0; kk < MAXTOK; ++kk) {
                    const int i = tid + kk * NT;
                    jn[kk] = NIL;
                    wn[kk] = 1.0;
                    if (i < P && slot[i] < 0) {
                        const int j = ptr[i];
                        wn[kk] = sc[i];
                        if (j != NIL) { wn[kk] *= sc[j]; jn[kk] = ptr[j]; pending |= (jn[kk] != NIL) ? 1 : 0; }
                    }
                }
                __syncthreads();
#pragma unroll
                for (int kk = 0; kk < MAXTOK; ++kk) {
                    const int i = tid + kk * NT;
                    if (i < P && slot[i] < 0) { sc[i] = wn[kk]; ptr[i] = (uint16_t)jn[kk]; }
                }
                if (!__syncthreads_or(pending)) break;
            }
        };
        // Siblings.  The children of p, from p - 1 leftwards, have ascending rank, i.e. they are merged
        // into p in that order; the one after child i is the nearest token on i's left that outranks
        // i, as long as it does not outrank p as well.  ptr[] holds that left neighbour: cut the lists.
        for (int i = tid; i < P; i += NT) {
            if (slot[i] >= 0) continue;
            const int l = ptr[i];
            if (l != NIL && rk[l] >= rk[par[i]]) ptr[i] = NIL;     // (a survivor has rank 0xFFFF)
        }
        __syncthreads();
        list_products(ae);                                     // sc[i] = product of f over the siblings merged after i
        // edge coefficient of a removed token within its parent: g_i times the f of the later siblings;
        // own coefficient of any token: the f of all its children = f of the first child (the token on
        // its left, if that is a child) times the f of that child's later siblings.
        {
            double edge[MAXTOK], own[MAXTOK];
#pragma unroll
            for (int kk = 0; kk < MAXTOK; ++kk) {
                const int i = tid + kk * NT;
                edge[kk] = 0.0; own[kk] = 1.0;
                if (i >= P) continue;
                if (slot[i] < 0) edge[kk] = a0[i] * sc[i];
                if (i > 0 && slot[i - 1] < 0 && par[i - 1] == i) own[kk] = ae[i - 1] * sc[i - 1];
            }
            __syncthreads();
#pragma unroll
            for (int kk = 0; kk < MAXTOK; ++kk) {
                const int i = tid + kk * NT;
                if (i >= P) continue;
                if (slot[i] < 0) ae[i] = edge[kk];
                a0[i] = own[kk];
            }
        }
        // Ancestors: the weight of a raw token in its survivor's row is its own coefficient times the
        // edge coefficients up the tree.
        for (int i = tid; i < P; i += NT) {
            if (slot[i] >= 0) continue;
            const int q = par[i];
            ptr[i] = (slot[q] < 0) ? (uint16_t)q : (uint16_t)NIL;
        }
        __syncthreads();
        list_products(ae);                                     // sc[i] = product of the edge coefficients of i's removed ancestors
        for (int i = tid; i < P; i += NT) wu[i] = (slot[i] < 0) ? sc[i] * (ae[i] * a0[i]) : a0[i];
    }
}

// ------------------------------------------------------------------ 4. fold
// Keys and values of the survivors, FOLD_ROWS of them a workgroup: a key row is copied, a value row is the
// weighted sum of the raw rows of its run (the removed tokens left of the survivor, and itself),
// copied where the run is empty.  The loads are what takes the time (the runs of a unit are its whole
// prompt), so they go over the chip: 16 bytes a lane, 64 / LPR rows an instruction, four in
// flight; a run of LONG tokens or more is shared by the workgroup's waves.  Sums in fp64, rounded to
// the cache format once.  A prompt that fits the cache has no compress kernel before it: the few words of bookkeeping
// a token are written here (77 tokens: one launch of 5 us less).  Measured, with the wave-local steps of the sort (compress, then compress + fold):
// 24 units, 1237 tokens to 333 (d 64): 231 -> 50 + 16 us; 128 units, 2048 to 512 (d 128): 372 -> 59 + 59;
// 256 units, 4096 to 410: 795 -> 129 + 119 (the compress kernel's share by now: see there).
constexpr int FOLD_ROWS = 16, FOLD_WAVES = 8, LONG = 64;
template <class TT, int D>
__global__ __launch_bounds__(64 * FOLD_WAVES)
void wkv_prefill_fold(WkvCache c, const void* __restrict__ k_, const void* __restrict__ v_,
                      const double* __restrict__ weight, const double* __restrict__ a, int P, int unit0, int blocks, int merging)
{
    constexpr int ROWB = D * TT::BYTES, LPR = ROWB / 16, G = 64 / LPR;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int u = unit0 + blockIdx.x / blocks, s0 = (blockIdx.x % blocks) * FOLD_ROWS;
    const int L = min(P, c.m), here = min(FOLD_ROWS, L - s0);
    const size_t tok = (size_t)c.units * ROWB;
    const char* kb = reinterpret_cast<const char*>(k_) + (size_t)u * ROWB;
    const char* vb = reinterpret_cast<const char*>(v_) + (size_t)u * ROWB;
    char* Kc = reinterpret_cast<char*>(c.K) + ((size_t)u * c.m + s0) * ROWB;
    char* Vc = reinterpret_cast<char*>(c.V) + ((size_t)u * c.m + s0) * ROWB;
    const int32_t* pu = c.pos + (size_t)u * c.m;
    const double* wu = weight + (size_t)u * P;
    __shared__ int token[FOLD_ROWS + 1];                      // of survivor s0 - 1, s0, ...
    __shared__ double part[FOLD_WAVES][D];
    if (P <= c.m) {                                           // uniform: nothing is removed, no compress kernel ran
        if (tid <= here) token[tid] = s0 + tid - 1;
        if (tid < here) {
            const int i = s0 + tid;
            const size_t at = (size_t)u * c.m + i;
            const double ai = a[(size_t)u * P + i], s = (c.score_mode == 0) ? ai / (double)(P - i) : ai;
            if (!(s == s) || s == INFINITY) atomicAdd(&c.status[1], 1);
            c.a[at] = ai;
            c.pos[at] = i;
            c.nxt[at] = (i + 1 < P) ? i + 1 : -1;
        }
    } else if (tid <= here) {
        token[tid] = (s0 + tid > 0) ? pu[s0 + tid - 1] : -1;
    }
    __syncthreads();
    for (int i = tid; i < here * LPR; i += 64 * FOLD_WAVES) {
        uint32_t w[4];
        load_words<4>(kb + (size_t)token[i / LPR + 1] * tok + (i % LPR) * 16, w);
        *reinterpret_cast<u32x4_t*>(Kc + (size_t)(i / LPR) * ROWB + (i % LPR) * 16) = u32x4_t{ w[0], w[1], w[2], w[3] };
    }
    const int grp = lane / LPR, at = lane % LPR;
    // acc[e] += sum over rows first, first + stride, ... <= last of weight * V[row][8 at + e], then over the wave's groups
    auto sum_rows = [&](double (&acc)[8], int first, int last, int stride) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = 0.0;
        for (int k0 = first; k0 <= last; k0 += 4 * stride) {
            uint32_t raw[4][4];
            double w[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int k = min(k0 + j * stride, last);
                w[j] = (k0 + j * stride <= last) ? wu[k] : 0.0;
                load_words<4>(vb + (size_t)k * tok + at * 16, raw[j]);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (k0 + j * stride <= last)                  // (a repeated row must not add 0 x infinity)
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[e] = fma(w[j], (double)frag_elem<TT>(raw[j], e), acc[e]);
        }
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int off = LPR; off < 64; off <<= 1) acc[e] += __shfl_xor(acc[e], off);
    };
    for (int r = wid; r < here; r += FOLD_WAVES) {            // one wave per row
        const int last = token[r + 1], first = merging ? token[r] + 1 : last;
        char* dst = Vc + (size_t)r * ROWB;
        if (first == last) {                                  // nothing folds into this token
            if (grp == 0) {
                uint32_t w[4];
                load_words<4>(vb + (size_t)last * tok + at * 16, w);
                *reinterpret_cast<u32x4_t*>(dst + at * 16) = u32x4_t{ w[0], w[1], w[2], w[3] };
            }
        } else if (last - first < LONG) {
            double acc[8];
            sum_rows(acc, first + grp, last, G);
            if (grp == 0)
#pragma unroll
                for (int e = 0; e < 8; ++e) store_elem_f64<TT>(dst, at * 8 + e, acc[e]);
        }
    }
    for (int r = 0; r < here; ++r) {                          // uniform over the workgroup
        const int last = token[r + 1], first = token[r] + 1;
        if (!merging || last - first < LONG) continue;
        double acc[8];
        sum_rows(acc, first + wid * G + grp, last, FOLD_WAVES * G);
        if (grp == 0)
#pragma unroll
            for (int e = 0; e < 8; ++e) part[wid][at * 8 + e] = acc[e];
        __syncthreads();
        if (tid < D) {
            double y = 0.0;
#pragma unroll
            for (int w = 0; w < FOLD_WAVES; ++w) y += part[w][tid];
            store_elem_f64<TT>(Vc + (size_t)r * ROWB, tid, y);
        }
        __syncthreads();                                      // the partial sums have been read
    }
}

// How many tiles of 16 tokens a wave of rows takes.  Two share slicing, value loads and permutes, but are half as many workgroups with twice the
// last stretch of each (the diagonal, and the loop's end on an emptying chip) and two waves a SIMD instead of three, so both the loop and the launch must be long.
// Whole prompts, one tile | two, ms: fp16 d 128: 128 units x 4096 5.56 | 5.41, 256 x 4096 10.46 | 10.11, 192 x 3072 4.71 | 4.71, 1024 x 2048
// 10.85 | 11.18, 1024 x 1024 3.26 | 3.58; bf16: 128 x 4096 5.89 | 5.96, 192 x 4096 8.10 | 7.98, 256 x 4096
// 10.55 | 9.98, 384 x 3072 9.15 | 8.98, 512 x 2048 5.58 | 5.67.  Rows of 128 bytes: fp16 256 x 4096 7.75 | 7.64, 384 x 3072 6.76 | 6.87,
// bf16 384 x 4096 11.88 | 12.04 (before the lowest digit was left out), so never.
// In those launches a workgroup of scores has eight waves instead of four, which halves the slicing: 256 x 4096 fp16 4.08 | 4.05 ms, bf16 3.84 | 3.60, but 128 x 2048
// 0.612 | 0.629 and 96 x 1024 0.152 | 0.170.  (All of these with a stack in both forms; without it 128 x 2048 5 % and 256 x 4096 3 % less, for both.)
inline bool two_tiles_a_wave(long long tiles, int P) { return P >= 3072 && tiles >= 49152; }
// Whether two waves share a tile, each taking every other tile of its loop.  Small launches last as long as their longest loop;
// but every part slices all the rows it shares with fewer waves, which pays until the chip is full: for short prompts early.
// Whole prompts, one wave | two, us (fp16 d 128; bf16 d 128; fp16 d 64; bf16 d 64; - not taken):
//   128 units x 128 (1024 tiles) 71 | 67; 72 | 68; 61 | 61; -            128 x 256 (2048) 112 | 119; 132 | 130; -; 91 | 97
//   64 x 384 (1536) 126 | 120; 129 | 123; 106 | 98; -                    128 x 384 (3072) 145 | 170; 156 | 177; 119 | 136; -
//   24 x 1024 (1536) 270 | 214; 274 | 218; 205 | 183; 204 | 184          48 x 1024 (3072) 331 | 301; 339 | 302; 250 | 219; 250 | 226
//   96 x 512 (3072) 196 | 198; 198 | 205; 153 | 149; -                   32 x 2048 (4096) 649 | 586; 655 | 607; 486 | 426; 547 | 450
//   8 x 4096 (2048) 810 | 646; 1063 | 709; 584 | 452; 584 | 463          16 x 4096 (4096) 1039 | 1026; 1062 | 1105; 759 | 744; 827 | 772
// (bf16 d 128 at 16 x 4096 with one key channel at 20: 1218 | 1191, 12 x 4096 1056 | 1036, 9 x 4096 1126 | 1044, so the line stays for all.)
// From 3072 tokens on one unit more for some partitions is felt, so units count in rounds of all eight: fp16 d 128, d 64 17 x 3800 (3 a partition, as 24)
// 1175 | 1307, -; 18 x 3500 981 | 1102; 697 | 749; 20 x 3200 850 | 948; 625 | 647; bf16 927 | 961; 628 | 672; fp16 9 x 4096 (as 16) 1017 | 1000.
inline bool two_waves_a_tile(int units, int ntiles, int P) {
    const long long counted = P >= 3072 ? (units + XCDS - 1) / XCDS * (long long)XCDS : units;
    return counted * ntiles <= (P < 512 ? 1536 : 4096);
}

template <class TT, int D>
hipError_t run(const WkvCache& c, const void* q, const void* k, const void* v, void* out,
               double* lse, double* a, int P, hipStream_t stream)
{
    constexpr int NW = 4;
    const int ntiles = (P + TILE - 1) / TILE;
    const long long tiles = (long long)c.units * ntiles;
    auto contract = [&](auto tiles_c, auto split_c) {
        constexpr int T = decltype(tiles_c)::value, S = decltype(split_c)::value, TPG = NW / S * T, NS = 4 * T, TPS = NS / S;
        const int groups = (ntiles + TPG - 1) / TPG, groups_s = (ntiles + TPS - 1) / TPS;
        launches(c.units, groups, 64 * NW, [&](int u0, int n) {
            hipLaunchKernelGGL((wkv_prefill_rows<TT, D, NW, T, S>), dim3(xcd_grid(n, groups)), dim3(64 * NW), 0, stream, q, k, v, out, lse, P, c.units, u0);
        });
        launches(c.units, groups_s, 64 * NS, [&](int u0, int n) {
            hipLaunchKernelGGL((wkv_prefill_scores<TT, D, NS, S>), dim3(xcd_grid(n, groups_s)), dim3(64 * NS), 0, stream, q, k, lse, a, P, c.units, u0);
        });
        if constexpr (NS == 8) {
            const int groups_m = ((ntiles + 1) / 2 + MARKED_WAVES - 1) / MARKED_WAVES;
            launches(c.units, groups_m, 64 * MARKED_WAVES, [&](int u0, int n) {
                hipLaunchKernelGGL((wkv_prefill_scores_marked<TT, D>), dim3(xcd_grid(n, groups_m)), dim3(64 * MARKED_WAVES), 0, stream, q, k, lse, a, P,
                                   c.units, u0);
            });
        }
    };
    using std::integral_constant;
    if (two_waves_a_tile(c.units, ntiles, P)) {
        contract(integral_constant<int, 1>{}, integral_constant<int, 2>{});
    } else if (D == 64 || !two_tiles_a_wave(tiles, P)) {
        contract(integral_constant<int, 1>{}, integral_constant<int, 1>{});
    } else {
        if constexpr (D == 128) contract(integral_constant<int, 2>{}, integral_constant<int, 1>{});
    }
    if (P > c.m) {
        // The kernel's limit is one for all threads of the process and all prompts: always the longest prompt's, so that no
        // call lowers it between another one's setting and its launch.
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&wkv_prefill_compress),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)wkv_prefill_lds_bytes(WKV_PREFILL_MAX_TOKENS));
        if (e != hipSuccess) return e;
        const size_t lds = wkv_prefill_lds_bytes(P);
        // the row log-sum-exps have been used: their place takes the weights of the tokens
        launches(c.units, 1, 1024, [&](int u0, int n) {
            hipLaunchKernelGGL(wkv_prefill_compress, dim3(n), dim3(1024), lds, stream, c, a, lse, P, u0);
        });
    }
    const int blocks = ((P < c.m ? P : c.m) + FOLD_ROWS - 1) / FOLD_ROWS;
    const int merging = c.merge_mode == 0 && P > c.m;
    launches(c.units, blocks, 64 * FOLD_WAVES, [&](int u0, int n) {
        hipLaunchKernelGGL((wkv_prefill_fold<TT, D>), dim3(n * blocks), dim3(64 * FOLD_WAVES), 0, stream, c, k, v, lse, a, P, u0, blocks, merging);
    });
    return hipGetLastError();
}

}  // namespace

size_t wkv_prefill_lds_bytes(int P) { return (size_t)P * 34 + 1024 * 4 + 64 * 2; }

// ---- scratch of wkv_prefill_noalloc: a static device array, so that the call allocates nothing.
// Every GPU holds its own copy at its own address; in host code the array's name is only a
// stand-in for hipGetSymbolAddress, never an address to hand to a kernel.
static __device__ __align__(256) unsigned char wkv_noalloc_scratch[WKV_NOALLOC_SCRATCH_BYTES];

hipError_t wkv_prefill_static_scratch(int device, double** ptr)
{
    constexpr int MAX_DEVICES = 64;
    static std::mutex mu;
    static void* addr[MAX_DEVICES] = {};
    if (device < 0 || device >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(wkv_noalloc_scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[device] = p;
    }
    *ptr = static_cast<double*>(addr[device]);
    return hipSuccess;
}

hipError_t wkv_launch_prefill(const WkvCache& c, int dtype, int head_dim, const void* q, const void* k,
                              const void* v, void* out, double* lse, double* a, int P, hipStream_t stream)
{
    if (dtype == 1 && head_dim == 64)  return run<TF16, 64>(c, q, k, v, out, lse, a, P, stream);
    if (dtype == 1 && head_dim == 128) return run<TF16, 128>(c, q, k, v, out, lse, a, P, stream);
    if (dtype == 2 && head_dim == 64)  return run<TBF16, 64>(c, q, k, v, out, lse, a, P, stream);
    if (dtype == 2 && head_dim == 128) return run<TBF16, 128>(c, q, k, v, out, lse, a, P, stream);
    return hipErrorInvalidValue;
}
