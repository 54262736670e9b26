// Row-wise top-k selection (paper Sec. 4.1 workload table: Top-K; Sec. 4.2: selection sort -> radix
// select; Table 1: `radix_select`, "coarse + refine pass"): the kernels of its three states and the C ABI.
// One workgroup per row.  A value's key is its bit pattern made monotone (sign bit flipped for
// non-negative values, all bits for negative ones; -0.0 takes +0.0's key), so "k-th largest value" is
// "k-th largest unsigned key" and can be found digit by digit from histograms.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <atomic>

#include "../../include/topk_lineage.h"

namespace {

struct TopkArgs {
    const float* x;
    int32_t* idx;
    float* val;
    int64_t n, k, ld;
};

__device__ __forceinline__ uint32_t key_of(float v)
{
    uint32_t b = __float_as_uint(v);
    if (b == 0x80000000u) b = 0;
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Inclusive prefix sum over the wave, by data-parallel moves: rows of 16 first, then the last lane of a row to the next row
// and of the lower half to the upper one.
__device__ __forceinline__ int row_scan(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);      // row_shr:1, 2, 4, 8; lanes that have no source add 0
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    return v;
}
__device__ __forceinline__ int wave_scan(int v)
{
    v = row_scan(v);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);      // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);      // row_bcast:31 into rows 2 and 3
    return v;
}

// The wave's largest value, in lane 63.
__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
    auto with = [&](uint32_t o) { v = o > v ? o : v; };
    with(__builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false));
    with(__builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false));
    with(__builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false));
    with(__builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false));
    with(__builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false));
    with(__builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false));
    return v;
}

// The workgroup's part of a prefix sum whose waves have done theirs (`s`, inclusive): one barrier.  `wsum` is T/64 ints of
// LDS that nobody reads any more.
template <int T>
__device__ __forceinline__ int join_scan(int s, int* wsum, int* total)
{
    static_assert(T / 64 <= 16, "the waves' sums are one row of lanes");
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (lane == 63) wsum[wave] = s;
    __syncthreads();
    const int sums = row_scan(lane < T / 64 ? wsum[lane] : 0);
    *total = __builtin_amdgcn_readlane(sums, T / 64 - 1);
    return s + (wave > 0 ? __builtin_amdgcn_readlane(sums, wave - 1) : 0);
}

// Inclusive prefix sum of v over the workgroup's T threads; *total receives the sum over all of them.  Two barriers; safe to
// call back to back.  (With shuffles, and the waves' sums added up one by one, a scan took 1700 cycles of a 12 000-cycle
// selection; most instructions of these kernels run once, from a cold instruction cache, so short code counts.)
template <int T>
__device__ __forceinline__ int block_scan(int v, int* wsum, int* total)
{
    const int s = wave_scan(v);
    __syncthreads();                      // the previous call's readers are done with wsum
    return join_scan<T>(s, wsum, total);
}

// Where this lane's `n` entries go in a list whose length is *length, in no particular order; all lanes of the wave take part.
// (One addition per wave: hundreds of lanes that add to one word of LDS wait for each other.)
__device__ __forceinline__ int take_places(int n, int* length)
{
    const int s = wave_scan(n);
    int first = 0;
    if ((threadIdx.x & 63) == 63 && s > 0) first = atomicAdd(length, s);
    return __builtin_amdgcn_readlane(first, 63) + s - n;
}

// Ordered compaction shared by all states.  Each thread owns a contiguous run of elements [lo, hi) and
// classifies element i through `cls(i)`: 2 = above the threshold, 1 = equal to it, 0 = below.  Selected
// are all of class 2 and the first `take_equal` of class 1 in index order; they are written in index
// order, values taken from `value(i)`.  Rows shorter than 65536 elements need one scan (both counts
// packed into one word), longer ones two.
template <int T, typename CLS, typename VAL>
__device__ __forceinline__ void compact(const TopkArgs& a, int64_t lo, int64_t hi, int take_equal, int* wsum, CLS cls, VAL value)
{
    int gt = 0, eq = 0;
    for (int64_t i = lo; i < hi; ++i) {
        const int c = cls(i);
        gt += c == 2;
        eq += c == 1;
    }
    int total, g, e;
    if (a.n < 65536) {
        const int both = block_scan<T>(gt | (eq << 16), wsum, &total) - (gt | (eq << 16));
        g = both & 0xFFFF;                             // class-2 elements before this thread's run
        e = (int)((uint32_t)both >> 16);               // class-1 elements before it
    } else {
        g = block_scan<T>(gt, wsum, &total) - gt;
        e = block_scan<T>(eq, wsum, &total) - eq;
    }
    int32_t* idx = a.idx + (int64_t)blockIdx.x * a.k;
    float* val = a.val + (int64_t)blockIdx.x * a.k;
    for (int64_t i = lo; i < hi; ++i) {
        const int c = cls(i);
        if (c == 2 || (c == 1 && e < take_equal)) {
            const int64_t pos = g + (e < take_equal ? e : take_equal);
            if (pos < a.k) {                            // always true for NaN-free rows
                idx[pos] = (int32_t)i;
                val[pos] = value(i);
            }
        }
        g += c == 2;
        e += c == 1;
    }
}

// ---- T0: selection ------------------------------------------------------------------------------
constexpr int SEL_T = 256;
constexpr int SEL_MAX_N = 65536;

__global__ __launch_bounds__(SEL_T) void topk_selection(TopkArgs a)
{
    __shared__ unsigned char taken[SEL_MAX_N];
    __shared__ float wv[SEL_T / 64];
    __shared__ int wi[SEL_T / 64];
    __shared__ int wsum[SEL_T / 64];
    const float* row = a.x + (int64_t)blockIdx.x * a.ld;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = (int)a.n;
    constexpr int NONE = 0x7FFFFFFF;
    for (int i = tid; i < n; i += SEL_T) taken[i] = 0;
    __syncthreads();
    // a candidate (v, i) beats the best so far when there is none, when it is larger, or equal and earlier
    auto beats = [](float v, int i, float bv, int bi) { return i != NONE && (bi == NONE || v > bv || (v == bv && i < bi)); };
    for (int64_t round = 0; round < a.k; ++round) {
        float bv = 0.0f;
        int bi = NONE;
        for (int i = tid; i < n; i += SEL_T) {
            if (taken[i]) continue;
            const float v = row[i];
            if (beats(v, i, bv, bi)) { bv = v; bi = i; }
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const float ov = __shfl_xor(bv, o, 64);
            const int oi = __shfl_xor(bi, o, 64);
            if (beats(ov, oi, bv, bi)) { bv = ov; bi = oi; }
        }
        if (lane == 0) { wv[wave] = bv; wi[wave] = bi; }
        __syncthreads();
        if (tid == 0) {
            for (int w = 1; w < SEL_T / 64; ++w)
                if (beats(wv[w], wi[w], bv, bi)) { bv = wv[w]; bi = wi[w]; }
            if (bi != NONE) taken[bi] = 1;
        }
        __syncthreads();
    }
    const int64_t seg = (a.n + SEL_T - 1) / SEL_T;
    const int64_t lo = tid * seg < a.n ? tid * seg : a.n, hi = lo + seg < a.n ? lo + seg : a.n;
    compact<SEL_T>(a, lo, hi, 0, wsum, [&](int64_t i) { return taken[i] ? 2 : 0; }, [&](int64_t i) { return row[i]; });
}

// The digit d of a histogram of nb bins with  #(keys with a larger digit) < remaining <= #(keys with digit >= d),
// how many of the keys with that digit are still wanted, and how many there are.  The caller has a barrier between the
// counting and this call; the results are readable by every thread on return.
struct Digit { int digit, left, count; };
template <int T>
__device__ __forceinline__ void pick_digit(const int* hist, int nb, int remaining, int* wsum, Digit* out)
{
    const int tid = threadIdx.x;
    const int ch = nb >= T ? nb / T : 1;                   // bins per thread, a contiguous chunk
    const bool active = tid * ch < nb;
    int s = 0;
    if (active)
        for (int c = 0; c < ch; ++c) s += hist[tid * ch + c];
    int total;
    const int incl = join_scan<T>(wave_scan(s), wsum, &total);
    const int above = total - incl;                         // keys in the chunks above this thread's
    if (active && above < remaining && remaining <= above + s) {
        int acc = above;
        for (int d = tid * ch + ch - 1; d >= tid * ch; --d) {
            if (acc + hist[d] >= remaining) {
                *out = Digit{d, remaining - acc, hist[d]};
                break;
            }
            acc += hist[d];
        }
    }
    __syncthreads();
}

// Adds four neighbouring elements per lane to a histogram, at once where they share a bin, and at once for the wave where all
// of its elements do (sorted, smooth and equal rows: additions to one word of LDS wait for each other, 4096 of them 4 us).
// All lanes of the wave take part.
__device__ __forceinline__ void count_bins(int* hist, const uint32_t (&bin)[4], const bool (&on)[4])
{
    const bool all = on[0] && on[1] && on[2] && on[3], alike = all && bin[0] == bin[1] && bin[1] == bin[2] && bin[2] == bin[3];
    if (__any(alike)) {
        const uint32_t first = __builtin_amdgcn_readfirstlane(bin[0]);
        if (__all(alike && bin[0] == first)) {
            if ((threadIdx.x & 63) == 0) atomicAdd(&hist[first], 4 * 64);
            return;
        }
    }
    if (alike) {
        atomicAdd(&hist[bin[0]], 4);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (on[e]) atomicAdd(&hist[bin[e]], 1);
    }
}

// The keys that share the k-th largest one's first digit, listed in LDS: once they are few, one wave finishes, six bits a
// step, in a histogram of one bin per lane, while the others wait at one barrier; it stops as soon as all that are left are
// taken.  Taken are the keys above `thr` and the first `equal` of those that equal it.
// (T2, which used to make two more histogram passes of five barriers each: 64 rows x 4096, k = 512, 7.2 -> 5.0 us, 1204 cycles
// of loads, 1400 of counting, 1100 for the digit, 1400 for the list, 2300 here and 900 of compaction; 64 x 1024, k = 64, 8.7 ->
// 4.5, of which 2 were additions of elements that do not exist to one bin; 128 x 16384, k = 1000, 20.7 -> 9.8; 4 x 9000, k = 100,
// 22.7 -> 7.7; 4000 x 1000, k = 10, 93 -> 30.)
constexpr int FEW_KEYS = 512;
struct Cut { uint32_t thr; int equal; };

// called by a whole wave; `count` <= FEW_KEYS keys that agree in the bits from `shift` up, which are `prefix`'s
__device__ __forceinline__ Cut cut_of_listed(const uint32_t* keys, volatile int* h, int count, int remaining, uint32_t prefix, int shift)
{
    constexpr int ITEMS = FEW_KEYS / 64;
    const int lane = threadIdx.x & 63;
    uint32_t key[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) key[j] = j * 64 + lane < count ? keys[j * 64 + lane] : ~prefix;
    int size = count;
    while (shift > 0 && (size != remaining || prefix == 0)) {
        const int low = shift < 6 ? 0 : shift - 6;
        h[lane] = 0;                                        // (one wave: LDS serves its requests in order)
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < ITEMS; ++j)
            if (key[j] >> shift == prefix >> shift) atomicAdd((int*)&h[63 - ((key[j] >> low) & 63)], 1);      // (bits from `shift` up are the same in all)
        __builtin_amdgcn_wave_barrier();
        const int mine = h[lane], incl = wave_scan(mine);   // lane l: the digit 63 - l
        const int at = __ffsll((unsigned long long)__ballot(incl >= remaining)) - 1;
        size = __builtin_amdgcn_readlane(mine, at);
        remaining -= __builtin_amdgcn_readlane(incl, at) - size;
        prefix = ((prefix >> low | 63u) - (uint32_t)at) << low;
        shift = low;
    }
    return size == remaining && prefix != 0 ? Cut{prefix - 1, 0} : Cut{prefix, remaining};
}

// ---- T1 / T2: radix select ----------------------------------------------------------------------
// NPASS histogram passes over digits of B0, B1, ... bits, most significant first (they add up to 32).
// RESIDENT: the thread's ITEMS consecutive keys are loaded once (16 bytes at a time) and every pass
// runs from registers; otherwise every pass reads the row again (any n).
template <int T, int BINS, bool RESIDENT>
struct RadixShared {
    int hist[BINS];
    int wsum[T / 64];
    Digit found;
};
template <int T, int BINS>
struct RadixShared<T, BINS, true> : RadixShared<T, BINS, false> {
    uint32_t few[FEW_KEYS];
    int bins[64], listed;
    Cut cut;
};
template <int T, int ITEMS, bool RESIDENT, int NPASS, int B0, int B1, int B2, int B3>
__global__ __launch_bounds__(T) void topk_radix(TopkArgs a)
{
    static_assert(B0 + B1 + B2 + B3 == 32 && NPASS >= 1 && NPASS <= 4, "the digits cover the key");
    constexpr int MAXB = B0 > B1 ? (B0 > B2 ? (B0 > B3 ? B0 : B3) : (B2 > B3 ? B2 : B3)) : (B1 > B2 ? (B1 > B3 ? B1 : B3) : (B2 > B3 ? B2 : B3));
    constexpr int BITS[4] = {B0, B1, B2, B3};
    __shared__ RadixShared<T, 1 << MAXB, RESIDENT> sh;
    auto& hist = sh.hist;
    auto& wsum = sh.wsum;
    Digit& found = sh.found;
    const float* row = a.x + (int64_t)blockIdx.x * a.ld;
    const int tid = threadIdx.x;
    const int64_t n = a.n;

    // resident form: the thread's values as loaded (bit patterns; the key is three ALU operations away).
    // Elements past n are held as the pattern whose key is 0, below every non-NaN key.
    constexpr uint32_t PAD_BITS = 0xFFFFFFFFu;
    uint32_t held[RESIDENT ? ITEMS : 1];
    int mine = 0;                                           // the thread's elements that exist
    if constexpr (RESIDENT) {
        static_assert(ITEMS % 4 == 0, "16-byte loads");
        const int64_t left = n - (int64_t)tid * ITEMS;
        mine = left < 0 ? 0 : left < ITEMS ? (int)left : ITEMS;
#pragma unroll
        for (int j = 0; j < ITEMS; j += 4) {
            const int64_t i = (int64_t)tid * ITEMS + j;
            if (i + 3 < n) {
                const float4 v = *(const float4*)(row + i);
                held[j] = __float_as_uint(v.x); held[j + 1] = __float_as_uint(v.y); held[j + 2] = __float_as_uint(v.z); held[j + 3] = __float_as_uint(v.w);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) held[j + e] = i + e < n ? __float_as_uint(row[i + e]) : PAD_BITS;
            }
        }
    }
    if (tid == 0) {
        found = Digit{0, 0, 0};
        if constexpr (RESIDENT) sh.listed = 0;
    }

    uint32_t prefix = 0, mask = 0;
    int remaining = (int)a.k, shift = 32;
#pragma unroll
    for (int p = 0; p < NPASS; ++p) {
        const int bits = BITS[p], nb = 1 << bits;
        shift -= bits;
        for (int i = tid; i < nb; i += T) hist[i] = 0;
        __syncthreads();
        if constexpr (RESIDENT) {
            // (what does not exist is not counted: thousands of additions to one bin of LDS would wait for each other)
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) {
                const uint32_t key = key_of(__uint_as_float(held[j]));
                if (j < mine && (key & mask) == prefix) atomicAdd(&hist[(key >> shift) & (nb - 1)], 1);
            }
        } else {
            for (int64_t i = tid; i < n; i += T) {
                const uint32_t key = key_of(row[i]);
                if ((key & mask) == prefix) atomicAdd(&hist[(key >> shift) & (nb - 1)], 1);
            }
        }
        __syncthreads();
        pick_digit<T>(hist, nb, remaining, wsum, &found);
        prefix |= (uint32_t)found.digit << shift;
        mask |= (uint32_t)(nb - 1) << shift;
        remaining = found.left;
        if constexpr (RESIDENT) {
            const int count = found.count;
            if (p + 1 < NPASS && count <= FEW_KEYS) {
                int in_digit = 0;
#pragma unroll
                for (int j = 0; j < ITEMS; ++j) in_digit += j < mine && (key_of(__uint_as_float(held[j])) & mask) == prefix;
                int at = take_places(in_digit, &sh.listed);
#pragma unroll
                for (int j = 0; j < ITEMS; ++j) {
                    const uint32_t key = key_of(__uint_as_float(held[j]));
                    if (j < mine && (key & mask) == prefix) sh.few[at++] = key;
                }
                __syncthreads();
                if (tid < 64) {
                    const Cut c = cut_of_listed(sh.few, sh.bins, count, remaining, prefix, shift);
                    if (tid == 0) sh.cut = c;
                }
                __syncthreads();
                prefix = sh.cut.thr;
                remaining = sh.cut.equal;
                break;
            }
        }
    }
    // taken: the elements whose keys lie above prefix, and the first `remaining` of those equal to it
    const uint32_t thr = prefix;
    if constexpr (RESIDENT) {
        int gt = 0, eq = 0;
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const uint32_t key = key_of(__uint_as_float(held[j]));
            gt += j < mine && key > thr;
            eq += j < mine && key == thr;
        }
        int total;
        const int both = block_scan<T>(gt | (eq << 16), wsum, &total) - (gt | (eq << 16));
        int g = both & 0xFFFF, e = (int)((uint32_t)both >> 16);
        if (gt + eq == 0) return;
        int32_t* idx = a.idx + (int64_t)blockIdx.x * a.k;
        float* val = a.val + (int64_t)blockIdx.x * a.k;
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const uint32_t key = key_of(__uint_as_float(held[j]));
            const bool above = j < mine && key > thr, equal = j < mine && key == thr;
            const int pos = g + (e < remaining ? e : remaining);
            if ((above || (equal && e < remaining)) && pos < a.k) {         // (pos < k: always true for NaN-free rows)
                idx[pos] = tid * ITEMS + j;
                val[pos] = __uint_as_float(held[j]);
            }
            g += above;
            e += equal;
        }
    } else {
        const int64_t seg = (n + T - 1) / T;
        const int64_t lo = tid * seg < n ? tid * seg : n, hi = lo + seg < n ? lo + seg : n;
        compact<T>(a, lo, hi, remaining, wsum,
                   [&](int64_t i) { const uint32_t key = key_of(row[i]); return key > thr ? 2 : key == thr ? 1 : 0; },
                   [&](int64_t i) { return row[i]; });
    }
}

// ---- T1 on long rows ------------------------------------------------------------------------------
// One workgroup of 1024 lanes per row (up to 32 rows are cut, below), 16 bytes per lane and load; what bounds it is what
// one CU can fetch.  The general form reads the row five times: three histogram passes and two of ordered compaction.
// The filter reads it twice (8 x 131072, k = 64, not cut: 256 lanes took 460 us, the general form 94, this one 27.5, 23
// since its scans are short, 18.5 and 16 of them for k = 1, where the second read is one lane's; 128 x 200000, k = 100:
// 1426 -> 40) and everything else works on few keys:
//   1. each lane keeps the largest value of four interleaved groups of elements (4096 groups in all);
//   2. the k-th largest of the 4096 maxima is a lower bound of the row's k-th largest value (k groups each hold an
//      element at least that large): two 11-bit digits of it, the rest zero, are bound enough;
//   3. the row is read again, by the lanes only whose own maxima reach the bound, and the elements that reach it are
//      listed in LDS (k = 64 of 131072 normal values: about 65; k = 2048: about 2840 of the 4096 there is room for);
//   4. radix select on the list, a counting sort of it by index, ordered compaction.
// A list that overflows (long runs of values equal to the threshold, rows that put the large values into few groups)
// or k above half the groups takes the general form, after one of the filter's reads or both: six or seven passes.
// Which rows come here (times relative to 256 lanes and five passes, normal values unless noted):
//   up to 512 rows, every length: the general form 0.58 at 4097 elements and k = 64, rows of one value 0.7 to 0.95;
//   more rows, beyond 5000 elements: the workgroups of 256 share the CUs better, 1024 rows of 4097 take 1.05 and 8192
//   rows 1.32 (of one value 1.7), of 5000 0.70 and 0.85 (1.13), of 6000 0.60 and 0.66 (1.05).
// The filter pays from 12288 elements on: general / filter 8192 elements, k = 512, 0.34 / 0.40; 12288 0.30 / 0.31;
// 20000 0.26 / 0.24; 32768 0.23 / 0.17; and where the list overflows its two reads are lost (12288 zeros 0.65 / 0.83;
// rows in ascending order, whose neighbours fall into one bin of the histograms, 0.41 / 0.29).
constexpr int LONG_T = 1024;
constexpr int LONG_GROUPS = 4 * LONG_T;
constexpr int LONG_CAP = 4096;                  // listed elements: 4 per lane
constexpr int LONG_MAX_K = LONG_GROUPS / 2;
constexpr int LONG_MAX_REACH = LONG_GROUPS / 4 * 3;
constexpr int64_t LONG_MANY_ROWS = 512, LONG_MANY_N = 5000, LONG_FILTER_N = 12288;     // (4096 groups need an element each)
typedef float float4_u __attribute__((ext_vector_type(4), aligned(4)));      // rows start at any element

// f(four values, index of the first, how many of them exist) for every run of four that belongs to this lane,
// 16 bytes a load, UNROLL loads in flight
template <int UNROLL, typename F>
__device__ __forceinline__ void for_each_of_lane(const float* row, int64_t n, F f)
{
    const int64_t whole = n & ~(int64_t)3;
    int64_t i = (int64_t)threadIdx.x * 4;
    for (; i + (int64_t)(UNROLL - 1) * LONG_GROUPS < whole; i += (int64_t)UNROLL * LONG_GROUPS) {
        float4_u v[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) v[u] = *(const float4_u*)(row + i + (int64_t)u * LONG_GROUPS);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) f(v[u], i + (int64_t)u * LONG_GROUPS, 4);
    }
    for (; i < n; i += LONG_GROUPS) {
        float4_u v = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        if (i < whole) v = *(const float4_u*)(row + i);
        else
#pragma unroll
            for (int e = 0; e < 3; ++e)
                if (i + e < n) v[e] = row[i + e];
        f(v, i, i < whole ? 4 : (int)(n - i));
    }
}

struct LongShared {
    int hist[2048];
    uint32_t bits[LONG_CAP];                    // the listed elements' patterns, in order of arrival
    int32_t idx[LONG_CAP];
    uint16_t bucketed[LONG_CAP], ordered[LONG_CAP];
    int wsum[LONG_T / 64];
    int wcount[2][LONG_T / 64];
    int bins[64];
    uint32_t few_keys[FEW_KEYS];
    Digit found;
    Cut cut;
    int listed, few;
};

// the k-th largest of the keys held, digit by digit from the top; `passes` digits of 11, 11, 10 bits, the rest zero
template <int ITEMS>
__device__ __forceinline__ uint32_t select_key(LongShared& sh, const uint32_t (&key)[ITEMS], int count, int passes, int& remaining)
{
    const int tid = threadIdx.x;
    uint32_t prefix = 0, mask = 0;
    int shift = 32;
    for (int p = 0; p < passes; ++p) {
        const int bits = p < 2 ? 11 : 10, nb = 1 << bits;
        shift -= bits;
        for (int i = tid; i < nb; i += LONG_T) sh.hist[i] = 0;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ITEMS; ++j)
            if (j * LONG_T + tid < count && (key[j] & mask) == prefix) atomicAdd(&sh.hist[(key[j] >> shift) & (nb - 1)], 1);
        __syncthreads();
        pick_digit<LONG_T>(sh.hist, nb, remaining, sh.wsum, &sh.found);
        prefix |= (uint32_t)sh.found.digit << shift;
        mask |= (uint32_t)(nb - 1) << shift;
        remaining = sh.found.left;
    }
    return prefix;
}

// the cut between the k largest of the keys held and the rest
template <int ITEMS>
__device__ __forceinline__ Cut select_cut(LongShared& sh, const uint32_t (&key)[ITEMS], int count, int k)
{
    const int tid = threadIdx.x;
    int remaining = k;
    if (tid == 0) sh.few = 0;
    const uint32_t first = select_key(sh, key, count, 1, remaining);
    const int in_digit = sh.found.count;
    if (in_digit > FEW_KEYS) {
        remaining = k;
        const uint32_t thr = select_key(sh, key, count, 3, remaining);
        return Cut{thr, remaining};
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
        if (j * LONG_T + tid < count && key[j] >> 21 == first >> 21) sh.few_keys[atomicAdd(&sh.few, 1)] = key[j];
    __syncthreads();
    if (tid < 64) {
        const Cut c = cut_of_listed(sh.few_keys, sh.bins, in_digit, remaining, first, 21);
        if (tid == 0) sh.cut = c;
    }
    __syncthreads();
    return sh.cut;
}

// any k, any values: every pass reads the row
__device__ void long_row_general(const TopkArgs& a, const float* row, LongShared& sh)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint32_t prefix = 0, mask = 0;
    int remaining = (int)a.k, shift = 32;
    for (int p = 0; p < 3; ++p) {
        const int bits = p < 2 ? 11 : 10, nb = 1 << bits;
        shift -= bits;
        for (int i = tid; i < nb; i += LONG_T) sh.hist[i] = 0;
        __syncthreads();
        for_each_of_lane<4>(row, a.n, [&](float4_u v, int64_t, int count) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t key = key_of(v[e]);
                if (e < count && (key & mask) == prefix) atomicAdd(&sh.hist[(key >> shift) & (nb - 1)], 1);
            }
        });
        __syncthreads();
        pick_digit<LONG_T>(sh.hist, nb, remaining, sh.wsum, &sh.found);
        prefix |= (uint32_t)sh.found.digit << shift;
        mask |= (uint32_t)(nb - 1) << shift;
        remaining = sh.found.left;
    }
    // ordered compaction: a wave owns a contiguous run of whole 256-element steps
    const int64_t seg = (a.n + LONG_GROUPS - 1) / LONG_GROUPS * 256;
    const int64_t lo = wave * seg < a.n ? wave * seg : a.n, hi = lo + seg < a.n ? lo + seg : a.n;
    auto fetch = [&](int64_t i, float (&v)[4], bool (&in)[4]) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            in[u] = i + u * 64 + lane < hi;
            v[u] = in[u] ? row[i + u * 64 + lane] : 0.0f;
        }
    };
    float v[4];
    bool in[4];
    int gt = 0, eq = 0;
    for (int64_t i = lo; i < hi; i += 256) {
        fetch(i, v, in);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            gt += __popcll(__ballot(in[u] && key_of(v[u]) > prefix));
            eq += __popcll(__ballot(in[u] && key_of(v[u]) == prefix));
        }
    }
    if (lane == 0) { sh.wcount[0][wave] = gt; sh.wcount[1][wave] = eq; }
    __syncthreads();
    int64_t g = 0, e = 0;
    for (int w = 0; w < wave; ++w) { g += sh.wcount[0][w]; e += sh.wcount[1][w]; }
    int32_t* idx = a.idx + (int64_t)blockIdx.x * a.k;
    float* val = a.val + (int64_t)blockIdx.x * a.k;
    const uint64_t below = ((uint64_t)1 << lane) - 1;
    for (int64_t i = lo; i < hi; i += 256) {
        fetch(i, v, in);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t key = key_of(v[u]);
            const uint64_t mg = __ballot(in[u] && key > prefix), me = __ballot(in[u] && key == prefix);
            const int64_t le = e + __popcll(me & below);
            if (in[u] && (key > prefix || (key == prefix && le < remaining))) {
                const int64_t pos = g + __popcll(mg & below) + (le < remaining ? le : remaining);
                if (pos < a.k) {                        // always true for NaN-free rows
                    idx[pos] = (int32_t)(i + u * 64 + lane);
                    val[pos] = v[u];
                }
            }
            g += __popcll(mg);
            e += __popcll(me);
        }
    }
}

// The k largest of the `listed` elements in LDS, in index order: those that `cut` takes, where it is known.
constexpr int SHORT_K = LONG_T / 4;
__device__ void finish_list(const TopkArgs& a, LongShared& sh, int listed, bool known, Cut cut)
{
    const int tid = threadIdx.x;
    uint32_t key[LONG_CAP / LONG_T];
    int total;
    int32_t pos[LONG_CAP / LONG_T];
#pragma unroll
    for (int j = 0; j < LONG_CAP / LONG_T; ++j) {
        const int c = j * LONG_T + tid;
        key[j] = c < listed ? key_of(__uint_as_float(sh.bits[c])) : 0;
        pos[j] = c < listed ? sh.idx[c] : 0;
    }
    if (!known) cut = select_cut(sh, key, listed, (int)a.k);
    const uint32_t thr = cut.thr;
    const int remaining = cut.equal;
    int32_t* idx = a.idx + (int64_t)blockIdx.x * a.k;
    float* val = a.val + (int64_t)blockIdx.x * a.k;
    // counting sort by index: 2048 buckets of consecutive indices, then the rank among the bucket's few elements
    int shift = 0;
    while (((a.n - 1) >> shift) >= 2048) ++shift;
    sh.hist[2 * tid] = sh.hist[2 * tid + 1] = 0;
    __syncthreads();
    int slot[LONG_CAP / LONG_T];
#pragma unroll
    for (int j = 0; j < LONG_CAP / LONG_T; ++j)
        if (j * LONG_T + tid < listed) slot[j] = atomicAdd(&sh.hist[pos[j] >> shift], 1);
    __syncthreads();
    const int h0 = sh.hist[2 * tid], h1 = sh.hist[2 * tid + 1];
    const int start = block_scan<LONG_T>(h0 + h1, sh.wsum, &total) - h0 - h1;
    sh.hist[2 * tid] = start;
    sh.hist[2 * tid + 1] = start + h0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < LONG_CAP / LONG_T; ++j)
        if (j * LONG_T + tid < listed) sh.bucketed[sh.hist[pos[j] >> shift] + slot[j]] = (uint16_t)(j * LONG_T + tid);
    __syncthreads();
#pragma unroll
    for (int j = 0; j < LONG_CAP / LONG_T; ++j)
        if (j * LONG_T + tid < listed) {
            const int b = pos[j] >> shift, first = sh.hist[b], last = b + 1 < 2048 ? sh.hist[b + 1] : listed;
            int rank = 0;
            for (int c = first; c < last; ++c) rank += sh.idx[sh.bucketed[c]] < pos[j];
            sh.ordered[first + rank] = (uint16_t)(j * LONG_T + tid);
        }
    __syncthreads();
    const int lo = tid * (LONG_CAP / LONG_T);
    int c[LONG_CAP / LONG_T], gt = 0, eq = 0;
#pragma unroll
    for (int j = 0; j < LONG_CAP / LONG_T; ++j) {
        c[j] = lo + j < listed ? sh.ordered[lo + j] : -1;
        key[j] = c[j] >= 0 ? key_of(__uint_as_float(sh.bits[c[j]])) : 0;
        gt += c[j] >= 0 && key[j] > thr;
        eq += c[j] >= 0 && key[j] == thr;
    }
    const int both = block_scan<LONG_T>(gt | (eq << 16), sh.wsum, &total) - (gt | (eq << 16));
    int g = both & 0xFFFF, e = both >> 16;
#pragma unroll
    for (int j = 0; j < LONG_CAP / LONG_T; ++j) {
        if (c[j] < 0) break;
        if (key[j] > thr || (key[j] == thr && e < remaining)) {
            const int at = g + (e < remaining ? e : remaining);
            if (at < a.k) {
                idx[at] = sh.idx[c[j]];
                val[at] = __uint_as_float(sh.bits[c[j]]);
            }
        }
        g += key[j] > thr;
        e += key[j] == thr;
    }
}

// k <= LONG_MAX_K; false (nothing written) when the list does not hold the row's candidates
__device__ bool long_row_filtered(const TopkArgs& a, const float* row, LongShared& sh)
{
    float top[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    auto larger = [](float v, float w) { return __builtin_amdgcn_fmed3f(v, w, INFINITY); };
    for_each_of_lane<8>(row, a.n, [&](float4_u v, int64_t, int) {
#pragma unroll
        for (int e = 0; e < 4; ++e) top[e] = larger(v[e], top[e]);
    });
    uint32_t key[LONG_CAP / LONG_T];
#pragma unroll
    for (int e = 0; e < 4; ++e) key[e] = key_of(top[e]);
    int remaining = (int)a.k;
    const uint32_t bound = select_key(sh, key, LONG_GROUPS, 2, remaining);
    // groups whose maxima reach the bound: each puts an element on the list at least, and far more of them than k means
    // that a run of equal values is the threshold (2048 x 12289 zeros, k = 64: 428 -> 407 us,
    // 383 with 256 lanes and five passes; 64 x 131072: 395 -> 392, 595)
    if ((int)a.k - remaining + sh.found.count > LONG_MAX_REACH) {
        __syncthreads();                        // (the general form clears the histogram)
        return false;
    }
    bool full = false;
    if (key[0] >= bound || key[1] >= bound || key[2] >= bound || key[3] >= bound)
        // (four values are tested at once: with a test per element 8 x 131072, k = 64 took 40 us)
        for_each_of_lane<8>(row, a.n, [&](float4_u v, int64_t i, int count) {
            if (!full && key_of(larger(larger(v[0], v[1]), larger(v[2], v[3]))) >= bound)
                for (int e = 0; e < count; ++e) {
                    const float x = e == 0 ? v[0] : e == 1 ? v[1] : e == 2 ? v[2] : v[3];
                    if (key_of(x) < bound) continue;
                    const int at = atomicAdd(&sh.listed, 1);
                    if (at >= LONG_CAP) {
                        full = true;
                        break;
                    }
                    sh.bits[at] = __float_as_uint(x);
                    sh.idx[at] = (int32_t)(i + e);
                }
        });
    __syncthreads();
    const int listed = sh.listed;
    if (listed > LONG_CAP || listed < a.k) return false;            // fewer than k only where NaNs hid a group's elements
    finish_list(a, sh, listed, false, Cut{});
    return true;
}

__host__ __device__ inline bool long_row_takes_filter(int64_t n, int64_t k) { return n > LONG_FILTER_N && k <= LONG_MAX_K; }

__global__ __launch_bounds__(LONG_T) void topk_long(TopkArgs a)
{
    __shared__ LongShared sh;
    const float* row = a.x + (int64_t)blockIdx.x * a.ld;
    if (threadIdx.x == 0) { sh.found = Digit{0, 0, 0}; sh.listed = 0; }      // a row of NaNs may leave a digit unfound
    if (long_row_takes_filter(a.n, a.k) && long_row_filtered(a, row, sh)) return;
    long_row_general(a, row, sh);
}

// ---- T1 on few long rows ---------------------------------------------------------------------------
// One workgroup reads a row no faster than one CU can fetch, and most CUs have no row.  Here a row is cut into parts of 4096
// elements (blocks of 256 in turn, of 32 where k neighbours have to be shared out), a workgroup each: it keeps its elements in
// registers, finds its own `want`-th largest, digit by digit until few keys share what has been found, and lists its elements
// from there up; of those that equal it, if there are more than there is room for, the first.  A second kernel, one
// workgroup per row, finds the k largest of the lists.  Where there is room for it `want` is k: each part has listed its k
// largest, the first of equal ones first, so the row's are among them.  Otherwise it is what a part holds of k elements spread at
// random, or of k neighbours, and the result is checked, not assumed: in the order of larger keys and then smaller indices a
// part's list is complete down to its bound, or to the last one listed that equals it, so the result holds if k of the listed
// elements come no later than the first of these.  A row for which they do not is read again by the one workgroup as if it had
// not been cut.
// 8 x 131072, k = 64, uncut / cut: normal values 26.8 / 12.5 us, uniform ones 29.1 / 13.9, normal around -10 27.3 / 12.9, rounded to
// bf16 26.9 / 15.3, to halves 29.3 / 19.5, one value 392 / 45, sorted 25.8 / 13.9; k = 500, for which there is no room: normal
// 38.1 / 14.4, one value 393 / 45, sorted 26.0 / 19.3; 31 x 197076, k = 1, normal 26.9 / 23.6, sorted 29.0 / 27.1.  (With 120
// elements listed per part whatever k is, bounds no finer than the first digit where more than 512 keys share it, equal elements
// beyond the room sent to the uncut form, and bounds joined by additions to one word of LDS: normal 15.2, uniform 36, one value
// 400, sorted 18.0 and for k = 500 42; 31 x 197076 29.4 and 46.)
//
// The lists are device memory of the loaded library (one copy per GPU, held until the process ends), because the interface
// lends no scratch.  A call's rows take consecutive slots from a ticket; the first part to arrive claims the row's slot for the
// address of the row's output, which no other call that runs at the same time can share, later parts join it, and the second
// kernel gives it back.  A part that finds its slot held by another call's row (more than PART_SLOTS rows in flight on several
// streams) leaves: the second kernel then sees that not all parts came, and reads the row itself.  Nothing waits for anything.
constexpr int PART_N = 4 * LONG_T;
constexpr int PART_SLOTS = 128, PART_LIST = LONG_CAP, PART_MAX = 64;       // rows, elements listed per row, parts per row
struct PartSlot {
    unsigned long long owner;           // address of the row's indices, 0: free
    unsigned int arrived;
    uint2 part[PART_MAX];               // elements from the bound up (as many are listed as there is room for) and bound of each part
    unsigned int last[PART_MAX];        // where they are more: index of the last one listed that equals the bound
    uint2 list[PART_LIST];              // pattern and index; part i's begin at i * room
};
__device__ PartSlot part_slots[PART_SLOTS];
struct PartArgs { int parts, room, want, lanes; unsigned int room_inverse, first_slot; };     // room_inverse: 2^32 / room, rounded up

__global__ __launch_bounds__(LONG_T) void topk_parts(TopkArgs a, PartArgs p)
{
    __shared__ int hist[2048];              // (less than topk_merge holds)
    __shared__ int wsum[2][LONG_T / 64];
    __shared__ uint32_t few[FEW_KEYS];
    __shared__ int bins[64], listed, ok;
    __shared__ Digit found;
    __shared__ Cut cut;
    const int tid = threadIdx.x, row_no = (int)blockIdx.x / p.parts, part = (int)blockIdx.x % p.parts;
    const float* row = a.x + (int64_t)row_no * a.ld;
    PartSlot& slot = part_slots[(p.first_slot + (unsigned)row_no) % PART_SLOTS];
    // blocks of 4 << p.lanes elements, four per lane
    const int first = (((tid >> p.lanes) * p.parts + part) << (p.lanes + 2)) + 4 * (tid & ((1 << p.lanes) - 1));      // (PART_MAX parts: below 2^18)
    const int there = first >= a.n ? 0 : first + 4 <= a.n ? 4 : (int)a.n - first;
    float4_u held = {0, 0, 0, 0};
    if (there == 4) held = *(const float4_u*)(row + first);
    else
        for (int e = 0; e < there; ++e) held[e] = row[first + e];
    if (tid == 0) {
        const unsigned long long tag = (unsigned long long)(uintptr_t)(a.idx + (int64_t)row_no * a.k);
        unsigned long long seen = 0;
        ok = __hip_atomic_compare_exchange_strong(&slot.owner, &seen, tag, __ATOMIC_ACQUIRE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) || seen == tag;
        listed = 0;
        found = Digit{0, 0, 0};
    }
    hist[tid] = hist[LONG_T + tid] = 0;
    __syncthreads();
    if (!ok) return;
    uint32_t key[4], bin[4];
    bool on[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        key[e] = key_of(held[e]);
        bin[e] = key[e] >> 21;
        on[e] = e < there;
    }
    count_bins(hist, bin, on);
    __syncthreads();
    pick_digit<LONG_T>(hist, 2048, p.want, wsum[0], &found);
    // the elements of the digit found and of those above it, where there is room for them; else from the want-th largest up
    uint32_t bound = (uint32_t)found.digit << 21;         // (fewer than `want` elements: 0, all of them are listed)
    int shift = 21, left = found.left, count = found.count;
    while (shift > 0 && p.want - left + count > p.room && count > FEW_KEYS) {       // 11 bits more, then the last 10
        const int low = shift > 11 ? shift - 11 : 0, bits = shift - low;
        hist[tid] = hist[LONG_T + tid] = 0;
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            bin[e] = (key[e] >> low) & ((1u << bits) - 1);
            on[e] = e < there && key[e] >> shift == bound >> shift;
        }
        count_bins(hist, bin, on);
        __syncthreads();
        pick_digit<LONG_T>(hist, 1 << bits, left, wsum[0], &found);
        bound |= (uint32_t)found.digit << low;
        left = found.left;
        count = found.count;
        shift = low;
    }
    if (shift > 0 && p.want - left + count > p.room) {
        int in_digit = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) in_digit += e < there && key[e] >> shift == bound >> shift;
        int at = take_places(in_digit, &listed);
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (e < there && key[e] >> shift == bound >> shift) few[at++] = key[e];
        __syncthreads();
        if (tid < 64) {
            const Cut c = cut_of_listed(few, bins, count, left, bound, shift);
            if (tid == 0) cut = c;
        }
        __syncthreads();
        bound = cut.equal > 0 ? cut.thr : cut.thr + 1;
    }
    // (more than there is room for only where `bound` is the want-th largest key itself)
    int gt = 0, eq = 0, totals;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        gt += e < there && key[e] > bound;
        eq += e < there && key[e] == bound;
    }
    const int before = join_scan<LONG_T>(wave_scan(gt | (eq << 16)), wsum[1], &totals) - (gt | (eq << 16));
    const int above = totals & 0xFFFF, equal = totals >> 16, keep = p.room - above;
    if (gt + eq > 0) {
        uint2* list = slot.list + part * p.room;
        int g = before & 0xFFFF, e0 = before >> 16;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const bool is_gt = e < there && key[e] > bound, is_eq = e < there && key[e] == bound;
            if (is_gt || (is_eq && e0 < keep)) list[g + (e0 < keep ? e0 : keep)] = make_uint2(__float_as_uint(held[e]), (uint32_t)(first + e));
            if (is_eq && e0 == keep - 1) slot.last[part] = (unsigned)(first + e);
            g += is_gt;
            e0 += is_eq;
        }
    }
    if (tid == 0) {
        slot.part[part] = make_uint2((unsigned)(above + equal), bound);
        __hip_atomic_fetch_add(&slot.arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

constexpr int MERGE_LDS = sizeof(LongShared) + PART_MAX * sizeof(uint2) + 5 * sizeof(unsigned int);     // (one struct of them all measured 0.1 us slower)
__global__ __launch_bounds__(LONG_T) void topk_merge(TopkArgs a, PartArgs p)
{
    constexpr int ITEMS = PART_LIST / LONG_T;
    __shared__ LongShared sh;
    __shared__ uint2 part[PART_MAX];
    __shared__ unsigned long long bound;
    __shared__ unsigned int lowest, highest, tied;
    const int tid = threadIdx.x;
    const float* row = a.x + (int64_t)blockIdx.x * a.ld;
    PartSlot& slot = part_slots[(p.first_slot + blockIdx.x) % PART_SLOTS];
    const unsigned long long tag = (unsigned long long)(uintptr_t)(a.idx + (int64_t)blockIdx.x * a.k);
    // all that may be wanted is loaded at once: each wait is a trip to what another XCD has written
    const unsigned long long owner = slot.owner;
    const unsigned int arrived = slot.arrived;
    const uint2 mine = tid < PART_MAX ? slot.part[tid] : make_uint2(0, 0);
    const unsigned int last = tid < PART_MAX ? slot.last[tid] : 0;
    uint2 entry[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) entry[j] = slot.list[j * LONG_T + tid];
    sh.hist[tid] = sh.hist[LONG_T + tid] = 0;
    const bool held = owner == tag;
    // An element's place in the order of the row, larger keys and then smaller indices first.  For k > want: from which place on
    // all parts' lists are complete.
    auto order_of = [](uint32_t key, uint32_t index) { return (unsigned long long)key << 32 | ~index; };
    const bool left_out = mine.x > (unsigned)p.room;
    if (tid < PART_MAX) {
        static_assert(PART_MAX == 64, "a part per lane of one wave");
        const bool is_part = tid < p.parts;
        const uint32_t key = __builtin_amdgcn_readlane(wave_max(is_part ? mine.y : 0u), 63), low = ~__builtin_amdgcn_readlane(wave_max(is_part ? ~mine.y : 0u), 63);
        const uint32_t index = ~__builtin_amdgcn_readlane(wave_max(is_part && left_out && mine.y == key ? ~last : 0u), 63);
        part[tid] = mine;
        if (tid == 0) {
            sh.found = Digit{0, 0, 0};
            sh.listed = sh.few = 0;
            lowest = low;
            bound = a.k > p.want ? order_of(key, index) : 0;
            highest = tied = 0;
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);                 // every wave's loads of the list have come (a barrier does not wait for them)
    __syncthreads();
    // (all of the slot has been read; while it is held nobody else changes it)
    if (held && tid == 0) {
        __hip_atomic_store(&slot.arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&slot.owner, 0ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (held && arrived == (unsigned)p.parts) {
        bool there[ITEMS];
        uint32_t key[ITEMS], top = 0;
        int sure = 0, all_sure = (int)a.k;
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const unsigned i = j * LONG_T + tid, of = __umulhi(i, p.room_inverse);
            there[j] = of < (unsigned)p.parts && i - of * p.room < part[of < PART_MAX ? of : 0].x;
            key[j] = key_of(__uint_as_float(entry[j].x));
            sure += there[j] && order_of(key[j], entry[j].y) >= bound;
            if (there[j] && key[j] > top) top = key[j];
        }
        top = wave_max(top);
        if ((tid & 63) == 63) atomicMax(&highest, top);
        if (a.k > p.want) join_scan<LONG_T>(wave_scan(sure), sh.wsum, &all_sure);
        else __syncthreads();
        if (all_sure >= a.k) {
            // The keys lie between the lowest bound and the highest key: 2047 bins over that range (a few bins of the key's
            // top bits would hold nearly all of them, and additions to one bin wait for each other).
            const uint32_t range = highest - lowest;
            int shift = range < 2048 ? 0 : 21 - __clz(range);                   // range >> shift: 1024 .. 2047
            if (range >> shift > 2046) ++shift;
            auto place_of = [&](uint32_t k) { return k - lowest + (1u << shift); };       // (bins from 1: see cut_of_listed on 0)
            uint32_t bin[ITEMS];
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) bin[j] = place_of(key[j]) >> shift;
#pragma unroll
            for (int j = 0; j < ITEMS; ++j)
                if (there[j]) atomicAdd(&sh.hist[bin[j]], 1);
            __syncthreads();
            pick_digit<LONG_T>(sh.hist, 2048, (int)a.k, sh.wsum, &sh.found);
            const uint32_t digit = sh.found.digit;
            const int count = sh.found.count;
            Cut c = {digit << shift, sh.found.left};
            const bool known = count <= FEW_KEYS || shift == 0;
            if (count <= FEW_KEYS) {
                int in_digit = 0;
#pragma unroll
                for (int j = 0; j < ITEMS; ++j) in_digit += there[j] && bin[j] == digit;
                int to = take_places(in_digit, &sh.few);
#pragma unroll
                for (int j = 0; j < ITEMS; ++j)
                    if (there[j] && bin[j] == digit) sh.few_keys[to++] = place_of(key[j]);
                __syncthreads();
                if (tid < 64) {
                    const Cut w = cut_of_listed(sh.few_keys, sh.bins, count, sh.found.left, digit << shift, shift);
                    if (tid == 0) sh.cut = w;
                }
                __syncthreads();
                c = sh.cut;
            }
            // those that may be taken: the k keys above c.thr where the cut is a clean one, and what equals it (or shares its bin,
            // many as they are) where not
            const bool clean = known && c.equal == 0;
            const uint32_t first = clean ? c.thr + 1 : c.thr;
            int taken = 0;
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) taken += there[j] && place_of(key[j]) >= first;
            int to = take_places(taken, &sh.listed);
#pragma unroll
            for (int j = 0; j < ITEMS; ++j)
                if (there[j] && place_of(key[j]) >= first) {
                    sh.bits[to] = entry[j].x;
                    sh.idx[to++] = (int32_t)entry[j].y;
                }
            __syncthreads();
            const int k = (int)a.k, q = tid >> 2;           // four lanes for one
            if (clean && k <= SHORT_K) {
                // their order by index is each one's rank among them
                if (q < k) {
                    const int32_t index = sh.idx[q];
                    int rank = 0;
                    for (int i = tid & 3; i < k; i += 4) rank += sh.idx[i] < index;
                    rank += __shfl_xor(rank, 1, 64);
                    rank += __shfl_xor(rank, 2, 64);
                    if ((tid & 3) == 0) {
                        a.idx[(int64_t)blockIdx.x * a.k + rank] = index;
                        a.val[(int64_t)blockIdx.x * a.k + rank] = __uint_as_float(sh.bits[q]);
                    }
                }
                return;
            }
            // (the cut as a key again; a clean one's lies above the key 0, which no number has)
            const uint32_t from = first + lowest - (1u << shift);
            finish_list(a, sh, sh.listed, known, Cut{clean ? (from > 0 ? from - 1 : 0) : from, c.equal});
            return;
        }
        // the row's k-th largest lies at the key of the bound or below: where more elements than the filter can list lie from there up,
        // it is not tried
        if (tid < p.parts && left_out && mine.y == (unsigned)(bound >> 32)) atomicAdd(&tied, mine.x);
        __syncthreads();
    }
    if (tied <= LONG_CAP && long_row_takes_filter(a.n, a.k) && long_row_filtered(a, row, sh)) return;
    long_row_general(a, row, sh);
}

// Gives the slots back that topk_parts has claimed, one workgroup per row, when topk_merge could not be launched.
__global__ void topk_give_back(TopkArgs a, PartArgs p)
{
    PartSlot& slot = part_slots[(p.first_slot + blockIdx.x) % PART_SLOTS];
    if (threadIdx.x != 0 || slot.owner != (unsigned long long)(uintptr_t)(a.idx + (int64_t)blockIdx.x * a.k)) return;
    __hip_atomic_store(&slot.arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&slot.owner, 0ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// Which rows are cut: up to 32 of them (beyond, one workgroup per row has enough CUs: uncut / cut, k = 16, 64 x 32768 16.1 /
// 16.0 us, 64 x 131072 26.4 / 32.6, 128 x 131072 29.1 / 52.0, when each part listed up to 120 elements), longer than the resident
// state takes.  Uncut / cut: 1 x 17000, k = 16, 14.7 / 9.3; 24 x 24000, k = 200, 21.7 / 13.1; 8 x 131072, k = 64, 26.7 / 12.4; 1 x
// 200000, k = 16, 27.4 / 10.4; 24 x 200000, k = 16, 34.7 / 21.0.  More than SHORT_K elements are put in order by finish_list: their
// line lies where cutting paid when that sorted the whole list (k = 500, 8 x 32768 21.4 / 20.0, 8 x 50000 27.0 / 20.9, now 27.3 /
// 12.9; 1 x 131072, k = 1500, 48.1 / 15.3); with a list of candidates only it would pay from PART_FROM_N on (8 x 17000 15.6 /
// 13.8, 8 x 32768 18.9 / 14.5).
constexpr int64_t PART_FROM_N = 16384, PART_FROM_N_MANY = 49152, PART_ROWS = 32;
PartArgs parts_of(int64_t batch, int64_t n, int64_t k)
{
    const int64_t parts = (n + PART_N - 1) / PART_N;
    if (batch < 1 || batch > PART_ROWS || n <= (k <= SHORT_K ? PART_FROM_N : PART_FROM_N_MANY) || parts > PART_MAX || k < 1) return PartArgs{};
    const int room = (int)(PART_LIST / parts), most = room - room / 16;      // (a sixteenth is left for elements that share the last one's first digits)
    const unsigned room_inverse = (unsigned)((((uint64_t)1 << 32) + room - 1) / room);
    if (k <= most) return PartArgs{(int)parts, room, (int)k, 6, room_inverse, 0};
    // Of k elements spread at random a part holds more than `spread` once in a million, of k neighbours dealt out in blocks of 32 at
    // most `run`, and one more shows that they were all.  (Blocks of 256 are read a little faster: 32 x 50000, k = 100, 16.4 us
    // against 16.7.)
    const double mean = (double)k / (double)parts;
    const int spread = (int)__builtin_ceil(mean + 5 * __builtin_sqrt(mean) + 8), run = 32 * (int)(((k + 62) / 32 + parts - 1) / parts);
    if (spread > most || run >= most) return PartArgs{};
    return PartArgs{(int)parts, room, spread > run ? spread : run + 1, 3, room_inverse, 0};
}
std::atomic<unsigned> part_ticket{0};

constexpr int RES_ITEMS = 16;

struct Plan {
    int status = GEMM_OK;
    bool empty = false;
    TopkArgs a{};
    int threads = 0;
    int items = 0;          // T2: keys per lane
    PartArgs parts{};       // T1: a row's parts (0: rows are not cut)
    hipStream_t stream = nullptr;
    topk_query_t q{};
};

Plan make_plan(int variant, const topk_desc_t* d, const float* x, const void* idx, const void* val, bool need_ptrs)
{
    Plan p;
    auto fail = [&](int s) { p.status = s; return p; };
    if (variant < 0 || variant >= TOPK_VARIANT_COUNT) return fail(GEMM_ERR_BAD_VARIANT);
    if (!d) return fail(GEMM_ERR_BAD_ARG);
    if (d->batch < 0 || d->n < 0 || d->k < 0 || d->k > d->n || d->ld < d->n || d->flags != 0 || d->reserved != 0) return fail(GEMM_ERR_BAD_ARG);
    if (d->n >= ((int64_t)1 << 31) || d->batch >= ((int64_t)1 << 31)) return fail(GEMM_ERR_BAD_ARG);
    p.empty = d->batch == 0 || d->k == 0;
    if (need_ptrs && !p.empty && (!x || !idx || !val)) return fail(GEMM_ERR_BAD_ARG);
    p.a = TopkArgs{x, (int32_t*)idx, (float*)val, d->n, d->k, d->ld};
    p.stream = (hipStream_t)d->stream;

    uint32_t holds = 0, required = 0;
    if (d->n <= SEL_MAX_N) holds |= TOPK_COND_ROW_IN_LDS;
    if (d->n <= 1024 * RES_ITEMS) holds |= TOPK_COND_ROW_IN_REGISTERS;
    if ((!x || ((uintptr_t)x & 15u) == 0) && d->ld % 4 == 0) holds |= TOPK_COND_ALIGN16;
    const char* path = "";
    topk_query_t& q = p.q;
    switch (variant) {
    case TOPK_T0_SELECTION:
        required = TOPK_COND_ROW_IN_LDS;
        path = "selection(k arg-max rounds)";
        p.threads = SEL_T; q.passes = (int32_t)(d->k < 0x7FFFFFFF ? d->k : 0x7FFFFFFF); q.lds_bytes = SEL_MAX_N + 48;
        break;
    case TOPK_T1_RADIX_SELECT:
        p.parts = parts_of(d->batch, d->n, d->k);
        if (p.parts.parts > 0) {
            path = "parts of 4096 listed and merged, else group-maxima filter";
            p.threads = LONG_T; q.passes = 1; q.lds_bytes = MERGE_LDS;
            break;
        }
        // (the lines: see topk_long; a launch holds fewer than 2^32 threads, so 2^22 rows and more stay with 256 lanes each)
        if (d->n > (d->batch > LONG_MANY_ROWS ? LONG_MANY_N : 4096) && d->batch < ((int64_t)1 << 32) / LONG_T) {
            const bool filter = long_row_takes_filter(d->n, d->k);
            path = filter ? "group-maxima filter, else radix-select(11+11+10), 1024 lanes" : "radix-select(11+11+10, streaming, 1024 lanes)";
            p.threads = LONG_T; q.passes = filter ? 2 : 5; q.lds_bytes = sizeof(LongShared);
            break;
        }
        path = "radix-select(8+8+8+8, streaming)";
        p.threads = 256; q.passes = 5; q.lds_bytes = sizeof(RadixShared<256, 256, false>);
        break;
    default:
        required = TOPK_COND_ROW_IN_REGISTERS | TOPK_COND_ALIGN16;
        // 1024 lanes per row: 64 rows keep a quarter of the CUs busy, so the work per lane is what counts
        // (batch 64, n 4096, k 512: 15.5 us with 256 lanes x 16 keys, 10.2 us with 1024 lanes x 4 keys)
        p.threads = 1024;
        p.items = d->n <= 1024 * 4 ? 4 : RES_ITEMS;
        path = p.items == 4 ? "radix-select(11+11+10, 4 keys/lane x 1024)" : "radix-select(11+11+10, 16 keys/lane x 1024)";
        q.passes = 4; q.lds_bytes = sizeof(RadixShared<1024, 2048, true>);
        break;
    }
    q.required = required; q.holds = holds; q.violated = required & ~holds;
    q.threads = p.threads;
    q.grid = p.empty ? 0 : d->batch * (p.parts.parts > 0 ? p.parts.parts : 1);
    strncpy(q.path, path, sizeof(q.path) - 1);
    if (q.violated) p.status = GEMM_ERR_PRECONDITION;
    return p;
}

thread_local hipError_t last_topk_launch_error = hipSuccess;

}  // namespace

extern "C" {

int topk_query(int variant, const topk_desc_t* d, const float* x, topk_query_t* out)
{
    if (!out) return GEMM_ERR_BAD_ARG;
    Plan p = make_plan(variant, d, x, nullptr, nullptr, /*need_ptrs=*/false);
    memset(out, 0, sizeof(*out));
    if (p.status == GEMM_OK || p.status == GEMM_ERR_PRECONDITION) *out = p.q;
    return p.status;
}

int topk_run(int variant, const topk_desc_t* d, const float* x, int32_t* idx, float* val)
{
    Plan p = make_plan(variant, d, x, idx, val, /*need_ptrs=*/true);
    if (p.status != GEMM_OK) return p.status;
    if (p.empty) return GEMM_OK;
    (void)hipGetLastError();
    hipError_t e = hipSuccess;
    const dim3 grid((unsigned)d->batch);
    if (variant == TOPK_T0_SELECTION)
        hipLaunchKernelGGL(topk_selection, grid, dim3(SEL_T), 0, p.stream, p.a);
    else if (p.parts.parts > 0) {
        p.parts.first_slot = part_ticket.fetch_add((unsigned)d->batch, std::memory_order_relaxed);
        hipLaunchKernelGGL(topk_parts, dim3((unsigned)p.q.grid), dim3(LONG_T), 0, p.stream, p.a, p.parts);
        e = hipGetLastError();
        if (e == hipSuccess) {
            hipLaunchKernelGGL(topk_merge, grid, dim3(LONG_T), 0, p.stream, p.a, p.parts);
            e = hipGetLastError();
            if (e != hipSuccess) {
                hipLaunchKernelGGL(topk_give_back, grid, dim3(64), 0, p.stream, p.a, p.parts);
                (void)hipGetLastError();
            }
        }
    } else if (variant == TOPK_T1_RADIX_SELECT && p.threads == LONG_T)
        hipLaunchKernelGGL(topk_long, grid, dim3(LONG_T), 0, p.stream, p.a);
    else if (variant == TOPK_T1_RADIX_SELECT)
        hipLaunchKernelGGL((topk_radix<256, 1, false, 4, 8, 8, 8, 8>), grid, dim3(256), 0, p.stream, p.a);
    else if (p.items == 4)
        hipLaunchKernelGGL((topk_radix<1024, 4, true, 3, 11, 11, 10, 0>), grid, dim3(1024), 0, p.stream, p.a);
    else
        hipLaunchKernelGGL((topk_radix<1024, RES_ITEMS, true, 3, 11, 11, 10, 0>), grid, dim3(1024), 0, p.stream, p.a);
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) last_topk_launch_error = e;
    return e == hipSuccess ? GEMM_OK : GEMM_ERR_LAUNCH;
}

const char* topk_last_launch_error(void) { return hipGetErrorString(last_topk_launch_error); }

const char* topk_variant_name(int v)
{
    static const char* names[] = {"T0_selection", "T1_radix_select", "T2_resident_coarse_refine"};
    return (v >= 0 && v < TOPK_VARIANT_COUNT) ? names[v] : "?";
}

const char* topk_variant_intent(int v)
{
    static const char* intents[] = {"(start of lineage)", "radix_select", "keys resident in registers; coarse + refine pass"};
    return (v >= 0 && v < TOPK_VARIANT_COUNT) ? intents[v] : "?";
}

const char* topk_cond_name(uint32_t bit)
{
    switch (bit) {
    case TOPK_COND_ROW_IN_LDS: return "ROW_IN_LDS";
    case TOPK_COND_ROW_IN_REGISTERS: return "ROW_IN_REGISTERS";
    case TOPK_COND_ALIGN16: return "ALIGN16";
    default: return "?";
    }
}

int topk_variant_count(void) { return TOPK_VARIANT_COUNT; }

}  // extern "C"
