// Per-query selection and exact re-scoring (gfx950).
//
//  select_kernel   exact k'-th best of a query's candidate keys; writes it as the admission key
//                  for the next scan stage and cuts the list down to its k' best keys in place.
//  rescore_kernel  for the k' rows kept by the scan: inner product with the fp32 query from
//                  the EXACT datastore copy, products and sum in double, one rounding to
//                  fp32; final ranking (score descending, id ascending); first k written.
//                  This is what makes the result that of the paper's exact dense retriever
//                  (Section 5.1) although the scan ran in bf16/fp16.  It also checks that
//                  result: the gap between the exact rank-k score and the scan's score of the
//                  worst kept candidate must exceed what the scan's rounding can do to a
//                  score (judged from the rounding errors seen on the candidates themselves);
//                  a query that fails the check, or whose list lost entries, is queued for
//  exact_scan_kernel / exact_finish_kernel: every row of the exact copy is scored exactly
//                  against the queued queries, the rows that reach the query's exact rank-k
//                  key are collected, and the best k of them are the answer.  Both kernels
//                  are always launched and return at once when nothing is queued.
#include <type_traits>

#include <atomic>

#include "ralm_common.h"
#include "ralm_kernels.h"

namespace ralm {

namespace {

constexpr int SEL_THREADS = 1024;   // of the workgroups that rank a list (lists known to be short take fewer)

// Exact rank-th best (1-based) key of c[0, n), n >= rank >= 1, by a radix descent over the 64-bit
// ranking key, 8 bits per pass from the top.  A pass histograms the digit of the keys that match
// the prefix found so far; wave 0 walks the 256 bins from the best digit down to the one that
// holds the wanted key.  As soon as that bin holds a single key the descent stops and one more
// pass over the list fetches that key (scores are mostly distinct, so this usually happens
// before the id bits are reached).  Called by all NT threads of a workgroup; keys must be
// distinct.
struct RadixShared {
    uint32_t hist[256];
    uint32_t digit, remaining, bin;
    u64 kth;
};

template <int NT>
__device__ u64 radix_kth(const u64 *__restrict__ c, uint32_t n, uint32_t rank, RadixShared &sh)
{
    const int tid = threadIdx.x, lane = tid & 63;
    u64 prefix = 0, mask = 0;
    uint32_t remaining = rank;
    bool single = false;
    for (int shift = 56; shift >= 0; shift -= 8) {
        if (tid < 256) sh.hist[tid] = 0;
        __syncthreads();
        for (uint32_t i = tid; i < n; i += NT) {
            const u64 key = c[i];
            if ((key & mask) == prefix) atomicAdd(&sh.hist[(uint32_t)(key >> shift) & 255u], 1u);
        }
        __syncthreads();
        if (tid < 64) {
            // lane l owns digits 255-4l .. 252-4l, best first
            uint32_t h[4], tot = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                h[j] = sh.hist[255 - 4 * lane - j];
                tot += h[j];
            }
            uint32_t incl = tot;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t y = __shfl_up(incl, o, 64);
                if (lane >= o) incl += y;
            }
            uint32_t run = incl - tot;   // keys in better digits than this lane's
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (run < remaining && run + h[j] >= remaining) {
                    sh.digit = 255 - 4 * lane - j;
                    sh.remaining = remaining - run;
                    sh.bin = h[j];
                }
                run += h[j];
            }
        }
        __syncthreads();
        prefix |= (u64)sh.digit << shift;
        mask |= 0xffull << shift;
        remaining = sh.remaining;
        if (sh.bin == 1) {
            single = shift > 0;
            break;
        }
    }
    u64 kth = prefix;
    if (single) {   // the only key under the prefix is the wanted one
        for (uint32_t i = tid; i < n; i += NT) {
            const u64 key = c[i];
            if ((key & mask) == prefix) sh.kth = key;
        }
        __syncthreads();
        kth = sh.kth;
    }
    __syncthreads();   // sh may be reused by the caller's next call
    return kth;
}

// ---- the best `rank` keys of a list -----------------------------------------------------------
// The digits of a radix descent are a poor histogram for scores: the top byte of a float is its
// sign and most of its exponent, so thousands of keys fall into two or three bins and their LDS
// atomics queue on one address.  Here the bins divide the range of the list's scores evenly (the map
// from score to bin is monotone, so it never reorders keys), which spreads the bulk and leaves a
// handful of keys in the bin that holds the wanted one; those are ranked by counting.  Lists of up
// to SEL_REGS keys per thread are read once and stay in registers.  What bounds it now is that one
// read and the barriers.  15872 keys, one list per workgroup: 81 lists 23 -> 10 us, 1024
// lists 65 -> 38 us, 2341 lists 227 -> 113 us.  A range that is not positive and finite, or a bin with more keys
// than SEL_BIN_KEYS (many equal or nearly equal scores), takes the radix descent.
constexpr int SEL_REGS = 16, SEL_BIN_KEYS = 1024;

template <int NT>
struct SelectShared {
    union {
        uint32_t hist[2 * NT];
        RadixShared radix;
    };
    u64 bin_keys[SEL_BIN_KEYS];
    uint32_t lo[NT / 64], hi[NT / 64], total[NT / 64];
    uint32_t bin, rest, in_bin, n_bin, n_out;
    uint32_t early_bin, early_bits, n_above;
    u64 kth;
};

// Exact rank-th best key of c[0, n), n >= rank >= 1, and the keys that reach it (exactly `rank`:
// keys are distinct) in out[0, rank), in any order.  All NT threads of a workgroup; out is in
// LDS and complete when the function returns; c is not read after that.
// early: the wanted key, or if 0 < early_rank < rank a better one that at least early_rank of the list reach, as few as the bins tell apart.
// REGS: keys per thread that are held in registers.  FITS: n <= REGS * NT, so that the form that walks a longer list in memory is not compiled.
template <int NT, int REGS = SEL_REGS, bool FITS = false>
__device__ __forceinline__ u64 select_best(const u64 *__restrict__ c, uint32_t n, uint32_t rank, SelectShared<NT> &sh, u64 *out,
                                           uint32_t early_rank, u64 &early)
{
    constexpr int SEL_BINS = 2 * NT, SEL_WAVES = NT / 64;
    const bool want_early = early_rank > 0 && early_rank < rank;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool in_regs = FITS || n <= (uint32_t)(REGS * NT);
    u64 reg[REGS];
    if (in_regs) {
#pragma unroll
        for (int i = 0; i < REGS; ++i) {
            const uint32_t at = (uint32_t)(i * NT + tid);
            reg[i] = at < n ? c[at] : 0ull;    // 0 is no key: scores of any value have non-zero keys
        }
    }
    // f(key) for every key of the list and for zeros in between; every thread takes part in each step
    auto each = [&](auto f) __attribute__((always_inline)) {
        if (in_regs) {
#pragma unroll
            for (int i = 0; i < REGS; ++i)
                if ((uint32_t)(i * NT) < n) f(reg[i]);
        } else {
            for (uint32_t i = 0; i < n; i += NT) f(i + tid < n ? c[i + tid] : 0ull);
        }
    };

    // range of the score bits
    uint32_t lo = 0xffffffffu, hi = 0u;
    each([&](u64 key) {
        const uint32_t b = (uint32_t)(key >> 32);
        lo = key && b < lo ? b : lo;
        hi = key && b > hi ? b : hi;
    });
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t l2 = __shfl_xor(lo, o, 64), h2 = __shfl_xor(hi, o, 64);
        lo = l2 < lo ? l2 : lo;
        hi = h2 > hi ? h2 : hi;
    }
    if (lane == 0) {
        sh.lo[wave] = lo;
        sh.hi[wave] = hi;
    }
    for (int i = tid; i < SEL_BINS; i += NT) sh.hist[i] = 0;
    if (tid == 0) {
        sh.n_bin = sh.n_out = sh.n_above = 0;
        sh.early_bits = 0xffffffffu;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < SEL_WAVES; ++w) {
        lo = sh.lo[w] < lo ? sh.lo[w] : lo;
        hi = sh.hi[w] > hi ? sh.hi[w] : hi;
    }
    const float s_lo = bits_score(lo), range = bits_score(hi) - s_lo, scale = (float)SEL_BINS / range;
    // (NaN compares false; scale may overflow for a range of denormals)
    bool even = range > 0.f && range < __builtin_inff() && scale < __builtin_inff();
    auto bin_of = [&](u64 key) __attribute__((always_inline)) {
        const uint32_t b = (uint32_t)((bits_score((uint32_t)(key >> 32)) - s_lo) * scale);
        return b < (uint32_t)SEL_BINS ? b : (uint32_t)SEL_BINS - 1u;
    };
    if (even) {
        each([&](u64 key) {
            if (key) atomicAdd(&sh.hist[bin_of(key)], 1u);
        });
        __syncthreads();
        // thread t owns bins SEL_BINS-1-2t and SEL_BINS-2-2t, best first
        const uint32_t h0 = sh.hist[SEL_BINS - 1 - 2 * tid], h1 = sh.hist[SEL_BINS - 2 - 2 * tid];
        uint32_t incl = h0 + h1;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o, 64);
            if (lane >= o) incl += y;
        }
        if (lane == 63) sh.total[wave] = incl;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < SEL_WAVES; ++w) incl += w < wave ? sh.total[w] : 0u;
        uint32_t better = incl - h0 - h1;     // keys in better bins than this thread's
        if (better < rank && rank <= incl) {
            const bool first = rank <= better + h0;
            sh.bin = (uint32_t)(SEL_BINS - 1 - 2 * tid - (first ? 0 : 1));
            sh.rest = rank - better - (first ? 0u : h0);
            sh.in_bin = first ? h0 : h1;
        }
        if (want_early && better < early_rank && early_rank <= incl)
            sh.early_bin = (uint32_t)(SEL_BINS - 1 - 2 * tid - (early_rank <= better + h0 ? 0 : 1));
        __syncthreads();
        even = sh.in_bin <= (uint32_t)SEL_BIN_KEYS;
    }
    u64 kth;
    if (even) {
        const uint32_t bin = sh.bin, in_bin = sh.in_bin, rest = sh.rest, early_bin = want_early ? sh.early_bin : bin;
        each([&](u64 key) {
            if (!key) return;
            const uint32_t b = bin_of(key);
            if (b == bin) sh.bin_keys[atomicAdd(&sh.n_bin, 1u)] = key;
            else if (b == early_bin) atomicMin(&sh.early_bits, (uint32_t)(key >> 32));
        });
        __syncthreads();
        for (uint32_t i = tid; i < in_bin; i += NT) {
            const u64 mine = sh.bin_keys[i];
            uint32_t better = 0;
            for (uint32_t j = 0; j < in_bin; ++j) better += sh.bin_keys[j] > mine ? 1u : 0u;
            if (better == rest - 1) sh.kth = mine;
        }
        __syncthreads();
        kth = sh.kth;
        // the worst score of the bin that holds the early rank; in the wanted key's own bin that key itself
        early = early_bin == bin ? kth : (u64)sh.early_bits << 32;
    } else {
        __syncthreads();
        kth = radix_kth<NT>(c, n, rank, sh.radix);
        early = kth;
    }
    each([&](u64 key) {
        const bool keep = key >= kth;         // kth is a key, so zeros never pass
        const unsigned long long m = __builtin_amdgcn_ballot_w64(keep);
        if (m) {                              // wave-uniform: one atomic per wave step
            uint32_t at = 0;
            if (lane == 0) at = atomicAdd(&sh.n_out, (uint32_t)__popcll(m));
            at = __builtin_amdgcn_readfirstlane(at) +
                 __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            if (keep && at < rank) out[at] = key;
        }
    });
    __syncthreads();
    return kth;
}

// The admission key that select_best found early, or the k'-th best key if `early` lies too near rank k.  Whoever is not admitted scores
// less than the key, so the gap between the scores at rank k and at the key is what is left of the check's margin where the sample holds a query's
// best rows all together (copies of one row have no gap at all).  It has to be `apart` times the score: more than the
// check asks for (early_gap in ralm_api.hip).  out: the k' best keys; all threads, behind select_best.
template <int NT>
__device__ __forceinline__ u64 with_margin(u64 early, u64 kth, const u64 *out, int k, int k_prime, float apart, SelectShared<NT> &sh)
{
    if (early == kth) return kth;   // uniform
    const float at = key_score(early);
    for (int base = 0; base < k_prime; base += NT) {
        const int i = base + threadIdx.x;
        const float s = key_score(out[i < k_prime ? i : 0]);   // (s - apart |s| rises with s)
        const unsigned long long m = __builtin_amdgcn_ballot_w64(i < k_prime && s > at && s - at >= apart * fabsf(s));
        if ((threadIdx.x & 63) == 0 && m) atomicAdd(&sh.n_above, (uint32_t)__popcll(m));
    }
    __syncthreads();
    return sh.n_above >= (uint32_t)k ? early : kth;
}

// What select_kernel and the re-score do with a query's list before they read it: the length that the
// stage left is recorded, and a list that was sent more keys than it has slots, of which it kept the first
// `cap`, is marked.  Returns the number of keys in the list.
__device__ uint32_t list_length(uint32_t n, int64_t q, uint32_t cap, uint32_t *__restrict__ lost, int32_t *__restrict__ flags,
                                int stage)
{
    if (threadIdx.x == 0) {
        // entries the scan sent to this list in the stage that just ended, plus the (at most k') kept before
        if (stage < MAX_STAGE_SUMS) {
            reinterpret_cast<uint32_t *>(reinterpret_cast<unsigned char *>(flags) + stage_offset(gridDim.x, stage))[q] = n;
            if (q == 0) flags[FLAG_STAGES] = stage + 1;
        }
        if (n > cap) {
            if (lost[q] == 0) atomicAdd(flags + FLAG_LADDER_OVERFLOWS, 1);
            lost[q] = 1;
        }
    }
    return n < cap ? n : cap;
}

// Per query: the list is cut down to its k' best keys in place, and a key of rank tau_rank <= k' among them becomes the admission
// key of the next scan stage (tau_rank 0: there is none; with_margin: or the k'-th best).  A list that was sent more keys than
// it has slots kept only the first `cap` of them: it is processed as it is (its k'-th best key
// is still a valid lower bound, the rows behind those keys were all scanned) and the query is
// marked in `lost`, so that it is answered by the exact pass at the end of the call.
//
// tau_rank < k' is the rank that the final k'-th best key has in the sample scanned so far, with room for chance
// (early_rank in ralm_api.hip): the list then still ends up with k' keys that reach it, out of a fraction of the scores that the
// sample's own k'-th best would admit.  If chance or the order of the rows has it otherwise, rows between the two were not admitted: the check
// of the result (certify) takes the admission key for the score of the best row that may be missing.
template <int NT>
__global__ __launch_bounds__(NT) void select_kernel(u64 *__restrict__ cand, uint32_t *__restrict__ cnt,
                                                             uint32_t cap, int k, int k_prime, int tau_rank, float apart, u64 *__restrict__ tau,
                                                             uint32_t *__restrict__ lost, int32_t *__restrict__ flags,
                                                             int stage)
{
    extern __shared__ __align__(16) unsigned char smem[];
    u64 *out = reinterpret_cast<u64 *>(smem);   // [k_prime]
    __shared__ SelectShared<NT> sh;

    const int64_t q = blockIdx.x;
    const int tid = threadIdx.x;
    u64 *c = cand + q * (int64_t)cap;
    const u64 before = tau[q];
    const uint32_t n = list_length(cnt[q * CNT_PITCH], q, cap, lost, flags, stage);
    if (n < (uint32_t)k_prime) {    // fewer than k' candidates exist so far: keep admitting everything
        if (tid == 0) cnt[q * CNT_PITCH] = n;   // (tau is 0 still)
        return;
    }
    u64 early, kth;
    // A short list: less code to fetch, for a kernel that is over in a few microseconds.  81 lists of about 200 keys 7.6 us in the general
    // form, 7.0 by one wave in registers (bracketing the score with ballots), 5.7.
    // (Not FITS, here and in the re-score: 2200 queries, k' = 128 and 256, over 50 000 x 768 took 543 and 703 us a call so, 522 and 682 as it is.)
    if (n <= (uint32_t)(2 * NT)) kth = select_best<NT, 2>(c, n, (uint32_t)k_prime, sh, out, (uint32_t)tau_rank, early);
    else kth = select_best<NT>(c, n, (uint32_t)k_prime, sh, out, (uint32_t)tau_rank, early);
    for (int i = tid; i < k_prime; i += NT) c[i] = out[i];
    early = with_margin<NT>(early, kth, out, k, k_prime, apart, sh);
    if (tid == 0) {
        if (tau_rank > 0) {   // (an admission key is never lowered: what it kept out stays out)
            tau[q] = early > before ? early : before;
        }
        cnt[q * CNT_PITCH] = (uint32_t)k_prime;
    }
}

// The first select of a ladder, of the lists that a scan left as scores (ScanParams::scores_only).  The k' blocks of 32
// rows whose best scores are the highest hold the k' best keys: so many rows score at least as much as the least of those, and a
// block that is left out has no better one (of blocks with that very best the first are taken, whose rows have the lower ids).  So
// 2 KB of bests and k' x 128 bytes are read per query, and not 128 KB of keys.  A thread has one best and four scores: what bounds it is
// the chain, and how much code is fetched for it (one wave per query with 8 bests and 32 scores per lane, all unrolled: 17 us for 3 lists).
// With 128 KB of keys and now: 3 lists 9.5, 9.0 us, 81 lists 12.2, 12.1, 2341 lists 113, 32.
constexpr int SF_THREADS = 512;
__global__ __launch_bounds__(SF_THREADS) void select_first_kernel(u64 *__restrict__ cand, uint32_t *__restrict__ cnt, uint32_t cap, int k, int k_prime,
                                                                  int tau_rank, float apart, int64_t tile_stride, u64 *__restrict__ tau,
                                                                  uint32_t *__restrict__ lost, int32_t *__restrict__ flags, int stage)
{
    constexpr int PER = FIRST_KEYS * 32 / SF_THREADS;   // scores per thread
    static_assert(FIRST_ROWS / 32 == SF_THREADS, "one block of 32 rows per thread");
    __shared__ SelectShared<SF_THREADS> sh;
    __shared__ u64 s_key[FIRST_KEYS * 32], s_out[FIRST_KEYS];
    const int64_t q = blockIdx.x;
    const int tid = threadIdx.x;
    u64 *c = cand + q * (int64_t)cap;
    const float *scores = reinterpret_cast<const float *>(c);
    const uint32_t best = reinterpret_cast<const uint32_t *>(scores + FIRST_ROWS)[tid];   // (all of them lie in the list)
    const uint32_t n = list_length(cnt[q * CNT_PITCH], q, cap, lost, flags, stage);        // more than FIRST_ROWS / 2
    const int nb = (int)((n + 31) / 32);
    if (tid < nb) s_key[tid] = (u64)best << 32 | (uint32_t)(0x7fffffff - tid);   // distinct, and the first of equal ones the better
    __syncthreads();
    u64 early;
    select_best<SF_THREADS, 1, true>(s_key, (uint32_t)nb, (uint32_t)k_prime, sh, s_out, 0, early);
    float f[PER];
    int32_t at[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int j = i * SF_THREADS + tid;   // 32 threads a block
        at[i] = j < k_prime * 32 ? key_id(s_out[j >> 5]) * 32 + (j & 31) : 0x7fffffff;
        f[i] = (uint32_t)at[i] < n ? scores[at[i]] : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int64_t row = (int64_t)(at[i] / SCAN_BM) * tile_stride * SCAN_BM + at[i] % SCAN_BM;
        if (i * SF_THREADS + tid < k_prime * 32) s_key[i * SF_THREADS + tid] = (uint32_t)at[i] < n ? make_key(f[i], (int32_t)row) : 0ull;
    }
    __syncthreads();
    const u64 kth = select_best<SF_THREADS, PER, true>(s_key, (uint32_t)k_prime * 32, (uint32_t)k_prime, sh, s_out, (uint32_t)tau_rank, early);
    if (tid < k_prime) c[tid] = s_out[tid];
    early = with_margin<SF_THREADS>(early, kth, s_out, k, k_prime, apart, sh);
    if (tid == 0) {
        tau[q] = early;
        cnt[q * CNT_PITCH] = (uint32_t)k_prime;
    }
}

// every exact score ends in this sum over the wave's 64 lane sums (fixed order: the re-score and
// the exact pass must give a row the same number)
__device__ __forceinline__ double wave_sum(double x) { return wave64_sum(x); }

// The exact score, as the re-score and the exact pass form it: lane l of a wave takes the
// elements 4l .. 4l+3, 256+4l .., adds their products (squared differences) to its sum in that
// order, and the 64 lane sums are added in a fixed order (wave_sum).  Products and sums in double;
// the caller rounds the total once to fp32.
template <bool L2>
__device__ __forceinline__ void exact_accum4(double &sum, const float4 &x, const float4 &y)
{
    if constexpr (L2) {
        const double d0 = (double)y.x - (double)x.x, d1 = (double)y.y - (double)x.y;
        const double d2 = (double)y.z - (double)x.z, d3 = (double)y.w - (double)x.w;
        sum += d0 * d0;
        sum += d1 * d1;
        sum += d2 * d2;
        sum += d3 * d3;
    } else {
        sum += (double)x.x * (double)y.x;
        sum += (double)x.y * (double)y.y;
        sum += (double)x.z * (double)y.z;
        sum += (double)x.w * (double)y.w;
    }
}

// elements j .. j+3 of a row of the exact copy, widened exactly to fp32
template <int EX>
__device__ __forceinline__ float4 exact_load4(const void *__restrict__ exact, int64_t row_off, int j)
{
    if constexpr (EX == DT_F32) {
        return *reinterpret_cast<const float4 *>(static_cast<const float *>(exact) + row_off + j);
    } else {
        const uint2 h = *reinterpret_cast<const uint2 *>(static_cast<const uint16_t *>(exact) + row_off + j);
        return make_float4(f16_bits_to_f32(h.x & 0xffffu), f16_bits_to_f32(h.x >> 16), f16_bits_to_f32(h.y & 0xffffu),
                           f16_bits_to_f32(h.y >> 16));
    }
}

constexpr int RS_ROWS = 4;             // rows that a wave scores together: their loads are in flight at once
constexpr int RS_COUNT_MAX = 256;      // up to this many candidates are ranked by counting

// What a wave learns from the rows that it scores (the sums are those of its lanes together).
struct RowStats {
    u64 min_scan = ~0ull;             // worst scan key
    double e2 = 0.0, x2max = 0.0;     // sum of squared scan errors, largest squared row norm
};

// Exact scores of the candidates list[begin, end), whose scan keys are in LDS, by the NW waves of a workgroup: the
// exact key of list[c] goes to keys[c].  A wave takes RS_ROWS rows at a time, whose loads are in flight
// together.  stats: whether the check's numbers are wanted.
template <int EX, bool L2, int NW>
__device__ __forceinline__ RowStats score_rows(const u64 *list, int begin, int end, const float *__restrict__ qv, float q_sq,
                                               const void *__restrict__ exact, int64_t ld, int d, bool stats, u64 *keys)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    RowStats st;
    for (int c0 = begin + wave; c0 < end; c0 += NW * RS_ROWS) {
        int64_t row_off[RS_ROWS];
        double sum[RS_ROWS], x2[RS_ROWS];
#pragma unroll
        for (int u = 0; u < RS_ROWS; ++u) {
            const int c = c0 + u * NW;
            row_off[u] = (int64_t)key_id(list[c < end ? c : c0]) * ld;   // past the end: the first row again
            sum[u] = x2[u] = 0.0;
        }
        for (int j = lane * 4; j < d; j += 256) {
            float4 x[RS_ROWS];
#pragma unroll
            for (int u = 0; u < RS_ROWS; ++u) x[u] = exact_load4<EX>(exact, row_off[u], j);
            const float4 y = *reinterpret_cast<const float4 *>(qv + j);
#pragma unroll
            for (int u = 0; u < RS_ROWS; ++u) {
                exact_accum4<L2>(sum[u], x[u], y);
                if (stats)
                    x2[u] += (double)x[u].x * (double)x[u].x + (double)x[u].y * (double)x[u].y +
                             (double)x[u].z * (double)x[u].z + (double)x[u].w * (double)x[u].w;
            }
        }
#pragma unroll
        for (int u = 0; u < RS_ROWS; ++u) {
            const int c = c0 + u * NW;
            if (c < end) {   // wave-uniform
                const u64 skey = list[c];
                st.min_scan = skey < st.min_scan ? skey : st.min_scan;
                const double t = wave_sum(sum[u]);
                const float score = L2 ? (float)(-t) : (float)t;
                if (stats) {
                    const double r2 = wave_sum(x2[u]);
                    const double e = (double)(key_score(skey) - q_sq) - (double)score;
                    st.e2 += e * e;
                    st.x2max = r2 > st.x2max ? r2 : st.x2max;
                }
                if (lane == 0) keys[c] = make_key(score, key_id(skey));
            }
        }
    }
    return st;
}

// |q|^2, every thread of the workgroup gets it: part of the scan's score under L2, and of the rounding bound
template <int NT>
__device__ __forceinline__ void query_norm2_part(const float *__restrict__ qv, int d, double *s_q2 /* [NT / 64] in LDS */)
{
    double q2 = 0.0;
    for (int j = threadIdx.x; j < d; j += NT) q2 += (double)qv[j] * (double)qv[j];
    q2 = wave_sum(q2);
    if ((threadIdx.x & 63) == 0) s_q2[threadIdx.x >> 6] = q2;
}
template <int NT>
__device__ __forceinline__ double query_norm2_sum(const double *s_q2)   // behind a barrier
{
    double q2 = 0.0;
    for (int w = 0; w < NT / 64; ++w) q2 += s_q2[w];
    return q2;
}
template <int NT>
__device__ __forceinline__ double query_norm2(const float *__restrict__ qv, int d, double *s_q2)
{
    query_norm2_part<NT>(qv, d, s_q2);
    __syncthreads();
    return query_norm2_sum<NT>(s_q2);
}

// floor: the admission key of the last stage; truncated: the list lost entries.
// The margin of query q and the verdict of the check (one thread): `rank_k` is the key at rank k of the
// n re-scored candidates, the statistics are those of all of them.
template <bool L2>
__device__ void certify(const CertifyParams &cert, float *__restrict__ out_margin, int64_t q, int cnt_pitch, int n, int k,
                        int k_prime, int d, double q2, u64 rank_k, u64 min_scan, double e2, double x2m, u64 floor, bool truncated)
{
    const float q_sq = L2 ? (float)q2 : 0.f;
    // rows that reach the worst kept key were not admitted if the last stage's admission key lies above it
    const bool open = floor > min_scan && n >= k_prime;
    // margin: exact score at rank k minus the scan's score of the worst kept candidate.  A row
    // that was not kept has a scan score at most the latter (the admission key's, if that is higher), so it can belong in the top k only
    // if the scan mis-scored it by at least the margin.
    float margin;
    if (n < k)
        margin = __builtin_nanf("");
    else if (n < k_prime)
        margin = __builtin_inff();   // every row of the datastore was re-scored
    else
        margin = key_score(rank_k) - (key_score(open ? floor : min_scan) - q_sq);
    if (out_margin) out_margin[q] = margin;
    if (!cert.flags) return;
    // what the scan's rounding can do to a score: the deterministic bound (every rounding
    // error aligned; rows outside the candidates are taken to be no longer than the longest
    // candidate), and the spread actually seen on this query's candidates
    const double qn = sqrt(q2), xn = sqrt(x2m);
    const double uq = cert.u_query, ux = cert.u_rows;
    double hard = (uq + ux + uq * ux) * qn * xn + (double)d * 5.9604644775390625e-08 * qn * xn;
    if (L2) hard = 2.0 * hard + (ux * ux + (double)d * 5.9604644775390625e-08) * x2m;
    const double soft = n > 0 ? 8.0 * sqrt(e2 / (double)n) : 0.0;
    const bool all_rows = n < k_prime && !truncated;
    const double m = (double)margin;
    const bool soft_ok = all_rows || (!truncated && n >= k && (m > soft || (soft == 0.0 && m >= 0.0 && !open)));
    uint32_t *status = reinterpret_cast<uint32_t *>(reinterpret_cast<unsigned char *>(cert.flags) + status_offset());
    status[q] = soft_ok ? (all_rows || m > hard ? STATUS_SOFT | STATUS_HARD : STATUS_SOFT) : 0u;
    if (!soft_ok && n >= k) {
        // answered again by the exact pass: every row whose exact key reaches the exact
        // rank-k key found here (a lower bound of the true one) is collected in the list
        const int at = atomicAdd(cert.flags + FLAG_FALLBACKS, 1);
        cert.fb_list[at] = (int32_t)q;
        cert.tau_exact[q] = rank_k;
        cert.cnt_rw[q * cnt_pitch] = 0u;
    }
}

// Re-score of the candidates, final ranking, and the check of the result (see CertifyParams).
// EX: DT_F32 or DT_F16 exact rows.  L2: the score is minus the squared distance; the scan's
// score of a row is then 2<q, x> - |x|^2, so |q|^2 is subtracted from it wherever the two are
// compared.
// What bounds it: the gather of Q k' rows for large batches, and for few queries the latency of
// one wave's rows, which is why a wave takes RS_ROWS of them at a time (k' = 64: each of the 16
// waves has its four rows in flight at once) and why the list is cut down here and not by a launch of
// its own.  With the last select (a launch of its own before): Q = 1, k' = 64: 26 -> 14 us;
// Q = 1024: 103 -> 50 us.
template <int EX, bool L2, int RS_THREADS>
__global__ __launch_bounds__(RS_THREADS) void rescore_kernel(const u64 *__restrict__ cand,
                                                      const uint32_t *__restrict__ cnt, int cnt_pitch, uint32_t cap,
                                                      int k_prime, int kp2, const float *__restrict__ queries,
                                                      const void *__restrict__ exact, int64_t ld, int d,
                                                      int k, int32_t *__restrict__ out_ids,
                                                      float *__restrict__ out_scores,
                                                      float *__restrict__ out_margin, const CertifyParams cert)
{
    constexpr int RS_WAVES = RS_THREADS / 64;
    extern __shared__ __align__(16) unsigned char smem[];
    u64 *keys = reinterpret_cast<u64 *>(smem);   // [kp2] exact keys
    u64 *list = keys + kp2;                      // [k_prime] the candidates' scan keys
    __shared__ SelectShared<RS_THREADS> sel;
    __shared__ u64 s_min_scan[RS_WAVES];
    __shared__ double s_e2[RS_WAVES], s_x2[RS_WAVES], s_q2[RS_WAVES];
    __shared__ uint32_t s_rank[RS_COUNT_MAX];

    const int64_t q = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const u64 *mine = cand + q * (int64_t)cap;
    const float *qv = queries + q * (int64_t)d;
    const bool stats = out_margin || cert.flags;   // wave-uniform

    // the list's length and its first keys travel while |q|^2 is formed (every list has that many slots, or it is the caches')
    uint32_t n_list = cnt[q * cnt_pitch];
    if (stats) query_norm2_part<RS_THREADS>(qv, d, s_q2);
    if (tid < RS_COUNT_MAX) s_rank[tid] = 0;
    // what the check needs at the end travels with the rows
    const bool checks = cert.flags && tid == 0;
    const u64 floor = checks ? cert.tau_exact[q] : 0ull;
    const uint32_t lost_before = checks && cert.lost ? cert.lost[q] : 0u;
    const uint32_t raw_length = n_list;
    n_list = cert.flags ? list_length(n_list, q, cap, cert.lost, cert.flags, cert.stage) : (n_list < cap ? n_list : cap);
    int n = (int)n_list;
    if (n > k_prime) {
        n = k_prime;
        u64 none;
        if (n_list <= 2 * RS_THREADS) {   // less code to fetch, see select_kernel
            select_best<RS_THREADS, 2>(mine, n_list, (uint32_t)k_prime, sel, list, 0, none);
        } else {
            select_best<RS_THREADS>(mine, n_list, (uint32_t)k_prime, sel, list, 0, none);
        }
    } else {
        for (int i = tid; i < n; i += RS_THREADS) list[i] = mine[i];
    }
    __syncthreads();
    const double q2 = L2 && stats ? query_norm2_sum<RS_THREADS>(s_q2) : 0.0;
    const RowStats st = score_rows<EX, L2, RS_WAVES>(list, 0, n, qv, L2 ? (float)q2 : 0.f, exact, ld, d, stats, keys);
    if (lane == 0) {
        s_min_scan[wave] = st.min_scan;
        s_e2[wave] = st.e2;
        s_x2[wave] = st.x2max;
    }

    const u64 *ranked;   // descending by key
    if (kp2 <= RS_COUNT_MAX) {
        // every candidate counts the better ones, RS_THREADS / kp2 threads share the counting (equal keys,
        // a cached id listed twice, keep their order)
        __syncthreads();
        const int i = tid & (kp2 - 1), part = tid / kp2, parts = RS_THREADS / kp2;
        if (i < n) {
            const u64 key = keys[i];
            uint32_t better = 0;
            for (int j = part; j < n; j += parts) better += keys[j] > key || (keys[j] == key && j < i) ? 1u : 0u;
            if (better) atomicAdd(&s_rank[i], better);
        }
        __syncthreads();
        if (tid < n) list[s_rank[tid]] = keys[tid];
        __syncthreads();
        ranked = list;
    } else {
        for (int c = n + tid; c < kp2; c += RS_THREADS) keys[c] = 0ull;
        __syncthreads();
        sort_keys<RS_THREADS, true>(keys, kp2);
        ranked = keys;
    }

    for (int r = tid; r < k; r += RS_THREADS) {
        const bool have = r < n;
        const u64 key = have ? ranked[r] : 0ull;
        out_ids[q * k + r] = have ? key_id(key) : -1;
        out_scores[q * k + r] = have ? key_score(key) : -__builtin_inff();
    }
    if (stats && tid == 0) {
        RowStats all = {s_min_scan[0], s_e2[0], s_x2[0]};
        for (int w = 1; w < RS_WAVES; ++w) {
            all.min_scan = s_min_scan[w] < all.min_scan ? s_min_scan[w] : all.min_scan;
            all.e2 += s_e2[w];
            all.x2max = s_x2[w] > all.x2max ? s_x2[w] : all.x2max;
        }
        certify<L2>(cert, out_margin, q, cnt_pitch, n, k, k_prime, d, L2 ? q2 : query_norm2_sum<RS_THREADS>(s_q2), n >= k ? ranked[k - 1] : 0ull,
                    all.min_scan, all.e2, all.x2max, floor, lost_before != 0 || raw_length > cap);
    }
}

// The same in two launches for many candidates per query, whose list a select has cut down before: the rows
// are scored by several workgroups per query, and one more ranks them.  In one workgroup the phases of a query
// (its list, its rows, its sort) follow each other on a CU with nothing beside them, and few queries leave most
// of the chip idle.  The exact keys go to the list's slots [k', 2 k') and the statistics of
// part p to the four slots from 2 k' + 4 p on (lists have at least 16384 slots).
// Neighbour rounds: 256 queries, k' = 2048, 1024 fp16 elements 6376 -> 6230 us; 16 queries 813 -> 596 us; 64 queries,
// k' = 512, squared distance: 68 -> 36 us for the select and both launches; 800 queries, k' = 512: 1874 -> 1854 us.
constexpr int RP_THREADS = 512, RP_WAVES = RP_THREADS / 64;

template <int EX, bool L2>
__global__ __launch_bounds__(RP_THREADS) void rescore_rows_kernel(u64 *__restrict__ cand, const uint32_t *__restrict__ cnt,
                                                                  uint32_t cap, int k_prime, const float *__restrict__ queries,
                                                                  const void *__restrict__ exact, int64_t ld, int d)
{
    extern __shared__ __align__(16) unsigned char smem[];
    u64 *list = reinterpret_cast<u64 *>(smem);   // [rows of a part]
    __shared__ u64 s_min_scan[RP_WAVES];
    __shared__ double s_e2[RP_WAVES], s_x2[RP_WAVES], s_q2[RP_WAVES];

    const int64_t q = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int part = blockIdx.y, per = (k_prime + (int)gridDim.y - 1) / (int)gridDim.y;
    u64 *mine = cand + q * (int64_t)cap;
    const float *qv = queries + q * (int64_t)d;
    const int n = (int)cnt[q * CNT_PITCH];       // at most k'
    const int begin = part * per;
    const int rows = n - begin < per ? (n - begin > 0 ? n - begin : 0) : per;
    for (int i = tid; i < rows; i += RP_THREADS) list[i] = mine[begin + i];
    const double q2 = L2 ? query_norm2<RP_THREADS>(qv, d, s_q2) : 0.0;
    __syncthreads();
    const RowStats st = score_rows<EX, L2, RP_WAVES>(list, 0, rows, qv, L2 ? (float)q2 : 0.f, exact, ld, d, true,
                                                     mine + k_prime + begin);
    if (lane == 0) {
        s_min_scan[wave] = st.min_scan;
        s_e2[wave] = st.e2;
        s_x2[wave] = st.x2max;
    }
    __syncthreads();
    if (tid == 0) {
        RowStats all = {s_min_scan[0], s_e2[0], s_x2[0]};
        for (int w = 1; w < RP_WAVES; ++w) {
            all.min_scan = s_min_scan[w] < all.min_scan ? s_min_scan[w] : all.min_scan;
            all.e2 += s_e2[w];
            all.x2max = s_x2[w] > all.x2max ? s_x2[w] : all.x2max;
        }
        u64 *to = mine + 2 * k_prime + 4 * part;
        to[0] = all.min_scan;
        to[1] = (u64)__double_as_longlong(all.e2);
        to[2] = (u64)__double_as_longlong(all.x2max);
    }
}

template <bool L2, int NT>
__global__ __launch_bounds__(NT) void rescore_rank_kernel(const u64 *__restrict__ cand, const uint32_t *__restrict__ cnt,
                                                          uint32_t cap, int k_prime, int kp2, int parts,
                                                          const float *__restrict__ queries, int d, int k,
                                                          int32_t *__restrict__ out_ids, float *__restrict__ out_scores,
                                                          float *__restrict__ out_margin, const CertifyParams cert)
{
    extern __shared__ __align__(16) unsigned char smem[];
    u64 *keys = reinterpret_cast<u64 *>(smem);   // [kp2]
    __shared__ double s_q2[NT / 64];
    const int64_t q = blockIdx.x;
    const int tid = threadIdx.x;
    const u64 *mine = cand + q * (int64_t)cap;
    const int n = (int)cnt[q * CNT_PITCH];       // at most k'
    for (int c = tid; c < kp2; c += NT) keys[c] = c < n ? mine[k_prime + c] : 0ull;
    const double q2 = query_norm2<NT>(queries + q * (int64_t)d, d, s_q2);
    __syncthreads();
    sort_keys<NT, true>(keys, kp2);
    for (int r = tid; r < k; r += NT) {
        const bool have = r < n;
        const u64 key = have ? keys[r] : 0ull;
        out_ids[q * k + r] = have ? key_id(key) : -1;
        out_scores[q * k + r] = have ? key_score(key) : -__builtin_inff();
    }
    if (tid == 0) {
        RowStats all;
        for (int p = 0; p < parts; ++p) {
            const u64 *from = mine + 2 * k_prime + 4 * p;
            const double e2 = __longlong_as_double((long long)from[1]), x2 = __longlong_as_double((long long)from[2]);
            all.min_scan = from[0] < all.min_scan ? from[0] : all.min_scan;
            all.e2 += e2;
            all.x2max = x2 > all.x2max ? x2 : all.x2max;
        }
        certify<L2>(cert, out_margin, q, CNT_PITCH, n, k, k_prime, d, q2, n >= k ? keys[k - 1] : 0ull, all.min_scan, all.e2,
                    all.x2max, cert.flags ? cert.tau_exact[q] : 0ull, cert.lost && cert.lost[q] != 0);
    }
}

// ---- exact pass for the queries whose scan result could not be trusted -------------------------
// All rows of the exact copy are scored exactly against up to QG of those queries at a time and
// every row whose exact key reaches the query's bound is appended to the query's list.  The
// arithmetic is that of the re-score (same order of the sums), so a row gets the same number.
constexpr int XS_THREADS = 256, XS_WAVES = XS_THREADS / 64, XS_QG = 8;

template <int EX, bool L2>
__global__ __launch_bounds__(XS_THREADS) void exact_scan_kernel(const float *__restrict__ queries,
                                                                const void *__restrict__ exact, int64_t ld,
                                                                int64_t N, int d, int qgroup,
                                                                const int32_t *__restrict__ fb_list,
                                                                const int32_t *__restrict__ flags,
                                                                const u64 *__restrict__ tau_exact,
                                                                u64 *__restrict__ cand, uint32_t *__restrict__ cnt,
                                                                uint32_t cap)
{
    extern __shared__ __align__(16) unsigned char smem[];
    float *qs = reinterpret_cast<float *>(smem);     // [qgroup][d]
    __shared__ u64 s_tau[XS_QG];
    __shared__ float s_tsc[XS_QG];                   // score part of the bound: a cheap first test
    __shared__ int32_t s_q[XS_QG];

    const int F = flags[FLAG_FALLBACKS];
    if (F <= 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t wave0 = (int64_t)blockIdx.x * XS_WAVES + wave, n_waves = (int64_t)gridDim.x * XS_WAVES;

    for (int g0 = 0; g0 < F; g0 += qgroup) {
        const int nq = F - g0 < qgroup ? F - g0 : qgroup;
        __syncthreads();
        if (tid < nq) {
            const int32_t q = fb_list[g0 + tid];
            s_q[tid] = q;
            s_tau[tid] = tau_exact[q];
            s_tsc[tid] = key_score(tau_exact[q]);
        }
        __syncthreads();
        for (int qi = 0; qi < nq; ++qi) {
            const float *src = queries + (int64_t)s_q[qi] * d;
            for (int j = tid * 4; j < d; j += XS_THREADS * 4)
                *reinterpret_cast<float4 *>(qs + (size_t)qi * d + j) = *reinterpret_cast<const float4 *>(src + j);
        }
        __syncthreads();

        for (int64_t row = wave0; row < N; row += n_waves) {
            const int64_t row_off = row * ld;
            double sum[XS_QG];
#pragma unroll
            for (int qi = 0; qi < XS_QG; ++qi) sum[qi] = 0.0;
            for (int j = lane * 4; j < d; j += 256) {
                const float4 x = exact_load4<EX>(exact, row_off, j);
#pragma unroll
                for (int qi = 0; qi < XS_QG; ++qi) {
                    if (qi < nq) {   // wave-uniform
                        const float4 y = *reinterpret_cast<const float4 *>(qs + (size_t)qi * d + j);
                        exact_accum4<L2>(sum[qi], x, y);
                    }
                }
            }
#pragma unroll
            for (int qi = 0; qi < XS_QG; ++qi) {
                if (qi < nq) {
                    const double t = wave_sum(sum[qi]);
                    const float sc = L2 ? (float)(-t) : (float)t;
                    if (lane == 0 && sc >= s_tsc[qi]) {   // a key that reaches the bound has a score that does
                        const u64 key = make_key(sc, (int32_t)row);
                        if (key >= s_tau[qi]) {
                            const int32_t q = s_q[qi];
                            const uint32_t at = atomicAdd(cnt + (int64_t)q * CNT_PITCH, 1u);
                            if (at < cap) cand[(int64_t)q * cap + at] = key;
                        }
                    }
                }
            }
        }
    }
}

// The exact pass on the fp64 matrix cores (inner product, rows that are whole 256-byte steps).
// v_mfma_f64_16x16x4: operand A of lane l is element (i = l%16, k = l/16), operand B element
// (k = l/16, j = l%16), and the lane receives D(i = 4v + l/16, j = l%16) in its v-th result,
// v = 0..3.  i runs over 16 consecutive rows, j over up to 16 queued queries, so one pass over the
// exact copy serves 16 queries at the cost of one, with sums in double and no reduction across
// lanes.  A lane holds elements 4*CH*u + CH*(l/16) .. + CH-1 of its row (CH elements per 16-byte
// load); the queries sit in LDS as floats in the order the instructions consume them.  The sums
// are formed in another order than the re-score forms them, so a row's score may differ from the
// re-score's in the last place of the fp32 result (rarely: both are double sums rounded once);
// rows are therefore collected from one fp32 step BELOW the bound's score on, which keeps the k
// rows that defined the bound in the list whatever the order, and the final ranking uses this
// kernel's scores only.
constexpr int XM_NW = 8, XM_QG = 16;

template <int EX, int SEG>
__global__ __launch_bounds__(XM_NW * 64) void exact_scan_mfma_kernel(const float *__restrict__ queries,
                                                                      const void *__restrict__ exact, int64_t ld,
                                                                      int64_t N, int d,
                                                                      const int32_t *__restrict__ fb_list,
                                                                      const int32_t *__restrict__ flags,
                                                                      const u64 *__restrict__ tau_exact,
                                                                      u64 *__restrict__ cand, uint32_t *__restrict__ cnt,
                                                                      uint32_t cap)
{
    constexpr int CH = EX == DT_F32 ? 4 : 8;   // elements per 16-byte piece
    constexpr int ES = EX == DT_F32 ? 4 : 2;
    typedef double d4 __attribute__((ext_vector_type(4)));
    extern __shared__ __align__(16) unsigned char smem[];
    float *qf = reinterpret_cast<float *>(smem);   // [d / 4 instructions][4 k][16 j]
    __shared__ float s_tsc[XM_QG];
    __shared__ int32_t s_q[XM_QG];

    const int F = flags[FLAG_FALLBACKS];
    if (F <= 0) return;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, kq = lane >> 4;
    const int NC = d / (4 * CH), nsegs = NC / SEG;
    const int64_t nblk = (N + 15) / 16;
    const int64_t blk0 = (int64_t)blockIdx.x * XM_NW + wave, blk_step = (int64_t)gridDim.x * XM_NW;
    const unsigned char *base = static_cast<const unsigned char *>(exact) + kq * 16;

    for (int g0 = 0; g0 < F; g0 += XM_QG) {
        const int nq = F - g0 < XM_QG ? F - g0 : XM_QG;
        __syncthreads();
        if (tid < XM_QG) {
            int32_t q = -1;
            float tsc = __builtin_inff();
            if (tid < nq) {
                q = fb_list[g0 + tid];
                const uint32_t b = (uint32_t)(tau_exact[q] >> 32);
                tsc = bits_score(b ? b - 1u : 0u);   // one fp32 step below the bound's score
            }
            s_q[tid] = q;
            s_tsc[tid] = tsc;
        }
        __syncthreads();
        for (int i = tid; i < XM_QG * d; i += XM_NW * 64) {
            const int qi = i / d, e = i - qi * d;
            const float v = qi < nq ? queries[(int64_t)s_q[qi] * d + e] : 0.f;
            const int t = CH * (e / (4 * CH)) + e % CH, k = (e / CH) & 3;
            qf[(size_t)t * 64 + k * 16 + qi] = v;
        }
        __syncthreads();
        const float my_tsc = s_tsc[r16];
        const int64_t my_q = s_q[r16];

        int64_t blk = blk0;
        if (blk >= nblk) continue;
        auto row_of = [&](int64_t b) {
            int64_t row = b * 16 + r16;
            row = row < N ? row : N - 1;   // rows past the end re-read the last one; their results are dropped
            return base + row * ld * ES;
        };
        const unsigned char *row = row_of(blk);
        int seg = 0;
        d4 acc = {0.0, 0.0, 0.0, 0.0};
        uint4 buf0[SEG], buf1[SEG];
        auto load = [&](uint4(&buf)[SEG], const unsigned char *rw, int sg) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < SEG; ++c) buf[c] = *reinterpret_cast<const uint4 *>(rw + (size_t)(sg * SEG + c) * 64);
        };
        auto item = [&](uint4(&cur)[SEG], uint4(&nxt)[SEG]) __attribute__((always_inline)) -> bool {
            const bool last_seg = seg + 1 == nsegs;
            const int64_t blk_n = last_seg ? blk + blk_step : blk;
            const bool more = blk_n < nblk;
            const unsigned char *row_n = last_seg ? row_of(more ? blk_n : blk) : row;
            if (more) load(nxt, row_n, last_seg ? 0 : seg + 1);
            const float *ql = qf + (size_t)seg * (SEG * CH * 64) + lane;
#pragma unroll
            for (int c = 0; c < SEG; ++c) {
                double a[CH];
                if constexpr (EX == DT_F32) {
                    a[0] = (double)__uint_as_float(cur[c].x);
                    a[1] = (double)__uint_as_float(cur[c].y);
                    a[2] = (double)__uint_as_float(cur[c].z);
                    a[3] = (double)__uint_as_float(cur[c].w);
                } else {
                    a[0] = (double)f16_bits_to_f32(cur[c].x & 0xffffu);
                    a[1] = (double)f16_bits_to_f32(cur[c].x >> 16);
                    a[2] = (double)f16_bits_to_f32(cur[c].y & 0xffffu);
                    a[3] = (double)f16_bits_to_f32(cur[c].y >> 16);
                    a[4] = (double)f16_bits_to_f32(cur[c].z & 0xffffu);
                    a[5] = (double)f16_bits_to_f32(cur[c].z >> 16);
                    a[6] = (double)f16_bits_to_f32(cur[c].w & 0xffffu);
                    a[7] = (double)f16_bits_to_f32(cur[c].w >> 16);
                }
#pragma unroll
                for (int e = 0; e < CH; ++e)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[e], (double)ql[(size_t)(c * CH + e) * 64], acc, 0, 0, 0);
            }
            if (last_seg) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int64_t rw = blk * 16 + 4 * v + kq;
                    const float sc = (float)acc[v];
                    if (rw < N && sc >= my_tsc) {
                        const uint32_t at = atomicAdd(cnt + my_q * CNT_PITCH, 1u);
                        if (at < cap) cand[my_q * cap + at] = make_key(sc, (int32_t)rw);
                    }
                }
                acc = d4{0.0, 0.0, 0.0, 0.0};
                blk = blk_n;
                seg = 0;
                row = row_n;
            } else {
                ++seg;
            }
            return !more;
        };
        load(buf0, row, 0);
        for (;;) {
            if (item(buf0, buf1)) break;
            if (item(buf1, buf0)) break;
        }
    }
}

// Final ranking of an exact-pass query: the k best keys of its list, sorted, written out.
__global__ __launch_bounds__(SEL_THREADS) void exact_finish_kernel(const u64 *__restrict__ cand,
                                                                   const uint32_t *__restrict__ cnt, uint32_t cap,
                                                                   int k, int kp2, const int32_t *__restrict__ fb_list,
                                                                   int32_t *__restrict__ flags,
                                                                   int32_t *__restrict__ out_ids,
                                                                   float *__restrict__ out_scores,
                                                                   int32_t *__restrict__ host_mark)
{
    extern __shared__ __align__(16) unsigned char smem[];
    u64 *keys = reinterpret_cast<u64 *>(smem);   // [kp2]
    __shared__ RadixShared sh;
    __shared__ uint32_t s_out;

    const int F = flags[FLAG_FALLBACKS];
    const int tid = threadIdx.x;
    for (int i = blockIdx.x; i < F; i += gridDim.x) {
        const int64_t q = fb_list[i];
        const uint32_t n = cnt[q * CNT_PITCH];
        const u64 *c = cand + q * (int64_t)cap;
        __syncthreads();
        if (n > cap || n < (uint32_t)k) {
            // more rows reach the bound than a list holds (n < k cannot happen: the k rows that
            // defined the bound reach it): this query stays unanswered and is counted
            for (int r = tid; r < k; r += SEL_THREADS) {
                out_ids[q * k + r] = -1;
                out_scores[q * k + r] = __builtin_nanf("");
            }
            if (tid == 0) {
                atomicAdd(flags + FLAG_UNANSWERED, 1);
                if (host_mark) __hip_atomic_store(host_mark, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
            }
            continue;
        }
        const u64 kth = radix_kth<SEL_THREADS>(c, n, (uint32_t)k, sh);
        if (tid == 0) s_out = 0;
        for (int r = tid; r < kp2; r += SEL_THREADS) keys[r] = 0ull;
        __syncthreads();
        for (uint32_t e = tid; e < n; e += SEL_THREADS) {
            const u64 key = c[e];
            if (key >= kth) {
                const uint32_t at = atomicAdd(&s_out, 1u);
                if (at < (uint32_t)kp2) keys[at] = key;
            }
        }
        __syncthreads();
        sort_keys<SEL_THREADS, true>(keys, kp2);
        for (int r = tid; r < k; r += SEL_THREADS) {
            out_ids[q * k + r] = key_id(keys[r]);
            out_scores[q * k + r] = key_score(keys[r]);
        }
    }
}

}  // namespace

hipError_t launch_select(u64 *cand, uint32_t *cnt, uint32_t cap, int32_t k, int32_t k_prime, int32_t tau_rank, float apart, int64_t Q, u64 *tau,
                         uint32_t *lost, int32_t *flags, int32_t stage, int64_t expected, hipStream_t stream)
{
    if (Q <= 0) return hipSuccess;
    const size_t smem = (size_t)k_prime * sizeof(u64);
    // lists that should be short are ranked by small workgroups, eight to a CU instead of two: 2341 lists of
    // about 128 keys 11 us instead of 20 (any length is right in either)
    if (expected <= 512)
        hipLaunchKernelGGL(select_kernel<256>, dim3((unsigned)Q), dim3(256), smem, stream, cand, cnt, cap, k, k_prime,
                           tau_rank, apart, tau, lost, flags, stage);
    else
        hipLaunchKernelGGL(select_kernel<SEL_THREADS>, dim3((unsigned)Q), dim3(SEL_THREADS), smem, stream, cand, cnt, cap,
                           k, k_prime, tau_rank, apart, tau, lost, flags, stage);
    return hipGetLastError();
}

hipError_t launch_select_first(u64 *cand, uint32_t *cnt, uint32_t cap, int32_t k, int32_t k_prime, int32_t tau_rank, float apart, int64_t tile_stride, int64_t Q, u64 *tau,
                               uint32_t *lost, int32_t *flags, int32_t stage, hipStream_t stream)
{
    if (Q <= 0) return hipSuccess;
    if (k_prime > FIRST_KEYS || cap < FIRST_ROWS) return hipErrorInvalidValue;
    hipLaunchKernelGGL(select_first_kernel, dim3((unsigned)Q), dim3(SF_THREADS), 0, stream, cand, cnt, cap, k, k_prime, tau_rank, apart, tile_stride, tau, lost,
                       flags, stage);
    return hipGetLastError();
}

hipError_t launch_rescore(const u64 *cand, const uint32_t *cnt, int cnt_pitch, uint32_t cap, int32_t k_prime, const float *queries,
                          int64_t Q, const void *exact, int32_t exact_dtype, int64_t ld, int32_t d, int32_t metric,
                          int32_t k, int32_t *out_ids, float *out_scores, float *out_margin,
                          const CertifyParams &cert, int64_t expected, hipStream_t stream)
{
    if (Q <= 0) return hipSuccess;
    int kp2 = 2;
    while (kp2 < k_prime) kp2 <<= 1;
    const size_t smem = (size_t)(kp2 + k_prime) * sizeof(u64);
#define RALM_RS_NT(EXV, L2V, NTV)                                                                              \
    do {                                                                                                     \
        auto kern = rescore_kernel<EXV, L2V, NTV>;                                                           \
        static std::atomic<bool> attr_done{false};                                                           \
        if (!attr_done.load(std::memory_order_acquire)) {                                                    \
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),                         \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024);       \
            if (e != hipSuccess) return e;                                                                   \
            attr_done.store(true, std::memory_order_release);                                                \
        }                                                                                                    \
        hipLaunchKernelGGL(kern, dim3((unsigned)Q), dim3(NTV), smem, stream, cand, cnt, \
                       cnt_pitch, cap, k_prime, kp2, queries, exact, ld, d, k, out_ids, out_scores, out_margin, cert);                     \
    } while (0)
    // A CU holds one large workgroup or eight small ones, which overlap one query's chain of list, rows and ranking with
    // the others' gathers.  From two rounds of large ones on small ones are the better, 1024 queries, k' = 64: 50 us instead of 91,
    // 2341: 96 instead of 200; with few candidates already where the second round is nearly empty, whole calls with small and large ones:
    // 300 over 200 000 x 768 251 and 255, 500 284 and 289, 300 over 30 000 97 and 103, but 256 152 and 151, and 300 with k' = 256 361 and 357.
    // Fewer queries, or many candidates each, need the large workgroup's waves; so do long
    // lists, of which a small one holds only 4096 keys in registers (the one stage of a small datastore).  Whole calls
    // with small and large ones: 512 queries over 16384 rows of 64, k = 5, 134 and 67, over 8000 rows 86 and 62, 1024
    // over 8000 101 and 89, 3000 over 16384 451 and 353, over 8000 227 and 233, k = 100 364 and 410.
    const bool short_lists = expected <= SEL_REGS * 256 || (expected <= SEL_REGS * 512 && Q >= 2048);
#define RALM_RS(EXV, L2V)                                  \
    do {                                                   \
        if ((Q >= 512 || (Q > 256 && k_prime <= 64)) && k_prime <= RS_COUNT_MAX && short_lists) RALM_RS_NT(EXV, L2V, 256); \
        else RALM_RS_NT(EXV, L2V, SEL_THREADS);            \
    } while (0)
    if (exact_dtype == DT_F16) {
        if (metric == METRIC_L2) RALM_RS(DT_F16, true);
        else RALM_RS(DT_F16, false);
    } else {
        if (metric == METRIC_L2) RALM_RS(DT_F32, true);
        else RALM_RS(DT_F32, false);
    }
#undef RALM_RS
#undef RALM_RS_NT
    return hipGetLastError();
}

hipError_t launch_rescore_cut(u64 *cand, const uint32_t *cnt, uint32_t cap, int32_t k_prime, const float *queries, int64_t Q,
                              const void *exact, int32_t exact_dtype, int64_t ld, int32_t d, int32_t metric, int32_t k,
                              int32_t *out_ids, float *out_scores, float *out_margin, const CertifyParams &cert,
                              hipStream_t stream)
{
    if (Q <= 0) return hipSuccess;
    int kp2 = 2;
    while (kp2 < k_prime) kp2 <<= 1;
    // four workgroups of eight waves fill a CU; a part is at least four rows per wave
    int64_t parts = (1024 + Q - 1) / Q;
    const int64_t most = (k_prime + RP_WAVES * RS_ROWS - 1) / (RP_WAVES * RS_ROWS);
    if (parts > most) parts = most;
    const dim3 grid((unsigned)Q, (unsigned)parts), block(RP_THREADS);
    const size_t rows_smem = (size_t)((k_prime + parts - 1) / parts) * sizeof(u64);
    if (exact_dtype == DT_F16) {
        if (metric == METRIC_L2)
            hipLaunchKernelGGL((rescore_rows_kernel<DT_F16, true>), grid, block, rows_smem, stream, cand, cnt, cap, k_prime, queries, exact, ld, d);
        else
            hipLaunchKernelGGL((rescore_rows_kernel<DT_F16, false>), grid, block, rows_smem, stream, cand, cnt, cap, k_prime, queries, exact, ld, d);
    } else {
        if (metric == METRIC_L2)
            hipLaunchKernelGGL((rescore_rows_kernel<DT_F32, true>), grid, block, rows_smem, stream, cand, cnt, cap, k_prime, queries, exact, ld, d);
        else
            hipLaunchKernelGGL((rescore_rows_kernel<DT_F32, false>), grid, block, rows_smem, stream, cand, cnt, cap, k_prime, queries, exact, ld, d);
    }
    const size_t smem = (size_t)kp2 * sizeof(u64);
#define RALM_RANK(L2V, NTV)                                                                                             \
    hipLaunchKernelGGL((rescore_rank_kernel<L2V, NTV>), dim3((unsigned)Q), dim3(NTV), smem, stream, cand, cnt, cap,     \
                       k_prime, kp2, (int)parts, queries, d, k, out_ids, out_scores, out_margin, cert)
    if (metric == METRIC_L2) {
        if (kp2 <= 512) RALM_RANK(true, 256);
        else RALM_RANK(true, 1024);
    } else {
        if (kp2 <= 512) RALM_RANK(false, 256);
        else RALM_RANK(false, 1024);
    }
#undef RALM_RANK
    return hipGetLastError();
}

hipError_t launch_exact_pass(const float *queries, int64_t Q, const void *exact, int32_t exact_dtype, int64_t ld,
                             int64_t N, int32_t d, int32_t metric, int32_t k, const int32_t *fb_list, int32_t *flags,
                             const u64 *tau_exact, u64 *cand, uint32_t *cnt, uint32_t cap, int32_t *out_ids,
                             float *out_scores, int32_t *host_mark, int n_cu, hipStream_t stream)
{
    if (Q <= 0) return hipSuccess;
    // as many of the queries at a time as fit 64 KB of LDS in fp32, at most XS_QG
    int qgroup = (64 * 1024) / (d * 4);
    if (qgroup > XS_QG) qgroup = XS_QG;
    if (qgroup < 1) return hipErrorInvalidValue;   // d <= 16384 is checked by the caller
    const size_t smem = (size_t)qgroup * d * 4;
    // both kernels return at once when no query needs them; their grids do not depend on that count,
    // which only the device knows
    int64_t rows_per_pass = (int64_t)n_cu * 4 * XS_WAVES;
    int64_t grid = N < rows_per_pass ? (N + XS_WAVES - 1) / XS_WAVES : (int64_t)n_cu * 4;
#define RALM_XS(EXV, L2V)                                                                                       \
    do {                                                                                                        \
        auto kern = exact_scan_kernel<EXV, L2V>;                                                                \
        static std::atomic<bool> attr_done{false};                                                              \
        if (!attr_done.load(std::memory_order_acquire)) {                                                       \
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),                            \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 64 * 1024);          \
            if (e != hipSuccess) return e;                                                                      \
            attr_done.store(true, std::memory_order_release);                                                   \
        }                                                                                                       \
        hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(XS_THREADS), smem, stream, queries, exact, ld, N, d, \
                           qgroup, fb_list, flags, tau_exact, cand, cnt, cap);                                  \
    } while (0)
    // matrix-core form: inner product, rows of a multiple of 4 sixteen-byte pieces per lane, queries of
    // a group within 128 KB of LDS
    const int nc = d / (exact_dtype == DT_F32 ? 16 : 32);
    const bool mfma = metric == METRIC_IP && d % (exact_dtype == DT_F32 ? 64 : 128) == 0 && d <= 2048;
#define RALM_XM(EXV, SEGV)                                                                                      \
    do {                                                                                                        \
        auto kern = exact_scan_mfma_kernel<EXV, SEGV>;                                                          \
        static std::atomic<bool> attr_done{false};                                                              \
        if (!attr_done.load(std::memory_order_acquire)) {                                                       \
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),                            \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);         \
            if (e != hipSuccess) return e;                                                                      \
            attr_done.store(true, std::memory_order_release);                                                   \
        }                                                                                                       \
        const int64_t nblk = (N + 15) / 16, wgs = (int64_t)n_cu * ((size_t)d * 64 * 2 <= 150 * 1024 ? 2 : 1);   \
        const int64_t g = nblk < wgs * XM_NW ? (nblk + XM_NW - 1) / XM_NW : wgs;                                \
        hipLaunchKernelGGL(kern, dim3((unsigned)g), dim3(XM_NW * 64), (size_t)d * 64, stream, queries, exact, ld, N, \
                           d, fb_list, flags, tau_exact, cand, cnt, cap);                                       \
    } while (0)
#define RALM_XM_SEG(EXV)                  \
    do {                                  \
        if (nc % 8 == 0) RALM_XM(EXV, 8); \
        else if (nc % 6 == 0) RALM_XM(EXV, 6); \
        else RALM_XM(EXV, 4);             \
    } while (0)
    if (exact_dtype == DT_F16) {
        if (metric == METRIC_L2) RALM_XS(DT_F16, true);
        else if (mfma) RALM_XM_SEG(DT_F16);
        else RALM_XS(DT_F16, false);
    } else {
        if (metric == METRIC_L2) RALM_XS(DT_F32, true);
        else if (mfma) RALM_XM_SEG(DT_F32);
        else RALM_XS(DT_F32, false);
    }
#undef RALM_XM_SEG
#undef RALM_XM
#undef RALM_XS
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    int kp2 = 2;
    while (kp2 < k) kp2 <<= 1;
    const int64_t fgrid = Q < 256 ? Q : 256;
    hipLaunchKernelGGL(exact_finish_kernel, dim3((unsigned)fgrid), dim3(SEL_THREADS), (size_t)kp2 * sizeof(u64), stream,
                       cand, cnt, cap, k, kp2, fb_list, flags, out_ids, out_scores, host_mark);
    return hipGetLastError();
}

}  // namespace ralm
