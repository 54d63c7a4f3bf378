// What the scan kernels share: tile order, loads that go straight to LDS, parking of admitted scores (gfx950 only).
#pragma once
#include "ralm_common.h"
#include "ralm_kernels.h"

namespace ralm {

namespace {

template <bool F16>
__device__ __forceinline__ f32x16 mfma32(const uint4 &a, const uint4 &b, const f32x16 &c)
{
    if constexpr (F16)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a),
                                                      __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

#define RALM_LDS __attribute__((address_space(3)))
#define RALM_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

// datastore tile of the t-th tile a launch visits (see ScanParams)
__device__ __forceinline__ int64_t visited_tile(const ScanParams &p, int64_t t)
{
    if (p.tile_skip) {
        // tile counts fit 32 bits (N < 2^31 rows): a 32-bit division, not an emulated 64-bit one
        const uint32_t g1 = (uint32_t)p.tile_skip - 1u, t32 = (uint32_t)t;
        const uint32_t q = t32 / g1;
        t = (int64_t)q * p.tile_skip + (t32 - q * g1) + 1;
    }
    return (p.tile_begin + t) * p.tile_stride;
}

struct PushList {
    RALM_LDS uint32_t *count;   // entries appended so far (may exceed cap; the excess went to global)
    RALM_LDS u64 *keys;         // [cap]
    RALM_LDS uint32_t *qs;      // [cap]
    uint32_t cap;
};

__device__ __forceinline__ void push_global(const ScanParams &p, int q, u64 key)
{
    const uint32_t at = atomicAdd(p.cnt + (int64_t)q * CNT_PITCH, 1u);
    if (at < p.cap) p.cand[(int64_t)q * p.cap + at] = key;
}

// All threads of the workgroup, after a barrier that follows the last append: moves the first n parked
// entries to the global lists and empties the LDS list.  GROUP (batches of up to 256 queries, one
// query tile): the entries of each query are counted in LDS first (`tally`, one word per query): a query's length is then moved once per
// flush and not once per entry.  Adds to one length are served one after the other wherever they come
// from (about 13 ns each here), so a stage that admits 3800 scores per query was bound by them.  Q = 8,
// 1M x 768, k' = 64, refining by 64 at once: whole call 328 -> 271 us.  With more queries an entry of a
// flush seldom shares its query with another.
template <int NT, bool GROUP>
__device__ __forceinline__ void flush_parked(const ScanParams &p, const PushList pl, RALM_LDS uint32_t *tally, uint32_t n)
{
    if constexpr (GROUP) {
        for (int q = threadIdx.x; q < p.Q; q += NT) tally[q] = 0;
        __syncthreads();
#pragma unroll 1
        for (uint32_t e = threadIdx.x; e < n; e += NT) {   // an entry's place among its query's, kept beside the query
            const uint32_t q = pl.qs[e];
            pl.qs[e] = q | __hip_atomic_fetch_add(tally + q, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) << 8;
        }
        __syncthreads();
        for (int q = threadIdx.x; q < p.Q; q += NT) {
            const uint32_t m = tally[q];
            if (m) tally[q] = atomicAdd(p.cnt + (int64_t)q * CNT_PITCH, m);
        }
        __syncthreads();
#pragma unroll 1
        for (uint32_t e = threadIdx.x; e < n; e += NT) {
            const uint32_t q = pl.qs[e] & 255u, at = tally[q] + (pl.qs[e] >> 8);
            if (at < p.cap) p.cand[(int64_t)q * p.cap + at] = pl.keys[e];
        }
    } else {
        for (uint32_t e = threadIdx.x; e < n; e += NT) push_global(p, (int)pl.qs[e], pl.keys[e]);
    }
    __syncthreads();
    if (threadIdx.x == 0) *pl.count = 0;
    __syncthreads();
}

// LDS chunk swizzle: row r of a strip stores its global 16-byte chunk c at chunk slot c ^ swz(r).
// Chosen so that 8 or 16 consecutive rows reading the same global chunk touch distinct
// 16-byte bank groups, for both 128 B and 256 B of LDS banking.
// CPR = 16-byte chunks per strip row: 4 (64-byte rows), 8 (128-byte rows) or 16 (256-byte rows).
template <int CPR>
__device__ __forceinline__ int swz(int r)
{
    static_assert(CPR == 4 || CPR == 8 || CPR == 16, "strip row of 64, 128 or 256 bytes");
    if constexpr (CPR == 16)
        return r & 15;
    else if constexpr (CPR == 8)
        return (r ^ (r >> 3)) & 7;
    else
        return ((r >> 2) & 1) | ((((r >> 1) ^ (r >> 3)) & 1) << 1);
}

// 64 lanes x 16 bytes, from  base + per-lane byte offset,  to 1 KB of LDS starting at lds_base
// (base and lds_base are wave-uniform).  Written as inline asm so that the compiler does not
// track it: completion is awaited by hand with s_waitcnt vmcnt(n) (loads complete in order).
//
// NT: the load is marked non-temporal.  Datastore rows that no other workgroup will read (the
// batch fits one query tile) are streamed that way: they do not displace the query tile in L2,
// and a pure read stream reaches a higher HBM rate with it.  Rows that several query tiles share
// through L2, and the queries themselves, are loaded with the default policy.
template <bool NT>
__device__ __forceinline__ void dma_1kb(const unsigned char *base, uint32_t voff, uint32_t lds_base)
{
    if constexpr (NT)
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds_base), "v"(voff), "s"(base)
                     : "memory");
    else
        asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_base), "v"(voff), "s"(base)
                     : "memory");
}
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

}  // namespace

}  // namespace ralm
