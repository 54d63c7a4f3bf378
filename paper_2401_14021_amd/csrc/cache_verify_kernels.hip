// Speculative retrieval from the per-request caches, the verification compare, and the
// small elementwise helpers (gfx950).
//
//  cache_lookup_kernel  Q.retrieve(q_i) of Alg. 1: rank the request's cached rows with the
//                       retriever's own metric (Section 3 "Speculative retrieval", Fig. 2)
//                       and return the top one.  Scores are formed exactly as the final
//                       scores of the knowledge-base retrieval (double products and sum,
//                       one rounding to fp32; only the order of the double additions
//                       differs), so a cached entry gets the same number from both and
//                       "top-1 of the knowledge base is cached => it is the cache's top-1"
//                       holds.
//  cache_lookup_mfma_kernel  the same lookup with the sums formed on the fp64 matrix cores
//                       (inner product, rows that are whole 256-byte steps).
//  verify_kernel        m = argmin_i (d^_i != d_i) of Alg. 1, per request.
//  cache_insert_kernel  Q.insert(C.retrieve(..)) of Alg. 1: the ids a verification step
//                       retrieved go into the request's cache (Section 3 "Batched
//                       verification": top-1 or top-k update; Section 5.3: the next n rows
//                       after a retrieved one), skipping ids already cached, first in first
//                       out once the cache is full.
#include <atomic>
#include <type_traits>

#include "ralm_common.h"
#include "ralm_kernels.h"

namespace ralm {

namespace {

constexpr int CL_GS = 16;          // lanes that share one cached row
constexpr int CL_ROWS = 64 / CL_GS;   // rows per wave step
constexpr int CL_LDS_BYTES = 100 * 1024;   // queries of a request, widened to double

__device__ __forceinline__ void clamp_range(const int64_t *off, int64_t r, int64_t Qt, int64_t &lo, int64_t &hi)
{
    lo = off[r];
    hi = off[r + 1];
    lo = lo < 0 ? 0 : (lo > Qt ? Qt : lo);
    hi = hi < lo ? lo : (hi > Qt ? Qt : hi);
}

// Queries that no request owns get id -1 / score -inf; the NT threads of one workgroup, for up to FILL_MAX_R requests and FILL_MAX_QT
// queries.  If the ranges reach from the first query to the last all are owned, in whatever order they are.  Otherwise every range is marked in
// a bit map in LDS (owned, of (Qt + 31) / 32 words).  More queries are answered by a launch over the whole chip: this workgroup took 157
// us for 2^20 of which 4 are owned, with the launch 7.5 (for 4096 5.2 and 5.9); ranges that are not in order (they should be),
// each query looked for in all of them, 16 000 for 16384 queries and 4096 ranges.
constexpr int64_t FILL_MAX_R = 4096, FILL_MAX_QT = 4096;
template <int NT>
__device__ __forceinline__ void answer_unowned(const int64_t *__restrict__ off, int64_t R, int64_t Qt, int32_t *__restrict__ ids,
                                               float *__restrict__ scores, uint32_t *owned)
{
    const int64_t first = off[0] < 0 ? 0 : (off[0] > Qt ? Qt : off[0]), end = off[R] < 0 ? 0 : (off[R] > Qt ? Qt : off[R]);
    if (first == 0 && end == Qt) return;
    __syncthreads();
    const int n = (int)Qt;
    for (int w = threadIdx.x; w * 32 < n; w += NT) owned[w] = 0u;
    __syncthreads();
    for (int64_t r = threadIdx.x; r < R; r += NT) {
        int64_t lo, hi;
        clamp_range(off, r, Qt, lo, hi);
        for (int q = (int)lo; q < (int)hi; q = (q | 31) + 1) {   // a word at a time
            const int to = (q | 31) < (int)hi ? 32 : (int)hi & 31;
            atomicOr(owned + (q >> 5), (~0u << (q & 31)) & (to == 32 ? ~0u : (1u << to) - 1u));
        }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < n; q += NT) {
        if (owned[q >> 5] >> (q & 31) & 1u) continue;
        ids[q] = -1;
        scores[q] = -__builtin_inff();
    }
}

// A lookup whose requests are split over several workgroups.  Their best keys meet in partial[query] by an atomic max; who is the last
// of a request to have sent its own decodes them.  The arrivals are counted in the request's first answer, which holds -1 before.
// In a launch of its own the decoding cost 4 us on the GPU and 2.5 us on the host.  Where a few requests have 32 or 64 workgroups each, their
// arrivals one after the other take longer than that launch replayed from a graph (4 x 4 x 4096 entries of 392 14.4 us, 13.5; as ordinary calls 16.1, 17.7).
// The order of maximum, count and decoding rests on gfx950 and not on the memory model, whose release and acquire write back and
// invalidate a whole L2 (+3 us with 256 workgroups): the words are touched by agent-scope atomics alone, which are carried out at memory for all
// XCDs; a wave waits for its own with vmcnt, the barrier joins the waves, and only then is the arrival sent.
constexpr int64_t SPLIT_MAX_R = 512;   // more requests are not split: every wave reads all offsets, 64 at a time; not measured beyond
__device__ __forceinline__ void merge_parts(const u64 *__restrict__ partial, int64_t q_lo, int64_t q_hi, int parts, int32_t *ids,
                                            float *scores)
{
    __shared__ int s_last;
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): this wave's maxima are in place
    __syncthreads();
    if (threadIdx.x == 0)
        s_last = __hip_atomic_fetch_add(ids + q_lo, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == parts - 2;
    __syncthreads();
    if (!s_last) return;
    for (int64_t q = q_lo + threadIdx.x; q < q_hi; q += blockDim.x) {
        const u64 b = __hip_atomic_load(partial + q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ids[q] = b ? key_id(b) : -1;
        scores[q] = b ? key_score(b) : -__builtin_inff();
    }
}
// Ranges that are not in order (they should be) may overlap, and with them the places that count arrivals: every request
// is then served by its first workgroup alone.
__device__ __forceinline__ bool ranges_in_order(const int64_t *__restrict__ off, int64_t R)
{
    bool sorted = true;
    for (int64_t r = threadIdx.x & 63; r < R; r += 64) sorted = sorted && off[r] <= off[r + 1];
    return __all(sorted);
}

// What cache_lookup_kernel needs before its rows and after them, its first argument.  It is read again from the arguments at the
// end, and the request's range from LDS: kept all the time they took scalar registers that the loop over the rows needs (arguments: 512
// requests x up to 8 queries x 4096 entries of 392 861 -> 978 us; range: 200 requests x 8 queries x 2048 entries of 600 286 -> 332, of 768 by
// squared distance 410 -> 423).
struct LookupEnd {
    const int64_t *q_offsets;
    int64_t R, Qt;
    int32_t *ids;
    float *scores;
    u64 *partial;   // NULL: a request has one workgroup
    int fill;       // answer the queries that no request owns
};
__device__ __forceinline__ LookupEnd lookup_end()
{
    typedef const __attribute__((address_space(4))) LookupEnd *Args;
    Args args = (Args)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(args));
    return {args->q_offsets, args->R, args->Qt, args->ids, args->scores, args->partial, args->fill};
}

// elements (c*CL_GS + sub)*4 .. +4 of a cached row, c = 0 .. NCH-1, widened exactly to fp32 (zeros
// for a missing row and past d)
template <int EX, int NCH>
__device__ __forceinline__ void cl_load_row(float4 (&x)[NCH], const void *__restrict__ exact, int64_t ld, int32_t id,
                                            bool ok, int sub, int d)
{
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
        const int j = (c * CL_GS + sub) * 4;
        x[c] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (ok && j < d) {
            if constexpr (EX == DT_F32) {
                x[c] = *reinterpret_cast<const float4 *>(static_cast<const float *>(exact) + (int64_t)id * ld + j);
            } else {
                const uint2 h = *reinterpret_cast<const uint2 *>(static_cast<const uint16_t *>(exact) + (int64_t)id * ld + j);
                x[c] = make_float4(f16_bits_to_f32(h.x & 0xffffu), f16_bits_to_f32(h.x >> 16),
                                   f16_bits_to_f32(h.y & 0xffffu), f16_bits_to_f32(h.y >> 16));
            }
        }
    }
}

constexpr int CL_QB = 4;    // queries scored together (independent sums hide the latency of the adds)
static_assert(CL_QB == 4, "the block dispatch in cache_lookup_kernel is written out for blocks of 4");

// NCH = float4 chunks of a row held by one lane (row element (c*CL_GS + sub)*4 .. +4).
// One block of NW waves per request.  A wave step scores CL_ROWS cached rows against all of the
// request's queries: the rows are gathered from the exact copy (while the previous rows are
// being scored: the loads of the next step are issued first), widened to double ONCE, and every
// query, kept in LDS as doubles, costs one fused multiply-add per element on top of that;
// CL_QB queries are scored together, whose independent sums hide the latency of the adds, and
// the 16 lane sums of a row meet through DPP.
// L2: the score is minus the squared distance (KNN-LM datastores) instead of the inner product.
// MAXQ (8 or 16): queries of a request held in LDS at a time (more are served in groups); their
// bests sit in registers, which is why wide rows take 8.
// LIST: the keys of all (query, cached row) pairs go to `list` instead of the best to the outputs (a template
// parameter: tested at run time it cost the lookup a quarter of its time).
template <int EX, int NCH, int NW, bool L2, int MAXQ, bool LIST>
__global__ __launch_bounds__(NW * 64) void cache_lookup_kernel(
    const LookupEnd to, const int32_t *__restrict__ cache_ids, const int32_t *__restrict__ cache_len, int C,
    const float *__restrict__ queries,
    const void *__restrict__ exact, int64_t ld, int64_t N, int d, int qgroup,
    u64 *__restrict__ list, uint32_t *__restrict__ list_len)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int dq = (d + 63) & ~63;                                  // a query's doubles in LDS
    double *qs = reinterpret_cast<double *>(smem);                  // [qgroup][dq], see below
    u64 *best = reinterpret_cast<u64 *>(qs + (size_t)qgroup * dq);  // [NW waves][CL_ROWS][qgroup]

    // gridDim.y workgroups share a request (few requests: spread each over many CUs); they then
    // merge their best keys (merge_parts)
    const int64_t r = blockIdx.x;
    const int part = blockIdx.y;
    int parts = gridDim.y;
    __shared__ int s_merge, s_fill;   // workgroups that merge (0: this one's bests are the answer); whether it answers the unowned
    __shared__ int64_t s_lo, s_hi;    // the request's queries
    if (!LIST) {
        const bool in_order = !to.partial || ranges_in_order(to.q_offsets, to.R);
        if (!in_order) {
            if (part > 0) return;
            parts = 1;
        }
        if (threadIdx.x == 0) {
            s_merge = to.partial && in_order ? parts : 0;
            s_fill = to.fill && r == 0;
        }
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int sub = lane % CL_GS, slot = lane / CL_GS;
    int64_t q_lo, q_hi;
    clamp_range(to.q_offsets, r, to.Qt, q_lo, q_hi);
    if (!LIST && threadIdx.x == 0) {
        s_lo = q_lo;
        s_hi = q_hi;
    }
    int len = cache_len[r];
    len = len < 0 ? 0 : (len > C ? C : len);
    const int32_t *ids = cache_ids + r * (int64_t)C;
    const int e_step = parts * NW * CL_ROWS;
    if (LIST && part == 0)
        for (int64_t q = q_lo + tid; q < q_hi; q += NW * 64) list_len[q] = (uint32_t)len;

    for (int64_t g0 = q_lo; g0 < q_hi; g0 += qgroup) {
        const int nq = (int)((q_hi - g0) < qgroup ? (q_hi - g0) : qgroup);
        __syncthreads();
        // A lane scores elements (c*16 + sub)*4 .. +3 of a row.  The query's elements are laid
        // out so that, for one c, the first two of the 16 lanes' four are contiguous (256 bytes),
        // then the last two: the two 16-byte reads of a lane are then free of bank conflicts.
        for (int i = tid * 4; i < nq * d; i += NW * 256) {
            const int qi = i / d, j = i - qi * d;
            const float4 y = *reinterpret_cast<const float4 *>(queries + g0 * d + i);
            double *dst = qs + (size_t)qi * dq + ((j >> 6) * 64) + ((j >> 2) & 15) * 2;
            dst[0] = (double)y.x;
            dst[1] = (double)y.y;
            dst[32] = (double)y.z;
            dst[33] = (double)y.w;
        }
        for (int i = tid; i < NW * CL_ROWS * qgroup; i += NW * 64) best[i] = 0ull;
        __syncthreads();
        u64 *my_best = best + (wave * CL_ROWS + slot) * qgroup;
        // best (score, id) per query so far, in registers of the row's first lane: the comparison
        // is two float compares, and a key is formed only once, at the end
        float best_sc[MAXQ];
        int32_t best_id[MAXQ];
#pragma unroll
        for (int i = 0; i < MAXQ; ++i) {
            best_sc[i] = -__builtin_inff();
            best_id[i] = -1;
        }

        int e0 = (part * NW + wave) * CL_ROWS;
        float4 xn[NCH];   // the next step's rows, in flight while this step's are scored
        int32_t id_n = e0 + slot < len ? ids[e0 + slot] : -1;
        bool ok_n = id_n >= 0 && (int64_t)id_n < N;
        cl_load_row<EX, NCH>(xn, exact, ld, id_n, ok_n, sub, d);
        for (; e0 < len; e0 += e_step) {
            const int32_t id = id_n;
            const bool ok = ok_n;
            double x[NCH][4];
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                x[c][0] = (double)xn[c].x;
                x[c][1] = (double)xn[c].y;
                x[c][2] = (double)xn[c].z;
                x[c][3] = (double)xn[c].w;
            }
            const int e_n = e0 + e_step + slot;
            id_n = e_n < len ? ids[e_n] : -1;
            ok_n = id_n >= 0 && (int64_t)id_n < N;
            cl_load_row<EX, NCH>(xn, exact, ld, id_n, ok_n, sub, d);

            // U queries q0 .. q0+U-1 against this step's rows
            auto score = [&](auto u_tag, auto q0_tag) __attribute__((always_inline)) {
                constexpr int U = decltype(u_tag)::value, q0 = decltype(q0_tag)::value;
                const double *qv[U];
                double sum[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    qv[u] = qs + (size_t)(q0 + u) * dq + sub * 2;
                    sum[u] = 0.0;
                }
#pragma unroll
                for (int c = 0; c < NCH; ++c) {
                    if ((c * CL_GS + sub) * 4 < d) {
#pragma unroll
                        for (int u = 0; u < U; ++u) {
                            const double2 y01 = *reinterpret_cast<const double2 *>(qv[u] + c * 64);
                            const double2 y23 = *reinterpret_cast<const double2 *>(qv[u] + c * 64 + 32);
                            if constexpr (L2) {
                                const double d0 = y01.x - x[c][0], d1 = y01.y - x[c][1];
                                const double d2 = y23.x - x[c][2], d3 = y23.y - x[c][3];
                                sum[u] += d0 * d0;
                                sum[u] += d1 * d1;
                                sum[u] += d2 * d2;
                                sum[u] += d3 * d3;
                            } else {
                                sum[u] += x[c][0] * y01.x;
                                sum[u] += x[c][1] * y01.y;
                                sum[u] += x[c][2] * y23.x;
                                sum[u] += x[c][3] * y23.y;
                            }
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const double t = row16_sum(sum[u]);
                    const float sc = (L2 ? (float)(-t) : (float)t) + 0.0f;   // -0 counts as +0, as in a key
                    if constexpr (LIST) {
                        if (sub == 0 && e0 + slot < len) list[(g0 + q0 + u) * C + e0 + slot] = ok ? make_key(sc, id) : 0ull;
                        continue;
                    }
                    // higher score, then lower id (ids of missing rows are -1 and never win)
                    const bool better = ok && (sc > best_sc[q0 + u] || (sc == best_sc[q0 + u] && id < best_id[q0 + u]));
                    best_sc[q0 + u] = better ? sc : best_sc[q0 + u];
                    best_id[q0 + u] = better ? id : best_id[q0 + u];
                }
            };
            // query blocks of CL_QB, the last one with as many sums as there are queries left
            // (block starts are compile-time constants: the bests are indexed statically)
            auto block = [&](auto q0_tag) __attribute__((always_inline)) {
                constexpr int q0 = decltype(q0_tag)::value;
                const int left = nq - q0;
                if (left >= 4) score(std::integral_constant<int, 4>{}, q0_tag);
                else if (left == 3) score(std::integral_constant<int, 3>{}, q0_tag);
                else if (left == 2) score(std::integral_constant<int, 2>{}, q0_tag);
                else if (left == 1) score(std::integral_constant<int, 1>{}, q0_tag);
            };
            block(std::integral_constant<int, 0>{});
            if (nq > 4) block(std::integral_constant<int, 4>{});
            if constexpr (MAXQ > 8) {
                if (nq > 8) block(std::integral_constant<int, 8>{});
                if (nq > 12) block(std::integral_constant<int, 12>{});
            }
        }
        if (LIST) continue;
        if (sub == 0) {
#pragma unroll
            for (int i = 0; i < MAXQ; ++i)
                if (i < nq && best_id[i] >= 0) my_best[i] = make_key(best_sc[i], best_id[i]);
        }
        __syncthreads();
        const LookupEnd end = lookup_end();
        const bool merge = s_merge != 0;
        for (int qi = tid; qi < nq; qi += NW * 64) {
            u64 b = 0ull;
            for (int w = 0; w < NW * CL_ROWS; ++w) {
                const u64 v = best[w * qgroup + qi];
                b = v > b ? v : b;
            }
            if (merge) {
                if (b) atomicMax(reinterpret_cast<unsigned long long *>(end.partial + g0 + qi), b);
            } else {
                end.ids[g0 + qi] = b ? key_id(b) : -1;
                end.scores[g0 + qi] = b ? key_score(b) : -__builtin_inff();
            }
        }
    }
    if (LIST) return;
    __syncthreads();
    if (s_merge && s_lo < s_hi) {
        const LookupEnd end = lookup_end();
        merge_parts(end.partial, s_lo, s_hi, s_merge, end.ids, end.scores);
    }
    if (s_fill) {
        const LookupEnd end = lookup_end();
        answer_unowned<NW * 64>(end.q_offsets, end.R, end.Qt, end.ids, end.scores, reinterpret_cast<uint32_t *>(smem));
    }
}

// ---- the same lookup on the fp64 matrix cores (inner-product metric) ---------------------------
// v_mfma_f64_4x4x4 multiplies four independent 4x4x4 blocks: operand A of lane l is element
// (i = l%4, k = l/16) of block (l/4)%4, operand B element (k = l/16, j = l%4) of that block, and
// the lane receives D(i = l/16, j = l%4).  Block b takes cached rows 4b .. 4b+3 of a step of 16
// rows and all blocks take the same 4 queries, so lane l feeds row l%16 and gets the score of row
// 4*((l/4)%4) + l/16 against query l%4: a step of 16 rows x 4 queries x 4 elements per
// instruction, sums in double, and no reduction across lanes.  A lane holds elements
// 4*CH*u + CH*(l/16) .. + CH-1 of its row (CH elements per 16-byte load: whole 64-byte pieces of
// a row per load instruction); the queries sit in LDS as doubles in the order the instructions
// consume them ([group of 4][instruction][k][j]: a wave reads 128 contiguous bytes, no bank
// conflicts).  More than 4 queries: one more instruction per group and element, same row operand.
constexpr int CM_NW = 8;
constexpr int CM_MAX_GROUPS = 4;     // groups of 4 queries whose doubles are in LDS at a time

// SEG = 16-byte pieces of a row that a lane has in flight per buffer; it divides the number of
// pieces per lane and row, d / (4 * CH).  LIST: as above; tested at run time it took the registers of fp32 rows of 64
// elements past 128 and with them the second workgroup of a CU, 30 to
// 60 % of the time (500 requests x 4096 rows 87 us, 69 as a template parameter; 2000 x 2 queries x 64 rows 22.4 and 14.1).
template <int EX, int SEG, bool LIST>
__global__ __launch_bounds__(CM_NW * 64) void cache_lookup_mfma_kernel(
    const int32_t *__restrict__ cache_ids, const int32_t *__restrict__ cache_len, int C,
    const float *__restrict__ queries, int64_t Qt, const int64_t *__restrict__ q_offsets,
    const void *__restrict__ exact, int64_t ld, int64_t N, int d, int ng_max,
    int32_t *spec_ids, float *spec_scores, u64 *partial, int fill, u64 *__restrict__ list, uint32_t *__restrict__ list_len)
{
    constexpr int CH = EX == DT_F32 ? 4 : 8;        // elements per 16-byte piece
    constexpr int ES = EX == DT_F32 ? 4 : 2;
    extern __shared__ __align__(16) unsigned char smem[];
    const int T = d / 4;                             // instructions per step and query group
    double *bq = reinterpret_cast<double *>(smem);   // [ng_max][T][4 k][4 j]
    u64 *best = reinterpret_cast<u64 *>(bq + (size_t)ng_max * T * 16);   // [4 * ng_max]

    const int64_t r = blockIdx.x;
    const int part = blockIdx.y;
    int parts = gridDim.y;
    if (!LIST && partial && !ranges_in_order(q_offsets, gridDim.x)) {
        if (part > 0) return;
        parts = 1;
        partial = nullptr;
    }
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int r16 = lane & 15, kq = lane >> 4;            // row of the step and k index this lane feeds
    const int ro = ((lane >> 2) & 3) * 4 + (lane >> 4);   // row of the step whose score this lane receives
    const int jq = lane & 3;                              // ... against this query of a group
    const int32_t *ids = cache_ids + r * (int64_t)C;
    // Rows that are one step of the request's waves or less are dealt out to its workgroups in turn: one workgroup after the other, the rows of 16
    // requests x 1024 entries by 16 went to the first eight (768 fp32 19.1 us, 17.9; 1 x 300 by 5 18.3, 13.5).  More are better off one after
    // the other, where the last workgroups have a step less (257 x 1024 by 3 of 1024 fp16 in turn 149, 136), and so are more workgroups than
    // CUs, where they make room for the next (the k best of 171 x 300 by 3 in turn 44.3, 37.6).
    const bool in_turn = C <= parts * (CM_NW * 16) && gridDim.x * gridDim.y <= 256;
    const int blk_first = in_turn ? wave * parts + part : part * CM_NW + wave, blk_step = parts * CM_NW;
    // What the first rows depend on, at once (a slot of the cache is there whether it is used or not; a split request has read all offsets
    // before): the ids of the rows this lane feeds and receives in its wave's first step and in the next.  Its rows then travel while
    // the queries are laid out; one after the other, 64 requests x 1024 entries of 768 took 41.6 us, now 39.9; the k best of 32 x 8 x 2048 of 1024 fp16 61.6 and 51.1.
    auto slot_at = [&](int e) { return e < C ? ids[e] : -1; };
    const int32_t feed_0 = slot_at(blk_first * 16 + r16), out_0 = slot_at(blk_first * 16 + ro);
    const int32_t feed_1 = slot_at((blk_first + blk_step) * 16 + r16), out_1 = slot_at((blk_first + blk_step) * 16 + ro);
    int64_t q_lo, q_hi;
    clamp_range(q_offsets, r, Qt, q_lo, q_hi);
    int len = cache_len[r];
    len = len < 0 ? 0 : (len > C ? C : len);
    const int NC = d / (4 * CH);                          // pieces per lane and row
    const int nsegs = NC / SEG;
    const int nblk = (len + 15) / 16;
    const unsigned char *base = static_cast<const unsigned char *>(exact) + kq * 16;
    if (LIST && part == 0)
        for (int64_t q = q_lo + tid; q < q_hi; q += CM_NW * 64) list_len[q] = (uint32_t)len;

    auto row_of = [&](int32_t id) {
        const bool ok = id >= 0 && (int64_t)id < N;
        return base + (int64_t)(ok ? id : 0) * ld * ES;
    };
    auto load = [&](uint4(&buf)[SEG], const unsigned char *rw, int sg) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < SEG; ++c) buf[c] = *reinterpret_cast<const uint4 *>(rw + (size_t)(sg * SEG + c) * 64);
    };

    for (int64_t g0 = q_lo; g0 < q_hi; g0 += 4 * ng_max) {
        const int nq = (int)((q_hi - g0) < 4 * ng_max ? (q_hi - g0) : 4 * ng_max);
        const int n_groups = (nq + 3) >> 2;
        if (g0 > q_lo) __syncthreads();   // (a barrier waits for all loads)
        auto run = [&](auto ng_tag) __attribute__((always_inline)) {
            constexpr int NG = decltype(ng_tag)::value;
            // the first step's rows are on their way while the queries are laid out
            uint4 buf0[SEG], buf1[SEG];
            if (blk_first < nblk) load(buf0, row_of(blk_first * 16 + r16 < len ? feed_0 : -1), 0);
            // four threads take the four queries of a group, piece by piece of four elements
#pragma unroll 1
            for (int g = 0; g < NG; ++g) {
                const int qi = g * 4 + (tid & 3);
                const float *src = queries + (g0 + qi) * d;
#pragma unroll 1
                for (int e = (tid >> 2) * 4; e < d; e += CM_NW * 64) {
                    const float4 v = qi < nq ? *reinterpret_cast<const float4 *>(src + e) : make_float4(0.f, 0.f, 0.f, 0.f);
                    double *to = bq + ((size_t)g * T + CH * (e / (4 * CH)) + e % CH) * 16 + ((e / CH) & 3) * 4 + (tid & 3);
                    to[0] = (double)v.x;
                    to[16] = (double)v.y;
                    to[32] = (double)v.z;
                    to[48] = (double)v.w;
                }
            }
            for (int i = tid; i < 4 * ng_max; i += CM_NW * 64) best[i] = 0ull;
            __syncthreads();
            int blk = blk_first;
            if (blk >= nblk) return;
            float best_sc[NG];
            int32_t best_id[NG];
            double acc[NG];
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                best_sc[g] = -__builtin_inff();
                best_id[g] = -1;
                acc[g] = 0.0;
            }
            // ids of the rows this lane feeds and receives, for this step and (ahead) the next
            auto id_at = [&](int e) { return e < len ? ids[e] : -1; };
            auto used = [&](int e, int32_t id) { return e < len ? id : -1; };
            int32_t id_out = used(blk * 16 + ro, out_0);
            const unsigned char *row = row_of(used(blk * 16 + r16, feed_0));
            int32_t id_feed_n = used((blk + blk_step) * 16 + r16, feed_1), id_out_n = used((blk + blk_step) * 16 + ro, out_1);
            int seg = 0;
            // one (step, segment) item: issue the next item's loads, multiply this one's pieces
            auto item = [&](uint4(&cur)[SEG], uint4(&nxt)[SEG]) __attribute__((always_inline)) -> bool {
                const bool last_seg = seg + 1 == nsegs;
                const int blk_n = last_seg ? blk + blk_step : blk;
                const bool more = blk_n < nblk;
                const unsigned char *row_n = last_seg ? row_of(id_feed_n) : row;
                if (more) load(nxt, row_n, last_seg ? 0 : seg + 1);
                const double *bl = bq + (size_t)seg * (SEG * CH * 16) + kq * 4 + jq;
#pragma unroll
                for (int c = 0; c < SEG; ++c) {
                    {
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
                        for (int e = 0; e < CH; ++e) {
#pragma unroll
                            for (int g = 0; g < NG; ++g)
                                acc[g] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[e], bl[((size_t)g * T + c * CH + e) * 16], acc[g], 0, 0, 0);
                        }
                    }
                }
                if (last_seg) {
                    const bool ok = id_out >= 0 && (int64_t)id_out < N;
#pragma unroll
                    for (int g = 0; g < NG; ++g) {
                        const float sc = (float)acc[g] + 0.0f;   // -0 counts as +0, as in a key
                        if constexpr (LIST) {
                            if (g * 4 + jq < nq && blk * 16 + ro < len)
                                list[(g0 + g * 4 + jq) * C + blk * 16 + ro] = ok ? make_key(sc, id_out) : 0ull;
                            acc[g] = 0.0;
                            continue;
                        }
                        // higher score, then lower id
                        const bool better = ok && g * 4 + jq < nq &&
                                            (sc > best_sc[g] || (sc == best_sc[g] && id_out < best_id[g]));
                        best_sc[g] = better ? sc : best_sc[g];
                        best_id[g] = better ? id_out : best_id[g];
                        acc[g] = 0.0;
                    }
                    blk = blk_n;
                    seg = 0;
                    row = row_n;
                    id_out = id_out_n;
                    if (more) {
                        id_feed_n = id_at((blk + blk_step) * 16 + r16);
                        id_out_n = id_at((blk + blk_step) * 16 + ro);
                    }
                } else {
                    ++seg;
                }
                return !more;
            };
            for (;;) {
                if (item(buf0, buf1)) break;
                if (item(buf1, buf0)) break;
            }
#pragma unroll
            for (int g = 0; g < NG; ++g)
                if (best_id[g] >= 0)
                    atomicMax(reinterpret_cast<unsigned long long *>(best + g * 4 + jq), make_key(best_sc[g], best_id[g]));
        };
        if (n_groups == 1) run(std::integral_constant<int, 1>{});
        else if (n_groups == 2) run(std::integral_constant<int, 2>{});
        else if (n_groups == 3) run(std::integral_constant<int, 3>{});
        else run(std::integral_constant<int, 4>{});
        if (LIST) continue;
        __syncthreads();
        for (int qi = tid; qi < nq; qi += CM_NW * 64) {
            const u64 b = best[qi];
            if (partial) {
                if (b) atomicMax(reinterpret_cast<unsigned long long *>(partial + g0 + qi), b);
            } else {
                spec_ids[g0 + qi] = b ? key_id(b) : -1;
                spec_scores[g0 + qi] = b ? key_score(b) : -__builtin_inff();
            }
        }
    }
    if (!LIST && partial && q_lo < q_hi) merge_parts(partial, q_lo, q_hi, parts, spec_ids, spec_scores);
    if (!LIST && fill && r == 0)
        answer_unowned<CM_NW * 64>(q_offsets, gridDim.x, Qt, spec_ids, spec_scores, reinterpret_cast<uint32_t *>(smem));
}

__global__ __launch_bounds__(256) void verify_kernel(const int32_t *__restrict__ spec,
                                                     const int32_t *__restrict__ truth,
                                                     int64_t true_stride, int64_t Qt,
                                                     const int64_t *__restrict__ q_offsets, int64_t R,
                                                     int32_t *__restrict__ first_mismatch)
{
    // one wave per request; lanes look at 64 consecutive steps at a time
    const int lane = threadIdx.x & 63;
    const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= R) return;
    int64_t lo, hi;
    clamp_range(q_offsets, r, Qt, lo, hi);
    const int64_t s = hi - lo;
    int64_t m = s;
    for (int64_t base = 0; base < s; base += 64) {
        const int64_t i = base + lane;
        const bool differ = i < s && spec[lo + i] != truth[(lo + i) * true_stride];
        const unsigned long long mask = __ballot(differ);
        if (mask) {
            m = base + __ffsll((long long)mask) - 1;
            break;
        }
    }
    if (lane == 0) first_mismatch[r] = (int32_t)m;
}

// Cache update.  One workgroup per request; the request's cache row sits in LDS.  The candidates'
// order matters (once the ring is full an insertion evicts an entry, and a later candidate may be that
// entry), but only the slots that the next insertions take can change meanwhile.  So candidates
// are taken 64 at a time, one per lane:
//   1. wave 0 takes the next 64 slots in insertion order (the "zone") out of LDS into registers, one
//      per lane;
//   2. every wave compares the 64 candidates with its part of the remaining slots (an id read from
//      LDS serves all lanes): whoever is found there is a member whatever happens in the zone;
//   3. where none of the others is in the zone as it was (nothing waits there to be evicted before it is asked for), those that no
//      earlier one of the batch equals take the zone's slots in order, all at once;
//   4. otherwise wave 0 walks them in order: a member of the zone as it is by then is skipped, anyone
//      else takes the zone's next slot.
// A batch ends early when its zone is used up, unless the zone is the whole ring: then it goes round (step 4).
// What bounds it: step 2's LDS reads, len / (4 waves) of them per 64 candidates (eight of a wave's travel together), four
// barriers and the candidates' ids from memory.  The former version gave one wave to a request and spread one candidate's test over its
// lanes, a chain of len / 256 LDS reads per candidate.  64 requests x 80 candidates into caches of one entry, us: one
// candidate at a time 34, in batches that end with the ring 87, now 15.  512 requests x up to 160 candidates, caches
// of 4096: 456 us one at a time, 71 in batches, 28 with step 3 and an exclusive or and a minimum per slot for a compare and its scalar
// or, 32 requests x 640 candidates, caches of 2048: 811, 97, 32.
constexpr int CI_THREADS = 512, CI_WAVES = CI_THREADS / 64;

__global__ __launch_bounds__(CI_THREADS) void cache_insert_kernel(
    int32_t *__restrict__ cache_ids, int32_t *__restrict__ cache_len, int32_t *__restrict__ cache_head, int C,
    const int32_t *__restrict__ truth, int64_t true_stride, int64_t Qt, const int64_t *__restrict__ q_offsets,
    const int32_t *__restrict__ first_mismatch, int p, int n_next, int64_t N)
{
    extern __shared__ __align__(16) int32_t cs[];   // [C rounded up to 256]; slots >= len hold -1
    __shared__ u64 s_member[CI_WAVES];
    __shared__ int s_len, s_head, s_taken;
    const int64_t r = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int64_t q_lo, q_hi;
    clamp_range(q_offsets, r, Qt, q_lo, q_hi);
    int64_t n = q_hi - q_lo;
    if (first_mismatch) {
        int64_t fm = first_mismatch[r];
        fm = fm < 0 ? 0 : fm;
        if (fm + 1 < n) n = fm + 1;        // steps up to and including the first mis-speculated one
    }
    if (n <= 0) return;
    int len = cache_len[r];
    len = len < 0 ? 0 : (len > C ? C : len);
    int head = cache_head[r];
    head = head < 0 || head >= C ? 0 : head;
    int32_t *ids = cache_ids + r * (int64_t)C;
    const int cpad = (C + 255) & ~255;
    for (int x = tid; x < cpad; x += CI_THREADS) cs[x] = x < len ? ids[x] : -1;

    // candidates in order: step, then rank, then successor offset
    const int64_t per_rank = n_next > 0 ? n_next : 1, per_step = per_rank * p, total = per_step * n;
    const int first = n_next > 0 ? 1 : 0;
    auto candidate = [&](int64_t c) __attribute__((always_inline)) -> int32_t {   // -1: none
        if (c >= total) return -1;
        int64_t step, rank, off;
        if (total <= 0x7fffffffLL) {   // wave-uniform: 64-bit divisions are emulated
            const uint32_t c32 = (uint32_t)c, ps = (uint32_t)per_step, pr = (uint32_t)per_rank;
            const uint32_t s32 = c32 / ps, in_step = c32 - s32 * ps, k32 = in_step / pr;
            step = s32;
            rank = k32;
            off = in_step - k32 * pr;
        } else {
            step = c / per_step;
            rank = (c - step * per_step) / per_rank;
            off = c - step * per_step - rank * per_rank;
        }
        const int64_t t = truth[(q_lo + step) * true_stride + rank];
        const int64_t e64 = t + first + off;
        return t >= 0 && e64 < N ? (int32_t)e64 : -1;
    };
    // The barriers order LDS alone: the ids of the next batch travel across them, and so do the stores of the last one's.
    auto meet = [&]() __attribute__((always_inline)) { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
    int32_t e_next = candidate(lane);
    int64_t next_at = 0;               // the first candidate that e_next holds
    __syncthreads();
    for (int64_t base = 0; base < total;) {
        const int32_t e = base == next_at ? e_next : candidate(base + lane);
        next_at = base + 64;
        e_next = candidate(next_at + lane);
        // 64 places without a candidate (an unfilled rank, successors past the datastore's end): the rest of the last
        // place's rank has none either.  65536 successors of each of 64 ids at the end, four requests: 46 ms batch by
        // batch, 0.03 ms this way
        if (!__any(e >= 0)) {              // the same in every wave
            const int64_t c = base + 63;
            base = c < total ? (c / per_rank + 1) * per_rank : total;
            continue;
        }
        // the zone: the slots behind the last entry, or the oldest entries once the ring is full
        const int zone_at = len < C ? len : head, room = len < C ? C - len : C;
        const int zone_n = room < 64 ? room : 64;
        int slot = zone_at + lane;
        slot = slot >= C ? slot - C : slot;
        meet();                   // the row is in LDS; the last batch's zone is back in it
        int32_t zone = -1;
        if (wave == 0 && lane < zone_n) {
            zone = cs[slot];
            cs[slot] = -1;
        }
        meet();
        // the least exclusive or with a slot: zero if one equals (a compare per slot would write a scalar that the next one reads)
        uint32_t apart = ~0u;
        auto nearer = [&](uint32_t a, uint32_t b) __attribute__((always_inline)) {
            const uint32_t m = a < b ? a : b;
            apart = m < apart ? m : apart;
        };
        for (int x = wave * 32; x < len; x += CI_WAVES * 32) {   // (slots from len on hold -1)
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int4 v = *reinterpret_cast<const int4 *>(cs + x + i * 4);   // one address: every lane gets it
                nearer((uint32_t)(v.x ^ e), (uint32_t)(v.y ^ e));
                nearer((uint32_t)(v.z ^ e), (uint32_t)(v.w ^ e));
            }
        }
        const bool member = apart == 0;
        const u64 found = __ballot(member && e >= 0);
        if (lane == 0) s_member[wave] = found;
        meet();
        if (wave == 0) {
            u64 todo = __ballot(e >= 0);
            u64 safe = 0;
            for (int w = 0; w < CI_WAVES; ++w) safe |= s_member[w];
            todo &= ~safe;
            int used = 0, taken = 64;      // used: the zone's slot that takes the next insertion
            bool round = false;            // the zone is the ring and has been gone round
            const int n_todo = __popcll((long long)todo);
            if (n_todo > 12 && (n_todo <= zone_n || len < C || zone_n < C)) {   // (so few are walked faster than compared)
                u64 repeated = 0, in_zone = 0;
                for (int c0 = 0; c0 < 64 && !(todo & in_zone); c0 += 8) {   // (the walk it is as soon as one is found in the zone)
#pragma unroll
                    for (int i = 0; i < 8; ++i) {
                        const int c = c0 + i;
                        const int32_t ec = __builtin_amdgcn_readlane(e, c);
                        repeated |= __ballot(e == ec) & (~1ull << c);
                        in_zone |= __ballot(zone == ec) && ec >= 0 ? 1ull << c : 0ull;
                    }
                }
                const u64 fresh = todo & ~repeated;
                const int n_fresh = __popcll((long long)fresh);
                if (!(todo & in_zone)) {   // wave-uniform
                    used = n_fresh < zone_n ? n_fresh : zone_n;
                    const int rank = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(fresh >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)fresh, 0u));
                    const bool mine = (fresh >> lane) & 1;
                    // no slot left in the zone for the first of these: it opens the next batch
                    const u64 left = __ballot(mine && rank >= zone_n);
                    if (left) taken = __ffsll((long long)left) - 1;
                    // to the zone's lane `rank`; the others' go to lane 63, which listens only if there are no others
                    const int32_t sent = __builtin_amdgcn_ds_permute((mine ? rank : 63) * 4, e);
                    zone = lane < used ? sent : zone;
                    todo = 0;
                }
            }
            while (todo) {                 // wave-uniform
                const int c = __ffsll((long long)todo) - 1;
                const int32_t ec = __builtin_amdgcn_readlane(e, c);
                if (!__any(zone == ec)) {
                    if (used == zone_n) {
                        if (len < C || zone_n < C) {   // no slot left in the zone: this candidate opens the next batch
                            taken = c;
                            break;
                        }
                        used = 0;
                        round = true;
                    }
                    if (lane == used) zone = ec;
                    ++used;
                }
                todo &= todo - 1;
            }
            if (lane < zone_n) {
                cs[slot] = zone;
                if (lane < used || round) ids[slot] = zone;
            }
            if (lane == 0) {
                s_taken = taken;
                s_len = len < C ? len + used : len;
                const int h = head + used;
                s_head = len < C ? head : (h >= C ? h - C : h);
            }
        }
        meet();
        base += s_taken;
        len = s_len;
        head = s_head;
    }
    if (tid == 0) {
        cache_len[r] = len;
        cache_head[r] = head;
    }
}

// The k best entries of a request's cache for each of its queries.  The lookup kernels above leave the
// key of every (query, cache slot) pair in list[q * C + slot], 0 where the slot holds no row, and the
// number of slots in list_len[q]; here a workgroup sorts one query's keys and writes the first k.  A cached
// row is thus read and widened once for all queries of its request; with a workgroup per query that gathered
// the rows for itself a call took 256 us for 32 requests x 8 queries x 2048 fp16 rows of 1024, and
// 105 us for 16 x 4 x 1000 by squared distance; now 100 and 61 us.
template <int NT>
__global__ __launch_bounds__(NT) void cache_rank_kernel(const u64 *__restrict__ list, const uint32_t *__restrict__ list_len,
                                                        int C, int k, int32_t *__restrict__ out_ids,
                                                        float *__restrict__ out_scores)
{
    extern __shared__ __align__(16) unsigned char smem[];
    u64 *keys = reinterpret_cast<u64 *>(smem);   // [C rounded up to a power of two]
    const int64_t q = blockIdx.x;
    const int len = (int)list_len[q];            // at most C
    int n2 = 2;
    while (n2 < len) n2 <<= 1;
    for (int i = threadIdx.x; i < n2; i += NT) keys[i] = i < len ? list[q * C + i] : 0ull;
    __syncthreads();
    sort_keys<NT, true>(keys, n2);
    for (int i = threadIdx.x; i < k; i += NT) {
        const u64 key = i < len ? keys[i] : 0ull;
        out_ids[q * k + i] = key ? key_id(key) : -1;
        out_scores[q * k + i] = key ? key_score(key) : -__builtin_inff();
    }
}

// Candidate lists for the k-entry cache retrieval by the re-score (cache_topk_by_rescore): every query of a request gets the request's
// valid cached ids as ranking keys (score part 0), in any order; one workgroup per request.
__global__ __launch_bounds__(256) void cache_keys_kernel(const int32_t *__restrict__ cache_ids,
                                                         const int32_t *__restrict__ cache_len, int C, int64_t Qt,
                                                         const int64_t *__restrict__ q_offsets, int64_t N,
                                                         u64 *__restrict__ keys, uint32_t *__restrict__ cnt)
{
    __shared__ uint32_t s_n;
    const int64_t r = blockIdx.x;
    int64_t q_lo, q_hi;
    clamp_range(q_offsets, r, Qt, q_lo, q_hi);
    if (q_hi <= q_lo) return;
    int len = cache_len[r];
    len = len < 0 ? 0 : (len > C ? C : len);
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    for (int x = threadIdx.x; x < len; x += 256) {
        const int32_t id = cache_ids[r * (int64_t)C + x];
        if (id >= 0 && (int64_t)id < N) {
            const uint32_t at = atomicAdd(&s_n, 1u);
            const u64 key = make_key(0.f, id);
            for (int64_t q = q_lo; q < q_hi; ++q) keys[q * C + at] = key;
        }
    }
    __syncthreads();
    for (int64_t q = q_lo + threadIdx.x; q < q_hi; q += 256) cnt[q] = s_n;
}

__global__ void fill_u32_kernel(uint32_t *p, uint32_t v, int64_t n)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}
// Before a lookup: the merge slots and, in the first answer of each of the R requests, the count of arrivals (merge_parts); the answer
// of queries that no request owns.  partial == NULL, every_row == 0: not wanted.
__global__ void lookup_init_kernel(u64 *partial, const int64_t *__restrict__ q_offsets, int64_t R, int32_t *ids, float *scores,
                                   int every_row, int64_t Qt)
{
    const int64_t n = R > Qt ? R : Qt, step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += step) {
        if (partial && i < Qt) partial[i] = 0ull;
        if (every_row && i < Qt) {
            ids[i] = -1;
            scores[i] = -__builtin_inff();
        }
        if (partial && !every_row && i < R) {
            int64_t lo, hi;
            clamp_range(q_offsets, i, Qt, lo, hi);
            if (lo < hi) ids[lo] = -1;
        }
    }
}

// query preparation: queries rounded to the scan dtype, zero padded to [Qpad, dpad]
// L2: the scan scores a row as 2<q, x> - |x|^2, its squared norm being stored behind the row as the
// sum of two scan-dtype numbers (columns d and d+1): the query is doubled and gets -1 in both.
// The same launch clears two ranges of 32-bit words (the call's counters and list lengths), which
// saves three tiny launches per retrieval call.
template <int DT, bool L2>
__global__ void query_prep_kernel(const float *__restrict__ q, int64_t Q, int d, uint16_t *__restrict__ out,
                                  int64_t Qpad, int dpad, uint32_t *__restrict__ z0, int64_t n0,
                                  uint32_t *__restrict__ z1, int64_t n1)
{
    const int64_t n = Qpad * dpad;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n0; i += (int64_t)gridDim.x * blockDim.x)
        z0[i] = i == FLAG_QUERIES ? (uint32_t)Q : (i == FLAG_MARK ? (uint32_t)Q ^ FLAG_MARK_XOR : 0u);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n1; i += (int64_t)gridDim.x * blockDim.x) z1[i] = 0u;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t row = i / dpad;
        const int col = (int)(i % dpad);
        uint32_t bits = 0;
        if (row < Q && col < d) bits = f32_to_scan_bits<DT>(L2 ? 2.f * q[row * d + col] : q[row * d + col]);
        if (L2 && row < Q && (col == d || col == d + 1)) bits = f32_to_scan_bits<DT>(-1.f);
        out[i] = (uint16_t)bits;
    }
}

template <int DT>
__global__ void convert_rows_kernel(const float *__restrict__ src, int64_t src_ld, uint16_t *__restrict__ dst,
                                    int64_t dst_ld, int64_t N, int d8)
{
    // one 8-element chunk per thread step
    const int64_t n = N * d8;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t row = i / d8;
        const int c = (int)(i % d8) * 8;
        const float4 a = *reinterpret_cast<const float4 *>(src + row * src_ld + c);
        const float4 b = *reinterpret_cast<const float4 *>(src + row * src_ld + c + 4);
        *reinterpret_cast<uint4 *>(dst + row * dst_ld + c) = pack8<DT>(a, b);
    }
}

// Scan copy for the squared-distance metric: one wave per row.  dst row = the d elements rounded
// to the scan dtype (skipped when dst is src: fp16 keys that are their own scan copy), then the
// row's squared norm (summed in double from the source) as hi + lo in the scan dtype, then six
// zeros: 8 extra columns, 16 bytes.
template <int SRC, int DT>
__global__ __launch_bounds__(256) void l2_scan_copy_kernel(const void *src, int64_t src_ld,
                                                            uint16_t *dst, int64_t dst_ld, int64_t N, int d,
                                                            int in_place)
{
    const int lane = threadIdx.x & 63;
    // rows are strided over a bounded grid: one block per four rows would exceed the 2^32 work-items
    // of a launch from 67M rows on
    for (int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); row < N; row += (int64_t)gridDim.x * 4) {
        double sum = 0.0;
        for (int c = lane * 8; c < d; c += 512) {
            float4 a, b;
            if constexpr (SRC == DT_F32) {
                const float *s = static_cast<const float *>(src) + row * src_ld + c;
                a = *reinterpret_cast<const float4 *>(s);
                b = *reinterpret_cast<const float4 *>(s + 4);
            } else {
                const uint4 h = *reinterpret_cast<const uint4 *>(static_cast<const uint16_t *>(src) + row * src_ld + c);
                a = make_float4(f16_bits_to_f32(h.x & 0xffffu), f16_bits_to_f32(h.x >> 16),
                                f16_bits_to_f32(h.y & 0xffffu), f16_bits_to_f32(h.y >> 16));
                b = make_float4(f16_bits_to_f32(h.z & 0xffffu), f16_bits_to_f32(h.z >> 16),
                                f16_bits_to_f32(h.w & 0xffffu), f16_bits_to_f32(h.w >> 16));
            }
            sum += (double)a.x * (double)a.x + (double)a.y * (double)a.y + (double)a.z * (double)a.z +
                   (double)a.w * (double)a.w + (double)b.x * (double)b.x + (double)b.y * (double)b.y +
                   (double)b.z * (double)b.z + (double)b.w * (double)b.w;
            if (!in_place) *reinterpret_cast<uint4 *>(dst + row * dst_ld + c) = pack8<DT>(a, b);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
        if (lane == 0) {
            const uint32_t hi = f32_to_scan_bits<DT>((float)sum);
            const float hi_f = DT == DT_F16 ? f16_bits_to_f32(hi) : __uint_as_float(hi << 16);
            const uint32_t lo = f32_to_scan_bits<DT>((float)(sum - (double)hi_f));
            *reinterpret_cast<uint4 *>(dst + row * dst_ld + d) = make_uint4(hi | (lo << 16), 0u, 0u, 0u);
        }
    }
}

int grid_for(int64_t n, int block)
{
    int64_t g = (n + block - 1) / block;
    if (g > 256 * 32) g = 256 * 32;
    if (g < 1) g = 1;
    return (int)g;
}

template <int EX, bool L2, bool LIST>
hipError_t launch_cache_ex_form(const int32_t *cache_ids, const int32_t *cache_len, int32_t C, int64_t R,
                           const float *queries, int64_t Qt, const int64_t *q_offsets, const void *exact,
                           int64_t ld, int64_t N, int32_t d, int32_t *spec_ids, float *spec_scores,
                           u64 *partial, int fill, u64 *list, uint32_t *list_len, int parts, hipStream_t stream)
{
    int qgroup = CL_LDS_BYTES / (((d + 63) & ~63) * 8);
    const int nch = (d + CL_GS * 4 - 1) / (CL_GS * 4);
    const int maxq = nch <= 12 ? 16 : 8;
    if (qgroup > maxq) qgroup = maxq;
    if (qgroup < 1) return hipErrorInvalidValue;
    static_assert(64 * 8 >= FILL_MAX_QT / 8, "the bit map of answer_unowned fits the doubles of one query");
    // a lane keeps its NCH chunks in registers (as doubles, and the next rows' as floats), which
    // bounds the waves a block can hold
#define RALM_CL(NCHV, NWV, MAXQV)                                                                           \
    do {                                                                                                    \
        auto kern = cache_lookup_kernel<EX, NCHV, NWV, L2, MAXQV, LIST>;                                    \
        static std::atomic<bool> attr_done{false};                                                          \
        if (!attr_done.load(std::memory_order_acquire)) {                                                   \
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),                        \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);     \
            if (e != hipSuccess) return e;                                                                  \
            attr_done.store(true, std::memory_order_release);                                               \
        }                                                                                                   \
        hipLaunchKernelGGL(kern, dim3((unsigned)R, (unsigned)parts), dim3(NWV * 64),                        \
                           (size_t)qgroup * ((d + 63) & ~63) * 8 + (size_t)NWV * CL_ROWS * qgroup * sizeof(u64),   \
                           stream,                                                                          \
                           LookupEnd{q_offsets, R, Qt, spec_ids, spec_scores, partial, fill}, cache_ids, cache_len, C, \
                           queries, exact, ld, N, d, qgroup, list, list_len);                               \
    } while (0)
    if (nch <= 4) RALM_CL(4, 8, 16);
    else if (nch <= 8) RALM_CL(8, 8, 16);
    else if (nch <= 12) RALM_CL(12, 8, 16);
    else if (nch <= 16) RALM_CL(16, 4, 8);
    else if (nch <= 32) RALM_CL(32, 4, 8);
    else return hipErrorInvalidValue;
#undef RALM_CL
    return hipGetLastError();
}

template <int EX, bool L2>
hipError_t launch_cache_ex(const int32_t *cache_ids, const int32_t *cache_len, int32_t C, int64_t R,
                           const float *queries, int64_t Qt, const int64_t *q_offsets, const void *exact,
                           int64_t ld, int64_t N, int32_t d, int32_t *spec_ids, float *spec_scores,
                           u64 *partial, int fill, u64 *list, uint32_t *list_len, int parts, hipStream_t stream)
{
    return list ? launch_cache_ex_form<EX, L2, true>(cache_ids, cache_len, C, R, queries, Qt, q_offsets, exact, ld, N, d, spec_ids,
                                                     spec_scores, partial, fill, list, list_len, parts, stream)
                : launch_cache_ex_form<EX, L2, false>(cache_ids, cache_len, C, R, queries, Qt, q_offsets, exact, ld, N, d,
                                                      spec_ids, spec_scores, partial, fill, list, list_len, parts, stream);
}

// The matrix-core form of the lookup, for the shapes it is written for: inner product, rows of a
// multiple of 16 sixteen-byte pieces (d % 64 == 0 for fp32 rows, d % 128 == 0 for fp16 rows).
template <int EX>
bool cache_mfma_fits(int32_t d)
{
    const int nc = d / (EX == DT_F32 ? 16 : 32);
    return d % (EX == DT_F32 ? 64 : 128) == 0 && nc >= 4 && (size_t)d * 32 <= 64 * 1024;
}

// 16-byte pieces of a row that a lane of the matrix-core form has in flight; LIST: see the kernels.
// Four take half the registers, and two workgroups fit a CU: for requests that are split and fill the chip (64 x 1024 entries of 768
// 38.8 and 37.4, 300 x 4 x 2000 302 and 292), and where one workgroup to a CU would leave a second round of few (350 x 300 73 and
// 66).  Fewer workgroups than CUs would pair up and leave others idle (100 x 1024 by 2 56.0 and 60.4), and full rounds of
// whole requests are the better for long loads (256 x 4 x 1024 121 and 125, 512 x 4 x 2048 467 and 475).  So are workgroups of many
// elements, with the longest and with four: fp16 rows of 1024, 400 x 1 x 4096 whole 661, 723, 400 x 4 x 700 whole 124, 132, 64 x 1 x 4096 by 4 95.2, 101,
// 300 x 4 x 300 whole 62.9, 62.9; fp32 rows of 768 450 x 4 x 2048 whole 427, 446, 300 x 1 x 4096 by 4 563, 555, 400 x 4 x 700 whole 149, 144, of 128 400 x 2 x 4096 whole 154, 134.
// Lists: workgroups of one step of rows, of which there are at most two to a CU.  The k best, with the longest and with four: 16 requests x 8 queries x 2048
// fp16 rows of 1024 35.3, 34.1, 33 x 8 x 1024 fp32 rows of 768 45.7, 42.9, 300 x 64 23.8, 21.0; more rows 128 x 4 x 2048 fp16 116, 122, 600 x 1 x 2048 531, 587.
template <int EX, bool LIST>
int lookup_pieces(int32_t d, int64_t R, int32_t C, int parts)
{
    const int nc = d / (EX == DT_F32 ? 16 : 32);
    constexpr int FEW = EX == DT_F32 ? 1 << 20 : 1 << 19;   // elements of a workgroup's rows
    if (LIST ? (parts > 1 || (R > 256 && R <= 512)) && C <= parts * (CM_NW * 16) : (R * parts >= 256 && (int64_t)C * d <= (int64_t)parts * FEW && (parts > 1 || (R > 256 && R < 512)))) return 4;
    return nc % 8 == 0 ? 8 : (nc % 6 == 0 ? 6 : 4);
}

template <int EX, bool LIST>
hipError_t launch_cache_mfma_form(const int32_t *cache_ids, const int32_t *cache_len, int32_t C, int64_t R,
                             const float *queries, int64_t Qt, const int64_t *q_offsets, const void *exact,
                             int64_t ld, int64_t N, int32_t d, int32_t *spec_ids, float *spec_scores,
                             u64 *partial, int fill, u64 *list, uint32_t *list_len, int parts, hipStream_t stream)
{
    // a group of 4 queries takes d * 32 bytes of LDS (2 KB at least, and a bit map of FILL_MAX_QT queries 512); up to 64 KB, so that two requests share a CU
    int ng = (int)((64 * 1024) / ((size_t)d * 32));
    ng = ng > CM_MAX_GROUPS ? CM_MAX_GROUPS : ng;
    const size_t smem = (size_t)ng * d * 32 + (size_t)4 * ng * sizeof(u64);
#define RALM_CM(SEGV)                                                                                       \
    do {                                                                                                    \
        auto kern = cache_lookup_mfma_kernel<EX, SEGV, LIST>;                                               \
        static std::atomic<bool> attr_done{false};                                                          \
        if (!attr_done.load(std::memory_order_acquire)) {                                                   \
            hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),                        \
                                               hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024);      \
            if (e != hipSuccess) return e;                                                                  \
            attr_done.store(true, std::memory_order_release);                                               \
        }                                                                                                   \
        hipLaunchKernelGGL(kern, dim3((unsigned)R, (unsigned)parts), dim3(CM_NW * 64), smem, stream, cache_ids, \
                           cache_len, C, queries, Qt, q_offsets, exact, ld, N, d, ng, spec_ids, spec_scores,   \
                           partial, fill, list, list_len);                                                  \
    } while (0)
    switch (lookup_pieces<EX, LIST>(d, R, C, parts)) {
        case 8: RALM_CM(8); break;
        case 6: RALM_CM(6); break;
        default: RALM_CM(4);
    }
#undef RALM_CM
    return hipGetLastError();
}

template <int EX>
hipError_t launch_cache_mfma(const int32_t *cache_ids, const int32_t *cache_len, int32_t C, int64_t R,
                             const float *queries, int64_t Qt, const int64_t *q_offsets, const void *exact,
                             int64_t ld, int64_t N, int32_t d, int32_t *spec_ids, float *spec_scores,
                             u64 *partial, int fill, u64 *list, uint32_t *list_len, int parts, hipStream_t stream)
{
    return list ? launch_cache_mfma_form<EX, true>(cache_ids, cache_len, C, R, queries, Qt, q_offsets, exact, ld, N, d, spec_ids,
                                                   spec_scores, partial, fill, list, list_len, parts, stream)
                : launch_cache_mfma_form<EX, false>(cache_ids, cache_len, C, R, queries, Qt, q_offsets, exact, ld, N, d,
                                                    spec_ids, spec_scores, partial, fill, list, list_len, parts, stream);
}

}  // namespace

namespace {

// whether the rows take the matrix-core form of the lookup
bool lookup_on_matrix_cores(int32_t exact_dtype, int32_t metric, int32_t d)
{
    return metric == METRIC_IP && (exact_dtype == DT_F16 ? cache_mfma_fits<DT_F16>(d) : cache_mfma_fits<DT_F32>(d));
}

// the form of the lookup kernels that fits the rows
hipError_t launch_lookup(const int32_t *cache_ids, const int32_t *cache_len, int32_t C, int64_t R, const float *queries, int64_t Qt,
                         const int64_t *q_offsets, const void *exact, int32_t exact_dtype, int64_t ld, int64_t N, int32_t d,
                         int32_t metric, int32_t *spec_ids, float *spec_scores, u64 *partial, int fill, u64 *list, uint32_t *list_len,
                         int parts, hipStream_t stream)
{
#define RALM_CACHE(FN) \
    FN(cache_ids, cache_len, C, R, queries, Qt, q_offsets, exact, ld, N, d, spec_ids, spec_scores, partial, fill, list, list_len, parts, stream)
    const bool mfma = lookup_on_matrix_cores(exact_dtype, metric, d);
    if (exact_dtype == DT_F16) {
        if (metric == METRIC_L2) return RALM_CACHE((launch_cache_ex<DT_F16, true>));
        if (mfma) return RALM_CACHE(launch_cache_mfma<DT_F16>);
        return RALM_CACHE((launch_cache_ex<DT_F16, false>));
    }
    if (metric == METRIC_L2) return RALM_CACHE((launch_cache_ex<DT_F32, true>));
    if (mfma) return RALM_CACHE(launch_cache_mfma<DT_F32>);
    return RALM_CACHE((launch_cache_ex<DT_F32, false>));
#undef RALM_CACHE
}

}  // namespace

// Few cached rows are done whole about when the slots of a split request are cleared, in one launch instead of two.  On the matrix
// cores by their elements, in steps of 128 rows, GPU time and time in a stream of calls, by 1 and by as many as can be, one request x 4 queries: one step, fp32 rows of 640
// 13.2, 12.6 and 13.4, 14.5, fp16 rows of 1024 15.0, 14.8 and 15.1, 14.9; two, 129 fp32 rows of 512 13.7, 11.0 and 14.1, 14.7, of 640 16.4, 11.8 and 16.5,
// 14.6, 160 fp16 rows of 512 12.6, 10.6 and 12.9, 14.7; more, 33 x 1 x 300 fp32 rows of 64 6.3, 7.8, 384 of 128 9.5, 7.6 and 12.1, 14.7.  On the vector units, fp32
// rows and few queries: 16 x 1 x 160 of 392 10.0, 9.7 and 12.1, 14.7, 1 x 4 x 100 11.0, 11.3 and 11.9, 14.5; 8 x 8 x 129 19.0, 14.4 and 19.3, 14.6, 16 x 1 x 160 of 712 12.3, 10.8 and 12.6, 13.7 (once 11.2).
// The lines lie where the GPU time of a whole request is that of the three launches which a split one once took (384 of 128 9.0).
bool done_whole(int64_t R, int64_t Qt, int32_t C, int32_t exact_dtype, int32_t metric, int32_t d, bool mfma)
{
    const bool f16 = exact_dtype == DT_F16;
    if (mfma) return (int64_t)C * d <= (C > 256 ? 40000 : (C > 128 ? (f16 ? 81920 : 65536) : (f16 ? 131072 : 81920)));
    return !f16 && metric == METRIC_IP && (C <= 128 ? Qt <= 4 * R && d <= 640 : C <= 160 && Qt <= R && d <= 448);
}

// Workgroups per request, at most one for every 64 cached rows begun.  Up to 256 requests have one round at least that is as full as it
// can be, of 256 workgroups on 256 CUs: 33 requests x 1024 fp32 rows of 768 by 8 (264 workgroups) 38.7 us, by 7 31.9; 100 x 1024 by 3 76.8, by 2
// 55.4; 70 x 2048 by 4 113.6, by 3 80.9.  Fewer are never the better where the sums or the loads' latency take the time: 1 request x 8
// queries x 256 fp16 rows of 392 by 1 35.3, by 4 15.6, 96 x 8 x 500 by 1 87.4, by 2 51.4, 8 x 1 x 129 of 1000 by squared distance by 1 33.7,
// by 3 17.6.  Whether more rounds pay, a model of them says, a workgroup to a CU (lookup_pieces may fit two, which it leaves out): a round costs 7
// us until rows flow, and then its rows at what a CU takes alone (38 KB a us) or its share of the chip's 6000; more than one workgroup needs slots cleared and a merge (6 us).
// 300 x 1024 of 768 by 1 212, by 3 164.
int lookup_parts(int64_t R, int32_t C, int64_t row_bytes)
{
    if (R > SPLIT_MAX_R) return 1;
    const int64_t most = (C + 63) / 64, round = R < 256 ? 256 / R : 1;
    const double bytes = (double)C * (double)row_bytes;
    int best = 1;
    double least = 0.0;
    for (int p = (int)(round < most ? round : most); p <= 256 && p <= most; ++p) {
        const int64_t wgs = R * p, full = wgs / 256, rest = wgs % 256;
        const double per_cu = rest > 0 && 6000.0 / (double)rest < 38.0 ? 6000.0 / (double)rest : 38.0;
        const double us = 7.0 * (double)(full + (rest > 0)) + (p > 1 ? 6.0 : 0.0) +
                          bytes / p / 1000.0 * ((double)full * 256.0 / 6000.0 + (rest > 0 ? 1.0 / per_cu : 0.0));
        if (least == 0.0 || us < least + 0.1) {   // (of equals the one with more workgroups)
            least = us;
            best = p;
        }
    }
    return best;
}

// Workgroups per request of the list form: two workgroups per CU, or one where the request's queries, as doubles in LDS, leave no room
// for two; each with rows for half a step of its waves (matrix cores: 8 waves of 16 rows) or a whole one (vector units: 8 or 4
// waves of 4 rows).  With 64 rows each, 16 requests x 8 queries x 64 fp16 rows of 1024 by squared distance were four
// steps one after the other: 43 us, now 20.  As many as run at once.  Of two to a CU, where they leave more than a fifth of the places empty (a
// quarter if that is one per request), one more:
// by as many and by one more, 33 requests x 2048 fp16 rows of 1024 65.9, 69.6, 150 x 2048 136, 147, 400 x 1024 185, 189; 171 x 1024 105, 98, 200 x 1024
// 99.8, 94.8, 257 x 2048 346, 270, 300 x 1024 181, 146; one to a CU, 100 x 1024 of 1200 by squared distance 347, 450.
int list_parts(int64_t R, int32_t C, bool mfma, int32_t d)
{
    const int rows = mfma ? 64 : (d <= 768 ? 32 : 16), wgs = mfma || d <= 1024 ? 512 : 256;
    const int64_t at_once = R < wgs ? wgs / R : 1, most = (C + rows - 1) / rows;
    const bool full = wgs == 256 || R * 4 >= wgs * 3 || R * at_once * 5 >= wgs * 4;
    const int64_t want = full ? at_once : at_once + 1;
    return (int)(want < most ? want : most);
}

LookupRoute lookup_route(int64_t R, int64_t Qt, int32_t C, int32_t exact_dtype, int32_t metric, int32_t d, bool scratch, bool every_row,
                         bool list)
{
    const bool mfma = lookup_on_matrix_cores(exact_dtype, metric, d);
    LookupRoute to{};
    if (list) to.parts = list_parts(R, C, mfma, d);
    else if (!scratch || done_whole(R, Qt, C, exact_dtype, metric, d, mfma)) to.parts = 1;
    else to.parts = lookup_parts(R, C, (int64_t)d * (exact_dtype == DT_F16 ? 2 : 4));
    if (mfma) {
        if (exact_dtype == DT_F16) to.pieces = list ? lookup_pieces<DT_F16, true>(d, R, C, to.parts) : lookup_pieces<DT_F16, false>(d, R, C, to.parts);
        else to.pieces = list ? lookup_pieces<DT_F32, true>(d, R, C, to.parts) : lookup_pieces<DT_F32, false>(d, R, C, to.parts);
    }
    if (list) return to;
    // Without merge slots to clear the lookup's first workgroup answers the queries that no request owns
    to.fill = every_row && to.parts == 1 && R <= FILL_MAX_R && Qt <= FILL_MAX_QT;
    to.init = (to.parts > 1 || (every_row && !to.fill)) && Qt > 0;
    return to;
}

hipError_t launch_cache_lookup(const int32_t *cache_ids, const int32_t *cache_len, int32_t C, int64_t R,
                               const float *queries, int64_t Qt, const int64_t *q_offsets,
                               const void *exact, int32_t exact_dtype, int64_t ld, int64_t N, int32_t d,
                               int32_t metric, int32_t *spec_ids, float *spec_scores, bool every_row, u64 *partial,
                               hipStream_t stream)
{
    LookupRoute to{};
    if (R > 0) to = lookup_route(R, Qt, C, exact_dtype, metric, d, partial != nullptr, every_row, false);
    else to.init = every_row && Qt > 0;
    if (to.parts <= 1) partial = nullptr;
    if (to.init) {
        hipLaunchKernelGGL(lookup_init_kernel, dim3(grid_for(Qt > R ? Qt : R, 256)), dim3(256), 0, stream, partial, q_offsets,
                           R, spec_ids, spec_scores, every_row ? 1 : 0, Qt);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (R <= 0) return hipSuccess;
    return launch_lookup(cache_ids, cache_len, C, R, queries, Qt, q_offsets, exact, exact_dtype, ld, N, d, metric, spec_ids,
                         spec_scores, partial, to.fill ? 1 : 0, nullptr, nullptr, to.parts, stream);
}

// fp16 rows on the vector units are 8-byte pieces, with few of them in flight; that pays where a row serves several
// queries and not where there are enough queries for a workgroup each to fill the chip.  By the lookup kernels and
// by the re-score, squared distance, us: 256 requests x 1 query x 2048 rows of 1024 elements 518 and 188; 128 x 1 x 2048 of
// 2000 1125 and 317, 256 x 2 x 2048 2409 and 651, 256 x 4 x 512 577 and 339; inner product, 256 x 1 x 2048 of 392 216 and 119.
// fp32 rows were at least as fast by the lookup kernels in every shape tried (64 to 2048 cached rows, 1 to 8 queries).
bool cache_topk_by_rescore(int32_t exact_dtype, int32_t metric, int32_t d, int64_t R, int64_t Qt, int32_t C)
{
    if (d > CACHE_LOOKUP_MAX_D) return true;
    if (exact_dtype != DT_F16 || lookup_on_matrix_cores(exact_dtype, metric, d)) return false;
    if (d > 1024) return Qt >= 128 && (Qt <= 2 * R || (Qt >= 256 && C > 64));
    return Qt >= 256 && Qt <= R && (int64_t)C * d >= 128 * 768;
}

hipError_t launch_cache_lookup_topk(const int32_t *cache_ids, const int32_t *cache_len, int32_t C, int64_t R,
                                    const float *queries, int64_t Qt, const int64_t *q_offsets, const void *exact,
                                    int32_t exact_dtype, int64_t ld, int64_t N, int32_t d, int32_t metric, int32_t k,
                                    int32_t *out_ids, float *out_scores, u64 *list, uint32_t *list_len, hipStream_t stream)
{
    if (Qt <= 0) return hipSuccess;
    hipError_t e = launch_fill_u32(list_len, 0u, Qt, stream);   // queries that no request owns have no entries
    if (e != hipSuccess) return e;
    if (R > 0) {
        e = launch_lookup(cache_ids, cache_len, C, R, queries, Qt, q_offsets, exact, exact_dtype, ld, N, d, metric, nullptr,
                          nullptr, nullptr, 0, list, list_len,
                          lookup_route(R, Qt, C, exact_dtype, metric, d, true, false, true).parts, stream);
        if (e != hipSuccess) return e;
    }
    int c2 = 2;
    while (c2 < C) c2 <<= 1;
    if (c2 <= 512)
        hipLaunchKernelGGL(cache_rank_kernel<256>, dim3((unsigned)Qt), dim3(256), (size_t)c2 * 8, stream, list, list_len, C, k,
                           out_ids, out_scores);
    else
        hipLaunchKernelGGL(cache_rank_kernel<1024>, dim3((unsigned)Qt), dim3(1024), (size_t)c2 * 8, stream, list, list_len, C, k,
                           out_ids, out_scores);
    return hipGetLastError();
}

hipError_t launch_verify(const int32_t *spec, const int32_t *truth, int64_t true_stride, int64_t Qt,
                         const int64_t *q_offsets, int64_t R, int32_t *first_mismatch, hipStream_t stream)
{
    if (R <= 0) return hipSuccess;
    hipLaunchKernelGGL(verify_kernel, dim3((unsigned)((R + 3) / 4)), dim3(256), 0, stream, spec, truth,
                       true_stride, Qt, q_offsets, R, first_mismatch);
    return hipGetLastError();
}

hipError_t launch_cache_insert(int32_t *cache_ids, int32_t *cache_len, int32_t *cache_head, int32_t C, int64_t R,
                               const int32_t *truth, int64_t true_stride, int64_t Qt, const int64_t *q_offsets,
                               const int32_t *first_mismatch, int32_t p, int32_t n_next, int64_t N,
                               hipStream_t stream)
{
    if (R <= 0) return hipSuccess;
    const size_t smem = (size_t)((C + 255) & ~255) * sizeof(int32_t);
    static std::atomic<bool> attr_done{false};   // per instantiation; setting it twice is harmless
    if (!attr_done.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(cache_insert_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, CACHE_INSERT_MAX_C * 4);
        if (e != hipSuccess) return e;
        attr_done.store(true, std::memory_order_release);
    }
    hipLaunchKernelGGL(cache_insert_kernel, dim3((unsigned)R), dim3(CI_THREADS), smem, stream, cache_ids, cache_len,
                       cache_head, C, truth, true_stride, Qt, q_offsets, first_mismatch, p, n_next, N);
    return hipGetLastError();
}

hipError_t launch_cache_keys(const int32_t *cache_ids, const int32_t *cache_len, int32_t C, int64_t R, int64_t Qt,
                             const int64_t *q_offsets, int64_t N, u64 *keys, uint32_t *cnt, hipStream_t stream)
{
    hipError_t e = launch_fill_u32(cnt, 0u, Qt, stream);
    if (e != hipSuccess || R <= 0) return e;
    hipLaunchKernelGGL(cache_keys_kernel, dim3((unsigned)R), dim3(256), 0, stream, cache_ids, cache_len, C, Qt,
                       q_offsets, N, keys, cnt);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t stream)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for(n, 256)), dim3(256), 0, stream, p, v, n);
    return hipGetLastError();
}
hipError_t launch_l2_scan_copy(const void *src, int32_t src_dtype, int64_t src_ld, void *dst, int32_t dst_dtype,
                               int64_t dst_ld, int64_t N, int32_t d, hipStream_t stream)
{
    if (N <= 0) return hipSuccess;
    const int in_place = src == dst ? 1 : 0;
    const int64_t blocks = (N + 3) / 4;
    const dim3 grid((unsigned)(blocks < (1 << 20) ? blocks : (1 << 20))), block(256);
    uint16_t *out = static_cast<uint16_t *>(dst);
    if (src_dtype == DT_F16) {
        if (dst_dtype == DT_F16)
            hipLaunchKernelGGL((l2_scan_copy_kernel<DT_F16, DT_F16>), grid, block, 0, stream, src, src_ld, out, dst_ld, N, d, in_place);
        else
            hipLaunchKernelGGL((l2_scan_copy_kernel<DT_F16, DT_BF16>), grid, block, 0, stream, src, src_ld, out, dst_ld, N, d, in_place);
    } else {
        if (dst_dtype == DT_F16)
            hipLaunchKernelGGL((l2_scan_copy_kernel<DT_F32, DT_F16>), grid, block, 0, stream, src, src_ld, out, dst_ld, N, d, in_place);
        else
            hipLaunchKernelGGL((l2_scan_copy_kernel<DT_F32, DT_BF16>), grid, block, 0, stream, src, src_ld, out, dst_ld, N, d, in_place);
    }
    return hipGetLastError();
}

hipError_t launch_query_prep(const float *q, int64_t Q, int32_t d, uint16_t *out, int64_t Qpad, int32_t dpad,
                             int32_t scan_dtype, int32_t metric, uint32_t *z0, int64_t n0, uint32_t *z1, int64_t n1,
                             hipStream_t stream)
{
    const int64_t n = Qpad * dpad;
    if (n <= 0) return hipSuccess;
    const dim3 grid(grid_for(n, 256)), block(256);
    if (scan_dtype == DT_F16) {
        if (metric == METRIC_L2)
            hipLaunchKernelGGL((query_prep_kernel<DT_F16, true>), grid, block, 0, stream, q, Q, d, out, Qpad, dpad, z0, n0, z1, n1);
        else
            hipLaunchKernelGGL((query_prep_kernel<DT_F16, false>), grid, block, 0, stream, q, Q, d, out, Qpad, dpad, z0, n0, z1, n1);
    } else {
        if (metric == METRIC_L2)
            hipLaunchKernelGGL((query_prep_kernel<DT_BF16, true>), grid, block, 0, stream, q, Q, d, out, Qpad, dpad, z0, n0, z1, n1);
        else
            hipLaunchKernelGGL((query_prep_kernel<DT_BF16, false>), grid, block, 0, stream, q, Q, d, out, Qpad, dpad, z0, n0, z1, n1);
    }
    return hipGetLastError();
}

hipError_t launch_convert_rows(const float *src, int64_t src_ld, void *dst, int32_t dst_dtype, int64_t dst_ld,
                               int64_t N, int32_t d, hipStream_t stream)
{
    const int64_t n = N * (d / 8);
    if (n <= 0) return hipSuccess;
    if (dst_dtype == DT_F16)
        hipLaunchKernelGGL(convert_rows_kernel<DT_F16>, dim3(grid_for(n, 256)), dim3(256), 0, stream, src,
                           src_ld, static_cast<uint16_t *>(dst), dst_ld, N, d / 8);
    else
        hipLaunchKernelGGL(convert_rows_kernel<DT_BF16>, dim3(grid_for(n, 256)), dim3(256), 0, stream, src,
                           src_ld, static_cast<uint16_t *>(dst), dst_ld, N, d / 8);
    return hipGetLastError();
}

}  // namespace ralm
