// Fused scoring + threshold selection scan over the datastore (gfx950).
//
// This is the knowledge-base retrieval C.retrieve(q_1..q_s) of Alg. 1 (the batched
// verification step) for the exact dense retriever of Section 5.1: every datastore row is
// scored against every query of the batch by inner product.  The [N, Q] score matrix is
// never written: scores come out of the matrix cores (bf16 or fp16 inputs, fp32
// accumulation) and each one is compared at once with its query's admission key; the few
// that pass are appended to that query's candidate list.
//
// Tiling: a workgroup of 4 or 8 waves owns a 256-row x BN-query tile (64,
// 128 and 256 queries on 8 waves, two per SIMD; 32 queries: half of the rows, on 4 waves; a first stage of few tiles of more than 32
// queries: a quarter of the rows); the reduction dimension is walked in strips of BK elements.  Datastore rows are the A operand of v_mfma_f32_32x32x16, queries the B operand, so
// every accumulator register of a lane belongs to ONE query (column = lane % 32) and the lane
// can hold that query's threshold in a register.
//
// scan_dma_kernel takes bf16 / fp16 datastore copies, and fp32 rows as they are (rounded to bf16
// between the operand read and the multiply).  Strips go from global memory straight into LDS
// (global_load_lds_dwordx4, no VGPR staging) through a ring of S stages that runs ahead of the
// multiply and keeps running across tile boundaries; the 16-byte chunks of a row are XOR-swizzled
// on the way in (by choosing which global chunk each lane fetches) so that the MFMA operand reads
// (32 rows, same chunk) are free of bank conflicts.  What happens to a tile's scores depends on
// how many of them a launch keeps (KEEP_*): thresholds that admit a few per tile, thresholds that
// admit hundreds or more, or every score into empty lists.
//
// Work items (row tile, query tile) are dealt to a persistent grid so that workgroups that
// run at the same time on one XCD (workgroup b lands on XCD b % 8) hold consecutive items:
// all query tiles of a row tile, then the next row tile.  The row tile's second to last
// readers therefore hit that XCD's L2.
//
// Launches with selective thresholds of batches whose queries fit the registers of a workgroup are served by
// scan_held_kernels.hip.
#include <type_traits>

#include <atomic>

#include "../../include/ralm.h"
#include "scan_device.h"

namespace ralm {

namespace {

// acc[i][j][v] of a wave is the score of datastore row
//     row0 + (wm*TM + i)*32 + (v/4)*8 + (lane/32)*4 + v%4
// against query  q0 + (wn*TN + j)*32 + lane%32.  A score is admitted (appended to its query's
// candidate list) iff its ranking key is >= the query's admission key.

// Parked epilogue (pipelined kernel).  A column of a 32x32 block that may hold an admitted score is put aside as it is, its
// 16 scores and where they belong, in a list of the wave's own: no atomics and no waits between the multiplies.  sort_aside()
// tests the scores later, 128 at a time, and parks the admitted ones in a list of the workgroup's, which flush_parked() moves
// to the global lists.  An entry that finds that list full goes to its global list directly, so nothing is ever lost.
// Tested and parked at once, with an LDS read back and an LDS atomic waited for while the other waves come to the next rendezvous, admission
// cost 379 us of 4004 in the last stage of 256 neighbour queries over 10M x 1024 (54 scores a tile).  Whole rounds at once and put aside:
// these 6211, 6089 us, 64 queries by squared distance over 2M x 1024 899, 842, 2341 over 4M x 768 13 451, 13 305.
//
// The common case (no lane of the wave holds an admitted score) must be a handful of
// instructions: the pipelined kernel's last stage contains 16 copies of the test, and
// anything bulky in it pushes that stage out of the instruction cache.  So the rare case does
// not unroll over the 16 values (registers cannot be indexed dynamically, LDS can).
constexpr int PARK_MIN = 512, PARK_MAX = 1024;   // parked admitted scores per workgroup (12 bytes each)
constexpr int ASIDE_MAX = 28, ASIDE_BYTES = 72;  // columns that a wave puts aside: 16 scores, a row and a query each

// How the LDS behind a launch's ring is used: `tau_n` admission keys, `park` parked scores, `aside` columns per wave.  Long
// lists are sorted out and flushed less often, so they get what the admission keys leave.
struct ParkLayout {
    int tau_n, park, aside;
    int flush_every;   // tiles (a power of two) from one look at the parked entries to the next
};

// Epilogue of a launch that keeps every score into empty lists (the first stage of a ladder): the
// score of the launch's r-th row goes to slot r of its query's list, no atomics.  A lane's 16
// values are 4 runs of 4 consecutive rows: 8 stores of two keys each.  Rows past the datastore's
// end are the launch's last ones: their slots lie behind the list's length, which leaves them out.
__device__ __forceinline__ void store_block_all(const ScanParams &p, const f32x16 &out, int32_t row_id0, int64_t pos0,
                                                int q, bool qok)
{
    if (!qok) return;
    u64 *dst = p.cand + (int64_t)q * p.cap + pos0;
    typedef unsigned long long u64x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int c = 0; c < 4; ++c) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int v = c * 4 + h * 2;
            const u64x2 two = {make_key(out[v], row_id0 + c * 8 + h * 2), make_key(out[v + 1], row_id0 + c * 8 + h * 2 + 1)};
            *reinterpret_cast<u64x2 *>(dst + c * 8 + h * 2) = two;
        }
    }
}

// The same where a select that looks at few of these scores follows (launch_select_first): the scores alone, half the bytes, in the first
// 64 KB of the query's list, and behind them the best score of every 32 rows, as the high word of a key.  Slot r is the launch's r-th row, so
// the row's number need not be kept.
__device__ __forceinline__ void store_block_scores(const ScanParams &p, const f32x16 &out, int32_t row_id0, int32_t n_rows, int64_t pos0,
                                                   int q, bool qok)
{
    uint32_t best = 0;   // (no score's word)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const uint32_t b = row_id0 + (v >> 2) * 8 + (v & 3) < n_rows ? score_bits(out[v]) : 0u;   // rows past the end are the last row again
        best = b > best ? b : best;
    }
    const uint32_t other = lane_xor<32>(best);   // the other lanes' 16 of the 32 rows
    best = other > best ? other : best;
    if (!qok) return;
    float *dst = reinterpret_cast<float *>(p.cand + (int64_t)q * p.cap);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const f32x4 four = {out[c * 4], out[c * 4 + 1], out[c * 4 + 2], out[c * 4 + 3]};
        *reinterpret_cast<f32x4 *>(dst + pos0 + c * 8) = four;
    }
    if ((threadIdx.x & 32) == 0) reinterpret_cast<uint32_t *>(dst + FIRST_ROWS)[pos0 >> 5] = best;
}

// Epilogue of a launch whose thresholds admit many of a tile's scores.  Taken one by one (above) they
// fill the parking list many times over, and every one that finds it full costs a round trip to its
// query's length.  Here the tile's scores stay in the accumulators, each lane counts those of its
// columns that are admitted, the counts meet per query in LDS (`tally`, one word per column), the
// lengths move once per tile and query, and the keys are stored where their lane's share of the
// list begins.  All threads of the workgroup; tally is zero on entry and on return.
// 256 queries, 1024 fp16 elements, k' = 2048, tiles that admit half of their scores: 292 -> 55 us
// for a launch of 40 tiles.
template <int TM, int TN, int NT>
__device__ __forceinline__ void select_tile_counted(const ScanParams &p, const f32x16 (&acc)[TM][TN], RALM_LDS uint32_t *tally,
                                                    int32_t row_id0, int32_t n_rows, int q0, int col0, int BN,
                                                    const u64 (&tkey)[TN], const float (&tsc)[TN])
{
    uint32_t pass[TM][TN], at[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const bool every = tkey[j] == 0ull;   // fewer than k' keys so far: everything is admitted
        uint32_t n = 0;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            uint32_t m = 0;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int32_t row = row_id0 + i * 32 + (v >> 2) * 8 + (v & 3);
                const bool in = row < n_rows && (every || acc[i][j][v] >= tsc[j]) && make_key(acc[i][j][v], row) >= tkey[j];
                m |= in ? 1u << v : 0u;
            }
            pass[i][j] = m;
            n += (uint32_t)__popc(m);
            // (kept as the word it is: the compiler would keep the 16 conditions and run out of registers)
            asm("" : "+v"(pass[i][j]));
            RALM_SCHED_FENCE();
        }
        at[j] = n ? __hip_atomic_fetch_add(tally + col0 + j * 32, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) : 0u;
    }
    __syncthreads();
    for (int c = threadIdx.x; c < BN; c += NT) {
        const uint32_t m = tally[c];
        if (m) tally[c] = atomicAdd(p.cnt + (int64_t)(q0 + c) * CNT_PITCH, m);   // padding columns have none
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        uint32_t to = tally[col0 + j * 32] + at[j];
        u64 *dst = p.cand + (int64_t)(q0 + col0 + j * 32) * p.cap;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                if (pass[i][j] & (1u << v)) {
                    // the keys are formed again: kept from above they would not fit the registers
                    float score = acc[i][j][v];
                    int32_t row = row_id0;
                    asm("" : "+v"(score), "+v"(row));
                    if (to < p.cap) dst[to] = make_key(score, row + i * 32 + (v >> 2) * 8 + (v & 3));
                    ++to;
                }
            }
            RALM_SCHED_FENCE();
        }
    }
    __syncthreads();
    for (int c = threadIdx.x; c < BN; c += NT) tally[c] = 0;
    __syncthreads();
}

// What a launch keeps of a tile's scores, and how they get to the lists:
enum {
    KEEP_PARKED,    // the few that pass selective thresholds, by way of lists in LDS (select_block)
    KEEP_COUNTED,   // those that pass thresholds which admit many of a tile (select_tile_counted)
    KEEP_ALL,       // every score, into empty lists (store_block_all)
    KEEP_SCORES     // the same as scores and bests of 32 (store_block_scores)
};

// A counted launch of one narrow query tile parks nothing, and its admission keys and counts have places that the compiler knows: with places
// from the launch it took 5 % longer over fp32 rows (whole calls, k' = 512, 130 000 x 384: 33 queries 98 us, 95; 64 queries 106, 103).
template <int BN, int KEEP>
constexpr bool layout_fixed = KEEP == KEEP_COUNTED && BN <= 128;
template <int BN>
constexpr ParkLayout fixed_layout{BN, PARK_MIN, 4, 1};

// ---- direct-to-LDS pipelined kernel ----------------------------------------------------------
// eight fp32 values (two 16-byte chunks) -> eight bf16, round to nearest even, as an MFMA operand
__device__ __forceinline__ uint4 round8_bf16(const uint4 &lo, const uint4 &hi)
{
    typedef float f32x8 __attribute__((ext_vector_type(8)));
    const f32x8 f = {__uint_as_float(lo.x), __uint_as_float(lo.y), __uint_as_float(lo.z), __uint_as_float(lo.w),
                     __uint_as_float(hi.x), __uint_as_float(hi.y), __uint_as_float(hi.z), __uint_as_float(hi.w)};
    return __builtin_bit_cast(uint4, __builtin_convertvector(f, bf16x8));
}

constexpr int TAU_LDS_MAX_Q = 2560;   // admission keys of up to this many queries are kept in LDS (by the widest query tile)

// The instruction stream of a stage is laid out by hand (one wave per SIMD: nothing else fills
// the issue slots between MFMAs).  After each MFMA exactly one "side" instruction follows: an
// LDS operand read for the next k-step, or one 1 KB global->LDS load of the strip that is S-1
// stages ahead.  sched_barrier keeps the compiler from regrouping them.  In a tile's last
// k-step the MFMA results are written to VGPRs and each block's selection test runs two MFMAs
// behind its last multiply, so the selection costs no separate pass over the accumulators.
//
// The ring has S slots and the issue cursor runs D stages ahead of the multiply.  D = S - 1 (the
// loads issued during stage t refill the slot of stage t - 1) or D = S (they refill the slot of
// stage t itself, once every wave has read the operands of the stage's last k-step out of it: a
// ring of two 64-element strips then does the work of four 32-element strips, with half the
// rendezvous per multiply and whole 128-byte lines per request).  The rendezvous of a stage
// sits in k-step RK, behind that k-step's operand reads; the query part of the new strip is
// requested after it in the same k-step, the datastore part in the next k-step.  RK = KS - 2 is
// the k-step whose reads are the stage's last, which D = S needs.
//
// A32: the datastore rows are fp32 (a datastore scanned as it is).  They travel to LDS as they
// are, twice the bytes per strip row, and are rounded to bf16 between the operand read and the
// multiply (two 16-byte reads and four conversions per operand instead of one read).
// KEEP: what is kept of the scores (KEEP_*).
template <bool F16, int WM, int WN, int TM, int TN, int BK, int S, bool NTA, int D = S - 1, int RK = 0,
          bool A32 = false, int KEEP = KEEP_PARKED>
__global__ __launch_bounds__(WM *WN * 64) void scan_dma_kernel(const ScanParams p, const int nqt, const ParkLayout launched)
{
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32;
    const ParkLayout lay = layout_fixed<BN, KEEP> ? fixed_layout<BN> : launched;
    constexpr int ESA = A32 ? 4 : 2;                       // bytes of a datastore element
    constexpr int ROWB_A = BK * ESA, ROWB_B = BK * 2;      // bytes of one strip row (datastore, queries)
    constexpr int CPR_A = ROWB_A / 16, CPR_B = ROWB_B / 16;   // 16-byte chunks per strip row
    constexpr int RPI_A = 64 / CPR_A, RPI_B = 64 / CPR_B;  // rows covered by one wave load
    constexpr int NW = WM * WN, NT = NW * 64;     // waves (4: one per SIMD, 8: two per SIMD), threads
    constexpr int NA = BM / RPI_A / NW, NB = BN / RPI_B / NW;   // wave loads per wave and stage
    constexpr int LPS = NA + NB;
    constexpr int A_BYTES = BM * ROWB_A, B_BYTES = BN * ROWB_B, STAGE = A_BYTES + B_BYTES;
    static_assert(!(A32 && F16), "fp32 rows are rounded to bf16");
    constexpr int KS = BK / 16;
    constexpr int NM = TM * TN, NR = TM + TN;
    constexpr int LAG = NM > 2 ? 2 : NM - 1;     // selection runs this many MFMAs behind
    constexpr int RV = NR - 1;                   // slot of k-step RK after which the stage rendezvous sits
    // a workgroup tile covers the whole 256-row tile of the ladder, half or a quarter of it
    constexpr int PARTS = SCAN_BM / BM;
    static_assert((NW == 4 || NW == 8) && (PARTS == 1 || PARTS == 2 || PARTS == 4) && PARTS * BM == SCAN_BM &&
                      NA >= 1 && NB >= 1,
                  "tile shape");
    static_assert(S >= 2 && (D == S - 1 || D == S) && D >= 2 && KS % 2 == 0, "ring depth / k-steps per stage");
    static_assert(RK >= 0 && RK + 1 < KS && (D < S || RK == KS - 2), "rendezvous position");
    static_assert(LPS * (D - 1) < 64, "vmcnt range");

    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t lds0 = (uint32_t)(size_t)(RALM_LDS unsigned char *)smem;
    RALM_LDS u64 *tau_lds = (RALM_LDS u64 *)(smem + S * STAGE);
    PushList pl;
    pl.keys = tau_lds + lay.tau_n;
    pl.qs = (RALM_LDS uint32_t *)(pl.keys + lay.park);
    pl.count = pl.qs + lay.park;
    pl.cap = (uint32_t)lay.park;
    // columns put aside, wave by wave; in their place, while there are none, the counts per query column of a flush or of a counted launch
    RALM_LDS uint32_t *tally = pl.count + 4;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int fr = lane & 31;
    const int la_r = lane / CPR_A, la_c = lane % CPR_A;   // row and chunk of this lane in a wave load
    const int lb_r = lane / CPR_B, lb_c = lane % CPR_B;

    // item indices fit 32 bits: at most 2^23 row tiles times a few query tiles (host checks)
    const int G = (int)gridDim.x;
    const int vb = (int)(blockIdx.x % 8) * (G / 8) + (int)(blockIdx.x / 8);
    const int n_tiles = (int)p.n_row_tiles * PARTS;      // workgroup tiles of this launch
    const int total = n_tiles * nqt;
    // first datastore row of the rt-th workgroup tile
    auto tile_row0 = [&](int rt) __attribute__((always_inline)) -> int64_t {
        if constexpr (PARTS == 1) return visited_tile(p, rt) * SCAN_BM;
        else return visited_tile(p, rt / PARTS) * SCAN_BM + (rt % PARTS) * BM;
    };
    const int KT = p.dpad / BK;
    const int n_mine = vb < total ? (total - vb + G - 1) / G : 0;
    if constexpr (KEEP == KEEP_ALL || KEEP == KEEP_SCORES) {
        // every list ends up with one entry per row of the launch; only its last tile can be partial
        if (blockIdx.x == 0) {
            const int64_t rows = (p.n_row_tiles - 1) * SCAN_BM, left = p.N - visited_tile(p, p.n_row_tiles - 1) * SCAN_BM;
            for (int q = tid; q < p.Q; q += NT) p.cnt[(int64_t)q * CNT_PITCH] = (uint32_t)(rows + (left < SCAN_BM ? left : SCAN_BM));
        }
    }
    if constexpr (KEEP == KEEP_COUNTED)
        for (int c = tid; c < BN; c += NT) tally[c] = 0;
    if (n_mine == 0) return;
    const unsigned char *Xb = static_cast<const unsigned char *>(p.X);
    const unsigned char *Qb = reinterpret_cast<const unsigned char *>(p.Qs);
    const uint32_t ldx2 = (uint32_t)p.ldx * (uint32_t)ESA, dpad2 = (uint32_t)p.dpad * 2u;   // row pitches in bytes
    const int32_t n_rows = (int32_t)p.N;

    if (tid == 0) *pl.count = 0;
    if (lay.tau_n)
        for (int q = tid; q < p.Q; q += NT) tau_lds[q] = p.tau[q];
    RALM_LDS float *aside_scores = (RALM_LDS float *)tally + wave * (lay.aside * (ASIDE_BYTES / 4));
    RALM_LDS int32_t *aside_rows = (RALM_LDS int32_t *)(aside_scores + lay.aside * 16), *aside_queries = aside_rows + lay.aside;
    int n_aside = 0;   // wave-uniform
    auto sort_aside = [&]() __attribute__((always_inline)) {
        // 128 scores at a time, so that one half's LDS reads travel with the other's; a place for all that are admitted by one add
#pragma unroll 1
        for (int base = 0; base < n_aside * 16; base += 128) {
            u64 key[2];
            int query[2];
            bool in[2];
            unsigned long long m[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int i = base + h * 64 + lane, at = i < n_aside * 16 ? i : 0, e = at >> 4, v = at & 15;
                const float score = aside_scores[at];
                const int32_t row = aside_rows[e] + (v >> 2) * 8 + (v & 3);
                query[h] = aside_queries[e];
                key[h] = make_key(score, row);
                in[h] = i < n_aside * 16 && row < n_rows && score == score;
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                in[h] = in[h] && key[h] >= (lay.tau_n ? tau_lds[query[h]] : p.tau[query[h]]);
                m[h] = __builtin_amdgcn_ballot_w64(in[h]);
            }
            const uint32_t n0 = (uint32_t)__builtin_popcountll(m[0]), n = n0 + (uint32_t)__builtin_popcountll(m[1]);
            if (n == 0) continue;   // wave-uniform
            uint32_t first = 0;
            if (lane == 0) first = __hip_atomic_fetch_add(pl.count, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            first = __builtin_amdgcn_readfirstlane(first);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (in[h]) {
                    const uint32_t at = first + (h ? n0 : 0u) + __builtin_amdgcn_mbcnt_hi((uint32_t)(m[h] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m[h], 0u));
                    if (at < pl.cap) {
                        pl.keys[at] = key[h];
                        pl.qs[at] = (uint32_t)query[h];
                    } else {
                        push_global(p, query[h], key[h]);
                    }
                }
            }
        }
        n_aside = 0;
    };
    // one 32x32 block of this wave: out[v] for row row0 + (v/4)*8 + v%4 + 4 (lane/32) and query q0 + lane%32
    auto select_block = [&](const f32x16 &out, int32_t row0, int q0, float tsc) __attribute__((always_inline)) {
        float m = out[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) m = fmaxf(m, out[v]);
        // tsc is -inf where the key admits everything and NaN for padding columns: one compare
        bool cand = m >= tsc;
        unsigned long long mask = __builtin_amdgcn_ballot_w64(cand);
        while (mask) {   // wave-uniform
            const int n = __builtin_popcountll(mask);
            if (n_aside > 0 && n_aside + n > lay.aside) sort_aside();
            uint32_t l = lane;   // (opaque, so that nothing of what follows is kept in registers)
            asm volatile("" : "+v"(l));
            const int at = n_aside + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            const bool mine = cand && at < lay.aside;
            if (mine) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const f32x4 t = {out[c * 4], out[c * 4 + 1], out[c * 4 + 2], out[c * 4 + 3]};
                    *(RALM_LDS f32x4 *)(aside_scores + at * 16 + c * 4) = t;
                }
                aside_rows[at] = row0 + (int32_t)(l >> 5) * 4;
                aside_queries[at] = q0 + (int)(l & 31);
            }
            n_aside = n_aside + n < lay.aside ? n_aside + n : lay.aside;
            cand = cand && !mine;
            mask = __builtin_amdgcn_ballot_w64(cand);
        }
    };

    // ---- issue cursor: runs S-1 stages ahead of the multiply, also across tile boundaries ----
    // per-lane constants of the loads: byte offset (tile row, swizzled chunk) of each wave load
    // inside a strip that lies fully inside the datastore; strips at its edges are clamped instead
    uint32_t a_voff[NA], b_voff[NB];
    auto a_tile_row = [&](int j) __attribute__((always_inline)) { return (uint32_t)((wave * NA + j) * RPI_A + la_r); };
    auto a_tile_chunk = [&](int j) __attribute__((always_inline)) {
        return (uint32_t)((la_c ^ swz<CPR_A>((int)a_tile_row(j) & 15)) << 4);
    };
#pragma unroll
    for (int j = 0; j < NA; ++j) a_voff[j] = __umul24(a_tile_row(j), ldx2) + a_tile_chunk(j);   // row < 2^8, ldx2 < 2^24
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int row = (wave * NB + j) * RPI_B + lb_r;
        b_voff[j] = (uint32_t)row * dpad2 + (uint32_t)((lb_c ^ swz<CPR_B>(row & 15)) << 4);
    }
    // (row tile, query tile) of an item advance by (G / nqt, G % nqt) from one item of this
    // workgroup to its next: no division in the loop
    const int step_rt = G / nqt;
    const int step_qt = G % nqt;
    int is_rt = vb / nqt;
    int is_qt = vb % nqt;
    int is_kt = 0, is_buf = 0;
    // wave-uniform state of the stage being issued
    const unsigned char *is_abase = nullptr, *is_bbase = nullptr, *is_aload = nullptr;
    uint32_t is_rowmax = 0, is_kmax = 0, is_lds = 0;
    bool is_inside = false;   // the strip needs no clamping
    auto issue_begin = [&]() __attribute__((always_inline)) {
        if (is_kt == 0) {
            // The cursor is never stopped: past this workgroup's last tile it fetches (valid)
            // strips that nobody multiplies, so the steady-state loop has no conditionals.
            const int rt = is_rt < n_tiles ? is_rt : 0;
            int64_t row0 = tile_row0(rt);
            int64_t left = p.N - 1 - row0;                  // rows past N re-read row N-1 ...
            if (left < 0) {                                 // ... also a half tile that starts past it
                row0 = p.N - 1;
                left = 0;
            }
            is_abase = Xb + row0 * p.ldx * ESA;
            is_bbase = Qb + (int64_t)is_qt * BN * p.dpad * 2;
            is_rowmax = (uint32_t)(left < BM - 1 ? left : BM - 1);
        }
        // chunks past d re-read the row's last valid one (the query side is zero there): inside a
        // strip by clamping the chunk offset, for a strip that lies past d entirely by stepping
        // the strip's base back to that chunk
        const int kleft = (p.d - 16 / ESA - is_kt * BK) * ESA;   // the row's last chunk, from the strip's start
        is_kmax = (uint32_t)(kleft < 0 ? 0 : (kleft < ROWB_A - 16 ? kleft : ROWB_A - 16));
        is_aload = is_abase + (kleft < 0 ? kleft : 0);
        is_inside = is_rowmax == (uint32_t)(BM - 1) && kleft >= ROWB_A - 16;
        is_lds = lds0 + is_buf * STAGE + wave * (NA * 1024);
    };
    auto issue_part = [&](int idx) __attribute__((always_inline)) {
        if (idx < NA) {
            uint32_t voff = a_voff[idx];
            if (!is_inside) {   // wave-uniform, rare: the datastore's last rows or last columns
                const uint32_t row = a_tile_row(idx), chunk = a_tile_chunk(idx);
                const uint32_t r = row < is_rowmax ? row : is_rowmax;
                const uint32_t c = chunk < is_kmax ? chunk : is_kmax;
                voff = __umul24(r, ldx2) + c;
            }
            dma_1kb<NTA>(is_aload, voff, is_lds + idx * 1024);
        } else {
            const int j = idx - NA;
            dma_1kb<false>(is_bbase, b_voff[j], lds0 + is_buf * STAGE + A_BYTES + (wave * NB + j) * 1024);
        }
    };
    auto issue_end = [&]() __attribute__((always_inline)) {
        is_abase += ROWB_A;
        is_bbase += ROWB_B;
        is_buf = is_buf + 1 == S ? 0 : is_buf + 1;
        if (++is_kt == KT) {
            is_kt = 0;
            is_rt += step_rt;
            is_qt += step_qt;
            if (is_qt >= nqt) {
                is_qt -= nqt;
                ++is_rt;
            }
        }
    };

    for (int st = 0; st < D; ++st) {
        issue_begin();
#pragma unroll
        for (int idx = 0; idx < LPS; ++idx) issue_part(idx);
        issue_end();
    }

    // Operand read offsets of this lane inside a stage (bytes) for k-step 0.  A lane multiplies the
    // 8 elements 16 kk + 8 (lane / 32) .. of its row in k-step kk: one 16-byte chunk of 2-byte
    // elements, chunk slot (2 kk + lane / 32) ^ swz, or the two chunks 4 kk + 2 (lane / 32), + 1 of
    // fp32 rows.  Either way the k-step's offset is the k-step 0 offset with (16 kk elements, in
    // bytes) XOR-ed in: the row part is a multiple of the row size and lies above those bits.
    const int hi = lane >> 5;
    const int a_off0 = (wm * TM * 32 + fr) * ROWB_A + (((A32 ? 2 * hi : hi) ^ swz<CPR_A>(fr & 15)) << 4);
    const int b_off0 = A_BYTES + (wn * TN * 32 + fr) * ROWB_B + ((hi ^ swz<CPR_B>(fr & 15)) << 4);
    static_assert((KS - 1) * 16 * ESA < ROWB_A && (KS - 1) * 32 < ROWB_B && A_BYTES % ROWB_B == 0,
                  "k-step offset stays inside the row");
    uint4 fa[2][TM], fb[2][TN];
    auto read_frag = [&](int slot, const unsigned char *sbase, int kk, int idx) __attribute__((always_inline)) {
        // in the order the MFMAs need them: A0, all of B, then A1..
        if (idx == 0 || idx > TN) {
            const int i = idx == 0 ? 0 : idx - TN;
            const unsigned char *at = sbase + (a_off0 ^ (kk * 16 * ESA)) + i * 32 * ROWB_A;
            if constexpr (A32)
                fa[slot][i] = round8_bf16(*reinterpret_cast<const uint4 *>(at),
                                          *reinterpret_cast<const uint4 *>(sbase + ((a_off0 ^ (kk * 16 * ESA)) ^ 16) +
                                                                           i * 32 * ROWB_A));
            else
                fa[slot][i] = *reinterpret_cast<const uint4 *>(at);
        } else {
            const int j = idx - 1;
            fb[slot][j] = *reinterpret_cast<const uint4 *>(sbase + (b_off0 ^ (kk << 5)) + j * 32 * ROWB_B);
        }
    };

    // stage 0 must be in LDS before the first operand read
    wait_vmcnt<LPS *(D - 1)>();
    __syncthreads();
#pragma unroll
    for (int idx = 0; idx < NR; ++idx) read_frag(0, smem, 0, idx);

    int buf = 0;
    int cur_rt = vb / nqt;
    int cur_qt = vb % nqt;
    for (int it = 0; it < n_mine; ++it) {
        f32x16 acc[TM][TN];
        const int32_t row0 = (int32_t)tile_row0(cur_rt);
        const int q0 = cur_qt * BN;
        // admission keys of this lane's TN queries
        // tsc: the score a value must reach to be looked at more closely; -inf for a key of 0
        // (admit everything; its score bits decode to NaN), NaN (which nothing reaches) for padding columns
        u64 tkey[TN];
        float tsc[TN];
        bool qok[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            const int q = q0 + (wn * TN + j) * 32 + fr;
            qok[j] = q < p.Q;
            tkey[j] = qok[j] ? (lay.tau_n ? tau_lds[q] : p.tau[q]) : ~0ull;
            tsc[j] = qok[j] ? (tkey[j] == 0ull ? -__builtin_inff() : key_score(tkey[j])) : __builtin_nanf("");
        }

        // one stage; FIRST: accumulators start from zero; LAST: selection fused into the last k-step;
        // COLS of the wave's TN column blocks are multiplied
        auto stage = [&](auto first_tag, auto last_tag, auto cols_tag) __attribute__((always_inline)) {
            constexpr int COLS = decltype(cols_tag)::value, NMC = TM * COLS;
            // (counted launches select after the stage, from the accumulators)
            constexpr bool FIRST = decltype(first_tag)::value, LAST = decltype(last_tag)::value && KEEP != KEEP_COUNTED;
            const unsigned char *sb = smem + buf * STAGE;
            const int nbuf = buf + 1 == S ? 0 : buf + 1;
#pragma unroll
            for (int kk = 0; kk < KS; ++kk) {
                // Two waves share a SIMD (and its matrix core): the one further along its stage
                // issues first, so that they take turns in k-step-long runs instead of
                // interleaving instruction by instruction (measured: 2 % faster).
                if constexpr (NW == 8) {
                    if (kk >= 3) __builtin_amdgcn_s_setprio(3);
                    else if (kk == 2) __builtin_amdgcn_s_setprio(2);
                    else if (kk == 1) __builtin_amdgcn_s_setprio(1);
                    else __builtin_amdgcn_s_setprio(0);
                }
                const int cur = kk & 1;
                const bool last_kk = kk + 1 == KS;
                const unsigned char *nsb = last_kk ? smem + nbuf * STAGE : sb;
                const int nkk = last_kk ? 0 : kk + 1;
                // side instructions of this k-step: the operand reads of the next k-step (for the
                // last k-step: of the next stage), then the global->LDS loads (the rendezvous sits
                // inside k-step RK; the query part of the strip is requested after it in that
                // k-step, the datastore part in the next)
                const int nd = kk == RK + 1 ? NA : (kk == RK ? NB : 0);
                const int d0 = kk == RK + 1 ? 0 : NA;
                f32x16 outs[LAG + 1];
                RALM_SCHED_FENCE();
#pragma unroll
                for (int m = 0; m < (NM > LPS + NR ? NM : LPS + NR) + LAG; ++m) {
                    if (m < NMC) {
                        const int i = m / COLS, j = m % COLS;
                        if constexpr (FIRST) {
                            if (kk == 0) {
                                f32x16 zero;
#pragma unroll
                                for (int v = 0; v < 16; ++v) zero[v] = 0.f;
                                acc[i][j] = mfma32<F16>(fa[cur][i], fb[cur][j], zero);
                            } else if (LAST && last_kk) {
                                outs[m % (LAG + 1)] = mfma32<F16>(fa[cur][i], fb[cur][j], acc[i][j]);
                            } else {
                                acc[i][j] = mfma32<F16>(fa[cur][i], fb[cur][j], acc[i][j]);
                            }
                        } else {
                            if (LAST && last_kk)
                                outs[m % (LAG + 1)] = mfma32<F16>(fa[cur][i], fb[cur][j], acc[i][j]);
                            else
                                acc[i][j] = mfma32<F16>(fa[cur][i], fb[cur][j], acc[i][j]);
                        }
                    }
                    if (m < NR)
                        read_frag(cur ^ 1, nsb, nkk, m);
                    else if (m - NR < nd)
                        issue_part(d0 + m - NR);
                    if (kk == RK && m == RV) {
                        // Rendezvous.  After it: the next stage is complete in LDS for every
                        // wave, and every wave has finished reading the slot that the loads
                        // issued from here on refill: the previous stage's (D = S - 1), or this
                        // stage's own (D = S; its last operand reads were issued just above
                        // and are awaited first).  No LDS data is written by ds instructions
                        // that another wave reads without a later full barrier, so no LDS fence
                        // is needed; the asm statements keep the compiler from moving memory
                        // operations across the barrier.
                        wait_vmcnt<LPS *(D - 2)>();
                        if constexpr (D == S) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                        asm volatile("" ::: "memory");
                        __builtin_amdgcn_s_barrier();
                        asm volatile("" ::: "memory");
                        issue_begin();
                    }
                    if (LAST && last_kk && m >= LAG && m - LAG < NMC) {
                        const int mm = m - LAG, i = mm / COLS, j = mm % COLS;
                        if constexpr (KEEP == KEEP_ALL)
                            store_block_all(p, outs[mm % (LAG + 1)], row0 + (wm * TM + i) * 32 + (lane >> 5) * 4,
                                            (int64_t)cur_rt * BM + (wm * TM + i) * 32 + (lane >> 5) * 4,
                                            q0 + (wn * TN + j) * 32 + fr, qok[j]);
                        else if constexpr (KEEP == KEEP_SCORES)
                            store_block_scores(p, outs[mm % (LAG + 1)], row0 + (wm * TM + i) * 32 + (lane >> 5) * 4, n_rows,
                                               (int64_t)cur_rt * BM + (wm * TM + i) * 32 + (lane >> 5) * 4,
                                               q0 + (wn * TN + j) * 32 + fr, qok[j]);
                        else
                            select_block(outs[mm % (LAG + 1)], row0 + (wm * TM + i) * 32, q0 + (wn * TN + j) * 32, tsc[j]);
                    }
                    RALM_SCHED_FENCE();
                }
                if (kk == RK + 1) issue_end();
                RALM_SCHED_FENCE();
            }
            buf = nbuf;
        };

        // A wave whose query columns are all padding (the batch's last query tile is ragged) has
        // nothing to multiply or select: it only keeps its part of the load ring and the
        // rendezvous going, and reads the operands of the next tile's first k-step at the end.
        auto stage_idle = [&]() __attribute__((always_inline)) {
            const int nbuf = buf + 1 == S ? 0 : buf + 1;
            RALM_SCHED_FENCE();
            wait_vmcnt<LPS *(D - 2)>();
            if constexpr (D == S) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // its last reads of the slot
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            issue_begin();
#pragma unroll
            for (int idx = NA; idx < LPS; ++idx) issue_part(idx);   // query part, as in k-step RK
#pragma unroll
            for (int idx = 0; idx < NA; ++idx) issue_part(idx);     // datastore part, as in k-step RK + 1
            issue_end();
#pragma unroll
            for (int idx = 0; idx < NR; ++idx) read_frag(((KS - 1) & 1) ^ 1, smem + nbuf * STAGE, 0, idx);
            RALM_SCHED_FENCE();
            buf = nbuf;
        };
        const bool wave_idle = q0 + wn * TN * 32 >= p.Q;   // wave-uniform

        auto tile = [&](auto cols) __attribute__((always_inline)) {
            if (KT == 1) {
                stage(std::true_type{}, std::true_type{}, cols);
            } else {
                stage(std::true_type{}, std::false_type{}, cols);
                for (int kt = 1; kt + 1 < KT; ++kt) stage(std::false_type{}, std::false_type{}, cols);
                stage(std::false_type{}, std::true_type{}, cols);
            }
        };
        if (wave_idle) {
            for (int kt = 0; kt < KT; ++kt) stage_idle();
        } else if constexpr (TN == 2 && NTA && !A32 && KEEP == KEEP_PARKED) {
            // One query tile of 16-bit rows in whole lines: a wave of whose two column blocks the second is all padding
            // multiplies the first only.  Waves w and w + 4, which hold the same columns, share a SIMD, so this idles that
            // SIMD and the others set the tile's time; what is gained is power, and little.  What comes here are rows of more
            // than 768 elements or less than 257, and middle stages: 200 queries over 2M x 1024 1081 -> 1061 us a call, 224 1129 -> 1113, 200
            // over 1M x 2048 1113 -> 1096, 200 over 4M x 256 657 -> 649, 140 and 170 over 2M x 1024 the same within the noise.
            if (q0 + (wn * TN + 1) * 32 >= p.Q) tile(std::integral_constant<int, 1>{});   // wave-uniform
            else tile(std::integral_constant<int, TN>{});
        } else {
            tile(std::integral_constant<int, TN>{});
        }

        if constexpr (KEEP == KEEP_COUNTED) {
            if (wave_idle) {   // nothing was multiplied: nothing passes
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
            }
            select_tile_counted<TM, TN, NT>(p, acc, tally, row0 + wm * TM * 32 + (lane >> 5) * 4, n_rows, q0, wn * TN * 32 + fr,
                                            BN, tkey, tsc);
        }
        // tile end: every few tiles the parked entries move to the global lists
        if constexpr (KEEP == KEEP_PARKED) {
            const bool last_tile = it + 1 == n_mine, look = last_tile || (it & (lay.flush_every - 1)) == lay.flush_every - 1;
            if (look || n_aside * 2 > lay.aside) sort_aside();
            if (look) {
                __syncthreads();
                const uint32_t n = *pl.count;   // uniform: read after the barrier
                const uint32_t parked = n < pl.cap ? n : pl.cap;
                if (parked >= pl.cap / 4 || (last_tile && parked > 0)) {
                    if (BN <= 128 || p.Q <= 256) flush_parked<NT, true>(p, pl, tally, parked);
                    else flush_parked<NT, false>(p, pl, tally, parked);
                }
            }
        }
        cur_rt += step_rt;
        cur_qt += step_qt;
        if (cur_qt >= nqt) {
            cur_qt -= nqt;
            ++cur_rt;
        }
    }
    wait_vmcnt<0>();   // the run-ahead loads must land before this workgroup's LDS is released
}

template <bool F16, int WM, int WN, int TM, int TN, int BK, int S, bool NTA, int D = S - 1, int RK = 0,
          bool A32 = false, int KEEP = KEEP_PARKED>
hipError_t launch_dma_variant(const ScanParams &p, int n_cu, hipStream_t stream)
{
    constexpr int BM = WM * TM * 32, BN = WN * TN * 32, NW = WM * WN;
    constexpr size_t ring = (size_t)S * (BM * (A32 ? 4 : 2) + BN * 2) * BK;
    constexpr size_t lds = ring <= 64 * 1024 ? 76 * 1024 : 160 * 1024;   // two workgroups to a CU, or one
    ParkLayout lay;
    lay.tau_n = BN <= 128 ? BN : (p.Q <= TAU_LDS_MAX_Q ? (int)((p.Q + 255) / 256 * 256) : 0);
    static_assert(ring + (BN <= 128 ? BN : TAU_LDS_MAX_Q) * 8 + PARK_MIN * 12 + 16 + NW * 2 * ASIDE_BYTES <= lds && NW * 2 * ASIDE_BYTES >= BN * 4,
                  "LDS budget; the counts fit the columns put aside");
    int left = (int)(lds - ring) - lay.tau_n * 8 - PARK_MIN * 12 - 16;
    lay.aside = left / (NW * ASIDE_BYTES) & ~1;   // (even: the lists begin on 16-byte boundaries)
    if (lay.aside > ASIDE_MAX) lay.aside = ASIDE_MAX;
    left -= lay.aside * NW * ASIDE_BYTES;
    lay.park = PARK_MIN + (left / 12 & ~3);
    if (lay.park > PARK_MAX) lay.park = PARK_MAX;
    if (layout_fixed<BN, KEEP>) {
        static_assert(NW * fixed_layout<BN>.aside * ASIDE_BYTES >= BN * 4 && ring + BN * 8 + PARK_MIN * 12 + 16 + NW * fixed_layout<BN>.aside * ASIDE_BYTES <= lds);
        lay = fixed_layout<BN>;
    }
    const size_t smem = ring + (size_t)lay.tau_n * 8 + (size_t)lay.park * 12 + 16 + (size_t)lay.aside * NW * ASIDE_BYTES;
    auto kern = scan_dma_kernel<F16, WM, WN, TM, TN, BK, S, NTA, D, RK, A32, KEEP>;
    static std::atomic<bool> attr_done{false};   // per instantiation; setting it twice is harmless
    if (!attr_done.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        attr_done.store(true, std::memory_order_release);
    }
    const int nqt = (int)((p.Q + BN - 1) / BN);
    const int64_t total = p.n_row_tiles * (SCAN_BM / BM) * nqt;
    if (total <= 0) return hipSuccess;
    if (total > 0x7fffffffLL) return hipErrorInvalidValue;   // the kernel counts items in 32 bits
    // the parked entries are looked at before they are expected to fill a quarter of their places
    const int64_t a_tile = p.admits * (p.Q < BN ? p.Q : BN) * BM / (p.n_row_tiles * SCAN_BM) + 1;
    lay.flush_every = a_tile * 4 <= lay.park ? 4 : (a_tile * 2 <= lay.park ? 2 : 1);
    const int per_cu = lds * 2 <= 160 * 1024 && !p.one_per_cu ? 2 : 1;
    int64_t grid = (int64_t)n_cu * per_cu;
    if (total < grid) grid = total;
    grid = (grid + 7) / 8 * 8;
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(NW * 64), smem, stream, p, nqt, lay);
    return hipGetLastError();
}

// Thresholds that few of a tile's scores pass.
// NTA: one query tile and rows of whole lines.  Nobody shares the rows through L2, they are streamed
// non-temporally (strips of whole 128-byte lines; with 64-byte strips a line would be requested
// twice, a stage apart, and would have to stay in L2 in between).
template <bool F16, bool NTA>
hipError_t launch_dma(const ScanParams &p, int n_cu, hipStream_t stream)
{
    switch (scan_bn_for(p.Q)) {
        // up to 32 queries: half tiles, two workgroups to a CU: a launch of few tiles spreads over twice as many
        // workgroups, and one's selection and flush are covered by the other's loads.  Against whole tiles, one
        // workgroup to a CU: Q = 8 over 1M x 768 271 -> 261 us, over 300K 118 -> 116 us, 1M x 392 216 -> 207 us.
        // With CUs reserved there is one to a CU (Q = 8 over 21M x 768 4606 -> 4782 us): two to each would leave none
        // free, and a lookup of 8 requests issued 1.5 ms into that call took 2.6 ms instead of 0.05
        case 32: return launch_dma_variant<F16, 4, 1, 1, 1, 64, 3, NTA, 3, 2>(p, n_cu, stream);
        // 64 and 128 queries: 8 waves (two per SIMD, wave tiles of 64 x 32 and 128 x 32), so that one wave's
        // waits are covered by the other's multiplies; with 4 waves of twice the width they were 5 % and 3 % slower
        case 64: return launch_dma_variant<F16, 4, 2, 2, 1, 64, 3, NTA, 3, 2>(p, n_cu, stream);
        case 128: return launch_dma_variant<F16, 2, 4, 4, 1, 64, 3, NTA, 3, 2>(p, n_cu, stream);
        // two slots of 64-element strips, refilled in place (D = S): same LDS as four 32-element
        // slots, half the rendezvous and half the L2 requests per multiply
        default: return launch_dma_variant<F16, 2, 4, 4, 2, 64, 2, NTA, 2, 2>(p, n_cu, stream);
    }
}

// launches that keep many or all of their scores (NTA: see launch_dma)
template <bool F16, bool NTA, int KEEP>
hipError_t launch_kept(const ScanParams &p, int n_cu, hipStream_t stream)
{
    switch (scan_bn_for(p.Q)) {
        case 32: return launch_dma_variant<F16, 4, 1, 1, 1, 64, 3, NTA, 3, 2, false, KEEP>(p, n_cu, stream);
        case 64: return launch_dma_variant<F16, 4, 2, 2, 1, 64, 3, NTA, 3, 2, false, KEEP>(p, n_cu, stream);
        case 128: return launch_dma_variant<F16, 2, 4, 4, 1, 64, 3, NTA, 3, 2, false, KEEP>(p, n_cu, stream);
        default: return launch_dma_variant<F16, 2, 4, 4, 2, 64, 2, NTA, 2, 2, false, KEEP>(p, n_cu, stream);
    }
}

// More than 32 queries (whose tiles are halves as it is), and whole tiles would leave half of the CUs idle.
bool few_tiles(const ScanParams &p, int n_cu)
{
    const int bn = scan_bn_for(p.Q);
    return p.Q > 32 && p.n_row_tiles * ((p.Q + bn - 1) / bn) * 2 <= n_cu;
}

// A first stage of few tiles (64 where the lists have 16384 slots) leaves most CUs without one, and a workgroup that has one
// waits for its strips one after the other.  Quarter tiles spread it over four times as many workgroups, with deeper
// rings.  us per launch, 62 whole tiles and 248 quarters of 768 elements: 40 queries 13.2, 9.0; 81 18.2, 12.0; 200 31.8, 17.3; 500 41.7,
// 36.9; 3 queries, which have half tiles anyway, 8.1, 8.4.  Whole calls of one or two stages, whole tiles and quarters: 40 over 300 000 x 16
// 56.2, 54.5, 300 over 300 000 x 64 152, 143, 200 over 5000 x 768 54, 38, 300 over 20 000 x 4096 311, 294, 500 over 20 000 x 8192 576, 561;
// fp32 rows: 40 over 300 000 x 64 65.9, 64.9, 100 over 300 000 x 768 230, 220, 400 over 20 000 x 8192 903, 840.
template <bool F16, int KEEP>
hipError_t launch_quarter(const ScanParams &p, int n_cu, hipStream_t stream)
{
    switch (scan_bn_for(p.Q)) {
        case 64: return launch_dma_variant<F16, 2, 2, 1, 1, 64, 6, false, 6, 2, false, KEEP>(p, n_cu, stream);
        case 128: return launch_dma_variant<F16, 2, 4, 1, 1, 64, 5, false, 5, 2, false, KEEP>(p, n_cu, stream);
        default: return launch_dma_variant<F16, 2, 4, 1, 2, 64, 3, false, 3, 2, false, KEEP>(p, n_cu, stream);
    }
}
template <int KEEP>
hipError_t launch_quarter_f32(const ScanParams &p, int n_cu, hipStream_t stream)
{
    switch (scan_bn_for(p.Q)) {
        case 64: return launch_dma_variant<false, 2, 2, 1, 1, 64, 4, false, 3, 0, true, KEEP>(p, n_cu, stream);
        case 128: return launch_dma_variant<false, 2, 4, 1, 1, 32, 5, false, 5, 0, true, KEEP>(p, n_cu, stream);
        default: return launch_dma_variant<false, 2, 4, 1, 2, 32, 4, false, 4, 0, true, KEEP>(p, n_cu, stream);
    }
}

template <bool F16>
hipError_t launch_16(const ScanParams &p, int route, bool nt, int n_cu, hipStream_t stream)
{
    if (route == RALM_SCAN_ALL_QUARTERS)
        return p.scores_only ? launch_quarter<F16, KEEP_SCORES>(p, n_cu, stream) : launch_quarter<F16, KEEP_ALL>(p, n_cu, stream);
    if (route == RALM_SCAN_ALL)
        return p.scores_only ? launch_kept<F16, false, KEEP_SCORES>(p, n_cu, stream) : launch_kept<F16, false, KEEP_ALL>(p, n_cu, stream);
    if (route == RALM_SCAN_COUNTED)
        return nt ? launch_kept<F16, true, KEEP_COUNTED>(p, n_cu, stream) : launch_kept<F16, false, KEEP_COUNTED>(p, n_cu, stream);
    return nt ? launch_dma<F16, true>(p, n_cu, stream) : launch_dma<F16, false>(p, n_cu, stream);
}

// fp32 rows: batches of one query tile stream them as they are and round on the way to the
// matrix cores (32-element strips for 128 and 256 queries: an fp32 strip row is 128 bytes).
// Several query tiles share the rows through L2 (default cache policy); 11.5 ms per query tile at
// 21M x 768 against 6.5 ms from a bf16 copy, so callers with many tiles are better off with a copy.
template <bool NTA, int KEEP>
hipError_t launch_f32(const ScanParams &p, int n_cu, hipStream_t stream)
{
    switch (scan_bn_for(p.Q)) {
        case 32: return launch_dma_variant<false, 4, 1, 1, 1, 64, 4, NTA, 3, 0, true, KEEP>(p, n_cu, stream);
        case 64: return launch_dma_variant<false, 4, 1, 1, 2, 64, 3, NTA, 3, 2, true, KEEP>(p, n_cu, stream);
        case 128: return launch_dma_variant<false, 2, 4, 4, 1, 32, 3, NTA, 3, 0, true, KEEP>(p, n_cu, stream);
        default: return launch_dma_variant<false, 2, 4, 4, 2, 32, 2, NTA, 2, 0, true, KEEP>(p, n_cu, stream);
    }
}

}  // namespace

constexpr int64_t COUNT_MIN = 8;

int scan_bn_for(int64_t Q)
{
    if (Q <= 32) return 32;
    if (Q <= 64) return 64;
    if (Q <= 128) return 128;
    return 256;
}

// Rows that are whole 128-byte lines.  Otherwise neighbouring strips share the lines that they meet in, and
// a line that was streamed past L2 is fetched again: 100 queries over 2M rows of 904 bf16 elements read
// 1.75 times the rows' bytes and take 1277 us, 994 us (1.08 times) with the default policy; 8 queries over 1M x
// 392: 256 and 216 us.
bool whole_lines(const ScanParams &p)
{
    return (p.ldx * (p.in_dtype == DT_F32 ? 4 : 2)) % 128 == 0 && reinterpret_cast<uintptr_t>(p.X) % 128 == 0;
}

int scan_route(const ScanParams &p, int n_cu)
{
    // every score into empty lists: fixed list positions
    const bool all_kept = p.lists_empty && p.tile_skip == 0 && p.n_row_tiles > 0 && p.n_row_tiles * SCAN_BM <= (int64_t)p.cap;
    if (all_kept) return few_tiles(p, n_cu) ? RALM_SCAN_ALL_QUARTERS : RALM_SCAN_ALL;
    // Thresholds that may admit COUNT_MIN or more of a tile's 256 scores per query: the admitted
    // scores of a tile are counted and stored together, which takes about 20 us a tile of 256 queries whatever their number.  Parked they take
    // time by their number: rounds of 144 neighbour queries over 2M x 1024 (k' = 1024) 1410 us with the line at 2, 1373 at 3, 1370 at
    // 8, 1375 at 16, of 256 over 10M x 1024 (k' = 2048) 6044 at 2, 5988 at 5, and about 90 us more with no counted launches.
    // Rows whose admitted scores come in bursts, whole calls that the line divides, with it at 2 over with it at 8 (mean, and the one that is best
    // at 2): up to 256 queries over stores in corpus order 1.067 (128 calls, 0.999), sorted by cluster 1.044 (118, 0.954: 256 queries, k' =
    // 256, over 1M x 512 417, 437 us), of rows that come 40 to 150 times 1.027 (32, 1.000); more queries in corpus order 1.018 (31, 0.994), sorted by
    // cluster 0.983 (28, 0.939: 2200, k' = 256, over 130 000 x 384 fp32 943, 1004).  200 queries, k' = 128, over 2M x 768 in corpus order 814, 775.
    if (p.admits >= COUNT_MIN * p.n_row_tiles) return RALM_SCAN_COUNTED;
    return scan_held_takes(p, n_cu) ? RALM_SCAN_HELD : RALM_SCAN_PARKED;
}

hipError_t launch_scan(const ScanParams &p, int n_cu, hipStream_t stream)
{
    const int route = scan_route(p, n_cu);
    const bool nt = p.Q <= 256 && whole_lines(p);
    if (route == RALM_SCAN_HELD) return launch_scan_held(p, nt, n_cu, stream);
    if (p.in_dtype == DT_F32) {
        if (route == RALM_SCAN_ALL_QUARTERS)
            return p.scores_only ? launch_quarter_f32<KEEP_SCORES>(p, n_cu, stream) : launch_quarter_f32<KEEP_ALL>(p, n_cu, stream);
        if (route == RALM_SCAN_ALL)
            return p.scores_only ? launch_f32<false, KEEP_SCORES>(p, n_cu, stream) : launch_f32<false, KEEP_ALL>(p, n_cu, stream);
        if (route == RALM_SCAN_COUNTED) return nt ? launch_f32<true, KEEP_COUNTED>(p, n_cu, stream) : launch_f32<false, KEEP_COUNTED>(p, n_cu, stream);
        return nt ? launch_f32<true, KEEP_PARKED>(p, n_cu, stream) : launch_f32<false, KEEP_PARKED>(p, n_cu, stream);
    }
    return p.in_dtype == DT_F16 ? launch_16<true>(p, route, nt, n_cu, stream) : launch_16<false>(p, route, nt, n_cu, stream);
}

}  // namespace ralm
