// The scan with the queries held in registers (gfx950 only); see scan_kernels.hip for what a scan does.
//
// A workgroup of 4 waves, one per SIMD, keeps the queries of one query tile for a whole launch: every wave holds TN blocks of 32
// of them over the full reduction length in its registers (TN = 2, 768 elements: 384 of the 512 that a lane has), and only
// datastore rows move.  They go through a ring of 32-row tiles that takes all of LDS but 16 KB.  The tiled kernel
// streams as many bytes of queries from L2 to LDS as of rows, and reads 6 operands from LDS per 8 multiplies and wave (5 per 4 in
// its tile of 128 queries); here it is no query bytes and 4 operands per 8 multiplies (TN = 2) or per 4 (TN = 1).  In a stream of
// calls the matrix cores are busy 0.77 to 0.78 of the cycles with 256 and 1024 queries, at 1.3 and 1.6 GHz of 2.4: power sets
// the time.  Up to 128 queries wait for the rows (0.54 busy).
//
// us per call, tiled and held behind the same first stage: 200 queries over 6M x 768 2251, 2111; 1024 over 10M x 768 12755, 12102;
// 81 over 1M x 768 318, 298; 140 over 1M x 768 434, 400; 90 over 777001 x 392 in corpus order 257, 183.
#include <atomic>

#include "scan_device.h"

namespace ralm {

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int HELD_BM = 32, HELD_RING_STRIPS = 36;   // rows of a tile; 64-element strips of 32 rows in the ring
constexpr int HELD_PARK = 512;                       // parked admitted scores per workgroup
constexpr int HELD_LIST = 28;                        // blocks' columns that a wave puts aside

// KT: 64-element strips of a row.  NTA: see dma_1kb.
//
// Loads: wave w fetches rows 8 w .. 8 w + 7 of every strip, one 1 KB load each, S - 1 tiles ahead.  A tile's strips are two
// halves.  In the last strip of a half the waves meet: the next half is then complete in LDS for all of them, and the
// half before this one, which everyone has read, may be overwritten.
//
// Multiplies: a lone wave per SIMD has nothing to cover its waits, so operands are read a strip ahead, and a block of
// scores is tested under the multiplies of the next one.  A score is one chain of multiplies in the order of its elements, as in the
// tiled kernel: added by even and odd k-steps, products that cancel in order may overflow to both infinities, and the row is lost.
template <bool F16, int KT, int TN, bool NTA>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1)))
void scan_held_kernel(ScanParams p, const int nqt, const int streams_per_xcd)
{
    constexpr int BN = TN * 128;
    constexpr int S = HELD_RING_STRIPS / KT;                 // tiles in the ring
    constexpr int STRIP = HELD_BM * 128, TILE = KT * STRIP;  // bytes
    constexpr int H = (KT + 1) / 2;                          // strips of a tile's first half
    constexpr int PARTS = SCAN_BM / HELD_BM;
    constexpr int SETS = KT % 2 ? 3 : 2;                     // operand sets: strips take turns, an odd count's first has its own
    constexpr int QREGS = KT * TN * 16;                      // registers that hold the queries
    constexpr int FRAGS_ACC = QREGS <= 128 ? 0 : (QREGS < 256 ? QREGS / 4 : 64);   // operands of these in accumulation registers
    static_assert(TN == 1 || TN == 2, "column blocks of a wave");
    static_assert(KT >= 5 && S >= 2 && (S - 1) * KT < 64 && QREGS <= 384, "ring, registers");

    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t lds0 = (uint32_t)(size_t)(RALM_LDS unsigned char *)smem;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int fr = lane & 31, hi = lane >> 5;
    RALM_LDS u64 *tau_lds = (RALM_LDS u64 *)(smem + HELD_RING_STRIPS * STRIP);
    PushList pl;
    pl.keys = tau_lds + BN;
    pl.qs = (RALM_LDS uint32_t *)(pl.keys + HELD_PARK);
    pl.count = pl.qs + HELD_PARK;
    pl.cap = HELD_PARK;
    RALM_LDS uint32_t *tally = pl.count + 4;   // [128], for the flush of up to 128 queries
    RALM_LDS float *held_scores = (RALM_LDS float *)(tally + (TN == 1 ? 128 : 0)) + wave * (HELD_LIST * 18);
    RALM_LDS int32_t *held_rows = (RALM_LDS int32_t *)(held_scores + HELD_LIST * 16), *held_columns = held_rows + HELD_LIST;

    // workgroup b runs on XCD b % 8; the query tiles of a stream of rows are neighbours on one XCD
    const int idx = (int)(blockIdx.x / 8), slot = idx / nqt, qt = idx % nqt;
    if (slot >= streams_per_xcd) return;
    const int n_streams = streams_per_xcd * 8, stream = slot * 8 + (int)(blockIdx.x % 8);
    const int n_tiles = (int)p.n_row_tiles * PARTS;
    const int n_mine = stream < n_tiles ? (n_tiles - stream + n_streams - 1) / n_streams : 0;
    if (n_mine == 0) return;
    auto tile_row0 = [&](int rt) __attribute__((always_inline)) -> int64_t {
        return visited_tile(p, rt / PARTS) * SCAN_BM + (rt % PARTS) * HELD_BM;
    };
    // from here on the batch is this workgroup's query tile
    {
        const int q0 = qt * BN;
        p.Qs += (int64_t)q0 * p.dpad;
        p.tau += q0;
        p.cand += (int64_t)q0 * p.cap;
        p.cnt += (int64_t)q0 * CNT_PITCH;
        p.Q = p.Q - q0 < BN ? p.Q - q0 : BN;
    }
    const int32_t n_rows = (int32_t)p.N;
    if (tid == 0) *pl.count = 0;
    if (tid < BN) tau_lds[tid] = tid < p.Q ? p.tau[tid] : ~0ull;

    // this wave's queries: elements 64 kt + 16 kk + 8 hi .. + 7 of columns 32 (TN wave + j) + fr
    const int column0 = wave * TN * 32;
    uint4 fb[KT][4][TN];
    {
        const uint16_t *src = p.Qs + (int64_t)(column0 + fr) * p.dpad + hi * 8;
#pragma unroll
        for (int kt = 0; kt < KT; ++kt)
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                    fb[kt][kk][j] = *reinterpret_cast<const uint4 *>(src + (int64_t)j * 32 * p.dpad + kt * 64 + kk * 16);
    }
    // where they are kept is said here: left to itself the compiler copies them to and fro
#pragma unroll
    for (int kt = 0; kt < KT; ++kt)
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int j = 0; j < TN; ++j) {
                u32x4 t = __builtin_bit_cast(u32x4, fb[kt][kk][j]);
                if ((kt * 4 + kk) * TN + j < FRAGS_ACC) asm volatile("" : "+a"(t));
                else asm volatile("" : "+v"(t));
                fb[kt][kk][j] = __builtin_bit_cast(uint4, t);
            }
    __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0): the queries have arrived before the first counted load
    __syncthreads();
    // the score that a value must reach to be looked at more closely; -inf for a key of 0 (admit everything), +inf for padding columns
    float tsc[TN];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
        const int c = column0 + j * 32 + fr;
        const u64 t = tau_lds[c];
        tsc[j] = c < p.Q ? (t == 0ull ? -__builtin_inff() : key_score(t)) : __builtin_inff();
    }

    // ---- load cursor ----
    const unsigned char *Xb = static_cast<const unsigned char *>(p.X);
    const uint32_t ldx2 = (uint32_t)p.ldx * 2u;
    const uint32_t l_row = (uint32_t)(wave * 8 + (lane >> 3));
    const uint32_t l_chunk = (uint32_t)(((lane & 7) ^ swz<8>((int)l_row & 15)) << 4);
    // the last strip may reach past d: chunks there re-read the row's last valid one (the query side is zero there)
    const uint32_t l_kmax = (uint32_t)((p.d - 8 - (KT - 1) * 64) * 2);
    const uint32_t l_chunk_last = l_chunk < l_kmax ? l_chunk : l_kmax;
    int is_rt = stream, is_buf = 0;
    const unsigned char *is_base = nullptr;
    uint32_t is_voff = 0, is_lds = 0;
    auto issue_begin = [&]() __attribute__((always_inline)) {   // next tile of the cursor
        // past this workgroup's last tile the cursor fetches (valid) strips that nobody multiplies
        int64_t row0 = tile_row0(is_rt < n_tiles ? is_rt : 0);
        int64_t left = p.N - 1 - row0;   // rows past N re-read row N - 1, also a tile that starts past it
        if (left < 0) {
            row0 = p.N - 1;
            left = 0;
        }
        is_base = Xb + row0 * p.ldx * 2;
        const uint32_t r = left < HELD_BM - 1 && l_row > (uint32_t)left ? (uint32_t)left : l_row;
        is_voff = __umul24(r, ldx2);     // row < 2^5, ldx2 < 2^24
        is_lds = lds0 + is_buf * TILE + wave * 1024;
        is_buf = is_buf + 1 == S ? 0 : is_buf + 1;
        is_rt += n_streams;
    };
    auto issue = [&](int kt) __attribute__((always_inline)) {
        dma_1kb<NTA>(is_base + kt * 128, is_voff + (kt + 1 == KT ? l_chunk_last : l_chunk), is_lds + kt * STRIP);
    };
    for (int t = 0; t < S - 1; ++t) {
        issue_begin();
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) issue(kt);
    }

    const uint32_t a_off0 = (uint32_t)(fr * 128 + ((hi ^ swz<8>(fr & 15)) << 4));
    uint4 fa[SETS][4];
    auto set_of = [](int kt) constexpr { return KT % 2 && kt == 0 ? 2 : kt & 1; };
    auto read_a = [&](const unsigned char *base, int kt, int kk) __attribute__((always_inline)) {
        fa[set_of(kt)][kk] = *reinterpret_cast<const uint4 *>(base + (a_off0 ^ (kk << 5)) + kt * STRIP);
    };
    auto rendezvous = [&](auto allowed) __attribute__((always_inline)) {   // that many loads are newer than what is needed
        wait_vmcnt<decltype(allowed)::value>();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
    rendezvous(std::integral_constant<int, (S - 1) * KT - H>{});   // the first tile's first half
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) read_a(smem, 0, kk);

    int buf = 0;
    int cur_rt = stream;
    int32_t prev_row0 = 0;
    f32x16 acc[TN];   // one per column block
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[0][v] = acc[TN - 1][v] = 0.f;

    // Columns of a block that may hold an admitted score are put aside as they are, 16 scores and where they belong, in a list
    // of this wave's own: no atomics and no waits between two multiplies.  sort_out() tests the scores later, 64 at a
    // time.  Tested at once, in a stage whose thresholds admit 320 scores per query of 1024 over 4.3M rows, they cost
    // the matrix cores a tenth of their time (5505 us, tiled kernel 5350; with the list 5000 or less).
    int held = 0;   // wave-uniform
    auto sort_out = [&]() __attribute__((always_inline)) {
#pragma unroll 1
        for (int i = lane; i < held * 16; i += 64) {
            const int e = i >> 4, v = i & 15;
            const float score = held_scores[i];
            const int32_t row = held_rows[e] + (v >> 2) * 8 + (v & 3);
            const int c = held_columns[e];
            const u64 key = make_key(score, row);
            if (row < n_rows && score == score && key >= tau_lds[c]) {
                const uint32_t at = __hip_atomic_fetch_add(pl.count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (at < pl.cap) {
                    pl.keys[at] = key;
                    pl.qs[at] = (uint32_t)c;
                } else {
                    push_global(p, c, key);
                }
            }
        }
        held = 0;
    };
    auto select = [&](int j, float m, int32_t row0) __attribute__((always_inline)) {
        bool cand = m >= tsc[j];
        unsigned long long mask = __builtin_amdgcn_ballot_w64(cand);
        while (mask) {   // wave-uniform
            const int n = __builtin_popcountll(mask);
            if (held > 0 && held + n > HELD_LIST) sort_out();
            uint32_t l = lane;   // (opaque, so that nothing of what follows is kept in registers)
            asm volatile("" : "+v"(l));
            const int at = held + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            const bool mine = cand && at < HELD_LIST;
            if (mine) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const f32x4 t = {acc[j][c * 4], acc[j][c * 4 + 1], acc[j][c * 4 + 2], acc[j][c * 4 + 3]};
                    *(RALM_LDS f32x4 *)(held_scores + at * 16 + c * 4) = t;
                }
                held_rows[at] = row0 + (int32_t)(l >> 5) * 4;
                held_columns[at] = column0 + j * 32 + (int)(l & 31);
            }
            held = held + n < HELD_LIST ? held + n : HELD_LIST;
            cand = cand && !mine;
            mask = __builtin_amdgcn_ballot_w64(cand);
        }
    };
    auto flush = [&](uint32_t least) __attribute__((always_inline)) {
        sort_out();
        __syncthreads();
        const uint32_t n = *pl.count;   // uniform: read after the barrier
        if (n >= least) flush_parked<256, TN == 1>(p, pl, tally, n < pl.cap ? n : pl.cap);
    };

#pragma unroll 1
    for (int it = 0; it < n_mine; ++it) {
        const unsigned char *cb = smem + buf * TILE;
        buf = buf + 1 == S ? 0 : buf + 1;
        const unsigned char *nb = smem + buf * TILE;
        const int32_t row0 = (int32_t)tile_row0(cur_rt);
        cur_rt += n_streams;
        issue_begin();
#pragma unroll
        for (int kt = 0; kt < KT; ++kt) {
            // Every 1024 rows the parked entries move on.  No wave parks between this barrier and every wave's read of the
            // count: the next entries come in the last strip, behind the rendezvous of the first half.
            if (kt == 1 && it > 0 && it % (SCAN_BM / HELD_BM * 4) == 0) flush(pl.cap / 4);
            if (kt == H - 1) rendezvous(std::integral_constant<int, (S - 2) * KT + H - 1>{});
            if (kt == KT - 1) rendezvous(std::integral_constant<int, (S - 2) * KT + KT - H - 1>{});
            RALM_SCHED_FENCE();
            // Two column blocks take turns; a tile's first and last strips do one after the other, so that the block that is
            // complete is tested under the other's multiplies.
            const bool grouped = TN == 2 && (kt == 0 || kt == KT - 1);
            float m = 0.f;
#pragma unroll
            for (int i = 0; i < 4 * TN; ++i) {
                const int kk = TN == 1 ? i : (grouped ? i % 4 : i / 2), j = TN == 1 ? 0 : (grouped ? i / 4 : i % 2);
                if (kt == 0 && kk == 0) {
                    f32x16 zero;
#pragma unroll
                    for (int v = 0; v < 16; ++v) zero[v] = 0.f;
                    acc[j] = mfma32<F16>(fa[set_of(kt)][kk], fb[kt][kk][j], zero);
                } else {
                    acc[j] = mfma32<F16>(fa[set_of(kt)][kk], fb[kt][kk][j], acc[j]);
                }
                if (i % TN == 0) {
                    if (kt + 1 < KT) read_a(cb, kt + 1, i / TN);
                    else read_a(nb, 0, i / TN);
                }
                if (i == 2 * TN + 1) issue(kt);
                RALM_SCHED_FENCE();
                if constexpr (TN == 2) {
                    // the first block's last multiply lies two or more back in the last strip, the second's in the next tile's first
                    const int tested = kt == KT - 1 && i >= 5 ? 0 : (kt == 0 && i >= 1 && i <= 3 ? 1 : -1);
                    if (tested >= 0) {
                        const int part = kt == 0 ? i - 1 : i - 5;
                        if (part == 0) m = acc[tested][0];
#pragma unroll
                        for (int v = 5 * part + 1; v <= 5 * part + 5; ++v) m = fmaxf(m, acc[tested][v]);
                        if (part == 2) {
                            if (kt > 0) select(0, m, row0);
                            else if (it > 0) select(1, m, prev_row0);
                        }
                        RALM_SCHED_FENCE();
                    }
                }
            }
        }
        if constexpr (TN == 1) {   // half as many multiplies per row: they wait for the rows, not the rows for them
            float m = -__builtin_inff();
#pragma unroll
            for (int v = 0; v < 16; ++v) m = fmaxf(m, acc[0][v]);
            select(0, m, row0);
        }
        prev_row0 = row0;
    }
    if constexpr (TN == 2) {
        float m = acc[1][0];
#pragma unroll
        for (int v = 1; v < 16; ++v) m = fmaxf(m, acc[1][v]);
        select(1, m, prev_row0);
    }
    flush(1);
    wait_vmcnt<0>();   // the run-ahead loads must land before this workgroup's LDS is released
}

// queries of a tile
int scan_held_bn(const ScanParams &p) { return p.Q <= 128 || p.dpad > 768 ? 128 : 256; }

// Streams of rows per XCD; each takes a workgroup for every query tile.  As many as the CUs hold at once leave CUs idle where
// their number is no multiple of the query tiles (seven tiles on 32 CUs: 4).  So a launch of several query tiles may have more workgroups than
// CUs: the hardware starts the rest as the first ones end, tile by tile of a stream, and what is idle is less than one of
// several rounds.  A round more costs a load of the queries and a ring that fills, 12 us (256 queries over 6M x 768 in 1, 2, 4 and 8 rounds
// 2233, 2246, 2271, 2315 us); a hundredth of the CUs gains 0.4 hundredths of the time, because power sets the clock.  Both in
// tiles of 32 rows: a tile of 256 queries x 768 takes 2.4 us.  Whole calls over 4M x 768, in one round and in the number that this takes:
// 1280 queries 6297, 6269 us (three), 1792 8944, 8628 (two), 2304 11 713, 11 195 (two).  With CUs reserved a second round would
// start on them, so there is one.
int64_t held_streams(const ScanParams &p, int n_cu)
{
    const int64_t bn = scan_held_bn(p), nqt = (p.Q + bn - 1) / bn, per_xcd = n_cu / 8, n_tiles = p.n_row_tiles * (SCAN_BM / HELD_BM);
    int64_t best = per_xcd / nqt;
    if (nqt == 1 || p.one_per_cu) return best;
    int64_t least = 0;
    for (int64_t rounds = 1; rounds <= 16; ++rounds) {
        const int64_t streams = rounds * per_xcd / nqt;
        if (streams < 1) continue;
        const int64_t cost = rounds * (11 + (n_tiles + 8 * streams - 1) / (8 * streams));
        if (least == 0 || cost < least) {
            least = cost;
            best = streams;
        }
    }
    return best;
}

template <bool F16, int KT, int TN, bool NTA>
hipError_t launch_variant(const ScanParams &p, int n_cu, hipStream_t stream)
{
    constexpr size_t smem = (size_t)HELD_RING_STRIPS * HELD_BM * 128 + TN * 128 * 8 + (size_t)HELD_PARK * 12 + 16 +
                            (TN == 1 ? 128 * 4 : 0) + 4 * HELD_LIST * 72;
    static_assert(smem <= 160 * 1024, "LDS budget");
    auto kern = scan_held_kernel<F16, KT, TN, NTA>;
    static std::atomic<bool> attr_done{false};   // per instantiation; setting it twice is harmless
    if (!attr_done.load(std::memory_order_acquire)) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        attr_done.store(true, std::memory_order_release);
    }
    const int nqt = (int)((p.Q + TN * 128 - 1) / (TN * 128));
    const int streams = (int)held_streams(p, n_cu);
    hipLaunchKernelGGL(kern, dim3((unsigned)(8 * nqt * streams)), dim3(256), smem, stream, p, nqt, streams);
    return hipGetLastError();
}

template <bool F16, int KT, int TN>
hipError_t launch_kt(const ScanParams &p, bool nt, int n_cu, hipStream_t stream)
{
    return nt ? launch_variant<F16, KT, TN, true>(p, n_cu, stream) : launch_variant<F16, KT, TN, false>(p, n_cu, stream);
}

template <bool F16>
hipError_t launch_type(const ScanParams &p, bool nt, int n_cu, hipStream_t stream)
{
    if (scan_held_bn(p) == 128) {
        switch (p.dpad / 64) {
#define RALM_HELD(KT) case KT: return launch_kt<F16, KT, 1>(p, nt, n_cu, stream);
            RALM_HELD(5) RALM_HELD(6) RALM_HELD(7) RALM_HELD(8) RALM_HELD(9) RALM_HELD(10) RALM_HELD(11) RALM_HELD(12)
            RALM_HELD(13) RALM_HELD(14) RALM_HELD(15) RALM_HELD(16) RALM_HELD(17)
#undef RALM_HELD
        }
    } else {
        switch (p.dpad / 64) {
#define RALM_HELD(KT) case KT: return launch_kt<F16, KT, 2>(p, nt, n_cu, stream);
            RALM_HELD(5) RALM_HELD(6) RALM_HELD(7) RALM_HELD(8) RALM_HELD(9) RALM_HELD(10) RALM_HELD(11) RALM_HELD(12)
#undef RALM_HELD
        }
    }
    return hipErrorInvalidValue;
}

}  // namespace

// us per call, tiled and held, unless something else is said.
bool scan_held_takes(const ScanParams &p, int n_cu)
{
    if (p.in_dtype == DT_F32) return false;
    // Up to 64 queries the tiled kernel's stream of queries is small and its rows come at the rate of a pure read: 50 over 4M x 768
    // 991, 1036, 64 over 2M x 384 310, 345, x 512 382, 409, x 1024 688, 695 (70 over 4M x 768: 1073, 1010).  Only copies of 1032
    // columns and more for the squared distance would gain: 64 over 2M 759, 728, 8 706, 697.  Rows that are no whole lines it
    // fetches at less: 8 over 1M x 392 in corpus order 197, 169, 4 over 2M x 904 740, 614, 60 over 1M x 600 329, 251, 1 over
    // 1M x 328 167, 148.  With CUs reserved up to 32 queries leave half of a CU's LDS to other kernels, and this one takes all.
    if (p.Q <= 64 && (whole_lines(p) || (p.Q <= 32 && p.one_per_cu))) return false;
    // The queries fit the registers; of rows of more than 768 elements only 128 per workgroup, whose multiplies then read LDS as fast
    // as it gives: 200 over 2M x 1024 1063, 1276, 256 1114, 1203, 512 1955, 2049, but 250 over 1M x 1000 775, 656, 1000 over 1M x
    // 904 2037, 1879.  Rows of less than 257 elements are too few multiplies for a tile's two rendezvous; those of 257 to 512
    // gain: 129 over 1M x 320 237, 226, 256 257, 257, 200 over 2M x 512 579, 551.
    const int kt = p.dpad / 64, bn = scan_held_bn(p);
    if (kt < 5 || kt > 17 || (kt > 12 && p.Q > 128 && whole_lines(p))) return false;
    // Several query tiles: columns and CUs that are left idle cost the tiled kernel less.  Where at most a twentieth of both is idle in one round, or two
    // tiles of 128 queries share the rows (135 over 1M x 904 680, 564), they are held.
    const int64_t nqt = (p.Q + bn - 1) / bn, per_xcd = n_cu / 8, n_tiles = p.n_row_tiles * (SCAN_BM / HELD_BM);
    const int64_t streams = held_streams(p, n_cu);
    if (streams < 1) return false;   // (nearly all CUs reserved, or more query tiles than 16 rounds hold)
    if (nqt > 1 && !(nqt == 2 && bn == 128) && p.Q * (per_xcd / nqt) * 20 < per_xcd * bn * 19) {
        // Otherwise if a quarter of the columns is idle at most.  Queries and both times, each line on one card and in turn:
        // over 4M x 768    300: 2484, 2474   400: 2704, 2656   450: 2864, 2685   550: 3634, 3654   600: 3759, 3713
        //                  700: 3857, 3737   850: 4998, 4880   1100: 6238, 6148   1280: 6448, 6270   1792: 8927, 8628
        // over 1M x 768    400: 780, 746   600: 1058, 1044   768: 1157, 1124   1100: 1726, 1698   1500: 2162, 2099
        // over 500 000 x 768   600: 607, 599   850: 776, 755   1500: 1204, 1196   3000: 2352, 2315
        // Two tiles over rows that are no whole lines at any size: 300 over 1M x 648 755, 657, over 4M x 392 1634, 1515, over 1M x 392 544, 548.
        // More than eight tiles only if a twentieth of the columns is idle at most.  That gives away 2341, whose last tile is nearly empty: 12 290,
        // 12 010 over 4M x 768.
        // over 4M x 768    2304: 11 505, 11 195   4352: 22 991, 21 634   8448: 47 471, 42 647
        // over 1M x 768    2304: 3435, 3378   8192: 12 427, 12 378   16 384: 25 658, 24 325   65 536: 104 091, 96 386   131 072: 208 373, 192 334
        // Beyond 32 tiles an XCD holds only some of a stream's at a time, and the later ones read its rows again: 8448 queries fetch 3.0 times the
        // rows' bytes from HBM (2304 1.18, 1280 1.13, 1024 1.00), the tiled kernel 34 times.
        // Tiles of 128 up to four: 300 over 1M x 1000 1120, 894, 500 over 1M x 904 1117, 1096, but 700 1498, 1549 and 1200 2430, 2530.
        // Below 64 tiles of rows for a workgroup there is little in it: 390 over 300 000 x 768 336, 336, 768 481, 486.
        if (p.one_per_cu || n_tiles < 512 * streams) return false;
        const int64_t columns = nqt * bn;
        if (bn == 128 ? nqt > 4 : (nqt > 8 && p.Q * 20 < columns * 19)) return false;
        if (!(nqt == 2 && !whole_lines(p)) && p.Q * 4 < columns * 3) return false;
        // Of up to 512 elements, which are no whole lines, admitted scores (below) interrupt few multiplies: a tile may admit a score for every six
        // strips.  With all stages that the limit below lets through, and with this one (k' = 64; the last stage of 1M rows admits 1.05 a
        // tile): 600 queries over 1M x 392 743, 754, 734, 1100 1193, 1244, 1193; over 1M x 328 600 669, 707, in tiles, 1100 1078, 1160, in tiles;
        // 1100 over 2M x 328 1873, 1939, 1868; 1500 over 600 000 x 456 1134, 1168, in tiles; 1500 over 4M x 456 5547, 5059, 5057.
        if (nqt > 2 && kt <= 8 && p.admits * bn * 6 > kt * n_tiles) return false;
    }
    // several query tiles share the stream of rows, and short rows are few multiplies between two rendezvous: 1000 queries
    // over 2M x 384 1520, 1567, 512 over 2M x 512 1047, 1042.  Rows that are no whole lines cost the tiled kernel more: 512 over
    // 1M x 560 694, 620
    if (nqt > 1 && kt <= 8 && whole_lines(p)) return false;
    // A workgroup loads 128 TN queries before its first row: at least 8 tiles each.  (On the safe side for rows that are no whole lines:
    // 120 queries over 400 000 x 392, whose middle stage has 7.8 tiles for each, 128, 117.)
    if (n_tiles < 64 * streams) return false;
    // Admitted scores interrupt a lone wave.  p.admits is what the k'-th best of the rows scanned so far would admit: the figures are of launches
    // that scanned with that key.  Stages scan with a better one now and admit about half as many where the rows' order allows it, so the lines are
    // on the safe side.  us per launch by such scores per tile of 32 rows: 26: 120, 159; 18: 61, 72; 10 (81
    // queries): 42, 44; 5.7: 578, 565; 4.7: 476, 516; 3.3 (100 queries): 235, 207; 2.3: 337, 294; 1.6: 1357, 1183; 0.8: 1968, 1870.
    // Rows that are no whole lines, in corpus order: 11 a tile (90 queries over 777001 x 392, the first of two such stages in tiles or
    // not) 244, 214 us a round.  There and in stores sorted by cluster the lines are on the safe side: 200 queries whose middle stage is
    // beyond 16 (29 a tile) and is left in tiles, or not: over 500 000 x 392 248, 194, over 600 000 x 600 292, 253, over 500 000 x
    // 904 364, 314; beyond 4, whole lines sorted by cluster: 200 queries, k' = 256, over 4M x 768 1990, 1468, 100 over 1M x 768 334, 298.
    // In random order (whole calls, the stages beyond 4 a tile in tiles or not): 81 over 1M x 768 (10 a tile) 298, 307, 200 over 200 000 x
    // 768 (27) 141, 153, 100 over 150 000 x 768 (14) 99, 91.
    const int64_t most = whole_lines(p) ? 4 : 16;
    return p.admits * (p.Q < bn ? p.Q : bn) <= most * n_tiles;
}

hipError_t launch_scan_held(const ScanParams &p, bool nt, int n_cu, hipStream_t stream)
{
    return p.in_dtype == DT_F16 ? launch_type<true>(p, nt, n_cu, stream) : launch_type<false>(p, nt, n_cu, stream);
}

}  // namespace ralm
