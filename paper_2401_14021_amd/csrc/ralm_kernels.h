// Launchers of the retrieval kernels (internal to libralm.so).  Every launcher only
// enqueues work on `stream`; argument validation happens in the C-ABI layer.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ralm {

typedef unsigned long long u64;

constexpr int SCAN_BM = 256;       // datastore rows per tile of the stage ladder (a workgroup takes one, or parts of 128, 64 or 32 rows)
constexpr int SCAN_BK = 64;        // reduction elements staged per pipeline step
constexpr int SCAN_QPAD = 256;     // query matrix is zero-padded to a multiple of this
// 32-bit words from one query's list length to the next: a 128-byte line each.  Every admitted score
// moves its query's length by one atomic add, and adds to one line are served one after the
// other (about 3 ns each, wherever they come from); packed lengths put 32 queries on a line, so a
// stage that admits many scores was bound by a handful of lines and not by the scan: 100M-style keys,
// 64 queries, k' = 512, the stage that admits 16.5 K scores per query: 3013 us packed, 895 us padded;
// 256 queries, k' = 2048, 248 tiles that admit 524 K scores: 264 us -> 133 us; 81 queries over 1M x
// 768, the stage behind the first: 72 us -> 43 us.
constexpr int CNT_PITCH = 32;

struct ScanParams {
    const void *X;          // scan copy [N, ldx]
    int64_t ldx;            // elements
    int64_t N;
    int32_t d;              // reduction length: columns of X that are scored (multiple of 8)
    int32_t in_dtype;       // DT_* of X
    const uint16_t *Qs;     // converted queries [Qpad, dpad], zero padded
    int32_t dpad;           // multiple of SCAN_BK
    int32_t Q;
    const u64 *tau;         // [Q] admission keys (0 = admit everything)
    u64 *cand;              // [Q, cap]
    uint32_t *cnt;          // [Q] list lengths, CNT_PITCH words apart
    uint32_t cap;
    int64_t n_row_tiles;    // tiles visited in this stage
    int64_t tile_stride;    // visited tile t is datastore tile (tile_begin + m(t)) * tile_stride, where m(t) = t
    int32_t tile_skip;      // if tile_skip == 0, else the t-th positive integer that is no multiple of tile_skip
    int64_t tile_begin;
    int64_t admits;         // scores that the k'-th best of the rows scanned so far would admit per query: what the thresholds are
                            // expected to admit at most (any number is handled)
    int32_t one_per_cu;     // 1: never more workgroups than the CUs that launch_scan is given
    int32_t lists_empty;    // 1: every list is empty and every score of this launch is kept, so list positions
                            // follow from the row's place in the launch (no atomics)
    int32_t scores_only;    // 1, with lists_empty: the lists are left as launch_select_first reads them
};

// query tile width chosen for Q
int scan_bn_for(int64_t Q);
hipError_t launch_scan(const ScanParams &p, int n_cu, hipStream_t stream);
int scan_route(const ScanParams &p, int n_cu);   // RALM_SCAN_*: the kernel that launch_scan takes for p
// whether a launch whose thresholds admit few scores is better served by the kernel that holds the queries in registers
bool scan_held_takes(const ScanParams &p, int n_cu);
bool whole_lines(const ScanParams &p);   // rows that are whole 128-byte lines
hipError_t launch_scan_held(const ScanParams &p, bool nt, int n_cu, hipStream_t stream);   // nt: rows stream past L2

hipError_t launch_fill_u32(uint32_t *p, uint32_t v, int64_t n, hipStream_t stream);

// fp32 [Q, d] -> scan dtype [Qpad, dpad], zero padded
// also clears the n0 words at z0 (the flag block, but for its number of queries and its mark) and the n1 words at z1
hipError_t launch_query_prep(const float *q, int64_t Q, int32_t d, uint16_t *out, int64_t Qpad,
                             int32_t dpad, int32_t scan_dtype, int32_t metric, uint32_t *z0, int64_t n0,
                             uint32_t *z1, int64_t n1, hipStream_t stream);
hipError_t launch_l2_scan_copy(const void *src, int32_t src_dtype, int64_t src_ld, void *dst, int32_t dst_dtype,
                               int64_t dst_ld, int64_t N, int32_t d, hipStream_t stream);

hipError_t launch_convert_rows(const float *src, int64_t src_ld, void *dst, int32_t dst_dtype,
                               int64_t dst_ld, int64_t N, int32_t d, hipStream_t stream);

// A retrieval call's workspace begins with its flag block (FLAG_BLOCK_BYTES: 32-bit words FLAG_*), one status
// word per query (STATUS_*, padded to a multiple of SCAN_QPAD queries) and, stage by stage of the ladder, the
// length of every query's list when the stage ended.  They are per query, and summed by the calls that report them,
// because one counter for all queries costs 15 ns per query and launch: adds to one address are
// served one after the other (2341 queries: 35 us per select, 70 us per re-score).
constexpr int FLAG_BLOCK_BYTES = 1024, MAX_STAGE_SUMS = 40;
constexpr uint32_t STATUS_SOFT = 1, STATUS_HARD = 2;   // of a query's status word: the check's verdicts
__host__ __device__ inline int64_t padded_queries(int64_t Q) { return (Q + SCAN_QPAD - 1) / SCAN_QPAD * SCAN_QPAD; }
__host__ __device__ inline size_t status_offset() { return FLAG_BLOCK_BYTES; }   // bytes from the flag block
__host__ __device__ inline size_t stage_offset(int64_t Q, int stage)
{
    return FLAG_BLOCK_BYTES + (size_t)padded_queries(Q) * 4 * (1 + stage);
}
enum {
    FLAG_UNANSWERED = 0,        // answered with id -1 / score NaN
    FLAG_LADDER_OVERFLOWS = 1,  // candidate list lost entries during the scan (answered by the exact pass)
    FLAG_FALLBACKS = 2,         // answered by the exact pass
    FLAG_STAGES = 3,            // stages of the ladder whose list lengths were recorded
    FLAG_QUERIES = 4,           // queries of the call
    FLAG_MARK = 5               // FLAG_QUERIES ^ FLAG_MARK_XOR: the block is that of a call
};
constexpr uint32_t FLAG_MARK_XOR = 0x5ca1ab1eu;

// What the re-score needs to check its own result and to queue a query for the exact pass; all
// pointers NULL: no check (flags == NULL decides).
struct CertifyParams {
    int32_t *flags;        // flag block
    uint32_t *lost;        // [Q] != 0: the query's list lost entries during the scan
    int32_t stage;         // of the ladder's last stage
    uint32_t *cnt_rw;      // [Q] list lengths (CNT_PITCH), reset for queued queries
    u64 *tau_exact;        // [Q] in: admission key of the ladder's last stage; out: exact rank-k key of a queued query
    int32_t *fb_list;      // [Q] out: queued queries
    float u_query, u_rows; // unit roundoff applied by the scan to the query / to the rows (0: not rounded)
};

// per query: the list cand[q, 0..cnt[q]) is cut down, in place, to its k' best keys (cnt[q] <- min(cnt[q], k')); the admission key
// tau[q] is raised to one that at least the best tau_rank <= k' of them reach, to the k'-th best itself if tau_rank = k' or if the other would
// lie nearer to the score at rank k than `apart` times that (0: it stays).  A list
// that was sent more than cap keys holds the first cap of them: lost[q] is set and the query
// counted once in flags[FLAG_LADDER_OVERFLOWS].
// The lists' lengths before the cut are recorded behind the flag block if stage < MAX_STAGE_SUMS.
// expected: keys that a list should hold (any number is handled).
hipError_t launch_select(u64 *cand, uint32_t *cnt, uint32_t cap, int32_t k, int32_t k_prime, int32_t tau_rank, float apart, int64_t Q, u64 *tau,
                         uint32_t *lost, int32_t *flags, int32_t stage, int64_t expected,
                         hipStream_t stream);

// The same behind a launch that kept every score as scores (ScanParams::scores_only) of every tile_stride-th tile, for k' = FIRST_KEYS at most
// and at least FIRST_ROWS / 2 rows: the list's area holds FIRST_ROWS scores and the best of every 32 of them.
constexpr int FIRST_ROWS = 16384, FIRST_KEYS = 64;
hipError_t launch_select_first(u64 *cand, uint32_t *cnt, uint32_t cap, int32_t k, int32_t k_prime, int32_t tau_rank, float apart, int64_t tile_stride, int64_t Q, u64 *tau,
                               uint32_t *lost, int32_t *flags, int32_t stage, hipStream_t stream);

// per query: exact scores of the k' best rows of its list, final ranking, top k out;
// with cert.flags: the result is checked and queries that fail are queued for launch_exact_pass
// with cert.flags, cand are the lists as the ladder's last stage left them: more than k' keys are
// cut down to the k' best first and the stage's lengths recorded, as by launch_select
// expected: keys that a list should hold (any number is handled)
hipError_t launch_rescore(const u64 *cand, const uint32_t *cnt, int cnt_pitch, uint32_t cap, int32_t k_prime,
                          const float *queries, int64_t Q, const void *exact, int32_t exact_dtype, int64_t ld,
                          int32_t d, int32_t metric, int32_t k, int32_t *out_ids, float *out_scores,
                          float *out_margin, const CertifyParams &cert, int64_t expected, hipStream_t stream);

constexpr int RESCORE_CUT_MIN = 257;   // k' from which launch_rescore_cut is used
// the same with the check, for lists that launch_select has cut down to their k' best (at least 16384 slots,
// CNT_PITCH); overwrites the slots behind the k' keys
hipError_t launch_rescore_cut(u64 *cand, const uint32_t *cnt, uint32_t cap, int32_t k_prime, const float *queries, int64_t Q,
                              const void *exact, int32_t exact_dtype, int64_t ld, int32_t d, int32_t metric, int32_t k,
                              int32_t *out_ids, float *out_scores, float *out_margin, const CertifyParams &cert,
                              hipStream_t stream);

// exact scan + final ranking for the queries queued by the re-score (two launches that return at
// once when none is queued).  host_mark (may be NULL): device address of a word in pinned host memory that is set to 1 where
// a query stays unanswered
hipError_t launch_exact_pass(const float *queries, int64_t Q, const void *exact, int32_t exact_dtype, int64_t ld,
                             int64_t N, int32_t d, int32_t metric, int32_t k, const int32_t *fb_list, int32_t *flags,
                             const u64 *tau_exact, u64 *cand, uint32_t *cnt, uint32_t cap, int32_t *out_ids,
                             float *out_scores, int32_t *host_mark, int n_cu, hipStream_t stream);

// How a cache lookup is launched (R > 0); scratch: the caller has given merge slots, every_row: see launch_cache_lookup,
// list: the k best
struct LookupRoute {
    int parts;    // workgroups per request; more than one merge
    int pieces;   // 16-byte pieces of a row that a lane has in flight; 0: the rows are read by the vector units
    bool init;    // a launch before the lookup clears the merge slots or answers the queries that no request owns
    bool fill;    // the lookup's first workgroup answers these queries
};
LookupRoute lookup_route(int64_t R, int64_t Qt, int32_t C, int32_t exact_dtype, int32_t metric, int32_t d, bool scratch, bool every_row,
                         bool list);

// every_row: queries that no request owns are answered with id -1 / score -inf
hipError_t launch_cache_lookup(const int32_t *cache_ids, const int32_t *cache_len, int32_t C, int64_t R,
                               const float *queries, int64_t Qt, const int64_t *q_offsets,
                               const void *exact, int32_t exact_dtype, int64_t ld, int64_t N, int32_t d,
                               int32_t metric, int32_t *spec_ids, float *spec_scores, bool every_row, u64 *partial,
                               hipStream_t stream);

constexpr int CACHE_LOOKUP_MAX_D = 2048;   // the lookup kernels hold a row in registers
// whether the k best cached entries are found by launch_cache_keys and launch_rescore instead of the next function
bool cache_topk_by_rescore(int32_t exact_dtype, int32_t metric, int32_t d, int64_t R, int64_t Qt, int32_t C);
// the k best cached entries per query; list [Qt, C] and list_len [Qt] are scratch
hipError_t launch_cache_lookup_topk(const int32_t *cache_ids, const int32_t *cache_len, int32_t C, int64_t R,
                                    const float *queries, int64_t Qt, const int64_t *q_offsets, const void *exact,
                                    int32_t exact_dtype, int64_t ld, int64_t N, int32_t d, int32_t metric, int32_t k,
                                    int32_t *out_ids, float *out_scores, u64 *list, uint32_t *list_len, hipStream_t stream);

constexpr int CACHE_INSERT_MAX_C = 16384;   // a request's cache row is held in LDS during an update
hipError_t launch_cache_insert(int32_t *cache_ids, int32_t *cache_len, int32_t *cache_head, int32_t C, int64_t R,
                               const int32_t *truth, int64_t true_stride, int64_t Qt, const int64_t *q_offsets,
                               const int32_t *first_mismatch, int32_t p, int32_t n_next, int64_t N,
                               hipStream_t stream);
hipError_t launch_knnlm_probs(const int32_t *ids, const float *scores, int64_t Q, int32_t k, const int32_t *values,
                              int64_t N, double T, int32_t *tokens, float *weights, int32_t *top_token,
                              float *top_prob, hipStream_t stream);
// keys[q, 0..cnt[q]) = ranking keys (score 0) of the valid ids cached by the request that owns query q
hipError_t launch_cache_keys(const int32_t *cache_ids, const int32_t *cache_len, int32_t C, int64_t R, int64_t Qt,
                             const int64_t *q_offsets, int64_t N, u64 *keys, uint32_t *cnt, hipStream_t stream);
hipError_t launch_verify(const int32_t *spec, const int32_t *truth, int64_t true_stride, int64_t Qt,
                         const int64_t *q_offsets, int64_t R, int32_t *first_mismatch,
                         hipStream_t stream);

}  // namespace ralm
