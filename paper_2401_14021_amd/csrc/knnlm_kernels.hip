// KNN-LM neighbour distribution (Section 5.3): from the k retrieved entries of a query to
// weights over their target tokens.
//
//  knnlm_probs_kernel  weight_i = exp(s_i / T) / sum_j exp(s_j / T) over the query's retrieved
//                      entries (s = retrieval score: larger is closer), token_i = values[id_i];
//                      the probability of a token is the sum of the weights of the entries that
//                      carry it; the most probable token (smallest id on ties) is reported.
//                      All of it in double, rounded once to fp32 on output.
#include "../../include/ralm.h"
#include "ralm_common.h"
#include "ralm_kernels.h"

namespace ralm {

namespace {

template <int S>
__device__ __forceinline__ double xor_f64(double x)
{
    return __hiloint2double((int)lane_xor<S>((uint32_t)__double2hiint(x)), (int)lane_xor<S>((uint32_t)__double2loint(x)));
}
// x of all the workgroup's threads joined by f, every thread gets it; red: [NT / 64] in LDS
template <int NT, class F>
__device__ __forceinline__ double block_join(double x, double *red, F f)
{
    x = f(x, xor_f64<32>(x));
    x = f(x, xor_f64<16>(x));
    x = f(x, xor_f64<8>(x));
    x = f(x, xor_f64<4>(x));
    x = f(x, xor_f64<2>(x));
    x = f(x, xor_f64<1>(x));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
    __syncthreads();
    double t = red[0];
    for (int w = 1; w < NT / 64; ++w) t = f(t, red[w]);
    return t;
}

// One workgroup per query, KP_MAX_PER entries per thread at most: what bounds it is the chain of ids, scores and tokens from memory, exp, sort
// and sums, of which a thread with more entries has more in a row, and with many queries how many of their workgroups a CU holds
// (launch_knnlm_probs has the line and the times).
template <int KP_THREADS, int KP_MAX_PER>
__global__ __launch_bounds__(KP_THREADS) void knnlm_probs_kernel(
    const int32_t *__restrict__ ids, const float *__restrict__ scores, int k, int kp2,
    const int32_t *__restrict__ values, int64_t N, double T, int32_t *__restrict__ tokens,
    float *__restrict__ weights, int32_t *__restrict__ top_token, float *__restrict__ top_prob)
{
    extern __shared__ __align__(16) unsigned char smem[];
    double *e = reinterpret_cast<double *>(smem);     // [kp2] weight of the entry at each rank
    u64 *keys = reinterpret_cast<u64 *>(e + kp2);      // [kp2] (token, rank), sorted by token then rank
    constexpr int KP_WAVES = KP_THREADS / 64;
    static_assert((RALM_MAX_K & (RALM_MAX_K - 1)) == 0, "the entries are padded to a power of two");
    __shared__ double red[KP_WAVES];
    __shared__ double s_p[KP_WAVES];
    __shared__ int32_t s_tok[KP_WAVES];

    const int64_t q = blockIdx.x;
    const int tid = threadIdx.x;
    const int32_t *id = ids + q * k;
    const float *sc = scores + q * k;

    double best = -__builtin_inf();
    for (int i = tid; i < k; i += KP_THREADS) {
        const int32_t j = id[i];
        if (j >= 0 && (int64_t)j < N) {
            const double s = (double)sc[i];
            best = s > best ? s : best;
        }
    }
    best = block_join<KP_THREADS>(best, red, [](double a, double b) { return b > a ? b : a; });

    double part = 0.0;
    for (int i = tid; i < kp2; i += KP_THREADS) {
        double x = 0.0;
        u64 key = ~0ull;
        if (i < k) {
            const int32_t j = id[i];
            const bool ok = j >= 0 && (int64_t)j < N;
            int32_t tok = -1;
            if (ok) {
                x = exp(((double)sc[i] - best) / T);
                tok = values[j];
                key = ((u64)((uint32_t)tok ^ 0x80000000u) << 32) | (uint32_t)i;
            }
            tokens[q * k + i] = tok;
        }
        e[i] = x;
        keys[i] = key;
        part += x;
    }
    const double Z = block_join<KP_THREADS>(part, red, [](double a, double b) { return a + b; });
    for (int i = tid; i < k; i += KP_THREADS) {
        const double w = Z > 0.0 ? e[i] / Z : 0.0;
        e[i] = w;
        weights[q * k + i] = (float)w;
    }
    if (!top_token && !top_prob) return;
    __syncthreads();

    // entries grouped by token, ranks ascending inside a group
    sort_keys<KP_THREADS, false>(keys, kp2);
    // weights into the sorted order, so that a group's are neighbours
    double sorted[KP_MAX_PER];
#pragma unroll
    for (int c = 0; c < KP_MAX_PER; ++c) {
        const int i = c * KP_THREADS + tid;
        sorted[c] = i < kp2 && keys[i] != ~0ull ? e[(uint32_t)keys[i]] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < KP_MAX_PER; ++c)
        if (c * KP_THREADS + tid < kp2) e[c * KP_THREADS + tid] = sorted[c];
    __syncthreads();
    // the thread at the start of a group adds the group's weights in rank order, four entries' reads at a
    // time (one after the other, a token with many entries was a chain of as many LDS round trips)
    double my_p = -1.0;
    int32_t my_tok = -1;
    for (int i = tid; i < kp2; i += KP_THREADS) {
        const u64 key = keys[i];
        if (key == ~0ull) continue;
        const uint32_t t32 = (uint32_t)(key >> 32);
        if (i > 0 && (uint32_t)(keys[i - 1] >> 32) == t32) continue;
        double p = 0.0;
        bool more = true;
        for (int j = i; more && j < kp2; j += 4) {
            u64 kj[4];
            double ej[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int at = j + u < kp2 ? j + u : kp2 - 1;
                kj[u] = keys[at];
                ej[u] = e[at];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                more = more && j + u < kp2 && (uint32_t)(kj[u] >> 32) == t32 && kj[u] != ~0ull;
                p = more ? p + ej[u] : p;
            }
        }
        const int32_t tok = (int32_t)(t32 ^ 0x80000000u);
        if (p > my_p || (p == my_p && tok < my_tok)) {
            my_p = p;
            my_tok = tok;
        }
    }
    auto better = [&](double p2, int32_t t2) __attribute__((always_inline)) {
        if (p2 > my_p || (p2 == my_p && p2 >= 0.0 && t2 < my_tok)) {
            my_p = p2;
            my_tok = t2;
        }
    };
    better(xor_f64<32>(my_p), (int32_t)lane_xor<32>((uint32_t)my_tok));
    better(xor_f64<16>(my_p), (int32_t)lane_xor<16>((uint32_t)my_tok));
    better(xor_f64<8>(my_p), (int32_t)lane_xor<8>((uint32_t)my_tok));
    better(xor_f64<4>(my_p), (int32_t)lane_xor<4>((uint32_t)my_tok));
    better(xor_f64<2>(my_p), (int32_t)lane_xor<2>((uint32_t)my_tok));
    better(xor_f64<1>(my_p), (int32_t)lane_xor<1>((uint32_t)my_tok));
    if ((tid & 63) == 0) {
        s_p[tid >> 6] = my_p;
        s_tok[tid >> 6] = my_tok;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < KP_WAVES; ++w) better(s_p[w], s_tok[w]);
        const bool any = my_p >= 0.0;
        if (top_token) top_token[q] = any ? my_tok : -1;
        if (top_prob) top_prob[q] = any ? (float)my_p : 0.f;
    }
}

}  // namespace

hipError_t launch_knnlm_probs(const int32_t *ids, const float *scores, int64_t Q, int32_t k, const int32_t *values,
                              int64_t N, double T, int32_t *tokens, float *weights, int32_t *top_token,
                              float *top_prob, hipStream_t stream)
{
    if (Q <= 0) return hipSuccess;
    int kp2 = 2;
    while (kp2 < k) kp2 <<= 1;
    const size_t smem = (size_t)kp2 * 16;
    // More than 512 entries: with 512 threads four workgroups fit a CU, with 256 eight.  1024 entries each, us a call with 256, 512 and 1024
    // threads: 128 queries 16.3, 13.3, 13.3; 256 17.4, 13.3, 14.0; 512 20.7, 17.5, 25.5; 1024 28.0, 28.6, 48.0; 1025 29.7, 31.9, 57.2;
    // 2048 44.8, 47.2, 92.6; 4000 71, 84, 181.
    constexpr int64_t KP_FEW_QUERIES = 1024;
    static_assert(RALM_MAX_K <= 1024, "entries per thread");
    if (kp2 <= 512)
        hipLaunchKernelGGL((knnlm_probs_kernel<256, 2>), dim3((unsigned)Q), dim3(256), smem, stream, ids, scores, k, kp2,
                           values, N, T, tokens, weights, top_token, top_prob);
    else if (Q <= KP_FEW_QUERIES)
        hipLaunchKernelGGL((knnlm_probs_kernel<512, 2>), dim3((unsigned)Q), dim3(512), smem, stream, ids, scores, k, kp2,
                           values, N, T, tokens, weights, top_token, top_prob);
    else
        hipLaunchKernelGGL((knnlm_probs_kernel<256, 4>), dim3((unsigned)Q), dim3(256), smem, stream, ids, scores, k, kp2,
                           values, N, T, tokens, weights, top_token, top_prob);
    return hipGetLastError();
}

}  // namespace ralm
