// Shared device helpers of the retrieval library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ralm {

typedef unsigned long long u64;

enum { DT_F32 = 0, DT_BF16 = 1, DT_F16 = 2 };
enum { METRIC_IP = 0, METRIC_L2 = 1 };   // inner product; minus the squared Euclidean distance
constexpr int L2_EXTRA_COLS = 8;        // columns behind a scan-copy row that hold its squared norm

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---- ranking keys -----------------------------------------------------------------------
// A candidate (score, row id) is packed into one 64-bit key whose unsigned order is the
// library's ranking: larger key = better = (higher score, then lower id).  -0.0 is folded
// into +0.0 first so that equal floats always give equal score bits.
__device__ __forceinline__ uint32_t score_bits(float s)
{
    s += 0.0f;
    uint32_t u = __float_as_uint(s);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float bits_score(uint32_t b)
{
    uint32_t u = (b & 0x80000000u) ? (b & 0x7fffffffu) : ~b;
    return __uint_as_float(u);
}
__device__ __forceinline__ u64 make_key(float s, int32_t id)
{
    return ((u64)score_bits(s) << 32) | (uint32_t)(0x7fffffff - id);
}
__device__ __forceinline__ int32_t key_id(u64 key) { return 0x7fffffff - (int32_t)(uint32_t)key; }
__device__ __forceinline__ float key_score(u64 key) { return bits_score((uint32_t)(key >> 32)); }

// ---- element conversions ----------------------------------------------------------------
// fp32 -> bf16 bits, round to nearest even (finite inputs).
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}
__device__ __forceinline__ uint32_t f32_to_f16_bits(float f)
{
    _Float16 h = (_Float16)f;   // v_cvt_f16_f32, round to nearest even
    return (uint32_t)__builtin_bit_cast(unsigned short, h);
}
__device__ __forceinline__ float f16_bits_to_f32(uint32_t h)
{
    return (float)__builtin_bit_cast(_Float16, (unsigned short)h);
}
template <int DT>
__device__ __forceinline__ uint32_t f32_to_scan_bits(float f)
{
    return DT == DT_F16 ? f32_to_f16_bits(f) : f32_to_bf16_bits(f);
}
template <int DT>
__device__ __forceinline__ uint4 pack8(const float4 &a, const float4 &b)
{
    uint4 r;
    r.x = f32_to_scan_bits<DT>(a.x) | (f32_to_scan_bits<DT>(a.y) << 16);
    r.y = f32_to_scan_bits<DT>(a.z) | (f32_to_scan_bits<DT>(a.w) << 16);
    r.z = f32_to_scan_bits<DT>(b.x) | (f32_to_scan_bits<DT>(b.y) << 16);
    r.w = f32_to_scan_bits<DT>(b.z) | (f32_to_scan_bits<DT>(b.w) << 16);
    return r;
}

// ---- sums of doubles across lanes ------------------------------------------------------------
// Lane exchanges through DPP and readlane: a shuffle through LDS costs ~100 cycles of latency per
// level, and these sums sit at the end of every exact score.
template <int CTRL>
__device__ __forceinline__ double dpp_mov_f64(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
// sum over the 16 lanes of a row (lanes 16 r .. 16 r + 15); every lane gets its row's sum
__device__ __forceinline__ double row16_sum(double v)
{
    v += dpp_mov_f64<0xB1>(v);    // quad_perm [1,0,3,2]: lane ^ 1
    v += dpp_mov_f64<0x4E>(v);    // quad_perm [2,3,0,1]: lane ^ 2
    v += dpp_mov_f64<0x141>(v);   // row_half_mirror: the other quad of the 8 (quads are uniform by now)
    v += dpp_mov_f64<0x140>(v);   // row_mirror: the other half of the 16
    return v;
}
__device__ __forceinline__ double readlane_f64(double v, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), lane),
                            __builtin_amdgcn_readlane(__double2loint(v), lane));
}
// sum over the 64 lanes of a wave, always in this order; every lane gets it
__device__ __forceinline__ double wave64_sum(double v)
{
    v = row16_sum(v);
    return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}

// ---- bitonic sort of n (a power of two) 64-bit keys in LDS, largest first (DESC) or smallest first ----
// All NT threads of a workgroup; the keys were written before a barrier, and the result is complete
// behind the function's last one.  Steps with a stride of up to 64 exchange keys inside blocks of 128, which a
// wave holds in registers, two keys per lane (lane l: keys l and l + 64 of the block): 56 of the 66 steps of 2048
// keys.  What bounds a step in LDS is its bandwidth (32 bytes per pair of keys and 2-way bank conflicts
// at short strides).  256 workgroups of 1024 threads
// that read 2048 keys, sort them and write 1024: 28 us with all steps in LDS, now 15.6.
template <int S>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v)
{
    static_assert(S == 1 || S == 2 || S == 4 || S == 8 || S == 16 || S == 32, "lane ^ S");
    if constexpr (S == 1) return __builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, false);        // quad_perm [1,0,3,2]
    else if constexpr (S == 2) return __builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, false);   // quad_perm [2,3,0,1]
    else if constexpr (S == 4) return __builtin_amdgcn_ds_swizzle((int)v, 4 << 10 | 0x1f);
    else if constexpr (S == 8) return __builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false);  // row_ror:8
    else if constexpr (S == 16) return __builtin_amdgcn_ds_swizzle((int)v, 16 << 10 | 0x1f);
    else return (uint32_t)__shfl_xor((int)v, 32, 64);
}
// this lane's and lane ^ S's keys: the larger (or the smaller) one
template <int S>
__device__ __forceinline__ u64 exchange(u64 v, bool larger)
{
    const u64 p = (u64)lane_xor<S>((uint32_t)(v >> 32)) << 32 | lane_xor<S>((uint32_t)v);
    return (v > p) == larger ? v : p;
}
// strides S, S / 2, .. 1; desc_a, desc_b: the direction of the blocks that this lane's keys lie in
template <int S>
__device__ __forceinline__ void merge_lanes(u64 &a, u64 &b, bool desc_a, bool desc_b)
{
    const bool low = (threadIdx.x & S) == 0;
    a = exchange<S>(a, low == desc_a);
    b = exchange<S>(b, low == desc_b);
    if constexpr (S > 1) merge_lanes<S / 2>(a, b, desc_a, desc_b);
}
// the same for one key
template <int S>
__device__ __forceinline__ void merge_lane(u64 &a, bool desc)
{
    a = exchange<S>(a, ((threadIdx.x & S) == 0) == desc);
    if constexpr (S > 1) merge_lane<S / 2>(a, desc);
}
// the first n <= SIZE lanes' keys, n a power of two
template <int SIZE, bool DESC>
__device__ __forceinline__ void sort_lane(u64 &a, int n)
{
    if constexpr (SIZE > 2) sort_lane<SIZE / 2, DESC>(a, n);
    if (SIZE <= n) merge_lane<SIZE / 2>(a, ((threadIdx.x & SIZE) == 0) == DESC);   // uniform
}
// block sizes 2, 4, .. SIZE < 64
template <int SIZE, bool DESC>
__device__ __forceinline__ void sort_lanes(u64 &a, u64 &b)
{
    if constexpr (SIZE > 2) sort_lanes<SIZE / 2, DESC>(a, b);
    const bool desc = ((threadIdx.x & SIZE) == 0) == DESC;
    merge_lanes<SIZE / 2>(a, b, desc, desc);
}
// strides 64 .. 1 of a block size of 128 or more
__device__ __forceinline__ void merge_block(u64 &a, u64 &b, bool desc)
{
    const u64 hi = a > b ? a : b, lo = a > b ? b : a;
    a = desc ? hi : lo;
    b = desc ? lo : hi;
    merge_lanes<32>(a, b, desc, desc);
}

template <int NT, bool DESC>
__device__ __forceinline__ void sort_keys(u64 *keys, int n)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (n <= 64) {
        // one key per lane and no more steps than n keys need (as a padded block of 128 the neighbour distributions of
        // 20000 queries x 8 entries took 68 us, in LDS 58, now 54)
        if (wave == 0) {
            u64 a = lane < n ? keys[lane] : 0ull;
            sort_lane<64, DESC>(a, n);
            if (lane < n) keys[lane] = a;
        }
        __syncthreads();
        return;
    }
    for (int base = wave * 128; base < n; base += NT * 2) {
        u64 a = keys[base + lane], b = keys[base + 64 + lane];
        sort_lanes<32, DESC>(a, b);
        merge_lanes<32>(a, b, DESC, !DESC);
        merge_block(a, b, ((base & 128) == 0) == DESC);
        keys[base + lane] = a;
        keys[base + 64 + lane] = b;
    }
    __syncthreads();
    for (int size = 256; size <= n; size <<= 1) {
        for (int stride = size >> 1; stride >= 128; stride >>= 1) {
            for (int t = threadIdx.x; t < n / 2; t += NT) {
                const int lo = 2 * t - (t & (stride - 1));
                const int hi = lo + stride;
                const u64 a = keys[lo], b = keys[hi];
                if ((a < b) == (((lo & size) == 0) == DESC)) {
                    keys[lo] = b;
                    keys[hi] = a;
                }
            }
            __syncthreads();
        }
        for (int base = wave * 128; base < n; base += NT * 2) {
            u64 a = keys[base + lane], b = keys[base + 64 + lane];
            merge_block(a, b, ((base & size) == 0) == DESC);
            keys[base + lane] = a;
            keys[base + 64 + lane] = b;
        }
        __syncthreads();
    }
}

}  // namespace ralm
