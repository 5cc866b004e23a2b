// kb_gen.hip -- seeded input generator for gfx950.
//
// Element g of stream (seed, stream_id, sub) is word g mod 4 of Philox4x32-10
// block g / 4 (key = seed, counter = (lo32(b), hi32(b), sub, stream_id)),
// mapped to a uniform value by u = (x >> 8) 2^-24 and fmaf(u, p1 - p0, p0), or
// to a normal value by the Box-Muller transform evaluated in binary64 over the
// word pair of g's half-block.
//
// gen_kernel           one thread computes one Philox block and stores its (up
//                      to) four elements; interior blocks of an offset that is
//                      a multiple of 4 store with one 16-byte (fp32/u32) or
//                      8-byte (fp16/bf16) write;
// gen_normal16_kernel  4 million and more 16-bit normals: a binary32 first
//                      pass on a persistent grid, binary64 where it is not
//                      sure (the same bits);
// t3_kernel            one thread per Student-t value (a block each);
// perturb_kernel       planted changes, 16 bytes per thread.
// The work is bound by instruction issue (ten 32x32->64 multiply rounds per
// block, plus the logarithm, root, sine and cosine per normal pair).
#include <algorithm>

#include "kb_device.hpp"
#include "kb_internal.hpp"
#include "kb_math.hpp"

namespace kb {
namespace {

__device__ __forceinline__ float u01(uint32_t x) { return (float)(x >> 8) * 0x1p-24f; }

// The device's seeds for the binary64 functions (v_rcp_f64 and v_rsq_f64 are
// good to about 2^-24).
struct DeviceSeed {
    static __device__ __forceinline__ double rcp(double x) { return __builtin_amdgcn_rcp(x); }
    static __device__ __forceinline__ double rsq(double x) { return __builtin_amdgcn_rsq(x); }
    static __device__ __forceinline__ double frexp_mant(double x) { return __builtin_amdgcn_frexp_mant(x); }
    static __device__ __forceinline__ int frexp_exp(double x) { return __builtin_amdgcn_frexp_exp(x); }
    static __device__ __forceinline__ double ldexp(double x, int n) { return __builtin_ldexp(x, n); }
    // saturating (2^32 gives 2^32 - 1), which a C++ conversion does not promise
    static __device__ __forceinline__ uint32_t to_u32(float x) {
        uint32_t u;
        asm("v_cvt_u32_f32 %0, %1" : "=v"(u) : "v"(x));
        return u;
    }
    static __device__ __forceinline__ float log2(float x) { return __builtin_amdgcn_logf(x); }
    static __device__ __forceinline__ float sqrt32(float x) { return __builtin_amdgcn_sqrtf(x); }
};

// Box-Muller on one word pair, each branch rounded once to binary32.
__device__ __forceinline__ void box_muller(uint32_t xa, uint32_t xb, float& zc, float& zs) {
    double c, s;
    box_muller64<DeviceSeed>(xa, xb, c, s);
    zc = (float)c;
    zs = (float)s;
}

// binary32 -> binary16 storage as its own rounding.  The value is made
// opaque first: otherwise the compiler may fuse the multiply-add that
// produced it with the conversion into one mixed-precision instruction that
// rounds once, straight to binary16, where the definition rounds to binary32
// and then to binary16 (the two differ when the binary32 result lands on a
// binary16 tie).
__device__ __forceinline__ uint16_t to_f16_bits(float v) {
    asm volatile("" : "+v"(v));
    return f32_to_f16_bits(v);
}

template <int DT>
__device__ __forceinline__ void store_one(void* dst, uint64_t j, float v, uint32_t word) {
    if constexpr (DT == DT_U32) ((uint32_t*)dst)[j] = word;
    else if constexpr (DT == DT_F32) ((float*)dst)[j] = v;
    else if constexpr (DT == DT_F16) ((uint16_t*)dst)[j] = to_f16_bits(v);
    else ((uint16_t*)dst)[j] = f32_to_bf16_bits(v);
}

template <int DT>
__device__ __forceinline__ void store_four(void* dst, uint64_t j, const float v[4], u32x4 w) {
    if constexpr (DT == DT_U32) {
        *(uint4*)((uint32_t*)dst + j) = make_uint4(w.x, w.y, w.z, w.w);
    } else if constexpr (DT == DT_F32) {
        *(float4*)((float*)dst + j) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
        uint32_t h[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
            h[i] = DT == DT_F16 ? to_f16_bits(v[i]) : f32_to_bf16_bits(v[i]);
        *(uint2*)((uint16_t*)dst + j) = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
    }
}

template <int DIST, int DT>
__global__ __launch_bounds__(256) void gen_kernel(void* __restrict__ dst, uint64_t n, float p0,
                                                  float p1, uint32_t k0, uint32_t k1,
                                                  uint32_t stream_id, uint32_t sub,
                                                  uint64_t offset, uint64_t b_first,
                                                  uint64_t n_blocks) {
    const float width = p1 - p0;  // binary32, one rounding
    const uint64_t end = offset + n;
    const uint64_t n_whole = (offset & 3u) == 0 ? n >> 2 : 0;
    const uint64_t step = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n_blocks; t += step) {
        const uint64_t b = b_first + t;
        const u32x4 w = philox4x32_10({(uint32_t)b, (uint32_t)(b >> 32), sub, stream_id}, k0, k1);
        float v[4] = {0.f, 0.f, 0.f, 0.f};
        if constexpr (DIST == KB_DIST_UNIFORM) {
            v[0] = fmaf(u01(w.x), width, p0);
            v[1] = fmaf(u01(w.y), width, p0);
            v[2] = fmaf(u01(w.z), width, p0);
            v[3] = fmaf(u01(w.w), width, p0);
        } else if constexpr (DIST == KB_DIST_NORMAL) {
            float z[4];
            box_muller(w.x, w.y, z[0], z[1]);
            box_muller(w.z, w.w, z[2], z[3]);
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = fmaf(z[i], p1, p0);
        }
        // (offset a multiple of 4: block t is the output's elements 4 t ..
        // 4 t + 3, all of them inside for t < n / 4)
        if (t < n_whole) {
            store_four<DT>(dst, 4 * t, v, w);
        } else {
            const uint64_t g0 = 4 * b;
            const uint32_t words[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint64_t g = g0 + i;
                if (g >= offset && g < end) store_one<DT>(dst, g - offset, v[i], words[i]);
            }
        }
    }
}

// Normals stored in 16 bits.  The values are defined by the binary64 transform
// rounded to binary32, scaled, and rounded again to 16 bits; only about one in
// 600 fp16 values (one in eight times as many of bf16) lies close enough to a
// rounding boundary for more than 20 bits of the normal to matter, 2.5 in 100
// blocks of four at the worst shift (p0 = -p1).  So each normal is first formed
// in binary32 (rho32 and sincos32: the binary32 steps issue no faster than
// binary64's here, but a pair takes 40 of them instead of 75) as an interval.
// The errors are relative -- rho 2^-22.2 at most, the sine or cosine 2^-22.3,
// their product 2^-24, 7.7 units of 2^-24 in all -- so the definition's normal
// lies between z (1 - e) and z (1 + e), e = 1.25 * 2^-21 (10 units), and since
// its rounding to binary32, the scaling and the last rounding are monotone, an
// interval whose two ends are stored as the same bits stores the value's bits.
// A block with any other interval is put on the work-group's list and computed
// by the binary64 path after the loop, when the list fills whole waves: the
// outputs are the same bits as without the first pass.  Bound by instruction
// issue: 3 x 33.5 million fp16 values 157 -> 105 us.
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// Two binary32 values (no NaN) rounded to storage, packed.
template <int DT>
__device__ __forceinline__ uint32_t pack16(float a, float b) {
    asm volatile("" : "+v"(a), "+v"(b));  // (see to_f16_bits)
    if constexpr (DT == DT_F16) return __builtin_bit_cast(uint32_t, f16x2{(_Float16)a, (_Float16)b});
    else return __builtin_bit_cast(uint32_t, bf16x2{(__bf16)a, (__bf16)b});
}

// The stored bits of a word pair's two normals, and whether they are sure.
template <int DT>
__device__ __forceinline__ uint32_t normal_pair16(uint32_t xa, uint32_t xb, float p0, float p1, bool& sure) {
    constexpr float kLow = 1.0f - 0x1.4p-21f, kHigh = 1.0f + 0x1.4p-21f;
    bool sure_rho, sure_angle;
    const float rho = rho32<DeviceSeed>(xa, sure_rho);
    float sn, cs;
    sincos32(xb, sn, cs, sure_angle);
    const float zc = rho * cs, zs = rho * sn;
    const uint32_t lo = pack16<DT>(fmaf(zc * kLow, p1, p0), fmaf(zs * kLow, p1, p0));
    const uint32_t hi = pack16<DT>(fmaf(zc * kHigh, p1, p0), fmaf(zs * kHigh, p1, p0));
    sure = sure_rho && sure_angle && lo == hi;
    return lo;
}

// Block t of the output by the binary64 path.
template <int DT>
__device__ void normal_block64(void* dst, uint64_t n, float p0, float p1, uint32_t k0, uint32_t k1, uint32_t stream_id,
                               uint32_t sub, uint64_t b_first, uint64_t t) {
    const uint64_t b = b_first + t;
    const u32x4 w = philox4x32_10({(uint32_t)b, (uint32_t)(b >> 32), sub, stream_id}, k0, k1);
    float z[4], v[4];
    box_muller(w.x, w.y, z[0], z[1]);
    box_muller(w.z, w.w, z[2], z[3]);
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = fmaf(z[i], p1, p0);
    if (t < n >> 2) {
        store_four<DT>(dst, 4 * t, v, w);
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (4 * t + i < n) store_one<DT>(dst, 4 * t + i, v[i], 0u);
    }
}

// Launched from 2^20 blocks (4 million values) on: below that a thread of the
// persistent grid (8 work-groups per CU) has one block at most, and the list's
// pass over a few entries costs what the first pass saves (us, without -> with
// the first pass: 2^21 fp16 values 6.6 -> 7.4, 2^22 10.7 -> 9.9, 2^23 19.1 ->
// 14.8, 2^25 59.2 -> 38.7).
constexpr uint64_t kNormal16Blocks = 1u << 20;
constexpr uint64_t kNormal16Grid = 2048;
constexpr uint32_t kRedo = 1024;  // blocks a work-group's list holds

// The offset is a multiple of 4 (blocks and groups of four outputs coincide).
template <int DT>
__global__ __launch_bounds__(256) void gen_normal16_kernel(void* __restrict__ dst, uint64_t n, float p0, float p1,
                                                           uint32_t k0, uint32_t k1, uint32_t stream_id, uint32_t sub,
                                                           uint64_t b_first) {
    __shared__ uint64_t s_redo[kRedo];
    __shared__ uint32_t s_count;
    if (threadIdx.x == 0) s_count = 0u;
    __syncthreads();
    const uint64_t n_blocks = (n + 3) >> 2, n_whole = n >> 2;
    const uint64_t step = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n_blocks; t += step) {
        const uint64_t b = b_first + t;
        const u32x4 w = philox4x32_10({(uint32_t)b, (uint32_t)(b >> 32), sub, stream_id}, k0, k1);
        bool sure0, sure1;
        const uint32_t h0 = normal_pair16<DT>(w.x, w.y, p0, p1, sure0);
        const uint32_t h1 = normal_pair16<DT>(w.z, w.w, p0, p1, sure1);
        if (sure0 && sure1 && t < n_whole) {
            ((uint2*)dst)[t] = make_uint2(h0, h1);
        } else {
            const uint32_t i = atomicAdd(&s_count, 1u);
            if (i < kRedo) s_redo[i] = t;
            else normal_block64<DT>(dst, n, p0, p1, k0, k1, stream_id, sub, b_first, t);  // (list full)
        }
    }
    __syncthreads();
    const uint32_t count = min(s_count, kRedo);
    for (uint32_t i = threadIdx.x; i < count; i += blockDim.x)
        normal_block64<DT>(dst, n, p0, p1, k0, k1, stream_id, sub, b_first, s_redo[i]);
}

template <int DIST, int DT>
hipError_t launch_typed(void* dst, uint64_t n, float p0, float p1, uint64_t seed,
                        uint32_t stream_id, uint32_t sub, uint64_t offset, hipStream_t stream) {
    const uint64_t b_first = offset / 4;
    const uint64_t b_last = (offset + n - 1) / 4;
    const uint64_t n_blocks = b_last - b_first + 1;
    const uint64_t want = (n_blocks + 255) / 256;
    if constexpr (DIST == KB_DIST_NORMAL && DT != DT_F32) {
        if ((offset & 3u) == 0 && n_blocks >= kNormal16Blocks) {
            // up to 256 blocks a thread, so that the list (about one block in
            // 150 of fp16, fewer of bf16) stays well under its length; at the
            // worst shift it can fill, and its last blocks are computed in
            // place
            const uint64_t grid16 = std::max<uint64_t>(kNormal16Grid, (want + 255) / 256);
            hipLaunchKernelGGL((gen_normal16_kernel<DT>), dim3((unsigned)std::min(want, grid16)), dim3(256), 0, stream,
                               dst, n, p0, p1, (uint32_t)seed, (uint32_t)(seed >> 32), stream_id, sub, b_first);
            return hipGetLastError();
        }
    }
    const unsigned grid = (unsigned)(want < 16384 ? want : 16384);
    hipLaunchKernelGGL((gen_kernel<DIST, DT>), dim3(grid), dim3(256), 0, stream, dst, n, p0, p1,
                       (uint32_t)seed, (uint32_t)(seed >> 32), stream_id, sub, offset, b_first,
                       n_blocks);
    return hipGetLastError();
}

// Student-t with 3 degrees of freedom of one block's words, rounded once to
// binary32.
__device__ __forceinline__ float student_t3(u32x4 w) { return (float)student_t3_64<DeviceSeed>(w.x, w.y, w.z); }

// The storage bits of an arithmetic result rounded to the storage type
// (nearest even); a NaN result is stored as the type's positive quiet NaN,
// whatever NaN the operation produced (its sign and payload are the
// platform's choice).
template <int DT>
__device__ __forceinline__ uint32_t value_bits(float v) {
    const bool nan = __builtin_isnan(v);
    if constexpr (DT == DT_F32) return nan ? 0x7FC00000u : __float_as_uint(v);
    else if constexpr (DT == DT_F16) return nan ? 0x7E00u : to_f16_bits(v);
    else return nan ? 0x7FC0u : f32_to_bf16_bits(v);
}

// The exact binary32 widening of storage bits (kept a separate instruction,
// so the arithmetic after it is plain binary32 arithmetic).
template <int DT>
__device__ __forceinline__ float widen_value(uint32_t bits) {
    float x;
    if constexpr (DT == DT_F32) x = __uint_as_float(bits);
    else if constexpr (DT == DT_F16) x = f16_bits_to_f32(bits);
    else x = bf16_bits_to_f32(bits);
    asm volatile("" : "+v"(x));
    return x;
}

template <int DT>
__device__ __forceinline__ uint32_t load_bits(const void* src, uint64_t j) {
    if constexpr (DT == DT_F32) return ((const uint32_t*)src)[j];
    else return ((const uint16_t*)src)[j];
}

template <int DT>
__device__ __forceinline__ void store_bits(void* dst, uint64_t j, uint32_t bits) {
    if constexpr (DT == DT_F32) ((uint32_t*)dst)[j] = bits;
    else ((uint16_t*)dst)[j] = (uint16_t)bits;
}

// One thread per element: element g = offset + j is the Student-t of block g.
template <int DT>
__global__ __launch_bounds__(256) void t3_kernel(void* __restrict__ dst, uint64_t n, float p0, float p1,
                                                 uint32_t k0, uint32_t k1, uint32_t stream_id, uint32_t sub,
                                                 uint64_t offset) {
    const uint64_t step = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += step) {
        const uint64_t b = offset + j;
        const u32x4 w = philox4x32_10({(uint32_t)b, (uint32_t)(b >> 32), sub, stream_id}, k0, k1);
        store_bits<DT>(dst, j, value_bits<DT>(fmaf(student_t3(w), p1, p0)));
    }
}

unsigned elementwise_grid(uint64_t n) {
    const uint64_t want = (n + 255) / 256;
    return (unsigned)(want < 16384 ? want : 16384);
}

template <int DT>
hipError_t launch_t3(void* dst, uint64_t n, float p0, float p1, uint64_t seed, uint32_t stream_id,
                     uint32_t sub, uint64_t offset, hipStream_t stream) {
    hipLaunchKernelGGL((t3_kernel<DT>), dim3(elementwise_grid(n)), dim3(256), 0, stream, dst, n, p0, p1,
                       (uint32_t)seed, (uint32_t)(seed >> 32), stream_id, sub, offset);
    return hipGetLastError();
}

// ------------------------------------------------------------ softmax rows --
// One work-group per row (grid-striding over rows): the logits (the NORMAL
// stream, mean 0, standard deviation sigma) go to dst first, then the row's
// maximum, the binary64 sum of exp(x - max) and the quotients.  The sum is a
// fixed tree (each thread's elements in order, then 64-lane DPP sums, then
// the four waves in order), so it is the same bits on every call.
__device__ __forceinline__ float wave_max_float(float v) {
    v = fmaxf(v, __uint_as_float(dpp_u32<DPP_QUAD_XOR1>(__float_as_uint(v))));
    v = fmaxf(v, __uint_as_float(dpp_u32<DPP_QUAD_XOR2>(__float_as_uint(v))));
    v = fmaxf(v, __uint_as_float(dpp_u32<DPP_ROW_HALF_MIRROR>(__float_as_uint(v))));
    v = fmaxf(v, __uint_as_float(dpp_u32<DPP_ROW_MIRROR>(__float_as_uint(v))));
    const float a = fmaxf(__uint_as_float(readlane_u32(__float_as_uint(v), 0)),
                          __uint_as_float(readlane_u32(__float_as_uint(v), 16)));
    const float b = fmaxf(__uint_as_float(readlane_u32(__float_as_uint(v), 32)),
                          __uint_as_float(readlane_u32(__float_as_uint(v), 48)));
    return fmaxf(a, b);
}

__global__ __launch_bounds__(256) void softmax_rows_kernel(float* __restrict__ dst, uint64_t rows, uint64_t cols,
                                                           float sigma, uint32_t k0, uint32_t k1,
                                                           uint32_t stream_id, uint32_t sub) {
    __shared__ float s_max[4];
    __shared__ double s_sum[4];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (uint64_t row = blockIdx.x; row < rows; row += gridDim.x) {
        float* x = dst + row * cols;
        float m = -__builtin_inff();
        for (uint64_t j = threadIdx.x; j < cols; j += 256) {
            const uint64_t g = row * cols + j;
            const uint64_t b = g >> 2;
            const u32x4 w = philox4x32_10({(uint32_t)b, (uint32_t)(b >> 32), sub, stream_id}, k0, k1);
            const uint32_t k = (uint32_t)(g & 3u);
            float zc, zs;
            if (k < 2) box_muller(w.x, w.y, zc, zs);
            else box_muller(w.z, w.w, zc, zs);
            const float v = fmaf(k & 1u ? zs : zc, sigma, 0.0f);
            x[j] = v;
            m = fmaxf(m, v);
        }
        m = wave_max_float(m);
        if (lane == 0) s_max[wave] = m;
        __syncthreads();
        m = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
        double s = 0.0;
        for (uint64_t j = threadIdx.x; j < cols; j += 256) s += exp((double)x[j] - (double)m);
        s = wave_sum_f64(s);
        if (lane == 0) s_sum[wave] = s;
        __syncthreads();
        s = ((s_sum[0] + s_sum[1]) + s_sum[2]) + s_sum[3];
        for (uint64_t j = threadIdx.x; j < cols; j += 256) x[j] = (float)(exp((double)x[j] - (double)m) / s);
        __syncthreads();  // s_max / s_sum are reused by the next row
    }
}

// -------------------------------------------------------------- index draws --
// One wave: each round its 64 lanes draw blocks j0 .. j0 + 63 at once, then
// the draws are taken in order, each checked by all lanes against the
// indices accepted so far (in LDS) and appended if new.
__global__ __launch_bounds__(64) void indices_kernel(uint64_t* __restrict__ dst, uint32_t m, uint64_t n,
                                                     uint32_t k0, uint32_t k1, uint32_t stream_id, uint32_t sub) {
    __shared__ uint64_t s_idx[KB_MAX_INDICES];
    const uint32_t lane = threadIdx.x;
    uint32_t have = 0;
    // (at most 2^20 draws: with 2 m <= n each draw is new with probability
    // >= 1/2, so this bound only guarantees the loop ends)
    for (uint64_t j0 = 0; have < m && j0 < (1u << 20); j0 += 64) {
        const uint64_t b = j0 + lane;
        const u32x4 w = philox4x32_10({(uint32_t)b, (uint32_t)(b >> 32), sub, stream_id}, k0, k1);
        const uint64_t mine = (((uint64_t)w.y << 32) | w.x) % n;
        for (int l = 0; l < 64 && have < m; ++l) {
            const uint64_t x = readlane_u64(mine, l);
            bool seen = false;
            for (uint32_t i = lane; i < have; i += 64) seen |= s_idx[i] == x;
            if (__builtin_amdgcn_ballot_w64(seen) == 0) {
                if (lane == 0) s_idx[have] = x;
                ++have;
                __syncthreads();  // the new entry is visible to every lane's next scan
            }
        }
    }
    for (uint32_t i = lane; i < m; i += 64) dst[i] = i < have ? s_idx[i] : ~0ull;
}

// --------------------------------------------------------- planted changes --
// Ops 1-5 read word g mod 4 of block g / 4, ops 6-7 the whole block g
// (binary32 only).  In place (dst == src) is allowed: an element is read and
// written by one thread.
//
// A thread takes kVec consecutive elements (16 bytes; one memory access each
// way where all of them lie inside), and for ops 1-5 a Philox block and its
// normals serve the four elements they hold.  One thread per element
// computed every block four times and every Box-Muller pair twice.  Measured,
// per element before: last-bit flips with planted infinities in 20 fp16
// tensors of 12 million 748 -> 363 us; 262,144 fp32 plus normal noise 4.8 ->
// 2.7 us; the block-per-element ops, whose 16 multiplies stay, 38 -> 30 us for
// 16.8 million.

// The changed storage bits of one element; u: its word, z: its normal (op 3).
template <int DT, int OP>
__device__ __forceinline__ uint32_t perturb_word(uint32_t bits, uint32_t u, float z, float a, float b, float p) {
    if constexpr (OP == KB_PERTURB_ADD_UNIFORM) {
        return value_bits<DT>(widen_value<DT>(bits) + fmaf(u01(u), b - a, a));
    } else if constexpr (OP == KB_PERTURB_REL_UNIFORM) {
        const float x = widen_value<DT>(bits);
        return value_bits<DT>(fmaf(x, fmaf(u01(u), b - a, a), x));
    } else if constexpr (OP == KB_PERTURB_ADD_NORMAL) {
        return value_bits<DT>(widen_value<DT>(bits) + fmaf(z, a, 0.0f));
    } else if constexpr (OP == KB_PERTURB_SCALE_WHERE) {
        return u01(u) < p ? value_bits<DT>(widen_value<DT>(bits) * a) : bits;
    } else {
        return u01(u) < p ? bits ^ 1u : bits;
    }
}

// The same for the ops that take a whole block w.
template <int OP>
__device__ __forceinline__ uint32_t perturb_block(uint32_t bits, u32x4 w, float a, float b, float p) {
    const float v = u01(w.x);
    uint32_t out = bits;
    if constexpr (OP == KB_PERTURB_SPECIALS) {
        const uint32_t sign = w.y & 0x80000000u;
        if (v < a) out = sign | (w.z & 0x7FFFFFu) | 1u;  // a subnormal of that sign
        else if (v < b) out = sign;                     // a zero
        else if (v < p) out = sign | 0x7F800000u;       // an infinity
    } else {  // KB_PERTURB_ZERO_SUBNORMAL_REL
        const uint32_t mag = bits & 0x7FFFFFFFu;
        if (v < p) {
            if (mag == 0u) out = bits ^ 0x80000000u;               // flip the zero's sign
            else if (mag < 0x00800000u) out = bits & 0x80000000u;  // flush the subnormal
            else if (mag < 0x7F800000u) {                          // a finite normal value
                const float x = __uint_as_float(bits);
                out = __float_as_uint(fmaf(x, fmaf(u01(w.y), b - a, a), x));
            }
        }
    }
    return out;
}

template <int DT>
constexpr int kVec = DT == DT_F32 ? 4 : 8;  // elements of 16 bytes

// The changed bits of elements g0 .. g0 + V - 1 (g0 a multiple of 4 for ops
// 1-5), in place.
template <int DT, int OP, int V>
__device__ __forceinline__ void perturb_vec(uint32_t e[V], uint64_t g0, float a, float b, float p, uint32_t k0,
                                            uint32_t k1, uint32_t stream_id, uint32_t sub) {
    if constexpr (OP <= KB_PERTURB_FLIP_LSB_WHERE) {
#pragma unroll
        for (int q = 0; q < V; q += 4) {
            const uint64_t blk = (g0 + q) >> 2;
            const u32x4 w = philox4x32_10({(uint32_t)blk, (uint32_t)(blk >> 32), sub, stream_id}, k0, k1);
            const uint32_t u[4] = {w.x, w.y, w.z, w.w};
            float z[4] = {0.f, 0.f, 0.f, 0.f};
            if constexpr (OP == KB_PERTURB_ADD_NORMAL) {
                box_muller(w.x, w.y, z[0], z[1]);
                box_muller(w.z, w.w, z[2], z[3]);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) e[q + i] = perturb_word<DT, OP>(e[q + i], u[i], z[i], a, b, p);
        }
    } else {
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const uint64_t g = g0 + i;
            e[i] = perturb_block<OP>(
                e[i], philox4x32_10({(uint32_t)g, (uint32_t)(g >> 32), sub, stream_id}, k0, k1), a, b, p);
        }
    }
}

// Thread t takes elements V t - lead .. of the stream's range, where lead puts
// g on a multiple of 4 (ops 1-5, an offset that is none: the memory accesses
// are then single elements); elements outside [0, n) are skipped.  V: 16
// bytes, but 4 elements where lead is not zero: eight 16-bit elements read
// and written one by one are the longer chain (4099 fp16 scaled 4.1 us, 2.9
// with one thread per element, 3.0 now; 16.8 million of them at an offset of 1 33 us, 41, 22 now).
template <int DT, int OP, int V>
__global__ __launch_bounds__(256) void perturb_kernel(void* dst, const void* src, uint64_t n, float a, float b,
                                                      float p, uint32_t k0, uint32_t k1, uint32_t stream_id,
                                                      uint32_t sub, uint64_t offset, uint32_t lead,
                                                      uint64_t n_items) {
    const uint64_t n_whole = V == kVec<DT> && lead == 0u ? n / V : 0;
    const uint64_t step = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n_items; t += step) {
        const uint64_t j0 = t * V - lead;  // (wraps below zero for t = 0, lead > 0)
        uint32_t e[V];
        if (V == kVec<DT> && t < n_whole) {
            const uint4 x = ((const uint4*)src)[t];
            const uint32_t q[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
            for (int i = 0; i < V; ++i)
                e[i] = DT == DT_F32 ? q[i % 4] : (q[i / 2 % 4] >> (16 * (i & 1))) & 0xFFFFu;
            perturb_vec<DT, OP, V>(e, offset + j0, a, b, p, k0, k1, stream_id, sub);
            uint4 y;
            if constexpr (DT == DT_F32) y = make_uint4(e[0], e[1], e[2], e[3]);
            else y = make_uint4(e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[V - 4] | (e[V - 3] << 16), e[V - 2] | (e[V - 1] << 16));
            ((uint4*)dst)[t] = y;
        } else {
#pragma unroll
            for (int i = 0; i < V; ++i) e[i] = j0 + i < n ? load_bits<DT>(src, j0 + i) : 0u;
            perturb_vec<DT, OP, V>(e, offset + j0, a, b, p, k0, k1, stream_id, sub);
#pragma unroll
            for (int i = 0; i < V; ++i)
                if (j0 + i < n) store_bits<DT>(dst, j0 + i, e[i]);
        }
    }
}

template <int DT, int OP>
hipError_t launch_perturb_op(void* dst, const void* src, uint64_t n, float a, float b, float p, uint64_t seed,
                             uint32_t stream_id, uint32_t sub, uint64_t offset, hipStream_t stream) {
    const uint32_t lead = OP <= KB_PERTURB_FLIP_LSB_WHERE ? (uint32_t)(offset & 3u) : 0u;
    const auto launch = [&](auto kernel, uint64_t V) {
        const uint64_t n_items = n / V + (n % V + lead + V - 1) / V;
        hipLaunchKernelGGL(kernel, dim3(elementwise_grid(n_items)), dim3(256), 0, stream, dst, src, n, a, b, p,
                           (uint32_t)seed, (uint32_t)(seed >> 32), stream_id, sub, offset, lead, n_items);
    };
    if (lead == 0u || kVec<DT> == 4) launch(perturb_kernel<DT, OP, kVec<DT>>, kVec<DT>);
    else launch(perturb_kernel<DT, OP, 4>, 4);
    return hipGetLastError();
}

template <int DT>
hipError_t launch_perturb_dt(void* dst, const void* src, uint64_t n, int op, float a, float b, float p,
                             uint64_t seed, uint32_t stream_id, uint32_t sub, uint64_t offset, hipStream_t stream) {
    switch (op) {
        case KB_PERTURB_ADD_UNIFORM:
            return launch_perturb_op<DT, KB_PERTURB_ADD_UNIFORM>(dst, src, n, a, b, p, seed, stream_id, sub, offset, stream);
        case KB_PERTURB_REL_UNIFORM:
            return launch_perturb_op<DT, KB_PERTURB_REL_UNIFORM>(dst, src, n, a, b, p, seed, stream_id, sub, offset, stream);
        case KB_PERTURB_ADD_NORMAL:
            return launch_perturb_op<DT, KB_PERTURB_ADD_NORMAL>(dst, src, n, a, b, p, seed, stream_id, sub, offset, stream);
        case KB_PERTURB_SCALE_WHERE:
            return launch_perturb_op<DT, KB_PERTURB_SCALE_WHERE>(dst, src, n, a, b, p, seed, stream_id, sub, offset, stream);
        default:
            return launch_perturb_op<DT, KB_PERTURB_FLIP_LSB_WHERE>(dst, src, n, a, b, p, seed, stream_id, sub, offset, stream);
    }
}

// ------------------------------------------------------------------ scatter --
template <int DT>
__global__ __launch_bounds__(256) void scatter_kernel(void* dst, const void* ref, uint64_t n,
                                                      const uint64_t* __restrict__ idx, uint32_t m, int mode) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < m; i += gridDim.x * blockDim.x) {
        const uint64_t k = idx[i];
        if (k >= n) continue;
        if constexpr (DT == DT_F32) {
            const uint32_t sign = ((const uint32_t*)ref)[k] & 0x80000000u;
            ((uint32_t*)dst)[k] = mode == KB_SCATTER_NAN ? 0x7FC00000u : (sign | 0x7F800000u);
        } else {
            const uint16_t sign = (uint16_t)(((const uint16_t*)ref)[k] & 0x8000u);
            const uint16_t nan = DT == DT_F16 ? 0x7E00u : 0x7FC0u, inf = DT == DT_F16 ? 0x7C00u : 0x7F80u;
            ((uint16_t*)dst)[k] = mode == KB_SCATTER_NAN ? nan : (uint16_t)(sign | inf);
        }
    }
}

}  // namespace

hipError_t launch_gen_t3(void* dst, int dtype, uint64_t n, float p0, float p1, uint64_t seed,
                         uint32_t stream_id, uint32_t sub, uint64_t offset, hipStream_t stream) {
    switch (dtype) {
        case DT_F32: return launch_t3<DT_F32>(dst, n, p0, p1, seed, stream_id, sub, offset, stream);
        case DT_F16: return launch_t3<DT_F16>(dst, n, p0, p1, seed, stream_id, sub, offset, stream);
        default: return launch_t3<DT_BF16>(dst, n, p0, p1, seed, stream_id, sub, offset, stream);
    }
}

hipError_t launch_softmax_rows(float* dst, uint64_t rows, uint64_t cols, float sigma, uint64_t seed,
                               uint32_t stream_id, uint32_t sub, hipStream_t stream) {
    const unsigned grid = (unsigned)(rows < 65536 ? rows : 65536);
    hipLaunchKernelGGL(softmax_rows_kernel, dim3(grid), dim3(256), 0, stream, dst, rows, cols, sigma,
                       (uint32_t)seed, (uint32_t)(seed >> 32), stream_id, sub);
    return hipGetLastError();
}

hipError_t launch_indices(uint64_t* dst, uint32_t m, uint64_t n, uint64_t seed, uint32_t stream_id, uint32_t sub,
                          hipStream_t stream) {
    hipLaunchKernelGGL(indices_kernel, dim3(1), dim3(64), 0, stream, dst, m, n, (uint32_t)seed,
                       (uint32_t)(seed >> 32), stream_id, sub);
    return hipGetLastError();
}

hipError_t launch_perturb(void* dst, const void* src, int dtype, uint64_t n, int op, float a, float b, float p,
                          uint64_t seed, uint32_t stream_id, uint32_t sub, uint64_t offset, hipStream_t stream) {
    if (op == KB_PERTURB_SPECIALS)
        return launch_perturb_op<DT_F32, KB_PERTURB_SPECIALS>(dst, src, n, a, b, p, seed, stream_id, sub, offset, stream);
    if (op == KB_PERTURB_ZERO_SUBNORMAL_REL)
        return launch_perturb_op<DT_F32, KB_PERTURB_ZERO_SUBNORMAL_REL>(dst, src, n, a, b, p, seed, stream_id, sub,
                                                                       offset, stream);
    switch (dtype) {
        case DT_F32: return launch_perturb_dt<DT_F32>(dst, src, n, op, a, b, p, seed, stream_id, sub, offset, stream);
        case DT_F16: return launch_perturb_dt<DT_F16>(dst, src, n, op, a, b, p, seed, stream_id, sub, offset, stream);
        default: return launch_perturb_dt<DT_BF16>(dst, src, n, op, a, b, p, seed, stream_id, sub, offset, stream);
    }
}

hipError_t launch_scatter(void* dst, const void* ref, int dtype, uint64_t n, const uint64_t* idx, uint32_t m,
                          int mode, hipStream_t stream) {
    const unsigned grid = (unsigned)((m + 255) / 256);
    switch (dtype) {
        case DT_F32:
            hipLaunchKernelGGL(scatter_kernel<DT_F32>, dim3(grid), dim3(256), 0, stream, dst, ref, n, idx, m, mode);
            break;
        case DT_F16:
            hipLaunchKernelGGL(scatter_kernel<DT_F16>, dim3(grid), dim3(256), 0, stream, dst, ref, n, idx, m, mode);
            break;
        default:
            hipLaunchKernelGGL(scatter_kernel<DT_BF16>, dim3(grid), dim3(256), 0, stream, dst, ref, n, idx, m, mode);
    }
    return hipGetLastError();
}

hipError_t launch_gen(void* dst, int dtype, uint64_t n, int dist, float p0, float p1,
                      uint64_t seed, uint32_t stream_id, uint32_t sub, uint64_t offset,
                      hipStream_t stream) {
    if (dist == KB_DIST_U32)
        return launch_typed<KB_DIST_U32, DT_U32>(dst, n, p0, p1, seed, stream_id, sub, offset, stream);
    if (dist == KB_DIST_UNIFORM) {
        switch (dtype) {
            case DT_F32: return launch_typed<KB_DIST_UNIFORM, DT_F32>(dst, n, p0, p1, seed, stream_id, sub, offset, stream);
            case DT_F16: return launch_typed<KB_DIST_UNIFORM, DT_F16>(dst, n, p0, p1, seed, stream_id, sub, offset, stream);
            default: return launch_typed<KB_DIST_UNIFORM, DT_BF16>(dst, n, p0, p1, seed, stream_id, sub, offset, stream);
        }
    }
    switch (dtype) {
        case DT_F32: return launch_typed<KB_DIST_NORMAL, DT_F32>(dst, n, p0, p1, seed, stream_id, sub, offset, stream);
        case DT_F16: return launch_typed<KB_DIST_NORMAL, DT_F16>(dst, n, p0, p1, seed, stream_id, sub, offset, stream);
        default: return launch_typed<KB_DIST_NORMAL, DT_BF16>(dst, n, p0, p1, seed, stream_id, sub, offset, stream);
    }
}

}  // namespace kb
