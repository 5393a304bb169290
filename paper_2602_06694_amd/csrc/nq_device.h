// Device-side helpers shared by the kernel files of libnq_binlr (not installed): vector types,
// 16-bit float decoding, the fixed-point split of a chunk of activations, tile loads and the
// one-step multiply-accumulate of the streaming kernels (Section 3.1 Eq. 1 evaluated as two
// sign-matrix x vector products; Appendix E.2).
#pragma once
#include <type_traits>
#include "nq_internal.h"

namespace nq {

typedef int v4i __attribute__((ext_vector_type(4)));

__device__ inline float half_bits_to_float(uint16_t h) { return (float)__builtin_bit_cast(_Float16, h); }
__device__ inline float bf16_bits_to_float(uint16_t h) { return __builtin_bit_cast(float, (uint32_t)h << 16); }

__device__ inline float load_as_float(const void* p, int dtype, int64_t idx)
{
    if (dtype == NQ_F32) return ((const float*)p)[idx];
    if (dtype == NQ_F16) return half_bits_to_float(((const uint16_t*)p)[idx]);
    return bf16_bits_to_float(((const uint16_t*)p)[idx]);
}

// v times an fp16 scale, rounded once to fp32.  (Written as a fused operation because that takes the fp16 operand, or both, as it is;
// the zero it adds only turns -0 into +0, which is the same fixed point.)
__device__ __forceinline__ float times_half(float v, uint16_t s) { return __builtin_fmaf(v, half_bits_to_float(s), 0.0f); }

typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) v4u* gptr_v4u;    // global (not generic) address space
typedef const __attribute__((address_space(1))) v4f* gptr_v4f;
typedef const __attribute__((address_space(1))) uint16_t* gptr_u16;

// chunk c (16 consecutive elements) of token row `base` of the vector d describes, times its scale.  Whole chunks of rows that start
// 16-byte aligned (`vec`) are read 16 bytes at a time; with ANY those of all rows, at the alignment of an element, which global memory
// takes (six rows of 3001 fp16 elements: 8.0 -> 6.4 us for their quantisation launch; the kernels that quantise for themselves
// do without: the wider code costs a 1024 x 1024 layer at batch 1 0.24 of its 10.4 us).
template <bool ANY = false>
__device__ inline void load_chunk16(const QuantDesc& d, int64_t base, int c, bool vec, float v[16])
{
    typedef v4f v4f_elem __attribute__((aligned(4)));
    typedef v4u v4u_elem __attribute__((aligned(2)));
    typedef const __attribute__((address_space(1))) v4f_elem* gptr_v4f_elem;
    typedef const __attribute__((address_space(1))) v4u_elem* gptr_v4u_elem;
    typedef typename std::conditional<ANY, gptr_v4f_elem, gptr_v4f>::type gptr_v4f_any;
    typedef typename std::conditional<ANY, gptr_v4u_elem, gptr_v4u>::type gptr_v4u_any;
    const int j0 = c * 16;
    if ((ANY || vec) && j0 + 16 <= d.N) {
        // the scales are requested before the (type-dependent) loads of x, so that both are in flight together
        v4u sraw[2] = {v4u{0, 0, 0, 0}, v4u{0, 0, 0, 0}};
        if (d.scale) {
            const gptr_v4u sp = (gptr_v4u)(d.scale + j0);
            sraw[0] = sp[0];
            sraw[1] = sp[1];
        }
        if (d.dtype == NQ_F32) {
            // (global, not generic, address space: plain vector loads, exact wait counts)
            const gptr_v4f_any p = (gptr_v4f_any)((const float*)d.x + base + j0);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const v4f f = p[q];
                v[4 * q] = f.x; v[4 * q + 1] = f.y; v[4 * q + 2] = f.z; v[4 * q + 3] = f.w;
            }
        } else {
            const gptr_v4u_any p = (gptr_v4u_any)((const uint16_t*)d.x + base + j0);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const v4u u = p[q];
                uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint16_t lo = (uint16_t)(w[i] & 0xFFFFu), hi = (uint16_t)(w[i] >> 16);
                    v[8 * q + 2 * i] = d.dtype == NQ_F16 ? half_bits_to_float(lo) : bf16_bits_to_float(lo);
                    v[8 * q + 2 * i + 1] = d.dtype == NQ_F16 ? half_bits_to_float(hi) : bf16_bits_to_float(hi);
                }
            }
        }
        if (d.scale) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const v4u u = sraw[q];
                uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v[8 * q + 2 * i] = times_half(v[8 * q + 2 * i], (uint16_t)(w[i] & 0xFFFFu));
                    v[8 * q + 2 * i + 1] = times_half(v[8 * q + 2 * i + 1], (uint16_t)(w[i] >> 16));
                }
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int j = j0 + i;
            float f = 0.f;                                  // padding beyond N contributes nothing
            if (j < d.N) {
                f = load_as_float(d.x, d.dtype, base + j);
                if (d.scale) f *= half_bits_to_float(d.scale[j]);
            }
            v[i] = f;
        }
    }
}

// 2^e, -126 <= e <= 127
__device__ __forceinline__ float exp2_int(int e) { return __builtin_bit_cast(float, (e + 127) << 23); }
// exponent of the quantisation step of a token whose largest magnitude has the bits `m` (0 for a token of zeros or with a non-finite value):
// f 2^e with f in [0.5, 1) gives 2^(e - 22), at least the smallest normal number
constexpr uint32_t kMostBits = 0x7f61b1e6u;            // of 3.0e38: larger ones (infinities and NaNs among them) count as not finite
__device__ __forceinline__ int step_exponent(uint32_t m)
{
    const int se = (int)(m >> 23) - 126 - 22;
    return m != 0 && m <= kMostBits ? (se < -126 ? -126 : se) : 0;
}

// byte 0 of a, b, c, d -> one word (a lowest): three byte-permute instructions
__device__ __forceinline__ uint32_t pack_low_bytes(uint32_t a, uint32_t b, uint32_t c, uint32_t d)
{
    const uint32_t ab = __builtin_amdgcn_perm(b, a, 0x0c0c0400u);      // bytes: a.0, b.0, 0, 0
    const uint32_t cd = __builtin_amdgcn_perm(d, c, 0x0c0c0400u);
    return __builtin_amdgcn_perm(cd, ab, 0x05040100u);                 // ab.0, ab.1, cd.0, cd.1
}

// Four values to fixed point: q = rint(v / step), |q| <= 2^22, as q = 65536 hi + 256 mid + lo with signed bytes: the words of the
// four hi, mid and lo bytes.  Returns the sum of the four q.
// Five vector instructions per value instead of eleven: v / step + 1.5 * 2^23 leaves no fraction (one rounding, to nearest even), its bits are
// a constant plus q, and with 0x8080 added their low three bytes are lo + 128, mid + 128 and hi; the 128s go with one exclusive or per
// word.  (A token with a non-finite value gets any bytes: its constants make NaN of whatever they sum up to.)
__device__ __forceinline__ int quantize4(float v0, float v1, float v2, float v3, float inv_step, uint32_t& hi, uint32_t& mid, uint32_t& lo)
{
    constexpr float kRound = 12582912.0f;                              // 1.5 * 2^23, bits 0x4b400000
    constexpr uint32_t kBias = 0x8080u - 0x400000u;
    const uint32_t a = __builtin_bit_cast(uint32_t, __builtin_fmaf(v0, inv_step, kRound)) + kBias;
    const uint32_t b = __builtin_bit_cast(uint32_t, __builtin_fmaf(v1, inv_step, kRound)) + kBias;
    const uint32_t c = __builtin_bit_cast(uint32_t, __builtin_fmaf(v2, inv_step, kRound)) + kBias;
    const uint32_t d = __builtin_bit_cast(uint32_t, __builtin_fmaf(v3, inv_step, kRound)) + kBias;
    const uint32_t ab = __builtin_amdgcn_perm(b, a, 0x05010400u);      // bytes: a.0, b.0, a.1, b.1
    const uint32_t cd = __builtin_amdgcn_perm(d, c, 0x05010400u);
    lo = __builtin_amdgcn_perm(cd, ab, 0x05040100u) ^ 0x80808080u;
    mid = __builtin_amdgcn_perm(cd, ab, 0x07060302u) ^ 0x80808080u;
    hi = __builtin_amdgcn_perm(__builtin_amdgcn_perm(d, c, 0x0c0c0602u), __builtin_amdgcn_perm(b, a, 0x0c0c0602u), 0x05040100u);
    return (int)(a + b + (c + d) - 4u * (0x4b400000u + kBias));        // (modulo 2^32; the sum itself fits)
}

// a chunk of 16 values: its pieces go to dst, slices `slice_pieces` pieces apart; returns the sum of its q
template <bool STREAMED = false>
__device__ inline int quantize_chunk16(const float v[16], float inv_step, uint4* dst, int slice_pieces = 4)
{
    uint32_t hi[4], mid[4], lo[4];
    int sum = 0;                                            // |q| <= 2^22, 16 of them: fits
#pragma unroll
    for (int w = 0; w < 4; ++w) sum += quantize4(v[4 * w], v[4 * w + 1], v[4 * w + 2], v[4 * w + 3], inv_step, hi[w], mid[w], lo[w]);
    // the three slices of a chunk sit 4 pieces apart (see bq_piece): consecutive threads = consecutive
    // chunks of a step fill whole 64-byte lines with each of the three stores
    if (STREAMED) {
        // a buffer in global memory that the next launch reads: written around the cache
        typedef __attribute__((address_space(1))) v4u* gptr_wv4u;
        __builtin_nontemporal_store(v4u{hi[0], hi[1], hi[2], hi[3]}, (gptr_wv4u)dst);
        __builtin_nontemporal_store(v4u{mid[0], mid[1], mid[2], mid[3]}, (gptr_wv4u)dst + slice_pieces);
        __builtin_nontemporal_store(v4u{lo[0], lo[1], lo[2], lo[3]}, (gptr_wv4u)dst + 2 * slice_pieces);
    } else {
        dst[0] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
        dst[slice_pieces] = make_uint4(mid[0], mid[1], mid[2], mid[3]);
        dst[2 * slice_pieces] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
    }
    return sum;
}

// sign tiles are streamed once, never reused: keep them from displacing the (reused) activations
__device__ __forceinline__ v4u load_tile_words(const char* base, uint32_t off)
{
    return __builtin_nontemporal_load((gptr_v4u)(base + off));
}
__device__ __forceinline__ v4u load_global_v4u(const char* base, uint32_t off) { return *(gptr_v4u)(base + off); }

// one 64-column step of a token's quantised vector: [3 slices][4 chunks][16 signed bytes]
constexpr uint32_t kBqStepBytes = 4 * kSlices * 16;

// one 64-column step: eight bit planes, each one AND per register and one MFMA per column group
template <int NB>
__device__ __forceinline__ void mac_tile(v4i (&acc)[NB][8], const v4u w, const v4u (&b)[NB])
{
#pragma unroll
    for (int p = 0; p < 8; ++p) {
        const uint32_t mask = 0x01010101u << p;
        const v4i a = (v4i)(w & mask);
#pragma unroll
        for (int cg = 0; cg < NB; ++cg)
            acc[cg][p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, (v4i)b[cg], acc[cg][p], 0, 0, 0);
    }
}

// Reductions over a wavefront on the data-parallel-primitive path of the vector unit (no LDS traffic):
// quad exchanges, mirrored halves of a 16-lane row, then the four rows through scalar registers.
// The result is the same in every lane.
template <class T, class Op>
__device__ __forceinline__ T wave_reduce32(T v, Op op)
{
    static_assert(sizeof(T) == 4, "32-bit values");
    auto dpp = [](T x, auto ctrl) {
        return __builtin_bit_cast(T, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), decltype(ctrl)::value, 0xf, 0xf, true));
    };
    v = op(v, dpp(v, std::integral_constant<int, 0xB1>{}));      // quad_perm [1, 0, 3, 2]
    v = op(v, dpp(v, std::integral_constant<int, 0x4E>{}));      // quad_perm [2, 3, 0, 1]
    v = op(v, dpp(v, std::integral_constant<int, 0x141>{}));     // row_half_mirror
    v = op(v, dpp(v, std::integral_constant<int, 0x140>{}));     // row_mirror
    const int b = __builtin_bit_cast(int, v);
    const T r0 = __builtin_bit_cast(T, __builtin_amdgcn_readlane(b, 0)), r1 = __builtin_bit_cast(T, __builtin_amdgcn_readlane(b, 16));
    const T r2 = __builtin_bit_cast(T, __builtin_amdgcn_readlane(b, 32)), r3 = __builtin_bit_cast(T, __builtin_amdgcn_readlane(b, 48));
    return op(op(r0, r1), op(r2, r3));
}

// sum of a 64-bit integer over the wavefront (the halves travel separately, the additions are 64-bit)
__device__ __forceinline__ long long wave_sum64(long long v)
{
    auto dpp = [](long long x, auto ctrl) {
        const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned int)(unsigned long long)x, decltype(ctrl)::value, 0xf, 0xf, true);
        const int hi = __builtin_amdgcn_mov_dpp((int)(unsigned int)((unsigned long long)x >> 32), decltype(ctrl)::value, 0xf, 0xf, true);
        return (long long)(((unsigned long long)(unsigned int)hi << 32) | (unsigned int)lo);
    };
    v += dpp(v, std::integral_constant<int, 0xB1>{});
    v += dpp(v, std::integral_constant<int, 0x4E>{});
    v += dpp(v, std::integral_constant<int, 0x141>{});
    v += dpp(v, std::integral_constant<int, 0x140>{});
    long long t = 0;
#pragma unroll
    for (int r = 0; r < 64; r += 16) {
        const unsigned int lo = (unsigned int)__builtin_amdgcn_readlane((int)(unsigned int)(unsigned long long)v, r);
        const unsigned int hi = (unsigned int)__builtin_amdgcn_readlane((int)(unsigned int)((unsigned long long)v >> 32), r);
        t += (long long)(((unsigned long long)hi << 32) | lo);
    }
    return t;
}

}  // namespace nq
