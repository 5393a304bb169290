// Dense (prefill, batch >= 9) path of  y = s_out (.) (U (V^T (s_in (.) x)))   (Section 3.1 Eq. 1;
// Appendix E.3, "Binary GEMM Inference"): both contractions run on the fp16 matrix cores of gfx950.
//
//   pre   : x'' = s_in (.) x * 2^a_b                  per token b, 2^a_b puts max|x''| in [2^12, 2^13), clamped for max|x'| >= 2^113
//   gemm1 : T   = (X'' V) * g                         g = power of two so that |T| <= 2^14 for all data short of the clamp
//   gemm2 : y   = (T U^T) (.) s_out / (2^a_b * g)     fp32 accumulation throughout
//
// A product with signs, two columns at a time, on the SPARSE matrix instruction.  For signs s1, s2 of a pair of columns
//
//   s1 x1 + s2 x2 = s1 * (x1 + x2)  where s1 = s2,   s1 * (x1 - x2)  where they differ,
//
// so with the operand holding the sum AND the difference of every pair (rounded to fp16, as x'' itself would be: the same
// relative rounding on half as many terms of twice the square, hence the same error: over the layers and batches timed, 2.9 to
// 3.6e-4 of the result's norm in fp32 either way), a row of signs has exactly one nonzero, +-1, per pair -- two in any four operand positions, which is what v_smfmac_f32_16x16x64_f16 takes: 64 columns in the 16
// cycles in which the dense instruction does 32.  Nothing is pruned: the products left out are with exact zeros.
//
// The sign matrices stay in the 1-bit tile layout of the streaming kernels.  A wave owns 128 output rows (one tile row
// block) and builds the operand of each 16-row plane in registers: the signs s1 shifted to the sign bits of +-1.0 (two vector
// instructions per four weights), the positions from s1 xor s2 gathered once per tile (about 22 instructions for all eight
// planes).  2.8 vector instructions per matrix instruction at 64 tokens a tile, and they are what bounds the loop: the two share
// a SIMD's issue, each vector instruction costs about 2.5 of the matrix core's cycles (a loop of random operands sustains 4.15
// PFLOP/s without, 2.3 with them; the clock falls to 2.0 .. 2.2 GHz under it).  Signs from memory and activations go straight
// to LDS, without registers in between.
// Measured (MI355X, bf16 in and out, whole forwards), dense instruction -> this: 8192 x 28672 r = 3520 at 2048 tokens
// 390 -> 302 us; 28672 x 8192 at 512 tokens 116 -> 91 us; the first layer's two GEMMs on average 285 + 81 -> 207 + 65 us.
// Not taken: 128-token tiles at one wave per SIMD (half the vector instructions per matrix instruction, no second wave to
// hide the rest: level); 8-bit sparse operands in two slices (half the vector instructions, but the fixed point that outlier
// tokens then get is coarser than fp16); three 6-bit slices with block scales (finer than fp16, 1.5 times the matrix cycles: level).
//
// Where x'' is exact in fp16 as it stands (16-bit activations times power-of-two scales, for instance) the sums would be rounded for
// nothing.  Such layers (prefill_plain, from s_in and the type of x) take the operands one column at a time through the dense
// instruction, in the same kernels otherwise (PLAIN).
//
// fp16 (not bf16) operands: +-1 is exact in both and the MFMA rate is the same, but rounding x'
// and t to 8 mantissa bits breaks the 1e-3 parity bar while 11 bits hold it with margin.
//
// Operand order.  Of a step (64 columns) the lane group g of a tile holds columns 16 g + 4 v + b as byte b of word v; the pairs
// are (word 0, word 1) and (word 2, word 3) at one byte index, i.e. columns c and c + 4, and X'' and T are STORED as
// the pairs' sums and differences in the order in which the instruction meets them (pf_store_pairs).
#include <algorithm>
#include <cstdio>
#include <type_traits>

#include "nq_internal.h"

// M0 among an asm statement's written registers is what is meant here (the warning calls it reserved)
#pragma clang diagnostic ignored "-Winline-asm"

namespace nq {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned int v4u32 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) v4u32* gp_v4u32;

constexpr int kPfTokens = 64;           // tokens per workgroup tile (4 MFMA column groups)
constexpr int kPfWaves = 4;             // waves per workgroup, one 128-row block each
constexpr int kPfSlots = 4;             // 64-column steps staged in LDS at a time (one read, three on their way)
constexpr int kPfTrStride = 132;        // floats per token row of a wave's epilogue region (128 + 4: conflict-free both ways)

typedef _Float16 v16h __attribute__((ext_vector_type(16)));
enum { EPI_PARTIAL = 0, EPI_T = 1, EPI_Y = 2 };

struct GemmArgs {
    const _Float16* act;       // [m_pad][lda] halves: pair sums and differences (see above)
    const uint32_t* tiles;     // sign tiles of the weight: rows = outputs, columns = reduction
    float* partial;            // EPI_PARTIAL: [splits][m_pad][n_pad] raw accumulators
    _Float16* t_out;           // EPI_T: [m_pad][ldt]
    void* y_out;               // EPI_Y: [batch][n_real] elements of y_dtype
    int y_dtype;
    const float* tok_scale;    // EPI_Y: per token 1 / (2^a_b * g)
    const uint16_t* out_scale; // EPI_Y: fp16 [n_real]
    float t_scale;             // EPI_T: g
    const uint16_t* mid_scale; // EPI_T: rank-wise scale fp16 [n_pad] (zeros beyond n_real) or nullptr
    int lda, ldt;
    int n_real;                // real output rows
    int n_rb;                  // row blocks of the weight
    int nst;                   // 64-column steps of the reduction
    int m_tiles, n_tiles;      // workgroup grid
    int batch;                 // real tokens
    int splits, steps_per_split;
    int n_pad, m_pad;
    int m_rows;                // tokens of the tiles that are launched (at most m_pad)
};

__device__ __forceinline__ float h2f(uint16_t h) { return (float)__builtin_bit_cast(_Float16, h); }

// ---------------------------------------------------------------------------------------------
// pre-scale: one workgroup per token
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ float pf_load(const void* p, int dtype, int64_t i)
{
    if (dtype == NQ_F32) return ((const float*)p)[i];
    if (dtype == NQ_F16) return h2f(((const uint16_t*)p)[i]);
    return __builtin_bit_cast(float, (uint32_t)((const uint16_t*)p)[i] << 16);
}

// eight consecutive scaled inputs x'[k0..k0+7] of one token (zero beyond d_in)
__device__ __forceinline__ void pf_load8(const void* x, int dtype, const uint16_t* s_in, int64_t base, int k0, int d_in,
                                         bool vec, float v[8])
{
    if (vec && k0 + 8 <= d_in) {
        if (dtype == NQ_F32) {
            const float4 f0 = *(const float4*)((const float*)x + base + k0);
            const float4 f1 = *(const float4*)((const float*)x + base + k0 + 4);
            v[0] = f0.x; v[1] = f0.y; v[2] = f0.z; v[3] = f0.w; v[4] = f1.x; v[5] = f1.y; v[6] = f1.z; v[7] = f1.w;
        } else {
            const uint4 u = *(const uint4*)((const uint16_t*)x + base + k0);
            const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint16_t lo = (uint16_t)(w[i] & 0xFFFFu), hi = (uint16_t)(w[i] >> 16);
                v[2 * i] = dtype == NQ_F16 ? h2f(lo) : __builtin_bit_cast(float, (uint32_t)lo << 16);
                v[2 * i + 1] = dtype == NQ_F16 ? h2f(hi) : __builtin_bit_cast(float, (uint32_t)hi << 16);
            }
        }
        const uint4 su = *(const uint4*)(s_in + k0);
        const uint32_t sw[4] = {su.x, su.y, su.z, su.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[2 * i] *= h2f((uint16_t)(sw[i] & 0xFFFFu));
            v[2 * i + 1] *= h2f((uint16_t)(sw[i] >> 16));
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = k0 + i < d_in ? pf_load(x, dtype, base + k0 + i) * h2f(s_in[k0 + i]) : 0.f;
    }
}

// 16 consecutive values of a token (columns 16 g .. 16 g + 15 of a 64-column step), each times sc -> the sums and differences
// of their eight pairs as fp16, in the order the matrix instruction meets them: dst = the token's step + 8 g halves, the second
// eight go 32 halves further on.  A pair is (column c, column c + 4): bytes of one index in two words of a tile.
__device__ __forceinline__ void pf_store_pairs(_Float16* dst, const float v[16], float sc)
{
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        v8h o;
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            // (scaled by the power of two first: sums of values near fp32's largest would overflow)
            const int i = h + 2 * n;
            const float a = v[i] * sc, b = v[4 + i] * sc, c = v[8 + i] * sc, d = v[12 + i] * sc;
            o[4 * n] = (_Float16)(a + b);
            o[4 * n + 1] = (_Float16)(a - b);
            o[4 * n + 2] = (_Float16)(c + d);
            o[4 * n + 3] = (_Float16)(c - d);
        }
        *(v8h*)(dst + 32 * h) = o;
    }
}

// The same 16 columns as they are, for the dense instruction: half h (columns 16 g + 8 h ..) is piece (g & 1) * 4 + 2 h + (g >> 1) of
// the token's eight 16-byte pieces of a step, the one that lane group g reads as half h of its operand; inside it the columns are in
// the order in which pf_signs has words 2 h and 2 h + 1 of a tile.  dst = the token's step + ((g & 1) * 4 + (g >> 1)) * 8 halves.
__device__ __forceinline__ void pf_store_plain(_Float16* dst, const float v[16], float sc)
{
    constexpr int order[8] = {0, 2, 4, 6, 1, 3, 5, 7};
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        v8h o;
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] = (_Float16)(v[8 * h + order[i]] * sc);
        *(v8h*)(dst + 16 * h) = o;
    }
}
// chunk g (columns 16 g ..) of a token's step at `step`
template <bool PLAIN>
__device__ __forceinline__ void pf_store16(_Float16* step, int g, const float v[16], float sc)
{
    if (PLAIN) pf_store_plain(step + ((g & 1) * 4 + (g >> 1)) * 8, v, sc);
    else pf_store_pairs(step + g * 8, v, sc);
}

// one workgroup per token: max |x'|, then the pairs of x'' = x' * 2^a as fp16.  A thread takes 16 columns at a time; up to
// kPreHeld such chunks per thread stay in registers between the two passes (rows up to 32768 elements are read once); longer
// rows are read twice.  The workgroup is no wider than the row needs (pre_threads).
constexpr int kPreThreads = 1024;
constexpr int kPreHeld = 2;

// DT: the element type of x (a template parameter, so that the loads of the fast path sit in
// straight-line code: all of a thread's chunks are requested back to back, then converted).
template <int DT, bool PLAIN>
__global__ void __launch_bounds__(kPreThreads)
prefill_prescale_kernel(const void* __restrict__ x, const uint16_t* __restrict__ s_in, int d_in, int lda,
                        float g_t, int a_min, _Float16* __restrict__ xs, float* __restrict__ tok_scale)
{
    __shared__ float sm[kPreThreads / 64];
    constexpr int x_dtype = DT;
    const int tok = blockIdx.x;
    const int tid = threadIdx.x, threads = blockDim.x;
    const int64_t base = (int64_t)tok * d_in;
    constexpr int esz = DT == NQ_F32 ? 4 : 2;
    const int n16 = lda / 16;
    const bool held = n16 <= threads * kPreHeld;
    // rows that fit the registers: no branch around a load.  A chunk past the last whole one re-reads chunk 0 and counts as
    // zeros, the last, partial one is filled element by element.  (The loads are 16 bytes at the alignment of an element,
    // which global memory takes: rows of odd lengths are read as wide as those of model shapes.  333 rows of 4095 fp16
    // elements: 5.3 us, element by element 10.3.)
    const bool fast = held && d_in >= 16;
    const bool vec = (((size_t)d_in * esz) & 15) == 0;      // every token row starts 16-byte aligned
    float hv[kPreHeld][16];
    float m = 0.f;
    if (fast) {
        const int n_in = d_in / 16;
        typedef v4f v4f_any __attribute__((aligned(4)));
        typedef v4u32 v4u32_any __attribute__((aligned(2)));
        typedef const __attribute__((address_space(1))) v4f_any* gp_v4f;
        typedef const __attribute__((address_space(1))) v4u32_any* gp_v4u32_any;
        v4u32 xr[kPreHeld][2], sr[kPreHeld][2];
        v4f xf[kPreHeld][4];
        const char* const xrow = (const char*)x + (size_t)base * esz;
#pragma unroll
        for (int k = 0; k < kPreHeld; ++k) {
            const int c = tid + k * threads;
            const uint32_t cc = (uint32_t)(c < n_in ? c : 0);
            if (DT == NQ_F32) {
#pragma unroll
                for (int i = 0; i < 4; ++i) xf[k][i] = *(gp_v4f)(xrow + cc * 64u + 16u * i);
            } else {
#pragma unroll
                for (int i = 0; i < 2; ++i) xr[k][i] = *(gp_v4u32_any)(xrow + cc * 32u + 16u * i);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) sr[k][i] = *(gp_v4u32)((const char*)s_in + cc * 32u + 16u * i);
        }
#pragma unroll
        for (int k = 0; k < kPreHeld; ++k) {
            const bool valid = tid + k * threads < n_in;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                float xv[8];
                if (DT == NQ_F32) {
                    const v4f a = xf[k][2 * h], b = xf[k][2 * h + 1];
                    xv[0] = a.x; xv[1] = a.y; xv[2] = a.z; xv[3] = a.w;
                    xv[4] = b.x; xv[5] = b.y; xv[6] = b.z; xv[7] = b.w;
                } else {
                    const uint32_t w[4] = {xr[k][h].x, xr[k][h].y, xr[k][h].z, xr[k][h].w};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint16_t lo = (uint16_t)(w[i] & 0xFFFFu), hi = (uint16_t)(w[i] >> 16);
                        xv[2 * i] = DT == NQ_F16 ? h2f(lo) : __builtin_bit_cast(float, (uint32_t)lo << 16);
                        xv[2 * i + 1] = DT == NQ_F16 ? h2f(hi) : __builtin_bit_cast(float, (uint32_t)hi << 16);
                    }
                }
                const uint32_t sw[4] = {sr[k][h].x, sr[k][h].y, sr[k][h].z, sr[k][h].w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float v0 = xv[2 * i] * h2f((uint16_t)(sw[i] & 0xFFFFu));
                    const float v1 = xv[2 * i + 1] * h2f((uint16_t)(sw[i] >> 16));
                    hv[k][8 * h + 2 * i] = valid ? v0 : 0.f;
                    hv[k][8 * h + 2 * i + 1] = valid ? v1 : 0.f;
                    m = fmaxf(m, fmaxf(fabsf(hv[k][8 * h + 2 * i]), fabsf(hv[k][8 * h + 2 * i + 1])));
                }
            }
            if ((d_in & 15) && tid + k * threads == n_in) {
                pf_load8(x, x_dtype, s_in, base, n_in * 16, d_in, false, hv[k]);
                pf_load8(x, x_dtype, s_in, base, n_in * 16 + 8, d_in, false, hv[k] + 8);
#pragma unroll
                for (int i = 0; i < 16; ++i) m = fmaxf(m, fabsf(hv[k][i]));
            }
        }
    } else if (held) {
#pragma unroll
        for (int k = 0; k < kPreHeld; ++k) {
            const int c = tid + k * threads;
            if (c < n16) {
                pf_load8(x, x_dtype, s_in, base, c * 16, d_in, false, hv[k]);
                pf_load8(x, x_dtype, s_in, base, c * 16 + 8, d_in, false, hv[k] + 8);
#pragma unroll
                for (int i = 0; i < 16; ++i) m = fmaxf(m, fabsf(hv[k][i]));
            }
        }
    } else {
        for (int c = tid; c < n16; c += threads) {
            float v[16];
            pf_load8(x, x_dtype, s_in, base, c * 16, d_in, vec, v);
            pf_load8(x, x_dtype, s_in, base, c * 16 + 8, d_in, vec, v + 8);
#pragma unroll
            for (int i = 0; i < 16; ++i) m = fmaxf(m, fabsf(v[i]));
        }
    }
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    if ((tid & 63) == 0) sm[tid >> 6] = m;
    __syncthreads();
    m = sm[0];
    for (int w = 1; w < threads / 64; ++w) m = fmaxf(m, sm[w]);
    // 2^a with max * 2^a in [2^12, 2^13); a NaN/Inf token keeps a = 0 and poisons only itself
    float sc = 1.0f;
    if (m > 0.f && m <= 3.0e38f) {
        int e;
        (void)frexpf(m, &e);
        int a = 13 - e;
        a = a > 100 ? 100 : (a < a_min ? a_min : a);
        sc = ldexpf(1.0f, a);
    }
    // chunk c = columns 16 (c & 3) .. of step c >> 2
    _Float16* row = xs + (size_t)tok * lda;
    if (held) {
#pragma unroll
        for (int k = 0; k < kPreHeld; ++k) {
            const int c = tid + k * threads;
            if (c < n16) pf_store16<PLAIN>(row + (c >> 2) * 64, c & 3, hv[k], sc);
        }
    } else {
        for (int c = tid; c < n16; c += threads) {
            float v[16];
            pf_load8(x, x_dtype, s_in, base, c * 16, d_in, vec, v);
            pf_load8(x, x_dtype, s_in, base, c * 16 + 8, d_in, vec, v + 8);
            pf_store16<PLAIN>(row + (c >> 2) * 64, c & 3, v, sc);
        }
    }
    if (tid == 0) tok_scale[tok] = 1.0f / (sc * g_t);
}

// ---------------------------------------------------------------------------------------------
// GEMM:  C[token][n] = sum_k act[token][k] * sign(tiles[n][k])
// grid = (m_tiles * n_tiles, splits); block = 256 (4 waves x 128 output rows, 64 tokens)
// ---------------------------------------------------------------------------------------------
// 16 consecutive results of gemm 1 (columns n0 .. n0 + 15 of T, n0 a multiple of 16) of token `tok` -> T as gemm 2 reads it:
// times g, times the rank-wise scale of the three-scale variant where there is one (its own power of two is folded into g);
// columns beyond the real rank are exact zeros (they are padding of the next reduction).
template <bool PLAIN>
__device__ __forceinline__ void store_t16(const GemmArgs& a, int tok, int n0, const float c[16])
{
    float f[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) f[i] = a.t_scale;
    if (a.mid_scale && n0 < a.n_pad) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const uint4 m = *(const uint4*)(a.mid_scale + n0 + 8 * q);
            const uint32_t w[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                f[8 * q + 2 * i] *= h2f((uint16_t)(w[i] & 0xFFFFu));
                f[8 * q + 2 * i + 1] *= h2f((uint16_t)(w[i] >> 16));
            }
        }
    }
    float v[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = n0 + i < a.n_real ? c[i] * f[i] : 0.f;
    pf_store16<PLAIN>(a.t_out + (size_t)tok * a.ldt + (n0 >> 6) * 64, (n0 >> 4) & 3, v, 1.0f);
}

// A lane's 16 tile bytes as the sparse matrix instruction takes them.  Word v, byte b, bit p = the sign of (row 16 p + j, column
// 16 g + 4 v + b); the pairs are (word 0, word 1) and (word 2, word 3) of one byte index, and a group of four operand positions
// (two pairs: sum, difference, sum, difference) is one byte index, in the order 0, 2, 1, 3.
//   r01, r23: words 0 and 2 with bytes 0 and 1 (2 and 3) side by side in 16-bit halves: the signs of the pairs' first members
//   i0: 16-bit halves = planes 0 | 4 (bits 2 k) and 1 | 5 (bits 2 k + 1), bit 2 k = whether the signs of pair k differ; i1: 2 | 6, 3 | 7
struct PfBits { uint32_t r01, r23, i0, i1; };
__device__ __forceinline__ uint32_t pf_bfi(uint32_t m, uint32_t a, uint32_t b) { return (m & a) | (~m & b); }
__device__ __forceinline__ uint32_t pf_gather_nibbles(uint32_t a)
{
    return pf_bfi(0xF0F00F0Fu, a, pf_bfi(0x0000FFFFu, a >> 12, a << 12));
}
__device__ __forceinline__ PfBits pf_bits(const v4u32 w)
{
    const uint32_t fa = w.x ^ w.y, fb = w.z ^ w.w;
    PfBits b;
    b.r01 = __builtin_amdgcn_perm(w.z, w.x, 0x05040100u);
    b.r23 = __builtin_amdgcn_perm(w.z, w.x, 0x07060302u);
    b.i0 = pf_gather_nibbles(pf_bfi(0x33333333u, fa, fb << 2));
    b.i1 = pf_gather_nibbles(pf_bfi(0x33333333u, fa >> 2, fb));
    return b;
}
// masks and constants of the two functions below, in registers: as literals the compiler spends an AND and an OR where
// one v_and_or_b32 does
struct PfConst { uint32_t sign, one, even, base; };
__device__ __forceinline__ PfConst pf_const()
{
    PfConst k = {0x80008000u, 0x3C003C00u, 0x55555555u, 0x88888888u};
    asm volatile("" : "+s"(k.sign), "+v"(k.one), "+s"(k.even), "+v"(k.base));
    return k;
}
// the eight values (+-1.0) of plane p
template <int P>
__device__ __forceinline__ v4u32 pf_signs(const PfBits& b, const PfConst& k)
{
    v4u32 a;
    a.x = ((b.r01 << (15 - P)) & k.sign) | k.one;
    a.y = ((b.r23 << (15 - P)) & k.sign) | k.one;
    a.z = ((b.r01 << (7 - P)) & k.sign) | k.one;
    a.w = ((b.r23 << (7 - P)) & k.sign) | k.one;
    return a;
}
// positions of the nonzeros of planes P (low half) and P + 4 (high half), P = 0..3
template <int P>
__device__ __forceinline__ uint32_t pf_index(const PfBits& b, const PfConst& k)
{
    const uint32_t w = P < 2 ? b.i0 : b.i1;
    return ((P & 1 ? w >> 1 : w) & k.even) | k.base;
}

// four consecutive outputs o (already scaled) of y, row-major: one store at the alignment of an element (global memory takes
// it: rows of any length are written as wide as those of model shapes), or element by element in a row's last, partial group
// (`left` = elements to the row's end).  STREAM: non-temporal.  The second GEMM
// of an 11005 x 4095 r = 1663 layer at 333 tokens: 24 us, with element stores 41.
template <bool STREAM>
__device__ __forceinline__ void store_y4(void* y, int dtype, size_t at, int left, const v4f o)
{
    typedef uint32_t v2u32 __attribute__((ext_vector_type(2)));
    typedef v4f v4f_any __attribute__((aligned(4)));
    typedef v2u32 v2u32_any __attribute__((aligned(2)));
    if (left >= 4) {
        if (dtype == NQ_F32) {
            v4f_any* const p = (v4f_any*)((float*)y + at);
            if (STREAM) __builtin_nontemporal_store(o, p);
            else *p = o;
        } else {
            v2u32 pk;
            pk.x = (uint32_t)float_to_out16(o.x, dtype) | ((uint32_t)float_to_out16(o.y, dtype) << 16);
            pk.y = (uint32_t)float_to_out16(o.z, dtype) | ((uint32_t)float_to_out16(o.w, dtype) << 16);
            v2u32_any* const p = (v2u32_any*)((uint16_t*)y + at);
            if (STREAM) __builtin_nontemporal_store(pk, p);
            else *p = pk;
        }
    } else {
        if (left > 0) store_out(y, dtype, at, o.x);
        if (left > 1) store_out(y, dtype, at + 1, o.y);
        if (left > 2) store_out(y, dtype, at + 2, o.z);
    }
}
// the output scales of four consecutive rows n0 .. n0 + 3 (n0 a multiple of 4; zero past the end)
__device__ __forceinline__ v4f load_scale4(const uint16_t* scale, int n0, int n)
{
    v4f r = {0.f, 0.f, 0.f, 0.f};
    if (n0 + 4 <= n) {
        const uint2 sc = *(const uint2*)(scale + n0);
        r.x = h2f((uint16_t)(sc.x & 0xFFFFu));
        r.y = h2f((uint16_t)(sc.x >> 16));
        r.z = h2f((uint16_t)(sc.y & 0xFFFFu));
        r.w = h2f((uint16_t)(sc.y >> 16));
    } else {
        if (n0 < n) r.x = h2f(scale[n0]);
        if (n0 + 1 < n) r.y = h2f(scale[n0 + 1]);
        if (n0 + 2 < n) r.z = h2f(scale[n0 + 2]);
    }
    return r;
}

// C[token][n] = sum_k act[token][k] * sign(tiles[n][k]); grid = (m_tiles * n_tiles, splits), four waves x 128 output rows.
// TG = token groups of 16 per workgroup tile: 4 (64 tokens) normally; 2 (32 tokens) where 64-token tiles are too few to cover
// the chip, or leave a last round nearly empty (the sign operands then serve half as many matrix instructions: a step
// costs a CU 0.255 us against 0.34, but a tile is half as large).
// KS = 2: eight waves; waves 4..7 take the same rows and tokens as waves 0..3 but the second half of
// the workgroup's part of the reduction (with staging buffers of their own), and hand their
// accumulators to their partners through LDS before the epilogue.  Such a workgroup fills its CU by itself (two waves per
// SIMD), and the reduction is halved without partial sums in memory.
template <int EPI, int TG, int KS, bool PLAIN>
__global__ void __launch_bounds__(64 * kPfWaves * KS) __attribute__((amdgpu_waves_per_eu(2, TG == 4 ? 2 : 4)))
prefill_gemm_kernel(GemmArgs a)
{
    static_assert((TG == 2 && KS == 1) || (TG == 4 && (KS == 1 || KS == 2)), "32- or 64-token tiles; only the latter split their part in two");
    constexpr int WR = kPfWaves;
    constexpr int kTok = 16 * TG;
    // a slot holds one step: per wave the activations that it fetches (pieces of 8 tokens x 128 bytes), then its tile (1 KiB).
    // After the reduction the same memory serves the exchange of accumulators and the epilogue.
    constexpr int kPieces = 2 * TG / WR;                                // activation pieces per wave and step
    constexpr int kWaveBytes = (kPieces + 1) * 1024, kSlotBytes = WR * kWaveBytes;
    static_assert(kTok == 8 * kPieces * WR && kPieces <= 2, "a token group is two pieces");
    constexpr int kRing = kPfSlots * kSlotBytes, kEpiBytes = WR * 16 * kPfTrStride * 4;
    constexpr int kLdsBytes = KS * kRing > kEpiBytes ? KS * kRing : kEpiBytes;
    static_assert(KS == 1 || kLdsBytes >= WR * 2 * 8 * 64 * 16, "exchange of two token groups per round");
    __shared__ __attribute__((aligned(1024))) char lds_raw[kLdsBytes];
    const int lane = threadIdx.x & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int wave = wave_all % WR, grp = wave_all / WR;                // row block within the tile, part of the reduction
    const int g = lane >> 4, j = lane & 15;

    // workgroups that share a token tile run on the same XCD (ids are dealt round-robin to the
    // 8 XCDs) so the activation tile is fetched into that XCD's L2 once
    const int total = a.m_tiles * a.n_tiles;
    int id = blockIdx.x;
    {
        const int per = total / 8;
        if (id < per * 8) id = (id & 7) * per + (id >> 3);
    }
    const int m_tile = id / a.n_tiles, n_tile = id - m_tile * a.n_tiles;
    const int split = blockIdx.y;
    // (with KS = 2 the host makes the workgroup's part a multiple of eight steps: equal halves, both
    // multiples of four, so that all waves pass the same barriers)
    const int wg_begin = split * a.steps_per_split;
    const int wg_steps = max(0, min(a.nst, wg_begin + a.steps_per_split) - wg_begin);
    const int n_my = wg_steps / KS;
    const int s_begin = wg_begin + grp * n_my;

    const int rb = n_tile * WR + wave;
    const bool rb_valid = rb < a.n_rb;
    const int rb_ld = rb_valid ? rb : a.n_rb - 1;          // a wave past the last row block keeps loading valid memory
    const int m0 = m_tile * kTok;

    v4f acc[8][TG];
#pragma unroll
    for (int p = 0; p < 8; ++p)
#pragma unroll
        for (int tg = 0; tg < TG; ++tg) acc[p][tg] = v4f{0.f, 0.f, 0.f, 0.f};

    // Everything a step needs goes from memory to LDS without passing through registers, three steps ahead: each wave asks for
    // its own tile (1 KiB) and its share of the activations (pieces of 8 tokens x 128 bytes).  Lane l of a piece
    // fetches the 16 bytes (l & 7) ^ (l >> 3) of token l >> 3 (the place in LDS is the lane's): the lanes of a matrix operand
    // then read 16-byte pieces of 16 tokens without bank conflicts.
    constexpr int kDma = kPieces + 1;                                   // requests per wave and step
    const uint32_t row_bytes = (uint32_t)a.lda * 2;
    // (a request's immediate offset moves its LDS address too: 1024 per piece, taken back in the memory offset)
    uint32_t act_off[kPieces];
#pragma unroll
    for (int i = 0; i < kPieces; ++i)
        act_off[i] = (uint32_t)(lane >> 3) * row_bytes + (uint32_t)(((lane & 7) ^ (lane >> 3)) * 16) + i * (8 * row_bytes - 1024);
    const uint32_t tile_off = (uint32_t)lane * 16;
    const char* const act_base = (const char*)a.act + ((size_t)m0 + 8 * kPieces * wave) * row_bytes + (size_t)s_begin * 128;
    const char* const tile_base = (const char*)a.tiles + ((size_t)rb_ld * a.nst + s_begin) * (kTileWords * 4);
    const uint32_t lds_wave = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds_raw + (uint32_t)(grp * kRing + wave * kWaveBytes);
    // (the requests are written out because for the builtin the compiler waits for all of them before every LDS read.  They
    // have no register result.  M0, which holds the LDS address, is named as written: the compiler sets it before uses of its own, but
    // may set it once for several.)
#define PF_DMA1(lds_addr, voff, base)                                                                                      \
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(voff), "s"(base) : "memory", "m0")
#define PF_DMA2(lds_addr, voff0, voff1, base, OFF0, OFF1)                                                                  \
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %3 offset:" OFF0                          \
                 "\n\tglobal_load_lds_dwordx4 %2, %3 offset:" OFF1 ::"s"(lds_addr), "v"(voff0), "v"(voff1), "s"(base) : "memory", "m0")
    // part k = 0 .. 2 of the requests of step `step` (spread over the planes of the step before: issued together they leave
    // the matrix cores of their SIMD idle for 5 to 9 us in 100)
#define PF_REQUEST(slot, step, k)                                                                                          \
    do {                                                                                                                   \
        const uint32_t la = lds_wave + (slot) * kSlotBytes;                                                                \
        const char* const ab = act_base + (size_t)(step) * 128;                                                            \
        const char* const tb = tile_base + (size_t)(step) * (kTileWords * 4);                                              \
        if ((k) == 0) PF_DMA1(la + kPieces * 1024, tile_off, tb);                                                          \
        if (kPieces == 1 && (k) == 1) PF_DMA1(la, act_off[0], ab);                                                         \
        if (kPieces == 2 && (k) == 2) PF_DMA2(la, act_off[0], act_off[kPieces - 1], ab, "0", "1024");                      \
    } while (0)
    // all but the newest n of this wave's requests have arrived, and its own LDS reads are done; then the same for all waves
#define PF_WAIT(n) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(n) : "memory")

    // operand of token group tg, half h (positions 32 h + 8 g .. + 7 of the step): 16-byte piece (g & 1) * 4 + 2 h + (g >> 1) of
    // token 16 tg + j
    const int j7 = j & 7;
    const uint32_t rd0 = (uint32_t)((j >> 3) * (kPieces == 1 ? kWaveBytes : 1024) + j7 * 128 + ((((g & 1) * 4 + (g >> 1)) ^ j7) * 16));
    const char* const rd_h0 = lds_raw + grp * kRing + rd0;
    const char* const rd_h1 = lds_raw + grp * kRing + (rd0 ^ 32u);
    const char* const rd_tile = lds_raw + grp * kRing + wave * kWaveBytes + kPieces * 1024 + lane * 16;
#define PF_READ_B(SET, slot, tg)                                                                                           \
    do {                                                                                                                   \
        const int at = (slot) * kSlotBytes + (2 * (tg) / kPieces) * kWaveBytes + (2 * (tg) % kPieces) * 1024;              \
        const v8h lo = *(const v8h*)(rd_h0 + at);                                                                          \
        const v8h hi = *(const v8h*)(rd_h1 + at);                                                                          \
        bop[SET][tg] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);              \
    } while (0)
#define PF_READ_TILE(slot) (*(const v4u32*)(rd_tile + (slot) * kSlotBytes))

    // n_my is a multiple of 4 (the reduction is padded to 4 steps and so are the splits), and the loop body is branch-free:
    // requests past the end ask for the last step again.  Step s works on registers read during step s - 1; meanwhile
    // slot s + 1 is read, slots s + 2 and s + 3 fill, and step s + 4 is requested into the slot that step s has left.
    if (n_my > 0) {
        const int last = n_my - 1;
        v16h bop[2][TG];
        v4u32 w;
#pragma unroll
        for (int k = 0; k < kPfSlots; ++k)
#pragma unroll
            for (int part = 0; part < 3; ++part) PF_REQUEST(k, min(k, last), part);
        PF_WAIT(3 * kDma);
        w = PF_READ_TILE(0);
#pragma unroll
        for (int tg = 0; tg < TG; ++tg) PF_READ_B(0, 0, tg);
        const PfConst kc = pf_const();
        // the reads of the next step beside plane number k of this one
#define PF_READS(SET, slot, k)                                                                                             \
    do {                                                                                                                   \
        if ((k) == 0) w = PF_READ_TILE(slot);                                                                              \
        if ((k) < TG) PF_READ_B(SET, slot, (k) % TG);                                                                      \
    } while (0)
        if constexpr (PLAIN) {
            // half h of a lane's operand = the columns of words 2 h and 2 h + 1 of its tile: a dense instruction per plane, half and
            // token group
            PfBits b0 = {w.x, w.y, 0, 0}, b1 = {w.z, w.w, 0, 0};
            v4u32 au = pf_signs<0>(b0, kc);
#define PF_HALF(P, H, SET, NEXT, READS)                                                                                    \
    do {                                                                                                                   \
        const v8h aop = __builtin_bit_cast(v8h, au);                                                                       \
        NEXT;                                                                                                              \
        READS;                                                                                                             \
        _Pragma("unroll") for (int tg = 0; tg < TG; ++tg) {                                                                \
            const v16h b = bop[SET][tg];                                                                                   \
            const v8h half = (H) ? __builtin_shufflevector(b, b, 8, 9, 10, 11, 12, 13, 14, 15)                             \
                                 : __builtin_shufflevector(b, b, 0, 1, 2, 3, 4, 5, 6, 7);                                  \
            acc[P][tg] = __builtin_amdgcn_mfma_f32_16x16x32_f16(aop, half, acc[P][tg], 0, 0, 0);                           \
        }                                                                                                                  \
        _Pragma("unroll") for (int i = 0; i < TG; ++i) {                                                                   \
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                                             \
            __builtin_amdgcn_sched_group_barrier(0x002, 8 / TG, 0);                                                        \
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                                             \
        }                                                                                                                  \
        __builtin_amdgcn_sched_barrier(0);                                                                                 \
    } while (0)
#define PF_PLANE(P, SET, READS0, READS1)                                                                                   \
    do {                                                                                                                   \
        PF_HALF(P, 0, SET, au = pf_signs<P>(b1, kc), READS0);                                                              \
        if ((P) == 7) { b0 = PfBits{w.x, w.y, 0, 0}; b1 = PfBits{w.z, w.w, 0, 0}; }                                        \
        PF_HALF(P, 1, SET, au = pf_signs<((P) + 1) % 8>(b0, kc), READS1);                                                  \
    } while (0)
#define PF_STEP(SET, SLOT, step)                                                                                           \
    do {                                                                                                                   \
        PF_WAIT(2 * kDma);                                                                                                 \
        const int nx = min((step) + kPfSlots, last);                                                                       \
        constexpr int NS = ((SLOT) + 1) % kPfSlots, ST = 1 - (SET);                                                        \
        PF_PLANE(0, SET, PF_READS(ST, NS, 0), PF_REQUEST(SLOT, nx, 0));                                                    \
        PF_PLANE(1, SET, PF_READS(ST, NS, 1), PF_REQUEST(SLOT, nx, 1));                                                    \
        PF_PLANE(2, SET, PF_READS(ST, NS, 2), PF_REQUEST(SLOT, nx, 2));                                                    \
        PF_PLANE(3, SET, PF_READS(ST, NS, 3), );                                                                           \
        PF_PLANE(4, SET, , );                                                                                              \
        PF_PLANE(5, SET, , );                                                                                              \
        PF_PLANE(6, SET, , );                                                                                              \
        PF_PLANE(7, SET, , );                                                                                              \
    } while (0)
            for (int s = 0; s < n_my; s += 4) {
                PF_STEP(0, 0, s);
                PF_STEP(1, 1, s + 1);
                PF_STEP(0, 2, s + 2);
                PF_STEP(1, 3, s + 3);
            }
#undef PF_STEP
#undef PF_PLANE
#undef PF_HALF
        } else {
        PfBits bits = pf_bits(w);
        v4u32 au = pf_signs<0>(bits, kc);
        uint32_t ix0 = pf_index<0>(bits, kc), ix1 = 0, ix2 = 0, ix3 = 0;
        // one plane: the values of the next plane are built, and LDS is read, in the shadow of its matrix instructions
#define PF_PLANE(P, SET, IX, HALF, NEXT, READS, NVALU)                                                                     \
    do {                                                                                                                   \
        const v8h aop = __builtin_bit_cast(v8h, au);                                                                       \
        NEXT;                                                                                                              \
        READS;                                                                                                             \
        _Pragma("unroll") for (int tg = 0; tg < TG; ++tg)                                                                  \
            acc[P][tg] = __builtin_amdgcn_smfmac_f32_16x16x64_f16(aop, bop[SET][tg], acc[P][tg], (int)IX, 0, HALF);        \
        _Pragma("unroll") for (int i = 0; i < TG; ++i) {                                                                   \
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                                             \
            __builtin_amdgcn_sched_group_barrier(0x002, ((NVALU) + TG - 1) / TG, 0);                                       \
            if (i < 4) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                                  \
        }                                                                                                                  \
        __builtin_amdgcn_sched_barrier(0);                                                                                 \
    } while (0)
#define PF_STEP(SET, SLOT, step)                                                                                           \
    do {                                                                                                                   \
        PF_WAIT(2 * kDma);                                                                                                 \
        const int nx = min((step) + kPfSlots, last);                                                                       \
        constexpr int NS = ((SLOT) + 1) % kPfSlots, ST = 1 - (SET);                                                        \
        PF_PLANE(0, SET, ix0, 0, au = pf_signs<4>(bits, kc); ix1 = pf_index<1>(bits, kc), PF_READS(ST, NS, 0); PF_REQUEST(SLOT, nx, 0), 10);        \
        PF_PLANE(4, SET, ix0, 1, au = pf_signs<1>(bits, kc); ix2 = pf_index<2>(bits, kc), PF_READS(ST, NS, 1); PF_REQUEST(SLOT, nx, 1), 9);         \
        PF_PLANE(1, SET, ix1, 0, au = pf_signs<5>(bits, kc); ix3 = pf_index<3>(bits, kc), PF_READS(ST, NS, 2); PF_REQUEST(SLOT, nx, 2), 10);        \
        PF_PLANE(5, SET, ix1, 1, au = pf_signs<2>(bits, kc), PF_READS(ST, NS, 3), 8);                                      \
        PF_PLANE(2, SET, ix2, 0, au = pf_signs<6>(bits, kc), , 8);                                      \
        PF_PLANE(6, SET, ix2, 1, au = pf_signs<3>(bits, kc), , 8);                                      \
        PF_PLANE(3, SET, ix3, 0, au = pf_signs<7>(bits, kc); bits = pf_bits(w), , 28);                  \
        PF_PLANE(7, SET, ix3, 1, au = pf_signs<0>(bits, kc); ix0 = pf_index<0>(bits, kc), , 10);                           \
    } while (0)
        for (int s = 0; s < n_my; s += 4) {
            PF_STEP(0, 0, s);
            PF_STEP(1, 1, s + 1);
            PF_STEP(0, 2, s + 2);
            PF_STEP(1, 3, s + 3);
        }
#undef PF_STEP
#undef PF_PLANE
        }
#undef PF_READS
    }
    // nothing on its way into LDS any more, in no wave: the memory changes hands
    PF_WAIT(0);
#undef PF_WAIT
#undef PF_REQUEST
#undef PF_DMA1
#undef PF_DMA2
#undef PF_READ_B
#undef PF_READ_TILE

    float* const lds_f = (float*)&lds_raw[0];
    if (KS == 2) {
        // the second part's waves hand their accumulators to the first's, two token groups per round: a lane's 16
        // registers of a token group go to the same lane of the partner (no transposition here).
        // Every wave adds what it reads (the second half's sums are not used any further): no
        // branch around a write to the accumulators.
        float* const xr = lds_f + wave * (2 * 8 * 64 * 4);
#pragma unroll
        for (int round = 0; round < TG / 2; ++round) {
            if (grp == 1) {
#pragma unroll
                for (int tl = 0; tl < 2; ++tl)
#pragma unroll
                    for (int p = 0; p < 8; ++p) *(v4f*)(xr + ((tl * 8 + p) * 64 + lane) * 4) = acc[p][2 * round + tl];
            }
            __syncthreads();
#pragma unroll
            for (int tl = 0; tl < 2; ++tl) {
#pragma unroll
                for (int p = 0; p < 8; ++p) acc[p][2 * round + tl] += *(const v4f*)(xr + ((tl * 8 + p) * 64 + lane) * 4);
                // (eight reads in flight, not sixteen: registers)
                // The sums are complete before the barrier: only waves of the first part use them further on, and left to itself the compiler
                // moves the last round's reads past the barrier into the code of those, where the epilogue's regions of other waves
                // may already have been written over what is read.
#pragma unroll
                for (int p = 0; p < 8; ++p) asm volatile("" : "+v"(acc[p][2 * round + tl]));
            }
            __syncthreads();
        }
        if (grp == 1) return;
    }
    if (!rb_valid) {
        // columns of T beyond the last row block are padding of gemm 2's reduction (at most one row block of them): zeros
        if (EPI == EPI_T && rb == a.n_rb && rb * kTileRows < a.ldt) {
            const v8h z = {};
#pragma unroll
            for (int i = 0; i < kTok * 16 / 64; ++i) {
                const int c = lane + 64 * i;
                *(v8h*)(a.t_out + (size_t)(m0 + (c >> 4)) * a.ldt + rb * kTileRows + (c & 15) * 8) = z;
            }
        }
        return;
    }

    // Result layout: lane (g, j), register v of acc[p][tg]  <->  C[token m0 + 16 tg + j][row 128 rb + 16 p + 4 g + v],
    // i.e. a lane holds 4 consecutive rows of a token and a store straight from the accumulators
    // would write 64-byte pieces of 16 different output rows.  Each wave therefore turns its
    // results round in a private LDS region, 16 tokens at a time: written in the layout above,
    // read back as [token][128 rows], so that one store instruction covers two tokens x 512
    // contiguous bytes (eight tokens x 2 x 64 bytes for T).  Measured on 28672x8192 r=3520 at 2048 tokens: the stores
    // were 18 % of the time of a forward.
    float* const tr = lds_f + wave * (16 * kPfTrStride);
    const int rd_col = 4 * (lane & 31), rd_tok = lane >> 5;
    const int n0 = rb * kTileRows + rd_col;                 // the 4 rows this lane stores
    const v4f osc = EPI == EPI_Y ? load_scale4(a.out_scale, n0, a.n_real) : v4f{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int tg = 0; tg < TG; ++tg) {
        float f = 1.0f;
        if (EPI == EPI_Y) {
            const int tok = m0 + tg * 16 + j;
            f = tok < a.batch ? a.tok_scale[tok] : 0.f;
        }
#pragma unroll
        for (int p = 0; p < 8; ++p) {
            v4f c = acc[p][tg];
            if (EPI == EPI_Y) c *= f;
            *(v4f*)(tr + j * kPfTrStride + 16 * p + 4 * g) = c;
        }
        // (the region is private to the wave and a wave's LDS operations complete in order)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        if (EPI == EPI_T) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int t = (lane >> 3) + 8 * i, col = 16 * (lane & 7);
                float c[16];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const v4f r = *(const v4f*)(tr + t * kPfTrStride + col + 4 * q);
                    c[4 * q] = r.x; c[4 * q + 1] = r.y; c[4 * q + 2] = r.z; c[4 * q + 3] = r.w;
                }
                store_t16<PLAIN>(a, m0 + tg * 16 + t, rb * kTileRows + col, c);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int t = rd_tok + 2 * i;
                const int tok = m0 + tg * 16 + t;
                const v4f c = *(const v4f*)(tr + t * kPfTrStride + rd_col);
                if (EPI == EPI_PARTIAL) {
                    float* dst = a.partial + ((size_t)split * a.m_pad + tok) * a.n_pad + n0;
                    *(v4f*)dst = c;
                } else if (tok < a.batch) {
                    store_y4<true>(a.y_out, a.y_dtype, (size_t)tok * a.n_real + n0, a.n_real - n0, c * osc);
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
    }
}

// sum the split-K partials and apply the epilogue; one thread per four consecutive outputs (y) or 16 columns of T (the
// columns between the last row block and T's row length are padding of gemm 2's reduction: zeros)
template <int EPI, bool PLAIN>
__global__ void __launch_bounds__(256)
prefill_finalize_kernel(GemmArgs a)
{
    const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (EPI == EPI_T) {
        const int n16 = a.ldt / 16;
        if (idx >= (size_t)a.m_rows * n16) return;
        const int tok = (int)(idx / n16), n0 = (int)(idx % n16) * 16;
        v4f c4[4] = {};
        if (n0 < a.n_pad) {
            for (int s = 0; s < a.splits; ++s) {
                const float* src = a.partial + ((size_t)s * a.m_pad + tok) * a.n_pad + n0;
#pragma unroll
                for (int q = 0; q < 4; ++q) c4[q] += *(const v4f*)(src + 4 * q);
            }
        }
        float c[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) { c[4 * q] = c4[q].x; c[4 * q + 1] = c4[q].y; c[4 * q + 2] = c4[q].z; c[4 * q + 3] = c4[q].w; }
        store_t16<PLAIN>(a, tok, n0, c);
    } else {
        const int n4 = a.n_pad / 4;
        if (idx >= (size_t)a.m_rows * n4) return;
        const int tok = (int)(idx / n4), n0 = (int)(idx % n4) * 4;
        v4f c = {0.f, 0.f, 0.f, 0.f};
        for (int s = 0; s < a.splits; ++s) c += *(const v4f*)(a.partial + ((size_t)s * a.m_pad + tok) * a.n_pad + n0);
        if (tok < a.batch) {
            const float f = a.tok_scale[tok];
            store_y4<false>(a.y_out, a.y_dtype, (size_t)tok * a.n_real + n0, a.n_real - n0, c * f * load_scale4(a.out_scale, n0, a.n_real));
        }
    }
}

// ---------------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------------
static size_t al256(size_t v) { return (v + 255) / 256 * 256; }

struct PfLayout {
    int m_pad;                // tokens rounded up to whole 64-token tiles
    int k1, k2, n1_pad, n2_pad;
    int splits1, splits2;
    int tg1, tg2;             // token groups of 16 per workgroup tile of the two GEMMs (4 or 2)
    int ks1, ks2;             // parts of the reduction taken inside a workgroup (1 or 2)
    int m_tiles1, m_tiles2;   // token tiles launched
    size_t off_x, off_t, off_scale, off_partial, total;
};

// steps per split, rounded up to a multiple of 4 (as nst itself is): the kernel's loop body is four
// steps; of 8 where the workgroup halves its part once more (ks = 2: nst is then a multiple of 8 too)
static int steps_per_split4(int nst, int splits, int ks = 1)
{
    const int per = (nst + splits - 1) / splits, q = 4 * ks;
    return (per + q - 1) / q * q;
}

// Tiling of one GEMM: token groups per workgroup tile (4 = 64 tokens, 2 = 32 tokens), the number of workgroups the
// reduction is split over, and the halving inside a workgroup.  Cost model in microseconds, fitted to 3200 timings: both GEMMs
// of 11 layers from 512 x 512 r = 200 to 28672 x 8192 r = 3520 at 10 batches from 16 to 2048, every tile with 1 .. 16 parts (the
// choices are on average 0.3 % of a forward slower than the best of each, at most 11 %):
//  - a reduction step of a 64-token workgroup takes 0.377 us when it has its CU to itself, 0.68 when two share it (two is all
//    that fits), 0.654 where a workgroup of eight waves does two at once; of a 32-token workgroup 0.353 us alone, and a CU
//    completes one per 0.255 us (up to four fit);
//  - beside its steps a workgroup takes 9.5 us (64 tokens), 10.5 (eight waves), 6.9 (32 tokens): the first fetch and the epilogue;
//  - splitting costs the finalize launch (2.8 us) and per part 0.23 us and the write and re-read of one set of fp32
//    partial sums, 0.29 us per MB.
// Tiles are counted over the tokens that are there: 32-token tiles leave out the half of a last 64 that holds none (its rows of T stay unwritten and are only read
// for tokens that are not stored), and either tile is split.  us per forward, 64-token tiles alone split and 32-token ones in pairs / so: 11005 x 4095 r = 1663 at 333 tokens 45.9 / 38.7,
// 5000 x 5000 r = 1300 at 800 47.5 / 41.9, 4096 x 11008 r = 1664 at 150 41.1 / 38.7, 3262 x 4081 r = 820 at 137 31.9 / 29.9 (on this path; by default it takes the exact one); 40 layers from 600 to 28672 a side at 60 to 2048
// tokens on average 0.7 % slower than the best tiling of each GEMM.
// One column at a time (`plain`) the steps take 0.60, 1.05, 0.97, 0.49 and 0.35 us (each of ten tilings
// of the two GEMMs of six layers at 24 to 2048 tokens, against the same in pairs), the rest is the same.
struct GemmTiling { int tg, splits, ks; double us; };
struct StepCost { double alone4, two4, halves4, alone2, each2; };
// most32: into how many parts the reduction of 32-token tiles may be split
static GemmTiling choose_tiling(int batch, int n_rb, int nst, int n_pad, bool plain, int most32 = 16)
{
    const StepCost c = plain ? StepCost{0.60, 1.05, 0.97, 0.49, 0.35} : StepCost{0.377, 0.68, 0.654, 0.353, 0.255};
    const int cus = device_cu_count();
    const int n_tiles = (n_rb + kPfWaves - 1) / kPfWaves;
    const double partial_mb = (double)round_up(batch, kPfTokens) * n_pad * 4.0 / 1e6;
    GemmTiling best = {4, 1, 1, 0.0};
    double best_cost = 1e30;
    auto consider = [&](int tg, int splits, int ks) {
        const int wgs = (batch + 16 * tg - 1) / (16 * tg) * n_tiles * splits, per = steps_per_split4(nst, splits, ks);
        if ((splits - 1) * per >= nst) return;                 // parts without a step: fewer do the same
        double cost;
        if (ks == 2) {
            cost = (wgs + cus - 1) / cus * (per / 2 * c.halves4 + 10.5);
        } else {
            // full rounds of the CUs' slots, then the last, partial one
            const int per_cu = tg == 4 ? 2 : 4, full = wgs / (per_cu * cus), rem = wgs % (per_cu * cus), k = (rem + cus - 1) / cus;
            const double step_full = tg == 4 ? c.two4 : 4 * c.each2, step_rem = tg == 4 ? (k <= 1 ? c.alone4 : c.two4) : std::max(c.alone2, k * c.each2);
            const double fixed = tg == 4 ? 9.5 : 6.9;
            cost = full * (per * step_full + fixed) + (rem ? per * step_rem + fixed : 0.0);
        }
        if (splits > 1) cost += 2.8 + splits * (0.23 + 0.29 * partial_mb);
        if (tg == 2 && splits > 1) cost += 1.5;                // (what such a choice has to be estimated to gain: short GEMMs were up to 3 % slower)
        if (cost < best_cost) { best_cost = cost; best = {tg, splits, ks, cost}; }
    };
    for (int s = 1; s <= 16; ++s) {
        consider(4, s, 1);
        if (nst % 8 == 0) consider(4, s, 2);
        if (s <= most32) consider(2, s, 1);
    }
    return best;
}

// Token tiles of a launch.  A token tile's workgroups have an XCD of their own where the tiles are a multiple of eight, and its activations then come into one L2: seven tiles (15, 23, ..) of
// 32 tokens that leave every workgroup its CU take an eighth without tokens along.  us per forward, 7 / 8 tiles in both GEMMs: 2796 x 166 r = 78 at 196 tokens 15.4 / 14.9,
// 15 / 16: 2722 x 431 r = 207 at 461 18.6 / 18.0; 57 short forwards of seven and 8 k + 7 tiles 0.982 of the time on average, none above 1.014.  Past the line work counts: 17245 x 497
// r = 94 at 458 20.1 / 21.7; in parts (of which there are more than CUs soon) nothing is gained.
static int token_tiles(int batch, int tg, int splits, int n_rb)
{
    const int n = (batch + 16 * tg - 1) / (16 * tg), n_tiles = (n_rb + kPfWaves - 1) / kPfWaves;
    return tg == 2 && n % 8 == 7 && splits == 1 && (n + 1) * n_tiles <= device_cu_count() ? n + 1 : n;
}

static PfLayout pf_layout(int64_t d_out, int64_t d_in, int64_t r, int batch, bool plain)
{
    PfLayout L;
    L.m_pad = (int)round_up(batch, kPfTokens);
    L.k1 = (int)n_steps(d_in) * 64;
    L.k2 = (int)n_steps(r) * 64;
    L.n1_pad = (int)n_rowblocks(r) * kTileRows;
    L.n2_pad = (int)n_rowblocks(d_out) * kTileRows;
    const GemmTiling t1 = choose_tiling(batch, (int)n_rowblocks(r), (int)n_steps(d_in), L.n1_pad, plain);
    const GemmTiling t2 = choose_tiling(batch, (int)n_rowblocks(d_out), (int)n_steps(r), L.n2_pad, plain);
    L.tg1 = t1.tg; L.splits1 = t1.splits; L.ks1 = t1.ks;
    L.tg2 = t2.tg; L.splits2 = t2.splits; L.ks2 = t2.ks;
    if (opt(OPT_PF_TG1) >= 0) L.tg1 = opt(OPT_PF_TG1) == 2 ? 2 : 4;
    if (opt(OPT_PF_TG2) >= 0) L.tg2 = opt(OPT_PF_TG2) == 2 ? 2 : 4;
    if (opt(OPT_PF_SPLITS1) >= 0) L.splits1 = std::max(1, opt(OPT_PF_SPLITS1));
    if (opt(OPT_PF_SPLITS2) >= 0) L.splits2 = std::max(1, opt(OPT_PF_SPLITS2));
    if (opt(OPT_PF_KS1) >= 0) L.ks1 = opt(OPT_PF_KS1) == 2 ? 2 : 1;
    if (opt(OPT_PF_KS2) >= 0) L.ks2 = opt(OPT_PF_KS2) == 2 ? 2 : 1;
    // the in-workgroup split needs 64-token tiles and a reduction of whole groups of eight steps
    if (L.tg1 != 4 || n_steps(d_in) % 8 != 0) L.ks1 = 1;
    if (L.tg2 != 4 || n_steps(r) % 8 != 0) L.ks2 = 1;
    L.m_tiles1 = token_tiles(batch, L.tg1, L.splits1, (int)n_rowblocks(r));
    L.m_tiles2 = token_tiles(batch, L.tg2, L.splits2, (int)n_rowblocks(d_out));
    if (opt_flag(OPT_PF_VERBOSE))
        fprintf(stderr, "prefill tiling B=%d: gemm1 tg=%d tiles=%d splits=%d ks=%d, gemm2 tg=%d tiles=%d splits=%d ks=%d\n", batch, L.tg1, L.m_tiles1, L.splits1,
                L.ks1, L.tg2, L.m_tiles2, L.splits2, L.ks2);
    size_t o = 0;
    L.off_x = o; o += al256((size_t)L.m_pad * L.k1 * 2);
    L.off_t = o; o += al256((size_t)L.m_pad * L.k2 * 2);
    L.off_scale = o; o += al256((size_t)L.m_pad * 4);
    L.off_partial = o;
    size_t p1 = L.splits1 > 1 ? (size_t)L.splits1 * L.m_pad * L.n1_pad * 4 : 0;
    size_t p2 = L.splits2 > 1 ? (size_t)L.splits2 * L.m_pad * L.n2_pad * 4 : 0;
    o += al256(std::max(p1, p2));
    L.total = o;
    return L;
}

// The path's time on the tilings that it takes
double prefill_now_us(int64_t d_out, int64_t d_in, int64_t r, int batch)
{
    const int rb1 = (int)n_rowblocks(r), rb2 = (int)n_rowblocks(d_out);
    return 0.94 * (choose_tiling(batch, rb1, (int)n_steps(d_in), rb1 * kTileRows, false).us + choose_tiling(batch, rb2, (int)n_steps(r), rb2 * kTileRows, false).us) +
           0.67e-6 * batch * (double)(d_in + d_out);
}

// The path's time without what the caller's host side adds, as the exact path is costed against it (nq_api.hip).
double prefill_us(int64_t d_out, int64_t d_in, int64_t r, int batch)
{
    // (whole 64-token tiles, and the tilings among which the choice between the paths was fitted: a call that is exact stays so whatever is gained here)
    const int rb1 = (int)n_rowblocks(r), rb2 = (int)n_rowblocks(d_out), whole = (int)round_up(batch, kPfTokens);
    return 0.94 * (choose_tiling(whole, rb1, (int)n_steps(d_in), rb1 * kTileRows, false, 1).us +
                   choose_tiling(whole, rb2, (int)n_steps(r), rb2 * kTileRows, false, 1).us) + 0.67e-6 * batch * (double)(d_in + d_out);
}

size_t prefill_workspace_bytes(int64_t d_out, int64_t d_in, int64_t r, int batch, bool plain)
{
    return pf_layout(d_out, d_in, r, batch, plain).total;
}

template <int EPI, bool PLAIN>
static void launch_gemm(const GemmArgs& a, int tg, int ks, hipStream_t s)
{
    const dim3 grid(a.m_tiles * a.n_tiles, a.splits), block(64 * kPfWaves * ks);
    if (ks == 2) hipLaunchKernelGGL((prefill_gemm_kernel<EPI, 4, 2, PLAIN>), grid, block, 0, s, a);
    else if (tg == 4) hipLaunchKernelGGL((prefill_gemm_kernel<EPI, 4, 1, PLAIN>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((prefill_gemm_kernel<EPI, 2, 1, PLAIN>), grid, block, 0, s, a);
}

template <int EPI, bool PLAIN>
static int run_gemm(const GemmArgs& a, int tg, int ks, hipStream_t s)
{
    if (ks == 2 && (tg != 4 || a.nst % 8 != 0 || a.steps_per_split % 8 != 0)) {
        set_error("prefill: the in-workgroup split needs 64-token tiles and parts of whole groups of eight steps");
        return NQ_E_INVALID_ARG;
    }
    if (a.splits > 1) {
        launch_gemm<EPI_PARTIAL, PLAIN>(a, tg, ks, s);
        NQ_HIP(hipGetLastError());
        const size_t total = EPI == EPI_T ? (size_t)a.m_rows * (a.ldt / 16) : (size_t)a.m_rows * (a.n_pad / 4);
        hipLaunchKernelGGL((prefill_finalize_kernel<EPI, PLAIN>), dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, a);
    } else {
        launch_gemm<EPI, PLAIN>(a, tg, ks, s);
    }
    NQ_HIP(hipGetLastError());
    return NQ_OK;
}

// A product of a p-bit and a q-bit number has at most p + q bits, p where the other is a power of two, and fp16 holds 11.  Channels
// whose scale keeps every x of the type exact: of at most 3 significant bits for bf16 (8 bits), powers of two for fp16 and fp32
// (whose values may be 16-bit ones widened).  From one channel in sixteen on such a layer is taken one column at a time: with
// fewer, the pairs' rounding is at most 1.6 % more than that of the columns; general fp16 scales have one such channel in 256 or 1024.
__host__ __device__ static int plain_channel(uint16_t s, int x_dtype)
{
    return (s & 0x7FFFu) != 0 && (s & (x_dtype == NQ_BF16 ? 0xFFu : 0x3FFu)) == 0;
}
static __host__ __device__ bool plain_layer(int64_t channels, int64_t d_in) { return channels * 16 >= d_in; }

bool prefill_plain(const uint16_t* s_in, int64_t d_in, int x_dtype)
{
    int64_t n = 0;
    for (int64_t i = 0; i < d_in; ++i) n += plain_channel(s_in[i], x_dtype);
    return plain_layer(n, d_in);
}

__global__ void __launch_bounds__(1024) prefill_plain_kernel(const uint16_t* s_in, int d_in, int x_dtype, int* answer)
{
    __shared__ int sm[16];
    int n = 0;
    for (int i = threadIdx.x; i < d_in; i += 1024) n += plain_channel(s_in[i], x_dtype);
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int w = 1; w < 16; ++w) n += sm[w];
    *answer = plain_layer(n, d_in);
}

int launch_prefill_plain(const uint16_t* d_s_in, int64_t d_in, int x_dtype, int* answer)
{
    hipLaunchKernelGGL(prefill_plain_kernel, dim3(1), dim3(1024), 0, nullptr, d_s_in, (int)d_in, x_dtype, answer);
    NQ_HIP(hipGetLastError());
    return NQ_OK;
}

// width of a pre-scale workgroup: as many threads as the row has chunks of 16 columns for kPreHeld of them each
static int pre_threads(int lda)
{
    const int need = (lda / 16 + kPreHeld - 1) / kPreHeld;
    return std::min(kPreThreads, std::max(64, (need + 63) / 64 * 64));
}

template <bool PLAIN>
static int launch_prefill_as(const PrefillArgs& p, hipStream_t s)
{
    const PfLayout L = pf_layout(p.d_out, p.d_in, p.r, p.batch, PLAIN);
    char* ws = (char*)p.workspace;
    _Float16* xs = (_Float16*)(ws + L.off_x);
    _Float16* t = (_Float16*)(ws + L.off_t);
    float* tok_scale = (float*)(ws + L.off_scale);
    float* partial = (float*)(ws + L.off_partial);
    // |x''| < 2^13, so |t''| < d_in * 2^13; g brings that to <= 2^14, its pair sums to <= 2^15 (fp16 range 65504)
    int lg = 0;
    while (((int64_t)1 << lg) < p.d_in) ++lg;
    // (with a rank-wise scale, |s_mid| <= 2^mid_exp, T = X''V g s_mid stays within the same bound)
    const float g_t = ldexpf(1.0f, -(lg > 1 ? lg - 1 : 0) - (p.s_mid ? p.mid_exp : 0));

    // The token's power of two is clamped to 2^a_min .. 2^100: from max|x'| = 2^113 on x'' grows with it, up to 2^16 at 2^116 where fp16 and
    // with it the path's range end.  Sums of pairs are twice that, so they are clamped at 2^-101 (short of that only where the
    // token's factor 1 / (2^a g) would leave fp32).
    const bool room = 101 + (lg > 1 ? lg - 1 : 0) + (p.s_mid ? p.mid_exp : 0) <= 127;
    const int a_min = !PLAIN && room ? -101 : -100;
    const dim3 pgrid(p.batch), pblock(pre_threads(L.k1));
    if (p.x_dtype == NQ_F32)
        hipLaunchKernelGGL((prefill_prescale_kernel<NQ_F32, PLAIN>), pgrid, pblock, 0, s, p.x, p.s_in, (int)p.d_in, L.k1, g_t, a_min, xs, tok_scale);
    else if (p.x_dtype == NQ_F16)
        hipLaunchKernelGGL((prefill_prescale_kernel<NQ_F16, PLAIN>), pgrid, pblock, 0, s, p.x, p.s_in, (int)p.d_in, L.k1, g_t, a_min, xs, tok_scale);
    else
        hipLaunchKernelGGL((prefill_prescale_kernel<NQ_BF16, PLAIN>), pgrid, pblock, 0, s, p.x, p.s_in, (int)p.d_in, L.k1, g_t, a_min, xs, tok_scale);
    NQ_HIP(hipGetLastError());

    GemmArgs a{};
    a.m_pad = L.m_pad;
    a.batch = p.batch;
    a.partial = partial;
    // gemm1: T = X'' V
    a.act = xs; a.lda = L.k1; a.tiles = p.vt_tiles;
    a.t_out = t; a.ldt = L.k2; a.t_scale = g_t; a.mid_scale = p.s_mid;
    a.n_real = (int)p.r; a.n_rb = (int)n_rowblocks(p.r); a.nst = (int)n_steps(p.d_in);
    a.n_tiles = (a.n_rb + kPfWaves - 1) / kPfWaves;
    a.splits = L.splits1; a.steps_per_split = steps_per_split4(a.nst, a.splits, L.ks1);
    a.n_pad = L.n1_pad;
    a.m_tiles = L.m_tiles1;
    a.m_rows = a.m_tiles * 16 * L.tg1;
    int rc = run_gemm<EPI_T, PLAIN>(a, L.tg1, L.ks1, s);
    if (rc != NQ_OK) return rc;
    // gemm2: y = T U^T
    a.act = t; a.lda = L.k2; a.tiles = p.u_tiles;
    a.y_out = p.y; a.y_dtype = p.y_dtype; a.tok_scale = tok_scale; a.out_scale = p.s_out;
    a.n_real = (int)p.d_out; a.n_rb = (int)n_rowblocks(p.d_out); a.nst = (int)n_steps(p.r);
    a.n_tiles = (a.n_rb + kPfWaves - 1) / kPfWaves;
    a.splits = L.splits2; a.steps_per_split = steps_per_split4(a.nst, a.splits, L.ks2);
    a.n_pad = L.n2_pad;
    a.m_tiles = L.m_tiles2;
    a.m_rows = a.m_tiles * 16 * L.tg2;
    return run_gemm<EPI_Y, PLAIN>(a, L.tg2, L.ks2, s);
}

int launch_prefill(const PrefillArgs& p, hipStream_t s)
{
    return p.plain ? launch_prefill_as<true>(p, s) : launch_prefill_as<false>(p, s);
}

}  // namespace nq
