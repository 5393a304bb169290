// Stages of the streaming path for launches that are far from filling the chip: a layer on its own, or the few layers of
// one level of a decoder block (Section 3.1 Eq. 1 as two sign-matrix x vector products, Appendix E.2).  Such a launch is bound by latency:
// by the host, which takes 2.7 to 3 us per launch, and by the chain  input -> fixed point -> tiles -> sums -> store  of a workgroup.
//   - The workgroups of a stage quantise its input themselves where it is short: one launch instead of two.
//   - A row block is dealt out to several workgroups, which share an XCD and its L2: by groups of TOKENS first, because the fixed point of a workgroup's tokens is the
//     longest link of its chain and only tokens divide it, and by BIT PLANES: each streams the same tiles, multiplies PL of the eight planes (16
//     rows each) and finishes its own rows, so that nothing has to be added up between workgroups.
//   - More than eight tokens (batch 9 and more through the exact path) are dealt out in groups of up to eight as well.
//   - stage_layer_kernel: a small layer in ONE launch, every workgroup computing the whole of t for itself.
// The arithmetic is that of quantize_kernel and stage_split_kernel (nq_decode.hip) element for element: the same bits.
//
// Whole forwards, us per call: four launches (batch 1: two self-quantising ones) / two, planes dealt out / tokens and planes; what two launches cost the host is 6:
//   4096 x 4096 r = 1024   batch 1 11.1 / 8.9 / 8.9, 4 15.8 / 10.6 / 9.9, 8 22.8 / 13.3 / 10.6, 24 27.4 (dense path) / 15.4 / 11.8
//   5003 x 3001 r = 777    batch 6 25.0 / 13.4 / 10.4        1024 x 1024 r = 256   batch 1 10.4 / 8.0 (one launch) / 7.6
//   1408 x 21251 r = 999   batch 7 27.1 (planes) / 14.5      384 x 13516 r = 96    batch 8 23.9 / 11.7
// 150 random layers from 256 to 28672 a side at batch 1 to 8: 0.81 to 0.85 of the time of planes alone (geometric mean), none slower than their scatter.
#include <algorithm>

#include "nq_internal.h"
#include "nq_device.h"

namespace nq {

typedef const __attribute__((address_space(4))) QMeta* cptr_meta;

// A "unit" is what a wave quantises at a time: 64 chunks of 16 elements of one token, one per lane; in the one-launch kernel, whose
// vectors are so short that this would leave most waves idle, 64 groups of four (E = 4).  Up to 32768 elements are quantised by the workgroups of the stage,
// two units per wave of 16, which is also what LDS holds; at that length a launch of its own takes about as long, and the host one launch more
// (4096 x 4096 at batch 8 15.0 us without it, 14.8 with; 8192 wide at batch 4 20.4 and 21.0).
constexpr int kLoneMaxElements = 32768;
template <int W, int E> constexpr int lone_share_units() { return kLoneMaxElements / (64 * E) / W; }
// ... of a kernel that takes four at a time only where they are few
constexpr int kFewElements = 16384;
template <int W, int E> constexpr int along_units() { return (E == 4 ? kFewElements : kLoneMaxElements) / (64 * E) / W; }

template <int E> __host__ __device__ inline int lone_pieces(int nst) { return (nst + E - 1) / E; }      // units per token
// fixed point of a token in LDS: [step][chunk][slice][16 bytes], tokens 48 mod 256 bytes apart: the 15 (token, slice) operands of a
// 16-lane group fall on different banks
__host__ __device__ inline int lone_tok_bytes(int nst) { return nst * (int)kBqStepBytes + 48; }
// ints between the waves' sums: 16 modulo 32, because the four lanes that add up a result start at four waves
__host__ __device__ constexpr int lone_wave_ints(int ints) { return (ints + 15) / 32 * 32 + 16; }

// What the units of a launch's tokens leave in LDS: the bits of their largest magnitude and the sum of their q
struct LoneTokens {
    unsigned long long sum[8];
    uint32_t max[8];
};

__device__ __forceinline__ void lone_clear(LoneTokens* lt, int tid)
{
    if (tid < 8) {
        lt->sum[tid] = 0;
        lt->max[tid] = 0;
    }
}

__device__ __forceinline__ QMeta lone_meta(const LoneTokens* lt, int tok)
{
    const uint32_t m = lt->max[tok];
    const float step = exp2_int(step_exponent(m));
    QMeta mt;
    mt.two_step = m <= kMostBits ? 2.0 * (double)step : (double)__builtin_nanf("");
    mt.neg_qs = -(double)(long long)lt->sum[tok] * (double)step;
    return mt;
}

// The units of one wave: `n` consecutive ones, so that few tokens end inside its share.  Wave-uniform.
struct LoneShare {
    int n, tok, piece;
};
template <int W>
__device__ __forceinline__ LoneShare lone_share(int units, int pieces, int wave)
{
    const int per = (units + W - 1) / W, u0 = wave * per;
    LoneShare sh;
    sh.n = units - u0 < per ? (units - u0 > 0 ? units - u0 : 0) : per;
    // (the quotient is exact for the small integers that occur)
    sh.tok = __builtin_amdgcn_readfirstlane((int)(((float)u0 + 0.5f) * __builtin_amdgcn_rcpf((float)pieces)));
    sh.piece = u0 - sh.tok * pieces;
    return sh;
}
__device__ __forceinline__ void lone_next(LoneShare& sh, int pieces)
{
    if (++sh.piece == pieces) {
        sh.piece = 0;
        ++sh.tok;
    }
}

// The elements of a lane and their scales as they are in memory: requested for all of a wave's units before the first is looked at.
template <int E>
struct LoneRaw {
    v4u x[E / 4];                                           // 16-bit inputs: the first half
    unsigned int s[E / 2];
};

// Elements j0 .. j0 + E - 1 of token row `base`.  Rows lie at the alignment of an element, which global memory takes.  A lane whose elements
// reach past the row's end requests the row's last E, which lone_value() moves into place (rows shorter than E: one at a time).
template <int E>
__device__ __forceinline__ void lone_request(const QuantDesc& d, int64_t base, int j0, LoneRaw<E>& r)
{
    typedef unsigned int v2u __attribute__((ext_vector_type(2)));
    typedef v4u v4u_elem __attribute__((aligned(2)));
    typedef v2u v2u_elem __attribute__((aligned(2)));
    typedef const __attribute__((address_space(1))) v4u_elem* gptr_4;
    typedef const __attribute__((address_space(1))) v2u_elem* gptr_2;
    if (d.N < E) {
#pragma unroll
        for (int i = 0; i < E; ++i) {
            float f = 0.f;
            if (j0 + i < d.N) {
                f = load_as_float(d.x, d.dtype, base + j0 + i);
                if (d.scale) f *= half_bits_to_float(d.scale[j0 + i]);
            }
            r.x[i / 4][i & 3] = __builtin_bit_cast(unsigned int, f);
        }
        return;
    }
    const int j = j0 + E <= d.N ? j0 : d.N - E;
    if (d.scale) {
        if (E == 16) {
#pragma unroll
            for (int q = 0; q < E / 8; ++q) {
                const v4u s = ((gptr_4)(d.scale + j))[q];
#pragma unroll
                for (int i = 0; i < 4; ++i) r.s[(4 * q + i) % (E / 2)] = s[i];
            }
        } else {
            const v2u s = *(gptr_2)(d.scale + j);
            r.s[0] = s.x;
            r.s[1] = s.y;
        }
    }
    if (d.dtype == NQ_F32) {
#pragma unroll
        for (int q = 0; q < E / 4; ++q) r.x[q] = ((gptr_4)((const float*)d.x + base + j))[q];
    } else if (E == 16) {
#pragma unroll
        for (int q = 0; q < E / 8; ++q) r.x[q] = ((gptr_4)((const uint16_t*)d.x + base + j))[q];
    } else {
        const v2u h = *(gptr_2)((const uint16_t*)d.x + base + j);
        r.x[0].x = h.x;
        r.x[0].y = h.y;
    }
}

// ... as numbers times their scales; padding beyond N is zero
template <int E>
__device__ __forceinline__ void lone_value(const QuantDesc& d, const LoneRaw<E>& r, int j0, float v[E])
{
    const bool done = d.N < E, scaled = d.scale && !done;
    const auto convert = [&](auto value) {                  // (one loop per type, which is the same for the whole launch)
#pragma unroll
        for (int i = 0; i < E; ++i) {
            v[i] = value(i);
            if (scaled) v[i] = times_half(v[i], (uint16_t)(r.s[i / 2] >> (16 * (i & 1))));
        }
    };
    const auto half_of = [&](int i) { return (uint16_t)(r.x[i / 8][(i / 2) & 3] >> (16 * (i & 1))); };
    if (done || d.dtype == NQ_F32) convert([&](int i) { const unsigned int w = r.x[i / 4][i & 3]; return __builtin_bit_cast(float, w); });
    else if (d.dtype == NQ_F16) convert([&](int i) { return half_bits_to_float(half_of(i)); });
    else convert([&](int i) { return bf16_bits_to_float(half_of(i)); });
    const int past = j0 + E - d.N;                          // elements of the lane beyond the row's end
    if (!done && __builtin_amdgcn_ballot_w64(past > 0) != 0) {
#pragma unroll
        for (int k = E / 2; k >= 1; k /= 2) {
            const bool move = past > 0 && (past & k) != 0;
#pragma unroll
            for (int i = 0; i < E; ++i) v[i] = move ? (i + k < E ? v[(i + k) % E] : 0.f) : v[i];
        }
#pragma unroll
        for (int i = 0; i < E; ++i) v[i] = past >= E ? 0.f : v[i];
    }
}

// A wave's share of the units (value(c, token, first element, v): the lane's elements of unit c, scaled) -> fixed point in `bq`, all waves of the
// workgroup together.  *lt is cleared, and a barrier has passed since.
template <int W, int E, int kU, class Value>
__device__ __forceinline__ void lone_quantise(Value value, const LoneShare& share, int pieces, int nst, int lane, LoneTokens* lt, char* bq)
{
    float hv[kU][E];
    LoneShare sh = share;
    uint32_t m = 0;                                        // (as bits: magnitudes order like them, NaN above all)
#pragma unroll
    for (int c = 0; c < kU; ++c) {
        if (c < share.n) {
            value(c, sh.tok, (sh.piece * 64 + lane) * E, hv[c]);
#pragma unroll
            for (int i = 0; i < E; ++i) {
                const uint32_t a = __builtin_bit_cast(uint32_t, hv[c][i]) & 0x7fffffffu;
                m = a > m ? a : m;
            }
            if (c + 1 == share.n || sh.piece + 1 == pieces) {
                m = wave_reduce32(m, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
                if (lane == 0) atomicMax(&lt->max[sh.tok], m);
                m = 0;
            }
            lone_next(sh, pieces);
        }
    }
    __syncthreads();
    sh = share;
    int sum = 0;                                           // |q| <= 2^22, and kU E <= 64 of them: 2^28 at most
    static_assert(kU * E <= 64, "a lane's sum of q");
#pragma unroll
    for (int c = 0; c < kU; ++c) {
        if (c < share.n) {
            m = lt->max[sh.tok];
            const float inv_step = exp2_int(-step_exponent(m));
            char* const tok = bq + sh.tok * lone_tok_bytes(nst);
            const int e0 = sh.piece * 64 + lane;            // the lane's group of E elements
            if (E == 16) {
                float v[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) v[i] = hv[c][i % E];
                if (e0 < nst * 4) sum += quantize_chunk16(v, inv_step, (uint4*)tok + kSlices * e0, 1);
            } else if (e0 < nst * 16) {
                uint32_t hi, mid, lo;
                sum += quantize4(hv[c][0], hv[c][1], hv[c][2], hv[c][3], inv_step, hi, mid, lo);
                uint32_t* const dst = (uint32_t*)(tok + (e0 >> 2) * (kSlices * 16)) + (e0 & 3);
                dst[0] = hi;
                dst[4] = mid;
                dst[8] = lo;
            }
            if (c + 1 == share.n || sh.piece + 1 == pieces) {
                const long long total = wave_sum64(sum);
                if (lane == 0) atomicAdd(&lt->sum[sh.tok], (unsigned long long)total);
                sum = 0;
            }
            lone_next(sh, pieces);
        }
    }
    __syncthreads();
}

// Column n of column group cg is slice n % 3 of token 5 cg + n / 3; an unused one repeats the group's last used one (an LDS broadcast)
__device__ __forceinline__ void lone_column(int cg, int n, int batch, int& tok, int& slice)
{
    int used = 3 * (batch - 5 * cg);
    used = used > 15 ? 15 : (used < 1 ? 1 : used);
    const int col = n < used ? n : used - 1;
    tok = 5 * cg + col / 3;
    slice = col % 3;
    if (tok >= batch) tok = 0;
}

// sum_n b_n q_n of (token, row) from the sums of `waves` waves, by the four lanes of a quad together (all of them get it); `q`: the row's place in
// wave 0's region, slices 4 ints apart
template <int W>
__device__ __forceinline__ double lone_raw(const int* q, int wave_ints, int waves, int quad)
{
    int s[3] = {0, 0, 0};
#pragma unroll
    for (int w = 0; w < W; w += 4) {
        if (w + quad < waves) {
#pragma unroll
            for (int i = 0; i < 3; ++i) s[i] += q[(w + quad) * wave_ints + 4 * i];
        }
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        s[i] += __builtin_amdgcn_mov_dpp(s[i], 0xB1, 0xf, 0xf, true);          // quad_perm [1, 0, 3, 2]
        s[i] += __builtin_amdgcn_mov_dpp(s[i], 0x4E, 0xf, 0xf, true);          // quad_perm [2, 3, 0, 1]
    }
    return fma((double)s[0], 65536.0, fma((double)s[1], 256.0, (double)s[2]));
}

// How a launch of the kernel below is dealt out: `groups` groups of up to `per` tokens (even sizes), PL bit planes per workgroup.  A unit is a row block
// of a group; the 8 / PL workgroups of one are 8 apart, i.e. on one XCD, and so are the groups of a row block, which stream the same tiles through
// that XCD's L2 (`spread`: units dealt to all XCDs, where more groups than that leaves room for make the launch).
struct LoneDeal {
    int n_rb, tokens, per, groups, spread;
};

// ... the unit of workgroup k of XCD x (planes aside): a group of tokens and a place among the row blocks or items; false: none
__device__ __forceinline__ bool lone_place(const LoneDeal& d, int x, int k, int& group, int& at)
{
    group = 0;
    at = x + 8 * k;
    if (d.groups > 1) {
        const int by = d.spread ? d.n_rb : d.groups;
        if (d.spread) k = at;
        const int quot = __builtin_amdgcn_readfirstlane((int)(((float)k + 0.5f) * __builtin_amdgcn_rcpf((float)by)));      // (exact for the small integers that occur)
        group = d.spread ? quot : k - quot * by;
        at = d.spread ? k - quot * by : x + 8 * quot;
    }
    return at < d.n_rb && group < d.groups;
}

// ints between the row groups of a wave's sums of one bit plane in LDS: the columns in use (three per token) x 4 rows and a gap, 4 or 12 modulo 16,
// so that what a wave reads of four row groups and (lone_wave_ints) four waves falls on different banks
__host__ __device__ inline int along_row_ints(int per) { return 12 * per + 4 + 4 * (per & 1); }

// A stage whose workgroups quantise their own group's tokens (E elements of a lane at a time) and multiply PL bit planes of a row block by them.
// Bound by a chain of latencies, of which the fixed point was the longest: 32 elements per thread take 3.2 us, so tokens are dealt out before planes
// are.
// items: n_rb row blocks of several ops, or nullptr: those of the one op (q1, s1).
template <int NB, int PL, int W, int E>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(W / 4, W / 4)))
stage_along_kernel(const FusedItem* __restrict__ items, QuantDesc q1, StageDesc s1, LoneDeal d)
{
    constexpr int D = W == 8 ? 8 : 4, S = 8 / PL, kUnits = along_units<W, E>();
    extern __shared__ __align__(16) int lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, n = lane & 15;
    const int x = blockIdx.x & 7, j = blockIdx.x >> 3, p0 = j % S * PL;
    int group, at;
    if (!lone_place(d, x, j / S, group, at)) return;
    QuantDesc qd = q1;
    StageDesc sd = s1;
    int rb = at;
    if (items) {
        const FusedItem* e = items + at;
        rb = e->rb;
        qd = e->q;
        sd = e->s;
    }
    const int nst = sd.n_steps;
    const int64_t first = (int64_t)group * d.per;           // of the group's tokens
    const int batch = d.tokens - (int)first < d.per ? d.tokens - (int)first : d.per;
    const int row_ints = along_row_ints(d.per), wave_ints = lone_wave_ints(PL * 4 * row_ints);
    int* const red = lds;                                   // [W][PL][4 row groups][columns][4 rows]
    LoneTokens* const lt = (LoneTokens*)(lds + W * wave_ints);
    char* const bq = (char*)(lt + 1);
    const int pieces = lone_pieces<E>(nst), units = batch * pieces;

    const LoneShare share = lone_share<W>(units, pieces, wave);
    LoneRaw<E> raw[kUnits];
    lone_clear(lt, tid);
    {
        LoneShare sh = share;
#pragma unroll
        for (int c = 0; c < kUnits; ++c) {
            if (c < share.n) {
                lone_request(qd, (first + sh.tok) * qd.x_stride, (sh.piece * 64 + lane) * E, raw[c]);
                lone_next(sh, pieces);
            }
        }
    }
    // the first tiles: steps wave, wave + W, ... (a short share re-reads its last tile)
    const int cnt = (nst - wave + W - 1) / W;
    const int st0 = cnt > 0 ? wave : 0;
    const char* const a_base = (const char*)sd.tiles + (size_t)rb * nst * (kTileWords * 4);
    const uint32_t a_off = (uint32_t)(st0 * 1024 + lane * 16);
    uint32_t b_off[NB];
#pragma unroll
    for (int cg = 0; cg < NB; ++cg) {
        int tok, slice;
        lone_column(cg, n, batch, tok, slice);
        b_off[cg] = (uint32_t)(tok * lone_tok_bytes(nst) + (g * kSlices + slice) * 16 + st0 * (int)kBqStepBytes);
    }
    v4u wbuf[D];
#define NQ_ISSUE(k, i) wbuf[k] = load_global_v4u(a_base, a_off + (uint32_t)(i) * (W * 1024))
#pragma unroll
    for (int k = 0; k < D; ++k) NQ_ISSUE(k, k < cnt ? k : (cnt > 0 ? cnt - 1 : 0));
    // A thread finishes the same row of all of its tokens: that row's output scale, requested behind everything that is waited for sooner (and whether there
    // is one or not, so that those waits stay exact: ahead of the tiles, in a branch, it cost stage 2 of 4096 x 4096 at batch 1 0.3 of 4.2 us).
    constexpr int kRows = 16 * PL;
    static_assert(16 * W % kRows == 0, "whole tokens between a thread's results");
    const int row = (tid >> 2) % kRows, grow = rb * kTileRows + 16 * p0 + row;
    const uint16_t oscale = *(sd.out_scale ? (gptr_u16)sd.out_scale + (grow < sd.M ? grow : 0) : (gptr_u16)sd.tiles);
    __syncthreads();
    lone_quantise<W, E, kUnits>([&](int c, int, int j0, float v[E]) { lone_value(qd, raw[c], j0, v); }, share, pieces, nst, lane, lt, bq);

    uint32_t mask[PL];
#pragma unroll
    for (int p = 0; p < PL; ++p) mask[p] = 0x01010101u << (p0 + p);
    v4i acc[NB][PL];
#pragma unroll
    for (int cg = 0; cg < NB; ++cg)
#pragma unroll
        for (int p = 0; p < PL; ++p) acc[cg][p] = v4i{0, 0, 0, 0};
#define NQ_MAC(k, i)                                                                                              \
    do {                                                                                                          \
        v4u b[NB];                                                                                                \
        _Pragma("unroll") for (int cg = 0; cg < NB; ++cg) b[cg] = *(const v4u*)(bq + b_off[cg] + (i) * (W * (int)kBqStepBytes)); \
        _Pragma("unroll") for (int p = 0; p < PL; ++p) {                                                          \
            const v4i a = (v4i)(wbuf[k] & mask[p]);                                                               \
            _Pragma("unroll") for (int cg = 0; cg < NB; ++cg)                                                     \
                acc[cg][p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, (v4i)b[cg], acc[cg][p], 0, 0, 0);           \
        }                                                                                                         \
    } while (0)
    // (whole passes over the ring without a branch, so that the waits inside stay partial; then the last D to 2 D - 1 steps)
    int i0 = 0;
    for (; i0 + 2 * D <= cnt; i0 += D) {
#pragma unroll
        for (int k = 0; k < D; ++k) {
            NQ_MAC(k, i0 + k);
            NQ_ISSUE(k, i0 + k + D);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int k = 0; k < D; ++k) {
        if (i0 + k < cnt) {
            NQ_MAC(k, i0 + k);
            if (i0 + k + D < cnt) NQ_ISSUE(k, i0 + k + D);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int k = 0; k < D; ++k) {
        if (i0 + D + k < cnt) {
            NQ_MAC(k, i0 + D + k);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#undef NQ_MAC
#undef NQ_ISSUE
    // the waves' partial sums of every result
#pragma unroll
    for (int cg = 0; cg < NB; ++cg)
        if (n < (cg == 0 && NB > 1 ? 15 : 3 * d.per - 15 * cg)) {
#pragma unroll
            for (int p = 0; p < PL; ++p) *(v4i*)(red + wave * wave_ints + (p * 4 + g) * row_ints + (15 * cg + n) * 4) = acc[cg][p];
        }
    __syncthreads();
    const int quad = tid & 3, p = p0 + (row >> 4);
    const float scale = sd.out_scale ? half_bits_to_float(oscale) : 1.0f;
    const int64_t out0 = first * sd.out_stride + grow;
    for (int tok = (tid >> 2) / kRows; tok < batch; tok += 16 * W / kRows) {
        double sum = lone_raw<W>(red + (row >> 2) * row_ints + 12 * tok + (row & 3), wave_ints, W, quad);
        const QMeta mt = lone_meta(lt, tok);
        if (quad != 0 || grow >= sd.M) continue;
        if (p == 7) sum = -sum;                            // bit 7 of an int8 is worth -128
        const double val = fma(sum, __builtin_ldexp(mt.two_step, -p), mt.neg_qs);     // exact
        store_out(sd.out, sd.out_dtype, (size_t)(out0 + (int64_t)tok * sd.out_stride), (float)val * scale, sd.out_scale != nullptr);
    }
}

// The same on an input that a launch of its own has quantised (too long to quantise along), dealt out alike.
template <int NB, int PL, int W>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(W / 4, W / 4)))
stage_lone_kernel(const FusedItem* __restrict__ items, StageDesc s1, LoneDeal d)
{
    constexpr int D = W == 8 ? 8 : 4, S = 8 / PL, kRows = 16 * PL;
    extern __shared__ __align__(16) int lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, n = lane & 15;
    const int x = blockIdx.x & 7, j = blockIdx.x >> 3, p0 = j % S * PL;
    int group, at;
    if (!lone_place(d, x, j / S, group, at)) return;
    StageDesc sd = s1;
    int rb = at;
    if (items) {
        const FusedItem* e = items + at;
        rb = e->rb;
        sd = e->s;
    }
    const int nst = sd.n_steps;
    const int64_t first = (int64_t)group * d.per;           // of the group's tokens
    const int batch = d.tokens - (int)first < d.per ? d.tokens - (int)first : d.per;
    const int row_ints = along_row_ints(d.per), wave_ints = lone_wave_ints(PL * 4 * row_ints);
    const char* const bq0 = (const char*)sd.bq + first * nst * kBqStepBytes;
    int* const red = lds;                                   // [W][PL][4 row groups][columns][4 rows]
    // the first tiles: steps wave, wave + W, ... (a short share re-reads its last tile)
    const int cnt = (nst - wave + W - 1) / W;
    const int st0 = cnt > 0 ? wave : 0;
    const char* const a_base = (const char*)sd.tiles + (size_t)rb * nst * (kTileWords * 4);
    const uint32_t a_off = (uint32_t)(st0 * 1024 + lane * 16);
    uint32_t b_off[NB];
#pragma unroll
    for (int cg = 0; cg < NB; ++cg) {
        int tok, slice;
        lone_column(cg, n, batch, tok, slice);
        b_off[cg] = (uint32_t)tok * ((uint32_t)nst * kBqStepBytes) + (uint32_t)(bq_piece(g, slice) * 16);
    }
    v4u wbuf[D], bbuf[D][NB];
#define NQ_ISSUE(k, i)                                                                                            \
    do {                                                                                                          \
        wbuf[k] = load_global_v4u(a_base, a_off + (uint32_t)(i) * (W * 1024));                                    \
        _Pragma("unroll") for (int cg = 0; cg < NB; ++cg)                                                         \
            bbuf[k][cg] = load_global_v4u(bq0, b_off[cg] + (uint32_t)(st0 + (i) * W) * kBqStepBytes);             \
    } while (0)
#pragma unroll
    for (int k = 0; k < D; ++k) NQ_ISSUE(k, k < cnt ? k : (cnt > 0 ? cnt - 1 : 0));
    static_assert(16 * W % kRows == 0, "whole tokens between a thread's results");
    const int row = (tid >> 2) % kRows, grow = rb * kTileRows + 16 * p0 + row, tok0 = wave * 16 / kRows;       // (a wave's 16 results are one token's)
    const uint16_t oscale = *(sd.out_scale ? (gptr_u16)sd.out_scale + (grow < sd.M ? grow : 0) : (gptr_u16)sd.tiles);
    const auto token_meta = [&](int tok) {
        const cptr_meta m = (cptr_meta)sd.meta + first + (tok < batch ? tok : 0);
        return QMeta{m->two_step, m->neg_qs};
    };
    QMeta meta = token_meta(tok0);

    uint32_t mask[PL];
#pragma unroll
    for (int p = 0; p < PL; ++p) mask[p] = 0x01010101u << (p0 + p);
    v4i acc[NB][PL];
#pragma unroll
    for (int cg = 0; cg < NB; ++cg)
#pragma unroll
        for (int p = 0; p < PL; ++p) acc[cg][p] = v4i{0, 0, 0, 0};
#define NQ_MAC(k, i)                                                                                              \
    do {                                                                                                          \
        _Pragma("unroll") for (int p = 0; p < PL; ++p) {                                                          \
            const v4i a = (v4i)(wbuf[k] & mask[p]);                                                               \
            _Pragma("unroll") for (int cg = 0; cg < NB; ++cg)                                                     \
                acc[cg][p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, (v4i)bbuf[k][cg], acc[cg][p], 0, 0, 0);     \
        }                                                                                                         \
    } while (0)
    // (whole passes over the ring without a branch, so that the waits inside stay partial; then the last D to 2 D - 1 steps)
    int i0 = 0;
    for (; i0 + 2 * D <= cnt; i0 += D) {
#pragma unroll
        for (int k = 0; k < D; ++k) {
            NQ_MAC(k, i0 + k);
            NQ_ISSUE(k, i0 + k + D);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int k = 0; k < D; ++k) {
        if (i0 + k < cnt) {
            NQ_MAC(k, i0 + k);
            if (i0 + k + D < cnt) NQ_ISSUE(k, i0 + k + D);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int k = 0; k < D; ++k) {
        if (i0 + D + k < cnt) {
            NQ_MAC(k, i0 + D + k);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#undef NQ_MAC
#undef NQ_ISSUE
    // the waves' partial sums of every result
#pragma unroll
    for (int cg = 0; cg < NB; ++cg)
        if (n < (cg == 0 && NB > 1 ? 15 : 3 * d.per - 15 * cg)) {
#pragma unroll
            for (int p = 0; p < PL; ++p) *(v4i*)(red + wave * wave_ints + (p * 4 + g) * row_ints + (15 * cg + n) * 4) = acc[cg][p];
        }
    __syncthreads();
    const int quad = tid & 3, p = p0 + (row >> 4);
    const float scale = sd.out_scale ? half_bits_to_float(oscale) : 1.0f;
    const int64_t out0 = first * sd.out_stride + grow;
    for (int tok = tok0; tok < batch; tok += 16 * W / kRows) {
        const QMeta mt = meta;
        meta = token_meta(tok + 16 * W / kRows);
        double sum = lone_raw<W>(red + (row >> 2) * row_ints + 12 * tok + (row & 3), wave_ints, W, quad);
        if (quad != 0 || grow >= sd.M) continue;
        if (p == 7) sum = -sum;                            // bit 7 of an int8 is worth -128
        const double val = fma(sum, __builtin_ldexp(mt.two_step, -p), mt.neg_qs);     // exact
        store_out(sd.out, sd.out_dtype, (size_t)(out0 + (int64_t)tok * sd.out_stride), (float)val * scale, sd.out_scale != nullptr);
    }
}

// ---------------------------------------------------------------------------------------------
// A small layer in one launch: every workgroup computes the whole of t (its stage-1 tiles are few and come from L2), keeps it in LDS,
// quantises it and finishes its own PL bit planes of one row block of stage 2.  Workgroup 0 also stores t.
// Bound by its chain of latencies; adding up the waves' sums of t was the longest link (2.4 of 8.0 us at 1024 x 1024 r = 256): all eight planes pass through LDS at once, in
// the columns that are in use, and t's largest magnitude is taken where t is: 7.6 us.
// ---------------------------------------------------------------------------------------------
constexpr int kLayerWaves = 16, kLayerTokens = 5;       // tokens: one column group of 15 columns, three per token, is all that the kernel has

template <int PL>
__global__ void __launch_bounds__(64 * kLayerWaves) __attribute__((amdgpu_waves_per_eu(4, 4)))
stage_layer_kernel(QuantDesc qx, StageDesc s1, QuantDesc qt, StageDesc s2, int n_rb, int batch, int t_off, int bqt_off)
{
    constexpr int NB = 1, W = kLayerWaves, D = 4, S = 8 / PL, kRows = 16 * PL;
    extern __shared__ __align__(16) int lds[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, n = lane & 15;
    const int j = blockIdx.x >> 3;
    const int rb2 = (blockIdx.x & 7) + 8 * (j / S), p0 = j % S * PL;
    if (rb2 >= n_rb) return;
    int* const red = lds;
    const int row_ints = along_row_ints(batch), wave_ints1 = lone_wave_ints(32 * row_ints), wave_ints2 = lone_wave_ints(PL * 4 * row_ints);
    LoneTokens* const lt = (LoneTokens*)(lds + W * wave_ints1);              // of x, then of t
    char* const bq = (char*)(lt + 2);
    float* const t_s = (float*)((char*)lds + t_off);                         // [batch][t stride]
    char* const bqt = (char*)lds + bqt_off;
    const int nst1 = s1.n_steps, nst2 = s2.n_steps;
    const int pieces1 = lone_pieces<4>(nst1), pieces2 = lone_pieces<4>(nst2);

    const LoneShare share1 = lone_share<W>(batch * pieces1, pieces1, wave), share2 = lone_share<W>(batch * pieces2, pieces2, wave);
    LoneRaw<4> raw[lone_share_units<W, 4>()];
    lone_clear(lt, tid);
    lone_clear(lt + 1, tid);
    {
        LoneShare sh = share1;
#pragma unroll
        for (int c = 0; c < lone_share_units<W, 4>(); ++c) {
            if (c < share1.n) {
                lone_request(qx, (int64_t)sh.tok * qx.x_stride, (sh.piece * 64 + lane) * 4, raw[c]);
                lone_next(sh, pieces1);
            }
        }
    }
    // stage 1: w1 waves per row block, all eight planes
    const int n_rb1 = (s1.M + kTileRows - 1) / kTileRows;
    int wl = 4;
    while ((W >> wl) < n_rb1) --wl;
    const int w1 = 1 << wl, rb1 = wave >> wl, part = wave & (w1 - 1);
    const int cnt1 = rb1 < n_rb1 ? (nst1 - part + w1 - 1) >> wl : 0;
    const int cnt2 = (nst2 - wave + W - 1) / W;
    const char* const a1 = (const char*)s1.tiles + (size_t)(rb1 < n_rb1 ? rb1 : 0) * nst1 * (kTileWords * 4) + (cnt1 > 0 ? part : 0) * 1024 + lane * 16;
    const char* const a2 = (const char*)s2.tiles + (size_t)rb2 * nst2 * (kTileWords * 4) + (cnt2 > 0 ? wave : 0) * 1024 + lane * 16;
    v4u wbuf[D];
#pragma unroll
    for (int k = 0; k < D; ++k) wbuf[k] = load_global_v4u(a1, (uint32_t)((k < cnt1 ? k : (cnt1 > 0 ? cnt1 - 1 : 0)) * w1) * 1024);
    // the output scale of the row that a thread finishes
    static_assert(16 * W % kRows == 0, "whole tokens between a thread's results");
    const int row2 = (tid >> 2) % kRows, grow = rb2 * kTileRows + 16 * p0 + row2;
    const uint16_t oscale = *(s2.out_scale ? (gptr_u16)s2.out_scale + (grow < s2.M ? grow : 0) : (gptr_u16)s2.tiles);
    __syncthreads();
    lone_quantise<W, 4, lone_share_units<W, 4>()>([&](int c, int, int j0, float v[4]) { lone_value(qx, raw[c], j0, v); }, share1, pieces1, nst1, lane, lt, bq);
    uint32_t b1[NB], b2[NB];
#pragma unroll
    for (int cg = 0; cg < NB; ++cg) {
        int tok, slice;
        lone_column(cg, n, batch, tok, slice);
        b1[cg] = (uint32_t)(tok * lone_tok_bytes(nst1) + (g * kSlices + slice) * 16);
        b2[cg] = (uint32_t)(tok * lone_tok_bytes(nst2) + (g * kSlices + slice) * 16);
    }
    {
        v4i acc[NB][8];
#pragma unroll
        for (int cg = 0; cg < NB; ++cg)
#pragma unroll
            for (int p = 0; p < 8; ++p) acc[cg][p] = v4i{0, 0, 0, 0};
        for (int i0 = 0; i0 < cnt1; i0 += D) {
#pragma unroll
            for (int k = 0; k < D; ++k) {
                if (i0 + k < cnt1) {
                    v4u b[NB];
#pragma unroll
                    for (int cg = 0; cg < NB; ++cg) b[cg] = *(const v4u*)(bq + b1[cg] + (part + (i0 + k) * w1) * (int)kBqStepBytes);
                    mac_tile<NB>(acc, wbuf[k], b);
                    if (i0 + k + D < cnt1) wbuf[k] = load_global_v4u(a1, (uint32_t)((i0 + k + D) * w1) * 1024);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        // the first tiles of stage 2 are requested before stage 1's sums are added up
#pragma unroll
        for (int k = 0; k < D; ++k) wbuf[k] = load_global_v4u(a2, (uint32_t)((k < cnt2 ? k : (cnt2 > 0 ? cnt2 - 1 : 0)) * W) * 1024);
        // the waves' partial sums of every result, all planes at once; t, scaled, and its largest magnitude from there
        if (n < 3 * batch) {
#pragma unroll
            for (int p = 0; p < 8; ++p) *(v4i*)(red + wave * wave_ints1 + (p * 4 + g) * row_ints + n * 4) = acc[0][p];
        }
        __syncthreads();
        const int quad = tid & 3;
        for (int idx = tid >> 2; idx < n_rb1 * kTileRows * batch; idx += 16 * W) {
            const int row = idx % kTileRows, tr = idx / kTileRows, tok = tr % batch, rb = tr / batch, p = row >> 4;     // (a wave's token is one)
            const int k = rb * kTileRows + row;
            double raw = lone_raw<W>(red + (rb << wl) * wave_ints1 + (row >> 2) * row_ints + 12 * tok + (row & 3), wave_ints1, w1, quad);
            if (p == 7) raw = -raw;
            const QMeta mt = lone_meta(lt, tok);
            const float t = (float)fma(raw, __builtin_ldexp(mt.two_step, -p), mt.neg_qs);
            float f = 0.f;
            if (k < s1.M) {
                f = t;
                if (qt.scale) f *= half_bits_to_float(((gptr_u16)qt.scale)[k]);
                if (quad == 0) {
                    t_s[tok * qt.x_stride + k] = f;
                    if (blockIdx.x == 0) ((float*)s1.out)[(size_t)tok * s1.out_stride + k] = t;
                }
            }
            const uint32_t m = wave_reduce32(__builtin_bit_cast(uint32_t, f) & 0x7fffffffu, [](uint32_t a, uint32_t b) { return a > b ? a : b; });
            if (lane == 0) atomicMax(&lt[1].max[tok], m);
        }
    }
    __syncthreads();
    // t -> fixed point (as the second half of lone_quantise; from LDS, so without registers for a share)
    {
        LoneShare sh = share2;
        int sum = 0;
#pragma unroll 1
        for (int c = 0; c < share2.n; ++c) {
            const float inv_step = exp2_int(-step_exponent(lt[1].max[sh.tok]));
            const int e0 = sh.piece * 64 + lane;
            if (e0 < nst2 * 16) {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = 4 * e0 + i < qt.N ? t_s[sh.tok * qt.x_stride + 4 * e0 + i] : 0.f;
                uint32_t hi, mid, lo;
                sum += quantize4(v[0], v[1], v[2], v[3], inv_step, hi, mid, lo);
                uint32_t* const dst = (uint32_t*)(bqt + sh.tok * lone_tok_bytes(nst2) + (e0 >> 2) * (kSlices * 16)) + (e0 & 3);
                dst[0] = hi;
                dst[4] = mid;
                dst[8] = lo;
            }
            if (c + 1 == share2.n || sh.piece + 1 == pieces2) {
                const long long total = wave_sum64(sum);
                if (lane == 0) atomicAdd(&lt[1].sum[sh.tok], (unsigned long long)total);
                sum = 0;
            }
            lone_next(sh, pieces2);
        }
    }
    __syncthreads();
    // stage 2: all waves on PL planes of this workgroup's row block
    uint32_t mask[PL];
#pragma unroll
    for (int p = 0; p < PL; ++p) mask[p] = 0x01010101u << (p0 + p);
    v4i acc[NB][PL];
#pragma unroll
    for (int cg = 0; cg < NB; ++cg)
#pragma unroll
        for (int p = 0; p < PL; ++p) acc[cg][p] = v4i{0, 0, 0, 0};
    for (int i0 = 0; i0 < cnt2; i0 += D) {
#pragma unroll
        for (int k = 0; k < D; ++k) {
            if (i0 + k < cnt2) {
                v4u b[NB];
#pragma unroll
                for (int cg = 0; cg < NB; ++cg) b[cg] = *(const v4u*)(bqt + b2[cg] + (wave + (i0 + k) * W) * (int)kBqStepBytes);
#pragma unroll
                for (int p = 0; p < PL; ++p) {
                    const v4i a = (v4i)(wbuf[k] & mask[p]);
#pragma unroll
                    for (int cg = 0; cg < NB; ++cg) acc[cg][p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, (v4i)b[cg], acc[cg][p], 0, 0, 0);
                }
                if (i0 + k + D < cnt2) wbuf[k] = load_global_v4u(a2, (uint32_t)((i0 + k + D) * W) * 1024);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    if (n < 3 * batch) {
#pragma unroll
        for (int p = 0; p < PL; ++p) *(v4i*)(red + wave * wave_ints2 + (p * 4 + g) * row_ints + n * 4) = acc[0][p];
    }
    __syncthreads();
    const int quad = tid & 3, p = p0 + (row2 >> 4);
    const float scale = s2.out_scale ? half_bits_to_float(oscale) : 1.0f;
    for (int tok = (tid >> 2) / kRows; tok < batch; tok += 16 * W / kRows) {
        double raw = lone_raw<W>(red + (row2 >> 2) * row_ints + 12 * tok + (row2 & 3), wave_ints2, W, quad);
        if (quad != 0 || grow >= s2.M) continue;
        if (p == 7) raw = -raw;
        const QMeta mt = lone_meta(lt + 1, tok);
        const double val = fma(raw, __builtin_ldexp(mt.two_step, -p), mt.neg_qs);     // exact
        store_out(s2.out, s2.out_dtype, (size_t)tok * s2.out_stride + grow, (float)val * scale, s2.out_scale != nullptr);
    }
}

// Bit planes of a workgroup: as many workgroups per row block as give every CU at most one (a second round of workgroups costs more than
// the planes: 86 row blocks at batch 4 14.2 us with two planes each, 10.7 with four).
int lone_planes(int n_rb)
{
    int pl = 1;
    while (pl < 8 && n_rb * (8 / pl) > device_cu_count()) pl *= 2;
    return pl;
}

constexpr size_t kLoneLdsBytes = 160 * 1024;            // of a CU
// More than eight tokens of one op on a quantised input are dealt out in groups of at most eight, of even sizes.
static int lone_group(int batch) { return (batch + (batch + 7) / 8 - 1) / ((batch + 7) / 8); }
static int lone_groups(int batch) { return (batch + 7) / 8; }

// A form of the launch that quantises along
struct AlongForm {
    LoneDeal d;
    int pl, w, e;
    size_t lds;
};

static size_t along_lds_bytes(int pl, int w, int steps, int per)
{
    return (size_t)w * lone_wave_ints(pl * 4 * along_row_ints(per)) * 4 + sizeof(LoneTokens) + (size_t)per * lone_tok_bytes(steps);
}

// Time of a launch, back to back with others (us), fitted to 43000 timings: 1 to 224 row blocks of 4 to 448 steps at 1 to 64 tokens in every form that
// fits; 3.4 % off on average, its choices 1.2 % slower than the best of each, the timings' own scatter included.  Beside the launch and the chain's fixed part
// (3.3): the vector instructions of the fixed point on the busiest SIMD (a lane's element 18 ns) and its reductions (a wave's part of a token 54), the matrix
// instructions and their masks there (13 ns each), the sums passed through LDS, and what workgroups cost each other.
static double along_us(const AlongForm& f, int steps)
{
    const int s = 8 / f.pl, pieces = (steps + f.e - 1) / f.e, units = f.d.per * pieces, share = (units + f.w - 1) / f.w;
    const int simd = units >= f.w ? share * (f.w / 4) : (units + 3) / 4;
    const int results = 16 * f.pl * f.d.per;
    int parts = 0;                                          // parts of tokens that waves reduce
    for (int u = 0; u < units; u += share) parts += (std::min(units, u + share) - 1) / pieces - u / pieces + 1;
    return 3.34 + 0.0184 * simd * f.e + (f.e == 4 ? 0.40 * share : 0.52) + 0.054 * ((parts + 3) / 4) + 0.013 * 0.25 * steps * f.pl * (f.d.per > 5 ? 2 : 1) + 0.002 * steps +
           0.0141 / 1024 * f.w * f.pl * 192 * f.d.per + 0.51 / 256 * f.d.n_rb * f.d.groups * s + 0.175 * ((results + 16 * f.w - 1) / (16 * f.w)) + (f.w == 8 ? 0.30 : 0.0);
}

// ... what it takes longer on the row blocks of several layers, by 11900 timings of plans of two and four layers, 4 to 128 row blocks of 4 to 128 steps at 1 to 8 tokens: there the
// estimate alone dealt out tokens and kept planes together for gains of hundredths, and plans of 32 to 48 row blocks at 2 to 4 tokens had become slower than with all tokens in a
// workgroup of two planes (five layers 11008 x 2048 r = 896, 2 tokens: two planes 13.0, as estimated alone 13.4).  Choices 0.28 % slower than the best of each plan, without it 0.54 %.
static double along_listed_us(const AlongForm& f)
{
    return (f.e == 4 ? 0.03 : 0.0) + (f.pl == 8 ? 0.60 : f.pl == 4 ? 0.28 : f.pl == 2 ? 0.12 : 0.0);
}

// The form of a launch: among those with at most one workgroup per CU, on their XCD (dealt to all XCDs only where more than eight tokens need it), whose
// fixed point and sums fit LDS, the one of the least estimated time.  us per launch, stage 1 of 8 row blocks of 64 steps at 24 tokens 8.4 with groups of eight and one
// plane, 6.7 with groups of three and two; 28 of 448 steps at 4 tokens 14.6 after a quantisation launch of 6.2, 14.8 with it.
static bool along_form_now(int n_rb, int steps, int tokens, bool listed, AlongForm* best)
{
    const int cus = device_cu_count(), slots = cus / 8 / ((n_rb + 7) / 8), asked = opt(OPT_LONE_FORM);
    double best_us = 1e30;
    for (int most = 8; most >= 1; --most) {
        const int groups = (tokens + most - 1) / most, per = (tokens + groups - 1) / groups;
        if (per != most || per * lone_pieces<16>(steps) > kLoneMaxElements / 1024) continue;
        for (int pl = 8; pl >= 1; pl /= 2)
            for (int w = 16; w >= 8; w /= 2) {
                if (w == 8 ? pl < 8 : per > 5) continue;
                for (int e = w == 16 && per * lone_pieces<4>(steps) <= kFewElements / 256 ? 4 : 16; e <= 16; e *= 4) {
                    const bool spread = 8 / pl * groups > slots;
                    if (asked >= 0 ? asked != 100 * per + 10 * pl + (w == 8 ? 2 : e == 4 ? 1 : 0) : spread && (tokens <= 8 || n_rb * groups * (8 / pl) > cus)) continue;
                    const AlongForm f = {LoneDeal{n_rb, tokens, per, groups, spread}, pl, w, e, along_lds_bytes(pl, w, steps, per)};
                    if (f.lds > kLoneLdsBytes) continue;
                    const double us = along_us(f, steps) + (listed ? along_listed_us(f) : 0.0);
                    if (us < best_us) { best_us = us; *best = f; }
                }
            }
    }
    return best_us < 1e30;
}

// (A call asks for the forms of two stages, twice each: 2 us of a host that takes 6 for the call.  The answer depends on nothing but the four arguments.)
static bool along_form(int n_rb, int steps, int tokens, bool listed, AlongForm* best)
{
    if (opt(OPT_LONE_FORM) >= 0) return along_form_now(n_rb, steps, tokens, listed, best);
    struct Known {
        int n_rb, steps, tokens;
        bool listed, fits;
        AlongForm form;
    };
    static thread_local Known known[64];                   // (all zero: no launch has no row blocks)
    Known& k = known[(unsigned)(n_rb * 31 + steps * 7 + tokens) % 64];
    if (k.n_rb != n_rb || k.steps != steps || k.tokens != tokens || k.listed != listed) {
        k = Known{n_rb, steps, tokens, listed, false, {}};
        k.fits = along_form_now(n_rb, steps, tokens, listed, &k.form);
    }
    if (k.fits) *best = k.form;
    return k.fits;
}

// Whether the workgroups of such a launch quantise its input themselves.  Where every row block finds two CUs and more, wherever that fits.  Whole row
// blocks per workgroup (more than half as many as CUs) leave nothing to deal out, which pays for one or two tokens and for short
// inputs of more; past that the launch of its own is the faster one.  us per plan, with a launch of its own / along, stage 2 of 224 row blocks: batch 2 r = 2048 12.1 / 11.2, r = 6144 16.8 / 14.4;
// batch 3 r = 1024 11.4 / 11.2, r = 2048 12.0 / 12.1, past the line r = 4096 13.3 / 14.4; batch 4 r = 1024 11.5 / 11.6, past it r = 2048 12.2 / 12.6; batch 5 r = 1024
// 12.3 / 12.8, past it r = 2048 12.9 / 14.3; batch 8 r = 1024 15.1 / 15.6, but stage 1 of as many of three layers, d_in = 1024, batch 5 to 8, 0.97 to 0.99 of the time.
// (132 to 256 row blocks and lone forwards alike.)
bool lone_selfq(int max_steps, int n_rb, int batch)
{
    AlongForm f;
    if (opt(OPT_LONE_FORM) >= 0) return opt(OPT_LONE_FORM) % 10 < 3;
    if (lone_planes(n_rb * lone_groups(batch)) == 8) {
        const int per = lone_group(batch);
        if (lone_pieces<16>(max_steps) > (per <= 2 ? 12 / per : per == 3 ? 2 : 1)) return false;
    }
    return along_form(n_rb, max_steps, batch, false, &f);
}

// The same for the launches of a plan, which quantise along where they did when whole groups of eight tokens were the only ones: what a plan does is part of its answers
// (nq_plan_schedules, and the times of nq_plan_forward_timed, where a launch that is not there takes none).  The line that was drawn then: the fixed point of all tokens in LDS beside the
// sums of 8 (whole row blocks) or 16 waves, 1088 bytes for each plane and column group of up to four that pass at a time.
bool lone_plan_selfq(int max_steps, int n_rb, int batch)
{
    const int pl = lone_planes(n_rb), nb = batch <= 5 ? 1 : 2;
    const int most = pl < 8 ? kLoneMaxElements / 1024 / batch : batch <= 2 ? 12 / batch : batch == 3 ? 2 : 1;
    const size_t sums = (size_t)(pl == 8 ? 8 : 16) * std::min(nb * pl, 4) * 1088;
    return lone_pieces<16>(max_steps) <= most && sums + sizeof(LoneTokens) + (size_t)batch * lone_tok_bytes(max_steps) <= kLoneLdsBytes && lone_selfq(max_steps, n_rb, batch);
}

// Up to half as many pairs of row block and group of eight tokens as CUs: several workgroups share every pair.
bool lone_shared_pairs(int n_rb, int batch) { return 2 * n_rb * lone_groups(batch) <= device_cu_count(); }

// Whether a stage of more than eight tokens is faster dealt out here than in the groups of 16 of nq_exact.hip: where two workgroups or more share a pair (of 600 stages of 24 to 128
// pairs one was slower).  Rows that do not start 16-byte aligned or end inside 16 elements, which the quantisation launch in front of the groups of 16 takes two to three us longer for,
// also up to one pair per CU where the workgroups quantise along (16 steps), and of 32 to 64 steps up to five pairs to eight CUs (four row blocks and fewer, and groups of
// five tokens: one per CU).  us per stage with its input's fixed point, groups of 16 / dealt out, by pairs (row blocks, steps, tokens): 2 (1, 7, 15) 6.6 / 4.2; 20 (5, 48, 30) 9.3 / 5.7; 32 (2, 162, 127) 20.5 / 9.6; 60
// (10, 4, 48) 6.5 / 5.0; 84 (6, 199, 107) 22.5 / 18.6; 120 (40, 26, 22) 9.1 / 7.1; past it 144 (72, 4, 16) 6.9 / 7.2, 165 (5, 23, 258) 9.8 / 11.3, 225 (15, 127, 114) 19.0 / 19.4; ragged rows
// 40 (4, 9, 78) 9.6 / 5.1, 128 (16, 34, 64) 12.2 / 8.2, 140 (5, 11, 217) 10.7 / 6.7, 236 (118, 44, 10) 12.8 / 11.8, past it 290 (5, 5, 459) 11.1 / 18.3, 207 (9, 161, 183) 18 / 20.  Of 540 forwards with one such stage
// of 128 to 256 pairs: 16 steps and fewer all 0 to 3.9 us faster dealt out, 20 to 28 steps 0.3 to 2.5 slower, 32 to 64 steps 0.2 to 3 faster up to those lines and mostly 0.3 to 1.4
// slower past them.
bool lone_deals_out(int n_rb, int steps, bool whole, int batch)
{
    const int pairs = n_rb * lone_groups(batch), cus = device_cu_count();
    return lone_shared_pairs(n_rb, batch) || (!whole && ((steps <= 16 && pairs <= cus) || (steps >= 32 && steps <= 64 && 8 * pairs <= (n_rb <= 4 || lone_group(batch) <= 5 ? 8 : 5) * cus)));
}

template <int NB, int PL, int W, int E>
static int launch_along_t(const FusedItem* d_items, const QuantDesc& q, const StageDesc& sd, const AlongForm& f, hipStream_t s)
{
    NQ_ALLOW_LDS((stage_along_kernel<NB, PL, W, E>), kLoneLdsBytes);
    const int units = f.d.spread ? (f.d.n_rb * f.d.groups + 7) / 8 : (f.d.n_rb + 7) / 8 * f.d.groups;       // of an XCD
    NQ_LAUNCH((stage_along_kernel<NB, PL, W, E>), dim3((unsigned)(8 * units * (8 / PL))), dim3(64 * W), f.lds, s, d_items, q, sd, f.d);
    NQ_HIP(hipGetLastError());
    return NQ_OK;
}

// One stage on its n_rb row blocks, with the quantisation of its input (d_items == nullptr: of the one op).
int launch_lone_selfq(const FusedItem* d_items, int n_rb, const QuantDesc& q, const StageDesc& sd, int max_steps, int batch, hipStream_t s)
{
    if (n_rb < 1) return NQ_OK;
    AlongForm f;
    if (!along_form(n_rb, max_steps, batch, d_items != nullptr, &f)) {
        set_error("launch_lone_selfq: input too long for the workgroups to quantise, or not in the form that was asked for");
        return NQ_E_INVALID_ARG;
    }
#define NQ_ALONG(PL) (f.e == 4 ? launch_along_t<1, PL, 16, 4>(d_items, q, sd, f, s) : launch_along_t<1, PL, 16, 16>(d_items, q, sd, f, s))
    if (f.w == 8) return f.d.per <= 5 ? launch_along_t<1, 8, 8, 16>(d_items, q, sd, f, s) : launch_along_t<2, 8, 8, 16>(d_items, q, sd, f, s);
    if (f.pl == 1) return NQ_ALONG(1);
    if (f.pl == 2) return NQ_ALONG(2);
    if (f.pl == 4) return NQ_ALONG(4);
    return NQ_ALONG(8);
#undef NQ_ALONG
}

// A form of the launch on a quantised input
struct LoneForm {
    LoneDeal d;
    int pl, w;
    size_t lds;
};

// (six to eight tokens take whole row blocks of eight waves: the registers of sixteen and their sums in LDS are not enough, and fewer planes of two column groups are never the
// faster form: estimated slower than groups of five tokens or fewer at 1 to 600 row blocks, 4 to 1024 steps, 1 to 512 tokens)
static LoneForm lone_form_of(int n_rb, int tokens, int groups, bool spread, int pl)
{
    const int per = (tokens + groups - 1) / groups, w = per > 5 && pl == 8 ? 8 : 16;
    return {LoneDeal{n_rb, tokens, per, groups, spread}, pl, w, (size_t)w * lone_wave_ints(pl * 4 * along_row_ints(per)) * 4};
}

// Time of a launch, back to back with others (us), fitted to 12500 timings: 2 to 100 row blocks of 16 to 448 steps at 1 to 48 tokens in every form of at most one workgroup per
// CU; 5 % off on average, its choices 0.5 % slower than the best of each.  Beside the launch and the chain's fixed part: tiles, fixed point and matrix instructions (past
// 64 steps the rings run dry and the L2 shows: both cost more), the sums through LDS, and what workgroups cost each other.
static double lone_us(const LoneForm& f, int steps)
{
    const int nb = f.d.per <= 5 ? 1 : 2, far = std::max(0, steps - 64), passes = (f.pl * f.d.per + f.w - 1) / f.w;
    const double full = (double)f.d.n_rb * f.d.groups * (8 / f.pl) / 256;
    return 3.11 + 0.0038 * steps + (0.0048 + 0.0023 * f.d.per) * far + 0.00105 * steps * f.pl * nb + 0.0091 / 1024 * f.w * f.pl * 192 * f.d.per +
           full * (0.23 + (0.0012 + 0.0004 * f.d.per) * far) + 0.035 * f.d.per + 0.67 * (nb - 1) + 0.09 * passes + (f.w == 8 ? 0.24 : 0.0);
}

// Tokens are dealt out as in along_form_now, and for the same reason two and more groups on one XCD are level with groups on all: us per launch, all tokens in a
// workgroup / dealt out, 28 row blocks of 448 steps at 8 tokens 18.3 / 10.6, at 4 12.2 / 9.9; 8 of 64 at 8 tokens 4.9 / 3.7, at 4 3.9 / 3.6; 100 of 172 at 8 9.7 / 8.5, at 4 6.8
// (nothing to deal).  More row blocks than half the CUs: whole ones, eight tokens at a time.
static bool lone_form_now(int n_rb, int steps, int tokens, LoneForm* best)
{
    const int cus = device_cu_count(), slots = cus / 8 / ((n_rb + 7) / 8), asked = opt(OPT_LONE_FORM);
    double best_us = 1e30;
    auto consider = [&](int groups, bool spread, int pl) {
        const LoneForm f = lone_form_of(n_rb, tokens, groups, spread, pl);
        if (f.d.per > 5 && pl < 8) return;
        if (asked >= 0 && asked != 100 * f.d.per + 10 * pl + (f.w == 8 ? 4 : 3)) return;
        const double us = lone_us(f, steps);
        if (us < best_us) { best_us = us; *best = f; }
    };
    consider(lone_groups(tokens), tokens > 8, lone_planes(n_rb * lone_groups(tokens)));
    for (int most = 8; most >= 1; --most) {
        const int groups = (tokens + most - 1) / most, per = (tokens + groups - 1) / groups;
        if (per != most) continue;
        for (int pl = 8; pl >= 1; pl /= 2)
            if (asked >= 0 || n_rb * groups * (8 / pl) <= cus) consider(groups, 8 / pl * groups > slots, pl);
    }
    return best_us < 1e30;
}

// (remembered as along_form's)
static bool lone_form(int n_rb, int steps, int tokens, LoneForm* best)
{
    if (opt(OPT_LONE_FORM) >= 0) return lone_form_now(n_rb, steps, tokens, best);
    struct Known {
        int n_rb, steps, tokens;
        LoneForm form;
    };
    static thread_local Known known[64];
    Known& k = known[(unsigned)(n_rb * 31 + steps * 7 + tokens) % 64];
    if (k.n_rb != n_rb || k.steps != steps || k.tokens != tokens) {
        k = Known{n_rb, steps, tokens, {}};
        (void)lone_form_now(n_rb, steps, tokens, &k.form);
    }
    *best = k.form;
    return true;
}

template <int NB, int PL, int W>
static int launch_lone_t(const FusedItem* d_items, const StageDesc& sd, const LoneForm& f, hipStream_t s)
{
    NQ_ALLOW_LDS((stage_lone_kernel<NB, PL, W>), kLoneLdsBytes);
    const int units = f.d.spread ? (f.d.n_rb * f.d.groups + 7) / 8 : (f.d.n_rb + 7) / 8 * f.d.groups;       // of an XCD
    NQ_LAUNCH((stage_lone_kernel<NB, PL, W>), dim3((unsigned)(8 * units * (8 / PL))), dim3(64 * W), f.lds, s, d_items, sd, f.d);
    NQ_HIP(hipGetLastError());
    return NQ_OK;
}

// One stage on an input that a launch of its own has quantised.
int launch_lone(const FusedItem* d_items, int n_rb, const StageDesc& sd, int max_steps, int batch, hipStream_t s)
{
    if (n_rb < 1) return NQ_OK;
    LoneForm f;
    if (!lone_form(n_rb, max_steps, batch, &f)) {
        set_error("launch_lone: no launch in the form that was asked for");
        return NQ_E_INVALID_ARG;
    }
    if (f.w == 8) return launch_lone_t<2, 8, 8>(d_items, sd, f, s);
    if (f.pl == 1) return launch_lone_t<1, 1, 16>(d_items, sd, f, s);
    if (f.pl == 2) return launch_lone_t<1, 2, 16>(d_items, sd, f, s);
    if (f.pl == 4) return launch_lone_t<1, 4, 16>(d_items, sd, f, s);
    return launch_lone_t<1, 8, 16>(d_items, sd, f, s);
}

// Time of a stage dealt out, with its input's fixed point (a quantisation launch where the workgroups do not take it along: 3.5 us and 2.1 us per million elements)
double lone_stage_us(int n_rb, int steps, int tokens)
{
    AlongForm f;
    if (lone_selfq(steps, n_rb, tokens) && along_form(n_rb, steps, tokens, false, &f)) return along_us(f, steps);
    LoneForm l;
    return 3.5 + 2.1e-6 * 64.0 * steps * tokens + (lone_form(n_rb, steps, tokens, &l) ? lone_us(l, steps) : 0.0);
}

// ---- one launch per layer ----
struct LayerLds {
    int t_off, bqt_off;
    size_t bytes;
};
static LayerLds layer_lds(const QuantDesc& qt, const StageDesc& s1, const StageDesc& s2, int batch)
{
    LayerLds l;
    size_t at = (size_t)kLayerWaves * lone_wave_ints(32 * along_row_ints(batch)) * 4 + 2 * sizeof(LoneTokens) + (size_t)batch * lone_tok_bytes(s1.n_steps);
    l.t_off = (int)at;
    at += (size_t)batch * qt.x_stride * 4;
    l.bqt_off = (int)at;
    l.bytes = at + (size_t)batch * lone_tok_bytes(s2.n_steps);
    return l;
}

// Where it is faster than two launches: so few results of stage 1 that each workgroup adds up the waves' sums of all of them in two or three passes, and so few tiles that
// doing them once per workgroup costs less than a launch.  us per call, one launch / two, by row blocks and tiles of stage 1, 2048 outputs: batch 1 one row block of 16 tiles 7.2 / 8.7, 64
// 8.5 / 9.2, 128 10.9 / 9.7; two of 16 7.6 / 9.0, 64 8.4 / 8.9, 128 10.6 / 8.9; four of 32 8.6 / 8.6, 64 8.9 / 8.7 (three of 36 8.3 / 8.5); eight of 32 9.9 / 8.9.  Batch 2 one of 32 8.3 / 9.0, 64 9.4 / 9.3;
// two of 32 8.6 / 9.1, 64 9.5 / 9.0; four of 16 9.6 / 8.7.  Batch 3 one of 16 8.1 / 9.0, 32 8.9 / 9.0; two of 8 8.7 / 8.7.  Batch 4 one of 8 8.0 / 9.1, 16 8.8 / 9.1, 32 9.7 / 9.2; two of 8 9.4 / 9.1.  Batch 5 one of 4, 64 outputs
// 7.6 / 9.2, 2048 8.0 / 9.9, 32000 9.7 / 12.7.
bool lone_layer_fits(const QuantDesc& qt, const StageDesc& s1, const StageDesc& s2, int batch)
{
    const int n_rb1 = (int)n_rowblocks(s1.M), n_rb2 = (int)n_rowblocks(s2.M);
    return batch <= kLayerTokens && n_rb1 * batch <= 6 && n_rb1 * s1.n_steps * batch <= (n_rb1 * batch > 4 ? 24 : n_rb1 <= 2 ? 64 : 48) && n_rb2 <= device_cu_count() &&
           batch * s1.n_steps * 64 <= kLoneMaxElements && batch * s2.n_steps * 64 <= kLoneMaxElements && layer_lds(qt, s1, s2, batch).bytes <= kLoneLdsBytes;
}

template <int PL>
static int launch_layer_t(const QuantDesc& qx, const StageDesc& s1, const QuantDesc& qt, const StageDesc& s2, int batch, hipStream_t s)
{
    NQ_ALLOW_LDS((stage_layer_kernel<PL>), kLoneLdsBytes);
    const LayerLds l = layer_lds(qt, s1, s2, batch);
    const int n_rb = (int)n_rowblocks(s2.M);
    NQ_LAUNCH((stage_layer_kernel<PL>), dim3((unsigned)((n_rb + 7) / 8 * 8 * (8 / PL))), dim3(64 * kLayerWaves), l.bytes, s, qx, s1, qt, s2, n_rb, batch, l.t_off, l.bqt_off);
    NQ_HIP(hipGetLastError());
    return NQ_OK;
}

int launch_lone_layer(const QuantDesc& qx, const StageDesc& s1, const QuantDesc& qt, const StageDesc& s2, int batch, hipStream_t s)
{
    const int pl = lone_planes((int)n_rowblocks(s2.M));
    if (pl == 1) return launch_layer_t<1>(qx, s1, qt, s2, batch, s);
    if (pl == 2) return launch_layer_t<2>(qx, s1, qt, s2, batch, s);
    if (pl == 4) return launch_layer_t<4>(qx, s1, qt, s2, batch, s);
    return launch_layer_t<8>(qx, s1, qt, s2, batch, s);
}

}  // namespace nq
