// Products with the TRANSPOSED sign matrices from the resident tiles of a layer (the training-time siblings of the
// forward: Section 3.4 and Algorithm 1, Phase 3 need  V (U^T (s_out (.) g))  for the gradient of the input scales and of
// the input).  No second copy of the bits is made: a wave turns each 1 KiB tile round in registers and feeds it to the
// int8 matrix cores, against activations held as exact fixed point.
//
// Turning a tile round.  In the forward layout (nq_internal.h) lane (g, j) of a tile holds, in byte b of word v, bit p, the
// sign of row 16p + j, column 16g + 4v + b.  The transposed product reduces over ROWS, so a matrix-instruction operand needs a
// column per lane (its low four lane bits) and rows along the bytes.  The tile is loaded with its lanes renamed -- physical
// lane bits 0-1 = j bits 0-1, bits 2-3 = g, bits 4-5 = j bits 2-3: free, the address of a lane's 16 bytes is arbitrary --
// and then only a 4 x 4 byte transposition inside each quad of lanes is missing (two exchange steps of one DPP move and one
// byte permute per word).  After it, lane bits 0-3 are a column, lane bits 4-5 and the byte are row bits, and the eight bits of
// a byte are the row's remaining three: operand register i of half h is (word_v >> (4h + i)) & 0x01010101, for the columns
// 16g + 4v + b of word v.  That is 80 vector instructions per tile beside 32 matrix instructions of 16 cycles for 16 tokens.
//
// Fixed point with four byte slices (|q| < 2^31 of the token's maximum), exact int32 sums, joined and scaled in binary64,
// one rounding to fp32 when a result is stored: the error against binary64 is that of this one rounding (3.6e-8 of the
// result's norm on normal data, as with binary64 additions on the vector ALU, which this replaces: a product of 64
// tokens with a 4096 x 4096 r = 1024 layer took 235 us in passes of 8 tokens, 16 launches of 2 to 12 us; four launches of 3 to 9
// take 21).  The fixed point's own error is crest / 190 of that rounding, crest = the power of two above the token's maximum
// over the root mean square of its values.  A token of normal gradients times scales has 8 to 16 (the error grows by less than 0.4 %),
// one large element among 65536 has 256 and more: tokens with a crest above 16 take a fifth slice, 2^39, for which groups
// of 16 tokens with such a one are read once more.  (Five slices for all: the gradients of that layer 66 -> 72 us.)
#include <algorithm>

#include "nq_internal.h"
#include "nq_device.h"

namespace nq {

constexpr int kTSlices = 4;             // slices of every token; kTSlices + 1 of a wide one
constexpr int kTWaves = 8;              // waves of a workgroup share one (64 columns, 16 tokens) result: they split its row blocks
constexpr int kTTokens = 16;            // tokens of a workgroup: the 16 columns of one matrix instruction, one slice at a time
// the fixed-point bytes of a group of 16 tokens per 128-row block, [half][slice][token][4 pieces][16]: what one load instruction
// of the product kernel fetches is 1 KiB in one piece
constexpr uint32_t kTGroupRbBytes = 2 * kTSlices * 16 * 64;
constexpr uint32_t kTGroupRbBytes5 = 2 * 16 * 64;       // the fifth slices, in a region of their own: [half][token][4 pieces][16]

// input of the second product where the first one's reduction is dealt out to several workgroups: their sums in binary64, added up,
// scaled and rounded to fp32 (the intermediate u) while they are read
constexpr int kTParts = -1, kTMaxParts = 8;
constexpr int kTPartTokens = 32;        // most parts x tokens

// ---------------------------------------------------------------------------------------------
// scaled input -> fixed point.  One workgroup per token, as many threads as the token has groups of four rows (1024 at most): bound by latency, so a thread has
// little to do in turn.  Group q of 64 rows is word q >> 2 of piece q & 3 of those rows' four 16-byte pieces: piece (s, c) of a token holds, as four words
// i of four bytes, rows 64 s + 16 i + 4 c + (0..3) -- the order in which the turned-round tile meets its rows.  Launches of 64 tokens, 4096 rows 5.2 us (with 16 rows
// per thread and reductions through LDS permutes 5.6), 1024 rows 3.5 (4.0), 2500 rows 3.4 (5.5).
// ---------------------------------------------------------------------------------------------
struct TQuantArgs {
    const void* in;             // [batch][in_stride] of in_dtype; kTParts: [parts][batch][in_stride] binary64 to be added up
    int parts;
    const uint16_t* scale;      // fp16 [M] or nullptr
    uint8_t* bq;                // [groups of 16 tokens][n_pieces / 4][slices][16 tokens][4][16]
    uint8_t* bq5;               // [groups of 16 tokens][n_pieces / 4][16 tokens][4][16]: the fifth slice, of wide tokens only
    QMeta* meta;                // [batch]
    uint32_t* wide;             // [batch] whether the token has a fifth slice
    int M, in_dtype, in_stride;
    int n_pieces;               // 4 per 64 rows, whole row blocks
};

// the four scaled values of rows r0 .. r0 + 3 (rows past M are padding: zeros); binary64: an fp32 value times an fp16 scale is exact.  (DT = the type of the
// input; kTParts: from `u`, LDS)
template <int DT>
__device__ __forceinline__ void tq_load(const TQuantArgs& a, size_t base, int r0, double v[4], const float* u)
{
    typedef unsigned int v2u __attribute__((ext_vector_type(2)));
    typedef v4f v4f_any __attribute__((aligned(4)));       // rows of odd lengths: 16 and 8 bytes at the alignment of an element
    typedef v2u v2u_any __attribute__((aligned(2)));
    if (DT == kTParts) {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = r0 + k < a.M ? (double)u[r0 + k] : 0.0;
        return;
    }
    if (r0 + 4 <= a.M) {
        v4f xf;
        v2u xh, sc;
        if (DT == NQ_F32) xf = *(const __attribute__((address_space(1))) v4f_any*)((const float*)a.in + base + r0);
        else xh = *(const __attribute__((address_space(1))) v2u_any*)((const uint16_t*)a.in + base + r0);
        if (a.scale) sc = *(const __attribute__((address_space(1))) v2u*)(a.scale + r0);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint16_t h = (uint16_t)(xh[k >> 1] >> (16 * (k & 1)));
            v[k] = (double)(DT == NQ_F32 ? xf[k] : DT == NQ_F16 ? half_bits_to_float(h) : bf16_bits_to_float(h));
            if (a.scale) v[k] *= (double)half_bits_to_float((uint16_t)(sc[k >> 1] >> (16 * (k & 1))));
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = 0.0;
        if (r0 + k < a.M) {
            v[k] = (double)load_as_float(a.in, DT, (int64_t)(base + r0 + k));
            if (a.scale) v[k] *= (double)half_bits_to_float(a.scale[r0 + k]);
        }
    }
}

// low 32 bits of a binary64
__device__ __forceinline__ int low_word(double v) { return (int)(uint32_t)__builtin_bit_cast(uint64_t, v); }

// q of four values -> their word of every slice (slices 1 KiB apart); returns sum q.
// q (WIDE: hi and lo with q = 2^24 hi + lo) is taken from the low bits of a sum with a constant that leaves it no fraction: rounding
// and converting instructions for binary64 are several times as slow.
template <bool WIDE>
__device__ __forceinline__ double tq_store(const double v[4], double inv_step, bool bad, uint8_t* dst, uint8_t* dst5)
{
    constexpr int kS = kTSlices + (WIDE ? 1 : 0);
    constexpr double kLo = 0x1.8p52, kHi = 0x1.8p76;
    long long sum = 0;
    uint32_t d[kS][4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        int hi = 0, b;
        if (WIDE) {
            const double at = fma(v[k], inv_step, kHi);
            hi = low_word(at);                                              // |hi| <= 2^15
            b = low_word(fma(v[k], inv_step, kHi - at) + kLo);              // |lo| <= 2^23
            sum += ((long long)hi << 24) + b;
        } else {
            b = bad ? 0 : low_word(fma(v[k], inv_step, kLo));               // |q| < 0.992 * 2^31
            sum += b;
        }
        // the signed bytes from the lowest up (slice kS - 1); WIDE: those of lo, then of hi plus what lo carries
#pragma unroll
        for (int s = kS - 1; s >= 0; --s) {
            if (WIDE && s == kS - 4) b += hi;
            d[s][k] = (uint32_t)b;
            b = (b + 128) >> 8;
        }
    }
#pragma unroll
    for (int s = 0; s < kS; ++s) *(uint32_t*)(s < kTSlices ? dst + s * 1024 : dst5) = pack_low_bytes(d[s][0], d[s][1], d[s][2], d[s][3]);
    return (double)sum;                                                         // below 2^42
}

// op over each 16-lane row of the wavefront by data-parallel moves, the same in all lanes of a row; over the whole wavefront
template <class Op>
__device__ __forceinline__ double row_reduce_f64(double v, Op op)
{
    auto dpp = [](double x, auto ctrl) {
        const uint64_t b = __builtin_bit_cast(uint64_t, x);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, decltype(ctrl)::value, 0xf, 0xf, true);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), decltype(ctrl)::value, 0xf, 0xf, true);
        return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
    };
    v = op(v, dpp(v, std::integral_constant<int, 0xB1>{}));      // quad_perm [1, 0, 3, 2]
    v = op(v, dpp(v, std::integral_constant<int, 0x4E>{}));      // quad_perm [2, 3, 0, 1]
    v = op(v, dpp(v, std::integral_constant<int, 0x141>{}));     // row_half_mirror
    return op(v, dpp(v, std::integral_constant<int, 0x140>{})); // row_mirror
}
template <class Op>
__device__ __forceinline__ double wave_reduce_f64(double v, Op op)
{
    auto lane = [](double x, int l) {
        const uint64_t b = __builtin_bit_cast(uint64_t, x);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l), hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
        return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
    };
    v = row_reduce_f64(v, op);
    return op(op(lane(v, 0), lane(v, 16)), op(lane(v, 32), lane(v, 48)));
}

constexpr int kTQThreads = 1024;        // most threads of a workgroup

template <int DT>
__global__ void __launch_bounds__(kTQThreads) quantize_t_kernel(TQuantArgs a)
{
    __shared__ double sm_max[kTQThreads / 64], sm_sum[kTQThreads / 64], sm_sq[kTQThreads / 64];
    __shared__ int sm_bad[kTQThreads / 64];
    const int tok = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, threads = blockDim.x;
    const int groups = a.n_pieces * 4;                      // of four rows
    const size_t base = (size_t)tok * a.in_stride;
    double v[4], m = 0.0, sq = 0.0;
    int bad = 0;
    extern __shared__ float u[];                            // [M], kTParts only
    if (DT == kTParts) {
        typedef const __attribute__((address_space(1))) double* gptr_d;
        const gptr_d in = (gptr_d)a.in + base;
        const size_t part = (size_t)gridDim.x * a.in_stride;
        for (int r = tid; r < a.M; r += threads) {
            double p[kTMaxParts];                           // (as many loads in flight whatever the count: past it the last is read again)
#pragma unroll
            for (int k = 0; k < kTMaxParts; ++k) p[k] = in[(k < a.parts ? k : a.parts - 1) * part + r];
            double t = p[0];
#pragma unroll
            for (int k = 1; k < kTMaxParts; ++k) t += k < a.parts ? p[k] : 0.0;
            u[r] = (float)(a.scale ? t * (double)half_bits_to_float(a.scale[r]) : t);
        }
        __syncthreads();
    }
    // (a thread's first group stays in registers between the two passes; longer vectors re-read the others)
    for (int gr = tid + ((groups - 1 - tid) / threads) * threads; gr >= 0; gr -= threads) {
        if (gr >= groups) break;
        tq_load<DT>(a, base, 4 * gr, v, u);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double t = fabs(v[k]);
            if (!(t <= 1.0e300)) bad = 1;                   // NaN or infinity
            m = fmax(m, t);
            sq = fma(v[k], v[k], sq);
        }
    }
    const auto most = [](double x, double y) { return fmax(x, y); };
    const auto plus = [](double x, double y) { return x + y; };
    m = wave_reduce_f64(m, most);
    sq = wave_reduce_f64(sq, plus);
    bad = __builtin_amdgcn_ballot_w64(bad != 0) != 0;
    if ((tid & 63) == 0) { sm_max[wave] = m; sm_bad[wave] = bad; sm_sq[wave] = sq; }
    __syncthreads();
    // (lane l of every row looks at wave l's)
    const int other = (tid & 15) < threads / 64 ? tid & 15 : -1, other0 = other < 0 ? 0 : other;
    m = row_reduce_f64(sm_max[other0], most);
    bad = __builtin_amdgcn_ballot_w64(sm_bad[other0] != 0) != 0;
    sq = row_reduce_f64(other < 0 ? 0.0 : sm_sq[other0], plus);
    // step = 2^(e - 31), 2^(e - 39) wide, with the maximum at most 0.99 * 2^e: q fits its signed bytes, which hold +-0.996 * 2^31
    int e = 0;
    if (m > 0.0 && !bad && frexp(m, &e) > 0.99) ++e;
    const double top = ldexp(1.0, e);
    const bool wide = m > 0.0 && !bad && (double)a.M * top * top > 256.0 * sq;
    const double step = ldexp(1.0, e - (wide ? 39 : 31)), inv_step = ldexp(1.0, (wide ? 39 : 31) - e);
    double s = 0.0;
    const size_t group = (size_t)(tok >> 4) * (a.n_pieces >> 2);
    uint8_t* const dst = a.bq + group * (kTGroupRbBytes / 2) + (tok & 15) * 64;
    uint8_t* const dst5 = a.bq5 + group * (kTGroupRbBytes5 / 2) + (tok & 15) * 64;
    for (int gr = tid; gr < groups; gr += threads) {
        if (gr != tid) tq_load<DT>(a, base, 4 * gr, v, u);
        const int q = gr & 15, at = (q & 3) * 16 + (q >> 2) * 4;
        uint8_t* const to = dst + (size_t)(gr >> 4) * (kTGroupRbBytes / 2) + at;
        s += wide ? tq_store<true>(v, inv_step, false, to, dst5 + (size_t)(gr >> 4) * (kTGroupRbBytes5 / 2) + at) : tq_store<false>(v, inv_step, bad != 0, to, nullptr);
    }
    s = wave_reduce_f64(s, plus);                           // below 2^53: exact
    if ((tid & 63) == 0) sm_sum[wave] = s;
    __syncthreads();
    if (tid < 16) {
        const double tot = row_reduce_f64(other < 0 ? 0.0 : sm_sum[other0], plus);
        if (tid != 0) return;
        QMeta mt;
        mt.two_step = bad ? (double)__builtin_nanf("") : ldexp(1.0, e - 38);       // (the product joins five slices, the fifth of other tokens zero)
        mt.neg_qs = -tot * step;
        a.meta[tok] = mt;
        a.wide[tok] = wide;
    }
}

// ---------------------------------------------------------------------------------------------
// out[tok][col] = out_scale[col] * sum_row sign(row, col) v[tok][row], 64 columns x 16 tokens per workgroup
// grid = (64-column steps x 4 / NV, token groups, parts), block = 512.  NV = words of a tile's lane that a workgroup takes of the four,
// i.e. 16 NV of the 64 columns: where columns and token groups are few, two workgroups share a tile.  parts > 1: each takes its share
// of the row blocks, and the sums (exact) go to `partial` for the next quantisation to add up.
// ---------------------------------------------------------------------------------------------
struct TStageArgs {
    const uint32_t* tiles;
    const uint8_t* bq;
    const uint8_t* bq5;
    const QMeta* meta;
    const uint32_t* wide;
    const uint16_t* out_scale;      // fp16 [N] or nullptr
    float* out;                     // [batch][out_stride]
    double* partial;                // [parts][batch][out_stride] where the reduction is dealt out, else nullptr
    int N, n_steps, n_rb, out_stride, batch;
};

// rows of four bytes -> columns of four bytes inside each quad of lanes: byte b of lane t becomes byte t of lane b
__device__ __forceinline__ uint32_t quad_transpose(uint32_t w, uint32_t sel2, uint32_t sel1)
{
    const uint32_t a = (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0x4E, 0xF, 0xF, true);       // quad_perm [2,3,0,1]
    w = __builtin_amdgcn_perm(a, w, sel2);
    const uint32_t b = (uint32_t)__builtin_amdgcn_mov_dpp((int)w, 0xB1, 0xF, 0xF, true);       // quad_perm [1,0,3,2]
    return __builtin_amdgcn_perm(b, w, sel1);
}

// Bound: instruction issue and latency, not memory (a tile meets 16 tokens, so 1 KiB costs 512 matrix-core cycles of one
// SIMD).  Eight waves per workgroup because at the row counts of real layers (8 to 224 row blocks) a result's reduction is the
// only thing left to spread over the chip once columns and tokens have been.
template <int NV>
__global__ void __launch_bounds__(64 * kTWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) gemm_t_kernel(TStageArgs a)
{
    constexpr int kRing = 2;                                        // tiles in flight per wave
    __shared__ v4i red[2][kTWaves][NV][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int g = lane >> 4, n = lane & 15;
    const int st = blockIdx.x / (4 / NV), v0 = blockIdx.x % (4 / NV) * NV, t0 = blockIdx.y * kTTokens;
    const int tok = t0 + n < a.batch ? t0 + n : a.batch - 1;        // a column past the batch repeats the last token and is not stored
    const int tile_lane = (lane & 3) | ((lane >> 4) & 3) << 2 | ((lane >> 2) & 3) << 4;
    const uint32_t sel2 = lane & 2 ? 0x03020706u : 0x05040100u, sel1 = lane & 1 ? 0x03070105u : 0x06020400u;
    const char* w_base = (const char*)(a.tiles + (size_t)st * kTileWords) + 16 * tile_lane + 4 * v0;
    const size_t w_rb = (size_t)a.n_steps * (kTileWords * 4);
    const char* b_base = (const char*)a.bq + (size_t)blockIdx.y * a.n_rb * kTGroupRbBytes + 64 * n + 16 * g;
    // (what the epilogue needs is requested before the reduction, not behind it)
    const int col = st * kTileCols + 16 * g + 4 * (v0 + wave % NV);
    const double two_step = a.meta[tok].two_step, neg_qs = a.meta[tok].neg_qs;
    const bool wide = a.wide[tok] != 0;
    float osc[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) osc[k] = a.out_scale ? half_bits_to_float(a.out_scale[col + k < a.N ? col + k : 0]) : 1.0f;
    v4i acc[NV][kTSlices];
#pragma unroll
    for (int v = 0; v < NV; ++v)
#pragma unroll
        for (int s = 0; s < kTSlices; ++s) acc[v][s] = v4i{0, 0, 0, 0};
    // past the end the last tile is read again and not used
    const int last = a.n_rb - 1, first = blockIdx.z * kTWaves + wave, stride = gridDim.z * kTWaves;
    typedef unsigned int vNu __attribute__((ext_vector_type(NV)));
    vNu w[kRing];
    v4u b[kRing][2][kTSlices];
#define NQ_T_ISSUE(k, rb)                                                                                   \
    do {                                                                                                    \
        const int rr = (rb) < last ? (rb) : last;                                                           \
        w[k] = *(const __attribute__((address_space(1))) vNu*)(w_base + (size_t)rr * w_rb);                 \
        _Pragma("unroll") for (int h = 0; h < 2; ++h)                                                       \
            _Pragma("unroll") for (int s = 0; s < kTSlices; ++s)                                            \
                b[k][h][s] = load_global_v4u(b_base + (size_t)rr * kTGroupRbBytes, (uint32_t)((h * kTSlices + s) * 1024)); \
    } while (0)
#define NQ_T_MAC(k)                                                                                         \
    do {                                                                                                    \
        _Pragma("unroll") for (int v = 0; v < NV; ++v) {                                                    \
            const uint32_t t = quad_transpose(w[k][v], sel2, sel1);                                         \
            _Pragma("unroll") for (int h = 0; h < 2; ++h) {                                                 \
                v4u op;                                                                                     \
                _Pragma("unroll") for (int i = 0; i < 4; ++i) op[i] = (t >> (4 * h + i)) & 0x01010101u;     \
                _Pragma("unroll") for (int s = 0; s < kTSlices; ++s)                                        \
                    acc[v][s] = __builtin_amdgcn_mfma_i32_16x16x64_i8((v4i)op, (v4i)b[k][h][s], acc[v][s], 0, 0, 0); \
            }                                                                                               \
        }                                                                                                   \
    } while (0)
#pragma unroll
    for (int k = 0; k < kRing; ++k) {
        if (k == 0 || first + k * stride <= last) NQ_T_ISSUE(k, first + k * stride);
        __builtin_amdgcn_sched_barrier(0);
    }
    int rb = first;
    for (; rb + (kRing - 1) * stride < a.n_rb; rb += kRing * stride) {
#pragma unroll
        for (int k = 0; k < kRing; ++k) {
            NQ_T_MAC(k);
            NQ_T_ISSUE(k, rb + (k + kRing) * stride);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int k = 0; k < kRing - 1; ++k)
        if (rb + k * stride < a.n_rb) NQ_T_MAC(k);
#undef NQ_T_ISSUE
#undef NQ_T_MAC

    // the eight partial sums of every result, through LDS, two slices joined (a wave has met at most 8192 rows: 2^28); wave v
    // of the first NV takes word v0 + v
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int v = 0; v < NV; ++v) red[s][wave][v][lane] = (acc[v][2 * s] << 8) + acc[v][2 * s + 1];
    __syncthreads();
    double sum[2][4] = {};
    v4i low = {0, 0, 0, 0};
    if (wave < NV) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int k = 0; k < kTWaves; k += 4) {          // (four waves' sums stay in 32 bits)
                const v4i p = (red[s][k][wave][lane] + red[s][k + 1][wave][lane]) + (red[s][k + 2][wave][lane] + red[s][k + 3][wave][lane]);
#pragma unroll
                for (int i = 0; i < 4; ++i) sum[s][i] += (double)p[i];
            }
    }
    if (__builtin_amdgcn_ballot_w64(wide) != 0) {           // (the same in all waves)
#pragma unroll
        for (int v = 0; v < NV; ++v) acc[v][0] = v4i{0, 0, 0, 0};
        const char* const b5_base = (const char*)a.bq5 + (size_t)blockIdx.y * a.n_rb * kTGroupRbBytes5 + 64 * n + 16 * g;
        for (int r = first; r < a.n_rb; r += stride) {
            const vNu wr = *(const __attribute__((address_space(1))) vNu*)(w_base + (size_t)r * w_rb);
            v4u br[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                br[h] = load_global_v4u(b5_base + (size_t)r * kTGroupRbBytes5, (uint32_t)(h * 1024));
                if (!wide) br[h] = v4u{0, 0, 0, 0};         // (never written for this token)
            }
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                const uint32_t t = quad_transpose(wr[v], sel2, sel1);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    v4u op;
#pragma unroll
                    for (int i = 0; i < 4; ++i) op[i] = (t >> (4 * h + i)) & 0x01010101u;
                    acc[v][0] = __builtin_amdgcn_mfma_i32_16x16x64_i8((v4i)op, (v4i)br[h], acc[v][0], 0, 0, 0);
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int v = 0; v < NV; ++v) red[0][wave][v][lane] = acc[v][0];
        __syncthreads();
        if (wave < NV) {
#pragma unroll
            for (int k = 0; k < kTWaves; ++k) low += red[0][k][wave][lane];
        }
    }
    if (wave >= NV || t0 + n >= a.batch) return;
    // lane (g, n), register k: column 16 g + 4 v + k of the step, token n
    float r[4];
    if (a.partial) {
        double* const o = a.partial + ((size_t)blockIdx.z * a.batch + tok) * a.out_stride + col;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const double raw = fma(fma(sum[0][k], 65536.0, sum[1][k]), 256.0, (double)low[k]);
            if (col + k < a.N) o[k] = fma(raw, two_step, blockIdx.z == 0 ? neg_qs : 0.0);
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        // (below 2^47 without the fifth slice, then 2^55: rounded in binary64 at most)
        const double raw = fma(fma(sum[0][k], 65536.0, sum[1][k]), 256.0, (double)low[k]);
        double val = fma(raw, two_step, neg_qs);
        val *= (double)osc[k];
        r[k] = (float)val;
    }
    float* const o = a.out + (size_t)tok * a.out_stride + col;
    if ((a.out_stride & 3) == 0 && col + 4 <= a.N) {
        *(v4f*)o = v4f{r[0], r[1], r[2], r[3]};
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (col + k < a.N) o[k] = r[k];
    }
}

static size_t al256(size_t v) { return (v + 255) / 256 * 256; }

size_t gemm_t_scratch_bytes(int64_t M, int batch)
{
    return (size_t)((batch + kTTokens - 1) / kTTokens) * n_rowblocks(M) * (kTGroupRbBytes + kTGroupRbBytes5) + al256((size_t)batch * sizeof(QMeta)) +
           al256((size_t)batch * sizeof(uint32_t));
}

// half tiles where whole ones leave more than half of the CUs without a workgroup (16 steps x 4 groups: 8.3 us against 10; on 11
// layers from 300 x 300 to 28672 x 8192 at 1 to 512 tokens the faster of the two, or within 2 % of it)
static bool half_tiles(int64_t N, int batch)
{
    return (N + kTileCols - 1) / kTileCols * ((batch + kTTokens - 1) / kTTokens) <= device_cu_count() / 2;
}

// Workgroups that a product's reduction is dealt out to: where its columns and tokens give less than every fourth CU one and its waves
// have more than one row block each (few tokens of tall, narrow products, whose waves would walk them alone), as many as its sums leave room
// for in the memory of the fp32 intermediate of 64 tokens (32 in binary64).  Both products, 4 tokens: 65536 x 256 r = 64 97 -> 42 us,
// 9856 x 256 r = 82 27.4 -> 20.7, 4096 x 4096 r = 1024 19.1 -> 17.8; passes on the vector ALU took 63, 24.7 and 30.
int gemm_t_parts(int64_t M, int64_t N, int batch)
{
    const int64_t wgs = (N + kTileCols - 1) / kTileCols * ((batch + kTTokens - 1) / kTTokens) * (half_tiles(N, batch) ? 2 : 1);
    if (batch > 8 || wgs * 4 > device_cu_count()) return 1;         // (two parts are not worth adding up: 4096 x 4096 at 16 tokens 19.5 -> 21)
    int parts = 1;
    while (parts < kTMaxParts && parts * 2 * batch <= kTPartTokens && n_rowblocks(M) > kTWaves * parts) parts *= 2;
    return parts;
}

// A is [M][N] as sign tiles; out[tok][0..N) = out_scale (.) A^T (in_scale (.) in[tok][0..M)).  `scratch`: device,
// gemm_t_scratch_bytes(M, batch), 16-byte aligned.  parts > 1: the sums of that many shares of the rows go to `out` as
// binary64 [parts][batch][out_stride], without the output scale; in_parts > 1: `in` is such an array, whose total times
// in_scale is rounded to fp32 as it is read.
int launch_gemm_t(const uint32_t* tiles, int64_t M, int64_t N, const void* in, int in_dtype, int in_stride, const uint16_t* in_scale,
                  int in_parts, const uint16_t* out_scale, void* out, int out_stride, int parts, int batch, void* scratch, hipStream_t s)
{
    const int n_rb = (int)n_rowblocks(M);
    const int groups = (batch + kTTokens - 1) / kTTokens;
    uint8_t* bq = (uint8_t*)scratch;
    uint8_t* bq5 = bq + (size_t)groups * n_rb * kTGroupRbBytes;
    QMeta* meta = (QMeta*)(bq5 + (size_t)groups * n_rb * kTGroupRbBytes5);
    uint32_t* wide = (uint32_t*)((char*)meta + al256((size_t)batch * sizeof(QMeta)));
    const TQuantArgs q{in, in_parts, in_scale, bq, bq5, meta, wide, (int)M, in_dtype, in_stride, n_rb * 8};
    // (parts are added up by a thread per row; the rows, at most 8192 of them here, wait in LDS)
    const dim3 qgrid(batch), qblock(std::min(kTQThreads, (in_parts > 1 ? (int)M + 63 : q.n_pieces * 4 + 63) / 64 * 64));
    if (in_parts > 1) hipLaunchKernelGGL(quantize_t_kernel<kTParts>, qgrid, qblock, (size_t)M * sizeof(float), s, q);
    else if (in_dtype == NQ_F32) hipLaunchKernelGGL(quantize_t_kernel<NQ_F32>, qgrid, qblock, 0, s, q);
    else if (in_dtype == NQ_F16) hipLaunchKernelGGL(quantize_t_kernel<NQ_F16>, qgrid, qblock, 0, s, q);
    else hipLaunchKernelGGL(quantize_t_kernel<NQ_BF16>, qgrid, qblock, 0, s, q);
    NQ_HIP(hipGetLastError());
    const TStageArgs t{tiles, bq, bq5, meta, wide, out_scale, (float*)out, parts > 1 ? (double*)out : nullptr, (int)N, (int)n_steps(N), n_rb, out_stride, batch};
    const unsigned steps = (unsigned)((N + kTileCols - 1) / kTileCols);
    if (half_tiles(N, batch))
        hipLaunchKernelGGL(gemm_t_kernel<2>, dim3(steps * 2, (unsigned)groups, (unsigned)parts), dim3(64 * kTWaves), 0, s, t);
    else
        hipLaunchKernelGGL(gemm_t_kernel<4>, dim3(steps, (unsigned)groups, (unsigned)parts), dim3(64 * kTWaves), 0, s, t);
    NQ_HIP(hipGetLastError());
    return NQ_OK;
}

}  // namespace nq
