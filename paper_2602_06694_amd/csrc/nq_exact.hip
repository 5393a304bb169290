// The exact streaming product for more than eight tokens at a time: the arithmetic of the decode kernels (nq_decode.hip: 24-bit
// fixed point in three byte slices, exact int32 sums, the same roundings, hence the same bits) for groups of 16 tokens.
//
// A column group of the matrix instruction is ONE slice of 16 tokens, not three slices of five: the slices of a result sit in
// the same lane and register of three accumulators and are joined there, and a tile's masked words (32 vector instructions)
// are used by 24 matrix instructions instead of 8 or 16.  Nothing is staged: a 64-column step costs a wave 1 KiB of tile and
// 3 KiB of fixed point, both from L2 (the tiles of a layer of a few MB are read once per group of 16 tokens, and stay there).
// Eight waves of a workgroup split the reduction of one (row block, 16 tokens) result: at the sizes of real layers row blocks
// and token groups alone leave most of the chip idle.
// 64 tokens of a 4096 x 4096 r = 1024 layer: 20 us (four launches of 4 to 8 us, bound by latency) where passes of eight tokens
// took 32 launches and 185 us.
#include "nq_internal.h"
#include "nq_device.h"

namespace nq {

constexpr int kXWaves = 8, kXTokens = 16;

// grid = (row blocks x 8 / PL, token groups), block = 512.  PL = bit planes (16 rows each) a workgroup takes of its row block's
// eight: where row blocks and token groups are few, several workgroups read the same tiles and finish fewer rows each.
template <int PL>
__global__ void __launch_bounds__(64 * kXWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) stage_exact_kernel(StageDesc d, int batch)
{
    constexpr int kXRing = 4;                                       // steps in flight per wave
    constexpr int kRound = PL <= 2 ? kSlices : 1;                   // slices whose partial sums pass through LDS at a time
    __shared__ v4i red[kRound][kXWaves][PL][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int g = lane >> 4, n = lane & 15;
    const int rb = blockIdx.x / (8 / PL), p0 = blockIdx.x % (8 / PL) * PL, t0 = blockIdx.y * kXTokens;
    const int tok = t0 + n < batch ? t0 + n : batch - 1;            // a column past the batch repeats the last token and is not stored
    const char* w_base = (const char*)(d.tiles + (size_t)rb * d.n_steps * kTileWords) + 16 * lane;
    const char* b_base = (const char*)d.bq + (size_t)blockIdx.y * d.n_steps * kGroupStepBytes + 64 * n + 16 * g;
    // (what the epilogue needs is requested before the reduction, not behind it)
    const int row0 = rb * kTileRows + 16 * (p0 + wave % PL) + 4 * g;
    const QMeta mt = d.meta[tok];
    float osc[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) osc[v] = d.out_scale ? half_bits_to_float(((gptr_u16)d.out_scale)[row0 + v < d.M ? row0 + v : 0]) : 1.0f;
    v4i acc[kSlices][PL];
#pragma unroll
    for (int s = 0; s < kSlices; ++s)
#pragma unroll
        for (int p = 0; p < PL; ++p) acc[s][p] = v4i{0, 0, 0, 0};
    // steps wave, wave + 8, ...; past the end the last step is read again and not used
    const int last = d.n_steps - 1;
    v4u w[kXRing], b[kXRing][kSlices];
#define NQ_X_ISSUE(k, step)                                                                             \
    do {                                                                                                \
        const uint32_t ss = (uint32_t)((step) < last ? (step) : last);                                  \
        w[k] = load_global_v4u(w_base, ss * (kTileWords * 4));                                          \
        _Pragma("unroll") for (int s = 0; s < kSlices; ++s)                                             \
            b[k][s] = load_global_v4u(b_base, ss * kGroupStepBytes + 1024 * s);                            \
    } while (0)
#define NQ_X_MAC(k)                                                                                     \
    do {                                                                                                \
        const v4u wk = PL == 8 ? w[k] : w[k] >> (uint32_t)p0;                                           \
        _Pragma("unroll") for (int p = 0; p < PL; ++p) {                                                \
            const v4i a = (v4i)(wk & (0x01010101u << p));                                               \
            _Pragma("unroll") for (int s = 0; s < kSlices; ++s)                                         \
                acc[s][p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, (v4i)b[k][s], acc[s][p], 0, 0, 0); \
        }                                                                                               \
    } while (0)
#pragma unroll
    for (int k = 0; k < kXRing; ++k) {
        if (k == 0 || wave + k * kXWaves <= last) NQ_X_ISSUE(k, wave + k * kXWaves);
        __builtin_amdgcn_sched_barrier(0);
    }
    int st = wave;
    for (; st + (kXRing - 1) * kXWaves < d.n_steps; st += kXRing * kXWaves) {
#pragma unroll
        for (int k = 0; k < kXRing; ++k) {
            NQ_X_MAC(k);
            NQ_X_ISSUE(k, st + (k + kXRing) * kXWaves);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
#pragma unroll
    for (int k = 0; k < kXRing - 1; ++k)
        if (st + k * kXWaves < d.n_steps) NQ_X_MAC(k);
#undef NQ_X_ISSUE
#undef NQ_X_MAC

    // the partial sums of the eight waves, through LDS; wave p takes bit plane p0 + p.  (A plane below 7 of a shifted word is
    // worth 2^p, bit 7 of a byte 2^7 with a minus: int8)
    v4i sum[kSlices];
#pragma unroll
    for (int s0 = 0; s0 < kSlices; s0 += kRound) {
        if (s0) __syncthreads();
#pragma unroll
        for (int s = 0; s < kRound; ++s)
#pragma unroll
            for (int p = 0; p < PL; ++p) red[s][wave][p][lane] = acc[s0 + s][p];
        __syncthreads();
        if (wave < PL) {
#pragma unroll
            for (int s = 0; s < kRound; ++s) {
                sum[s0 + s] = v4i{0, 0, 0, 0};
#pragma unroll
                for (int k = 0; k < kXWaves; ++k) sum[s0 + s] += red[s][k][wave][lane];
                if (PL == 8 && wave == 7) sum[s0 + s] = -sum[s0 + s];
            }
        }
    }
    if (wave >= PL || t0 + n >= batch) return;
    // lane (g, n), register v: row 16 plane + 4 g + v, token n; joined and rounded as in the decode kernels' epilogue
    const double scale_p = __builtin_ldexp(mt.two_step, -wave);
    float r[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const double raw = fma((double)sum[0][v], 65536.0, fma((double)sum[1][v], 256.0, (double)sum[2][v]));
        const float z = (float)fma(raw, scale_p, mt.neg_qs);
        r[v] = z * osc[v];
    }
    const size_t at = (size_t)tok * d.out_stride + row0;
    if (d.out_dtype == NQ_F32 && (d.out_stride & 3) == 0 && row0 + 4 <= d.M) {
        *(__attribute__((address_space(1))) v4f*)((float*)d.out + at) = v4f{r[0], r[1], r[2], r[3]};
    } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
            if (row0 + v < d.M) store_out(d.out, d.out_dtype, at + v, r[v]);
    }
}

// Bit planes of a workgroup: whole row blocks where they give every second CU a workgroup; below that halves and quarters of them, until they do (a
// 4096 x 4096 r = 1024 layer at 64 tokens, 32 and 128 pairs of row block and group: quarters 12.1 -> 7.7 us, halves 6.7 -> 4.7;
// with the transposed product's rule the gradients of that layer 70.2 -> 66.1 us; of the three forms on 11 layers from 300 x 300
// to 28672 x 8192 at 12 to 512 tokens this rule's is the fastest or within 2 % of it)
static int exact_planes(int pairs)
{
    int pl = 8;
    while (pl > 2 && pairs * (8 / pl) <= device_cu_count() / 2) pl /= 2;
    return pl;
}

// Time of one stage: rounds of workgroups, one per CU, of 4.4 us and 0.057 us per step each.  With 7 us beside the stages and the
// quantisation per element (exact_us) fitted to 1150 forwards of 50 layers from 256 x 256 to 28672 x 28672 at 9 to 512 tokens: 6 % off on average.
static double exact_stage_us(int64_t M, int64_t N, int batch)
{
    const int pairs = (int)n_rowblocks(M) * ((batch + kXTokens - 1) / kXTokens), cus = device_cu_count();
    return (pairs * (8 / exact_planes(pairs)) + cus - 1) / cus * (4.36 + 0.0566 * n_steps(N));
}
double exact_us(int64_t d_out, int64_t d_in, int64_t r, int batch)
{
    return 7.0 + exact_stage_us(r, d_in, batch) + exact_stage_us(d_out, r, batch) + 2.14e-6 * batch * (double)(d_in + 3 * r);
}

// The path's time with stages dealt out where they are (nq_lone.hip): a stage in groups of 16 with its quantisation launch, or dealt out with its input's fixed point
double exact_now_us(int64_t d_out, int64_t d_in, int64_t r, int batch)
{
    const auto stage = [&](int64_t M, int64_t N) {
        const int n_rb = (int)n_rowblocks(M), steps = (int)n_steps(N);
        if (lone_deals_out(n_rb, steps, N % 16 == 0, batch)) return lone_stage_us(n_rb, steps, batch);
        return 3.5 + exact_stage_us(M, N, batch) + 2.14e-6 * batch * (double)N;
    };
    return stage(r, d_in) + stage(d_out, r);
}

int launch_stage_exact(const StageDesc& d, int batch, hipStream_t s)
{
    const int n_rb = (int)n_rowblocks(d.M), groups = (batch + kXTokens - 1) / kXTokens;
    const int pl = exact_planes(n_rb * groups);
    const dim3 grid((unsigned)(n_rb * (8 / pl)), (unsigned)groups), block(64 * kXWaves);
    if (pl == 8) hipLaunchKernelGGL(stage_exact_kernel<8>, grid, block, 0, s, d, batch);
    else if (pl == 4) hipLaunchKernelGGL(stage_exact_kernel<4>, grid, block, 0, s, d, batch);
    else hipLaunchKernelGGL(stage_exact_kernel<2>, grid, block, 0, s, d, batch);
    NQ_HIP(hipGetLastError());
    return NQ_OK;
}

}  // namespace nq
