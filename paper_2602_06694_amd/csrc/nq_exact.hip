// The exact streaming product for more than eight tokens at a time: the arithmetic of the decode kernels (nq_decode.hip: 24-bit
// fixed point in three byte slices, exact int32 sums, the same roundings, hence the same bits) for groups of 16 tokens.
//
// A column group of the matrix instruction is ONE slice of 16 tokens, not three slices of five: the slices of a result sit in
// the same lane and register of three accumulators and are joined there, and a tile's masked words (32 vector instructions)
// are used by 24 matrix instructions instead of 8 or 16.  Nothing is staged: a 64-column step costs a wave 1 KiB of tile and
// 3 KiB of fixed point, both from L2 (the tiles of a layer of a few MB are read once per group of 16 tokens, and stay there).
// Eight waves of a workgroup split the reduction of one (row block, 16 tokens) result: at the sizes of real layers row blocks
// and token groups alone leave most of the chip idle.
// 64 tokens of a 4096 x 4096 r = 1024 layer: 26 us (four launches of 4 to 12 us, bound by latency) where passes of eight tokens
// took 32 launches and 185 us.
#include "nq_internal.h"
#include "nq_device.h"

namespace nq {

constexpr int kXWaves = 8, kXTokens = 16, kXRing = 4;

// grid = (row blocks, token groups), block = 512
__global__ void __launch_bounds__(64 * kXWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) stage_exact_kernel(StageDesc d, int batch)
{
    __shared__ v4i red[kXWaves][8][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int g = lane >> 4, n = lane & 15;
    const int rb = blockIdx.x, t0 = blockIdx.y * kXTokens;
    const int tok = t0 + n < batch ? t0 + n : batch - 1;            // a column past the batch repeats the last token and is not stored
    const char* w_base = (const char*)(d.tiles + (size_t)rb * d.n_steps * kTileWords) + 16 * lane;
    const char* b_base = (const char*)d.bq + (size_t)tok * d.n_steps * kBqStepBytes + 16 * g;
    v4i acc[kSlices][8];
#pragma unroll
    for (int s = 0; s < kSlices; ++s)
#pragma unroll
        for (int p = 0; p < 8; ++p) acc[s][p] = v4i{0, 0, 0, 0};
    // steps wave, wave + 8, ...; past the end the last step is read again and not used
    const int last = d.n_steps - 1;
    v4u w[kXRing], b[kXRing][kSlices];
#define NQ_X_ISSUE(k, step)                                                                             \
    do {                                                                                                \
        const uint32_t ss = (uint32_t)((step) < last ? (step) : last);                                  \
        w[k] = load_global_v4u(w_base, ss * (kTileWords * 4));                                          \
        _Pragma("unroll") for (int s = 0; s < kSlices; ++s)                                             \
            b[k][s] = load_global_v4u(b_base, ss * kBqStepBytes + 64 * s);                              \
    } while (0)
#define NQ_X_MAC(k)                                                                                     \
    do {                                                                                                \
        _Pragma("unroll") for (int p = 0; p < 8; ++p) {                                                 \
            const v4i a = (v4i)(w[k] & (0x01010101u << p));                                             \
            _Pragma("unroll") for (int s = 0; s < kSlices; ++s)                                         \
                acc[s][p] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, (v4i)b[k][s], acc[s][p], 0, 0, 0); \
        }                                                                                               \
    } while (0)
#pragma unroll
    for (int k = 0; k < kXRing; ++k) {
        NQ_X_ISSUE(k, wave + k * kXWaves);
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

    // the partial sums of the eight waves, one slice per round through 64 KiB of LDS; wave p takes bit plane p
    v4i sum[kSlices];
#pragma unroll
    for (int s = 0; s < kSlices; ++s) {
        if (s) __syncthreads();
#pragma unroll
        for (int p = 0; p < 8; ++p) red[wave][p][lane] = acc[s][p];
        __syncthreads();
        sum[s] = v4i{0, 0, 0, 0};
#pragma unroll
        for (int k = 0; k < kXWaves; ++k) sum[s] += red[k][wave][lane];
        if (wave == 7) sum[s] = -sum[s];                            // plane 7 is the int8 sign bit: it sums -128 b q
    }
    if (t0 + n >= batch) return;
    // lane (g, n), register v: row 16 plane + 4 g + v, token n; joined and rounded as in the decode kernels' epilogue
    const int row0 = rb * kTileRows + 16 * wave + 4 * g;
    const QMeta mt = d.meta[tok];
    const double scale_p = __builtin_ldexp(mt.two_step, -wave);
    float r[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const double raw = fma((double)sum[0][v], 65536.0, fma((double)sum[1][v], 256.0, (double)sum[2][v]));
        const float z = (float)fma(raw, scale_p, mt.neg_qs);
        r[v] = z * (d.out_scale && row0 + v < d.M ? half_bits_to_float(((gptr_u16)d.out_scale)[row0 + v]) : 1.0f);
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

int launch_stage_exact(const StageDesc& d, int batch, hipStream_t s)
{
    hipLaunchKernelGGL(stage_exact_kernel, dim3((unsigned)n_rowblocks(d.M), (unsigned)((batch + kXTokens - 1) / kXTokens)),
                       dim3(64 * kXWaves), 0, s, d, batch);
    NQ_HIP(hipGetLastError());
    return NQ_OK;
}

}  // namespace nq
