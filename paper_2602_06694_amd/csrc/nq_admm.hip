// Latent-binary ADMM on one matrix in binary64 (Section 3.2 Step 2-2 and 2-3; Appendix B): the dense
// products on the fp64 matrix cores, a blocked Cholesky with its inverse, the SVID proxy update by power
// iteration, the dual update and the magnitude balancing.  Host code only sequences launches.
#include "nq_internal.h"
#include "nq_lb_admm.h"

#include <math.h>
#include <algorithm>
#include <mutex>
#include <type_traits>

namespace nq {

typedef double v4d __attribute__((ext_vector_type(4)));

// ============================================================================================
//  C = alpha op(A) op(B) + beta Cin + diag I   [, C2 = C + E]        (batched along blockIdx.z)
// ============================================================================================
struct GemmArgs {
    const double* A;
    const double* B;
    const double* Cin;     // read only when beta != 0 (may be C)
    double* C;
    const double* E;       // optional second output C2 = C + E (both with ldc)
    double* C2;
    int M, N, K;
    int lda, ldb, ldcin, ldc;
    long long sA, sB, sC;  // elements between batch members (Cin, C share sC)
    int trans_a;           // 0: A stored [M][K];  1: stored [K][M]
    int trans_b;           // 0: B stored [K][N];  1: stored [N][K]
    double alpha, beta, diag;
    int tile;              // 0: by size; 1 / 2 / 3: 128 x 128, 128 x 64, 64 x 64 (an in-place product needs a tile as wide as N)
    int lower_only;        // tiles that lie entirely above the diagonal are skipped
    int k_from_max;        // the reduction starts at max(first row, first column) of the tile: both operands
                           // are lower triangular in the sense  op(A)[i][k] = 0 for k < i,  op(B)[k][j] = 0 for k < j
    int k_parts;           // > 1 (unbatched only): blockIdx.z takes the reduction range [z, z + 1) * k_per_part and
    int k_per_part;        // writes its partial product to Cp[z]; beta, Cin and diag apply to part 0 only
    int lds_pad;           // bytes of LDS requested beyond the kernel's need (fewer workgroups per CU, room for other launches)
    int prio;              // the waves raise their priority: a launch on the critical path that shares the CUs with a
                           // long product on another stream then gets the issue slots first
    double* Cp[8];
};

constexpr int kGemmThreads = 256;
constexpr int kBK = 16;        // reduction depth of one LDS tile = four 16x16x4 matrix instructions

// A workgroup of four or eight waves (2 x 2, 2 x 4) owns a BM x BN tile of C; each wave (BM/2) x (BN/2 or BN/4) of it as
// 16 x 16 accumulator tiles.  v_mfma_f64_16x16x4_f64: lane l supplies A[l & 15][l >> 4] and B[l >> 4][l & 15],
// and holds C[4 v + (l >> 4)][l & 15] in element v of its four accumulators.  Operand tiles go through LDS, double
// buffered: the global loads of tile kt + 1 are in flight while tile kt is multiplied.  The LDS layout of an
// operand follows the memory layout of its source, so that both the staging stores and the operand reads are
// free of bank conflicts: a source that is contiguous along the reduction (A stored [M][K], B stored [N][K]) is kept
// as [i][k] with a row pitch of 17 doubles, one that is contiguous along the tile's rows or columns as [k][i] with
// a pitch of BM + 16.  Two workgroups fit a CU (registers and LDS; a 128 x 128 one has its eight waves for that), so one's staging overlaps the other's products.
// PF: tiles held in registers ahead of the one being multiplied (4 for the 64 x 64 tile, whose
// launches are mostly short reductions that would otherwise wait a full memory latency per 16 columns).
// Bound: binary64 matrix cores, 66 to 68 of 77.7 TFLOP/s on large products (49 to 62 before the fetches lost their branches and 128 wide tiles their second wave per SIMD).
// TA, TB: the transpose flags as compile-time constants (LDS offsets become immediates of the LDS instructions).
template <int BM, int BN, int PF, bool TA, bool TB, int WAVES>
__device__ __forceinline__ void dgemm_body(const GemmArgs& g, const int bx, const int by, const int bz, double* lds_gemm)
{
    constexpr int PK = kBK + 1;
    constexpr int PA = BM + 16, PB = BN + 16;
    constexpr int SA = BM * PK > kBK * PA ? BM * PK : kBK * PA;
    constexpr int SB = BN * PK > kBK * PB ? BN * PK : kBK * PB;
    constexpr int WN = WAVES / 2;          // waves side by side
    constexpr int TM = BM / 32, TN = BN / 16 / WN;
    constexpr int kThreads = 64 * WAVES, LA = BM * kBK / kThreads, LB = BN * kBK / kThreads;
    double* As = lds_gemm;                 // [2][SA]
    double* Bs = lds_gemm + 2 * SA;        // [2][SB]

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i0 = by * BM, j0 = bx * BN;
    if (g.lower_only && j0 > i0 + BM - 1) return;
    if (g.prio) __builtin_amdgcn_s_setprio(2);
    const double* A = g.A + (size_t)(g.k_parts > 1 ? 0 : bz) * g.sA;
    const double* B = g.B + (size_t)(g.k_parts > 1 ? 0 : bz) * g.sB;
    const int part = g.k_parts > 1 ? bz : 0;
    const int zb = g.k_parts > 1 ? 0 : bz;
    const int k_begin = g.k_from_max ? ((i0 > j0 ? i0 : j0) / kBK) * kBK : part * g.k_per_part;
    const int k_end = g.k_parts > 1 && k_begin + g.k_per_part < g.K ? k_begin + g.k_per_part : g.K;
    const int n_full = k_end > k_begin ? (k_end - k_begin) / kBK : 0, k_rest = k_end > k_begin ? (k_end - k_begin) % kBK : 0;      // whole tiles and what is left
    const int wm0 = wave / WN * (BM / 2), wn0 = wave % WN * (BN / WN);
    constexpr bool ta = TA, tb = TB;
    // What a thread fetches does not change from tile to tile except for the reduction offset: the pointers (rows and columns beyond the matrix are
    // clamped to its last one: they only reach results that are not stored), the element's depth inside a tile and its place in LDS are set up once; the loop only
    // advances the pointers.  Whole tiles are fetched without a branch, past the last one that one again: with masks and conditions around the loads the compiler
    // waited for all of them before the products that they are meant to run beside.
    double ra[PF][LA], rb[PF][LB];
    const double* pa[LA];
    const double* pb[LB];
    int ka[LA], kb[LB], sa[LA], sb[LB];
    const size_t step_a = ta ? (size_t)kBK * g.lda : kBK, step_b = tb ? kBK : (size_t)kBK * g.ldb;
#pragma unroll
    for (int p = 0; p < LA; ++p) {
        const int idx = p * kThreads + tid;
        const int i = ta ? idx % BM : idx / kBK, k = ta ? idx / BM : idx % kBK;
        const int gi = i0 + i < g.M ? i0 + i : g.M - 1;
        ka[p] = k;
        sa[p] = ta ? k * PA + i : i * PK + k;
        pa[p] = ta ? A + (size_t)(k_begin + k) * g.lda + gi : A + (size_t)gi * g.lda + k_begin + k;
    }
#pragma unroll
    for (int p = 0; p < LB; ++p) {
        const int idx = p * kThreads + tid;
        const int j = tb ? idx / kBK : idx % BN, k = tb ? idx % kBK : idx / BN;
        const int gj = j0 + j < g.N ? j0 + j : g.N - 1;
        kb[p] = k;
        sb[p] = tb ? j * PK + k : k * PB + j;
        pb[p] = tb ? B + (size_t)gj * g.ldb + k_begin + k : B + (size_t)(k_begin + k) * g.ldb + gj;
    }
    int left = n_full - 1;                 // whole tiles behind the one that the pointers are at
    auto fetch = [&](double (&ra)[LA], double (&rb)[LB]) {
#pragma unroll
        for (int p = 0; p < LA; ++p) ra[p] = *pa[p];
#pragma unroll
        for (int p = 0; p < LB; ++p) rb[p] = *pb[p];
        const size_t da = left > 0 ? step_a : 0, db = left > 0 ? step_b : 0;
        --left;
#pragma unroll
        for (int p = 0; p < LA; ++p) pa[p] += da;
#pragma unroll
        for (int p = 0; p < LB; ++p) pb[p] += db;
    };
    auto stash = [&](int buf, const double (&ra)[LA], const double (&rb)[LB]) {
#pragma unroll
        for (int p = 0; p < LA; ++p) As[buf * SA + sa[p]] = ra[p];
#pragma unroll
        for (int p = 0; p < LB; ++p) Bs[buf * SB + sb[p]] = rb[p];
    };

    v4d acc[TM][TN];
#pragma unroll
    for (int a = 0; a < TM; ++a)
#pragma unroll
        for (int b = 0; b < TN; ++b) acc[a][b] = v4d{0.0, 0.0, 0.0, 0.0};

    // per-lane offsets of the operand reads: element (row l & 15 of a 16-row group, depth l >> 4 of a group of four)
    const int a_off = ta ? (lane >> 4) * PA + wm0 + (lane & 15) : (wm0 + (lane & 15)) * PK + (lane >> 4);
    constexpr int a_dk = ta ? 4 * PA : 4, a_dt = ta ? 16 : 16 * PK;
    const int b_off = tb ? (wn0 + (lane & 15)) * PK + (lane >> 4) : (lane >> 4) * PB + wn0 + (lane & 15);
    constexpr int b_dk = tb ? 4 : 4 * PB, b_dt = tb ? 16 * PK : 16;
    auto multiply = [&](int buf) {
        const double* Ab = As + buf * SA + a_off;
        const double* Bb = Bs + buf * SB + b_off;
        // Where a wave has few products per column of operands, the next four columns' are on their way while these are multiplied; 128 x 128 tiles have
        // enough of them, and the compiler's own order leaves their fetches more room (4096 x 1024 x 4096 526 us, so ordered 562; 128 x 64 533 and 601 (transposed) -> 521 and 512).
        constexpr bool kAhead = BN < 128;
        double a[2][TM], b[2][TN];
        auto read = [&](int k4) {
#pragma unroll
            for (int t = 0; t < TM; ++t) a[k4 & 1][t] = Ab[k4 * a_dk + t * a_dt];
#pragma unroll
            for (int t = 0; t < TN; ++t) b[k4 & 1][t] = Bb[k4 * b_dk + t * b_dt];
        };
        if (kAhead) read(0);
#pragma unroll
        for (int k4 = 0; k4 < kBK / 4; ++k4) {
            if (!kAhead) read(k4);
            else if (k4 + 1 < kBK / 4) read(k4 + 1);
            if (kAhead) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int tm = 0; tm < TM; ++tm)
#pragma unroll
                for (int tn = 0; tn < TN; ++tn)
                    acc[tm][tn] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[k4 & 1][tm], b[k4 & 1][tn], acc[tm][tn], 0, 0, 0);
            if (kAhead) __builtin_amdgcn_sched_barrier(0);
        }
    };

    if (n_full > 0) {
#pragma unroll
        for (int t = 0; t < PF; ++t) fetch(ra[t], rb[t]);
        stash(0, ra[0], rb[0]);
        __syncthreads();
        int kt0 = 0;
        for (; kt0 + PF <= n_full; kt0 += PF) {
            // slot sl went to LDS one tile ago: refill it with the tile PF ahead, multiply tile kt, then stage tile kt + 1
#pragma unroll
            for (int sl = 0; sl < PF; ++sl) {
                const int buf = (kt0 + sl) & 1;
                fetch(ra[sl], rb[sl]);
                multiply(buf);
                stash(buf ^ 1, ra[(sl + 1) % PF], rb[(sl + 1) % PF]);
                __syncthreads();
            }
        }
#pragma unroll
        for (int sl = 0; sl + 1 < PF; ++sl) {
            if (kt0 + sl < n_full) {
                const int buf = (kt0 + sl) & 1;
                multiply(buf);
                stash(buf ^ 1, ra[sl + 1], rb[sl + 1]);
                __syncthreads();
            }
        }
    }
    if (k_rest > 0) {                      // the ragged last tile
        const size_t da = n_full > 0 ? step_a : 0, db = n_full > 0 ? step_b : 0;
#pragma unroll
        for (int p = 0; p < LA; ++p) ra[0][p] = ka[p] < k_rest ? pa[p][da] : 0.0;
#pragma unroll
        for (int p = 0; p < LB; ++p) rb[0][p] = kb[p] < k_rest ? pb[p][db] : 0.0;
        stash(0, ra[0], rb[0]);
        __syncthreads();
        multiply(0);
    }

    const bool first = part == 0;
    const double* Cin = g.Cin && first ? g.Cin + (size_t)zb * g.sC : nullptr;
    double* C = g.k_parts > 1 ? g.Cp[part] : g.C + (size_t)zb * g.sC;
#pragma unroll
    for (int tm = 0; tm < TM; ++tm)
#pragma unroll
        for (int tn = 0; tn < TN; ++tn)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = i0 + wm0 + tm * 16 + 4 * v + (lane >> 4);
                const int j = j0 + wn0 + tn * 16 + (lane & 15);
                if (i < g.M && j < g.N) {
                    double val = g.alpha * acc[tm][tn][v];
                    if (g.beta != 0.0 && first) val = fma(g.beta, Cin[(size_t)i * g.ldcin + j], val);
                    if (i == j && first) val += g.diag;
                    C[(size_t)i * g.ldc + j] = val;
                    if (g.C2) g.C2[(size_t)i * g.ldc + j] = val + g.E[(size_t)i * g.ldc + j];
                }
            }
}

template <int BM, int BN, int PF, bool TA, bool TB, int WAVES>
__global__ __launch_bounds__(64 * WAVES, BM == 128 && BN == 128 ? 3 : 2) void dgemm_kernel(GemmArgs g)
{
    extern __shared__ __align__(16) double lds_dyn[];
    int bx = (int)blockIdx.x, by = (int)blockIdx.y;
    if (BM == BN && g.lower_only && g.M == g.N) {   // tile t of those on and below the diagonal, row by row
        by = (int)((__builtin_sqrtf(8.0f * (float)bx + 1.0f) - 1.0f) * 0.5f);
        while (by * (by + 1) / 2 > bx) --by;
        while ((by + 1) * (by + 2) / 2 <= bx) ++by;
        bx -= by * (by + 1) / 2;
    }
    dgemm_body<BM, BN, PF, TA, TB, WAVES>(g, bx, by, (int)blockIdx.z, lds_dyn);
}

template <int BM, int BN> constexpr size_t gemm_lds_bytes()
{
    constexpr int PK = kBK + 1;
    constexpr int SA = BM * PK > kBK * (BM + 16) ? BM * PK : kBK * (BM + 16);
    constexpr int SB = BN * PK > kBK * (BN + 16) ? BN * PK : kBK * (BN + 16);
    return (size_t)2 * (SA + SB) * sizeof(double);
}

constexpr int kGemmMaxLdsPad = 32768;

template <int BM, int BN, int PF, bool TA, bool TB, int WAVES> static int launch_gemm_variant(const GemmArgs& g, int batch, hipStream_t s)
{
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    constexpr size_t lds = gemm_lds_bytes<BM, BN>();
    std::call_once(once, [] {
        if (lds + kGemmMaxLdsPad > 65536)
            attr_err = hipFuncSetAttribute((const void*)dgemm_kernel<BM, BN, PF, TA, TB, WAVES>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)(lds + kGemmMaxLdsPad));
    });
    NQ_HIP(attr_err);
    dim3 grid((g.N + BN - 1) / BN, (g.M + BM - 1) / BM, batch);
    // Of a square matrix' lower half only the tiles that do work are launched: of a grid of all of them XCD k (workgroup mod 8) would get block
    // column k, and with it 8 - k of 8 tiles (Gram product of r = 1024, 4096 rows: 191 -> 135 us)
    if (BM == BN && g.lower_only && g.M == g.N) grid = dim3(grid.x * (grid.x + 1) / 2, 1, batch);
    const size_t pad = (size_t)(g.lds_pad < 0 ? 0 : g.lds_pad > kGemmMaxLdsPad ? kGemmMaxLdsPad : g.lds_pad);
    hipLaunchKernelGGL((dgemm_kernel<BM, BN, PF, TA, TB, WAVES>), grid, dim3(64 * WAVES), lds + pad, s, g);
    NQ_HIP(hipGetLastError());
    return NQ_OK;
}

template <int BM, int BN, int PF, int WAVES = 4> static int launch_gemm_tile(const GemmArgs& g, int batch, hipStream_t s)
{
    if (g.trans_a) return g.trans_b ? launch_gemm_variant<BM, BN, PF, true, true, WAVES>(g, batch, s) : launch_gemm_variant<BM, BN, PF, true, false, WAVES>(g, batch, s);
    return g.trans_b ? launch_gemm_variant<BM, BN, PF, false, true, WAVES>(g, batch, s) : launch_gemm_variant<BM, BN, PF, false, false, WAVES>(g, batch, s);
}

// Tile choice: 128 x 64 by eight waves or 64 x 64 by four, whichever gives the fullest CU less to do (in halves of a 128 x 64 tile; a 64 x 64 tile's half takes 1.06 of it; a
// 128 x 64 workgroup alone on its CU 1.15).  us, 128 x 64 / 64 x 64: 4096 x 1024 x 4096 514 / 550, x 1024 134 / 146, 4096^3 2019 / 2043, past the line
// 2048 x 1024 x 4096 307 / 275, 3072 x 1024 x 2048 (384 tiles) 256 / 201, 1024 x 1024 x 4096 302 / 192.  The option "dgemm_tile" (1: 128 x 128, 2: 128 x 64, 3: 64 x 64) overrides it.
// Four waves on 128 x 128 and 128 x 64 tiles, fetched under conditions, took 549 us for the first (569 transposed), 2346 for 4096^3, and 64 x 64 ones 300 for the last.
static int launch_gemm(const GemmArgs& g, int batch, hipStream_t s)
{
    if (g.M < 1 || g.N < 1 || batch < 1) return NQ_OK;
    auto tiles = [&](int bm, int bn) {            // workgroups that do work (with lower_only: those not entirely above the diagonal)
        const int tr = (g.M + bm - 1) / bm, tc = (g.N + bn - 1) / bn;
        long long n = 0;
        for (int i = 0; i < tr; ++i) n += g.lower_only ? std::min(tc, (i * bm + bm - 1) / bn + 1) : tc;
        return n * batch;
    };
    int choice = g.tile ? g.tile : opt_or(OPT_DGEMM_TILE, 0);
    if (choice < 1 || choice > 3) {
        const int cus = device_cu_count();
        const long long wide = (tiles(128, 64) + cus - 1) / cus, narrow = (tiles(64, 64) + cus - 1) / cus;
        choice = (wide == 1 ? 2.3 : 2.0 * wide) <= 1.06 * narrow ? 2 : 3;
    }
    if (choice == 1) return launch_gemm_tile<128, 128, 2, 8>(g, batch, s);
    if (choice == 2) return launch_gemm_tile<128, 64, 2, 8>(g, batch, s);
    return launch_gemm_tile<64, 64, 4>(g, batch, s);
}

__host__ __device__ static GemmArgs gemm_args(int ta, int tb, int M, int N, int K, double alpha, const double* A, int lda, const double* B, int ldb,
                          double beta, const double* Cin, int ldcin, double* C, int ldc)
{
    GemmArgs g{};
    g.A = A; g.B = B; g.Cin = Cin; g.C = C; g.E = nullptr; g.C2 = nullptr;
    g.M = M; g.N = N; g.K = K; g.lda = lda; g.ldb = ldb; g.ldcin = ldcin; g.ldc = ldc;
    g.sA = g.sB = g.sC = 0;
    g.trans_a = ta; g.trans_b = tb; g.alpha = alpha; g.beta = beta; g.diag = 0.0;
    g.tile = 0; g.lower_only = 0; g.k_from_max = 0;
    g.k_parts = 1; g.k_per_part = 0; g.prio = 0; g.lds_pad = 0;
    for (double*& c : g.Cp) c = nullptr;
    return g;
}

// ============================================================================================
//  Cholesky of one diagonal block and the inverse of its factor (one workgroup)
// ============================================================================================
constexpr int kNB = 64;        // width of a block column of the factorisation (an earlier 128-wide diagonal-block kernel measured slower than two of 64)

// the value of lane J of every 16-lane row, in all lanes of the row
template <int J>
__device__ __forceinline__ double row_bcast(double v)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x150 + J, 0xf, 0xf, true);      // row_newbcast
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x150 + J, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
template <int N, int I = 0, class F>
__device__ __forceinline__ void static_for(F f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        static_for<N, I + 1>(f);
    }
}

// One workgroup of four waves.  The 64 x 64 block and its inverse are kept in LDS as lower 16 x 16 tiles; four rounds of
//   * waves 0 and 1 eliminate the diagonal tile's 16 columns, one lane per column and its 16 rows in registers.  Beside the tile
//     wave 0 carries the tiles below it, transposed (lanes 16 to 63: the panel comes out of the same row operations), wave 1 the identity
//     (lanes 16 to 31: the tile's inverse).  A pivot is LDL^T's: what the next one waits for is a move between lanes, a reciprocal (the hardware's estimate
//     and two Newton steps), a product and one multiply-add; the multipliers reach the lanes of a 16-lane row by data-parallel moves from a copy of the tile that every row keeps.  The 16
//     square roots and their reciprocals follow together, one per lane, and scale rows and columns (within an ulp or two).
//   * 16 x 16 x 16 products on the matrix cores: the next column of tiles at once, by three waves; the other tiles and the off-diagonal tiles of
//     the inverse (X_kj = -X_kk sum_p L_kp X_pj) by waves 2 and 3 beside the next elimination.
// Bound by the 64 dependent pivots: of 18 us on its own, 3.5 are loads, 4 x 1.7 eliminations (2.4 with lane reads into
// scalars, whose use by the next instruction waits), 3 x 1 the products and barriers between them.
// H (lower part) is overwritten by L; the block of Linv receives L^-1 with an exactly zero upper part.  A pivot that is
// not > 0 sets *status (the results are then meaningless, every thread still finishes).
// A21 != nullptr: the block is the first tile of the trailing update of the block column before it, whose inverted diagonal block is X11: first
//  P = A21 X11^T,  which goes to L21 (both with leading dimension ldh), and  A <- A - P P^T,  so that the update's other tiles can run beside this
// kernel's work.  Everything is requested at once and P stays in LDS (with the tiles' bodies below: step launch 24 -> 19 us on its own, 52 beside the product with W).
// lds: kPotrfLdsBytes bytes.
// registers for three waves per SIMD (168), so that such a workgroup fits beside one of the product with W (two waves of 144): otherwise it waits for its end
constexpr int kStepWavesPerEu = 3;
constexpr int kTilePitch = 17, kTileDoubles = 16 * kTilePitch;         // operand reads of all three forms are free of bank conflicts
constexpr int kPitchP = kNB + 1;
constexpr size_t kPotrfLdsBytes = (kNB * kPitchP + 10 * kTileDoubles) * sizeof(double);      // P and X11; then the block's tiles and its inverse's

__device__ __forceinline__ void potrf_inv_body(double* H, int ldh, double* Linv, int ldi, int o, int* status, int prio, const double* A21,
                                               const double* X11, double* L21, double* lds)
{
    if (prio) __builtin_amdgcn_s_setprio(3);
    static_assert(kNB == 64 && kGemmThreads == 256, "four tiles a side, four waves");
    static_assert(20 * kTileDoubles * sizeof(double) <= kPotrfLdsBytes, "the tiles go where P and X11 were");
    double* const A = lds;
    double* const X = lds + 10 * kTileDoubles;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int g = lane >> 4, n = lane & 15;
    auto tile = [](int i, int j) { return (i * (i + 1) / 2 + j) * kTileDoubles; };
    {
        v4d acc[3];
        int ti[3], tj[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            const int t = wave + 4 * u;
            ti[u] = t < 1 ? 0 : t < 3 ? 1 : t < 6 ? 2 : 3;
            tj[u] = t - ti[u] * (ti[u] + 1) / 2;
            if (t < 10)
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[u][v] = H[(size_t)(o + 16 * ti[u] + 4 * v + g) * ldh + o + 16 * tj[u] + n];
        }
        if (A21) {
            double* const P = lds;                 // [64][65]: rows of A21, then of P; a wave's 16 rows are its own
            double* const XT = lds + kNB * kPitchP;
            {
                const int row = threadIdx.x >> 2, c = threadIdx.x & 3;
                const double *pa = A21 + (size_t)row * ldh + 16 * c, *px = X11 + (size_t)row * ldi + 16 * c;
                double av[16], xv[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) av[k] = pa[k];
                if (c <= row >> 4)
#pragma unroll
                    for (int k = 0; k < 16; ++k) xv[k] = px[k];
#pragma unroll
                for (int k = 0; k < 16; ++k) P[row * kPitchP + 16 * c + k] = av[k];
                if (c <= row >> 4)
#pragma unroll
                    for (int k = 0; k < 16; ++k) XT[tile(row >> 4, c) + (row & 15) * kTilePitch + k] = xv[k];
            }
            __syncthreads();
            double a[16];
#pragma unroll
            for (int s = 0; s < 16; ++s) a[s] = P[(16 * wave + n) * kPitchP + 4 * s + g];
            v4d p[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) p[j] = v4d{0.0, 0.0, 0.0, 0.0};
            // (depth outside: four independent sums at a time; X11 is lower triangular)
#pragma unroll
            for (int s = 0; s < 16; ++s)
#pragma unroll
                for (int j = s / 4; j < 4; ++j)
                    p[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], XT[tile(j, s / 4) + n * kTilePitch + 4 * (s % 4) + g], p[j], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    P[(16 * wave + 4 * v + g) * kPitchP + 16 * j + n] = p[j][v];
                    L21[(size_t)(16 * wave + 4 * v + g) * ldh + 16 * j + n] = p[j][v];
                }
            __syncthreads();
            v4d sum[3];
#pragma unroll
            for (int u = 0; u < 3; ++u) sum[u] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int s = 0; s < kNB / 4; ++s)
#pragma unroll
                for (int u = 0; u < 3; ++u)
                    if (wave + 4 * u < 10)
                        sum[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(P[(16 * ti[u] + n) * kPitchP + g + 4 * s], P[(16 * tj[u] + n) * kPitchP + g + 4 * s], sum[u], 0, 0, 0);
#pragma unroll
            for (int u = 0; u < 3; ++u)
                if (wave + 4 * u < 10) acc[u] -= sum[u];
            __syncthreads();                       // everybody has read P: the tiles go where it was
        }
#pragma unroll
        for (int u = 0; u < 3; ++u)
            if (wave + 4 * u < 10)
#pragma unroll
                for (int v = 0; v < 4; ++v) A[tile(ti[u], tj[u]) + (4 * v + g) * kTilePitch + n] = acc[u][v];
    }
    __syncthreads();
    bool bad = false;

    // what waves do on the matrix cores; the operands are read as [row n][depth 4 s + g], or, for an untransposed right factor, [depth][column n]
    auto load_c = [&](const double* c) {
        v4d acc;
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[v] = c[(4 * v + g) * kTilePitch + n];
        return acc;
    };
    auto store_c = [&](double* c, v4d acc) {
#pragma unroll
        for (int v = 0; v < 4; ++v) c[(4 * v + g) * kTilePitch + n] = acc[v];
    };
    auto sub_aat = [&](int i, int j, int kb) {     // A_ij -= P_i P_j^T
        const double *pi = A + tile(i, kb) + n * kTilePitch + g, *pj = A + tile(j, kb) + n * kTilePitch + g;
        v4d acc = load_c(A + tile(i, j));
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-pi[4 * s], pj[4 * s], acc, 0, 0, 0);
        store_c(A + tile(i, j), acc);
    };
    auto sum_lx = [&](int k, int j) {              // X_kj <- sum over j <= p < k of L_kp X_pj
        v4d acc = {0.0, 0.0, 0.0, 0.0};
        for (int p = j; p < k; ++p) {
            const double *l = A + tile(k, p) + n * kTilePitch + g, *x = X + tile(p, j) + g * kTilePitch + n;
#pragma unroll
            for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(l[4 * s], x[4 * s * kTilePitch], acc, 0, 0, 0);
        }
        store_c(X + tile(k, j), acc);
    };
    auto finish_x = [&](int k, int j) {            // X_kj <- -X_kk X_kj
        const double *l = X + tile(k, k) + n * kTilePitch + g, *x = X + tile(k, j) + g * kTilePitch + n;
        v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-l[4 * s], x[4 * s * kTilePitch], acc, 0, 0, 0);
        store_c(X + tile(k, j), acc);
    };

    for (int kb = 0; kb < 4; ++kb) {
        // d: the diagonal tile's column n, in all four 16-lane rows of the wave (a value of lane j of a row reaches its other lanes by a
        // data-parallel move); v: the lane's other column
        double d[16], v[16], root = 0.0;
        const int below = kb + g;                  // the panel tile of wave 0's lanes
        if (wave < 2) {
            const double* const t = A + tile(kb, kb);
            const double* const p = A + tile(g > 0 && below < 4 ? below : kb, kb) + n * kTilePitch;
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                d[i] = t[i >= n ? i * kTilePitch + n : n * kTilePitch + i];
                v[i] = wave == 0 ? p[i] : (i == n ? 1.0 : 0.0);
            }
            double mine = 1.0;
            static_for<16>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                const double piv = row_bcast<j>(d[j]);
                if (!(piv > 0.0)) bad = true;
                double y = __builtin_amdgcn_rcp(piv);
                y = fma(y, fma(-piv, y, 1.0), y);
                y = fma(y, fma(-piv, y, 1.0), y);
                mine = n == j ? piv : mine;
                const double rd = n > j ? -d[j] * y : 0.0, rv = -v[j] * y;     // (columns that are done stay)
#pragma unroll
                for (int i = j + 1; i < 16; ++i) {
                    const double m = row_bcast<j>(d[i]);
                    d[i] = fma(m, rd, d[i]);
                    v[i] = fma(m, rv, v[i]);
                }
            });
            double y = __builtin_amdgcn_rsq(mine);
            double h = 0.5 * y;
            root = mine * y;
            double e = fma(-h, root, 0.5);
            root = fma(root, e, root);
            h = fma(h, e, h);
            e = fma(-h, root, 0.5);
            root = fma(root, e, root);
            h = fma(h, e, h);
            e = fma(-root, root, mine);
            root = fma(e, h, root);
            y = 2.0 * h;
            static_for<16>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                v[i] *= row_bcast<i>(y);
                d[i] *= y;
            });
            if (wave == 0 && g > 0 && below < 4) {
                double* const to = A + tile(below, kb) + n * kTilePitch;
#pragma unroll
                for (int i = 0; i < 16; ++i) to[i] = v[i];
            }
            if (wave == 1 && g == 1) {
                double* const to = X + tile(kb, kb) + n;
#pragma unroll
                for (int i = 0; i < 16; ++i) to[i * kTilePitch] = v[i];
            }
        }
        __syncthreads();                           // the panel and X_kk
        if (wave == 0 && g == 0) {
            double* const to = A + tile(kb, kb) + n;
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (i >= n) to[i * kTilePitch] = i == n ? root : d[i];
        }
        if (kb == 3) break;
        if (wave < 3 - kb) sub_aat(kb + 1 + wave, kb + 1, kb);
        __syncthreads();                           // the next column of tiles
        if (wave == 2) {
            if (kb > 0) finish_x(kb, 0);
            sum_lx(kb + 1, 0);
            if (kb == 0) sub_aat(3, 3, 0);
        } else if (wave == 3) {
            if (kb == 0) {
                sub_aat(2, 2, 0);
                sub_aat(3, 2, 0);
            } else if (kb == 1) {
                sub_aat(3, 3, 1);
                sum_lx(2, 1);
            } else {
                finish_x(2, 1);
                sum_lx(3, 1);
                sum_lx(3, 2);
            }
        }
    }
    if (wave < 3) finish_x(3, wave);
    __syncthreads();
    // (a wave stores whole rows)
#pragma unroll 4
    for (int q = 0; q < kNB / 4; ++q) {
        const int i = 4 * q + wave, at = tile(i >> 4, g) + (i & 15) * kTilePitch + n;
        if (lane <= i) H[(size_t)(o + i) * ldh + o + lane] = A[at];
        Linv[(size_t)(o + i) * ldi + o + lane] = lane <= i ? X[g <= (i >> 4) ? at : 0] : 0.0;
    }
    if (bad) *status = 1;
}

__global__ __launch_bounds__(kGemmThreads, kStepWavesPerEu) void potrf_inv_kernel(double* H, int ldh, double* Linv, int ldi, int o, int* status, int prio)
{
    extern __shared__ __align__(16) double lds_dyn[];
    potrf_inv_body(H, ldh, Linv, ldi, o, status, prio, nullptr, nullptr, nullptr, lds_dyn);
}

// One launch per block column k of the factorisation, after the diagonal block k has been factorised and inverted
// (X = L11^-1): the panel  P = A21 X^T  (the rows of L below the diagonal block), the trailing update  A22 -= P P^T
// (lower tiles), and the factorisation of the next diagonal block.  Nothing is handed from one workgroup to another:
//   * workgroup (0, 0) forms the first 64 rows of P, stores them as that block of L, applies  P P^T  to the diagonal
//     block k + 1 in its registers and factorises it (the long pole of the launch);
//   * workgroup (j, i + 1), j <= i, (i, j) != (0, 0), owns tile (i, j) of the trailing matrix: it forms the rows P_i and
//     P_j of the panel for itself (three 64 x 64 x 64 products instead of one; they cost little next to the
//     factorisation beside them) and subtracts  P_i P_j^T  from its tile; tile (i, 0) stores P_i as block i of L.
//   * with `S`, workgroup (i, tiles + 1 + j), j <= k, carries the inverse along: it forms P_i and the block
//     X_kj = -X_kk S_kj  of row k of L^-1 for itself (the first of the column also stores it) and adds  P_i X_kj  to  S_ij,
//     the sum of L_ip X_pj over p < i that row k + 1 + i of L^-1 waits for.  As many products as a tile of the trailing matrix takes, in the same
//     launch, while the diagonal block is factorised: what is left of the inversion afterwards is one row of blocks, where
//     inverting by halves took eight launches, 185 us for r = 1024.
// The last two run as one body (step_tile_body): everything is requested at once, a wave owns 16 rows of each product, whose first operand needs only its
// own rows, and what the other waves need of the first products passes through LDS.  (As three general products through memory, each waiting for its
// first tiles, they took 24 us, longer than the factorisation.)
// The panel is NOT written over A21: other workgroups still read A21, so L's blocks below the diagonal go to a matrix
// of their own (Lb; the diagonal blocks of L stay in H).  A step is then one launch of the factorisation's length
// where the panel, the update and the factorisation as launches of their own take three.
struct StepArgs {
    double* H;          // [..][ld]: A21, A22 (read and updated in place), diagonal blocks of L
    double* Lb;         // [..][ld]: L below the diagonal
    double* Linv;       // [..][ld]: the inverted diagonal blocks
    int ld, o, prio;    // o: first row / column of block column k
    int* status;
    int tiles;          // row blocks below block column k
    double* S;          // [..][ld] sums behind the rows of L^-1 still to come, or nullptr
};

constexpr size_t kStepLdsBytes = 2 * kNB * kPitchP * sizeof(double);       // two blocks, 65 KiB; beside the product with W (80.5) that still fits a CU

// INV = false: C -= P_i P_j^T with P_j from B = A21_j (the same as P_i where B is nullptr); INV = true: C (+)= P_i Y with Y = -X11 B, B = S_kj, or Y = X11
// (B nullptr).  P_i = A21_i X11^T.  store_p: where P_i goes, store_y: Y (leading dimension ld), or nullptr.
template <bool INV>
__device__ __forceinline__ void step_tile_body(const double* A21i, const double* X11, const double* B, double* C, bool add, double* store_p, double* store_y, int ld,
                                               double* lds)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int g = lane >> 4, n = lane & 15;
    auto tile = [](int i, int j) { return (i * (i + 1) / 2 + j) * kTileDoubles; };
    double* const R0 = lds;                        // X11's lower tiles, then P_i
    double* const R1 = lds + kNB * kPitchP;        // P_j, or S_kj and then Y
    const int row = threadIdx.x >> 2, c4 = threadIdx.x & 3;
    double x[16], b[16], ai[16];
    v4d acc[4], pi[4], q[4];
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = X11[(size_t)row * ld + 16 * c4 + k];
#pragma unroll
    for (int s = 0; s < 16; ++s) ai[s] = A21i[(size_t)(16 * wave + n) * ld + 4 * s + g];
    if (B)
#pragma unroll
        for (int s = 0; s < 16; ++s) b[s] = INV ? B[(size_t)row * ld + 16 * c4 + s] : B[(size_t)(16 * wave + n) * ld + 4 * s + g];
    if (c4 <= row >> 4)
#pragma unroll
        for (int k = 0; k < 16; ++k) R0[tile(row >> 4, c4) + (row & 15) * kTilePitch + k] = x[k];
    if (INV)
#pragma unroll
        for (int k = 0; k < 16; ++k) R1[row * kPitchP + 16 * c4 + k] = B ? b[k] : x[k];
    __syncthreads();
    auto times_xt = [&](const double (&a)[16], v4d (&p)[4]) {      // 16 rows times X11^T, which is upper triangular
#pragma unroll
        for (int c = 0; c < 4; ++c) p[c] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int s = 0; s < 16; ++s)
#pragma unroll
            for (int c = s / 4; c < 4; ++c)
                p[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[s], R0[tile(c, s / 4) + n * kTilePitch + 4 * (s % 4) + g], p[c], 0, 0, 0);
    };
    auto to_rows = [&](double* r, const v4d (&p)[4]) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) r[(16 * wave + 4 * v + g) * kPitchP + 16 * c + n] = p[c][v];
    };
    auto to_memory = [&](double* m, const v4d (&p)[4]) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) m[(size_t)(16 * wave + 4 * v + g) * ld + 16 * c + n] = p[c][v];
    };
    times_xt(ai, pi);
    if (!INV) {
        if (B) {
            times_xt(b, q);
            to_rows(R1, q);
        } else to_rows(R1, pi);
    } else if (B) {
#pragma unroll
        for (int c = 0; c < 4; ++c) q[c] = v4d{0.0, 0.0, 0.0, 0.0};
        for (int t = 0; t <= wave; ++t)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const double xs = -R0[tile(wave, t) + n * kTilePitch + 4 * s + g];
#pragma unroll
                for (int c = 0; c < 4; ++c) q[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(xs, R1[(16 * t + 4 * s + g) * kPitchP + 16 * c + n], q[c], 0, 0, 0);
            }
    }
    __syncthreads();                               // X11 (and S_kj) have been read
    to_rows(R0, pi);
    if (INV && B) to_rows(R1, q);
    if (store_p) to_memory(store_p, pi);
    if (INV && store_y) to_memory(store_y, q);
    v4d old[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        acc[c] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int v = 0; v < 4; ++v) old[c][v] = add ? C[(size_t)(16 * wave + 4 * v + g) * ld + 16 * c + n] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 16; ++s) {
        const double p = R0[(16 * wave + n) * kPitchP + 4 * s + g];
#pragma unroll
        for (int c = 0; c < 4; ++c)
            acc[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(p, INV ? R1[(4 * s + g) * kPitchP + 16 * c + n] : R1[(16 * c + n) * kPitchP + 4 * s + g], acc[c], 0, 0, 0);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[c] = INV ? old[c] + acc[c] : old[c] - acc[c];
    to_memory(C, acc);
}

__global__ __launch_bounds__(kGemmThreads, kStepWavesPerEu) void chol_step_kernel(StepArgs a)
{
    static_assert(kGemmThreads == 256 && kNB == 64, "both bodies are written for 256 threads and 64-wide blocks");
    extern __shared__ __align__(16) double lds_dyn[];
    const int ld = a.ld;
    const double* const X = a.Linv + (size_t)a.o * ld + a.o;
    double* const A21 = a.H + (size_t)(a.o + kNB) * ld + a.o;
    double* const L21 = a.Lb + (size_t)(a.o + kNB) * ld + a.o;
    if (blockIdx.y == 0) {
        if (blockIdx.x != 0) return;
        potrf_inv_body(a.H, ld, a.Linv, ld, a.o + kNB, a.status, a.prio, A21, X, L21, lds_dyn);
        return;
    }
    if (a.prio) __builtin_amdgcn_s_setprio(2);
    if ((int)blockIdx.y > a.tiles) {
        const int i = (int)blockIdx.x, j = (int)blockIdx.y - a.tiles - 1, k = a.o / kNB;
        step_tile_body<true>(A21 + (size_t)i * kNB * ld, X, j < k ? a.S + (size_t)a.o * ld + j * kNB : nullptr, a.S + (size_t)(a.o + (i + 1) * kNB) * ld + j * kNB, j < k,
                             nullptr, i == 0 && j < k ? a.Linv + (size_t)a.o * ld + j * kNB : nullptr, ld, lds_dyn);
        return;
    }
    const int i = (int)blockIdx.y - 1, j = (int)blockIdx.x;
    if (j > i || i == 0) return;                   // above the diagonal; (0, 0) is the diagonal block's
    step_tile_body<false>(A21 + (size_t)i * kNB * ld, X, j < i ? A21 + (size_t)j * kNB * ld : nullptr, a.H + (size_t)(a.o + kNB + i * kNB) * ld + a.o + kNB + j * kNB, true,
                          j == 0 ? L21 + (size_t)i * kNB * ld : nullptr, nullptr, ld, lds_dyn);
}

// A += the other parts, in their order, on the leading r x r part of [rp][rp] matrices (the partial Gram products of a
// split reduction; part 0 is A itself).
struct GramParts {
    const double* p[8];
    int n;
};
__global__ void add_parts_kernel(double* A, GramParts parts, int rp, int r)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= r) return;
    const size_t at = (size_t)blockIdx.y * rp + j;
    double v = A[at];
    for (int q = 1; q < parts.n; ++q) v += parts.p[q][at];
    A[at] = v;
}

// Identity outside the leading r x r part of a [rp][rp] matrix (the padding that keeps the block algorithms
// exact: an identity block factorises and inverts to itself); `zero_inside` also clears the leading part.
__global__ void pad_identity_kernel(double* A, int rp, int r, int zero_inside)
{
    const size_t n = (size_t)rp * rp;
    for (size_t e = (size_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (size_t)gridDim.x * blockDim.x) {
        const int i = (int)(e / rp), j = (int)(e % rp);
        if (i >= r || j >= r) A[e] = (i == j) ? 1.0 : 0.0;
        else if (zero_inside) A[e] = 0.0;
    }
}

// ============================================================================================
//  SVID: power iteration on |P| and the proxy / dual update
// ============================================================================================
constexpr int kRowsPerWg = 16;

__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
    return v;
}

// Sum over the workgroup of one value per thread (256 threads); every thread gets the result.
__device__ __forceinline__ double block_sum(double v, double* scratch4)
{
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) scratch4[threadIdx.x >> 6] = v;
    __syncthreads();
    return (scratch4[0] + scratch4[1]) + (scratch4[2] + scratch4[3]);
}

constexpr int kWParts = 8;      // the vector of a round is kept as eight partial vectors, added in a fixed order by its readers

__device__ __forceinline__ double w_at(const double* w8, int r, int k)
{
    return ((w8[k] + w8[r + k]) + (w8[2 * r + k] + w8[3 * r + k])) + ((w8[4 * r + k] + w8[5 * r + k]) + (w8[6 * r + k] + w8[7 * r + k]));
}

// One round of the power iteration in one pass over P [n][r]: for the 16 rows of this workgroup
//     a_i = sum_k |P[i][k]| b_k          with b = w / ||w||   (w: the unnormalised vector of the round before)
// and, unless `rows_only`, this workgroup's part of the next unnormalised vector  w'_k = sum_i |P[i][k]| a_i
// (partial[g][k]; a second kernel adds the parts in a fixed order).  `ones`: a_i = 1 instead (the start vector;
// its scale does not matter, the next round normalises).  w is staged in LDS (dynamic, r doubles).
__global__ __launch_bounds__(256) void power_pass_kernel(const double* P, int n, int r, const double* w8, int ones, int rows_only,
                                                          double* a_out, double* partial)
{
    extern __shared__ __align__(16) double w_s[];
    __shared__ double red[4];
    __shared__ double a_s[kRowsPerWg];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row0 = blockIdx.x * kRowsPerWg;
    if (!ones) {
        double q = 0.0;
        for (int k = tid; k < r; k += 256) {
            const double v = w_at(w8, r, k);
            w_s[k] = v;
            q = fma(v, v, q);
        }
        const double inv = 1.0 / sqrt(block_sum(q, red));           // its barriers also publish w_s
        constexpr int RW = kRowsPerWg / 4;                          // rows per wave, taken together
        double d[RW];
        const double* rowp[RW];
#pragma unroll
        for (int rr = 0; rr < RW; ++rr) {
            const int i = row0 + wave * RW + rr;
            d[rr] = 0.0;
            rowp[rr] = P + (size_t)(i < n ? i : n - 1) * r;        // a row beyond the end reads the last row, its result is dropped
        }
#pragma unroll 2
        for (int k = lane; k < r; k += 64) {
            const double wk = w_s[k];
#pragma unroll
            for (int rr = 0; rr < RW; ++rr) d[rr] = fma(fabs(rowp[rr][k]), wk, d[rr]);
        }
#pragma unroll
        for (int rr = 0; rr < RW; ++rr) {
            const int i = row0 + wave * RW + rr;
            const double v = wave_sum(d[rr]) * inv;
            if (lane == 0) {
                a_s[wave * RW + rr] = i < n ? v : 0.0;
                if (i < n) a_out[i] = v;
            }
        }
    } else if (tid < kRowsPerWg) {
        a_s[tid] = row0 + tid < n ? 1.0 : 0.0;
    }
    __syncthreads();
    if (rows_only) return;
    for (int k = tid; k < r; k += 256) {
        double c = 0.0;
#pragma unroll
        for (int rr = 0; rr < kRowsPerWg; ++rr) {
            const int i = row0 + rr;
            c = fma(fabs(P[(size_t)(i < n ? i : n - 1) * r + k]), a_s[rr], c);      // a_s = 0 beyond the end
        }
        partial[(size_t)blockIdx.x * r + k] = c;
    }
}

// w8[q][k] = sum over the parts g = q, q + 8, q + 16, ... of partial[g][k], added in index order by four threads per
// column whose results are combined in a fixed tree.
__global__ __launch_bounds__(256) void power_reduce_kernel(const double* partial, int n_parts, int r, double* w8)
{
    __shared__ double s[4][64];
    const int c = threadIdx.x & 63, t = threadIdx.x >> 6;
    const int k = blockIdx.x * 64 + c, q = blockIdx.y;
    double acc = 0.0;
    if (k < r)
        for (int g = q + kWParts * t; g < n_parts; g += kWParts * 4) acc += partial[(size_t)g * r + k];
    s[t][c] = acc;
    __syncthreads();
    if (t == 0 && k < r) w8[(size_t)q * r + k] = (s[0][c] + s[1][c]) + (s[2][c] + s[3][c]);
}

// Z = sign(P) (.) (a b^T) with b = w / ||w||  (power_iters = 0: the constant sum(w) / (n r), w = |P|^T 1),
// and the dual update in its two forms:  first = 0:  Lambda = P - Z  (P = X + Lambda_old, so this is
// Lambda_old + X - Z),  D = Z - Lambda;   first = 1 (initial state):  Lambda = 0,  D = Z.
__global__ __launch_bounds__(256) void svid_finish_kernel(const double* P, int n, int r, const double* a, const double* w8, int zero_rounds,
                                                           int first, double* Z, double* Lambda, double* D)
{
    extern __shared__ __align__(16) double w_s[];
    __shared__ double red[4];
    const int tid = threadIdx.x;
    double q = 0.0;
    for (int k = tid; k < r; k += 256) {
        const double v = w_at(w8, r, k);
        w_s[k] = v;
        q = zero_rounds ? q + v : fma(v, v, q);
    }
    const double tot = block_sum(q, red);
    const double scale = zero_rounds ? tot / ((double)n * (double)r) : 1.0 / sqrt(tot);
    const int row0 = blockIdx.x * kRowsPerWg;
    for (int k = tid; k < r; k += 256) {
        const double bk = zero_rounds ? scale : w_s[k] * scale;
#pragma unroll 4
        for (int rr = 0; rr < kRowsPerWg; ++rr) {
            const int i = row0 + rr;
            if (i >= n) break;
            const size_t e = (size_t)i * r + k;
            const double p = P[e];
            const double mag = zero_rounds ? scale : a[i] * bk;
            const double z = (p >= 0.0) ? mag : -mag;
            Z[e] = z;
            const double lam = first ? 0.0 : p - z;
            Lambda[e] = lam;
            D[e] = z - lam;
        }
    }
}

// ============================================================================================
//  Magnitude balancing (Step 2-3)
// ============================================================================================
__global__ __launch_bounds__(256) void sumsq_kernel(const double* X, const double* L, size_t count, double* partial)
{
    __shared__ double red[4];
    double q = 0.0;
    for (size_t e = (size_t)blockIdx.x * 256 + threadIdx.x; e < count; e += (size_t)gridDim.x * 256) {
        const double p = X[e] + L[e];
        q = fma(p, p, q);
    }
    const double t = block_sum(q, red);
    if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

constexpr int kSumParts = 256;

// One wave per row: scale[i] = mean_k |f p_ik| with f = eta (which = 0) or 1 / eta (which = 1), p = X + L, and the
// packed sign bits of the row (bit = 1 iff p >= 0; a NaN packs as 0).
__global__ __launch_bounds__(256) void balance_rows_kernel(const double* X, const double* L, int rows, int r, const double* parts_u,
                                                            const double* parts_v, int which, uint32_t* words, double* scale, double* eta_out)
{
    __shared__ double red[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const double su = block_sum(parts_u[tid], red);
    const double sv = block_sum(parts_v[tid], red);
    const double eta = sqrt(sqrt(sv) / sqrt(su));
    if (eta_out && blockIdx.x == 0 && tid == 0) *eta_out = eta;
    const double f = which == 0 ? eta : 1.0 / eta;
    const int i = blockIdx.x * 4 + wave;
    if (i >= rows) return;
    const int n_words = (r + 31) / 32;
    double acc = 0.0;
    for (int c = 0; c * 64 < r; ++c) {
        const int k = c * 64 + lane;
        double p = -1.0;
        if (k < r) {
            p = X[(size_t)i * r + k] + L[(size_t)i * r + k];
            acc += fabs(f * p);
        }
        const unsigned long long bits = __ballot(k < r && p >= 0.0);
        if (lane == 0) {
            words[(size_t)i * n_words + 2 * c] = (uint32_t)bits;
            if (2 * c + 1 < n_words) words[(size_t)i * n_words + 2 * c + 1] = (uint32_t)(bits >> 32);
        }
    }
    acc = wave_sum(acc);
    if (lane == 0) scale[i] = acc / (double)r;
}

// ============================================================================================
//  Host side: workspace layout and the sequence of launches
// ============================================================================================
static int64_t next_pow2(int64_t v) { int64_t p = 1; while (p < v) p <<= 1; return p; }
static size_t up256(size_t b) { return (b + 255) & ~(size_t)255; }

struct AdmmWs {
    int rp;            // padded side of the r x r matrices: 64 * 2^ceil(log2(ceil(r/64)))
    int rr;            // 64 * ceil(r/64): the part the factorisation touches
    double *H, *Linv, *Hinv, *T, *RHS, *P, *DU, *DV, *a, *w, *partial, *parts_u, *parts_v;
    double* G[3];      // three more [rp][rp] buffers for the parts of the Gram product's reduction (small ranks only, else nullptr)
    int* status;
    size_t bytes;
};

constexpr int kGramSixPartsMaxSide = 2048;

static AdmmWs carve(void* base, int64_t n, int64_t m, int64_t r)
{
    AdmmWs ws{};
    const int64_t q = (r + kNB - 1) / kNB;
    ws.rr = (int)(q * kNB);
    ws.rp = (int)(next_pow2(q) * kNB);
    const int64_t big = n > m ? n : m;
    size_t off = 0;
    auto take = [&](size_t count) { double* p = base ? (double*)((char*)base + off) : nullptr; off += up256(count * sizeof(double)); return p; };
    const size_t sq = (size_t)ws.rp * ws.rp;
    ws.H = take(sq); ws.Linv = take(sq); ws.Hinv = take(sq); ws.T = take(sq);
    // (a small Gram matrix has few tiles: its reduction is cut into six parts instead of three to fill the chip)
    for (double*& gp : ws.G) gp = ws.rp <= kGramSixPartsMaxSide ? take(sq) : nullptr;
    ws.RHS = take((size_t)big * r); ws.P = take((size_t)big * r);
    ws.DU = take((size_t)n * r); ws.DV = take((size_t)m * r);
    ws.a = take(big); ws.w = take((size_t)kWParts * r);
    ws.partial = take((size_t)((big + kRowsPerWg - 1) / kRowsPerWg) * r);
    ws.parts_u = take(kSumParts); ws.parts_v = take(kSumParts);
    ws.status = (int*)take(32);
    ws.bytes = off;
    return ws;
}

// SVID of P [rows][r] by `iters` rounds of power iteration; writes Z, Lambda and D = Z - Lambda.
static int svid(const AdmmWs& ws, const double* P, int rows, int r, int iters, int first, double* Z, double* Lambda, double* D, hipStream_t s)
{
    const int n_wg = (rows + kRowsPerWg - 1) / kRowsPerWg;
    const dim3 red_grid((r + 63) / 64, kWParts);
    const size_t lds = (size_t)r * sizeof(double);
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [] {        // r doubles of dynamic LDS plus the kernels' own few words can pass 64 KiB at the largest rank
        const int most = NQ_ADMM_MAX_RANK * (int)sizeof(double);
        attr_err = hipFuncSetAttribute((const void*)power_pass_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, most);
        if (attr_err == hipSuccess) attr_err = hipFuncSetAttribute((const void*)svid_finish_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, most);
    });
    NQ_HIP(attr_err);
    // w = |P|^T 1
    hipLaunchKernelGGL(power_pass_kernel, dim3(n_wg), dim3(256), lds, s, P, rows, r, (const double*)nullptr, 1, 0, ws.a, ws.partial);
    hipLaunchKernelGGL(power_reduce_kernel, red_grid, dim3(256), 0, s, ws.partial, n_wg, r, ws.w);
    for (int it = 0; it < iters; ++it) {
        // a = |P| b with b = w / ||w||; and, except in the last round, the next w = |P|^T a
        const int last = it + 1 == iters;
        hipLaunchKernelGGL(power_pass_kernel, dim3(n_wg), dim3(256), lds, s, P, rows, r, (const double*)ws.w, 0, last, ws.a, ws.partial);
        if (!last) hipLaunchKernelGGL(power_reduce_kernel, red_grid, dim3(256), 0, s, ws.partial, n_wg, r, ws.w);
    }
    hipLaunchKernelGGL(svid_finish_kernel, dim3(n_wg), dim3(256), lds, s, P, rows, r, (const double*)ws.a, (const double*)ws.w, iters == 0 ? 1 : 0, first,
                       Z, Lambda, D);
    NQ_HIP(hipGetLastError());
    return NQ_OK;
}

// H (leading rr x rr of [rp][rp], lower part) -> L in place, Linv = L^-1, Hinv = L^-T L^-1.
static int factor_and_invert(const AdmmWs& ws, hipStream_t s, int prio)
{
    const int rp = ws.rp, rr = ws.rr, q = rr / kNB;
    const bool fused = !opt_flag(OPT_ADMM_NO_FUSED_STEP);
    constexpr size_t potrf_lds = kPotrfLdsBytes;
    constexpr size_t step_lds = std::max(kPotrfLdsBytes, kStepLdsBytes);
    static std::once_flag once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(once, [] { attr_err = hipFuncSetAttribute((const void*)chol_step_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)step_lds); });
    NQ_HIP(attr_err);
    // where the blocks of L below the diagonal end up: a matrix of their own with the one-launch step (Hinv's buffer,
    // free until the last product below), in place of A21 with separate launches
    const double* const Lb = fused ? ws.Hinv : ws.H;
    // the inverse carried along by the step launches, in one of the buffers of the Gram product's parts (ranks that have them)
    const bool carried = fused && ws.G[0] != nullptr;
    hipLaunchKernelGGL(potrf_inv_kernel, dim3(1), dim3(kGemmThreads), potrf_lds, s, ws.H, rp, ws.Linv, rp, 0, ws.status, prio);
    for (int k = 0; k + 1 < q; ++k) {
        const int o = k * kNB;
        const int rem = rr - o - kNB;
        if (fused) {
            const int tiles = rem / kNB;
            StepArgs sa{ws.H, ws.Hinv, ws.Linv, rp, o, prio, ws.status, tiles, carried ? ws.G[0] : nullptr};
            hipLaunchKernelGGL(chol_step_kernel, dim3(tiles, tiles + 1 + (carried ? k + 1 : 0)), dim3(kGemmThreads), step_lds, s, sa);
            continue;
        }
        double* A21 = ws.H + (size_t)(o + kNB) * rp + o;
        // panel: L21 = A21 L11^-T, in place (a workgroup reads all of its rows before it writes them)
        GemmArgs p = gemm_args(0, 1, rem, kNB, kNB, 1.0, A21, rp, ws.Linv + (size_t)o * rp + o, rp, 0.0, nullptr, 0, A21, rp);
        p.tile = 3;                                // whole rows per workgroup: the product is in place
        p.prio = prio;
        int rc = launch_gemm(p, 1, s);
        if (rc != NQ_OK) return rc;
        // trailing update: A22 -= L21 L21^T (lower tiles only)
        double* A22 = ws.H + (size_t)(o + kNB) * rp + o + kNB;
        GemmArgs u = gemm_args(0, 1, rem, rem, kNB, -1.0, A21, rp, A21, rp, 1.0, A22, rp, A22, rp);
        u.lower_only = 1;
        u.prio = prio;
        rc = launch_gemm(u, 1, s);
        if (rc != NQ_OK) return rc;
        hipLaunchKernelGGL(potrf_inv_kernel, dim3(1), dim3(kGemmThreads), potrf_lds, s, ws.H, rp, ws.Linv, rp, o + kNB, ws.status, prio);
    }
    NQ_HIP(hipGetLastError());
    if (carried && q > 1) {
        // the last row of blocks of L^-1
        const int o = rr - kNB;
        GemmArgs x = gemm_args(0, 0, kNB, o, kNB, -1.0, ws.Linv + (size_t)o * rp + o, rp, ws.G[0] + (size_t)o * rp, rp, 0.0, nullptr, 0,
                               ws.Linv + (size_t)o * rp, rp);
        x.prio = prio;
        int rc = launch_gemm(x, 1, s);
        if (rc != NQ_OK) return rc;
    }
    // L^-1 block-recursively: with the halves of a diagonal block inverted (X11, X22), the block below the
    // diagonal of its inverse is  -X22 L21 X11;  all pairs of one level run as one batched launch.
    for (int b = kNB; !carried && b < rr; b *= 2) {
        const int pairs = (rr - b + 2 * b - 1) / (2 * b);       // pairs whose lower half holds real rows
        const long long stride = (long long)2 * b * rp + 2 * b;
        GemmArgs t = gemm_args(0, 0, b, b, b, 1.0, Lb + (size_t)b * rp, rp, ws.Linv, rp, 0.0, nullptr, 0, ws.T + (size_t)b * rp, rp);
        t.sA = t.sB = t.sC = stride;
        t.prio = prio;
        int rc = launch_gemm(t, pairs, s);
        if (rc != NQ_OK) return rc;
        GemmArgs x = gemm_args(0, 0, b, b, b, -1.0, ws.Linv + (size_t)b * rp + b, rp, ws.T + (size_t)b * rp, rp, 0.0, nullptr, 0,
                               ws.Linv + (size_t)b * rp, rp);
        x.sA = x.sB = x.sC = stride;
        x.prio = prio;
        rc = launch_gemm(x, pairs, s);
        if (rc != NQ_OK) return rc;
    }
    GemmArgs h = gemm_args(1, 0, rr, rr, rr, 1.0, ws.Linv, rp, ws.Linv, rp, 0.0, nullptr, 0, ws.Hinv, rp);
    h.k_from_max = 1;
    h.prio = prio;
    return launch_gemm(h, 1, s);
}

// Two more streams and four events, created once.  Two things run beside the factorisation, which is a chain of small
// launches that leaves most of the chip idle: the product with W (it does not depend on the factorisation), and the
// SVID of the factor just updated (nothing needs its result before that factor's NEXT update, a whole factor step later;
// the other factor's update only reads the new factor itself).
struct SideStream {
    hipStream_t stream = nullptr, svid = nullptr;
    hipEvent_t fork = nullptr, join = nullptr, updated = nullptr, svid_done = nullptr;
    hipError_t err = hipSuccess;
};

static SideStream& side_stream()
{
    static SideStream ss;
    static std::once_flag once;
    std::call_once(once, [] {
        ss.err = hipStreamCreateWithFlags(&ss.stream, hipStreamNonBlocking);
        if (ss.err == hipSuccess) ss.err = hipStreamCreateWithFlags(&ss.svid, hipStreamNonBlocking);
        if (ss.err == hipSuccess) ss.err = hipEventCreateWithFlags(&ss.svid_done, hipEventDisableTiming);
        if (ss.err == hipSuccess) ss.err = hipEventCreateWithFlags(&ss.fork, hipEventDisableTiming);
        if (ss.err == hipSuccess) ss.err = hipEventCreateWithFlags(&ss.join, hipEventDisableTiming);
        if (ss.err == hipSuccess) ss.err = hipEventCreateWithFlags(&ss.updated, hipEventDisableTiming);
    });
    return ss;
}

// One factor update of Eq. 5 and Eq. 6 for X [rows][r] given the other factor O [cols][r]:
//   op(W) is [rows][cols] (w_trans = 1: W is stored [cols][rows]).
// An SVID whose launches are still to be issued (to the side stream): the factor step that follows issues them behind its
// own first launch, so that the host does not hold that launch -- the head of the critical path -- back by twenty others.
struct PendingSvid {
    bool valid = false;
    int rows = 0;
    double *Z = nullptr, *Lambda = nullptr, *D = nullptr;
};

static int issue_pending_svid(const AdmmWs& ws, PendingSvid& pend, int r, int power_iters)
{
    if (!pend.valid) return NQ_OK;
    pend.valid = false;
    SideStream& ss = side_stream();
    NQ_HIP(hipStreamWaitEvent(ss.svid, ss.updated, 0));
    const int rc = svid(ws, ws.P, pend.rows, r, power_iters, 0, pend.Z, pend.Lambda, pend.D, ss.svid);
    if (rc != NQ_OK) return rc;
    NQ_HIP(hipEventRecord(ss.svid_done, ss.svid));
    return NQ_OK;
}

static int factor_step(const AdmmWs& ws, const double* W, int w_trans, int ldw, int rows, int cols, int r, const double* O, double rho, double lam,
                       int power_iters, double* X, double* Z, double* Lambda, double* D, hipStream_t s, PendingSvid& pend)
{
    const bool overlap = !opt_flag(OPT_ADMM_NO_OVERLAP);
    // the launches of the caller's stream are the critical path: where another stream shares the chip, their waves
    // ask for the issue slots first
    const int prio = overlap && !opt_flag(OPT_ADMM_NO_PRIO);
    SideStream& ss = side_stream();
    NQ_HIP(ss.err);
    // H = O^T O + (rho + lambda) I   (lower tiles), its factor and inverse
    GemmArgs gh = gemm_args(1, 0, r, r, cols, 1.0, O, r, O, r, 0.0, nullptr, 0, ws.H, ws.rp);
    gh.diag = rho + lam;
    gh.lower_only = 1;
    gh.prio = prio;
    // a long reduction over few tiles: three or six parts of the reduction side by side (into H, two buffers that are
    // free at this point, and three of their own), then added in a fixed order
    // (small ranks: six parts on 128 x 128 tiles -- wider tiles halve what the tiles fetch between them, and the
    // parts make up for their number: 232 -> 190 us for r = 1024, 4096 rows)
    const bool six = ws.G[0] && cols >= 1536 && r >= 256;
    const int parts = cols >= 768 ? (six ? 6 : 3) : 1;
    if (parts > 1) {
        gh.k_parts = parts;
        gh.k_per_part = ((cols + parts - 1) / parts + kBK - 1) / kBK * kBK;
        gh.Cp[0] = ws.H; gh.Cp[1] = ws.T; gh.Cp[2] = ws.Hinv;
        gh.Cp[3] = ws.G[0]; gh.Cp[4] = ws.G[1]; gh.Cp[5] = ws.G[2];
    }
    if (six) gh.tile = 1;
    int rc = launch_gemm(gh, parts, s);
    if (rc != NQ_OK) return rc;
    if (parts > 1) {
        GramParts gp{};
        gp.n = parts;
        for (int q = 0; q < parts; ++q) gp.p[q] = gh.Cp[q];
        hipLaunchKernelGGL(add_parts_kernel, dim3((r + 255) / 256, r), dim3(256), 0, s, ws.H, gp, ws.rp, r);
        NQ_HIP(hipGetLastError());
    }
    // (the product below needs this factor's own SVID, the one before the one that is issued here)
    if (overlap) NQ_HIP(hipStreamWaitEvent(ss.stream, ss.svid_done, 0));
    rc = issue_pending_svid(ws, pend, r, power_iters);        // the other factor's SVID, to its stream
    if (rc != NQ_OK) return rc;
    // RHS = op(W) O + rho (Z - Lambda), on the side stream (behind the SVID that produced Z and Lambda).  It is let go
    // once the Gram matrix is done: both fill the chip, so side by side neither gains, and the product would only keep
    // the Gram matrix -- the head of the critical path -- waiting for workgroup slots; what the product can hide behind
    // is the factorisation that follows.
    hipStream_t rs = overlap ? ss.stream : s;
    if (overlap) {
        NQ_HIP(hipEventRecord(ss.fork, s));
        NQ_HIP(hipStreamWaitEvent(ss.stream, ss.fork, 0));
    }
    GemmArgs gr = gemm_args(w_trans, 0, rows, r, cols, 1.0, W, ldw, O, r, rho, D, r, ws.RHS, r);
    // Beside the factorisation the product has the whole factorisation to finish in, and what
    // matters is that the factorisation's small launches find room at once -- with two workgroups of the product
    // on a CU (2 x 72 KiB of LDS) one of the chain (65 KiB) has to wait until one of them has finished its whole reduction
    // (measured: a panel update of 15 workgroups took 470-570 us instead of 8).  So the product then runs with at
    // most ONE workgroup per CU (its LDS request is padded past half a CU's), of eight waves: 585 us beside the chain, 526 alone, where
    // one of four took 800 and 720.
    const long long t128 = (long long)((rows + 127) / 128) * ((r + 127) / 128);
    if (overlap && opt_or(OPT_ADMM_PRODUCT_MODE, 0) != 1 && t128 >= 64) {
        gr.tile = 1;
        gr.lds_pad = 8704;                         // (2 x 80.5 KiB do not fit; what is left takes a workgroup of the factorisation, 65 KiB)
    }
    rc = launch_gemm(gr, 1, rs);
    if (rc != NQ_OK) return rc;
    if (overlap) NQ_HIP(hipEventRecord(ss.join, ss.stream));
    rc = factor_and_invert(ws, s, prio);
    if (rc != NQ_OK) return rc;
    if (overlap) {
        NQ_HIP(hipStreamWaitEvent(s, ss.join, 0));
        NQ_HIP(hipStreamWaitEvent(s, ss.svid_done, 0));       // P is about to be written
    }
    // X = RHS H^-1,  P = X + Lambda
    GemmArgs gx = gemm_args(0, 0, rows, r, r, 1.0, ws.RHS, r, ws.Hinv, ws.rp, 0.0, nullptr, 0, X, r);
    gx.E = Lambda;
    gx.C2 = ws.P;
    gx.prio = prio;
    rc = launch_gemm(gx, 1, s);
    if (rc != NQ_OK) return rc;
    if (!overlap || opt_flag(OPT_ADMM_INLINE_SVID)) return svid(ws, ws.P, rows, r, power_iters, 0, Z, Lambda, D, s);
    // The SVID goes to a stream of its own, so that the next product does not wait for it (four iterations of 4096 x 4096 r = 1024 10.72 -> 10.27 ms).  What keeps
    // the buffers apart: SVIDs follow one another (they read P; write Z, Lambda, D and the vectors); a factor's product waits for that factor's last SVID, which wrote
    // its D; the caller's stream writes P, reads RHS and Lambda only after it has waited for that product and for the SVID that still reads P.
    // (Its launches are issued by the next factor step, or by the caller after the last one.)
    NQ_HIP(hipEventRecord(ss.updated, s));
    pend.valid = true;
    pend.rows = rows; pend.Z = Z; pend.Lambda = Lambda; pend.D = D;
    return NQ_OK;
}

static int fail(int code, const char* msg)
{
    set_error(msg);
    return code;
}

static bool aligned8(const void* p) { return ((uintptr_t)p & 7u) == 0; }

static int check_shape(int64_t n, int64_t m, int64_t r)
{
    if (n < 1 || m < 1 || r < 1) return fail(NQ_E_SHAPE, "lb_admm: n, m, r must be >= 1");
    if (n > NQ_ADMM_MAX_DIM || m > NQ_ADMM_MAX_DIM || r > NQ_ADMM_MAX_RANK) return fail(NQ_E_SHAPE, "lb_admm: n, m or r beyond the supported size");
    if ((uint64_t)n * (uint64_t)m >= (1ull << 40)) return fail(NQ_E_SHAPE, "lb_admm: n * m too large");
    return NQ_OK;
}

}  // namespace nq

using namespace nq;

extern "C" int nq_lb_admm_workspace_bytes(int64_t n, int64_t m, int64_t r, size_t* bytes)
{
    if (!bytes) return fail(NQ_E_NULL, "lb_admm_workspace_bytes: bytes is NULL");
    const int rc = check_shape(n, m, r);
    if (rc != NQ_OK) return rc;
    *bytes = carve(nullptr, n, m, r).bytes;
    return NQ_OK;
}

extern "C" int nq_lb_admm(const double* W, int64_t n, int64_t m, int64_t r, const double* U0, const double* V0, int n_iters, double rho_start,
                          double rho_end, double lambda, int power_iters, double* U, double* V, double* Z_U, double* Z_V, double* Lambda_U,
                          double* Lambda_V, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!W || !U0 || !V0 || !U || !V || !Z_U || !Z_V || !Lambda_U || !Lambda_V || !workspace) return fail(NQ_E_NULL, "lb_admm: NULL pointer");
    int rc = check_shape(n, m, r);
    if (rc != NQ_OK) return rc;
    const void* ptrs[] = {W, U0, V0, U, V, Z_U, Z_V, Lambda_U, Lambda_V};
    for (const void* p : ptrs)
        if (!aligned8(p)) return fail(NQ_E_ALIGN, "lb_admm: a matrix pointer is not 8-byte aligned");
    if (((uintptr_t)workspace & 255u) != 0) return fail(NQ_E_ALIGN, "lb_admm: workspace is not 256-byte aligned");
    if (n_iters < 0 || power_iters < 0) return fail(NQ_E_INVALID_ARG, "lb_admm: n_iters and power_iters must be >= 0");
    if (!isfinite(rho_start) || !isfinite(rho_end) || !isfinite(lambda)) return fail(NQ_E_INVALID_ARG, "lb_admm: rho and lambda must be finite");
    const AdmmWs ws = carve(workspace, n, m, r);
    if (workspace_bytes < ws.bytes) return fail(NQ_E_INVALID_ARG, "lb_admm: workspace smaller than nq_lb_admm_workspace_bytes");
    hipStream_t s = (hipStream_t)stream;
    const int N = (int)n, M = (int)m, R = (int)r;

    NQ_HIP(hipMemsetAsync(ws.status, 0, 256, s));
    hipLaunchKernelGGL(pad_identity_kernel, dim3(256), dim3(256), 0, s, ws.H, ws.rp, R, 0);
    hipLaunchKernelGGL(pad_identity_kernel, dim3(256), dim3(256), 0, s, ws.Linv, ws.rp, R, 1);
    // (the inverse of L reads whole blocks of the matrix that holds L below its diagonal, in Hinv's buffer, also where they lie past
    // the last real block: times zeros, which the workspace's own bits need not survive)
    if (ws.rp > ws.rr) hipLaunchKernelGGL(pad_identity_kernel, dim3(256), dim3(256), 0, s, ws.Hinv, ws.rp, R, 0);
    NQ_HIP(hipGetLastError());
    if (U != U0) NQ_HIP(hipMemcpyAsync(U, U0, (size_t)n * r * sizeof(double), hipMemcpyDeviceToDevice, s));
    if (V != V0) NQ_HIP(hipMemcpyAsync(V, V0, (size_t)m * r * sizeof(double), hipMemcpyDeviceToDevice, s));
    // initial state: Z = SVID of the start factors, Lambda = 0
    rc = svid(ws, U, N, R, power_iters, 1, Z_U, Lambda_U, ws.DU, s);
    if (rc != NQ_OK) return rc;
    rc = svid(ws, V, M, R, power_iters, 1, Z_V, Lambda_V, ws.DV, s);
    if (rc != NQ_OK) return rc;
    PendingSvid pend;
    for (int k = 0; k < n_iters; ++k) {
        const double rho = n_iters <= 1 ? rho_start : rho_start + (rho_end - rho_start) * (double)k / (double)(n_iters - 1);
        rc = factor_step(ws, W, 0, M, N, M, R, V, rho, lambda, power_iters, U, Z_U, Lambda_U, ws.DU, s, pend);
        if (rc != NQ_OK) return rc;
        rc = factor_step(ws, W, 1, M, M, N, R, U, rho, lambda, power_iters, V, Z_V, Lambda_V, ws.DV, s, pend);
        if (rc != NQ_OK) return rc;
    }
    rc = issue_pending_svid(ws, pend, R, power_iters);
    if (rc != NQ_OK) return rc;
    if (n_iters > 0 && !opt_flag(OPT_ADMM_NO_OVERLAP)) {      // the last SVID may still be running on the side stream
        SideStream& ss = side_stream();
        NQ_HIP(hipStreamWaitEvent(s, ss.svid_done, 0));
    }
    int status = 0;
    NQ_HIP(hipMemcpyAsync(&status, ws.status, sizeof(int), hipMemcpyDeviceToHost, s));
    NQ_HIP(hipStreamSynchronize(s));
    if (status != 0) return fail(NQ_E_INVALID_ARG, "lb_admm: a pivot of the Cholesky factorisation was not positive (rho + lambda <= 0, or NaN in the input)");
    return NQ_OK;
}

extern "C" int nq_lb_admm_balance(const double* U, const double* Lambda_U, int64_t n, const double* V, const double* Lambda_V, int64_t m, int64_t r,
                                  uint32_t* U_words, uint32_t* V_words, double* s1, double* s2, double* eta, void* workspace,
                                  size_t workspace_bytes, void* stream)
{
    if (!U || !Lambda_U || !V || !Lambda_V || !U_words || !V_words || !s1 || !s2 || !eta || !workspace) return fail(NQ_E_NULL, "lb_admm_balance: NULL pointer");
    const int rc = check_shape(n, m, r);
    if (rc != NQ_OK) return rc;
    const void* ptrs[] = {U, Lambda_U, V, Lambda_V, s1, s2, eta};
    for (const void* p : ptrs)
        if (!aligned8(p)) return fail(NQ_E_ALIGN, "lb_admm_balance: a pointer is not 8-byte aligned");
    if (((uintptr_t)U_words & 3u) || ((uintptr_t)V_words & 3u)) return fail(NQ_E_ALIGN, "lb_admm_balance: word pointers must be 4-byte aligned");
    if (((uintptr_t)workspace & 255u) != 0) return fail(NQ_E_ALIGN, "lb_admm_balance: workspace is not 256-byte aligned");
    const AdmmWs ws = carve(workspace, n, m, r);
    if (workspace_bytes < ws.bytes) return fail(NQ_E_INVALID_ARG, "lb_admm_balance: workspace smaller than nq_lb_admm_workspace_bytes");
    hipStream_t s = (hipStream_t)stream;
    hipLaunchKernelGGL(sumsq_kernel, dim3(kSumParts), dim3(256), 0, s, U, Lambda_U, (size_t)n * r, ws.parts_u);
    hipLaunchKernelGGL(sumsq_kernel, dim3(kSumParts), dim3(256), 0, s, V, Lambda_V, (size_t)m * r, ws.parts_v);
    hipLaunchKernelGGL(balance_rows_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, U, Lambda_U, (int)n, (int)r, (const double*)ws.parts_u,
                       (const double*)ws.parts_v, 0, U_words, s1, eta);
    hipLaunchKernelGGL(balance_rows_kernel, dim3((unsigned)((m + 3) / 4)), dim3(256), 0, s, V, Lambda_V, (int)m, (int)r, (const double*)ws.parts_u,
                       (const double*)ws.parts_v, 1, V_words, s2, (double*)nullptr);
    NQ_HIP(hipGetLastError());
    return NQ_OK;
}

extern "C" int nq_dgemm(int trans_a, int trans_b, int64_t M, int64_t N, int64_t K, double alpha, const double* A, int64_t lda, const double* B,
                        int64_t ldb, double beta, double* C, int64_t ldc, void* stream)
{
    if (!A || !B || !C) return fail(NQ_E_NULL, "dgemm: NULL pointer");
    if (M < 1 || N < 1 || K < 1 || M > NQ_ADMM_MAX_DIM || N > NQ_ADMM_MAX_DIM || K > NQ_ADMM_MAX_DIM) return fail(NQ_E_SHAPE, "dgemm: M, N, K must be in [1, 65536]");
    if ((trans_a | trans_b) & ~1) return fail(NQ_E_INVALID_ARG, "dgemm: trans flags are 0 or 1");
    if (lda < (trans_a ? M : K) || ldb < (trans_b ? K : N) || ldc < N || lda > INT32_MAX || ldb > INT32_MAX || ldc > INT32_MAX)
        return fail(NQ_E_SHAPE, "dgemm: a leading dimension is smaller than its row length");
    if (!aligned8(A) || !aligned8(B) || !aligned8(C)) return fail(NQ_E_ALIGN, "dgemm: a pointer is not 8-byte aligned");
    GemmArgs g = gemm_args(trans_a, trans_b, (int)M, (int)N, (int)K, alpha, A, (int)lda, B, (int)ldb, beta, C, (int)ldc, C, (int)ldc);
    return launch_gemm(g, 1, (hipStream_t)stream);
}
