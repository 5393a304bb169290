// Dependent layers in ONE launch: a decoder block (or a stack of them) run level by level
// (q, k, v | o | gate, up | down -- the seven projections of Appendix D.3's figure, in the order the
// decode harness of Appendix D.1 calls them) by a persistent grid, batch 1.
//
// A layer forward is two sign-matrix x vector products (Section 3.1 Eq. 1; Appendix E.2), so a
// stack of L levels is 2 L phases, each depending on ALL outputs of the one before.  Run as
// launches, a phase costs a launch-to-launch latency (about 7 us measured) for well under 1 us of
// streaming.  Here one workgroup of 8 waves sits on every CU and walks its own list of tasks; a
// task is a run of 128-row blocks of one phase's sign matrix.  Nothing is ever waited for except data:
//
//  - every value that crosses from one phase to the next (t of stage 1; y where a later layer of
//    the same call reads it) is one 32-bit word, stored with ONE device-scope store and read with device-scope
//    loads.  The word is the fp32 value; the bits of one NaN that no value has (results that are NaN are stored with other bits) mean
//    "not there yet", and a consumer that meets them reads again: no flag, no counter, no fence, no ordering between
//    stores.  There are two copies of every such array, for launches of even and odd number: who stores a value in this launch's
//    copy clears it in the other, which nobody reads before the next launch.  The number lives in device memory and is
//    advanced by the last workgroup to leave, so a replay of a captured launch takes the copies in turn too.
//
// What bounds it: 256 dependent phases of 4.25 us per token of a 7B-shaped stack.  Of those the hand-over, from the last store to the last workgroup that has its
// input, is 1.3 to 2.7 us (a store, half a polling period and a read past the L2; 3.3 where 86 workgroups store, 4.8 where 104 read 11008 values, 6 for 28672), the
// fixed point 0.4 to 0.7 (0.8, 1.6), the products 0.7 to 1.9 (a long reduction or many rows: 2.9 to 5.5), adding them up and storing 0.3 to 0.45.  As pairs of value and
// launch number, read 16 elements per lane (a line per 16-byte request), hand-overs took 2.4 to 5 us (17 of 28672 values); whole row blocks per workgroup,
// loops over the longest input's groups without an exit and addresses spilled from phase to phase cost another 1.5 us: 1818 -> 1089 us per token.
//  - every wait is bounded by a wall-clock limit; a workgroup that gives up sets an error word
//    and leaves, the others see the word (or run into their own limit) and leave too: the grid
//    always drains.  (They clear the other copies of what their tasks would have stored first.)
//  - a workgroup requests the first sign tiles of its next task BEFORE it waits for that task's
//    input, so the weights stream while the dependency chain is being walked.
//
// The arithmetic is that of the streaming kernels element for element (same fixed-point split, same
// exact integer sums, same single roundings), so results are bit-identical to a sequence of
// nq_binlr_forward calls.
#include <algorithm>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "nq_internal.h"
#include "nq_device.h"

namespace nq {

constexpr int kExecWaves = 8;                      // two per SIMD
constexpr int kExecThreads = 64 * kExecWaves;
constexpr int kExecRing = 8;                       // sign tiles a wave keeps in flight
constexpr int kExecMaxSteps = 512;                 // longest reduction: 32768 elements (96 KiB of LDS as fixed point)
constexpr int kExecEpiInts = 3 * kTileRows + 16;   // per wave: the three slice columns x 128 rows, 16 banks on from wave to wave
constexpr int kExecWordBytes = 64;                 // the words of the reductions over a workgroup
constexpr int kExecHeld = 16;                      // groups of four elements of the input that a thread keeps in registers

// One task of one workgroup: a run of row blocks of one stage of one layer, with everything the
// kernel needs to know about that stage in the record itself -- a workgroup's records are
// consecutive in memory, so the next one is a neighbouring cache line, requested a task ahead.
// W = 1 << wl waves share a row block, 8 / W row blocks are worked on side by side.
struct ExecTask {
    const uint32_t* tiles;          // sign tiles of A (V^T or U)
    const void* in;                 // the input vector: plain elements of in_dtype (in_ll 0), words handed over (1), or none: the LDS array (2)
    const uint16_t* in_scale;       // fp16 [N] or nullptr
    const uint16_t* out_scale;      // fp16 [M rounded up to whole row blocks] or nullptr
    void* out;                      // plain output [M] of out_dtype, or nullptr
    unsigned int* out_ll;           // words [M] for the stages that read this output in the same launch (the copy of even launches), or nullptr
    int M, N, n_steps, in_dtype, out_dtype, in_ll;
    int rb0, n_rb, wl;
    int out_lds;                    // the (fp32) output also goes to the workgroup's LDS array, for its next task (in_ll == 2)
    int p0, pl;                     // pl > 0: bit planes p0 .. p0 + pl - 1 (16 rows each) of the one row block, all eight waves on it
};
static_assert(sizeof(ExecTask) == 96, "task record");
static_assert(kExecMaxSteps * 16 <= kExecHeld * kExecThreads, "a thread holds all of its groups");

struct ExecState {                  // device words shared by the launches of one executor
    unsigned int epoch;             // number of the NEXT launch
    unsigned int done;              // workgroups of the running launch that have left
    int error;                      // sticky: a wait ran into its limit
    int pad;
};

typedef __attribute__((address_space(1))) unsigned int* gptr_u32;

constexpr unsigned int kNotThere = 0xffffffffu;    // a NaN of these bits is never stored as a value

__device__ __forceinline__ void ll_store(unsigned int* p, unsigned int bits)
{
    // (global, not generic, address space: a flat store would count on both wait counters)
    __hip_atomic_store((gptr_u32)p, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned int ll_bits(float v) { return v == v ? __builtin_bit_cast(unsigned int, v) : 0x7fc00000u; }

// ---------------------------------------------------------------------------------------------
// LDS: [bq_bytes] the task's input as fixed point (layout of the global buffers of the streaming
// kernels) | [8][3][128] raw sums of the waves | sum of q, largest magnitude, flags
// ---------------------------------------------------------------------------------------------
// tasks[ti .. t_end) of this workgroup; SMALL: a lone workgroup whose tasks hand over through LDS only (state == nullptr)
template <bool SMALL>
__device__ __forceinline__ void exec_body(const ExecTask* __restrict__ tasks, int ti, const int t_end,
                                          ExecState* __restrict__ state, int bq_bytes, size_t copy_words, unsigned long long spin_ticks)
{
    extern __shared__ __align__(16) int lds[];
    constexpr int D = kExecRing;
    char* const lds_bq = (char*)lds;
    int* const lds_epi = (int*)(lds_bq + bq_bytes);
    // reductions over the workgroup go through LDS atomics (one instruction per wave each, no shuffle
    // chains): the sum of the quantised values, the largest magnitude (as the bits of a non-negative
    // float), "a value is not finite", "a wait gave up"
    // (two sets, of consecutive tasks: a task clears the other's while everybody is between its two barriers)
    struct Words {
        unsigned long long sum;
        unsigned int max;
    };
    Words* const words = (Words*)(lds_epi + kExecWaves * kExecEpiInts);
    int* const lds_abort = (int*)(words + 2);
    float* const lds_t = (float*)((char*)words + kExecWordBytes);     // an output kept in LDS for the next task of this workgroup

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 4, n = lane & 15;
    const unsigned int epoch = state ? state->epoch : 0u;   // written by the previous launch (or the host)
    const size_t now = epoch & 1u ? copy_words : 0, other = copy_words - now;      // this launch's copies and the others, from the even ones
    if (tid == 0) {
        *lds_abort = 0;
        words[0] = words[1] = Words{0, 0};
    }
    __syncthreads();

    v4u wbuf[D];
    // the wave's tile stream of one (task, group of row blocks)
    const char* a_base = nullptr;
    uint32_t a_off = 0;
    int cnt = 0, part = 0, w_of = 1;
    // requests the first D tiles of group `grp` of task `t` (branch-free: a short share re-reads its last tile)
#define NQ_PRIME(t, grp)                                                                           \
    do {                                                                                           \
        const int nst_ = (t).n_steps;                                                      \
        const int wl_ = (t).wl;                                                                    \
        const int sub_ = wave >> wl_;                                                              \
        part = wave - (sub_ << wl_);                                                               \
        w_of = 1 << wl_;                                                                           \
        const int rb_ = (t).rb0 + (grp) * (kExecWaves >> wl_) + sub_;                              \
        const bool act_ = rb_ < (t).rb0 + (t).n_rb;                                                \
        cnt = act_ ? (nst_ - part + w_of - 1) >> wl_ : 0;                                          \
        cnt = cnt < 0 ? 0 : cnt;                                                                   \
        a_base = (const char*)(t).tiles +                                                  \
                 (size_t)(act_ ? rb_ : (t).rb0) * nst_ * (kTileWords * 4);                         \
        a_off = (uint32_t)((cnt > 0 ? part : 0) * 1024 + lane * 16);                               \
        /* (ordinary loads: the workgroups that share a row block share its tiles in their L2) */  \
        _Pragma("unroll") for (int k = 0; k < D; ++k) {                                            \
            const int kk = k < cnt ? k : (cnt > 0 ? cnt - 1 : 0);                                  \
            wbuf[k] = load_global_v4u(a_base, a_off + (uint32_t)kk * (uint32_t)(w_of * 1024));     \
        }                                                                                          \
        a_off += (uint32_t)(D * w_of * 1024);                                                      \
    } while (0)

    // With the first tiles of a task go the scales it will need (static data, usually cold in the caches:
    // a round trip to memory each): the input scales of the groups this thread owns, where the input is
    // handed over by another stage, and the output scales of the rows this
    // thread finishes in the task's first group.  All of them are requested before the task's input is
    // waited for and converted only when they are used.  Read through a buffer that ends with the input:
    // a group past it, which is zero, gets the scale zero and not what an earlier task left there, which may be infinite.  (7B-shaped chain 1089 us;
    // 1125 to 1129 with a condition per group, here or where they are scaled; 1110 without either.)
    typedef unsigned int v2u __attribute__((ext_vector_type(2)));
    typedef const __attribute__((address_space(1))) v2u* gptr_v2u;
    constexpr int kScaled = 8;                              // groups whose scales come ahead: inputs of up to 16384 elements
    v2u sraw[kScaled];
#pragma unroll
    for (int k = 0; k < kScaled; ++k) sraw[k] = v2u{0, 0};
    uint16_t ps[2] = {0, 0};
#define NQ_PREFETCH_SCALES(t)                                                                      \
    do {                                                                                           \
        const uint16_t* const is_ = (t).in_scale;                                                  \
        const int n_ = (t).N;                                                                      \
        if (is_ && (t).in_ll == 1) {                                                               \
            const __amdgpu_buffer_rsrc_t r_ = __builtin_amdgcn_make_buffer_rsrc((void*)is_, 0, n_ * 2, 0x00020000); \
            _Pragma("unroll") for (int k_ = 0; k_ < kScaled; ++k_) {                               \
                if (k_ * kExecThreads + 64 * wave >= 16 * (t).n_steps) break;                      \
                sraw[k_] = __builtin_amdgcn_raw_buffer_load_b64(r_, (k_ * kExecThreads + tid) * 8, 0, 0); \
            }                                                                                      \
        }                                                                                          \
        const uint16_t* const os_ = (t).out_scale;                                         \
        const int per_ = kExecWaves >> (t).wl;                                                     \
        if ((t).pl > 0) {                                                                          \
            if (os_ && (tid >> 2) < 16 * (t).pl)                                                   \
                ps[0] = ((gptr_u16)os_)[(t).rb0 * kTileRows + 16 * (t).p0 + (tid >> 2)];           \
        } else _Pragma("unroll") for (int u = 0; u < 2; ++u) {                                     \
            const int idx_ = tid + u * kExecThreads;                                               \
            const int rb_ = (t).rb0 + (idx_ >> 7);                                                 \
            if (os_ && idx_ < per_ * kTileRows && rb_ < (t).rb0 + (t).n_rb)                        \
                ps[u] = ((gptr_u16)os_)[rb_ * kTileRows + (idx_ & 127)];                           \
        }                                                                                          \
    } while (0)

    ExecTask tk{};
    if (ti < t_end) {
        tk = tasks[ti];
        NQ_PRIME(tk, 0);
        NQ_PREFETCH_SCALES(tk);
    }

    while (ti < t_end) {
        const ExecTask& op = tk;                            // (wave-uniform: the record came through scalar loads)
        // the next record is requested now, a whole task before its fields are needed
        ExecTask nxt = tk;
        const bool more = ti + 1 < t_end;
        if (more) nxt = tasks[ti + 1];
        const int nst = op.n_steps;
        const int n_groups = 16 * nst;                      // groups of four elements: thread t owns t, t + 512, ... (whole lines per load)
        Words* const wd = words + (ti & 1);

        // ---- the task's input: load (waiting for it where another stage writes it), scale, quantise ----
        // (whole 16-byte loads; the arrays are padded)
        const unsigned int* const in_words = (const unsigned int*)op.in + (op.in_ll == 1 ? now : 0);
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)in_words, 0, op.in_ll == 1 ? ((op.N + 3) & ~3) * 4 : 0, 0x00020000);
        const unsigned long long t0 = __builtin_amdgcn_s_memrealtime();
        int gave_up = 0;
        v4u hv[kExecHeld];                                  // (as bits until they are scaled)
        // (whole steps of four: whether a wave has a k-th group is the same for all of its lanes)
        const int wave0 = 64 * wave;
        int t = tid;
        asm volatile("" : "+v"(t));                         // (addresses are formed here, not kept from task to task, which spills them)
        if (!SMALL && op.in_ll == 1) {
            // Read until everything is there (or the time is up: gave_up).  First the wave polls the last word of its first groups only (one
            // transaction per round, all lanes the same address), so that workgroups waiting far ahead of the running phase leave the
            // memory system alone; then it asks for the groups that are not complete yet, all of them before any is looked at.  (7B-shaped chain: 1110 us;
            // polling the first word 1121, four times as rarely 1143, without polling where a thread has one group 1168.)
            // (Device-scope loads; beyond the array the buffer returns zeros.)
            const int last = wave0 * 4 + 255 < op.N ? wave0 * 4 + 255 : op.N - 1;
            const int mine = wave0 < n_groups ? (n_groups - wave0 + kExecThreads - 1) / kExecThreads : 0;
            unsigned int todo = (1u << mine) - 1u;
            unsigned int spins = 0;
            bool waiting = wave0 * 4 < op.N;
            while (todo) {
                asm volatile("" ::: "memory");              // another workgroup writes this memory: load again every time
                if (waiting) {
                    waiting = __builtin_amdgcn_raw_buffer_load_b32(rsrc, last * 4, 0, 16) == kNotThere;
                    if (waiting) {
                        ++spins;
                        // (the clock and the error word are looked at every 16th round, and on the first: a limit of zero gives up at once)
                        if ((spins & 15u) == 1u && (__builtin_amdgcn_s_memrealtime() - t0 > spin_ticks ||
                                                    __hip_atomic_load(&state->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
                            gave_up = 1;
                            break;
                        }
                        __builtin_amdgcn_s_sleep(2);
                        continue;
                    }
                }
#pragma unroll
                for (int k = 0; k < kExecHeld; ++k)
                {
                    if (k * kExecThreads + wave0 >= n_groups) break;
                    if (todo & (1u << k)) hv[k] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (k * kExecThreads + t) * 16, 0, 16);
                }
#pragma unroll
                for (int k = 0; k < kExecHeld; ++k) {
                    if (k * kExecThreads + wave0 >= n_groups) break;
                    if (todo & (1u << k)) {
                        const int j = (k * kExecThreads + t) * 4;
                        bool missing = false;
#pragma unroll
                        for (int i = 0; i < 4; ++i) missing |= hv[k][i] == kNotThere && j + i < op.N;
                        if (__builtin_amdgcn_ballot_w64(missing) == 0) todo &= ~(1u << k);
                    }
                }
                if (todo && (__builtin_amdgcn_s_memrealtime() - t0 > spin_ticks ||
                             ((++spins & 15u) == 0 && __hip_atomic_load(&state->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0))) {
                    gave_up = 1;
                    break;
                }
                // (inputs of one group per thread, which most workgroups of the grid wait for: a pause; 1264 us without, 1119 with one for all)
                if (todo && op.N <= 4 * kExecThreads) __builtin_amdgcn_s_sleep(2);
            }
        } else {
            if (SMALL && op.in_ll == 2) __syncthreads();    // the LDS array of this workgroup's previous task is complete
#pragma unroll
            for (int k = 0; k < kExecHeld; ++k) {
                if (k * kExecThreads + wave0 >= n_groups) break;
                const int j = (k * kExecThreads + t) * 4;
                {
                    hv[k] = v4u{0, 0, 0, 0};
                    if (SMALL && op.in_ll == 2) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) hv[k][i] = j + i < op.N ? __builtin_bit_cast(unsigned int, lds_t[j + i]) : 0u;
                    } else if (j + 4 <= op.N) {             // (x is 16-byte aligned)
                        if (op.in_dtype == NQ_F32) {
                            hv[k] = *(gptr_v4u)((const float*)op.in + j);
                        } else {
                            const v2u h = *(gptr_v2u)((const uint16_t*)op.in + j);
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                const uint16_t b = (uint16_t)(h[i / 2] >> (16 * (i & 1)));
                                hv[k][i] = __builtin_bit_cast(unsigned int, op.in_dtype == NQ_F16 ? half_bits_to_float(b) : bf16_bits_to_float(b));
                            }
                        }
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (j + i < op.N) hv[k][i] = __builtin_bit_cast(unsigned int, load_as_float(op.in, op.in_dtype, j + i));
                    }
                    if (k < kScaled && op.in_scale) {
                        sraw[k % kScaled] = v2u{0, 0};
                        if (j + 4 <= op.N) sraw[k % kScaled] = *(gptr_v2u)(op.in_scale + j);
                    }
                }
            }
        }
        if (op.N & 3) {                                     // the one group that the input ends inside of
#pragma unroll
            for (int k = 0; k < kExecHeld; ++k) {
                const int j = (k * kExecThreads + t) * 4;
                if (j < op.N && j + 4 > op.N) {
                    uint16_t h[4] = {0, 0, 0, 0};
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (j + i >= op.N) hv[k][i] = 0;
                        else if (op.in_scale) h[i] = ((gptr_u16)op.in_scale)[j + i];
                    }
                    if (k < kScaled) sraw[k % kScaled] = v2u{(unsigned int)h[0] | (unsigned int)h[1] << 16, (unsigned int)h[2] | (unsigned int)h[3] << 16};
                    else if (op.in_scale)
#pragma unroll
                        for (int i = 0; i < 4; ++i) hv[k][i] = __builtin_bit_cast(unsigned int, times_half(__builtin_bit_cast(float, (unsigned int)hv[k][i]), h[i]));
                }
            }
        }
        unsigned int m = 0;                                 // (as bits: magnitudes order like them, NaN above all)
#pragma unroll
        for (int k = 0; k < kExecHeld; ++k) {
            if (k * kExecThreads + wave0 >= n_groups) break;
            {
                if (op.in_scale) {
                    // times the input scale, as the quantiser of the streaming path does: one fp32 product
                    const int j = (k * kExecThreads + t) * 4;
                    v2u sc = sraw[k % kScaled];
                    if (k < kScaled || j + 4 <= op.N) {
                        if (k >= kScaled) sc = *(gptr_v2u)(op.in_scale + j);
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            hv[k][i] = __builtin_bit_cast(unsigned int, times_half(__builtin_bit_cast(float, (unsigned int)hv[k][i]), (uint16_t)(sc[i / 2] >> (16 * (i & 1)))));
                    }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const unsigned int a = hv[k][i] & 0x7fffffffu;
                    m = a > m ? a : m;
                }
            }
        }
        // (a wave none of whose lanes owns a group goes straight to the barrier)
        const bool wave_works = wave0 < n_groups;
        if (wave_works) {
            m = wave_reduce32(m, [](unsigned int a, unsigned int b) { return a > b ? a : b; });
            if (lane == 0) atomicMax(&wd->max, m);          // one LDS atomic per wave
            if (gave_up) *lds_abort = 1;
        }
        __syncthreads();
        if (*lds_abort) break;                              // the whole workgroup leaves (same LDS word for all)
        m = wd->max;
        if (tid == 0) words[(ti + 1) & 1] = Words{0, 0};
        const float step = exp2_int(step_exponent(m));
        if (wave_works) {
            const float inv_step = exp2_int(-step_exponent(m));
            int sum = 0;                                    // |q| <= 2^22: 64 of them fit
            uint32_t* const first = (uint32_t*)lds_bq + 4 * bq_piece(t >> 2, 0) + (t & 3);
#pragma unroll
            for (int k = 0; k < kExecHeld; ++k) {
                if (k * kExecThreads + wave0 >= n_groups) break;
                {
                    uint32_t hi, mid, lo;
                    const v4f v = __builtin_bit_cast(v4f, hv[k]);
                    sum += quantize4(v[0], v[1], v[2], v[3], inv_step, hi, mid, lo);
                    uint32_t* const dst = first + k * (kExecThreads / 16) * (int)(kBqStepBytes / 4);
                    dst[0] = hi;
                    dst[16] = mid;
                    dst[32] = lo;
                }
            }
            const long long total = wave_sum64(sum);
            if (lane == 0) atomicAdd(&wd->sum, (unsigned long long)total);     // |sum| < 2^39: exact, whatever the order
        }
        __syncthreads();
        const double tot = (double)(long long)wd->sum;
        const double two_step = m <= kMostBits ? 2.0 * (double)step : (double)__builtin_nanf("");
        const double neg_qs = -tot * (double)step;

        // ---- the task's row blocks, 8 / W at a time ----
        const int per = kExecWaves >> tk.wl;
        const int n_grp = (tk.n_rb + per - 1) / per;
        const uint32_t b_lane = (uint32_t)(bq_piece(g, n < 3 ? n : 0) * 16);     // unused columns re-read slice 0
        // the value and its hand-over: rounded, then scaled in fp32, as the streaming kernels do
        auto finish = [&](int grow, double val, uint16_t scale) {
            float f = (float)val;
            if (op.out_scale) f *= half_bits_to_float(scale);
            if (op.out_ll) {
                // what a reader of the stored output would see: the value after its rounding to the output type
                float h = f;
                if (op.out_dtype == NQ_BF16) h = bf16_bits_to_float(float_to_bf16_bits(f));
                else if (op.out_dtype == NQ_F16) h = half_bits_to_float(float_to_f16_bits(f));
                ll_store(op.out_ll + now + grow, ll_bits(h));
                op.out_ll[other + grow] = kNotThere;
            }
            if (op.out) store_out(op.out, op.out_dtype, (size_t)grow, f, op.out_scale != nullptr);
            if (op.out_lds) lds_t[grow] = f;
        };
        // PL bit planes of one row block, all waves on it
        v4i acc[1][8];
        auto run_planes = [&](auto planes) {
            constexpr int PL = decltype(planes)::value;
            uint32_t mask[PL];
#pragma unroll
            for (int p = 0; p < PL; ++p) mask[p] = 0x01010101u << (tk.p0 + p);
#pragma unroll
            for (int p = 0; p < PL; ++p) acc[0][p] = v4i{0, 0, 0, 0};
            const char* const b_base = lds_bq + b_lane + wave * (int)kBqStepBytes;
            auto mac = [&](int k, int i) {
                const v4u b = *(const v4u*)(b_base + i * (kExecWaves * (int)kBqStepBytes));
#pragma unroll
                for (int p = 0; p < PL; ++p)
                    acc[0][p] = __builtin_amdgcn_mfma_i32_16x16x64_i8((v4i)(wbuf[k] & mask[p]), (v4i)b, acc[0][p], 0, 0, 0);
            };
            auto issue = [&](int k) {
                wbuf[k] = load_global_v4u(a_base, a_off);
                a_off += (uint32_t)(kExecWaves * 1024);
            };
            // whole passes over the ring without a branch, so that the waits inside stay partial (few planes: long reductions); then what is left
            int i0 = 0;
            if (PL <= 2) {
                for (; i0 + 2 * D <= cnt; i0 += D) {
#pragma unroll
                    for (int k = 0; k < D; ++k) {
                        mac(k, i0 + k);
                        issue(k);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
            for (; i0 < cnt; i0 += D) {
#pragma unroll
                for (int k = 0; k < D; ++k) {
                    if (i0 + k < cnt) {
                        mac(k, i0 + k);
                        if (i0 + k + D < cnt) issue(k);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
#pragma unroll
            for (int p = 0; p < PL; ++p)
                if (n < 3) *((v4i*)(lds_epi + wave * kExecEpiInts + n * kTileRows) + g + 4 * p) = acc[0][p];
        };
        if (tk.pl > 0) {
            if (tk.pl == 1) run_planes(std::integral_constant<int, 1>{});
            else if (tk.pl == 2) run_planes(std::integral_constant<int, 2>{});
            else if (tk.pl == 4) run_planes(std::integral_constant<int, 4>{});
            else run_planes(std::integral_constant<int, 8>{});
            __syncthreads();
            // a quad of lanes per row, two waves' sums each
            const int row = tid >> 2, grow = tk.rb0 * kTileRows + 16 * tk.p0 + row;
            if (row < 16 * tk.pl) {
                const int* q = lds_epi + (tid & 3) * kExecEpiInts + row;
                int s[3];
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    s[i] = q[i * kTileRows] + q[4 * kExecEpiInts + i * kTileRows];
                    s[i] += __builtin_amdgcn_mov_dpp(s[i], 0xB1, 0xf, 0xf, true);          // quad_perm [1, 0, 3, 2]
                    s[i] += __builtin_amdgcn_mov_dpp(s[i], 0x4E, 0xf, 0xf, true);          // quad_perm [2, 3, 0, 1]
                }
                if ((tid & 3) == 0 && grow < op.M) {
                    const int p = tk.p0 + (row >> 4);
                    double raw = fma((double)s[0], 65536.0, fma((double)s[1], 256.0, (double)s[2]));
                    if (p == 7) raw = -raw;                 // bit 7 of an int8 is worth -128
                    finish(grow, fma(raw, __builtin_ldexp(two_step, -p), neg_qs), ps[0]);         // exact
                }
            }
        } else for (int grp = 0; grp < n_grp; ++grp) {
            // (the output scales of the first group came with the task's first tiles; a later group requests its own now)
            if (grp > 0) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int idx = tid + u * kExecThreads;
                    const int rb = tk.rb0 + grp * per + (idx >> 7);
                    if (op.out_scale && idx < per * kTileRows && rb < tk.rb0 + tk.n_rb)
                        ps[u] = ((gptr_u16)op.out_scale)[rb * kTileRows + (idx & 127)];
                }
            }
            const uint16_t ps_now[2] = {ps[0], ps[1]};
#pragma unroll
            for (int p = 0; p < 8; ++p) acc[0][p] = v4i{0, 0, 0, 0};
            const int last = cnt > 0 ? cnt - 1 : 0;
            const int w_steps = w_of;
#define NQ_ISSUE(k)                                                              \
    do {                                                                         \
        wbuf[k] = load_tile_words(a_base, a_off);                                \
        a_off += (uint32_t)(w_steps * 1024);                                     \
    } while (0)
#define NQ_LDSB(i) (*(const v4u*)(lds_bq + b_lane + (part + ((i) < last ? (i) : last) * w_steps) * (int)kBqStepBytes))
            v4u bop[2][1];
            bop[0][0] = NQ_LDSB(0);
            for (int i0 = 0; i0 < cnt; i0 += D) {
#pragma unroll
                for (int k = 0; k < D; ++k) {
                    if (i0 + k < cnt) {
                        bop[(k + 1) & 1][0] = NQ_LDSB(i0 + k + 1);
                        mac_tile<1>(acc, wbuf[k], bop[k & 1]);
                        if (i0 + k + D < cnt) NQ_ISSUE(k);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
#undef NQ_LDSB
#undef NQ_ISSUE
            // the ring is empty: the next group's first tiles go out before the epilogue
            const int w_cur = 1 << tk.wl;
            if (grp + 1 < n_grp) NQ_PRIME(tk, grp + 1);

            // ---- epilogue: raw sums -> LDS, added over the W waves of a row block, scaled, stored ----
            if (grp > 0) __syncthreads();                   // (the regions of the group before; those of a task before are free since its successor's barriers)
            if (n < 3) {
                v4i* dst = (v4i*)(lds_epi + wave * kExecEpiInts + n * kTileRows) + g;
#pragma unroll
                for (int p = 0; p < 8; ++p) dst[4 * p] = p == 7 ? -acc[0][p] : acc[0][p];    // rows 16p + 4g .. +3; plane 7 holds -128 * sum
            }
            __syncthreads();
#pragma unroll 1
            for (int u = 0; u < 2; ++u) {
                const int idx = tid + u * kExecThreads;
                if (idx >= per * kTileRows) break;          // (whole waves: per * 128 is a multiple of 64)
                const int sub = idx >> 7, row = idx & 127;
                const int rb = tk.rb0 + grp * per + sub;
                const int grow = rb * kTileRows + row;
                if (idx < per * kTileRows && rb < tk.rb0 + tk.n_rb && grow < op.M) {
                    int h = 0, mm = 0, l = 0;
                    const int* q = lds_epi + sub * w_cur * kExecEpiInts + row;
                    // (the waves' sums requested together; a wave beyond the row block's W reads wave 0's region again and is not added)
#pragma unroll 1
                    for (int w0 = 0; w0 < w_cur; w0 += kExecWaves) {
#pragma unroll
                        for (int w = 0; w < kExecWaves; ++w) {
                            const int* qw = q + (w0 + w < w_cur ? w0 + w : 0) * kExecEpiInts;
                            const int a0 = qw[0], a1 = qw[kTileRows], a2 = qw[2 * kTileRows];
                            h += w0 + w < w_cur ? a0 : 0;
                            mm += w0 + w < w_cur ? a1 : 0;
                            l += w0 + w < w_cur ? a2 : 0;
                        }
                    }
                    const double raw = fma((double)h, 65536.0, fma((double)mm, 256.0, (double)l));
                    const double val = fma(raw, __builtin_ldexp(two_step, -(row >> 4)), neg_qs);    // exact
                    finish(grow, val, u ? ps_now[1] : ps_now[0]);
                }
            }
        }
        // The next task's first tiles and scales go out now, behind this task's stores and ahead of the wait
        // for that task's input.  (Not earlier: vector memory returns in order, so anything this task still
        // had to wait for -- a scale, a spilled register -- would have waited for those tiles as well.)
        if (more) {
            NQ_PRIME(nxt, 0);
            NQ_PREFETCH_SCALES(nxt);
        }
        ++ti;
        tk = nxt;
    }
#undef NQ_PRIME
#undef NQ_PREFETCH_SCALES

    // ---- leave: report a missed deadline; the last workgroup out advances the number ----
    // (A workgroup that gave up clears what the tasks it did not finish would have cleared: the next launch reads those copies.)
    for (; ti < t_end; ++ti) {
        const ExecTask t = tasks[ti];
        const int row0 = t.rb0 * kTileRows + 16 * t.p0, rows = t.pl > 0 ? 16 * t.pl : t.n_rb * kTileRows;
        for (int k = tid; k < rows; k += kExecThreads)
            if (t.out_ll && row0 + k < t.M) t.out_ll[other + row0 + k] = kNotThere;
    }
    __syncthreads();
    if (tid == 0 && state) {
        if (*lds_abort) __hip_atomic_store(&state->error, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned int left = __hip_atomic_fetch_add(&state->done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (left + 1 == gridDim.x) {
            __hip_atomic_store(&state->done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(&state->epoch, epoch + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

__global__ void __launch_bounds__(kExecThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
exec_kernel(const ExecTask* __restrict__ tasks, const int* __restrict__ task_begin,
            ExecState* __restrict__ state, int bq_bytes, size_t copy_words, unsigned long long spin_ticks)
{
    exec_body<false>(tasks, task_begin[blockIdx.x], task_begin[blockIdx.x + 1], state, bq_bytes, copy_words, spin_ticks);
}

// One small layer, both stages, by ONE workgroup in one launch: t stays in LDS between the stages
// (the two-stage GEMV of Appendix E.2 with its intermediate in shared memory).  The two task records are
// kernel arguments.
struct ExecPair {
    ExecTask t[2];
};
__global__ void __launch_bounds__(kExecThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
exec_small_kernel(ExecPair pair, int bq_bytes)
{
    exec_body<true>(pair.t, 0, 2, nullptr, bq_bytes, 0, 0ull);
}

// ---------------------------------------------------------------------------------------------
// host: the task lists
// ---------------------------------------------------------------------------------------------
struct PlannedTask {
    int wg, phase, layer, stage, rb0, n_rb, W, p0, pl;
};

// Levels are run as 2 phases each (stage 1 of every layer of the level, then stage 2).  Inside a
// phase the row blocks are dealt to the workgroups in runs of 8 / W with the largest W (waves per row
// block) for which every run finds a workgroup of its own; consecutive phases start where the one
// before stopped, so a workgroup's next task usually lies several phases ahead and its first tiles
// are in registers long before its input exists.  Every workgroup's list is in phase order, which
// is what makes the grid deadlock-free: the earliest unfinished phase depends on finished ones only.
static void plan_tasks(const int64_t* d_out, const int64_t* d_in, const int64_t* r, const int* level_of, int n,
                       int n_wg, std::vector<PlannedTask>& out)
{
    out.clear();
    int start = 0, slot[8] = {};
    for (int i0 = 0; i0 < n;) {
        int i1 = i0;
        while (i1 < n && level_of[i1] == level_of[i0]) ++i1;
        for (int stage = 0; stage < 2; ++stage) {
            const int phase = 2 * level_of[i0] + stage;
            std::vector<int> nrb(i1 - i0);
            for (int i = i0; i < i1; ++i) nrb[i - i0] = (int)n_rowblocks(stage == 0 ? r[i] : d_out[i]);
            // Where every row block finds a workgroup of its own, all of its waves take it; where the row blocks are few, each is dealt out by bit
            // planes to 8 / pl workgroups, which stream the same tiles and finish 16 pl rows each: on one XCD, whose L2 they share.
            // (Workgroup w runs on XCD w mod 8; `slot`: the next workgroup of each.)  At most every second workgroup of the grid, because all
            // of them read the whole input (up to three quarters / half / a quarter of it: 7B-shaped chain 1126 / 1110 / 1206 us, a 70B-shaped
            // block 62 / 61 / 88).
            int pl = 1, all = 0;
            for (int v : nrb) all += v;
            const int slots = n_wg / 8, deep = (all + 7) / 8;         // workgroups, row blocks per XCD
            while (pl < 8 && 2 * deep * (8 / pl) > slots) pl *= 2;
            if (n_wg % 8 == 0 && deep * (8 / pl) <= slots) {
                int x = 0;
                for (int i = i0; i < i1; ++i)
                    for (int rb = 0; rb < nrb[i - i0]; ++rb, x = (x + 1) % 8)
                        for (int p0 = 0; p0 < 8; p0 += pl, slot[x] = (slot[x] + 1) % slots)
                            out.push_back(PlannedTask{8 * slot[x] + x, phase, i, stage, rb, 1, kExecWaves, p0, pl});
                continue;
            }
            int W = kExecWaves;
            auto runs = [&](int w) {
                int u = 0;
                for (int v : nrb) u += (v + kExecWaves / w - 1) / (kExecWaves / w);
                return u;
            };
            while (W > 1 && runs(W) > n_wg) W /= 2;
            const int per = kExecWaves / W;
            const int total = runs(W);
            // runs per workgroup when even one wave per row block leaves more runs than workgroups
            const int each = (total + n_wg - 1) / n_wg;
            int run = 0;
            for (int i = i0; i < i1; ++i) {
                for (int rb = 0; rb < nrb[i - i0]; rb += per, ++run) {
                    const int wg = (start + run / each) % n_wg;
                    const int cnt = std::min(per, nrb[i - i0] - rb);
                    if (!out.empty() && out.back().wg == wg && out.back().phase == phase && out.back().layer == i &&
                        out.back().rb0 + out.back().n_rb == rb)
                        out.back().n_rb += cnt;                 // the same workgroup goes on with the same layer
                    else
                        out.push_back(PlannedTask{wg, phase, i, stage, rb, cnt, W, 0, 0});
                }
            }
            start = (start + (total + each - 1) / each) % n_wg;
        }
        i0 = i1;
    }
}

}  // namespace nq

using namespace nq;

struct nq_exec_s {
    int n, n_wg, device;
    std::vector<nq_handle> handles;
    void* alloc;                    // tasks | task_begin | state | words handed over, both copies
    ExecTask* tasks;
    int* task_begin;
    ExecState* state;
    int bq_bytes;
    size_t lds_bytes, copy_words;
    int n_tasks;
};

static int exec_fail(int code, const char* msg)
{
    set_error(msg);
    return code;
}

// the lists as records of 9 (with the bit planes) or of 7 words
static int plan_records(const char* who, const int64_t* d_out, const int64_t* d_in, const int64_t* r, const int* level_of, int n,
                        int n_workgroups, int record, int32_t* tasks_out, int capacity, int* n_tasks)
{
    const std::string w(who);
    if (!d_out || !d_in || !r || !level_of || !n_tasks) return exec_fail(NQ_E_NULL, (w + ": NULL pointer").c_str());
    if (n < 1 || n_workgroups < 1) return exec_fail(NQ_E_INVALID_ARG, (w + ": n and n_workgroups must be >= 1").c_str());
    for (int i = 0; i < n; ++i) {
        if (d_out[i] < 1 || d_in[i] < 1 || r[i] < 1) return exec_fail(NQ_E_SHAPE, (w + ": dimensions must be >= 1").c_str());
        if (level_of[i] < 0 || (i > 0 && level_of[i] < level_of[i - 1]))
            return exec_fail(NQ_E_INVALID_ARG, (w + ": levels must be >= 0 and listed in order").c_str());
    }
    std::vector<PlannedTask> t;
    plan_tasks(d_out, d_in, r, level_of, n, n_workgroups, t);
    // (7 words cannot tell the planes of a row block apart: it is listed once)
    if (record == 7) t.erase(std::remove_if(t.begin(), t.end(), [](const PlannedTask& p) { return p.p0 != 0; }), t.end());
    *n_tasks = (int)t.size();
    if (tasks_out) {
        if ((int)t.size() > capacity) return exec_fail(NQ_E_INVALID_ARG, (w + ": tasks_out too small").c_str());
        for (size_t k = 0; k < t.size(); ++k) {
            const int32_t rec[9] = {t[k].wg, t[k].phase, t[k].layer, t[k].stage, t[k].rb0, t[k].n_rb, t[k].W, t[k].p0, t[k].pl};
            std::copy(rec, rec + record, tasks_out + record * k);
        }
    }
    return NQ_OK;
}

extern "C" int nq_exec_plan_tasks(const int64_t* d_out, const int64_t* d_in, const int64_t* r, const int* level_of, int n,
                                  int n_workgroups, int32_t* tasks_out, int capacity, int* n_tasks)
{
    return plan_records("nq_exec_plan_tasks", d_out, d_in, r, level_of, n, n_workgroups, 7, tasks_out, capacity, n_tasks);
}

extern "C" int nq_exec_plan_lists(const int64_t* d_out, const int64_t* d_in, const int64_t* r, const int* level_of, int n,
                                  int n_workgroups, int32_t* tasks_out, int capacity, int* n_tasks)
{
    return plan_records("nq_exec_plan_lists", d_out, d_in, r, level_of, n, n_workgroups, 9, tasks_out, capacity, n_tasks);
}

// ---------------------------------------------------------------------------------------------
// a lone small layer at batch 1: both stages in one launch by one workgroup (see exec_small_kernel)
// ---------------------------------------------------------------------------------------------
namespace nq {

// Off by default: measured on config 1 (1024 x 1024, r = 256, 66 KB of bits) one workgroup doing all ten row
// blocks of the two stages in turn takes 13.3 us per forward where the two launches that spread them over ten
// CUs take 10.2 us -- on this chip the latency of a stage is a wave's instruction stream, not the launch, and a
// lone workgroup serialises what the CUs do side by side.  The option "small_layer_kb" gives the packed size
// (both factors, KiB) up to which a lone layer at batch 1 takes this path.
constexpr int kSmallLayerKiB = 0;

bool small_layer_fits(nq_handle h, int batch)
{
    if (batch != 1 || opt_flag(OPT_NO_SMALL_LAYER)) return false;
    if (h->d_in > 16384 || h->r > 8192) return false;       // one chunk per thread; t in LDS
    const size_t tile_bytes = (tile_words(h->r, h->d_in) + tile_words(h->d_out, h->r)) * 4;
    return tile_bytes <= (size_t)opt_or(OPT_SMALL_LAYER_KB, kSmallLayerKiB) * 1024;
}

int launch_small_layer(nq_handle h, const DecodeWorkspace& w, const void* x, void* y, bool unscaled, hipStream_t s)
{
    ExecPair p{};
    // waves per row block: as many as leave every row block of the stage a place in ONE round (else one wave each, several rounds)
    auto wl_for = [](int64_t n_rb) {
        int W = kExecWaves;
        while (W > 1 && n_rb * W > kExecWaves) W /= 2;
        int wl = 0;
        while ((1 << wl) < W) ++wl;
        return wl;
    };
    ExecTask& a = p.t[0];
    a.tiles = h->vt_tiles; a.in = x; a.in_ll = 0; a.in_scale = h->s_in; a.out_scale = nullptr;
    a.out = w.t; a.out_ll = nullptr; a.out_lds = 1;
    a.M = (int)h->r; a.N = (int)h->d_in; a.n_steps = (int)n_steps(h->d_in); a.in_dtype = h->x_dtype; a.out_dtype = NQ_F32;
    a.rb0 = 0; a.n_rb = (int)n_rowblocks(h->r); a.wl = wl_for(a.n_rb); a.pl = 0;
    ExecTask& b = p.t[1];
    b.tiles = h->u_tiles; b.in = nullptr; b.in_ll = 2; b.in_scale = h->s_mid; b.out_scale = unscaled ? nullptr : h->s_out;
    b.out = y; b.out_ll = nullptr; b.out_lds = 0;
    b.M = (int)h->d_out; b.N = (int)h->r; b.n_steps = (int)n_steps(h->r); b.in_dtype = NQ_F32; b.out_dtype = h->y_dtype;
    b.rb0 = 0; b.n_rb = (int)n_rowblocks(h->d_out); b.wl = wl_for(b.n_rb); b.pl = 0;
    const int bq_bytes = (int)std::max(n_steps(h->d_in), n_steps(h->r)) * (int)kBqStepBytes;
    const size_t lds_bytes = (size_t)bq_bytes + (size_t)kExecWaves * kExecEpiInts * 4 + kExecWordBytes + (size_t)round_up(h->r, 16) * 4;
    NQ_ALLOW_LDS(exec_small_kernel, 160 * 1024);
    hipLaunchKernelGGL(exec_small_kernel, dim3(1), dim3(kExecThreads), lds_bytes, s, p, bq_bytes);
    NQ_HIP(hipGetLastError());
    return NQ_OK;
}

}  // namespace nq

extern "C" int nq_exec_destroy(nq_exec e)
{
    if (!e) return NQ_OK;
    (void)hipDeviceSynchronize();
    if (e->alloc) (void)hipFree(e->alloc);
    delete e;
    return NQ_OK;
}

extern "C" int nq_exec_create(nq_exec* out, const nq_handle* hs, const void* const* xs, void* const* ys,
                              const int* level_of, int n)
{
    if (!out) return exec_fail(NQ_E_NULL, "nq_exec_create: out is NULL");
    *out = nullptr;
    if (!hs || !xs || !ys || !level_of) return exec_fail(NQ_E_NULL, "nq_exec_create: NULL array");
    if (n < 1) return exec_fail(NQ_E_INVALID_ARG, "nq_exec_create: n must be >= 1");
    std::vector<int> src(n, -1);
    std::vector<char> consumed(n, 0);
    for (int i = 0; i < n; ++i) {
        nq_handle h = hs[i];
        if (!h) return exec_fail(NQ_E_NULL, "nq_exec_create: NULL handle in list");
        if (h->flags & NQ_FLAG_DECODE_VALU) return exec_fail(NQ_E_UNSUPPORTED, "nq_exec_create: handle uses NQ_FLAG_DECODE_VALU");
        if (h->device != hs[0]->device) return exec_fail(NQ_E_INVALID_ARG, "nq_exec_create: handles live on different devices");
        if (n_steps(h->d_in) > kExecMaxSteps || n_steps(h->r) > kExecMaxSteps)
            return exec_fail(NQ_E_SHAPE, "nq_exec_create: d_in and r must be <= 32768");
        if (level_of[i] < 0 || (i > 0 && level_of[i] < level_of[i - 1]))
            return exec_fail(NQ_E_INVALID_ARG, "nq_exec_create: levels must be >= 0 and listed in order");
        if (!xs[i] || !ys[i]) return exec_fail(NQ_E_NULL, "nq_exec_create: x or y is NULL");
        if (((uintptr_t)xs[i] | (uintptr_t)ys[i]) & 15u) return exec_fail(NQ_E_ALIGN, "nq_exec_create: x and y must be 16-byte aligned");
        for (int j = 0; j < i; ++j)
            if (hs[j] == h) return exec_fail(NQ_E_INVALID_ARG, "nq_exec_create: a handle appears twice");
    }
    // data flow: an input is either outside memory, or exactly the output of a layer of an earlier level
    auto bytes_x = [&](int i) { return (size_t)hs[i]->d_in * (hs[i]->x_dtype == NQ_F32 ? 4 : 2); };
    auto bytes_y = [&](int i) { return (size_t)hs[i]->d_out * (hs[i]->y_dtype == NQ_F32 ? 4 : 2); };
    auto overlap = [](const void* a, size_t na, const void* b, size_t nb) {
        return (const char*)a < (const char*)b + nb && (const char*)b < (const char*)a + na;
    };
    for (int i = 0; i < n; ++i) {
        for (int j = 0; j < n; ++j) {
            if (j != i && overlap(ys[i], bytes_y(i), ys[j], bytes_y(j)))
                return exec_fail(NQ_E_INVALID_ARG, "nq_exec_create: two outputs overlap");
            if (!overlap(xs[i], bytes_x(i), ys[j], bytes_y(j))) continue;
            const bool same = xs[i] == ys[j] && hs[i]->d_in == hs[j]->d_out && hs[i]->x_dtype == hs[j]->y_dtype;
            if (!same || level_of[j] >= level_of[i])
                return exec_fail(NQ_E_INVALID_ARG,
                                 "nq_exec_create: an input may overlap an output only by BEING the output (same pointer, "
                                 "length and type) of a layer of an earlier level");
            src[i] = j;
            consumed[j] = 1;
        }
    }

    nq_exec e = new (std::nothrow) nq_exec_s();
    if (!e) return exec_fail(NQ_E_HIP, "nq_exec_create: out of host memory");
    e->n = n; e->device = hs[0]->device; e->alloc = nullptr;
    e->handles.assign(hs, hs + n);
    // up to two workgroups per CU, and only as many as can be resident together
    int per_cu = 0;
    std::vector<int64_t> d_out(n), d_in(n), r(n);
    int max_steps = 4;
    for (int i = 0; i < n; ++i) {
        d_out[i] = hs[i]->d_out; d_in[i] = hs[i]->d_in; r[i] = hs[i]->r;
        max_steps = std::max(max_steps, (int)std::max(n_steps(d_in[i]), n_steps(r[i])));
    }
    e->bq_bytes = max_steps * (int)kBqStepBytes;
    e->lds_bytes = (size_t)e->bq_bytes + (size_t)kExecWaves * kExecEpiInts * 4 + kExecWordBytes;
    hipError_t he = hipFuncSetAttribute((const void*)exec_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (he == hipSuccess)
        he = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, (const void*)exec_kernel, kExecThreads, e->lds_bytes);
    if (he != hipSuccess) { delete e; return hip_fail(he, "occupancy query (executor)", __FILE__, __LINE__); }
    if (per_cu < 1) { delete e; return exec_fail(NQ_E_UNSUPPORTED, "nq_exec_create: the executor's workgroup does not fit a CU"); }
    e->n_wg = device_cu_count() * std::min(per_cu, 2);

    std::vector<PlannedTask> planned;
    plan_tasks(d_out.data(), d_in.data(), r.data(), level_of, n, e->n_wg, planned);
    // per workgroup, in phase order (plan_tasks emits phases in order: a stable sort by workgroup keeps it)
    std::stable_sort(planned.begin(), planned.end(), [](const PlannedTask& a, const PlannedTask& b) { return a.wg < b.wg; });
    std::vector<int> begin(e->n_wg + 1, 0);
    for (size_t k = 0; k < planned.size(); ++k) begin[planned[k].wg + 1] += 1;
    for (int w = 0; w < e->n_wg; ++w) begin[w + 1] += begin[w];
    e->n_tasks = (int)planned.size();

    auto al = [](size_t v) { return (v + 255) / 256 * 256; };
    const size_t tasks_b = al(sizeof(ExecTask) * planned.size()), begin_b = al(sizeof(int) * begin.size()),
                 state_b = al(sizeof(ExecState));
    size_t words = 0;                                      // bytes of one copy
    std::vector<size_t> t_off(n), y_off(n);
    for (int i = 0; i < n; ++i) {
        t_off[i] = words; words += al((size_t)hs[i]->r * 4);
        y_off[i] = words; if (consumed[i]) words += al((size_t)hs[i]->d_out * 4);
    }
    e->copy_words = words / 4;
    const size_t total = tasks_b + begin_b + state_b + 2 * words;
    he = hipMalloc(&e->alloc, total);
    if (he != hipSuccess) { delete e; return hip_fail(he, "hipMalloc(executor)", __FILE__, __LINE__); }
    char* c = (char*)e->alloc;
    e->tasks = (ExecTask*)c; c += tasks_b;
    e->task_begin = (int*)c; c += begin_b;
    e->state = (ExecState*)c; c += state_b;
    char* const word_base = c;
    // the two stages of every layer
    std::vector<ExecTask> ops(2 * n);
    for (int i = 0; i < n; ++i) {
        nq_handle h = hs[i];
        ExecTask& a = ops[2 * i];
        a = ExecTask{};
        a.tiles = h->vt_tiles;
        a.in = src[i] >= 0 ? (const void*)(word_base + y_off[src[i]]) : xs[i];
        a.in_ll = src[i] >= 0;
        a.in_scale = h->s_in; a.out_scale = nullptr;
        a.out = h->ws.t;                                   // (so that nq_binlr_read_intermediate sees it)
        a.out_ll = (unsigned int*)(word_base + t_off[i]);
        a.M = (int)h->r; a.N = (int)h->d_in; a.n_steps = (int)n_steps(h->d_in);
        a.in_dtype = h->x_dtype; a.out_dtype = NQ_F32;
        ExecTask& b = ops[2 * i + 1];
        b = ExecTask{};
        b.tiles = h->u_tiles;
        b.in = word_base + t_off[i]; b.in_ll = 1;
        b.in_scale = h->s_mid; b.out_scale = h->s_out;
        b.out = ys[i];
        b.out_ll = consumed[i] ? (unsigned int*)(word_base + y_off[i]) : nullptr;
        b.M = (int)h->d_out; b.N = (int)h->r; b.n_steps = (int)n_steps(h->r);
        b.in_dtype = NQ_F32; b.out_dtype = h->y_dtype;
    }
    std::vector<ExecTask> tasks(planned.size());
    for (size_t k = 0; k < planned.size(); ++k) {
        tasks[k] = ops[2 * planned[k].layer + planned[k].stage];
        tasks[k].rb0 = planned[k].rb0;
        tasks[k].n_rb = planned[k].n_rb;
        tasks[k].p0 = planned[k].p0;
        tasks[k].pl = planned[k].pl;
        int wl = 0;
        while ((1 << wl) < planned[k].W) ++wl;
        tasks[k].wl = wl;
    }
    ExecState st0{1u, 0u, 0, 0};
    he = hipMemset(e->alloc, 0, total);
    if (he == hipSuccess) he = hipMemset(word_base, 0xff, 2 * words);      // kNotThere
    if (he == hipSuccess) he = hipMemcpy(e->tasks, tasks.data(), sizeof(ExecTask) * tasks.size(), hipMemcpyHostToDevice);
    if (he == hipSuccess) he = hipMemcpy(e->task_begin, begin.data(), sizeof(int) * begin.size(), hipMemcpyHostToDevice);
    if (he == hipSuccess) he = hipMemcpy(e->state, &st0, sizeof st0, hipMemcpyHostToDevice);
    if (he == hipSuccess) he = hipDeviceSynchronize();
    if (he != hipSuccess) {
        (void)hipFree(e->alloc);
        delete e;
        return hip_fail(he, "upload (executor)", __FILE__, __LINE__);
    }
    *out = e;
    return NQ_OK;
}

extern "C" int nq_exec_forward(nq_exec e, void* stream)
{
    if (!e) return exec_fail(NQ_E_NULL, "nq_exec_forward: NULL executor");
    // wall-clock limit of every wait, in ticks of the 100 MHz constant clock (default 2 s)
    const int us = opt(OPT_EXEC_SPIN_LIMIT_US);
    const unsigned long long ticks = us >= 0 ? (unsigned long long)us * 100ull : 200000000ull;
    hipLaunchKernelGGL(exec_kernel, dim3(e->n_wg), dim3(kExecThreads), e->lds_bytes, (hipStream_t)stream, e->tasks,
                       e->task_begin, e->state, e->bq_bytes, e->copy_words, ticks);
    NQ_HIP(hipGetLastError());
    return NQ_OK;
}

extern "C" int nq_exec_status(nq_exec e, void* stream)
{
    if (!e) return exec_fail(NQ_E_NULL, "nq_exec_status: NULL executor");
    NQ_HIP(hipStreamSynchronize((hipStream_t)stream));
    ExecState st;
    NQ_HIP(hipMemcpy(&st, e->state, sizeof st, hipMemcpyDeviceToHost));
    if (st.error) {
        // clear the word (and the count of a launch that may have been cut short cannot be off: every workgroup leaves through it)
        int zero = 0;
        NQ_HIP(hipMemcpy(&e->state->error, &zero, sizeof zero, hipMemcpyHostToDevice));
        return exec_fail(NQ_E_TIMEOUT, "nq_exec_status: a wait inside the executor ran into its time limit; outputs of that launch are incomplete");
    }
    return NQ_OK;
}

extern "C" int nq_exec_info(nq_exec e, int* n_workgroups, int* n_tasks, size_t* lds_bytes)
{
    if (!e) return exec_fail(NQ_E_NULL, "nq_exec_info: NULL executor");
    if (n_workgroups) *n_workgroups = e->n_wg;
    if (n_tasks) *n_tasks = e->n_tasks;
    if (lds_bytes) *lds_bytes = e->lds_bytes;
    return NQ_OK;
}
