// Minibatch passes of small nets: one launch per direction that walks all layers.
//
// Samples are independent of each other in (z),(a) and in (bp2), so the minibatch is cut into slices and every slice is
// walked through all layers by a cluster of workgroups of its own, on one XCD: consecutive layers are then separated by an
// exchange inside that XCD's L2 (0.6 us among 16 workgroups, 1.0 to 1.2 among XCDs), not by a kernel boundary (2.5 to 3.5 us
// with the first requests behind it).  The price is that every cluster reads all the weights, which is why wide nets take the
// kernels of minibatch_kernels.h.  us a layer, a launch a layer -> here: fp32 forward N = 64 2.7 -> 0.9, N = 256 3.0 -> 1.4, N = 512
// 3.6 -> 2.7; the pass with gradients, L = 16, N = 64, B = 8 96 -> 41 us, N = 256, B = 32 112 -> 62, bf16 N = 512, B = 256 147 -> 96 (with
// the 1.8 us of the launch that prepares the exchange).
// What bounds it: a step is a chain of latencies (poll 400 cycles, matrix instructions 32 per 4 indices and wave, the waves'
// sum through LDS, sigma, store), and from N = 384 on what a compute unit takes in, weights and words at 40 bytes a cycle.
//
//   task       one tile of output neurons (16 of fp32, 32 of bf16) of one layer for one slice of up to 16 samples, by the
//              matrix instructions of four waves that share the contraction; four more waves fetch weights, and add up,
//              publish and store the results, so that nothing stands in front of the polls in a computing wave's queue
//              (loads and stores of a wave are waited for in order; with all of it in four waves N = 256 took 2.3 us a step).
//   exchange   64-bit words (32 bits of values, 32-bit tag), agent scope, relaxed, in the order in which the matrix
//              instructions of the next layer take them.  A reader that sees the tag has the value: no fence, no flag.  The
//              words of a layer are overwritten two layers on: whoever writes there has read all of the layer between, whose
//              writers have read all of these.  The tag tells the layers, and the launches, apart.
//   weights    do not depend on the exchange: they are requested three tasks ahead, as whole lines, and come to LDS a task ahead.
//              (Requested straight into LDS they took 100 to 200 cycles a KB to issue.)
//   progress   no workgroup waits for one that may not be running.  Tasks are numbered, layer by layer; a task needs
//              tasks of lower numbers only.  Workgroups take a first number as they arrive.  When all of a cluster have
//              arrived they are resident, and walk on in steps of their count (fixed shares: one task each per layer).  Where
//              they have not after a while (other work holds the compute units) those that run draw every further number
//              from the counter, in order: the lowest unfinished task is then always some running workgroup's current one.
//              The placement (cluster = workgroup index mod 8) decides the speed only.  Waits are bounded all the same: one that gives up
//              makes its values NaN and raises a word that the gradients' launch (no descent step then) and the host look at.
//   sums       in an order fixed by the shape alone.
#pragma once
#include "lf_internal.h"

#include <algorithm>
#include <cstdlib>

namespace lf {
namespace cluster {
namespace {

typedef unsigned long long u64;

constexpr int kWaves = 4;
constexpr int kThreads = 64 * 2 * kWaves;       // the computing waves, then those that help
constexpr int kTasks = 8;                       // numbers of tasks kept in LDS
constexpr int kRedRow = 80;                     // floats between the rows of the waves' partial tiles in LDS
constexpr unsigned kOutside = 0xFFFFFFF0u;      // an offset past the end of every buffer: loads zeros
constexpr unsigned kPatience = 1u << 23;        // polls a wave spends in vain in all (seconds): no wait is endless
constexpr int kDevice = 16;                     // device scope of a buffer access
constexpr unsigned kArrivalPolls = 256;         // how long the workgroups of a cluster wait for each other's arrival

template <typename T> struct Shape;             // Q: contraction indices of a unit = output neurons of a tile; M: 16-row blocks of them
template <> struct Shape<float> { static constexpr int Q = 16, M = 1; };
template <> struct Shape<__bf16> { static constexpr int Q = 32, M = 2; };

__host__ __device__ constexpr int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Words of the state block of a cluster.  (LOST: of the first block, for the whole pass)
enum { ARRIVED = 0, DECISION = 1, EXITED = 2, BASE = 3, LOST = 4, STATE_WORDS = 32 };
enum { UNDECIDED = 0, TOGETHER = 1, IN_ORDER = 2 };

struct Args {
    int layers;                                 // steps of this launch
    int B, S, ST;                               // samples; of a slice; slices of a cluster
    int clusters, per_cluster, expected;        // clusters; workgroups of one; arrivals that make it complete
    int units, nap;                             // units of the widest layer; pause before the first poll
    const void* in;                             // forward: a^{l-1} of the first step.  backward: a^L
    const void* y;                              // backward, first launch: y (delta^L is formed here); else NULL
    const void* d_in;                           // backward: delta^{l+1} of the first step as the products' operand
    float* d_top; void* d_top_bf;               // backward, first launch: where delta^L goes
    float scale;
    char* out; long out_step;                   // a^l or delta^l (fp32) of the steps, and bytes from one to the next
    char* out_bf;  long out_bf_step;            // backward, bf16: the copy of delta^l
    const char* act; long act_step;             // backward: a^l
    u64* words;                                 // [2][slices][units][256]
    unsigned* state;                            // [clusters][STATE_WORDS]
    unsigned patience;
    int layer;                                  // of the first step
    int* lost_host;                             // pinned word, or null
    const void* w[kClusterLayers];
    const float* b[kClusterLayers];
    int n[kClusterLayers + 1];                  // n[m]: contraction of step m; n[m + 1]: its outputs
};

__device__ __forceinline__ unsigned load_state(const unsigned* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Where a wait gave up (site 4 of the handle's abort word).
__device__ __forceinline__ int abort_code(int l, int workgroup) { return (4 << 24) | (l << 10) | (workgroup & 0x3ff); }

// Where output neuron c of a tile lies in a wave's partial tile: row `row` (of 4 M), lane 16 * group + sample.
template <typename T, bool BWD> __device__ __forceinline__ void place_of(int c, int* row, int* group) {
    if constexpr (sizeof(T) == 4) { *row = c & 3; *group = c >> 2; }
    else if constexpr (!BWD) { *row = 4 * (c >> 4) + (c & 3); *group = (c >> 2) & 3; }
    else { *row = 4 * (c & 1) + ((c >> 1) & 3); *group = c >> 3; }
}

template <typename T, bool BWD, int KU>
__global__ __launch_bounds__(kThreads, 2) void k_cluster(const Args g) {
    constexpr int Q = Shape<T>::Q, M = Shape<T>::M;
    constexpr int PW = Q / 16;                  // values of a word
    constexpr int KL = M * KU;                  // KB of a tile's weights that each of the four helping waves moves
    constexpr unsigned es = sizeof(T);
    extern __shared__ __attribute__((aligned(16))) char s_weights[];        // two tiles of 4 KL KB
    __shared__ const void* s_w[kClusterLayers];
    __shared__ const float* s_b[kClusterLayers];
    __shared__ int s_n[kClusterLayers + 1];
    __shared__ unsigned s_number[kTasks];       // task i's number at i % kTasks
    __shared__ unsigned s_base;
    __shared__ __attribute__((aligned(16))) float s_red[2][kWaves][4 * M * kRedRow];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), i16 = lane & 15, group = lane >> 4;
    const int c = blockIdx.x & 7;
    if (c >= g.clusters) return;
    const int slice0 = c * g.ST, slices = min(g.ST, ceil_div(g.B, g.S) - slice0);     // of this cluster
    if (slices <= 0) return;
    unsigned* const state = g.state + c * STATE_WORDS;
    const int slices_all = g.ST * g.clusters;
    const bool draws = threadIdx.x == 64 * kWaves;
    if (draws) {
        const unsigned number = __hip_atomic_fetch_add(state + ARRIVED, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s_number[0] = number;
        s_base = load_state(state + BASE);
        unsigned expected = UNDECIDED;
        if (number == (unsigned)g.expected - 1)                             // the last of them: all are resident
            __hip_atomic_compare_exchange_strong(state + DECISION, &expected, (unsigned)TOGETHER, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    for (int m = threadIdx.x; m <= g.layers; m += kThreads) {
        s_n[m] = g.n[m];
        if (m < g.layers) { s_w[m] = g.w[m]; s_b[m] = g.b[m]; }
    }
    __syncthreads();                                                        // the tables and the first number
    auto size_of = [&](int m) { return __builtin_amdgcn_readfirstlane(s_n[m]); };
    // contraction index, or output neuron, of value v (of PW) of word e of lane group gr
    auto index_of = [&](int e, int v, int gr) { return BWD ? 4 * (PW * e + v) + gr : 4 * PW * gr + PW * e + v; };
    const unsigned base = __builtin_amdgcn_readfirstlane(s_base);

    // Tasks in ascending order of their numbers.
    struct Task { int m, slice, ct, K, N; };                                // m < 0: past the last
    int at_m = 0, at_tiles = ceil_div(size_of(1), Q);
    unsigned at_first = 0;                                                  // number of step at_m's first task
    auto task = [&](int i) {
        const unsigned number = __builtin_amdgcn_readfirstlane(s_number[i % kTasks]);
        while (at_m < g.layers && number >= at_first + (unsigned)(slices * at_tiles)) {
            at_first += (unsigned)(slices * at_tiles);
            if (++at_m < g.layers) at_tiles = ceil_div(size_of(at_m + 1), Q);
        }
        if (at_m >= g.layers) return Task{-1, 0, 0, 4, 4};
        int ct = (int)(number - at_first), st = 0;
        while (ct >= at_tiles) { ct -= at_tiles; ++st; }
        return Task{at_m, slice0 + st, ct, size_of(at_m), size_of(at_m + 1)};
    };

    if (wave >= kWaves) {
        // ---- the waves that fetch the weights, three tasks ahead, and that add up, publish and store the results
        const int w = wave - kWaves, t = threadIdx.x - 64 * kWaves;
        const int r8 = lane >> 3, r16 = lane >> 2;
        // my word of a published block (as the loads take them: two words of a lane side by side), and its sample
        const int e = 2 * (t >> 7) + (t & 1), ps = (t >> 1) & 15, pg = ((t >> 1) & 63) >> 4;
        auto fetch = [&](v4f (&raw)[KL], const Task& x) {
            const __amdgpu_buffer_rsrc_t W = make_buffer(s_w[max(x.m, 0)], x.m < 0 ? 0u : (unsigned)x.K * (unsigned)x.N * es);
            const int n0 = x.ct * Q;
            if constexpr (!BWD) {
                // 1 KB: a 128-byte line of eight rows (rows past the end repeat the last; their results are not stored)
                const int row_bytes = x.K * (int)es;
#pragma unroll
                for (int k = 0; k < KL; ++k) {
                    const int n = kWaves * k + w, h = n % (Q / 8), at = 128 * (n / (Q / 8)) + 16 * (lane & 7);
                    raw[k] = buffer_load_v4f(W, at < row_bytes ? (unsigned)min(n0 + 8 * h + r8, x.N - 1) * (unsigned)row_bytes + at : kOutside);
                }
            } else {
                // 1 KB: 64 bytes of sixteen rows
                const bool in = n0 * (int)es + 16 * (lane & 3) < x.N * (int)es;
#pragma unroll
                for (int k = 0; k < KL; ++k) {
                    const int row = 16 * (kWaves * k + w) + r16;
                    raw[k] = buffer_load_v4f(W, in && row < x.K ? ((unsigned)row * (unsigned)x.N + n0) * es + 16u * (lane & 3) : kOutside);
                }
            }
        };
        auto put = [&](const v4f (&raw)[KL], int i) {
            v4f* const to = reinterpret_cast<v4f*>(s_weights + (i & 1) * (4096 * KL)) + (BWD ? lane : 8 * r8 + ((lane & 7) ^ r8));
#pragma unroll
            for (int k = 0; k < KL; ++k) to[64 * (kWaves * k + w)] = raw[k];
        };
        v4f raw0[KL], raw1[KL];
        Task x0 = task(0);
        fetch(raw0, x0);
        unsigned mode = UNDECIDED, number = s_number[0];
        auto draw = [&](int i) {                                            // task i's number
            if (!draws) return;
            if (mode == TOGETHER) number += (unsigned)g.per_cluster;
            else number = __hip_atomic_fetch_add(state + ARRIVED, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_number[i % kTasks] = number;
        };
        if (draws) {
            for (unsigned polls = 0; mode == UNDECIDED; ++polls) {
                mode = load_state(state + DECISION);
                if (mode != UNDECIDED) break;
                if (polls < kArrivalPolls) { __builtin_amdgcn_s_sleep(4); continue; }
                unsigned expected = UNDECIDED;
                __hip_atomic_compare_exchange_strong(state + DECISION, &expected, (unsigned)IN_ORDER, __ATOMIC_RELAXED,
                                                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        for (int i = 1; i <= 3; ++i) draw(i);
        __syncthreads();                                                    // the next numbers
        Task x1 = task(1), x2 = task(2);
        fetch(raw1, x1);
        put(raw0, 0);
        fetch(raw0, x2);
        __syncthreads();                                                    // the first weights
        // Step i: task i + 1's weights go to LDS, task i + 3's are requested into the same registers; then task i's results.
        auto step = [&](int i, v4f (&raw)[KL]) {
            const int n0 = x0.ct * Q, b0 = x0.slice * g.S, nsamples = min(g.S, g.B - b0);
            const bool mine = ps < nsamples;
            float own[PW];                                                  // bias, or a^l
            unsigned at[PW];                                                // where my values go
#pragma unroll
            for (int z = 0; z < PW; ++z) {
                const int col = n0 + index_of(e, z, pg);
                at[z] = mine && col < x0.N ? (unsigned)(b0 + ps) * (unsigned)x0.N + col : kOutside;
                if constexpr (!BWD) {
                    own[z] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(make_buffer(s_b[x0.m], (unsigned)x0.N * 4u), 4u * col, 0, 0));
                } else {
                    const __amdgpu_buffer_rsrc_t A = make_buffer(g.act + (long)x0.m * g.act_step, (unsigned)g.B * (unsigned)x0.N * es);
                    const unsigned off = at[z] == kOutside ? kOutside : at[z] * es;
                    if constexpr (PW == 1) own[z] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(A, off, 0, 0));
                    else own[z] = __uint_as_float((unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(A, off, 0, 0) << 16);
                }
            }
            // (addresses are formed in front of the barrier: what follows it is on every other workgroup's path)
            const float* part[PW];
#pragma unroll
            for (int z = 0; z < PW; ++z) {
                int row, gr;
                place_of<T, BWD>(index_of(e, z, pg), &row, &gr);
                part[z] = s_red[i & 1][0] + row * kRedRow + 16 * gr + ps;
                asm volatile("" : "+v"(part[z]));
            }
            u64* word = g.words + (((size_t)((x0.m + 1) & 1) * slices_all + x0.slice) * g.units + x0.ct) * 256 + t;
            asm volatile("" : "+v"(word));
            const bool publish = x0.m + 1 < g.layers && mine;
            const u64 tag = (u64)(base + (unsigned)x0.m + 1u) << 32;
            __builtin_amdgcn_sched_barrier(0);
            put(raw, i + 1);
            const Task x3 = task(i + 3);
            draw(i + 4);
            fetch(raw, x3);
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();                                                // the four waves' parts
            __builtin_amdgcn_sched_barrier(0);
            float v[PW];
#pragma unroll
            for (int z = 0; z < PW; ++z) {
                float u = part[z][0];
#pragma unroll
                for (int q = 1; q < kWaves; ++q) u += part[z][q * 4 * M * kRedRow];
                v[z] = BWD ? u * (own[z] * (1.0f - own[z])) : sigmoidf(u + own[z]);
                if (at[z] == kOutside) v[z] = 0.0f;                         // past the layer's end: the next one's padding
            }
            typedef __bf16 v2 __attribute__((ext_vector_type(2)));
            unsigned bits;
            if constexpr (PW == 1) bits = __float_as_uint(v[0]);
            else bits = __builtin_bit_cast(unsigned, v2{(__bf16)v[0], (__bf16)v[1]});
            if (publish) __hip_atomic_store(word, tag | bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __builtin_amdgcn_sched_barrier(0);
            // (an offset outside the buffer stores nothing)
            const __amdgpu_buffer_rsrc_t out = make_buffer(g.out + (long)x0.m * g.out_step, (unsigned)g.B * (unsigned)x0.N * (BWD ? 4u : es));
            if constexpr (PW == 1) {
                __builtin_amdgcn_raw_buffer_store_b32(bits, out, at[0] == kOutside ? kOutside : 4u * at[0], 0, 0);
            } else if constexpr (!BWD) {                                    // (two neighbours)
                __builtin_amdgcn_raw_buffer_store_b32(bits, out, at[0] == kOutside ? kOutside : 2u * at[0], 0, 0);
            } else {
                const __amdgpu_buffer_rsrc_t copy = make_buffer(g.out_bf + (long)x0.m * g.out_bf_step, (unsigned)g.B * (unsigned)x0.N * 2u);
#pragma unroll
                for (int z = 0; z < 2; ++z) {
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[z]), out, at[z] == kOutside ? kOutside : 4u * at[z], 0, 0);
                    __builtin_amdgcn_raw_buffer_store_b16((short)(bits >> 16 * z), copy, at[z] == kOutside ? kOutside : 2u * at[z], 0, 0);
                }
            }
            x0 = x1; x1 = x2; x2 = x3;
        };
        for (int i = 0; x0.m >= 0; i += 2) {
            step(i, raw1);
            if (x0.m < 0) break;
            step(i + 1, raw0);
        }
        // the last to leave prepares the pass's next launch
        if (draws) {
            const unsigned gone = __hip_atomic_fetch_add(state + EXITED, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (gone == (unsigned)g.per_cluster - 1) {
                __hip_atomic_store(state + ARRIVED, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(state + DECISION, (unsigned)UNDECIDED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(state + EXITED, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(state + BASE, base + (unsigned)g.layers, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        return;
    }

    // ---- the waves that compute: units 4 s + wave of the contraction
    const __amdgpu_buffer_rsrc_t words = make_buffer(g.words, 2u * (unsigned)slices_all * (unsigned)g.units * 2048u);
    unsigned patience = g.patience;
    __syncthreads();                                                        // the next numbers
    __syncthreads();                                                        // the first weights
    Task x = task(0);
    for (int i = 0; x.m >= 0; ++i) {
        const int b0 = x.slice * g.S, nsamples = min(g.S, g.B - b0), units = ceil_div(x.K, Q);
        // the weights as the matrix instructions take them
        typedef unsigned v8u __attribute__((ext_vector_type(8)));
        v4f wf[BWD ? 1 : KU][M];
        v8u wb[BWD ? KU : 1];
        const char* const wt = s_weights + (i & 1) * (4096 * KL);
        if constexpr (!BWD) {
            const char* const p = wt + 1024 * (Q / 8) * (wave >> 1) + 1024 * (i16 >> 3) + 128 * (i16 & 7) +
                                  16 * ((4 * (wave & 1) + group) ^ (i16 & 7));
#pragma unroll
            for (int s = 0; s < KU; ++s)
#pragma unroll
                for (int h = 0; h < M; ++h) wf[s][h] = *reinterpret_cast<const v4f*>(p + 2048 * (Q / 8) * s + 2048 * h);
        } else {
#pragma unroll
            for (int s = 0; s < KU; ++s)
#pragma unroll
                for (int y = 0; y < Q / 4; ++y)
                    wb[s][y] = *reinterpret_cast<const unsigned*>(wt + 64 * Q * (kWaves * s + wave) + 256 * y + 4 * lane);
        }
        const Task next = task(i + 1);
        v4u xs[KU];                                                         // the units' four words' values, of my sample
        const bool mine = i16 < nsamples;
        if (x.m == 0) {
            const size_t row = (size_t)(b0 + min(i16, nsamples - 1)) * x.K;
#pragma unroll
            for (int s = 0; s < KU; ++s) {
                const int u = kWaves * s + wave;
                xs[s] = v4u{0, 0, 0, 0};
                if constexpr (!BWD) {                                       // (K is a multiple of 4 PW)
                    const int k = u * Q + index_of(0, 0, group);
                    if (mine && k < x.K) xs[s] = *reinterpret_cast<const v4u*>(static_cast<const T*>(g.in) + row + k);
                } else {
#pragma unroll
                    for (int y = 0; y < 4; ++y) {
                        float v[PW];
#pragma unroll
                        for (int z = 0; z < PW; ++z) {
                            const int k = u * Q + index_of(y, z, group);
                            v[z] = 0.0f;
                            if (!mine || k >= x.K) continue;
                            if (g.y) {                                      // (bp1)
                                const float a = (float)static_cast<const T*>(g.in)[row + k];
                                v[z] = g.scale * ((a - (float)static_cast<const T*>(g.y)[row + k]) * (a * (1.0f - a)));
                                if (u % ceil_div(x.N, Q) == x.ct) {         // the tiles of the first step share its stores
                                    g.d_top[row + k] = v[z];
                                    if constexpr (PW == 2) static_cast<__bf16*>(g.d_top_bf)[row + k] = (__bf16)v[z];
                                }
                            } else {
                                v[z] = (float)static_cast<const T*>(g.d_in)[row + k];
                            }
                        }
                        typedef __bf16 v2 __attribute__((ext_vector_type(2)));
                        if constexpr (PW == 1) xs[s][y] = __float_as_uint(v[0]);
                        else xs[s][y] = __builtin_bit_cast(unsigned, v2{(__bf16)v[0], (__bf16)v[1]});
                    }
                }
            }
        } else {
            // (units past the last one, and lanes past the slice's samples, load zeros from outside the buffer)
            const unsigned at = mine ? (((unsigned)(x.m & 1) * slices_all + x.slice) * (unsigned)g.units) * 2048u + 16u * lane : kOutside;
            const unsigned tag = mine ? base + (unsigned)x.m : 0u;
            for (int p = 0; p < g.nap; ++p) __builtin_amdgcn_s_sleep(1);
            for (;;) {
                v4u y[KU][2];
                unsigned bad = 0;
#pragma unroll
                for (int s = 0; s < KU; ++s) {
                    const int u = kWaves * s + wave;
                    const unsigned off = u < units ? at : kOutside;
                    y[s][0] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(words, off, 2048 * u, kDevice));
                    y[s][1] = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(words, off, 2048 * u + 1024, kDevice));
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < KU; ++s) {
                    const unsigned want = kWaves * s + wave < units ? tag : 0u;
                    bad |= ((y[s][0][1] ^ want) | (y[s][0][3] ^ want)) | ((y[s][1][1] ^ want) | (y[s][1][3] ^ want));
                    xs[s] = v4u{y[s][0][0], y[s][0][2], y[s][1][0], y[s][1][2]};
                }
                if (__all(bad == 0u)) break;
                if (patience == 0) {                                        // the pass is lost: NaN, and both words say so
                    xs[0][0] = 0x7fc07fc0u;
                    __hip_atomic_store(g.state + LOST, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (g.lost_host)
                        __hip_atomic_store(g.lost_host, abort_code(BWD ? g.layer - x.m : g.layer + x.m, (int)blockIdx.x), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_SYSTEM);
                    break;
                }
                if ((--patience & 255u) == 0 && load_state(g.state + LOST)) patience = 0;
                __builtin_amdgcn_s_sleep(1);
                asm volatile("" ::: "memory");
            }
        }
        v4f acc[M];
#pragma unroll
        for (int h = 0; h < M; ++h) acc[h] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < KU; ++s) {
            if constexpr (M == 1) {
#pragma unroll
                for (int y = 0; y < 4; ++y) {
                    const float w = BWD ? __uint_as_float(wb[BWD ? s : 0][y]) : wf[BWD ? 0 : s][0][y];
                    acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(w, __uint_as_float(xs[s][y]), acc[0], 0, 0, 0);
                }
            } else {
                const v8bf b = __builtin_bit_cast(v8bf, xs[s]);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    v8bf a;
                    if constexpr (!BWD) {
                        a = __builtin_bit_cast(v8bf, wf[s][h]);
                    } else {
                        v4u p;
#pragma unroll
                        for (int d = 0; d < 4; ++d)
                            p[d] = __builtin_amdgcn_perm(wb[s][2 * d + 1], wb[s][2 * d], h ? 0x07060302u : 0x05040100u);
                        a = __builtin_bit_cast(v8bf, p);
                    }
                    acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[h], 0, 0, 0);
                }
            }
        }
        float* const red = s_red[i & 1][wave] + lane;
#pragma unroll
        for (int h = 0; h < M; ++h)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[(4 * h + r) * kRedRow] = acc[h][r];
        __syncthreads();                                                    // the four waves' parts
        x = next;
    }
}

// Whatever the workspace held: every counter at its start, and no word with a tag that is waited for (those of a pass begin at 2).
__global__ void k_cluster_state(unsigned* state, u64* words, size_t n) {
    v4u* const pairs = reinterpret_cast<v4u*>(words);           // (the words of a unit are 256)
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n / 2; i += (size_t)gridDim.x * blockDim.x) pairs[i] = v4u{0, 0, 0, 0};
    if (blockIdx.x == 0 && threadIdx.x < 8 * STATE_WORDS) state[threadIdx.x] = threadIdx.x % STATE_WORDS == BASE ? 1u : 0u;
}

// Units of the contraction that each wave of a kernel takes, where the widest one of a launch has this many units.
int units_a_wave(int units) {
    const int ku = ceil_div(units, kWaves);
    return ku <= 4 ? ku : ku <= 6 ? 6 : 8;
}

template <typename T, bool BWD>
hipError_t launch_steps(const Args& g, int widest_contraction, hipStream_t s) {
    const int grid = g.per_cluster * 8;         // (workgroup x goes to XCD x mod 8)
    auto launch = [&](auto kernel, int KU) -> hipError_t {
        kernel<<<grid, kThreads, 2 * 4096 * Shape<T>::M * KU, s>>>(g);
        return hipGetLastError();
    };
    const int units = ceil_div(widest_contraction, Shape<T>::Q);
    if (units > 8 * kWaves) return hipErrorInvalidValue;
    switch (units_a_wave(units)) {
        case 1: return launch(k_cluster<T, BWD, 1>, 1);
        case 2: return launch(k_cluster<T, BWD, 2>, 2);
        case 3: return launch(k_cluster<T, BWD, 3>, 3);
        case 4: return launch(k_cluster<T, BWD, 4>, 4);
        case 6: return launch(k_cluster<T, BWD, 6>, 6);
        default: return launch(k_cluster<T, BWD, 8>, 8);
    }
}

// The launches of a direction: at most kClusterLayers steps each.
template <typename T, bool BWD>
hipError_t run(const ClusterPass& p, hipStream_t s) {
    const int all = BWD ? p.L - 2 : p.L - 1;            // steps of the pass
    for (int from = 0; from < all; from += kClusterLayers) {
        Args g{};
        g.layers = std::min(kClusterLayers, all - from);
        g.B = p.B; g.S = p.plan.S; g.ST = p.plan.ST;
        g.clusters = p.plan.clusters; g.per_cluster = p.plan.per_cluster; g.expected = p.plan.expected;
        g.units = p.plan.units; g.nap = p.plan.nap;
        int widest = 0;
        for (int i = 0; i <= g.layers; ++i) g.n[i] = BWD ? p.n[p.L - 1 - from - i] : p.n[from + i];
        for (int i = 0; i < g.layers; ++i) widest = std::max(widest, g.n[i]);
        g.words = p.words; g.state = p.state;
        g.patience = p.plan.patience; g.lost_host = p.lost_host;
        g.layer = BWD ? p.L - 1 - from : from + 2;
        for (int i = 0; i < g.layers; ++i) {
            const int l = BWD ? p.L - 1 - from - i : from + i + 2;      // the layer whose a^l or delta^l step i forms
            g.w[i] = p.w[(BWD ? l + 1 : l) - 2];
            if (!BWD) g.b[i] = p.b[l - 2];
        }
        if (!BWD) {
            g.in = from == 0 ? p.x : p.a + (size_t)(from - 1) * p.a_stride;
            g.out = p.a + (size_t)from * p.a_stride;
            g.out_step = (long)p.a_stride;
        } else {
            const int l = p.L - 1 - from;                               // of the first step
            g.out = p.d + (size_t)(l - 2) * p.d_stride; g.out_step = -(long)p.d_stride;
            if (sizeof(T) == 2) { g.out_bf = p.d_bf + (size_t)(l - 2) * p.d_bf_stride; g.out_bf_step = -(long)p.d_bf_stride; }
            g.act = p.a + (size_t)(l - 2) * p.a_stride; g.act_step = -(long)p.a_stride;
            if (from == 0) {
                g.in = p.a + (size_t)(p.L - 2) * p.a_stride;
                g.y = p.y; g.scale = p.scale;
                g.d_top = reinterpret_cast<float*>(p.d + (size_t)(p.L - 2) * p.d_stride);
                if (sizeof(T) == 2) g.d_top_bf = p.d_bf + (size_t)(p.L - 2) * p.d_bf_stride;
            } else {
                g.d_in = sizeof(T) == 2 ? static_cast<const void*>(p.d_bf + (size_t)(l - 1) * p.d_bf_stride)
                                        : static_cast<const void*>(p.d + (size_t)(l - 1) * p.d_stride);
            }
        }
        const hipError_t e = launch_steps<T, BWD>(g, widest, s);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// What a direction's launches take, in us: `start` a launch, and a step for each layer.  Every task of a launch moves and multiplies
// the units of the launch's widest contraction, whatever its own layer's (`unit`, from a least of `least` on), finds its place among the
// slices (`slice` each), and where workgroups have one task or none it also waits for its own layer's words (`wait` an index); two
// turns of tasks take the time of `pair` steps, more of them a step each.  The first step of the chain forms delta^L from a^L and y
// (`top` an index).
struct StepPrices { double start, least, base, unit, slice, wait, pair, top; };
constexpr StepPrices kForwardPrices[] = {{5.5, 0.915, 0.62, 0.178, 0.0094, 0.0011, 1.67, 0.0}, {5.5, 1.035, 0.62, 0.236, 0.0094, 0.0007, 1.96, 0.0}};
constexpr StepPrices kChainPrices[] = {{8.7, 0.825, 0.56, 0.197, 0.0061, 0.0, 1.55, 0.0102}, {9.0, 0.985, 0.673, 0.212, 0.0096, 0.0, 1.55, 0.0102}};
double steps_us(const ClusterPlan& p, const int* n, int L, bool bf16, bool backward) {
    const StepPrices& c = (backward ? kChainPrices : kForwardPrices)[bf16];
    const int Q = bf16 ? 32 : 16, all = backward ? L - 2 : L - 1;
    auto width = [&](int i) { return backward ? n[L - 1 - i] : n[i]; };         // contraction of step i, outputs of step i - 1
    double us = c.top * width(0);
    for (int from = 0; from < all; from += kClusterLayers) {
        const int to = std::min(all, from + kClusterLayers);
        int widest = 0;
        for (int i = from; i < to; ++i) widest = std::max(widest, width(i));
        const double step = std::max(c.least, c.base + c.unit * units_a_wave(ceil_div(widest, Q))) + c.slice * p.ST;
        us += c.start;
        for (int i = from; i < to; ++i) {
            const double turns = (double)p.ST * ceil_div(width(i + 1), Q) / p.per_cluster, one = step + c.wait * width(i);
            us += turns <= 1.0 ? one : std::max(one, std::max(c.pair, turns) * step);
        }
    }
    return us;
}
constexpr double kPrepare = 1.8;                // us of the launch that prepares the words (and up to half of one a MB)

}  // namespace
}  // namespace cluster

const unsigned* cluster_lost(const unsigned* state) { return state + cluster::LOST; }

ClusterPlan cluster_plan(const int* n, int L, int B, bool bf16) {
    using namespace cluster;
    ClusterPlan p{};
    const int Q = bf16 ? 32 : 16;
    int widest = 0;
    for (int i = 0; i < L; ++i) widest = std::max(widest, n[i]);
    // (what fewer layers would gain is less than 6 us a pass: L = 4, N = 64 10 -> 9 / 17 -> 12 us, N = 512 11 -> 14 / 15 -> 20)
    if (L < 5 || widest > 8 * kWaves * Q) return p;
    p.clusters = std::min(8, B);
    p.ST = ceil_div(B, 16 * p.clusters);
    p.S = ceil_div(B, p.clusters * p.ST);
    p.units = ceil_div(widest, Q);
    p.words = (size_t)2 * p.clusters * p.ST * p.units * 256;
    p.state_words = 8 * STATE_WORDS;
    p.grad_kind = grad_kind_of_all(n, L, B, bf16);
    if (p.ST > 255 || p.words * 8 >= 0xFFFFFFF0ull) return p;
    const int tasks = p.ST * p.units, ku = ceil_div(p.units, kWaves);
    p.per_cluster = std::min(tasks, 32);        // one a compute unit
    // LF_CLUSTER_INCOMPLETE=1: no cluster is ever complete, so that its workgroups draw every task (the tests' way there)
    const char* incomplete = std::getenv("LF_CLUSTER_INCOMPLETE");
    p.expected = p.per_cluster + (incomplete && incomplete[0] == '1' ? 1 : 0);
    // LF_CLUSTER_SPIN_LIMIT: polls before a wait gives up; 0 makes the first one that finds nothing fail (the tests' way there)
    const char* limit = std::getenv("LF_CLUSTER_SPIN_LIMIT");
    p.patience = limit ? (unsigned)std::strtoul(limit, nullptr, 10) : kPatience;
    // A poll that finds nothing costs a round trip, and its lines are taken from the writers: the first one is sent when the
    // words are about due.  us a layer forward, pauses of 0, 2, 4, 8, 14, 18 x 64 cycles: fp32 N = 64 1.19, 1.20, 1.20;
    // N = 256, B = 32 1.94, 1.77, 1.71, 1.83 (8);  N = 512, B = 16 3.20 (8), 3.00 (14), 3.09 (18);  bf16 N = 256, B = 32 1.69,
    // 1.64, 1.50, 1.47, 1.62;  N = 512, B = 256 2.43 (8), 2.18, 2.27.  With more than one task a layer for every workgroup the
    // words are there long before (fp32 N = 256, B = 512 3.13, 3.14, 3.15, 3.41 (8)).
    p.nap = tasks > p.per_cluster ? 0 : bf16 ? std::min(4 * ku, 22) : ku <= 4 ? ku : 2 * ku - 2;
    if (const char* e = std::getenv("LF_CLUSTER")) {
        p.forward = p.backward = e[0] == '1';   // (a tuning knob, read whenever a layout is made: the same for all of a handle)
        return p;
    }
    if (std::getenv("LF_GEMM_BIG")) return p;   // (which of the other kernels to take has been asked for)
    // What these kernels and those of one launch a layer take: fitted to 1700 uniform nets, L = 5 .. 64, N = 8 .. 512 (fp32) and 8 .. 1024
    // (bf16), B = 2 .. 32640, and 800 of unequal widths, within 5 to 8 % (root mean square) a side.  By the choice 17 of these nets take more
    // than 2 % longer than by a launch a layer, and 17 more than 10 % longer than by the better side; those it sends here gain 1.5 times.
    // us a pass forward / backward, a launch a layer -> here (the preparation with the forward pass), L = 8:
    //   fp32  N = 64, B = 32 19 -> 12 / 29 -> 15, B = 8192 145 -> 90 / 400 -> 128;  N = 256, B = 32 21 -> 17 / 31 -> 21, B = 300 27 -> 22 /
    //         43 -> 36, B = 512 29 -> 27 / 55 -> 42, B = 1024 37 -> 47 / 75 -> 70, B = 4096 114 -> 187 / 234 -> 265;  N = 384, B = 32 23 -> 20 /
    //         32 -> 28, B = 256 30 -> 28 / 46 -> 48, B = 512 39 -> 43 / 60 -> 72;  N = 512, B = 32 25 -> 28 / 33 -> 37, B = 256 34 -> 38 / 60 -> 67
    //   bf16  N = 256, B = 32 21 -> 15 / 31 -> 19, B = 512 24 -> 16 / 40 -> 28, B = 2048 42 -> 44 / 121 -> 80, B = 8192 114 -> 205 / 414 -> 324;
    //         N = 512, B = 32 22 -> 19 / 32 -> 29, B = 256 26 -> 20 / 45 -> 40, B = 384 30 -> 27 / 43 -> 57;  N = 768, B = 32 23 -> 27 / 33 -> 42, B =
    //         128 27 -> 27 / 52 -> 46, B = 256 35 -> 37 / 60 -> 70;  N = 1024, B = 32 24 -> 35 / 47 -> 52
    //   one layer of 512 among 64 (fp32) B = 32 20 -> 22 / 30 -> 24, B = 512 23 -> 28 / 50 -> 32;  64 and 1024 in turn (bf16) B = 32 22 -> 24 /
    //   37 -> 39, B = 512 31 -> 49 / 47 -> 70;  784, six of 256, 16 (bf16) B = 32 21 -> 22 / 31 -> 18
    // and what few layers make of the start, L = 5: fp32 N = 64, B = 32 12 -> 10 / 18 -> 13, N = 512 14 -> 17 / 20 -> 24.
    const double forward = steps_us(p, n, L, bf16, false);
    const double backward = steps_us(p, n, L, bf16, true) + all_gradients_us(n, L, B, bf16);
    p.forward = forward + kPrepare < layer_launches_us(n, L, B, bf16, false);
    p.backward = backward + (p.forward ? 0.0 : kPrepare) < layer_launches_us(n, L, B, bf16, true);
    p.forward = p.forward && p.backward;        // (the other kernels' descent step would not know of a lost forward pass)
    return p;
}

hipError_t launch_cluster_state(const ClusterPlan& plan, unsigned* state, unsigned long long* words, hipStream_t s) {
    cluster::k_cluster_state<<<256, 256, 0, s>>>(state, words, plan.words);
    return hipGetLastError();
}
hipError_t launch_cluster_forward(const ClusterPass& p, hipStream_t s) {
    return p.bf16 ? cluster::run<__bf16, false>(p, s) : cluster::run<float, false>(p, s);
}
hipError_t launch_cluster_chain(const ClusterPass& p, hipStream_t s) {
    return p.bf16 ? cluster::run<__bf16, true>(p, s) : cluster::run<float, true>(p, s);
}

}  // namespace lf
