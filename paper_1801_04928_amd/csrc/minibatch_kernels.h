// Minibatch (B > 1, and bf16 at any B) kernels that need neither LDS operand tiles nor a second pass: the three
// per-layer contractions as matrix instructions on fragments loaded straight from memory into registers.
//
//   forward (z),(a):  A_out[b][j] = sigma( sum_k A_in[b][k]  W[j][k]  + bias[j] )
//   chain   (bp2):    D_l[b][k]   = ( sum_j D_next[b][j] W_next[j][k] ) * A_l[b][k] (1 - A_l[b][k])
//   grads   (bp4):    nabla_w[j][k] = sum_b D[b][j] A_prev[b][k]        (bp3): nabla_b[j] = sum_b D[b][j]
//
// All three are  C[m][n] = sum_q P(m,q) Q(n,q)  with operands that are either contiguous along the contraction index
// q ("QC": element (i,q) at p[i*ld + q]) or along their own index ("IC": element (i,q) at p[q*ld + i]).  forward:
// P = A_in (QC), Q = W (QC).  chain: P = D_next (QC), Q = W_next (IC).  grads: P = D (IC), Q = A_prev (IC).
// Accumulation is fp32, in an order fixed by the shape alone, so results depend neither on k nor on the launch.
#pragma once
#include "lf_internal.h"

#include <algorithm>

namespace lf {
namespace direct {
namespace {

__host__ __device__ constexpr int ceil_div(int a, int b) { return (a + b - 1) / b; }

constexpr unsigned kOutside = 0xFFFFFFF0u;   // an offset past the end of every buffer: loads zeros
constexpr int kWaves = 4;                    // of every workgroup
constexpr int kSplitWorkgroups = 256;        // of a split chain product, at most: also the number of its arrival counters

// A unit of the contraction: the q's of one 64-byte piece of a QC row.  A 16 x 16 matrix instruction hands row
// (lane % 16) of its operand to a lane and one quarter (g = lane / 16) of the q's; which q's form a quarter is free as
// long as both operands agree.  Here lane group g holds q0 + PL g .. + PL - 1: 16 bytes of a QC row.
template <typename T> struct Unit;
template <> struct Unit<float> { static constexpr int Q = 16, PL = 4; };
template <> struct Unit<__bf16> { static constexpr int Q = 32, PL = 8; };

// One unit of NT 16-row tiles of an operand in registers.
template <typename T, bool IC, int NT> struct Operand;

// QC: tile t is rows i0 + 16 t .. + 15, and registers hold a pair of units: 128 bytes of every row, a whole cache line.
// The memory pipeline coalesces neighbouring lanes only, and the L2 serves a request per cycle and channel, of 64 bytes
// or of 128: eight neighbouring lanes load the line of a row (lane-per-row addressing, as the instructions want it,
// moves 16 bytes a cycle and compute unit instead of 64; half lines get half of the L2's rate).  A turn through 2 KB of
// LDS per tile that belong to the wave alone gives every lane its row.  LDS operations of a wave complete in order: no
// barrier, and the area can be overwritten by the next pair at once.  The 16-byte pieces of row i are placed by an
// exclusive or with i % 8: no bank conflicts either way.
template <typename T, int NT> struct Operand<T, false, NT> {
    static constexpr int kLdsVecs = 128 * NT;
    struct At {
        unsigned off[2 * NT];
        int qlane, write[2], read[2];
        __device__ At(int i0, int I, int ld) {
            const int lane = threadIdx.x & 63, row = lane >> 3, c = lane & 7, i = lane & 15, g = lane >> 4;
            qlane = Unit<T>::PL * c;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                write[h] = 8 * (row + 8 * h) + (c ^ row);
                read[h] = 8 * i + ((4 * h + g) ^ (i & 7));
            }
#pragma unroll
            for (int t = 0; t < 2 * NT; ++t)   // rows past the end repeat the last one (their results are not stored)
                off[t] = (unsigned)min(i0 + 8 * t + row, I - 1) * (unsigned)ld * (unsigned)sizeof(T) + 16u * c;
        }
    };
    struct Raw { v4f r[2 * NT]; };             // a pair, as loaded
    struct Op { v4f r[NT]; };                  // a unit, as the matrix instructions take it
    static __device__ __forceinline__ void load(Raw& x, __amdgpu_buffer_rsrc_t buf, const At& at, int q0, int K) {
        const bool ok = q0 + at.qlane < K;     // K is a multiple of PL
#pragma unroll
        for (int t = 0; t < 2 * NT; ++t)
            x.r[t] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(
                         buf, ok ? at.off[t] : kOutside, q0 * (int)sizeof(T), 0));
    }
    static __device__ __forceinline__ void put(const Raw& x, const At& at, v4f* lds) {
#pragma unroll
        for (int t = 0; t < 2 * NT; ++t) lds[128 * (t >> 1) + at.write[t & 1]] = x.r[t];
    }
    static __device__ __forceinline__ void take(Op& o, int unit, const At& at, const v4f* lds) {
#pragma unroll
        for (int t = 0; t < NT; ++t) o.r[t] = lds[128 * t + at.read[unit]];
    }
    static __device__ __forceinline__ float f32(const Op& o, int t, int e) { return o.r[t][e]; }
    static __device__ __forceinline__ v8bf bf(const Op& o, int t) { return __builtin_bit_cast(v8bf, o.r[t]); }
};

// IC: a lane loads NT consecutive i's of each of its PL q's; element t of each belongs to tile t, so tile t is the
// rows i0 + NT * (lane % 16) + t: a permutation of the NT * 16 rows that only the store has to know.
template <typename T, int NT> struct Operand<T, true, NT> {
    static constexpr int PL = Unit<T>::PL;
    static constexpr int W = NT * (int)sizeof(T) / 4;          // 32-bit words of one load
    static constexpr int kLdsVecs = 0;
    struct At {
        unsigned off;
        int qlane;
        __device__ At(int i0, int I, int ld) {
            const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
            qlane = PL * g;
            // columns past the end repeat the last ones (their results are not stored); I is a multiple of NT
            off = ((unsigned)qlane * (unsigned)ld + (unsigned)min(i0 + NT * i, I - NT)) * (unsigned)sizeof(T);
        }
    };
    struct Raw { unsigned r[PL][W]; };         // a unit, as loaded and as used
    typedef Raw Op;
    static __device__ __forceinline__ void load(Raw& x, __amdgpu_buffer_rsrc_t buf, const At& at, int ld, int q0, int K) {
#pragma unroll
        for (int e = 0; e < PL; ++e) {
            const unsigned off = q0 + at.qlane + e < K ? at.off : kOutside;
            const unsigned row = (unsigned)(q0 + e) * (unsigned)ld * (unsigned)sizeof(T);
            if constexpr (W == 4) {
                const v4u v = __builtin_bit_cast(v4u, __builtin_amdgcn_raw_buffer_load_b128(buf, off, row, 0));
#pragma unroll
                for (int c = 0; c < 4; ++c) x.r[e][c] = v[c];
            } else if constexpr (W == 2) {
                typedef unsigned v2u __attribute__((ext_vector_type(2)));
                const v2u v = __builtin_bit_cast(v2u, __builtin_amdgcn_raw_buffer_load_b64(buf, off, row, 0));
                x.r[e][0] = v[0];
                x.r[e][1] = v[1];
            } else {
                x.r[e][0] = __builtin_amdgcn_raw_buffer_load_b32(buf, off, row, 0);
            }
        }
    }
    static __device__ __forceinline__ float f32(const Raw& x, int t, int e) { return __uint_as_float(x.r[e][t]); }
    static __device__ __forceinline__ v8bf bf(const Raw& x, int t) {      // halves t % 2 of word t / 2 of the eight q's
        const unsigned sel = (t & 1) ? 0x07060302u : 0x05040100u;
        v4u v;
#pragma unroll
        for (int d = 0; d < 4; ++d) v[d] = __builtin_amdgcn_perm(x.r[2 * d + 1][t >> 1], x.r[2 * d][t >> 1], sel);
        return __builtin_bit_cast(v8bf, v);
    }
};

template <int W, int FROM, int TO>
__device__ __forceinline__ void interleave_ops() {              // operations FROM .. TO - 1: W writes, then reads
    if constexpr (FROM < TO) {
        if constexpr (FROM < W) {
            __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        } else {
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
        interleave_ops<W, FROM + 1, TO>();
    }
}
// Issue order of one unit as scheduling groups (mask 0x008 matrix instruction, 0x020 memory read, 0x100 LDS read, 0x200
// LDS write): after every matrix instruction its share of the W writes to LDS, each with the request that refills its
// register, and of the R reads, all within the first WINDOW of the M matrix instructions; behind each quarter (the one
// of four values of q) the IC requests that refill the registers it has read.  A SIMD often has a single wave, whose
// matrix instructions (32 cycles each in fp32) stand still while it issues anything in a row; left alone, the compiler
// puts a pair's 16 writes and 16 requests together, and the reads right in front of their use.  us per pass, before ->
// after: L = 32, N = 4096, B = 256 6966 -> 6005; L = 16, N = 2048, B = 64 396 -> 376; unequal widths, B = 100, 100 -> 95.
template <int M, int WINDOW, int W, int R, int IC, int I = 0>
__device__ __forceinline__ void interleave() {
    if constexpr (I < M) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        constexpr int ops = W + R, from = I < WINDOW ? I * ops / WINDOW : ops;
        constexpr int to = I + 1 < WINDOW ? (I + 1) * ops / WINDOW : ops;
        interleave_ops<W, from, to>();
        if constexpr (IC > 0 && (I + 1) % (M / 4) == 0) __builtin_amdgcn_sched_group_barrier(0x020, IC, 0);
        interleave<M, WINDOW, W, R, IC, I + 1>();
    }
}

// acc[mt][nt] += P Q^T of one 16*MT x 16*NT tile over the units of wave w of W that share the contraction: pairs of
// units are dealt to the waves in turn.  A QC operand is requested D pairs ahead of its way through LDS, which is half
// a pair ahead of its use; an IC operand E units ahead of its use.  lds: the workgroup's area, kLdsVecs vectors a wave.
template <typename T, bool P_IC, bool Q_IC, int MT, int NT>
__device__ __forceinline__ void contract(v4f (&acc)[MT][NT], float* lds, const void* p, unsigned p_bytes, int ldp, int m0,
                                         int M, const void* q, unsigned q_bytes, int ldq, int n0, int Nn, int K, int w,
                                         int W) {
    typedef Operand<T, P_IC, MT> OP;
    typedef Operand<T, Q_IC, NT> OQ;
    // requested ahead: as many pairs of QC units as about 96 registers hold, and at least four IC units (of 4 (MT + NT)
    // registers each in fp32: 128 for the gradients' 4 x 4 tiles)
    constexpr int kFit = 96 / (8 * (MT + NT));
    constexpr int D = kFit > 4 ? 4 : kFit;
    constexpr int E = D == 1 ? 4 : 2 * D;
    constexpr int U = (P_IC || Q_IC) ? E : 2 * D;               // units a turn of the loop
    constexpr int kMfmas = MT * NT * (sizeof(T) == 4 ? 4 : 1);  // matrix instructions a unit
    // bfloat16's matrix instructions are too short to cover the requests (N = 2048, B = 128: 466 -> 471 us interleaved)
    constexpr bool kInterleave = sizeof(T) == 4;
    const __amdgpu_buffer_rsrc_t P = make_buffer(p, p_bytes);
    const __amdgpu_buffer_rsrc_t Q = make_buffer(q, q_bytes);
    const typename OP::At pa(m0, M, ldp);
    const typename OQ::At qa(n0, Nn, ldq);
    v4f* const lp = reinterpret_cast<v4f*>(lds) + (threadIdx.x >> 6) * (OP::kLdsVecs + OQ::kLdsVecs);
    v4f* const lq = lp + OP::kLdsVecs;
    const int units = ceil_div(K, Unit<T>::Q), pairs = ceil_div(units, 2);
    // A QC operand goes through LDS by pairs; without one, a wave that has the contraction to itself ends with its last unit
    // (gradients, fp32, us a layer, pairs / units: N = 4096, B = 8 22.0 / 18.2;  N = 1500, B = 100 13.3 / 12.6).
    const int nu = P_IC && W == 1 ? units : (w < pairs ? 2 * ((pairs - w + W - 1) / W) : 0);
    // (units past the last one start at K or beyond and load zeros)
    auto q_of = [&](int j) { return (((j >> 1) * W + w) * 2 + (j & 1)) * Unit<T>::Q; };
    typename OP::Raw rp[P_IC ? E : D];
    typename OQ::Raw rq[Q_IC ? E : D];
    typename OP::Op op[2];
    typename OQ::Op oq[2];
    // unit j of an IC operand, or the pair that starts with unit j of a QC one, into slot d
    auto request_p = [&](int d, int j) {
        if constexpr (P_IC) OP::load(rp[d], P, pa, ldp, q_of(j), K);
        else OP::load(rp[d], P, pa, q_of(j), K);
    };
    auto request_q = [&](int d, int j) {
        if constexpr (Q_IC) OQ::load(rq[d], Q, qa, ldq, q_of(j), K);
        else OQ::load(rq[d], Q, qa, q_of(j), K);
    };
    auto put = [&](int d) {
        if constexpr (!P_IC) OP::put(rp[d], pa, lp);
        if constexpr (!Q_IC) OQ::put(rq[d], qa, lq);
    };
    auto take = [&](int unit) {
        if constexpr (!P_IC) OP::take(op[unit], unit, pa, lp);
        if constexpr (!Q_IC) OQ::take(oq[unit], unit, qa, lq);
    };
    auto multiply_ops = [&](const typename OP::Op& x, const typename OQ::Op& y) {
        if constexpr (sizeof(T) == 4) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(OP::f32(x, mt, e), OQ::f32(y, nt, e),
                                                                           acc[mt][nt], 0, 0, 0);
        } else {
            v8bf a[MT], b[NT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) a[mt] = OP::bf(x, mt);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) b[nt] = OQ::bf(y, nt);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    acc[mt][nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[mt], b[nt], acc[mt][nt], 0, 0, 0);
        }
    };
    auto multiply = [&](int u) {                                // unit u of a turn
        if constexpr (P_IC && Q_IC) multiply_ops(rp[u % E], rq[u % E]);
        else if constexpr (Q_IC) multiply_ops(op[u & 1], rq[u % E]);
        else multiply_ops(op[u & 1], oq[u & 1]);
    };
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[mt][nt] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int d = 0; d < (E > D ? E : D); ++d) {
        if (P_IC ? d < E : d < D) request_p(d, P_IC ? d : 2 * d);
        if (Q_IC ? d < E : d < D) request_q(d, Q_IC ? d : 2 * d);
    }
    __builtin_amdgcn_sched_barrier(0);
    put(0);
    if constexpr (!P_IC) request_p(0, 2 * D);
    if constexpr (!Q_IC) request_q(0, 2 * D);
    take(0);
    // One unit: the QC operands of the next one come from LDS (the first of a pair behind the pair's way there), the
    // slots that are free again are requested.  No branch inside the loop: on a path around a request or a use the
    // compiler's waits would have to cover loads that are younger than the unit needed.
    auto unit = [&](int u, int j) {
        __builtin_amdgcn_sched_barrier(0);                      // requests stay where they are written
        if (u & 1) {
            const int n = ((u + 1) / 2) % D;
            put(n);
            if constexpr (!P_IC) request_p(n, j + u + 1 + 2 * D);
            if constexpr (!Q_IC) request_q(n, j + u + 1 + 2 * D);
            take(0);
        } else {
            take(1);
        }
        multiply(u);
        if constexpr ((P_IC || Q_IC) && !kInterleave) __builtin_amdgcn_sched_barrier(0);
        if constexpr (P_IC) request_p(u % E, j + u + E);
        if constexpr (Q_IC) request_q(u % E, j + u + E);
        if constexpr (kInterleave) {
            constexpr int R = (P_IC ? 0 : MT) + (Q_IC ? 0 : NT), IC = (P_IC ? 1 : 0) + (Q_IC ? 1 : 0);
            constexpr int window = IC ? kMfmas / 2 : 3 * kMfmas / 4;
            if (u & 1) interleave<kMfmas, window, 2 * R, R, IC>();
            else interleave<kMfmas, window, 0, R, IC>();
        }
    };
    int j = 0;
    for (; j + U <= nu; j += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) unit(u, j);
    }
    if constexpr (P_IC) {
#pragma unroll
        for (int u = 0; u < U - 1; ++u)
            if (j + u < nu) unit(u, j);
    } else {
#pragma unroll
        for (int u = 0; u < U - 2; u += 2)
            if (j + u < nu) {
                unit(u, j);
                unit(u + 1, j);
            }
    }
}

// Where element r of lane (i = lane % 16, g = lane / 16) of acc[mt][nt] lies in the tile.
template <bool IC, int MT> __device__ __forceinline__ int tile_row(int mt, int idx) {      // idx = 4 g + r
    return IC ? MT * idx + mt : 16 * mt + idx;
}
template <bool IC, int NT> __device__ __forceinline__ int tile_col(int nt, int i) { return IC ? NT * i + nt : 16 * nt + i; }

constexpr int kPad = 4;
// LDS of a workgroup: the waves' operand areas (qc_tiles 16-row tiles of QC operands a wave), then the reduction's slices
constexpr size_t lds_bytes(int qc_tiles, int nt) {
    const int operands = kWaves * qc_tiles * 2048, slices = kWaves * 16 * (16 * nt + kPad) * 4;
    return operands > slices ? operands : slices;
}

// The waves' partial tiles are added in wave order through LDS, one 16-row slice (acc[mt]) at a time; `store(row, col,
// v4f)` then gets four consecutive columns of the tile.  Every thread of the workgroup calls it.
template <bool P_IC, bool Q_IC, int MT, int NT, typename Store>
__device__ __forceinline__ void reduce_waves(const v4f (&acc)[MT][NT], float* lds, Store store) {
    constexpr int TN = 16 * NT, LD = TN + kPad;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, i = lane & 15, g = lane >> 4;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) {
        __syncthreads();                                       // the slice before, or the waves' operand areas
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int r = 0; r < 4; ++r) lds[(wave * 16 + 4 * g + r) * LD + tile_col<Q_IC, NT>(nt, i)] = acc[mt][nt][r];
        __syncthreads();
        for (int v = t; v < 4 * TN; v += 64 * kWaves) {       // 16 rows of TN / 4 vectors
            const int idx = v / (TN / 4), c4 = (v % (TN / 4)) * 4;
            v4f s = *reinterpret_cast<const v4f*>(&lds[idx * LD + c4]);
            for (int q = 1; q < kWaves; ++q) s += *reinterpret_cast<const v4f*>(&lds[(q * 16 + idx) * LD + c4]);
            store(tile_row<P_IC, MT>(mt, idx), c4, s);
        }
    }
}

// The same for a tile whose contraction is split over workgroups as well: each stores its sum, and the last one to do so
// adds all of them, in the order of the splits, and stores the result.  No workgroup waits for another.  The sums pass
// through memory at device scope (aux 16) on either side: written through and acknowledged before the split is counted.
template <int MT, int NT, typename Store>
__device__ __forceinline__ void meet(const v4f (&acc)[MT][NT], float* lds, float* scratch, int tile, int splits, int split,
                                     Store store) {
    constexpr int TM = 16 * MT, TN = 16 * NT, kDevice = 16;
    unsigned* const arrived = reinterpret_cast<unsigned*>(scratch) + tile;
    const __amdgpu_buffer_rsrc_t buf = make_buffer(scratch + kSplitWorkgroups + (size_t)tile * splits * TM * TN,
                                                   (unsigned)splits * TM * TN * 4u);
    reduce_waves<false, true, MT, NT>(acc, lds, [&](int row, int col, v4f u) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, u), buf, ((split * TM + row) * TN + col) * 4, 0, kDevice);
    });
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0)
        lds[0] = (float)__hip_atomic_fetch_add(arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (lds[0] != (float)(splits - 1)) return;                 // (the same for every thread)
    if (threadIdx.x == 0) __hip_atomic_store(arrived, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    for (int v = threadIdx.x; v < TM * TN / 4; v += 64 * kWaves) {
        const int at = v * 16;
        v4f s = {0.0f, 0.0f, 0.0f, 0.0f};
        for (int z = 0; z < splits; z += 4) {                   // (past the last split: zeros from outside the buffer)
            v4f x[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                x[u] = __builtin_bit_cast(v4f, __builtin_amdgcn_raw_buffer_load_b128(buf, at + (z + u) * TM * TN * 4, 0, kDevice));
#pragma unroll
            for (int u = 0; u < 4; ++u) s += x[u];
        }
        store(v / (TN / 4), v % (TN / 4) * 4, s);
    }
}

// ---- forward ------------------------------------------------------------------------------------------------
struct ForwardArgs {
    const void* A_in; const void* W; const float* bias; void* A_out;
    unsigned a_bytes, w_bytes;
    int B, n_out, n_in;
    int tiles_m, tiles_n;
};

// Tile of workgroup x.  Workgroups go to the 8 XCDs in turn: an XCD takes an eighth of the tile columns, side by side,
// and the workgroups that share weights (equal tn) follow each other there, so its L2 serves all but the first.
// (Every eighth column instead: L = 10, N = 4096, fp32, B = 16 backward 42.1 -> 35.1 us a layer.)
__device__ __forceinline__ void tile_of(int x, int tiles_m, int tiles_n, int* tm, int* tn) {
    *tm = (x >> 3) % tiles_m;
    *tn = (x >> 3) / tiles_m + (x & 7) * ceil_div(tiles_n, 8);
}

template <typename T, int MT, int NT>
__global__ __launch_bounds__(64 * kWaves, 2) void k_forward_tile(const ForwardArgs g) {
    extern __shared__ __attribute__((aligned(16))) float lds[];
    int tm, tn;
    tile_of(blockIdx.x, g.tiles_m, g.tiles_n, &tm, &tn);
    if (tn >= g.tiles_n) return;
    const int m0 = tm * 16 * MT, n0 = tn * 16 * NT;
    v4f acc[MT][NT];
    contract<T, false, false, MT, NT>(acc, lds, g.A_in, g.a_bytes, g.n_in, m0, g.B, g.W, g.w_bytes, g.n_in, n0, g.n_out,
                                      g.n_in, __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), kWaves);
    reduce_waves<false, false, MT, NT>(acc, lds, [&](int row, int col, v4f z) {
        const int m = m0 + row, n = n0 + col;
        if (m >= g.B || n >= g.n_out) return;
        const v4f bs = *reinterpret_cast<const v4f*>(g.bias + n);
        typedef T v4t __attribute__((ext_vector_type(4)));
        const v4t a = {(T)sigmoidf(z[0] + bs[0]), (T)sigmoidf(z[1] + bs[1]), (T)sigmoidf(z[2] + bs[2]),
                       (T)sigmoidf(z[3] + bs[3])};
        *reinterpret_cast<v4t*>(static_cast<T*>(g.A_out) + (size_t)m * g.n_out + n) = a;
    });
}

// ---- backward -----------------------------------------------------------------------------------------------
struct GradJob {                    // (bp3), (bp4) of one layer
    const void* D_op;               // delta^l as the products' operand (fp32, or its bfloat16 copy)
    const float* D;                 // delta^l
    const void* A_prev;
    float* w; float* b; void* w_bf;
    unsigned d_bytes, a_bytes;
    int n_l, n_prev;
    int tiles_x, tile_blocks, blocks;   // workgroups: tile_blocks for nabla_w, the rest for nabla_b
    const unsigned* lost;               // none, or != 0 there: what a descent step would apply is not to be trusted
};
struct StepArgs {
    // the chain: delta^l from delta^{l+1}
    const void* D_next; const void* W_next; const void* A_l; float* D_l; void* D_l_bf;
    unsigned d_bytes, w_bytes;
    int n_l, n_next;
    int tiles_m, tiles_n, splits, chain_blocks;
    float* scratch;                     // splits > 1: how many of a tile's splits have arrived, and their partial tiles
    GradJob grad[2];
    int B;
    float sgd_eta;
};

// nabla_b[j] = sum_b D[b][j]: 32 columns a workgroup; eight row groups each add every 8th sample in ascending order,
// then the eight partial sums are added in group order.
__device__ __forceinline__ void bias_block(const GradJob& g, int x, int B, float sgd_eta, float* lds) {
    const int t = threadIdx.x, c = t & 31, rg = t >> 5;
    const int j = x * 32 + c;
    float s = 0.0f;
    if (j < g.n_l) {
        int b = rg;
        for (; b + 56 < B; b += 64) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = g.D[(size_t)(b + 8 * u) * g.n_l + j];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; b < B; b += 8) s += g.D[(size_t)b * g.n_l + j];
    }
    lds[rg * 32 + c] = s;
    __syncthreads();
    if (rg == 0 && j < g.n_l) {
        s = lds[c];
#pragma unroll
        for (int q = 1; q < 8; ++q) s += lds[q * 32 + c];
        if (sgd_eta == 0.0f) g.b[j] = s;
        else if (!g.lost || *g.lost == 0) g.b[j] = fmaf(-sgd_eta, s, g.b[j]);
    }
}

// R vectors of nabla_w (N consecutive columns of row m[r] from column n[r] on): stored, or applied to the weights, whose
// old values are then requested together (entries past the edges re-read the last ones and are not written).
template <int R, int N, typename At, typename Value>
__device__ __forceinline__ void put_grads(const GradJob& g, float sgd_eta, At at, Value value) {
    typedef float vf __attribute__((ext_vector_type(N)));
    typedef __bf16 vb __attribute__((ext_vector_type(N)));
    if (sgd_eta == 0.0f) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            int m, n;
            at(r, &m, &n);
            if (m >= g.n_l || n >= g.n_prev) continue;
            __builtin_nontemporal_store(__builtin_bit_cast(vf, value(r)),
                                        (__attribute__((address_space(1))) vf*)(g.w + (size_t)m * g.n_prev + n));
        }
        return;
    }
    vf old[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int m, n;
        at(r, &m, &n);
        old[r] = *(const __attribute__((address_space(1))) vf*)(
            g.w + (size_t)min(m, g.n_l - 1) * g.n_prev + min(n, g.n_prev - N));
    }
    if (g.lost && *g.lost) return;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int m, n;
        at(r, &m, &n);
        if (m >= g.n_l || n >= g.n_prev) continue;
        const vf v = __builtin_bit_cast(vf, value(r));
        vf o;
#pragma unroll
        for (int c = 0; c < N; ++c) o[c] = fmaf(-sgd_eta, v[c], old[r][c]);
        const size_t off = (size_t)m * g.n_prev + n;
        *(__attribute__((address_space(1))) vf*)(g.w + off) = o;
        if (g.w_bf) {                                  // bfloat16 storage: the weights the next pass multiplies with
            vb ob;
#pragma unroll
            for (int c = 0; c < N; ++c) ob[c] = (__bf16)o[c];
            *(__attribute__((address_space(1))) vb*)(static_cast<__bf16*>(g.w_bf) + off) = ob;
        }
    }
}

// nabla_w of one layer, workgroup x of tile_blocks.  SPLIT: the waves of a workgroup share one tile and its
// contraction; otherwise every wave has a tile of its own (2 x 2 of them a workgroup).
template <typename T, int GT, bool SPLIT>
__device__ __forceinline__ void grad_block(const GradJob& g, int x, int B, float sgd_eta, float* lds) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    v4f acc[GT][GT];
    if constexpr (SPLIT) {
        const int m0 = x / g.tiles_x * 16 * GT, n0 = x % g.tiles_x * 16 * GT;
        contract<T, true, true, GT, GT>(acc, lds, g.D_op, g.d_bytes, g.n_l, m0, g.n_l, g.A_prev, g.a_bytes, g.n_prev, n0,
                                        g.n_prev, B, wave, kWaves);
        reduce_waves<true, true, GT, GT>(acc, lds, [&](int row, int col, v4f s) {
            put_grads<1, 4>(g, sgd_eta, [&](int, int* m, int* n) { *m = m0 + row; *n = n0 + col; }, [&](int) { return s; });
        });
    } else {
        constexpr int wx = kWaves / 2;
        const int m0 = (x / g.tiles_x * 2 + wave / wx) * 16 * GT, n0 = (x % g.tiles_x * wx + wave % wx) * 16 * GT;
        if (m0 >= g.n_l || n0 >= g.n_prev) return;
        contract<T, true, true, GT, GT>(acc, lds, g.D_op, g.d_bytes, g.n_l, m0, g.n_l, g.A_prev, g.a_bytes, g.n_prev, n0,
                                        g.n_prev, B, 0, 1);
        const int lane = threadIdx.x & 63, i = lane & 15, gr = lane >> 4;
        typedef float vg __attribute__((ext_vector_type(GT)));
        put_grads<4 * GT, GT>(
            g, sgd_eta, [&](int r, int* m, int* n) { *m = m0 + GT * (4 * gr + (r & 3)) + (r >> 2); *n = n0 + GT * i; },
            [&](int r) {
                vg v;
#pragma unroll
                for (int nt = 0; nt < GT; ++nt) v[nt] = acc[r >> 2][nt][r & 3];
                return v;
            });
    }
}

// MEET: the chain's tiles are split along the contraction (an instance of its own: the few instructions that this takes cost the
// smallest nets 4 % where they stand beside the whole tiles').
template <typename T, int MT, int NT, int GT, bool GSPLIT, bool MEET>
__global__ __launch_bounds__(64 * kWaves, 2) void k_backward_step(const StepArgs g) {
    extern __shared__ __attribute__((aligned(16))) float lds[];
    int x = blockIdx.x;
    if (x < g.chain_blocks) {
        int tm, tn;                                             // (the splits of a tile follow each other on its XCD)
        tile_of(x, MEET ? g.tiles_m * g.splits : g.tiles_m, g.tiles_n, &tm, &tn);
        if (tn >= g.tiles_n) return;
        const int split = MEET ? tm / g.tiles_m : 0;
        if constexpr (MEET) tm %= g.tiles_m;
        const int m0 = tm * 16 * MT, n0 = tn * 16 * NT;
        v4f acc[MT][NT];
        contract<T, false, true, MT, NT>(acc, lds, g.D_next, g.d_bytes, g.n_next, m0, g.B, g.W_next, g.w_bytes, g.n_l, n0,
                                         g.n_l, g.n_next, split * kWaves + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6),
                                         MEET ? g.splits * kWaves : kWaves);
        auto finish = [&](int row, int col, v4f u) {
            const int m = m0 + row, n = n0 + col;
            if (m >= g.B || n >= g.n_l) return;
            const size_t o = (size_t)m * g.n_l + n;
            typedef T v4t __attribute__((ext_vector_type(4)));
            const v4t av = *reinterpret_cast<const v4t*>(static_cast<const T*>(g.A_l) + o);
            v4f d;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float a = (float)av[c];
                d[c] = u[c] * (a * (1.0f - a));
            }
            *reinterpret_cast<v4f*>(g.D_l + o) = d;
            if constexpr (sizeof(T) == 2) {
                const v4bf db = {(__bf16)d[0], (__bf16)d[1], (__bf16)d[2], (__bf16)d[3]};
                *reinterpret_cast<v4bf*>(static_cast<__bf16*>(g.D_l_bf) + o) = db;
            }
        };
        if constexpr (!MEET) reduce_waves<false, true, MT, NT>(acc, lds, finish);
        else meet<MT, NT>(acc, lds, g.scratch, tn * g.tiles_m + tm, g.splits, split, finish);
        return;
    }
    x -= g.chain_blocks;
    const bool second = x >= g.grad[0].blocks;
    if (second) x -= g.grad[0].blocks;
    const GradJob& j = second ? g.grad[1] : g.grad[0];
    if (x < j.tile_blocks) grad_block<T, GT, GSPLIT>(j, x, g.B, g.sgd_eta, lds);
    else bias_block(j, x - j.tile_blocks, g.B, g.sgd_eta, lds);
}

// The gradients of several layers, none of which depends on another.
struct AllGradArgs {
    struct Layer { const void* D_op; const float* D; const void* A_prev; float* w; float* b; void* w_bf; int n_l, n_prev; };
    Layer layer[kGradLayers];
    int first[kGradLayers + 1];         // workgroups of the layers before
    int layers, B;
    float sgd_eta;
    const unsigned* lost;
};

template <typename T, int GT, bool GSPLIT>
__global__ __launch_bounds__(64 * kWaves, 2) void k_all_gradients(const AllGradArgs g) {
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int lane = threadIdx.x & 63;
    const int at = __builtin_popcountll(__ballot(lane < g.layers && (int)blockIdx.x >= g.first[lane])) - 1;
    const AllGradArgs::Layer& in = g.layer[at];
    GradJob j;
    j.D_op = in.D_op; j.D = in.D; j.A_prev = in.A_prev; j.w = in.w; j.b = in.b; j.w_bf = in.w_bf;
    j.n_l = in.n_l; j.n_prev = in.n_prev; j.lost = g.lost;
    j.d_bytes = (unsigned)(g.B * in.n_l) * (unsigned)sizeof(T);
    j.a_bytes = (unsigned)(g.B * in.n_prev) * (unsigned)sizeof(T);
    constexpr int tm = GSPLIT ? 16 * GT : 2 * 16 * GT, tn = GSPLIT ? 16 * GT : kWaves / 2 * 16 * GT;
    j.tiles_x = ceil_div(in.n_prev, tn);
    j.tile_blocks = j.tiles_x * ceil_div(in.n_l, tm);
    const int x = (int)blockIdx.x - g.first[at];
    if (x < j.tile_blocks) grad_block<T, GT, GSPLIT>(j, x, g.B, g.sgd_eta, lds);
    else bias_block(j, x - j.tile_blocks, g.B, g.sgd_eta, lds);
}

bool fits_buffer(unsigned long long bytes) { return bytes < 0xFFFFFFF0ull; }

// Tile of a chain-side product, in 16 x 16 blocks.  A compute unit works through ceil(tiles / 256) of them; a tile
// costs, per q of the contraction, its 16 (mt + nt) operand rows (measured: as if each took 35 cycles per unit and 16
// rows, the rate the L2s give all compute units together) or its mt nt matrix instructions (32 cycles a unit for fp32,
// 4 for bf16, over four SIMDs), whichever is more.  Forward, us a layer, tiles 1x1, 1x2, 2x2, 2x4, 4x4:
//   fp32: N = 1024, B = 64: 4.4, 5.9, 7.9, 12, 20;  N = 2048, B = 64: 10.2, 9.3, 12.5, 20, 35;  N = 4096, B = 256: 108, 89, 73, 68, 64
//   bf16: N = 2048, B = 128: 9.1, 7.7, 6.3, 7.8, 11;  N = 4096, B = 256: 59, 45, 33, 26, 23
// Rows past the minibatch may be part of a tile where that saves a turn: B = 33 .. 48 beyond N = 8192 takes one turn of
// 4x4 tiles instead of two of 2x4 (bf16, N = 9216, B = 48: forward 65 -> 53, backward 94 -> 86; N = 10240, B = 40: 74 -> 62,
// 111 -> 99; fp32 within 1 % there, N = 16384: 313 -> 281, 573 -> 548).
// A bf16 chain product takes at least two columns a lane (one would be a two-byte load).
struct TileShape { int mt, nt, splits = 1; };

// cycles a unit of the contraction costs a compute unit
long tile_cycles(const TileShape& c, bool bf16) { return std::max(35 * (c.mt + c.nt), (bf16 ? 4 : 32) * c.mt * c.nt); }

TileShape chain_tile(int B, int n_out, bool bf16, bool chain) {
    TileShape best{1, 2};
    long best_cost = 0;
    static const TileShape candidates[] = {{4, 4}, {2, 4}, {2, 2}, {1, 2}, {1, 1}};
    for (const TileShape& c : candidates) {
        if (c.mt == 1 && c.nt == 1 && chain && bf16) continue;
        if (c.mt > 1 && c.mt / 2 >= ceil_div(B, 16)) continue;         // half of its rows would do
        const long tiles = (long)ceil_div(B, 16 * c.mt) * ceil_div(n_out, 16 * c.nt);
        const long cost = (tiles + 255) / 256 * tile_cycles(c, bf16);
        if (best_cost == 0 || cost < best_cost) { best_cost = cost; best = c; }
    }
    return best;
}

// How nabla_w of a layer is cut: 64 x 64 a wave where that gives at least four waves per compute unit; 32 x 32 a wave
// below; and where even those leave SIMDs idle and the minibatch is long enough to divide, 32 x 32 a workgroup whose
// waves share the samples.  Backward, us a layer, 64 / 32 / 32 split: fp32, N = 2048, B = 64: 14.3 / 18.5 / 31; N = 1024,
// B = 64: 11.1 / 8.8 / 10.7; N = 512, B = 128: 14 / 7.3 / 6.2, B = 512: 39 / 17 / 10; bf16, N = 1024, B = 256: 10.9 / 8.4 / 12.
enum GradKind { GRAD_WAVE_64, GRAD_WAVE_32, GRAD_SPLIT_32 };

GradKind grad_kind(int n_l, int n_prev, int B, bool bf16) {
    if ((long)ceil_div(n_l, 64) * ceil_div(n_prev, 64) >= 1024) return GRAD_WAVE_64;
    if ((long)ceil_div(n_l, 32) * ceil_div(n_prev, 32) < 1024 && B > (bf16 ? 96 : 48)) return GRAD_SPLIT_32;
    return GRAD_WAVE_32;
}

// The chain product of a few samples is the reading of W_next, by columns: a tile's workgroup walks a strip of it, 32 nt
// (bf16) or 64 nt (fp32) bytes wide, down all its rows.  Whole tiles alone make too few workgroups to keep memory busy (N =
// 4096, B = 8, bf16: 128 of 64-byte strips, 2.1 TB/s), so their contraction is split over workgroups that meet in memory,
// which costs about 2 us, and the strips become wider.  Backward, us a layer, whole tiles -> split (mt, nt, splits),
// weights in the cache (140 MB of them) | from memory (1.2 GB):
//   bf16  B = 8: N = 1024 7.0 -> 6.6, 1536 8.2 -> 7.4, 2048 10.0 -> 8.0 | 11.8 -> 8.1 (1, 2, 4);  2056 10.7 -> 9.5 | 12.2
//         -> 10.0, 2304 10.3 -> 9.2 | 13.1 -> 10.4 (1, 4, 4);  2560 12.1 -> 10.9 | 15.6 -> 13.2, 3072 14.9 -> 12.8 | 19.8
//         -> 16.1, 4096 18.6 -> 18.4 | 26.9 -> 22.6, 8192 57 -> 57 | 73 -> 66 (1, 4, 2);  four splits there: 10.4 | 12.2,
//         14.0 | 14.5, 20.9 | 22.1; B = 32: N = 1536 8.3 -> 7.6, 2048 10.1 -> 8.6 | 12.5 -> 9.0 (2, 2, 4);  3072 14.2 ->
//         14.3 | 20.0 -> 18.1, 4096 22.2 -> 19.1 | 28.1 -> 24.5, 6144 35 -> 35 | 51 -> 43 (2, 4, 2);  B = 64: N = 3072 15.0
//         -> 14.5 | 21.3 -> 18.0, 4096 23.0 -> 22.7 | 29.6 -> 25.8 (2, 4, 2);  4104 26.3 -> 25.6 | 35.2 -> 32.1, 8192 63 ->
//         62 | 81 -> 74 (4, 4, 2);  B = 40: 8128 72 -> 70 | 86 -> 82, 8192 62 -> 61 | 79 -> 73
//   fp32  B = 8: N = 1024 6.9 -> 6.4, 1536 9.1 -> 8.1 | 10.9 -> 8.4 (1, 2, 4);  2304 11.4 -> 10.8 | 14.8 -> 12.9, 3072 16.9
//         -> 16.2 | 22.5 -> 17.6 (1, 4, 4);  6144 45 -> 44 | 62 -> 57 (1, 4, 2);  B = 32: N = 3072 20.2 -> 21.6 | 26.0 ->
//         23.0, 3584 25.0 -> 24.4 | 31.4 -> 26.4 (2, 4, 4); 4096 30.3 -> 28.2 | 37.2 -> 33.1 (four splits: 31.0 | 34.5),
//         6144 53 -> 53 | 75 -> 66 (2, 4, 2);  B = 64: N = 4096 40.3 -> 36.9 | 50.4 -> 46.4 (2, 4, 2);  4104 44.1 -> 44.4 |
//         56.1 -> 51.2 (4, 4, 2)
// Nothing is gained, or little, below 1024 rows or columns (the meeting: N = 512, 768 20 to 30 % slower), for 17 .. 32
// samples between the ranges below (bf16 N = 2176 -1 | +7 %), and by longer minibatches, which have tiles enough.  fp32, 33
// samples and more: 4 x 4 blocks take the matrix cores as long as two of 2 x 4, and what their strips gain is lost where
// the gradients' matrix instructions beside them set the pace (B = 64, N = 4608: 45.5 -> 49.0 | 59.4 -> 58.5; B = 40: 43.4
// -> 42.5 | 57.6 -> 50.0, 5632 59 -> 61 | 74 -> 74).
TileShape split_shape(int rows, int n_l, bool bf16) {
    if (bf16) {
        if (rows <= 2 && n_l <= 2048) return {rows, 2, 4};
        if (rows == 1) return {1, 4, n_l <= 2304 ? 4 : 2};
        if (rows == 2 && n_l >= 3072) return {2, 4, 2};
        if (rows <= 4 && n_l >= 3072) return n_l <= 4096 ? TileShape{2, 4, 2} : TileShape{4, 4, 2};
    } else {
        if (rows == 1) return n_l <= 1984 ? TileShape{1, 2, 4} : TileShape{1, 4, n_l <= 4096 ? 4 : 2};
        if (rows == 2 && n_l >= 3072) return {2, 4, n_l <= 3584 ? 4 : 2};
        if (rows <= 4 && n_l >= 3072 && n_l <= 4096) return {2, 4, 2};
        if (rows <= 4 && n_l > 4096 && n_l <= (rows == 3 ? 5200 : 4352)) return {4, 4, 2};
    }
    return {0, 0, 1};
}

// Workgroups of a chain product in the grid.
int chain_blocks(const TileShape& t, int B, int n_l) {
    return ceil_div(ceil_div(n_l, 16 * t.nt), 8) * 8 * ceil_div(B, 16 * t.mt) * t.splits;
}

TileShape chain_shape(int B, int n_l, int n_next, bool bf16) {
    const TileShape whole = chain_tile(B, n_l, bf16, true);
    const TileShape t = std::min(n_l, n_next) < 1024 ? TileShape{0, 0, 1} : split_shape(ceil_div(B, 16), n_l, bf16);
    if (t.splits == 1 || ceil_div(B, 16 * t.mt) * ceil_div(n_l, 16 * t.nt) * t.splits > kSplitWorkgroups) return whole;
    if (n_next >= 2 * n_l) return t;
    // A contraction that is short beside the width is not worth the meeting.  us a pair of layers, whole -> split: bf16, B
    // = 64, 1024 rows x 4096 columns 25.4 -> 30.0, 2048 x 4096 37.1 -> 37.5, 3072 x 4096 49.6 -> 47.8;  B = 8, 1024 x 4096
    // 22.0 -> 22.9, 2048 x 4096 33.4 -> 31.7, 2048 x 8192 59.5 -> 59.6, 4096 x 8192 87 -> 84;  fp32, B = 8, 1024 x 4096
    // 28.8 -> 29.3, 2048 x 4096 41.4 -> 40.2.
    if (n_next < n_l && (n_next < 1536 || (B <= 32 ? 2 * n_next < n_l : 3 * n_next < 2 * n_l))) return whole;
    // Beside 32 x 32 gradients (of the layer with these weights) three workgroups are resident on a compute unit, four of
    // the fp32 ones with the fewest registers; where the splits make it more, or one more than whole tiles would, that turn
    // costs more than they bring: bf16, B = 8: N = 1152 (two) 7.2 -> 6.7, 1280 (three, for two) 8.9 -> 9.3 with the descent
    // step, 1536 (three) 8.2 -> 7.4, 1600 (four) 7.9 -> 9.4, 1920 9.6 -> 10.5;  fp32: 1152 6.9 -> 6.7, 1216 6.8 -> 7.6,
    // 1536 9.1 -> 8.1, 1600 9.0 -> 10.6, 1920 10.2 -> 13.5.
    if (grad_kind(n_next, n_l, B, bf16) != GRAD_WAVE_64) {
        const int grads = ceil_div(n_next, 64) * ceil_div(n_l, 64), resident = !bf16 && t.mt == 1 && t.nt == 4 ? 4 : 3;
        const int turns = ceil_div(chain_blocks(t, B, n_l) + grads, 256);
        if (turns > resident || turns > ceil_div(chain_blocks(whole, B, n_l) + grads, 256)) return whole;
    }
    return t;
}
size_t chain_scratch(int B, int n_l, int n_next, bool bf16) {  // floats: arrival counters, then the partial tiles
    const TileShape t = chain_shape(B, n_l, n_next, bf16);
    if (t.splits == 1) return 0;
    return kSplitWorkgroups + (size_t)ceil_div(B, 16 * t.mt) * ceil_div(n_l, 16 * t.nt) * t.splits * (16 * t.mt) * (16 * t.nt);
}

// What the direct kernels take for a layer of a bf16 net in us, for the choice between them and the wide-net kernels
// (gemm_plan, where the measurements are).  Turns of the compute units: `part` of a turn is lost where the last is not full.
double turns(double jobs, int units, double part) {
    if (jobs <= units) return 1.0;
    const double t = jobs / units, whole = (double)(long)t;
    return t > whole ? whole + part + (1.0 - part) * (t - whole) : whole;
}
// A chain-side product: the busiest XCD's tiles over its 32 compute units, a tile's units at the rate of the L2s, or at
// the rate at which memory feeds an XCD's L2 (3 cycles for each 16 operand rows that its 32 tiles of a turn read between
// them: from B = 2048 on every tile brings rows of its own).  With nothing beside it a second turn, once begun, takes
// as long as the first.  (The meeting of a split one is in backward_us's constants.)
double chain_us(int B, int n_out, int K, bool chain) {
    const TileShape t = chain ? chain_shape(B, n_out, K, true) : chain_tile(B, n_out, true, false);
    const int tm = ceil_div(B, 16 * t.mt), tn = ceil_div(n_out, 16 * t.nt);
    const double rows = std::min(tm, 32) * t.mt + std::max(1.0, 32.0 / tm) * t.nt;
    const double cycles = std::max((double)tile_cycles(t, true), 3.0 * rows);
    double n = turns((double)ceil_div(tn, 8) * tm * t.splits, 32, 0.76);
    if (!chain && n > 1.0 && n < 2.0) n = 2.0;
    return n * cycles * ceil_div(K, 32) / t.splits / 2400.0;
}
// (rows that are no whole 128-byte lines cost forward operands a third more, gradients a quarter)
double forward_us(int n_out, int n_in, int B) {
    return 2.8 + 0.915 * chain_us(B, n_out, n_in, false) * (n_in % 64 ? 1.34 : 1.0) + 0.06 * 2e-6 * n_out * n_in;
}
double grad_us(int n_l, int n_prev, int B) {
    const GradKind kind = grad_kind(n_l, n_prev, B, true);
    const int gt = kind == GRAD_WAVE_64 ? 4 : 2;
    const double waves = (double)ceil_div(n_l, 16 * gt) * ceil_div(n_prev, 16 * gt);
    const double units = kind == GRAD_SPLIT_32 ? 2 * ceil_div(B, 64) : ceil_div(B, 32);    // (in pairs where waves share them)
    const double wave = units * 35 * 2 * gt / 2400.0;
    // the stores, twice as long where rows are no whole 64-byte pieces and a layer's gradients exceed 200 MB (the cache does not
    // put the pieces together then: B = 40, N = 8120 109, 8128 72 us a layer)
    const bool pieces = n_prev % 16 && (double)n_l * n_prev > 50e6;
    const double stores = (pieces ? 1.012e-6 : 0.512e-6) * n_l * n_prev;
    return 1.27 * turns(waves, 1024, 0.4) * 4 * wave * (n_prev % 64 ? 1.24 : 1.0) + stores;
}
double backward_us(int n_l, int n_prev, int B, bool chain) {    // gradients of layer l, and the chain step below it
    return 3.08 + grad_us(n_l, n_prev, B) + (chain ? 0.878 * chain_us(B, n_prev, n_l, true) : 0.0);
}

// The same for nets of widths up to 1024, fp32 too, against which the kernels that walk all layers in one launch are set
// (cluster_plan, where the measurements are).  A chain-side product takes as many turns as the busiest XCD's tiles make on its 32
// compute units (whole columns of tiles go to an XCD); a turn is the units of a tile, dearer by `part` where rows are no whole lines,
// and what larger tiles take to start and end.
struct SmallProduct { double turns, tile; };
SmallProduct small_product(int B, int n_out, int K, bool bf16, bool chain, double unit, double part, double block) {
    const TileShape t = chain_tile(B, n_out, bf16, chain);
    const double jobs = (double)ceil_div(ceil_div(n_out, 16 * t.nt), 8) * ceil_div(B, 16 * t.mt);
    const double us = (double)tile_cycles(t, bf16) * ceil_div(K, bf16 ? 32 : 16) / 2400.0;
    const bool lines = (chain ? n_out : K) % (bf16 ? 64 : 32) == 0;
    return {std::max(1.0, jobs / 32), unit * us * (lines ? 1.0 : part) + block * (t.mt + t.nt - 2)};
}
double small_forward_us(int n_out, int n_in, int B, bool bf16) {
    const SmallProduct p = bf16 ? small_product(B, n_out, n_in, bf16, false, 0.62, 1.5, 0.35) : small_product(B, n_out, n_in, bf16, false, 0.886, 1.25, 0.506);
    return (bf16 ? 2.8 : 2.63) + p.tile + (p.turns - 1.0) * (0.35 + (bf16 ? 0.8 : 0.69) * p.tile) + (bf16 ? 1.65e-6 : 3.52e-6) * B * n_out;
}
// The units of the samples that one wave of a gradient tile walks (in pairs), and the waves, in 1024.
struct SmallGrads { double units, waves; };
SmallGrads small_grads(GradKind kind, int n_l, int n_prev, int B, bool bf16) {
    const int edge = kind == GRAD_WAVE_64 ? 64 : 32, q = bf16 ? 32 : 16;
    return {2.0 * ceil_div(B, kind == GRAD_SPLIT_32 ? 2 * kWaves * q : 2 * q),
            (double)ceil_div(n_l, edge) * ceil_div(n_prev, edge) * (kind == GRAD_SPLIT_32 ? kWaves : 1) / 1024.0};
}
double small_backward_us(int n_l, int n_prev, int B, bool bf16, bool chain) {      // as backward_us
    const GradKind kind = grad_kind(n_l, n_prev, B, bf16);
    const SmallGrads g = small_grads(kind, n_l, n_prev, B, bf16);
    const double unit = (bf16 ? 0.222 * g.waves : 0.048 + 0.108 * g.waves) * (kind == GRAD_SPLIT_32 ? (bf16 ? 2.14 : 2.49) : 1.0);
    const double us = (bf16 ? 3.33 : 3.55) + g.units * unit + (bf16 ? 1.63e-6 : 2.9e-6) * n_l * n_prev + (bf16 ? 2.9e-3 : 3.55e-3) * B;
    if (!chain) return us;
    const SmallProduct p = bf16 ? small_product(B, n_prev, n_l, bf16, true, 0.284, 2.47, 0.294) : small_product(B, n_prev, n_l, bf16, true, 0.26, 3.0, 0.12);
    return us + p.tile * (1.0 + (p.turns - 1.0) * (bf16 ? 3.9 : 1.85));
}

template <typename T, int MT, int NT>
hipError_t launch_forward(const ForwardArgs& g, hipStream_t s) {
    k_forward_tile<T, MT, NT><<<ceil_div(g.tiles_n, 8) * 8 * g.tiles_m, 64 * kWaves, lds_bytes(MT + NT, NT), s>>>(g);
    return hipGetLastError();
}

template <typename T>
hipError_t forward_any(ForwardArgs g, TileShape t, hipStream_t s) {
    g.tiles_m = ceil_div(g.B, 16 * t.mt);
    g.tiles_n = ceil_div(g.n_out, 16 * t.nt);
    if (t.mt == 4 && t.nt == 4) return launch_forward<T, 4, 4>(g, s);
    if (t.mt == 2 && t.nt == 4) return launch_forward<T, 2, 4>(g, s);
    if (t.mt == 2 && t.nt == 2) return launch_forward<T, 2, 2>(g, s);
    if (t.mt == 1 && t.nt == 2) return launch_forward<T, 1, 2>(g, s);
    return launch_forward<T, 1, 1>(g, s);
}

template <typename T, int MT, int NT, int GT, bool GSPLIT, bool MEET = false>
hipError_t launch_step(const StepArgs& g, hipStream_t s) {
    k_backward_step<T, MT, NT, GT, GSPLIT, MEET><<<g.chain_blocks + g.grad[0].blocks + g.grad[1].blocks, 64 * kWaves,
                                                   lds_bytes(MT, NT > GT ? NT : GT), s>>>(g);
    return hipGetLastError();
}

template <typename T, int GT, bool GSPLIT>
hipError_t step_any(StepArgs g, TileShape t, hipStream_t s) {
    // The shapes of split_shape.  Gradients whose waves share the samples are fp32 ones of more than 48 samples there,
    // which ride beside a chain step of other widths than their own (the descent step's).
    if constexpr (!GSPLIT || sizeof(T) == 4) {
        if (t.splits > 1 && t.mt == 4) return launch_step<T, 4, 4, GT, GSPLIT, true>(g, s);
        if (t.splits > 1 && t.mt == 2 && t.nt == 4) return launch_step<T, 2, 4, GT, GSPLIT, true>(g, s);
    }
    if constexpr (!GSPLIT) {
        if (t.splits > 1 && t.nt == 4) return launch_step<T, 1, 4, GT, GSPLIT, true>(g, s);
        if constexpr (sizeof(T) == 2)
            if (t.splits > 1 && t.mt == 2) return launch_step<T, 2, 2, GT, GSPLIT, true>(g, s);
        if (t.splits > 1) return launch_step<T, 1, 2, GT, GSPLIT, true>(g, s);
    }
    if (t.splits > 1) return hipErrorInvalidValue;
    if (t.mt == 4 && t.nt == 4) return launch_step<T, 4, 4, GT, GSPLIT>(g, s);
    if (t.mt == 2 && t.nt == 4) return launch_step<T, 2, 4, GT, GSPLIT>(g, s);
    if (t.mt == 2 && t.nt == 2) return launch_step<T, 2, 2, GT, GSPLIT>(g, s);
    if constexpr (sizeof(T) == 4)
        if (t.mt == 1 && t.nt == 1) return launch_step<T, 1, 1, GT, GSPLIT>(g, s);
    return launch_step<T, 1, 2, GT, GSPLIT>(g, s);
}

template <typename T, int GT, bool GSPLIT>
hipError_t launch_gradients_of(AllGradArgs& g, hipStream_t s) {
    const int tm = GSPLIT ? 16 * GT : 2 * 16 * GT, tn = GSPLIT ? 16 * GT : kWaves / 2 * 16 * GT;
    for (int i = 0; i < g.layers; ++i)
        g.first[i + 1] = g.first[i] + ceil_div(g.layer[i].n_prev, tn) * ceil_div(g.layer[i].n_l, tm) + ceil_div(g.layer[i].n_l, 32);
    k_all_gradients<T, GT, GSPLIT><<<g.first[g.layers], 64 * kWaves, lds_bytes(0, GT), s>>>(g);
    return hipGetLastError();
}

}  // namespace
}  // namespace direct

hipError_t launch_all_gradients(const GradStep* grads, int count, int B, bool bf16, float sgd_eta, hipStream_t s) {
    using namespace direct;
    if (count < 1 || count > kGradLayers) return hipErrorInvalidValue;
    AllGradArgs g{};
    g.layers = count;
    g.B = B; g.sgd_eta = sgd_eta; g.lost = grads[0].lost;
    for (int i = 0; i < count; ++i) {
        const GradStep& in = grads[i];
        const unsigned long long es = bf16 ? 2 : 4;
        if (in.kind != grads[0].kind || !fits_buffer(es * B * in.n_l) || !fits_buffer(es * B * in.n_prev)) return hipErrorInvalidValue;
        g.layer[i] = {bf16 ? in.D_bf : static_cast<const void*>(in.D), in.D, in.A_prev, in.w, in.b, in.w_bf, in.n_l, in.n_prev};
    }
    switch (grads[0].kind) {
        case GRAD_WAVE_64: return bf16 ? launch_gradients_of<__bf16, 4, false>(g, s) : launch_gradients_of<float, 4, false>(g, s);
        case GRAD_WAVE_32: return bf16 ? launch_gradients_of<__bf16, 2, false>(g, s) : launch_gradients_of<float, 2, false>(g, s);
        case GRAD_SPLIT_32: return bf16 ? launch_gradients_of<__bf16, 2, true>(g, s) : launch_gradients_of<float, 2, true>(g, s);
        default: return hipErrorInvalidValue;
    }
}

// As grad_kind, for the tiles of all layers.  us a backward pass, 64 / 32 / 32 split, the chain included: fp32, L = 16, N = 512, B =
// 128 74 / 71 / 78;  N = 256, B = 128 43 / 40 / 40;  N = 128, B = 512 59 / 39 / 34;  N = 64, B = 512 53 / 33 / 25;  L = 6, N = 256, B =
// 512 59 / 39 / 35;  bf16, L = 16, N = 512, B = 128 58 / 57 / 71.
int grad_kind_of_all(const int* n, int L, int B, bool bf16) {
    using namespace direct;
    long tiles64 = 0, tiles32 = 0;
    for (int i = 1; i < L; ++i) {
        tiles64 += (long)ceil_div(n[i], 64) * ceil_div(n[i - 1], 64);
        tiles32 += (long)ceil_div(n[i], 32) * ceil_div(n[i - 1], 32);
    }
    return tiles64 >= 1024 ? GRAD_WAVE_64 : tiles32 < 1024 && B > (bf16 ? 96 : 48) ? GRAD_SPLIT_32 : GRAD_WAVE_32;
}

double all_gradients_us(const int* n, int L, int B, bool bf16) {
    using namespace direct;
    const GradKind kind = (GradKind)grad_kind_of_all(n, L, B, bf16);
    double waves = 0.0, entries = 0.0, units = 0.0;
    for (int i = 1; i < L; ++i) {
        const SmallGrads g = small_grads(kind, n[i], n[i - 1], B, bf16);
        units = g.units;
        waves += g.waves;
        entries += (double)n[i] * n[i - 1];
    }
    const double unit = kind == GRAD_SPLIT_32 ? (bf16 ? 1.13 : 0.80) * waves : kind == GRAD_WAVE_64 ? (bf16 ? 1.97 : 0.71) + waves
                                              : (bf16 ? 0.21 + 0.81 * waves : 0.46 + 0.37 * waves);
    return units * unit + (bf16 ? 1.2e-6 : 3.1e-6) * entries + (bf16 ? 5.7e-3 : 5.6e-3) * B;
}

int chain_counters() { return direct::kSplitWorkgroups; }
size_t direct_chain_scratch_floats(int n_l, int n_next, int B, bool bf16) { return direct::chain_scratch(B, n_l, n_next, bf16); }

hipError_t launch_forward_direct(const void* W, const float* bias, const void* A_in, void* A_out, int n_out, int n_in,
                                 int B, bool bf16, hipStream_t s) {
    using namespace direct;
    const unsigned long long es = bf16 ? 2 : 4, ab = es * B * n_in, wb = es * n_out * n_in;
    if (!fits_buffer(ab) || !fits_buffer(wb)) return hipErrorInvalidValue;
    ForwardArgs g{};
    g.A_in = A_in; g.W = W; g.bias = bias; g.A_out = A_out;
    g.a_bytes = (unsigned)ab; g.w_bytes = (unsigned)wb;
    g.B = B; g.n_out = n_out; g.n_in = n_in;
    const TileShape t = chain_tile(B, n_out, bf16, false);
    return bf16 ? forward_any<__bf16>(g, t, s) : forward_any<float>(g, t, s);
}

hipError_t launch_backward_step(const ChainStep* c, const GradStep* grads, int ngrads, int B, bool bf16, float sgd_eta,
                                hipStream_t s) {
    using namespace direct;
    auto kind_of = [&](const GradStep& g) { return g.kind >= 0 ? (GradKind)g.kind : grad_kind(g.n_l, g.n_prev, B, bf16); };
    if (ngrads == 2 && kind_of(grads[0]) != kind_of(grads[1])) {
        const hipError_t e = launch_backward_step(c, grads, 1, B, bf16, sgd_eta, s);
        return e != hipSuccess ? e : launch_backward_step(nullptr, grads + 1, 1, B, bf16, sgd_eta, s);
    }
    const unsigned long long es = bf16 ? 2 : 4;
    StepArgs g{};
    g.B = B; g.sgd_eta = sgd_eta;
    TileShape t{1, 2};
    if (c) {
        const unsigned long long db = es * B * c->n_next, wb = es * c->n_next * c->n_l;
        if (!fits_buffer(db) || !fits_buffer(wb)) return hipErrorInvalidValue;
        t = chain_shape(B, c->n_l, c->n_next, bf16);
        if (t.splits > 1 && !c->scratch) return hipErrorInvalidValue;
        g.D_next = bf16 ? c->D_next_bf : static_cast<const void*>(c->D_next);
        g.W_next = c->W_next; g.A_l = c->A_l; g.D_l = c->D_l; g.D_l_bf = c->D_l_bf;
        g.d_bytes = (unsigned)db; g.w_bytes = (unsigned)wb;
        g.n_l = c->n_l; g.n_next = c->n_next;
        g.tiles_m = ceil_div(B, 16 * t.mt);
        g.tiles_n = ceil_div(c->n_l, 16 * t.nt);
        g.splits = t.splits;
        g.scratch = c->scratch;
        g.chain_blocks = chain_blocks(t, B, c->n_l);
    }
    const GradKind kind = ngrads > 0 ? kind_of(grads[0]) : GRAD_WAVE_32;
    const bool split = kind == GRAD_SPLIT_32;
    const int gt = kind == GRAD_WAVE_64 ? 4 : 2;
    for (int i = 0; i < ngrads; ++i) {
        const GradStep& in = grads[i];
        GradJob& j = g.grad[i];
        const unsigned long long db = es * B * in.n_l, ab = es * B * in.n_prev;
        if (!fits_buffer(db) || !fits_buffer(ab)) return hipErrorInvalidValue;
        j.D_op = bf16 ? in.D_bf : static_cast<const void*>(in.D);
        j.D = in.D; j.A_prev = in.A_prev; j.w = in.w; j.b = in.b; j.w_bf = in.w_bf; j.lost = in.lost;
        j.d_bytes = (unsigned)db; j.a_bytes = (unsigned)ab;
        j.n_l = in.n_l; j.n_prev = in.n_prev;
        const int tm = split ? 16 * gt : 2 * 16 * gt, tn = split ? 16 * gt : kWaves / 2 * 16 * gt;
        j.tiles_x = ceil_div(in.n_prev, tn);
        j.tile_blocks = j.tiles_x * ceil_div(in.n_l, tm);
        j.blocks = j.tile_blocks + ceil_div(in.n_l, 32);
    }
    if (g.chain_blocks + g.grad[0].blocks + g.grad[1].blocks == 0) return hipSuccess;
    switch (kind) {
        case GRAD_WAVE_64: return bf16 ? step_any<__bf16, 4, false>(g, t, s) : step_any<float, 4, false>(g, t, s);
        case GRAD_WAVE_32: return bf16 ? step_any<__bf16, 2, false>(g, t, s) : step_any<float, 2, false>(g, t, s);
        default: return bf16 ? step_any<__bf16, 2, true>(g, t, s) : step_any<float, 2, true>(g, t, s);
    }
}

}  // namespace lf
