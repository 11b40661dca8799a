// Wide bf16 nets: the three per-layer contractions of the pass as LDS-tiled MFMA GEMMs whose workgroups fill a compute
// unit, and the finish of a product that is split along its contraction; and the choice between these kernels and
// those of minibatch_kernels.h, which serve all other minibatch nets.
//
// All three are  C[m][n] = sum_q P(m,q) Q(n,q)  with operands that are either contiguous along the
// contraction index q ("QC": element (i,q) at p[i*ld + q]) or along their own index ("IC": element
// (i,q) at p[q*ld + i]).  forward: P = A_in (QC), Q = W (QC).  chain: P = D_next (QC), Q = W_next (IC).
// grads: P = D (IC), Q = A_prev (IC).  Accumulation is fp32 in the MFMA accumulators, in an order fixed
// by (N, B) alone, so results do not depend on k or on the launch.
#include "lf_internal.h"
#include "cluster_kernels.h"
#include "minibatch_kernels.h"

namespace lf {
namespace {

constexpr int kThreads = 256;
// the default plan (gemm_plan)
constexpr int kSplitTarget = 256, kChainSplitTarget = 128, kStreamGroups = 96, kStreamAlign = 32;

__host__ __device__ constexpr int ceil_div(int a, int b) { return (a + b - 1) / b; }

enum Epilogue { EPI_RAW = 0, EPI_SIGMOID = 1, EPI_SIGMA_PRIME = 2, EPI_GRAD = 3 };

struct GemmArgs {
    const void* P;  int ldp;               // rows of P index m
    const void* Q;  int ldq;               // rows of Q index n
    unsigned p_bytes, q_bytes;             // sizes of the two operand matrices (< 4 GiB each)
    int M, Nn, K;                          // C is M x Nn, contraction length K
    int k_tiles_per_split;                 // split-K: blockIdx.z handles this many BK tiles
    float* raw;                            // EPI_RAW: [splits][M][Nn] fp32
    const float* bias;                     // EPI_SIGMOID: [Nn]
    const void* act;                       // EPI_SIGMA_PRIME: A_l [M][Nn], type T
    void* out;                             // EPI_SIGMOID: T [M][Nn]; EPI_SIGMA_PRIME / EPI_GRAD: float [M][Nn]
    void* out_bf;                          // EPI_SIGMA_PRIME with bf16: bfloat16 copy of out (or null);
                                           // EPI_GRAD with sgd_eta: the bfloat16 weights to rewrite (or null)
    float sgd_eta;                         // EPI_GRAD: != 0 = out holds w^l in fp32 and receives w - eta * C
};

// Operands are addressed as one buffer each: a vector that lies outside the matrix (row past the end, or past the
// contraction length) is given an offset past the end of the buffer and loads zeros.  No branch surrounds a load, so
// the compiler can count the loads in flight.
constexpr unsigned kOutside = 0xFFFFFFF0u;

// MFMA operand (8 consecutive q for row i = lane % 32, starting at q0 + 8 (lane / 32)) from an LDS tile kept
// as [q][i].  ds_read_b64_tr_b16 works on groups of 16 lanes: source lane s supplies the address of four
// consecutive i, result lane r receives element (r % 4) of source lanes r/4, 4 + r/4, 8 + r/4, 12 + r/4.
// With source lane s pointing at row q = s/4, columns 4 (s % 4) .. +3, result lane r holds q = 0..3 at
// column r: four consecutive q of its own row.  Two such loads give the eight values.
typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
__device__ __forceinline__ v8bf lds_operand_transposed(const __bf16* tile, int ld, int i_base, int q0) {
    const int lane = threadIdx.x & 63, s16 = lane & 15;
    const int q = q0 + 8 * (lane >> 5) + (s16 >> 2);
    const int i = i_base + 16 * ((lane >> 4) & 1) + 4 * (s16 & 3);
    typedef __attribute__((address_space(3))) v4s* lds_v4s_ptr;
    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_ptr)(tile + q * ld + i));
    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s_ptr)(tile + (q + 4) * ld + i));
    const v8s both = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(v8bf, both);
}

// ================================================================================================
// bf16, large shapes: 256 x 256 tile, 512 threads
// ================================================================================================
// With 64 x 64 wave tiles one K = 16 step reads 4 KB of LDS per wave for 4 MFMAs (128 cycles): four
// busy SIMDs would need 128 bytes per clock, all the LDS has -- the matrix cores wait for operands half
// of the time.  Here a wave owns 64 x 128 (6 KB per 8 MFMAs: 96 bytes per clock), eight waves (4 x 2)
// share a 256 x 256 tile (128 flops per operand byte fetched, against 64), and LDS is double-buffered:
// tile t is multiplied while tile t+1 goes from registers to the other buffer and tile t+2 is
// requested, with one barrier per tile.  Two waves per SIMD cover each other's waits.
namespace big {
constexpr int kThreadsBig = 512;
constexpr int TM = 256, TN = 256, TK = 64;
constexpr int LDA = TK + 8;                // QC operand in LDS: [i][q]
constexpr int LDI = TM + 32;               // IC operand in LDS: [q][i]
constexpr int ELEMS = TM * LDA > TK * LDI ? TM * LDA : TK * LDI;     // per operand and buffer

// 16-byte pieces of one operand tile, four per thread
template <bool IC> struct StageBig;
template <> struct StageBig<false> {       // [i][q]: 8 threads cover the 64 q of one row
    v4f r[4];
    __device__ void load(__amdgpu_buffer_rsrc_t buf, int ld, int i0, int q0, int I, int Kq, bool live) {
        const int t = threadIdx.x, qv = (t & 7) * 8;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = (t >> 3) + 64 * u;
            const bool ok = live && (i0 + i < I) && (q0 + qv < Kq);
            const unsigned off = ((unsigned)(i0 + i) * (unsigned)ld + (unsigned)(q0 + qv)) * 2u;
            r[u] = buffer_load_v4f(buf, ok ? off : kOutside);
        }
    }
    __device__ void store(__bf16* s) const {
        const int t = threadIdx.x, qv = (t & 7) * 8;
#pragma unroll
        for (int u = 0; u < 4; ++u) *reinterpret_cast<v4f*>(s + ((t >> 3) + 64 * u) * LDA + qv) = r[u];
    }
};
template <> struct StageBig<true> {        // [q][i]: 32 threads cover the 256 i of one q
    v4f r[4];
    __device__ void load(__amdgpu_buffer_rsrc_t buf, int ld, int i0, int q0, int I, int Kq, bool live) {
        const int t = threadIdx.x, iv = (t & 31) * 8;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int q = (t >> 5) * 4 + u;
            const bool ok = live && (q0 + q < Kq) && (i0 + iv < I);
            const unsigned off = ((unsigned)(q0 + q) * (unsigned)ld + (unsigned)(i0 + iv)) * 2u;
            r[u] = buffer_load_v4f(buf, ok ? off : kOutside);
        }
    }
    __device__ void store(__bf16* s) const {
        const int t = threadIdx.x, iv = (t & 31) * 8, q = (t >> 5) * 4;
#pragma unroll
        for (int u = 0; u < 4; ++u) *reinterpret_cast<v4f*>(s + (q + u) * LDI + iv) = r[u];
    }
};

// Issue order of one tile's block, as scheduling groups (mask: 0x008 MFMA, 0x020 memory read, 0x100 LDS
// read, 0x200 LDS write).  A k = 16 step is 8 MFMAs; its operands (6 fragments, one or two LDS reads
// each) are read during the step before; the 8 LDS writes and the 8 requests alternate, two of each per
// step.
template <int R, int I>      // I = 8 * step + index of the MFMA within the step
__device__ __forceinline__ void interleave_from() {
    if constexpr (I < 32) {
        constexpr int step = I / 8, m = I % 8, per = (R + 7) / 8;
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if constexpr (step < 3 && m * per < R) __builtin_amdgcn_sched_group_barrier(0x100, per, 0);
        // a staged vector goes to LDS and its registers are requested again right away: every request
        // then has a whole tile's multiplications to come back
        if constexpr (m % 4 == 1) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
        if constexpr (m % 4 == 3) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        interleave_from<R, I + 1>();
    }
}
template <bool P_IC, bool Q_IC>
__device__ __forceinline__ void interleave() {
    constexpr int R = (P_IC ? 4 : 2) + (Q_IC ? 8 : 4);     // LDS reads per step (6, 10 or 12)
    __builtin_amdgcn_sched_group_barrier(0x100, R, 0);      // operands of step 0
    interleave_from<R, 0>();
}

template <bool P_IC, bool Q_IC, int EPI>
__global__ __launch_bounds__(kThreadsBig) void k_gemm_big(const GemmArgs g) {
    // Two buffers of two operand tiles; afterwards the staging areas of the epilogue.  Four separate arrays:
    // that writes to one buffer and reads of the other cannot touch the same memory is then visible to
    // the compiler, which may interleave them.
    __shared__ __attribute__((aligned(16))) __bf16 s_p0[ELEMS];
    __shared__ __attribute__((aligned(16))) __bf16 s_q0[ELEMS];
    __shared__ __attribute__((aligned(16))) __bf16 s_p1[ELEMS];
    __shared__ __attribute__((aligned(16))) __bf16 s_q1[ELEMS];

    // Which tile column and which split this workgroup takes.  Workgroups are dealt to the 8 XCDs round-robin
    // in x-first order, so with a multiple of 8 tile columns the XCD is x % 8: the split is taken from x (x % S
    // for S = 2, 4 or 8 splits), so that one XCD's workgroups all work in one range of the contraction and its L2
    // fetches only that part of the operand every tile column shares (P); the workgroups of one tile column and
    // split (they share Q's tiles) stay on one XCD, as before.  Only a matter of which workgroup does what.
    int tile_x = blockIdx.x, split = blockIdx.z;
    {
        const int S = gridDim.z;
        if (S > 1 && S <= 8 && (S & (S - 1)) == 0 && gridDim.x % 8 == 0) {
            split = (int)blockIdx.x % S;
            tile_x = (int)blockIdx.x / S + (int)(gridDim.x / S) * (int)blockIdx.z;
        }
    }
    const int m0 = blockIdx.y * TM, n0 = tile_x * TN;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 128;
    const int r32 = lane & 31, half = lane >> 5;

    const int kt_total = ceil_div(g.K, TK);
    const int kt_begin = split * g.k_tiles_per_split;
    const int kt_end = min(kt_total, kt_begin + g.k_tiles_per_split);
    const int T = kt_end - kt_begin;

    v16f acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    StageBig<P_IC> sp;
    StageBig<Q_IC> sq;
    const __amdgpu_buffer_rsrc_t P = make_buffer(g.P, g.p_bytes);
    const __amdgpu_buffer_rsrc_t Q = make_buffer(g.Q, g.q_bytes);
    auto request = [&](int t) {       // tiles past the end load zeros: no branch around a request
        sp.load(P, g.ldp, m0, (kt_begin + t) * TK, g.M, g.K, t < T);
        sq.load(Q, g.ldq, n0, (kt_begin + t) * TK, g.Nn, g.K, t < T);
    };
    auto multiply = [&](const __bf16* tp, const __bf16* tq) {
#pragma unroll
        for (int kk = 0; kk < TK; kk += 16) {
            v8bf a[2], b[4];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                if constexpr (P_IC) a[i] = lds_operand_transposed(tp, LDI, wm + i * 32, kk);
                else a[i] = *reinterpret_cast<const v8bf*>(&tp[(wm + i * 32 + r32) * LDA + kk + half * 8]);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if constexpr (Q_IC) b[j] = lds_operand_transposed(tq, LDI, wn + j * 32, kk);
                else b[j] = *reinterpret_cast<const v8bf*>(&tq[(wn + j * 32 + r32) * LDA + kk + half * 8]);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    };

    // One straight-line block per tile: tile t+1 goes from the registers to the other buffer (last read
    // before the barrier that ended the previous iteration), tile t+2 is requested, tile t is multiplied.
    // The order below is only the data flow; the instructions are interleaved by the groups declared after
    // it, so that the matrix cores run while LDS and memory instructions issue.
    auto tile_block = [&](const __bf16* cur_p, const __bf16* cur_q, __bf16* nxt_p, __bf16* nxt_q, int t) {
        sp.store(nxt_p);
        sq.store(nxt_q);
        request(t + 2);
        multiply(cur_p, cur_q);
        interleave<P_IC, Q_IC>();
        __syncthreads();
    };
    if (T > 0) {
        request(0);
        sp.store(s_p0);
        sq.store(s_q0);
        request(1);
        __syncthreads();
        for (int t = 0; t < T; t += 2) {
            tile_block(s_p0, s_q0, s_p1, s_q1, t);
            if (t + 1 < T) tile_block(s_p1, s_q1, s_p0, s_q0, t + 1);
        }
    }

    // Accumulator element e of lane (r32, half) in tile (i, j) is
    // C[m0 + wm + 32 i + 8 (e/4) + 4 half + e%4][n0 + wn + 32 j + r32].
    // Every epilogue turns the wave's accumulators through a private LDS area (all operand reads are behind
    // the last barrier), so that a lane handles 4 consecutive columns and a wave 2 rows x 512 contiguous
    // bytes per store instruction.  LDS operations of a wave complete in order: no barrier is needed.
    constexpr int LDE = 128 + 4;
    static_assert(2 * 32 * LDE * 4 <= ELEMS * 2, "two waves' staging areas fit one operand buffer");
    __bf16* const area = wave < 2 ? s_p0 : (wave < 4 ? s_q0 : (wave < 6 ? s_p1 : s_q1));
    float* stage = reinterpret_cast<float*>(area) + (wave & 1) * 32 * LDE;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                stage[(8 * (e >> 2) + 4 * half + (e & 3)) * LDE + j * 32 + r32] = acc[i][j][e];
#pragma unroll
        for (int it = 0; it < 16; ++it) {
            const int row = 2 * it + (lane >> 5), c4 = (lane & 31) * 4;
            const v4f v = *reinterpret_cast<const v4f*>(&stage[row * LDE + c4]);
            const int m = m0 + wm + i * 32 + row, n = n0 + wn + c4;
            if (m >= g.M || n >= g.Nn) continue;              // Nn is a multiple of 4
            const size_t o = (size_t)m * g.Nn + n;
            if constexpr (EPI == EPI_GRAD) {
                float* dst = static_cast<float*>(g.out) + o;
                if (g.sgd_eta != 0.0f) {           // the descent step fused in: fp32 master weights stepped in
                    const v4f w = *reinterpret_cast<const v4f*>(dst);     // place, the bfloat16 weights rewritten
                    const v4f s = {fmaf(-g.sgd_eta, v.x, w.x), fmaf(-g.sgd_eta, v.y, w.y),
                                   fmaf(-g.sgd_eta, v.z, w.z), fmaf(-g.sgd_eta, v.w, w.w)};
                    *reinterpret_cast<v4f*>(dst) = s;
                    const v4bf sb = {(__bf16)s.x, (__bf16)s.y, (__bf16)s.z, (__bf16)s.w};
                    *reinterpret_cast<v4bf*>(static_cast<__bf16*>(g.out_bf) + o) = sb;
                } else {
                    store_global_nt_v4f(dst, v);
                }
            } else if constexpr (EPI == EPI_RAW) {
                *reinterpret_cast<v4f*>(g.raw + (size_t)split * g.M * g.Nn + o) = v;
            } else if constexpr (EPI == EPI_SIGMOID) {
                const v4f bs = *reinterpret_cast<const v4f*>(g.bias + n);
                const v4bf a = {(__bf16)sigmoidf(v.x + bs.x), (__bf16)sigmoidf(v.y + bs.y),
                                (__bf16)sigmoidf(v.z + bs.z), (__bf16)sigmoidf(v.w + bs.w)};
                *reinterpret_cast<v4bf*>(static_cast<__bf16*>(g.out) + o) = a;
            } else {
                const v4bf ab = *reinterpret_cast<const v4bf*>(static_cast<const __bf16*>(g.act) + o);
                v4f d;
                v4bf db;
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float a = (float)ab[c];
                    d[c] = v[c] * (a * (1.0f - a));
                    db[c] = (__bf16)d[c];
                }
                *reinterpret_cast<v4f*>(static_cast<float*>(g.out) + o) = d;
                *reinterpret_cast<v4bf*>(static_cast<__bf16*>(g.out_bf) + o) = db;
            }
        }
    }
}

// The gradient product nabla_w = D^T A_prev as one stream of k-tiles over several output tiles.
// Its contraction (the minibatch) is short -- 8 k-tiles at B = 512 -- so a workgroup per output tile spends
// more time starting up (launch, first operands from memory) and storing its 256 KB of fp32 results than
// multiplying.  Here a workgroup is resident for the whole product and walks its tiles: the k-tiles of all of
// them form one stream through the same double-buffered pipeline, so the first operands of the next tile are
// requested, and written to LDS, while the current tile is still being multiplied.  At a tile's end every wave
// stores its accumulators straight to memory (for a fixed accumulator element a half wave holds 32
// consecutive columns of one row: one 128-byte line per row and store instruction; no LDS staging, which
// would collide with the next tile's operands) and goes on multiplying with operands that arrived before
// the stores were issued.
template <int DUMMY>
__global__ __launch_bounds__(kThreadsBig) void k_grad_stream(const GemmArgs g, int tiles_x, int tiles_total) {
    __shared__ __attribute__((aligned(16))) __bf16 s_p0[ELEMS];
    __shared__ __attribute__((aligned(16))) __bf16 s_q0[ELEMS];
    __shared__ __attribute__((aligned(16))) __bf16 s_p1[ELEMS];
    __shared__ __attribute__((aligned(16))) __bf16 s_q1[ELEMS];

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 128;
    const int r32 = lane & 31, half = lane >> 5;
    const int T = ceil_div(g.K, TK);                         // k-tiles per output tile
    // my tiles: blockIdx.x, blockIdx.x + gridDim.x, ...  (with a multiple of 8 tile columns and a grid that is a
    // multiple of 8, all of them lie in tile columns of one residue mod 8: the operands of one XCD's L2)
    const int first = blockIdx.x, stride = gridDim.x;
    const int mine = first < tiles_total ? (tiles_total - first + stride - 1) / stride : 0;

    v16f acc[2][4];
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
    };
    clear();

    StageBig<true> sp, sq;
    const __amdgpu_buffer_rsrc_t P = make_buffer(g.P, g.p_bytes);
    const __amdgpu_buffer_rsrc_t Q = make_buffer(g.Q, g.q_bytes);
    const __amdgpu_buffer_rsrc_t OUT = make_buffer(g.out, (unsigned)((size_t)g.M * g.Nn * 4u));
    // the k-tile the next request fetches: tile number req_tile of mine, k-tile req_kt of it
    int req_tile = 0, req_kt = 0;
    auto request = [&]() {          // past my last tile: loads of zeros, no branch around a request
        const bool live = req_tile < mine;
        const int t = first + req_tile * stride;
        const int m0 = (t / tiles_x) * TM, n0 = (t % tiles_x) * TN;
        sp.load(P, g.ldp, m0, req_kt * TK, g.M, g.K, live);
        sq.load(Q, g.ldq, n0, req_kt * TK, g.Nn, g.K, live);
        if (++req_kt == T) { req_kt = 0; ++req_tile; }
    };
    auto multiply = [&](const __bf16* tp, const __bf16* tq) {
#pragma unroll
        for (int kk = 0; kk < TK; kk += 16) {
            v8bf a[2], b[4];
#pragma unroll
            for (int i = 0; i < 2; ++i) a[i] = lds_operand_transposed(tp, LDI, wm + i * 32, kk);
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = lds_operand_transposed(tq, LDI, wn + j * 32, kk);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    };
    // Accumulator element e of lane (r32, half) in tile (i, j) is
    // C[m0 + wm + 32 i + 8 (e/4) + 4 half + e%4][n0 + wn + 32 j + r32].  The whole byte offset of a store goes
    // into the bounds-checked vector offset (a scalar offset would not be checked): a row past the end of the
    // matrix then lies outside the buffer (no store; the launcher guarantees the sum cannot wrap), a column
    // past the end is given an offset outside it.
    auto store_tile = [&](int tile_no) {
        const int t = first + tile_no * stride;
        const int m0 = (t / tiles_x) * TM, n0 = (t % tiles_x) * TN;
        const int n = n0 + wn + r32;
        const unsigned lane_off = ((unsigned)(m0 + wm + 4 * half) * (unsigned)g.Nn + (unsigned)n) * 4u;
        const unsigned row_bytes = (unsigned)g.Nn * 4u;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool col_ok = n + 32 * j < g.Nn;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const unsigned off = lane_off + 128u * j + (unsigned)(32 * i + 8 * (e >> 2) + (e & 3)) * row_bytes;
                    const float v = acc[i][j][e];      // (a copy: a bit cast of the vector element itself reads element 0)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), OUT, col_ok ? off : kOutside, 0, 2);
                }
            }
    };
    int kt_in_tile = 0, tile_no = 0;
    auto tile_block = [&](const __bf16* cur_p, const __bf16* cur_q, __bf16* nxt_p, __bf16* nxt_q) {
        sp.store(nxt_p);
        sq.store(nxt_q);
        request();
        multiply(cur_p, cur_q);
        interleave<true, true>();
        __syncthreads();
        if (++kt_in_tile == T) {
            store_tile(tile_no);
            clear();
            kt_in_tile = 0;
            ++tile_no;
        }
    };
    if (mine > 0) {
        request();
        sp.store(s_p0);
        sq.store(s_q0);
        request();
        __syncthreads();
        const int total = mine * T;
        for (int it = 0; it < total; it += 2) {
            tile_block(s_p0, s_q0, s_p1, s_q1);
            if (it + 1 < total) tile_block(s_p1, s_q1, s_p0, s_q0);
        }
    }
}

static_assert(2 * 2 * ELEMS * 2 <= 160 * 1024, "LDS of one compute unit");
}  // namespace big

// ================================================================================================
// bf16, large shapes: 128 x 256 tile, 256 threads, two workgroups per compute unit
// ================================================================================================
// The leapfrog schedule runs the chain product of one layer beside the gradient products of the layers
// above it.  The two are complementary -- the chain product is bound by the matrix cores, the gradient
// product by its N x N fp32 store stream -- but kernels whose workgroups fill a compute unit (the
// 256 x 256 kernel above: 512 threads, 147 KB of LDS) cannot share one: they take turns.  This kernel is
// sized for half a compute unit (256 threads, 60 KB of LDS, 256 registers), so that a workgroup of the
// chain product and one of a gradient product -- or two of one product in different phases -- are
// resident together: one multiplies while the other stores, loads or waits at a barrier.
// Same wave tile (64 x 128: 8 matrix instructions per 6 operand fragments), 2 x 2 waves, k-tiles of 32,
// LDS double-buffered, one barrier per k-tile; tile t is multiplied while tile t+1 goes from registers to
// the other buffer and tile t+2 is requested.  The epilogues store straight from the accumulators: for a
// fixed accumulator element the 32 lanes of a half wave hold 32 consecutive columns of one row, a whole
// 128-byte line of fp32 output.
namespace half {
constexpr int kThreadsHalf = 256;
constexpr int TM = 128, TN = 256, TK = 32;
constexpr int LDA = TK + 8;                // QC operand in LDS: [i][q]; 80-byte rows: 16 lanes' 16-byte reads
                                           // fall on 16 different bank groups
constexpr int LDI_P = TM + 32;             // IC operand in LDS: [q][i], rows 16 banks past a multiple of 64
constexpr int LDI_Q = TN + 32;
constexpr int P_ELEMS = TM * LDA > TK * LDI_P ? TM * LDA : TK * LDI_P;
constexpr int Q_ELEMS = TN * LDA > TK * LDI_Q ? TN * LDA : TK * LDI_Q;

// 16-byte pieces of one operand tile of I rows (of its own index), I / 64 per thread
template <int I, bool IC> struct StageHalf;
template <int I> struct StageHalf<I, false> {     // [i][q]: 4 threads cover the 32 q of one row
    v4f r[I / 64];
    __device__ void load(__amdgpu_buffer_rsrc_t buf, int ld, int i0, int q0, int Imax, int Kq, bool live) {
        const int t = threadIdx.x, qv = (t & 3) * 8;
#pragma unroll
        for (int u = 0; u < I / 64; ++u) {
            const int i = (t >> 2) + 64 * u;
            const bool ok = live && (i0 + i < Imax) && (q0 + qv < Kq);
            const unsigned off = ((unsigned)(i0 + i) * (unsigned)ld + (unsigned)(q0 + qv)) * 2u;
            r[u] = buffer_load_v4f(buf, ok ? off : kOutside);
        }
    }
    __device__ void store(__bf16* s) const {
        const int t = threadIdx.x, qv = (t & 3) * 8;
#pragma unroll
        for (int u = 0; u < I / 64; ++u) *reinterpret_cast<v4f*>(s + ((t >> 2) + 64 * u) * LDA + qv) = r[u];
    }
};
template <int I> struct StageHalf<I, true> {      // [q][i]: I / 8 threads cover the I entries of one q
    static constexpr int TPQ = I / 8, QPP = kThreadsHalf / TPQ, LDI = I + 32;
    v4f r[I / 64];
    __device__ void load(__amdgpu_buffer_rsrc_t buf, int ld, int i0, int q0, int Imax, int Kq, bool live) {
        const int t = threadIdx.x, iv = (t % TPQ) * 8;
#pragma unroll
        for (int u = 0; u < I / 64; ++u) {
            const int q = t / TPQ + QPP * u;
            const bool ok = live && (q0 + q < Kq) && (i0 + iv < Imax);
            const unsigned off = ((unsigned)(q0 + q) * (unsigned)ld + (unsigned)(i0 + iv)) * 2u;
            r[u] = buffer_load_v4f(buf, ok ? off : kOutside);
        }
    }
    __device__ void store(__bf16* s) const {
        const int t = threadIdx.x, iv = (t % TPQ) * 8;
#pragma unroll
        for (int u = 0; u < I / 64; ++u) *reinterpret_cast<v4f*>(s + (t / TPQ + QPP * u) * LDI + iv) = r[u];
    }
};

// Issue order of one k-tile's block (see big::interleave_from): 16 matrix instructions in two k = 16 steps;
// the second step's operands are read from LDS during the first; each of the six staged vectors is written
// to LDS and requested again back to back, one LDS write or one request after every matrix instruction.
template <int R, int I>
__device__ __forceinline__ void interleave_from() {
    if constexpr (I < 16) {
        constexpr int step = I / 8, m = I % 8, per = (R + 7) / 8;
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        if constexpr (step < 1 && m * per < R) __builtin_amdgcn_sched_group_barrier(0x100, per, 0);
        if constexpr (I >= 1 && I <= 12 && I % 2 == 1) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
        if constexpr (I >= 1 && I <= 12 && I % 2 == 0) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        interleave_from<R, I + 1>();
    }
}
template <bool P_IC, bool Q_IC>
__device__ __forceinline__ void interleave() {
    constexpr int R = (P_IC ? 4 : 2) + (Q_IC ? 8 : 4);
    __builtin_amdgcn_sched_group_barrier(0x100, R, 0);
    interleave_from<R, 0>();
}

template <bool P_IC, bool Q_IC, int EPI>
__global__ __launch_bounds__(kThreadsHalf, 2) void k_gemm_half(const GemmArgs g) {
    __shared__ __attribute__((aligned(16))) __bf16 s_p0[P_ELEMS];
    __shared__ __attribute__((aligned(16))) __bf16 s_q0[Q_ELEMS];
    __shared__ __attribute__((aligned(16))) __bf16 s_p1[P_ELEMS];
    __shared__ __attribute__((aligned(16))) __bf16 s_q1[Q_ELEMS];

    // (Workgroups are dealt to the 8 XCDs, each with an L2 of its own, round-robin by linear index, x fastest.
    // With a multiple of 8 tile columns an XCD therefore owns every 8th tile column and walks it row by row:
    // the workgroups resident on it together share a few operand tiles of either kind, which its L2 holds.)
    const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TN;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = (wave >> 1) * 64, wn = (wave & 1) * 128;
    const int r32 = lane & 31, half = lane >> 5;

    const int kt_total = ceil_div(g.K, TK);
    const int kt_begin = blockIdx.z * g.k_tiles_per_split;
    const int kt_end = min(kt_total, kt_begin + g.k_tiles_per_split);
    const int T = kt_end - kt_begin;

    v16f acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

    StageHalf<TM, P_IC> sp;
    StageHalf<TN, Q_IC> sq;
    const __amdgpu_buffer_rsrc_t P = make_buffer(g.P, g.p_bytes);
    const __amdgpu_buffer_rsrc_t Q = make_buffer(g.Q, g.q_bytes);
    auto request = [&](int t) {       // tiles past the end load zeros: no branch around a request
        sp.load(P, g.ldp, m0, (kt_begin + t) * TK, g.M, g.K, t < T);
        sq.load(Q, g.ldq, n0, (kt_begin + t) * TK, g.Nn, g.K, t < T);
    };
    auto multiply = [&](const __bf16* tp, const __bf16* tq) {
#pragma unroll
        for (int kk = 0; kk < TK; kk += 16) {
            v8bf a[2], b[4];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                if constexpr (P_IC) a[i] = lds_operand_transposed(tp, LDI_P, wm + i * 32, kk);
                else a[i] = *reinterpret_cast<const v8bf*>(&tp[(wm + i * 32 + r32) * LDA + kk + half * 8]);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if constexpr (Q_IC) b[j] = lds_operand_transposed(tq, LDI_Q, wn + j * 32, kk);
                else b[j] = *reinterpret_cast<const v8bf*>(&tq[(wn + j * 32 + r32) * LDA + kk + half * 8]);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    };
    auto tile_block = [&](const __bf16* cur_p, const __bf16* cur_q, __bf16* nxt_p, __bf16* nxt_q, int t) {
        sp.store(nxt_p);
        sq.store(nxt_q);
        request(t + 2);
        multiply(cur_p, cur_q);
        interleave<P_IC, Q_IC>();
        __syncthreads();
    };
    if (T > 0) {
        request(0);
        sp.store(s_p0);
        sq.store(s_q0);
        request(1);
        __syncthreads();
        for (int t = 0; t < T; t += 2) {
            tile_block(s_p0, s_q0, s_p1, s_q1, t);
            if (t + 1 < T) tile_block(s_p1, s_q1, s_p0, s_q0, t + 1);
        }
    }

    // Accumulator element e of lane (r32, half) in tile (i, j) is
    // C[m0 + wm + 32 i + 8 (e/4) + 4 half + e%4][n0 + wn + 32 j + r32]: for a fixed e a half wave holds 32
    // consecutive columns of one row, so every store instruction writes two whole 128-byte lines of fp32.
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int n = n0 + wn + j * 32 + r32;
            if (n >= g.Nn) continue;
            float bias = 0.0f;
            if constexpr (EPI == EPI_SIGMOID) bias = g.bias[n];
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int m = m0 + wm + i * 32 + 8 * (e >> 2) + 4 * half + (e & 3);
                if (m >= g.M) continue;
                const size_t o = (size_t)m * g.Nn + n;
                const float v = acc[i][j][e];
                if constexpr (EPI == EPI_GRAD) {
                    float* dst = static_cast<float*>(g.out) + o;
                    if (g.sgd_eta != 0.0f) {       // the descent step fused in: fp32 master weights stepped in
                        const float w = fmaf(-g.sgd_eta, v, *dst);       // place, the bfloat16 weights rewritten
                        *dst = w;
                        static_cast<__bf16*>(g.out_bf)[o] = (__bf16)w;
                    } else {
                        __builtin_nontemporal_store(v, (__attribute__((address_space(1))) float*)dst);
                    }
                } else if constexpr (EPI == EPI_RAW) {
                    g.raw[(size_t)blockIdx.z * g.M * g.Nn + o] = v;
                } else if constexpr (EPI == EPI_SIGMOID) {
                    static_cast<__bf16*>(g.out)[o] = (__bf16)sigmoidf(v + bias);
                } else {
                    const float a = (float)static_cast<const __bf16*>(g.act)[o];
                    const float d = v * (a * (1.0f - a));
                    static_cast<float*>(g.out)[o] = d;
                    static_cast<__bf16*>(g.out_bf)[o] = (__bf16)d;
                }
            }
        }
}

static_assert(2 * (P_ELEMS + Q_ELEMS) * 2 <= 80 * 1024, "two workgroups' LDS fit one compute unit");
}  // namespace half

// Split-K second stage: sum the raw partials in split order, then the layer's epilogue.  A thread takes four
// consecutive outputs (one row: every width is a multiple of 8), 16 bytes per load.
template <int EPI>
__global__ __launch_bounds__(kThreads) void k_split_finish(const float* __restrict__ raw, int splits, size_t count,
                                                           int Nn, const float* __restrict__ bias,
                                                           const __bf16* __restrict__ act, void* out, __bf16* out_bf) {
    const size_t o = ((size_t)blockIdx.x * kThreads + threadIdx.x) * 4;
    if (o >= count) return;
    v4f v = *reinterpret_cast<const v4f*>(raw + o);
    for (int z = 1; z < splits; ++z) v += *reinterpret_cast<const v4f*>(raw + (size_t)z * count + o);
    if constexpr (EPI == EPI_SIGMOID) {
        const v4f bs = *reinterpret_cast<const v4f*>(bias + o % Nn);
        const v4bf r = {(__bf16)sigmoidf(v[0] + bs[0]), (__bf16)sigmoidf(v[1] + bs[1]), (__bf16)sigmoidf(v[2] + bs[2]),
                        (__bf16)sigmoidf(v[3] + bs[3])};
        *reinterpret_cast<v4bf*>(static_cast<__bf16*>(out) + o) = r;
    } else {
        const v4bf av = *reinterpret_cast<const v4bf*>(act + o);
        v4f d;
        v4bf db;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float a = (float)av[c];
            d[c] = v[c] * (a * (1.0f - a));
            db[c] = (__bf16)d[c];
        }
        *reinterpret_cast<v4f*>(static_cast<float*>(out) + o) = d;
        *reinterpret_cast<v4bf*>(out_bf + o) = db;
    }
}

// eq. (bp3) for a minibatch: nabla_b[j] = sum_b D[b][j].  A workgroup owns 32 columns; its 8 row groups
// each add every 8th sample in ascending order, then the 8 partial sums are added in group order.
// sgd_eta != 0: nabla_b is b^l itself and receives b - eta * sum.
__global__ __launch_bounds__(kThreads) void k_bias_grad(const float* __restrict__ D, float* nabla_b, int N,
                                                        int B, float sgd_eta) {
    __shared__ float s_part[8][32];
    const int c = threadIdx.x & 31, rg = threadIdx.x >> 5;
    const int j = blockIdx.x * 32 + c;
    float s = 0.0f;
    if (j < N) {
        // eight rows requested at a time, added in ascending order
        int b = rg;
        for (; b + 56 < B; b += 64) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = D[(size_t)(b + 8 * u) * N + j];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += v[u];
        }
        for (; b < B; b += 8) s += D[(size_t)b * N + j];
    }
    s_part[rg][c] = s;
    __syncthreads();
    if (rg == 0 && j < N) {
        float t = s_part[0][c];
#pragma unroll
        for (int q = 1; q < 8; ++q) t += s_part[q][c];
        nabla_b[j] = sgd_eta != 0.0f ? fmaf(-sgd_eta, t, nabla_b[j]) : t;
    }
}

template <bool P_IC, bool Q_IC, int EPI>
hipError_t run_big(GemmArgs g, int splits, hipStream_t s) {
    const unsigned long long pb = (unsigned long long)(P_IC ? g.K : g.M) * g.ldp * 2ull;
    const unsigned long long qb = (unsigned long long)(Q_IC ? g.K : g.Nn) * g.ldq * 2ull;
    if (pb >= 0xFFFFFFF0ull || qb >= 0xFFFFFFF0ull) return hipErrorInvalidValue;
    g.p_bytes = (unsigned)pb;
    g.q_bytes = (unsigned)qb;
    const dim3 grid(ceil_div(g.Nn, big::TN), ceil_div(g.M, big::TM), splits);
    big::k_gemm_big<P_IC, Q_IC, EPI><<<grid, big::kThreadsBig, 0, s>>>(g);
    return hipGetLastError();
}

// The streamed gradient product (big::k_grad_stream): `groups` resident workgroups walk all output tiles.
hipError_t run_grad_stream(GemmArgs g, int groups, hipStream_t s) {
    const unsigned long long pb = (unsigned long long)g.K * g.ldp * 2ull, qb = (unsigned long long)g.K * g.ldq * 2ull;
    // (the result is addressed with 32-bit offsets that may point up to one tile of rows past its end)
    const unsigned long long ob = (unsigned long long)(g.M + big::TM) * g.Nn * 4ull;
    if (pb >= 0xFFFFFFF0ull || qb >= 0xFFFFFFF0ull || ob >= 0xFFFFFFF0ull) return hipErrorInvalidValue;
    g.p_bytes = (unsigned)pb;
    g.q_bytes = (unsigned)qb;
    const int tiles_x = ceil_div(g.Nn, big::TN), tiles = tiles_x * ceil_div(g.M, big::TM);
    big::k_grad_stream<0><<<groups < tiles ? groups : tiles, big::kThreadsBig, 0, s>>>(g, tiles_x, tiles);
    return hipGetLastError();
}

template <bool P_IC, bool Q_IC, int EPI>
hipError_t run_half(GemmArgs g, int splits, hipStream_t s) {
    const unsigned long long pb = (unsigned long long)(P_IC ? g.K : g.M) * g.ldp * 2ull;
    const unsigned long long qb = (unsigned long long)(Q_IC ? g.K : g.Nn) * g.ldq * 2ull;
    if (pb >= 0xFFFFFFF0ull || qb >= 0xFFFFFFF0ull) return hipErrorInvalidValue;
    g.p_bytes = (unsigned)pb;
    g.q_bytes = (unsigned)qb;
    const dim3 grid(ceil_div(g.Nn, half::TN), ceil_div(g.M, half::TM), splits);
    half::k_gemm_half<P_IC, Q_IC, EPI><<<grid, half::kThreadsHalf, 0, s>>>(g);
    return hipGetLastError();
}

}  // namespace

static int chain_splits(int n_out, int K, int B, int kernel, int target) {
    const bool half_tile = kernel == GEMM_HALF;
    const int tiles = half_tile ? ceil_div(n_out, half::TN) * ceil_div(B, half::TM)
                                : ceil_div(n_out, big::TN) * ceil_div(B, big::TM);
    const int kt = ceil_div(K, half_tile ? half::TK : big::TK), least = half_tile ? 8 : 4;
    int s = 1;
    while (tiles * s < target && s < 16 && kt / (s * 2) >= least) s *= 2;
    return s;
}

// What the wide-net kernels take for a layer, as direct::forward_us and backward_us.  Forward: turns of 256 compute
// units, a k-tile at a time, and the split's second pass over its partial sums.  Backward: the chain and the workers'
// streams side by side have a floor of 22 us a layer, to which come the partial sums, the turns of 96 resident
// workgroups through the samples, and the gradient stores.
static double wide_forward_us(int n_out, int n_in, int B) {
    const int s = chain_splits(n_out, n_in, B, GEMM_BIG, kSplitTarget);
    const double groups = (double)s * ceil_div(n_out, big::TN) * ceil_div(B, big::TM);
    return 8.3 + 1.09 * direct::turns(groups, 256, 0.9) * ceil_div(ceil_div(n_in, big::TK), s) * (n_in % 64 ? 1.12 : 1.0) +
           (s > 1 ? 0.352 * 4e-6 * s * B * n_out : 0.0) + 0.074 * 2e-6 * n_out * n_in;
}
static double wide_backward_us(int n_l, int n_prev, int B, bool chain) {
    const int s = chain ? chain_splits(n_prev, n_l, B, GEMM_BIG, kChainSplitTarget) : 1;
    const double tiles = (double)ceil_div(n_l, big::TM) * ceil_div(n_prev, big::TN);
    return 22.0 + (s > 1 ? 0.155 * 4e-6 * s * B * n_prev : 0.0) +
           0.706 * direct::turns(tiles, kStreamGroups, 1.0) * ceil_div(B, big::TK) +
           0.643e-6 * n_l * n_prev * (n_prev % kStreamAlign ? 1.31 : 1.0) + 0.54 * 2e-6 * B * n_prev;
}

// Which kernels a minibatch net takes, decided once per net from its widths n[0 .. L-1] and its storage type.
// The direct kernels (minibatch_kernels.h) serve every fp32 net; a bf16 net takes them or the kernels of this file, by
// default with 256 x 256 tiles for all three products (measured faster than 128 x 256 ones, alone and beside each other).
// The direct kernels read every operand once per 64 x 64 outputs at most, the wide ones once per 256 x 256: with many
// outputs or a long contraction that traffic decides; with few the wide kernels' second pass, their events and their
// whole tiles of 256 samples do.  Neither N nor B nor a number of tiles alone says which is faster, because turns of the
// chip are whole numbers: the two estimates above are compared, summed over the layers, forward and backward each for
// itself.  The forward constants are fitted to 230 uniform nets, N = 256 .. 16384, B = 1 .. 32768, L = 6 .. 8, the backward ones
// to 856, N = 512 .. 16384, B = 2 .. 2048, L = 6, 8 and 16.  On the latter the choice is within 4 % of the faster kernels
// for 97 % backward, 94 % forward; the worst are L = 16, N = 5120, B = 128 backward (28 %: its weights come from memory, which
// the estimates do not know of) and N = 8120, B = 128 forward (39 %: rows of no whole lines).  us a layer, direct / wide,
// k = 4:
//   forward   N = 2048: B = 1024 17 / 31, 2048 39 / 37, 4096 80 / 52;  N = 3072: B = 1024 33 / 55, 2048 85 / 71;
//             N = 4096: B = 256 17 / 38, 512 28 / 38, 1024 59 / 50, 4096 293 / 120;  N = 5120: B = 256 41 / 52, 768 73 / 75, 2048 230 / 139;
//             N = 6144: B = 128 36 / 42, 256 50 / 58, 640 85 / 85;  N = 8192: B = 64 37 / 38, 256 66 / 56, 512 108 / 79
//   backward  N = 1536: B = 768 31 / 35, 2048 75 / 57;  N = 2048: B = 1024 34 / 44, 2048 72 / 63;  N = 3072: B = 512 42 / 46, 768 60 / 52;
//             N = 4096: B = 256 40 / 47, 512 65 / 57, 4096 537 / 249;  N = 5120: B = 128 38 / 45, 256 63 / 53;
//             N = 6144: B = 64 45 / 51, 128 63 / 56, 512 146 / 103;  N = 7168: B = 96 69 / 73;  N = 8192: B = 64 71 / 80, 128 103 / 85, 512 256 / 146
// The streamed gradient product stores single columns, 32 neighbouring ones of a row at a time: where rows of nabla_w are
// no whole 128-byte lines (n_prev not a multiple of 32) every store is two partial lines, and the layer takes the
// kernel with a workgroup per tile, whose epilogue stores 512 bytes of a row at a time.  Backward, us a layer, streamed /
// per tile: N = 4360, B = 200 58 / 49; N = 5384, B = 300 85 / 73; N = 7000, B = 150 122 / 93; N = 8120, B = 500 181 / 163.
// How a wide net shares the chip between the chain and the workers: a kernel of either kind fills every compute
// unit it gets (registers, LDS), so two of them never share one; what can be shared is the set of compute
// units.  The chain product is split only two ways along K -- 128 workgroups, half the chip (and half the
// split's partial-sum traffic) -- the streamed gradient product keeps 96 workgroups resident, and the k workers
// run on two streams (worker j on stream j mod 2), so that at most two gradient products are in flight and the
// next chain kernel always finds compute units.  Measured at L = 48, N = 8192, B = 512, k = 8: 7.0 ms per backward
// pass against 8.0 ms with every kernel spread over the whole chip.  (The split does not depend on k: the
// gradients must be the same bits for every k.  A sequential pass, k = 1, would be faster with four splits.)
// Overrides for tests and A/B runs, read when the plan is made:
// LF_GEMM_BIG=0/1 forces the direct / wide-net kernels (also where a small net would take those of cluster_kernels.h); LF_GEMM_CHAIN_TILE = "big" or "half" picks the wide-net
// kernel of the forward and chain products, LF_GEMM_GRAD_TILE = "stream", "big" or "half" that of the gradient
// product of every layer; LF_GEMM_SPLIT_TARGET = workgroups the split of a chain-side product aims at (both products),
// LF_GEMM_CHAIN_SPLIT_TARGET = the same for the backward chain product alone; LF_GEMM_STREAM_GROUPS = resident
// workgroups of the streamed gradient product, which every layer then takes; LF_WORKER_STREAMS (read by the schedule) =
// streams the workers share.
GemmPlan gemm_plan(const int* n, int L, int B, bool bf16) {
    GemmPlan p{GEMM_DIRECT, GEMM_DIRECT, GEMM_DIRECT, kSplitTarget, kChainSplitTarget, kStreamGroups, kStreamAlign, 1};
    double fwd = 0.0, wide_fwd = 0.0, bwd = 0.0, wide_bwd = 0.0;
    for (int l = 2; bf16 && l <= L; ++l) {
        const int n_l = n[l - 1], n_prev = n[l - 2];
        fwd += direct::forward_us(n_l, n_prev, B);
        wide_fwd += wide_forward_us(n_l, n_prev, B);
        bwd += direct::backward_us(n_l, n_prev, B, l > 2);
        wide_bwd += wide_backward_us(n_l, n_prev, B, l > 2);
    }
    bool wide_forward = wide_fwd < fwd, wide_backward = wide_bwd < bwd;
    if (const char* e = getenv("LF_GEMM_BIG")) {
        if (e[0] == '0') wide_forward = wide_backward = false;
        if (e[0] == '1') wide_forward = wide_backward = bf16;
    }
    int tile = GEMM_BIG;
    if (const char* e = getenv("LF_GEMM_CHAIN_TILE")) tile = e[0] == 'b' ? GEMM_BIG : GEMM_HALF;
    if (wide_forward) p.forward = tile;
    if (wide_backward) {
        p.chain = tile;
        p.grad = GEMM_STREAM;
        p.worker_streams = 2;
        if (const char* e = getenv("LF_GEMM_GRAD_TILE")) {
            p.grad = e[0] == 'b' ? GEMM_BIG : (e[0] == 's' ? GEMM_STREAM : GEMM_HALF);
            p.stream_align = 1;
        }
    }
    if (const char* e = getenv("LF_GEMM_STREAM_GROUPS")) {
        const int t = atoi(e);
        if (t >= 8 && t <= 1024) { p.stream_groups = t; p.stream_align = 1; }
    }
    if (const char* e = getenv("LF_GEMM_SPLIT_TARGET")) {
        const int t = atoi(e);
        if (t >= 64 && t <= 2048) p.split_target = p.chain_split_target = t;
    }
    if (const char* e = getenv("LF_GEMM_CHAIN_SPLIT_TARGET")) {
        const int t = atoi(e);
        if (t >= 64 && t <= 2048) p.chain_split_target = t;
    }
    return p;
}

double layer_launches_us(const int* n, int L, int B, bool bf16, bool backward) {
    const GemmPlan plan = gemm_plan(n, L, B, bf16);
    const bool wide = (backward ? plan.chain : plan.forward) != GEMM_DIRECT;
    double us = backward ? 1.8 : 0.0;
    for (int l = 2; l <= L; ++l) {
        const int n_l = n[l - 1], n_prev = n[l - 2];
        if (wide) us += backward ? wide_backward_us(n_l, n_prev, B, l > 2) : wide_forward_us(n_l, n_prev, B);
        else us += backward ? direct::small_backward_us(n_l, n_prev, B, bf16, l > 2) : direct::small_forward_us(n_l, n_prev, B, bf16);
    }
    return backward ? us : std::max(us, 3.0 + 2.5 * (L - 1));      // (2.5: what the host takes to launch one)
}

size_t split_workspace_floats(int n_out, int B, bool bf16) {             // enough for any plan
    return bf16 ? (size_t)16 * B * n_out : 0;                            // no plan splits more than 16 ways
}

size_t noalloc_scratch_floats(const int* n, int L, int B, bool bf16, const GemmPlan& plan) {
    size_t used = 0, tiles_128 = 0, tiles_256 = 0;
    auto add = [&](size_t& most, int splits, int n_out) {
        if (splits > 1) most = std::max(most, (size_t)splits * B * n_out);
    };
    for (int l = 2; l < L; ++l) {
        const int n_out = n[l - 1], K = n[l];
        if (plan.chain != GEMM_DIRECT) add(used, chain_splits(n_out, K, B, plan.chain, plan.chain_split_target), n_out);
        add(tiles_256, chain_splits(n_out, K, B, GEMM_BIG, 128), n_out);
        const int tiles = ceil_div(n_out, 128) * ceil_div(B, 128), kt = ceil_div(K, bf16 ? 64 : 32);
        int s = 1;
        while (tiles * s < 512 && s < 16 && kt / (s * 2) >= 4) s *= 2;
        add(tiles_128, s, n_out);
    }
    const int N = *std::max_element(n, n + L);
    const bool wide = bf16 && (ceil_div(B, 256) * ceil_div(N, 256) >= 64 || (N >= 6144 && B >= 48) || (N >= 4096 && B >= 384));
    return std::max(used, wide ? std::min(tiles_128, tiles_256) : tiles_128);
}

hipError_t launch_fwd_gemm(const void* W, const float* bias, const void* A_in, void* A_out, float* raw,
                           int n_out, int n_in, int B, const GemmPlan& plan, hipStream_t s) {
    const int splits = chain_splits(n_out, n_in, B, plan.forward, plan.split_target);
    const bool half_tile = plan.forward == GEMM_HALF;
    GemmArgs g{};
    g.P = A_in; g.ldp = n_in; g.Q = W; g.ldq = n_in; g.M = B; g.Nn = n_out; g.K = n_in;
    g.k_tiles_per_split = ceil_div(ceil_div(n_in, half_tile ? half::TK : big::TK), splits);
    g.bias = bias; g.out = A_out; g.raw = raw;
    if (splits == 1)
        return half_tile ? run_half<false, false, EPI_SIGMOID>(g, 1, s) : run_big<false, false, EPI_SIGMOID>(g, 1, s);
    const hipError_t e = half_tile ? run_half<false, false, EPI_RAW>(g, splits, s)
                                   : run_big<false, false, EPI_RAW>(g, splits, s);
    if (e != hipSuccess) return e;
    const size_t count = (size_t)B * n_out;
    k_split_finish<EPI_SIGMOID><<<(unsigned)((count / 4 + kThreads - 1) / kThreads), kThreads, 0, s>>>(
        raw, splits, count, n_out, bias, nullptr, A_out, nullptr);
    return hipGetLastError();
}

hipError_t launch_chain_gemm(const void* W_next, const void* D_next_bf, const void* A_l, float* D_l, void* D_l_bf,
                             float* raw, int n_l, int n_next, int B, const GemmPlan& plan, hipStream_t s) {
    const int splits = chain_splits(n_l, n_next, B, plan.chain, plan.chain_split_target);
    const bool half_tile = plan.chain == GEMM_HALF;
    GemmArgs g{};
    g.P = D_next_bf; g.ldp = n_next; g.Q = W_next; g.ldq = n_l; g.M = B; g.Nn = n_l; g.K = n_next;
    g.k_tiles_per_split = ceil_div(ceil_div(n_next, half_tile ? half::TK : big::TK), splits);
    g.act = A_l; g.out = D_l; g.out_bf = D_l_bf; g.raw = raw;
    if (splits == 1)
        return half_tile ? run_half<false, true, EPI_SIGMA_PRIME>(g, 1, s) : run_big<false, true, EPI_SIGMA_PRIME>(g, 1, s);
    const hipError_t e = half_tile ? run_half<false, true, EPI_RAW>(g, splits, s)
                                   : run_big<false, true, EPI_RAW>(g, splits, s);
    if (e != hipSuccess) return e;
    const size_t count = (size_t)B * n_l;
    k_split_finish<EPI_SIGMA_PRIME><<<(unsigned)((count / 4 + kThreads - 1) / kThreads), kThreads, 0, s>>>(
        raw, splits, count, n_l, nullptr, static_cast<const __bf16*>(A_l), D_l, static_cast<__bf16*>(D_l_bf));
    return hipGetLastError();
}

hipError_t launch_grad_gemm(const float* D, const void* D_bf, const void* A_prev, float* nabla_w, float* nabla_b,
                            int n_l, int n_prev, int B, const GemmPlan& plan, bool whole_chip, float sgd_eta,
                            void* w_bf, hipStream_t s) {
    if ((sgd_eta != 0.0f) != (w_bf != nullptr)) return hipErrorInvalidValue;
    k_bias_grad<<<ceil_div(n_l, 32), kThreads, 0, s>>>(D, nabla_b, n_l, B, sgd_eta);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    GemmArgs g{};
    g.P = D_bf; g.ldp = n_l; g.Q = A_prev; g.ldq = n_prev; g.M = n_l; g.Nn = n_prev; g.K = B;
    g.out = nabla_w;
    g.sgd_eta = sgd_eta;
    g.out_bf = w_bf;
    g.k_tiles_per_split = ceil_div(B, plan.grad == GEMM_HALF ? half::TK : big::TK);
    if (plan.grad == GEMM_HALF) return run_half<true, true, EPI_GRAD>(g, 1, s);
    // the streamed kernel stores gradients only (the descent step keeps the tile-per-workgroup kernel), whole lines of
    // them, and addresses the result through one 32-bit buffer
    if (plan.grad == GEMM_STREAM && sgd_eta == 0.0f && n_prev % plan.stream_align == 0 &&
        (unsigned long long)(n_l + big::TM) * n_prev * 4ull < 0xFFFFFFF0ull)
        return run_grad_stream(g, whole_chip ? 256 : plan.stream_groups, s);
    return run_big<true, true, EPI_GRAD>(g, 1, s);
}

}  // namespace lf
