// Single-sample (B = 1) fp32 kernels: every step is bound by HBM traffic on the N x N matrix
// (one read of w^l forward, one read of w^{l+1} on the delta chain, one write of nabla_w^l), so the
// kernels are organised around coalesced 128-bit accesses, many loads in flight per wave, and
// reduction trees that depend on N alone (results are bit-identical for every launch shape and k).
#include "lf_internal.h"

namespace lf {

namespace {

constexpr int kThreads = 256;            // 4 waves per workgroup
constexpr int kWavesPerWg = kThreads / kWave;

__host__ __device__ constexpr int ceil_div(int a, int b) { return (a + b - 1) / b; }

// ------------------------------------------------------------------------------------------------
// eqs. (z),(a):  a_out[j] = sigma( sum_k W[j][k] a_in[k] + b[j] ),  W is rows x cols
// One wave owns R consecutive rows.  a_in is staged once per workgroup in LDS; a lane walks the row
// in float4 steps of stride 64 lanes, keeps one accumulator per row, and the 64 lane sums are
// combined in a fixed order (row rotations, then the four rows of 16 lanes).
template <int R, bool NT>
__global__ __launch_bounds__(kThreads) void k_fwd_gemv(const float* __restrict__ W,
                                                       const float* __restrict__ bias,
                                                       const float* __restrict__ a_in,
                                                       float* __restrict__ a_out, int rows, int cols) {
    extern __shared__ v4f s_a[];   // cols/4 float4
    const int nvec = cols >> 2;
    for (int v = threadIdx.x; v < nvec; v += kThreads) s_a[v] = reinterpret_cast<const v4f*>(a_in)[v];
    __syncthreads();

    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x >> 6;
    const int row0 = (blockIdx.x * kWavesPerWg + wave) * R;
    if (row0 >= rows) return;

    const v4f* wrow[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int row = min(row0 + r, rows - 1);   // rows past the end repeat the last one; not stored
        wrow[r] = reinterpret_cast<const v4f*>(W + (size_t)row * cols);
    }
    float acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r) acc[r] = 0.0f;

    constexpr int U = R == 2 ? 4 : 8;                    // float4 loads in flight per lane = R*U
    v4f w[U][R];
    auto request = [&](int u, int v) {
#pragma unroll
        for (int r = 0; r < R; ++r) w[u][r] = NT ? __builtin_nontemporal_load(&wrow[r][v]) : wrow[r][v];
    };
    auto add = [&](int u, int v) {
        const v4f a = s_a[v];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            acc[r] = fmaf(w[u][r].x, a.x, acc[r]);
            acc[r] = fmaf(w[u][r].y, a.y, acc[r]);
            acc[r] = fmaf(w[u][r].z, a.z, acc[r]);
            acc[r] = fmaf(w[u][r].w, a.w, acc[r]);
        }
    };
    int v = lane, left = nvec;                           // this lane's vector; vectors of the row from lane 0's on
#pragma unroll 1
    for (; left >= U * kWave; left -= U * kWave, v += U * kWave) {
#pragma unroll
        for (int u = 0; u < U; ++u) request(u, v + u * kWave);
#pragma unroll
        for (int u = 0; u < U; ++u) add(u, v + u * kWave);
    }
    // What is left of the row, U - 1 whole steps and a part of one at most: requested at once as well (U/2, U/4, .. 1 steps, then the
    // part), but for a step or two, which short rows end with sooner (widths 64-8192-64-8192-64 3.9 us a layer, 4.1 that way).
    // One step after the other, us a layer: N = 8000, L = 3 53 -> 50, 14000, L = 2 155 -> 142; non-temporal 46 -> 43, 126 -> 118.
    if (left > 2 * kWave) {
        const int steps = left / kWave;
        auto rest = [&](auto each) {
#pragma unroll
            for (int h = U / 2; h >= 1; h /= 2)
                if (steps & h) {
#pragma unroll
                    for (int u = 0; u < h; ++u) each(U - 2 * h + u, v + ((steps & (U - 2 * h)) + u) * kWave);
                }
            if (lane < left % kWave) each(U - 1, v + steps * kWave);
        };
        rest(request);
        rest(add);
    } else {
#pragma unroll 1
        for (; v < nvec; v += kWave) {
            request(0, v);
            add(0, v);
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const float z = wave_sum(acc[r]);
        if (lane == 0 && row0 + r < rows) a_out[row0 + r] = sigmoidf(z + bias[row0 + r]);
    }
}

// ------------------------------------------------------------------------------------------------
// eq. (bp2), stage 1: partial[p][k] = sum over the rows j of block p of W[j][k] * delta[j]; W is rows x cols.
// A workgroup covers one strip of 256 columns (a lane owns 4 consecutive columns, so each row is read
// as one contiguous 1 KiB segment) and RPW rows per wave; the four waves' sums are added in wave
// order through LDS.
template <int RPW>
__device__ __forceinline__ void chain_partial_block(const float* __restrict__ W, const float* __restrict__ delta,
                                                    float* __restrict__ partial, int rows, int cols, int strip, int block) {
    __shared__ v4f s_acc[kWavesPerWg][kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x >> 6;
    const int col = strip * (kWave * 4) + lane * 4;
    const int row_begin = (block * kWavesPerWg + wave) * RPW;
    v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
    if (col < cols) {
        const float* wp = W + (size_t)row_begin * cols + col;
        if (row_begin + RPW <= rows) {
            v4f w[RPW];
#pragma unroll
            for (int r = 0; r < RPW; ++r) w[r] = *reinterpret_cast<const v4f*>(wp + (size_t)r * cols);
#pragma unroll
            for (int r = 0; r < RPW; ++r) {
                const float d = delta[row_begin + r];
                acc.x = fmaf(w[r].x, d, acc.x);
                acc.y = fmaf(w[r].y, d, acc.y);
                acc.z = fmaf(w[r].z, d, acc.z);
                acc.w = fmaf(w[r].w, d, acc.w);
            }
        } else {
            for (int r = 0; r < RPW && row_begin + r < rows; ++r) {
                const v4f w = *reinterpret_cast<const v4f*>(wp + (size_t)r * cols);
                const float d = delta[row_begin + r];
                acc.x = fmaf(w.x, d, acc.x);
                acc.y = fmaf(w.y, d, acc.y);
                acc.z = fmaf(w.z, d, acc.z);
                acc.w = fmaf(w.w, d, acc.w);
            }
        }
    }
    s_acc[wave][lane] = acc;
    __syncthreads();
    if (wave == 0 && col < cols) {
        v4f t = s_acc[0][lane];
#pragma unroll
        for (int q = 1; q < kWavesPerWg; ++q) t += s_acc[q][lane];
        *reinterpret_cast<v4f*>(partial + (size_t)block * cols + col) = t;
    }
}
template <int RPW>
__global__ __launch_bounds__(kThreads) void k_chain_partial(const float* __restrict__ W, const float* __restrict__ delta,
                                                            float* __restrict__ partial, int rows, int cols) {
    chain_partial_block<RPW>(W, delta, partial, rows, cols, blockIdx.x, blockIdx.y);
}

// eq. (bp2), stage 2: delta_l[k] = (sum_p partial[p][k]) * a_l[k] * (1 - a_l[k]), p in ascending order.
__global__ __launch_bounds__(kThreads) void k_chain_finish(const float* __restrict__ partial,
                                                           const float* __restrict__ a_l,
                                                           float* __restrict__ delta_l, int N, int P) {
    const int k = blockIdx.x * kThreads + threadIdx.x;
    if (k >= N) return;
    const float a = a_l[k];
    float u = 0.0f;
    int p = 0;
    for (; p + 8 <= P; p += 8) {            // eight requested at a time, added in ascending order
        float v[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) v[c] = partial[(size_t)(p + c) * N + k];
#pragma unroll
        for (int c = 0; c < 8; ++c) u += v[c];
    }
    for (; p < P; ++p) u += partial[(size_t)p * N + k];
    delta_l[k] = u * (a * (1.0f - a));
}

// ------------------------------------------------------------------------------------------------
// eqs. (bp3),(bp4):  nabla_b[j] = delta[j];  nabla_w[j][k] = delta[j] * a_prev[k]  (rows x cols).
// Pure store stream.  A wave owns a strip of 256 columns (its a_prev values stay in registers) and
// RW rows, and writes each row segment with one non-temporal 128-bit store per lane.
// SGD: the gradient-descent step fused into the worker -- `nabla_w` and `nabla_b` are then w^l and b^l
// themselves and receive w - eta * nabla_w, b - eta * nabla_b (the gradient entry is rounded to fp32 exactly as
// it would have been stored, then one fused multiply-add); the gradients are not stored.
template <int RW, bool SGD>
__device__ __forceinline__ void grad_outer_block(const float* __restrict__ delta, const float* __restrict__ a_prev,
                                                 float* nabla_w, float* nabla_b, int rows, int cols, int nstrips, float eta,
                                                 int block) {
    const int lane = threadIdx.x & (kWave - 1);
    const int gw = block * kWavesPerWg + (threadIdx.x >> 6);   // global wave index
    const int strip = gw % nstrips;
    const int row0 = (gw / nstrips) * RW;
    if (row0 >= rows) return;
    const int col = strip * (kWave * 4) + lane * 4;
    if (strip == 0) {
        for (int r = lane; r < RW && row0 + r < rows; r += kWave) {
            if constexpr (SGD) nabla_b[row0 + r] = fmaf(-eta, delta[row0 + r], nabla_b[row0 + r]);
            else nabla_b[row0 + r] = delta[row0 + r];
        }
    }
    if (col >= cols) return;
    const v4f a = *reinterpret_cast<const v4f*>(a_prev + col);
    float* out = nabla_w + (size_t)row0 * cols + col;
    if constexpr (SGD) {
        constexpr int U = 8;                          // rows read ahead
#pragma unroll 1
        for (int r0 = 0; r0 < RW; r0 += U) {
            v4f w[U];
#pragma unroll
            for (int u = 0; u < U; ++u)   // rows past the end re-read the last one; not stored
                w[u] = *reinterpret_cast<const v4f*>(out + (size_t)(min(row0 + r0 + u, rows - 1) - row0) * cols);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (row0 + r0 + u >= rows) break;
                const float d = delta[row0 + r0 + u];
                const v4f g = {d * a.x, d * a.y, d * a.z, d * a.w};
                const v4f o = {fmaf(-eta, g.x, w[u].x), fmaf(-eta, g.y, w[u].y), fmaf(-eta, g.z, w[u].z),
                               fmaf(-eta, g.w, w[u].w)};
                *reinterpret_cast<v4f*>(out + (size_t)(r0 + u) * cols) = o;
            }
        }
    } else {
#pragma unroll 4
        for (int r = 0; r < RW; ++r) {
            if (row0 + r >= rows) break;
            const float d = delta[row0 + r];
            const v4f g = {d * a.x, d * a.y, d * a.z, d * a.w};
            __builtin_nontemporal_store(g, reinterpret_cast<v4f*>(out + (size_t)r * cols));
        }
    }
}
template <int RW, bool SGD>
__global__ __launch_bounds__(kThreads) void k_grad_outer(const float* __restrict__ delta, const float* __restrict__ a_prev,
                                                         float* nabla_w, float* nabla_b, int rows, int cols, int nstrips,
                                                         float eta) {
    grad_outer_block<RW, SGD>(delta, a_prev, nabla_w, nabla_b, rows, cols, nstrips, eta, blockIdx.x);
}

// Both in one launch: stage 1 of the chain step delta^{l+1} -> delta^l, and beside it the gradients (or the descent step) of a
// layer above, which do not wait for it.  A pass of a small net is a sequence of launches of about 3 us each, and this is
// one for two: us a pass, in line without / with it: widths 72-100-64-200-128-80-64-400 83 / 67,
// 84-996-6348-1364-1084-88 147 / 88;  N = 4100, L = 6 295 / 220;  N = 8192, L = 12 2021 / 1743 (the stores fill what the chain leaves of memory).
struct OuterArgs { const float* delta; const float* a_prev; float* w; float* b; int rows, cols, nstrips; float eta; };
template <int RPW, int RW, bool SGD>
__global__ __launch_bounds__(kThreads) void k_chain_partial_beside_grads(const float* __restrict__ W,
                                                                         const float* __restrict__ delta,
                                                                         float* __restrict__ partial, int rows, int cols,
                                                                         int strips, int chain_blocks, const OuterArgs g) {
    const int x = blockIdx.x;
    if (x < chain_blocks) chain_partial_block<RPW>(W, delta, partial, rows, cols, x % strips, x / strips);
    else grad_outer_block<RW, SGD>(g.delta, g.a_prev, g.w, g.b, g.rows, g.cols, g.nstrips, g.eta, x - chain_blocks);
}

// ------------------------------------------------------------------------------------------------
// eq. (bp1): delta_L = (a_L - y) * a_L * (1 - a_L), elementwise, fp32 or bfloat16 storage.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_output_error(const T* __restrict__ a_L,
                                                           const T* __restrict__ y,
                                                           float* __restrict__ delta_L,
                                                           __bf16* __restrict__ delta_bf, size_t count,
                                                           float scale, unsigned* clear, int clear_words) {
    if (clear && blockIdx.x == 0)
        for (int c = threadIdx.x; c < clear_words; c += kThreads) clear[c] = 0;
    const size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
    if (i >= count) return;
    const float a = (float)a_L[i];
    const float d = scale * ((a - (float)y[i]) * (a * (1.0f - a)));
    delta_L[i] = d;
    if (delta_bf) delta_bf[i] = (__bf16)d;
}

int chain_rows_per_wave(int rows) { return rows >= 4096 ? 16 : (rows >= 2048 ? 8 : 4); }

}  // namespace

int chain_partial_blocks(int rows) { return ceil_div(rows, kWavesPerWg * chain_rows_per_wave(rows)); }

// Rows a wave: one where the matrix is large or small, two in between (as few waves as fill the chip, as many bytes in flight).
// Weights that exceed the cache are read with non-temporal loads.  Forward pass, us, four rows a wave / one / one, non-temporal:
// N = 4100, L = 6 81 / 74 / 66;  N = 5000, L = 6 120 / 98 / 89;  N = 8192, L = 12 649 / 544 / 490 (6.0 TB/s);  L = 2, N = 12288
// 110 / 101 / 88, 16384 (two workgroups a compute unit, for the 64 KB of a^{l-1} that each holds) 182 / 201 / 163.
template <bool NT>
static void fwd_gemv(const float* W, const float* b, const float* a_in, float* a_out, int rows, int cols, hipStream_t s) {
    const size_t lds = (size_t)cols * sizeof(float), elems = (size_t)rows * cols;
    if (elems >= (size_t)2048 * 2048 && elems < (size_t)4096 * 4096)
        k_fwd_gemv<2, NT><<<ceil_div(rows, kWavesPerWg * 2), kThreads, lds, s>>>(W, b, a_in, a_out, rows, cols);
    else
        k_fwd_gemv<1, NT><<<ceil_div(rows, kWavesPerWg), kThreads, lds, s>>>(W, b, a_in, a_out, rows, cols);
}

hipError_t launch_fwd_gemv_f32(const float* W, const float* b, const float* a_in, float* a_out,
                               int rows, int cols, bool stream_weights, hipStream_t s) {
    if (stream_weights) fwd_gemv<true>(W, b, a_in, a_out, rows, cols, s);
    else fwd_gemv<false>(W, b, a_in, a_out, rows, cols, s);
    return hipGetLastError();
}

hipError_t launch_chain_gemvT_f32(const float* W_next, const float* delta_next, const float* a_l,
                                  float* delta_l, float* partial, int rows, int cols, hipStream_t s) {
    const int rpw = chain_rows_per_wave(rows);
    const int P = chain_partial_blocks(rows);
    const dim3 grid(ceil_div(cols, kWave * 4), P);
    if (rpw == 16) k_chain_partial<16><<<grid, kThreads, 0, s>>>(W_next, delta_next, partial, rows, cols);
    else if (rpw == 8) k_chain_partial<8><<<grid, kThreads, 0, s>>>(W_next, delta_next, partial, rows, cols);
    else k_chain_partial<4><<<grid, kThreads, 0, s>>>(W_next, delta_next, partial, rows, cols);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_chain_finish<<<ceil_div(cols, kThreads), kThreads, 0, s>>>(partial, a_l, delta_l, cols, P);
    return hipGetLastError();
}

template <bool SGD>
static void chain_partial_beside_grads(const float* W_next, const float* delta_next, float* partial, int rows, int cols,
                                       const OuterArgs& g, hipStream_t s) {
    constexpr int RW = 16;
    const int rpw = chain_rows_per_wave(rows), strips = ceil_div(cols, kWave * 4);
    const int chain_blocks = strips * chain_partial_blocks(rows);
    const int grid = chain_blocks + ceil_div(g.nstrips * ceil_div(g.rows, RW), kWavesPerWg);
    if (rpw == 16)
        k_chain_partial_beside_grads<16, RW, SGD><<<grid, kThreads, 0, s>>>(W_next, delta_next, partial, rows, cols, strips, chain_blocks, g);
    else if (rpw == 8)
        k_chain_partial_beside_grads<8, RW, SGD><<<grid, kThreads, 0, s>>>(W_next, delta_next, partial, rows, cols, strips, chain_blocks, g);
    else
        k_chain_partial_beside_grads<4, RW, SGD><<<grid, kThreads, 0, s>>>(W_next, delta_next, partial, rows, cols, strips, chain_blocks, g);
}

hipError_t launch_chain_gemvT_beside_grads_f32(const float* W_next, const float* delta_next, const float* a_l,
                                               float* delta_l, float* partial, int rows, int cols, const OuterStep& o,
                                               float sgd_eta, hipStream_t s) {
    const OuterArgs g{o.delta, o.a_prev, o.w, o.b, o.rows, o.cols, ceil_div(o.cols, kWave * 4), sgd_eta};
    if (sgd_eta != 0.0f) chain_partial_beside_grads<true>(W_next, delta_next, partial, rows, cols, g, s);
    else chain_partial_beside_grads<false>(W_next, delta_next, partial, rows, cols, g, s);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_chain_finish<<<ceil_div(cols, kThreads), kThreads, 0, s>>>(partial, a_l, delta_l, cols, chain_partial_blocks(rows));
    return hipGetLastError();
}

hipError_t launch_grad_outer_f32(const float* delta, const float* a_prev, float* nabla_w,
                                 float* nabla_b, int rows, int cols, float sgd_eta, hipStream_t s) {
    const int nstrips = ceil_div(cols, kWave * 4);
    constexpr int RW = 16;
    const int waves = nstrips * ceil_div(rows, RW);
    const int grid = ceil_div(waves, kWavesPerWg);
    if (sgd_eta != 0.0f)
        k_grad_outer<RW, true><<<grid, kThreads, 0, s>>>(delta, a_prev, nabla_w, nabla_b, rows, cols, nstrips,
                                                         sgd_eta);
    else
        k_grad_outer<RW, false><<<grid, kThreads, 0, s>>>(delta, a_prev, nabla_w, nabla_b, rows, cols, nstrips,
                                                          0.0f);
    return hipGetLastError();
}

hipError_t launch_output_error(const void* a_L, const void* y, float* delta_L, void* delta_bf,
                               size_t count, bool bf16, float scale, unsigned* clear, int clear_words, hipStream_t s) {
    const unsigned grid = (unsigned)((count + kThreads - 1) / kThreads);
    if (bf16)
        k_output_error<__bf16><<<grid, kThreads, 0, s>>>((const __bf16*)a_L, (const __bf16*)y, delta_L,
                                                         (__bf16*)delta_bf, count, scale, clear, clear_words);
    else
        k_output_error<float><<<grid, kThreads, 0, s>>>((const float*)a_L, (const float*)y, delta_L,
                                                        (__bf16*)delta_bf, count, scale, clear, clear_words);
    return hipGetLastError();
}

}  // namespace lf
