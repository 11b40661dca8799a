// Internal interface between the C-ABI layer (lf_api.hip) and the kernel files.
// Every launcher only enqueues work on `s` and returns the launch status.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "device_helpers.h"

namespace lf {

// ---- single-sample (B = 1) fp32 path: HBM-bound GEMV / outer-product kernels --------------------
// Matrices are rows x cols, row-major: w^l has n_l rows and n_{l-1} columns.

// Row blocks the transposed GEMV of eq. (bp2) is split into (its partial buffer is [P][cols]).
int chain_partial_blocks(int rows);

// eqs. (z),(a): a_out = sigma(W a_in + b); stream_weights: W is not worth keeping in the caches
hipError_t launch_fwd_gemv_f32(const float* W, const float* b, const float* a_in, float* a_out,
                               int rows, int cols, bool stream_weights, hipStream_t s);
// eq. (bp2): delta_l = (W_next^T delta_next) (.) a_l (1 - a_l); W_next is rows x cols, delta_next has rows
// entries, delta_l and a_l cols; partial: [chain_partial_blocks(rows)][cols]
hipError_t launch_chain_gemvT_f32(const float* W_next, const float* delta_next, const float* a_l,
                                  float* delta_l, float* partial, int rows, int cols, hipStream_t s);
// eqs. (bp3),(bp4): nabla_b = delta (rows entries); nabla_w[j][k] = delta[j] a_prev[k] (rows x cols).
// sgd_eta != 0: the descent step fused in -- nabla_w and nabla_b are then w^l and b^l themselves and receive
// w - eta nabla_w, b - eta nabla_b; the gradients are not stored.
hipError_t launch_grad_outer_f32(const float* delta, const float* a_prev, float* nabla_w,
                                 float* nabla_b, int rows, int cols, float sgd_eta, hipStream_t s);

// Both at once: the chain step, and beside its first kernel the gradients of a layer whose operands are there already.
struct OuterStep { const float* delta; const float* a_prev; float* w; float* b; int rows, cols; };
hipError_t launch_chain_gemvT_beside_grads_f32(const float* W_next, const float* delta_next, const float* a_l,
                                               float* delta_l, float* partial, int rows, int cols, const OuterStep& grads,
                                               float sgd_eta, hipStream_t s);

// ---- any B, either storage type ----------------------------------------------------------------

// eq. (bp1): delta_L = scale * (a_L - y) (.) a_L (1 - a_L) over count = B*N elements (scale: a power
// of two, see lf_set_cost_scale).  delta_bf (may be NULL) receives a bfloat16 copy of delta_L for the
// bf16 matrix kernels.  clear (may be NULL) receives `clear_words` zeros: the arrival counters of a split chain product.
hipError_t launch_output_error(const void* a_L, const void* y, float* delta_L, void* delta_bf,
                               size_t count, bool bf16, float scale, unsigned* clear, int clear_words, hipStream_t s);

// ---- minibatch path: which kernels ----------------------------------------------------------------

// DIRECT: the kernels of minibatch_kernels.h.  The others are the wide-net bf16 kernels: 256 x 256 tiles filling a
// compute unit, or 128 x 256 tiles sized so that two workgroups (of one product or of two) share a compute unit; the
// gradient product also as resident workgroups that stream through all their 256 x 256 tiles (STREAM).
enum GemmKernel { GEMM_DIRECT = 0, GEMM_BIG = 1, GEMM_HALF = 2, GEMM_STREAM = 3 };
struct GemmPlan {
    int forward;        // GemmKernel of the forward product,
    int chain;          // of the chain product
    int grad;           // and of the gradient product (chain and grad are either both DIRECT or neither)
    int split_target;   // workgroups the K split of a wide forward product aims at
    int chain_split_target;   // the same for the chain product of the backward pass
    int stream_groups;  // resident workgroups of the streamed gradient product
    int stream_align;   // the streamed product takes layers whose n_prev is a multiple of this
    int worker_streams; // streams the k workers share (worker j runs on stream j mod this)
};
// The plan of a net of L layers of n[0 .. L-1] neurons (decided once per net).
GemmPlan gemm_plan(const int* n, int L, int B, bool bf16);
// Floats of scratch that hold the split-K partials of a wide product with a B x n_out result under any plan.
size_t split_workspace_floats(int n_out, int B, bool bf16);
// Floats of chain scratch that lf_backward_leapfrog_noalloc charges a minibatch net of L layers of n[0 .. L-1] neurons for.
// This is the published limit of that call and does not follow the choice of kernels, which may change from one version
// to the next (the direct kernels use none of this scratch: the partial tiles of their split chain steps are in the
// handle's workspace, in this call too): the split-K partials of 128 x 128 tiles split to at most 512
// workgroups, or, for wide bf16 nets, those of 256 x 256 tiles split to at most 128 where they are fewer; and never
// less than what the plan's kernels do use.
size_t noalloc_scratch_floats(const int* n, int L, int B, bool bf16, const GemmPlan& plan);

// ---- minibatch path: wide bf16 nets ---------------------------------------------------------------

// eqs. (z),(a) for a minibatch: A_out[b][j] = sigma(sum_k A_in[b][k] W[j][k] + bias[j]); W is n_out x n_in.
// `raw` is the split-K scratch, split_workspace_floats(n_out, B, true) floats.
hipError_t launch_fwd_gemm(const void* W, const float* bias, const void* A_in, void* A_out, float* raw,
                           int n_out, int n_in, int B, const GemmPlan& plan, hipStream_t s);
// eq. (bp2) for a minibatch: D_l[b][k] = (sum_j D_next[b][j] W_next[j][k]) A_l[b][k] (1 - A_l[b][k]);
// W_next is n_next x n_l.  D_next_bf / D_l_bf are the bfloat16 copies used as matrix operands.
// raw: split_workspace_floats(n_l, B, true) floats.
hipError_t launch_chain_gemm(const void* W_next, const void* D_next_bf, const void* A_l, float* D_l, void* D_l_bf,
                             float* raw, int n_l, int n_next, int B, const GemmPlan& plan, hipStream_t s);
// eqs. (bp3),(bp4) for a minibatch: nabla_w[j][k] = sum_b D[b][j] A_prev[b][k] (n_l x n_prev);
// nabla_b[j] = sum_b D[b][j] (fixed summation order).
// sgd_eta != 0: the descent step fused into the epilogues -- nabla_w and nabla_b are then the fp32 master copy of w^l
// and b^l themselves and receive w - eta nabla_w, b - eta nabla_b, and w_bf, the bfloat16 weights, are rewritten as
// the master's rounding; the gradients are not stored.  whole_chip: nothing runs beside this product (the sequential
// pass), so the streamed kernel keeps a workgroup on every compute unit instead of the plan's share.
hipError_t launch_grad_gemm(const float* D, const void* D_bf, const void* A_prev, float* nabla_w, float* nabla_b,
                            int n_l, int n_prev, int B, const GemmPlan& plan, bool whole_chip, float sgd_eta,
                            void* w_bf, hipStream_t s);

// ---- minibatch path: direct kernels (fp32; bf16 nets that are not wide) -----------------------------

// eqs. (z),(a) for a minibatch (as launch_fwd_gemm), one launch, no scratch (the chain step takes some where few samples
// meet a wide layer).
hipError_t launch_forward_direct(const void* W, const float* bias, const void* A_in, void* A_out, int n_out, int n_in,
                                 int B, bool bf16, hipStream_t s);
struct ChainStep {      // eq. (bp2): delta^l from delta^{l+1} (as launch_chain_gemm; fp32 nets have no *_bf)
    const void* W_next; const float* D_next; const void* D_next_bf; const void* A_l; float* D_l; void* D_l_bf;
    int n_l, n_next;
    float* scratch;     // direct_chain_scratch_floats() floats (NULL where that is 0); its first chain_counters() words are 0
};                      // when the first chain step of a pass starts, and again when a step has ended
int chain_counters();
size_t direct_chain_scratch_floats(int n_l, int n_next, int B, bool bf16);
struct GradStep {       // eqs. (bp3), (bp4) of one layer (as launch_grad_gemm)
    const float* D; const void* D_bf; const void* A_prev; float* w; float* b; void* w_bf;
    int n_l, n_prev;
    int kind = -1;                  // how nabla_w is cut (a GradKind of minibatch_kernels.h), -1: as the layer's shape has it
    const unsigned* lost = nullptr; // a word of the device's, or none: while it is not 0 no descent step is taken
};
// One launch that takes a chain step (or none: NULL) and the gradients of up to two layers, none of which depends on
// another.  What a product's sums look like depends on its shape, B, the type and `kind` alone, not on what it is launched with.
hipError_t launch_backward_step(const ChainStep* chain, const GradStep* grads, int ngrads, int B, bool bf16,
                                float sgd_eta, hipStream_t s);

// The gradients of up to kGradLayers layers, all of one kind and with one `lost`, in one launch (none depends on another); and the kind
// that such a launch takes for all layers of a net.
constexpr int kGradLayers = 64;
hipError_t launch_all_gradients(const GradStep* grads, int count, int B, bool bf16, float sgd_eta, hipStream_t s);
int grad_kind_of_all(const int* n, int L, int B, bool bf16);
// For the choice of the kernels that walk all layers (cluster_plan), in us: such a gradients' launch, beyond its start; and a direction of
// a net of widths up to 1024 by a launch a layer.
double all_gradients_us(const int* n, int L, int B, bool bf16);
double layer_launches_us(const int* n, int L, int B, bool bf16, bool backward);

// ---- minibatch path: small nets (cluster_kernels.h) -------------------------------------------------

constexpr int kClusterLayers = 64;      // steps of one launch
struct ClusterPlan {
    bool forward, backward;             // whether the net's passes take these kernels
    int grad_kind;                      // how the gradients of all layers are cut, backward
    int clusters, per_cluster;          // clusters; workgroups of one
    int expected;                       // workgroups that make a cluster complete
    int S, ST;                          // samples of a slice; slices of a cluster
    int units;                          // units of the widest layer
    int nap;                            // pause before the first poll, in units of 64 cycles
    unsigned patience;                  // polls before a wait gives up
    size_t words;                       // exchanged words
    int state_words;
};
// The plan of a net of L layers of n[0 .. L-1] neurons (decided once per net).
ClusterPlan cluster_plan(const int* n, int L, int B, bool bf16);
struct ClusterPass {
    ClusterPlan plan;
    int L, B; const int* n; bool bf16;
    const void* x; const void* y; float scale;
    const void* const* w; const float* const* b;    // index l - 2
    char* a; size_t a_stride;           // a^l at a + (l - 2) a_stride
    char* d; size_t d_stride;           // delta^l, fp32
    char* d_bf; size_t d_bf_stride;     // its bfloat16 copy
    unsigned long long* words; unsigned* state;
    int* lost_host;                     // pinned word that a wait which gives up raises, as the device addresses it, or null
};
// The device's word, in the state: raised by a wait of this pass that gave up.
const unsigned* cluster_lost(const unsigned* state);
// Clears the words and the state: in front of a pass's first launch.
hipError_t launch_cluster_state(const ClusterPlan& plan, unsigned* state, unsigned long long* words, hipStream_t s);
// a^2 .. a^L
hipError_t launch_cluster_forward(const ClusterPass& p, hipStream_t s);
// delta^L .. delta^2
hipError_t launch_cluster_chain(const ClusterPass& p, hipStream_t s);

}  // namespace lf
