// Internal interface between the host driver (api.hip) and the kernel files.
// Not installed; the public interface is include/deeppcr.h.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

namespace deeppcr {

// Widths up to kMaxWidth use the per-width kernels (one workgroup or wave
// holds a whole block); kMaxWidth < w <= kMaxWideWidth use the tiled kernels
// of wide.hip.
constexpr int kMaxWidth = 128;
constexpr int kMaxWideWidth = 1024;

// The Newton convergence maxima are reduced into kRedShards slots each
// (slot = workgroup index mod kRedShards) to keep atomic contention low; the
// host takes the max over the slots after its one read-back per iteration.
// Reduction area: max|dZ| slots, then max|Z| slots (both cleared by the
// forward layer evaluation), then max|F| slots (the residual of the iterate,
// written by the forward layer evaluation; cleared by launch_zero_words).
constexpr int kRedShards = 256;
constexpr int kRedDZ = 0, kRedZ = kRedShards, kRedF = 2 * kRedShards;
constexpr int kRedWords = 3 * kRedShards;

// Layer kinds: code = 2 * activation + residual, activation 0 = tanh,
// 1 = logistic sigmoid, 2 = ReLU (derivative 0 at 0; a NaN input gives NaN).  The residual form is
// f(z) = z + alpha * sigma(W z + b), the plain form f(z) = sigma(W z + b).
constexpr int kNumLayerKinds = 6;
__host__ __device__ inline bool layer_residual(int layer) { return (layer & 1) != 0; }

// sigma(a) for the layer's activation; *d receives sigma'(a).
__device__ inline float activate(int layer, float a, float* d) {
    const int act = layer >> 1;
    if (act == 0) {
        const float t = tanhf(a);
        *d = 1.f - t * t;
        return t;
    }
    if (act == 1) {
        const float s = 1.f / (1.f + expf(-a));
        *d = s * (1.f - s);
        return s;
    }
    // NaN passes through (as max(a, 0) does in the usual frameworks)
    *d = a > 0.f ? 1.f : 0.f;
    return (a > 0.f || __builtin_isnan(a)) ? a : 0.f;
}

// Orders the LDS accesses of one wave (a barrier for the wave only).
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A batch of w x w blocks addressed as base + b*bstride + m*rstride (floats).
// Row strides may be negative (the transposed system is stored reversed).
// trans = 1: element (i, k) of block m is stored at [k*w + i].
struct BlockSrc {
    const float* base;
    long long bstride;
    long long rstride;
    int trans;
};

// A batch of length-w vectors, addressed like BlockSrc.
struct VecSrc {
    const float* base;
    long long bstride;
    long long rstride;
};

struct VecDst {
    float* base;
    long long bstride;
    long long rstride;
};

// ------------------------------------------------------------ layer kernels
// Forward Newton step: for every (b, l) evaluate the layer at Zprev = Z[b,l-1]
// (z0[b] for l = 0), write r[b,l] = f_l(Zprev) - Z[b,l] and, for l >= 1,
// the Jacobian block J_l into A ([B, L, w, w], forward row order).  The grid
// also clears the max|dZ| and max|Z| slots of `red` and reduces max|r| into
// its kRedF slots.  Widths up to 8 and above kMaxWidth (launch_layer_vectors
// has the others).
hipError_t launch_forward_eval(const float* W, const float* bias, const float* z0,
                               const float* Z, float* A, float* r, unsigned* red,
                               int B, int L, int w, int layer, float alpha,
                               hipStream_t stream);

// Z[b, l] = f_0(z0[b]) for every l.
hipError_t launch_initial_guess(const float* W, const float* bias, const float* z0,
                                float* Z, int B, int L, int w, int layer, float alpha,
                                hipStream_t stream);

// Z += x over n floats; red[kRedDZ + slot] = max bits of |x|,
// red[kRedZ + slot] = max bits of |Z| (atomic max on the IEEE bit patterns of
// non-negative floats, which orders NaN above Inf).
hipError_t launch_update_reduce(float* Z, const float* x, long long n, unsigned* red,
                                hipStream_t stream);

// Backward: Jacobian blocks of the transposed system in reversed row order,
// A[m = L-l] = J_l^T for l >= 1 (stored as J_l itself, i.e. to be read
// transposed), right-hand side rrev[m] = G if m == 0 else 0, and dscale[b, l]
// = c sigma'(a_l) in natural order; widths as launch_forward_eval.
hipError_t launch_backward_assemble(const float* W, const float* bias, const float* z0,
                                    const float* Z, const float* G, float* A, float* rrev,
                                    float* dscale, int B, int L, int w, int layer,
                                    float alpha, hipStream_t stream);

// dz0[b] = J_0^T Lambda[b, 0].
hipError_t launch_dz0(const float* W, const float* dscale, const float* Lambda, float* dz0,
                      int B, int L, int w, int layer, hipStream_t stream);

// dW[l] = sum_b (dscale*Lambda)[b,l] Zprev[b,l]^T, db[l] = sum_b (dscale*Lambda)[b,l].
hipError_t launch_wgrad(const float* z0, const float* Z, const float* dscale,
                        const float* Lambda, float* dW, float* db, int B, int L, int w,
                        hipStream_t stream);

// r = F - Z over n floats; max |r| bits into the kRedF slots of red.
hipError_t launch_residual(const float* F, const float* Z, float* r, long long n, unsigned* red,
                           hipStream_t stream);

// p[0 .. n) = 0 (a kernel, so that the call can sit in a captured graph).
hipError_t launch_zero_words(unsigned* p, int n, hipStream_t stream);
// out (host-mapped): out[0..2] = max over the kRedDZ, kRedZ, kRedF slots of
// red, then out[3] = seq.
hipError_t launch_measures(const unsigned* red, unsigned* out, unsigned seq, hipStream_t stream);

// dW[l] = sum_b Lambda[b,l] sigma(Zprev[b,l])^T, db[l] = sum_b Lambda[b,l]
// (pre-activation layers W sigma(z) + b; activation act: 0 tanh, 1 sigmoid,
// 2 ReLU).
hipError_t launch_wgrad_pre(const float* z0, const float* Z, const float* Lambda, float* dW,
                            float* db, int B, int L, int w, int act, hipStream_t stream);

// dst[b, l] = src[b, l] for every (b, l) (used when L = 1).
hipError_t launch_copy_rows(const VecSrc& src, const VecDst& dst, int B, int L, int w,
                            hipStream_t stream);

// ----------------------------------------------------------- small widths
// One PCR level with a lane group per row (w <= 3), and the layer evaluation
// with one thread per state element (w <= 8; forward and backward layouts as in
// launch_forward_eval / launch_backward_assemble).
bool small_width(int w);
hipError_t launch_pcr_level_small(const BlockSrc& Ain, const VecSrc& rin, float* Aout,
                                  const VecDst& rout, int B, int L, int w, int s,
                                  hipStream_t stream);
hipError_t launch_eval_small(bool bwd, const float* W, const float* bias, const float* z0,
                             const float* Z, const float* G, float* A, float* r, float* dscale,
                             unsigned* red, int B, int L, int w, int layer, float alpha,
                             hipStream_t stream);

// -------------------------------------------- solve on stored blocks, chunks
// How a solve (widths up to kMaxWidth) is cut, with its estimated time in us:
// chunks of m rows (0: substitution of all rows); walk: block_down finds every
// chunk's x_in itself from the chunk ends' P and q.
struct BlockPlan {
    int m;
    bool walk;
};
double block_plan(int B, int L, int w, BlockPlan* plan);
// The maps x_end = P x_in + q of chunks 0 .. C-2 of Lc rows (P [B, C-1, w, w],
// chunk 0 not written; q [B, C-1, w]).
// With y (w <= 16) A holds layer weights, not blocks: J = diag(d) W (+ I),
// d = y.d + b bstride + m rstride at row m; transposed, r is read at row 0 only.
struct LayerScale {
    const float* d;
    long long bstride, rstride;
    int residual;
};
hipError_t launch_block_up(const BlockSrc& A, const LayerScale* y, const VecSrc& r, float* P,
                           float* q, int B, int L, int w, int Lc, int C, hipStream_t st);
// The substitution inside every chunk, from xe [B, C-1, w], the solution at
// the chunk ends (P null), or from P and xe = q (unused for C = 1).  With red
// the solution is added to x (the Newton iterate), its maxima reduced into red.
hipError_t launch_block_down(const BlockSrc& A, const LayerScale* y, const VecSrc& r,
                             const VecDst& x, const float* xe, const float* P, unsigned* red,
                             int B, int L, int w, int Lc, int C, hipStream_t st);

// ------------------------------------------------------- chunked MLP solve
// The Newton solve (rows l = 0 .. L-1, operator of row l from layer l) and
// the transposed solve (rows m = 0 .. L, operator of row m from layer L - m,
// the last row being dz0) of MLP layers by chunks of Lc rows, widths
// panel_width accepts; WP = panel_pad(w) is the padded width of P, q, xe.
struct PanelArgs {
    const float* W;   // [L, w, w]
    const char* S;    // the weights split (PanelSplit), or null
    const float* scale;  // their factors, and whether there may be any
    const unsigned* odd;  // but 1: *odd == stamp
    unsigned stamp;
    const float* d;   // [B, L, w] c sigma'
    const float* r;   // [B, L, w] residuals; transposed: G [B, w]
    const float* xe;  // [B, C-1, WP] solution at the chunk ends
    float* P;         // [B, C-1, WP, WP] chunk products (chunk 0 not written)
    float* q;         // [B, C-1, WP] chunk vectors
    float* Z;         // [B, L, w] iterate, updated by the apply pass
    float* Lambda;    // [B, L, w]
    float* dz0;       // [B, w]
    unsigned* red;    // maxima of the update (apply pass)
    int B, L, w;
    int rows;         // L, transposed: L + 1
    int Lc, C;        // rows per chunk, ceil(rows / Lc)
    int residual;
};
// The weights (bwd: transposed) as bf16 parts in operand order, split_bytes
// (out null: not), and the factors of their results, split_scales of them.
struct PanelSplit {
    char* out;
    float* scale;
    unsigned* odd;
    unsigned stamp;
};
size_t split_bytes(int L, int w);
size_t split_scales(int L, int w);
bool panel_width(int w);
int panel_pad(int w);
int panel_chunks(int B, int rows, int w);
// d (and, forward, r and, if want_max, its maximum; clears the max|dZ|, max|Z|
// slots of red); with split the weights as well, once per call.
hipError_t launch_layer_vectors(bool bwd, const float* W, const float* bias, const float* z0,
                                const float* Z, float* d, float* r, unsigned* red, bool want_max,
                                int B, int L, int w, int layer, float alpha,
                                const PanelSplit* split, hipStream_t st);
// P of chunks 1 .. C-2 and q of chunks 0 .. C-2 (C >= 2).
hipError_t launch_chunk_pass(bool bwd, const PanelArgs& a, hipStream_t st);
// Every row from its chunk's x_in (xe of the chunk before; 0 in the first).
hipError_t launch_apply_pass(bool bwd, const PanelArgs& a, hipStream_t st);

// ------------------------------------------------------- sequential passes
// Layers l0 .. l1-1 of the sequential forward pass (one workgroup per system;
// reads Z[:, l0-1], or z0 when l0 = 0), and the sequential adjoint pass over
// layers l1-1 down to l0 (starting from G when l1 = L, else Lambda[:, l1-1]).
hipError_t launch_seq_forward(const float* W, const float* bias, const float* z0, float* Z, int B,
                              int L, int w, int layer, float alpha, int l0, int l1,
                              hipStream_t stream);
hipError_t launch_seq_backward(const float* W, const float* bias, const float* z0, const float* Z,
                               const float* G, float* Lambda, float* dz0, int B, int L, int w,
                               int layer, float alpha, int l0, int l1, hipStream_t stream);

// ------------------------------------------------- collapsed-skip ResNet
// Blocks of s layers, G = L / s blocks per system, X [B, G, w] the block
// outputs; act: 0 tanh, 1 sigmoid, 2 ReLU.
// Block evaluation at the iterate: r[b,g] = F_g(X[b,g-1]) - X[b,g] and, for
// g >= 1, A[b,g] = I + P_g (forward order); clears the max|dZ|, max|Z| slots.
hipError_t launch_resnet_block_eval(const float* W, const float* bias, const float* z0,
                                    const float* X, float* A, float* r, unsigned* red, int B,
                                    int G, int w, int skip, int act, hipStream_t stream);
// X[b, g] = F_0(z0[b]) for every g.
hipError_t launch_resnet_initial_guess(const float* W, const float* bias, const float* z0,
                                       float* X, int B, int G, int w, int skip, int act,
                                       hipStream_t stream);
// Z [B, L, w]: the layers inside each block run from X[b, g-1]; row gs+s-1 = X[b, g].
hipError_t launch_resnet_expand(const float* W, const float* bias, const float* z0,
                                const float* X, float* Z, int B, int G, int w, int skip, int act,
                                hipStream_t stream);
// Backward blocks at the stored states Z: A[b, G-g] = I + P_g (g >= 1, to be
// read transposed), rrev[b, m] = G[b] if m == 0 else 0.
hipError_t launch_resnet_block_jac(const float* W, const float* z0, const float* Z,
                                   const float* Gv, float* A, float* rrev, int B, int G, int w,
                                   int skip, int act, hipStream_t stream);
// Lambda [B, L, w] inside every block from mu [B, G, w] (block-output
// adjoints, natural order), and dz0.
hipError_t launch_resnet_intra_adjoint(const float* W, const float* z0, const float* Z,
                                       const float* mu, float* Lambda, float* dz0, int B, int G,
                                       int w, int skip, int act, hipStream_t stream);

// The collapsed-skip ResNet's sequential passes (one workgroup per system):
// forward layers l0 .. l1-1, and the reverse-mode adjoints over layers l1-1
// down to l0 (Lambda, and dz0 when l0 = 0).
hipError_t launch_resnet_seq_forward(const float* W, const float* bias, const float* z0, float* Z,
                                     int B, int L, int w, int skip, int act, int l0, int l1,
                                     hipStream_t stream);
hipError_t launch_resnet_seq_backward(const float* W, const float* z0, const float* Z,
                                      const float* G, float* Lambda, float* dz0, int B, int L,
                                      int w, int skip, int act, int l0, int l1,
                                      hipStream_t stream);

// ----------------------------------------------------- row-chunked solve
// The rows of each system cut into chunks of Lc rows (natural order; the
// last chunk may be shorter); rev = 1 runs the transposed system in reversed
// internal row order.  Chunk-local PCR level with stride s keeping every
// chunk's coupling to the row outside it (except the chunk holding internal
// row 0): Aout [B, L, w, w] and rout [B, L, w] contiguous, internal order.
int chunk_count(int L, int Lc);
void chunk_level_work(int B, int L, int w, int Lc, int rev, int s, double* bytes,
                      double* flops);
hipError_t launch_chunk_level(const BlockSrc& Ain, const VecSrc& rin, float* Aout, float* rout,
                              int B, int L, int w, int Lc, int rev, int s, hipStream_t stream);
// The chains left after the chunk-local levels with strides below s, solved
// by substitution into every row's map (P_j, q_j; q only in the chunk
// holding internal row 0), for the widths chunk_chain_width accepts; Ain and
// rin are the level buffers (contiguous, internal order), Pout and qout the
// same layout.
bool chunk_chain_width(int w);
void chunk_chain_work(int B, int L, int w, int Lc, int rev, int s, double* bytes,
                      double* flops);
hipError_t launch_chunk_chain(const float* Ain, const float* rin, float* Pout, float* qout,
                              int B, int L, int w, int Lc, int rev, int s, hipStream_t stream);
// xin [B, chunk_count, w]: the carry-in of every chunk (internal chunk order)
// from the chunk-end rows of P (the final operators) and q (final vectors).
hipError_t launch_chunk_carry(const float* P, const float* q, float* xin, int B, int L, int w,
                              int Lc, int rev, hipStream_t stream);
// x (natural-order destination) = q + P xin of each row's chunk.
hipError_t launch_chunk_apply(const float* P, const float* q, const float* xin, const VecDst& x,
                              int B, int L, int w, int Lc, int rev, hipStream_t stream);

// ------------------------------------------------------------ wide widths
// kMaxWidth < w <= kMaxWideWidth: the same operations as launch_pcr_level,
// launch_forward_eval, launch_initial_guess, launch_backward_assemble (blocks
// stored as J_l, read transposed), launch_dz0 and launch_wgrad, and one
// layer l of the sequential passes (the backward uses dz0 as its scratch for
// the scaled adjoint until the last step).
bool wide_width(int w);
hipError_t launch_pcr_level_wide(const BlockSrc& Ain, const VecSrc& rin, float* Aout,
                                 const VecDst& rout, int B, int L, int w, int s,
                                 hipStream_t stream);
hipError_t launch_forward_eval_wide(const float* W, const float* bias, const float* z0,
                                    const float* Z, float* A, float* r, unsigned* red, int B,
                                    int L, int w, int layer, float alpha, hipStream_t stream);
hipError_t launch_initial_guess_wide(const float* W, const float* bias, const float* z0, float* Z,
                                     int B, int L, int w, int layer, float alpha,
                                     hipStream_t stream);
hipError_t launch_backward_assemble_wide(const float* W, const float* bias, const float* z0,
                                         const float* Z, const float* G, float* A, float* rrev,
                                         float* dscale, int B, int L, int w, int layer,
                                         float alpha, hipStream_t stream);
// Whether a solve of `rows` rows goes row by row instead of by PCR levels;
// the layers' d and r (as launch_layer_vectors); one row of the forward solve
// in place (r_l becomes the solution), l >= 1; one row of the transposed solve
// (Lambda_{l-1}, or dz0 at l = 0, from Lambda_l, or G at l = L - 1).
bool wide_substitution(int B, int rows, int w);
hipError_t launch_wide_vectors(bool bwd, const float* W, const float* bias, const float* z0,
                               const float* Z, float* d, float* r, unsigned* red, int B, int L,
                               int w, int layer, float alpha, hipStream_t stream);
hipError_t launch_wide_step(const float* W, const float* d, float* r, int B, int L, int w,
                            int residual, int l, hipStream_t stream);
hipError_t launch_wide_step_t(const float* W, const float* d, const float* G, float* Lambda,
                              float* dz0, int B, int L, int w, int residual, int l,
                              hipStream_t stream);
hipError_t launch_dz0_wide(const float* W, const float* dscale, const float* Lambda, float* dz0,
                           int B, int L, int w, int layer, hipStream_t stream);
hipError_t launch_wgrad_wide(const float* z0, const float* Z, const float* dscale,
                             const float* Lambda, float* dW, float* db, int B, int L, int w,
                             hipStream_t stream);
hipError_t launch_seq_forward_wide(const float* W, const float* bias, const float* z0, float* Z,
                                   int B, int L, int w, int layer, float alpha, int l,
                                   hipStream_t stream);
hipError_t launch_seq_backward_wide(const float* W, const float* bias, const float* z0,
                                    const float* Z, const float* G, float* Lambda, float* dz0,
                                    int B, int L, int w, int layer, float alpha, int l,
                                    hipStream_t stream);

// ------------------------------------------------------------- tiny path
// Whole Newton + PCR forward solve in one workgroup with everything in LDS,
// for batches that fit in 64 KiB.  result[0] = status (0 ok, 2 no
// convergence, 3 non-finite), result[1] = solves, result[2] = bits of the
// last max|dZ| (update rule) or of the last residual norm (residual rule).
// Z_init may be null or alias Z.
struct StopRule {
    int residual;  // 0: max|dZ| < tol * max(1, max|Z|) after each update;
                   // 1: max|F| <= atol or <= rtol * max|F_0| before each solve
    float tol, atol, rtol;
    int max_iter;
};
bool tiny_eligible(int B, int L, int w);
size_t tiny_lds_bytes(int B, int L, int w);
hipError_t launch_newton_tiny(const float* W, const float* bias, const float* z0, float* Z,
                              const float* Z_init, int B, int L, int w, int layer, float alpha,
                              const StopRule& rule, unsigned* result, hipStream_t stream);

}  // namespace deeppcr
