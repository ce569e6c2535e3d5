// Internal launch interface between the C-ABI layer (api.hip) and the kernel files.
// Every launcher validates nothing (the C-ABI layer did), enqueues on `st` and returns 0 or a
// DLAYER_ERR_LAUNCH code with the thread-local message set.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace dl {

// ---- elementwise.hip
int launch_rmsnorm_fwd(const void* x, const void* gamma, int64_t T, int64_t D, float eps, void* h,
                       float* rstd, hipStream_t st);
// a norm and the rotary table (launch_rope_table) in one launch
int launch_rmsnorm_fwd_rope_table(const void* x, const void* gamma, int64_t T, int64_t D, float eps, void* h, float* rstd, float* cos,
                                  float* sin, int64_t seq, int64_t head_dim, float base, hipStream_t st);
size_t rmsnorm_bwd_workspace(int64_t T, int64_t D);
// the two halves of launch_rmsnorm_bwd: dx and the partial rows in `workspace`; then dgamma from them, of one norm or
// (ws_b, dgamma_b not null) two of the same shape.  h (or null): the forward's output, written again from x and rstd
int launch_rmsnorm_bwd_rows(const void* x, const void* gamma, const float* rstd, const void* dh,
                            const void* dres, int64_t T, int64_t D, void* dx, void* h, void* workspace, hipStream_t st);
// The second half as an argument for a launch that has room for it: column sums of nrows partial rows of D, one norm or (b not
// null) two
struct GainSums { const float *pa, *pb; void *outa, *outb; int nrows, D, accumulate; };
GainSums rmsnorm_bwd_gain_sums(const void* ws_a, void* dgamma_a, const void* ws_b, void* dgamma_b, int64_t T, int64_t D, int accumulate);
int launch_gain_sums(const GainSums& s, hipStream_t st);
int launch_rmsnorm_bwd_gain(const void* ws_a, void* dgamma_a, const void* ws_b, void* dgamma_b, int64_t T, int64_t D,
                            int accumulate, hipStream_t st);
int launch_rmsnorm_bwd(const void* x, const void* gamma, const float* rstd, const void* dh,
                       const void* dres, int64_t T, int64_t D, void* dx, void* dgamma,
                       int accumulate, void* workspace, hipStream_t st);
int launch_rope(void* z, int64_t batch, int64_t seq, int64_t n_heads, int64_t head_dim, float base,
                int layout, int inverse, hipStream_t st);
// cos and sin of angle(p, i) = p * base^(-2 i / head_dim) for p < seq, i < head_dim / 2, evaluated in
// fp64 and stored as fp32 [seq][head_dim / 2]
int launch_rope_table(float* cos, float* sin, int64_t seq, int64_t head_dim, float base, hipStream_t st);
int launch_swiglu_fwd(const void* g, const void* u, int64_t n, void* a, hipStream_t st);
int launch_swiglu_bwd(const void* g, const void* u, const void* da, int64_t n, void* dg, void* du,
                      hipStream_t st);
// g, u: [rows, cols] with leading dimension ld_gu; a with its own (padded) one
int launch_swiglu_fwd_rows(const void* g, const void* u, int64_t rows, int64_t cols, int64_t ld_gu, void* a,
                           int64_t ld_a, hipStream_t st);
// out[c][r] = in[r][c]; out has leading dimension ld_out >= R
int launch_transpose(const void* in, void* out, int64_t R, int64_t C, int64_t ld_out, hipStream_t st);
// up to 8 transposes (each R, C multiples of 64) in one launch
constexpr int kMaxTransposeGroup = 8;
struct TransposeJob { const void* in; void* out; int64_t R, C, ld_out; };
int launch_transpose_group(const TransposeJob* jobs, int n, hipStream_t st);
int launch_embed_fwd(const void* table, const int64_t* ids, int64_t T, int64_t V, int64_t D,
                     void* x0, hipStream_t st);
size_t embed_bwd_workspace(int64_t T, int64_t V);
int launch_embed_bwd(const void* dx0, const int64_t* ids, int64_t T, int64_t V, int64_t D,
                     void* dtable, void* workspace, hipStream_t st);

// ---- gemm.hip
// Compute units of the current device: 256 on a whole MI355X, fewer on a partition of one.  256 where there is no device to
// ask (a plan made on the host).
int compute_units();
// C[M,N] (bf16, row-major, leading dimension ldc) = sum over segments s of opA_s * opB_s
//        (+ R[M,N] if R) (+ C if accumulate), fp32 accumulation.
// Segment operands are bf16 row-major.  a_kmajor: A_s is [M, K_s] (lda >= K_s) else [K_s, M]
// (lda >= M).  b_kmajor: B_s is [N, K_s] else [K_s, N].  K_s % 64 == 0, N % 8 == 0.
struct GemmSeg {
  const void* a;
  const void* b;
  int64_t lda, ldb;
  int K;
};
struct GemmArgs {
  GemmSeg seg[3];
  int nseg;
  int M, N;
  void* c;
  int64_t ldc;
  const void* r;  // optional residual, same leading dimension as c
  int accumulate;
  bool a_kmajor, b_kmajor;
};
int launch_gemm(const GemmArgs& g, hipStream_t st);
// The product is dO [tokens][heads][head_dim] for a coming attention backward: where it runs on one-tile kernels that hold
// whole heads, their epilogue writes what attn_delta_kernel would (the same bits), and *done is set.  o: as c; lse, delta, lse2:
// [batch][heads][seq].
struct DeltaEpilogue { const void* o; const float* lse; float *delta, *lse2; int seq, heads, head_dim; };
int launch_gemm_delta(const GemmArgs& g, const DeltaEpilogue& d, bool* done, hipStream_t st);
// Up to 8 independent problems in one launch, both operands mn-major (the weight-gradient products).
int launch_gemm_group(const GemmArgs* gs, int n, hipStream_t st);
// the same, and the gain sums of a layer's norms: in the same launch where that is of one-tile kernels, before it otherwise
int launch_gemm_group_gains(const GemmArgs* gs, int n, const GainSums& gains, hipStream_t st);
// The same for k-major products whose outputs are [tokens][heads][head_dim], with the rotary embedding
// applied in the epilogue (on the fp32 accumulators) to the problems whose bit is set in rotate_mask.
// cos, sin: [seq][head_dim / 2] fp32 (launch_rope_table); position of a row = row % seq.
struct RopeEpilogue { const float *cos, *sin; int seq, head_dim, layout; unsigned rotate_mask; };
int launch_gemm_group_rope(const GemmArgs* gs, int n, const RopeEpilogue* rope, hipStream_t st);
// g = x Wg^T, u = x Wu^T and a = silu(g) * u (from the fp32 sums) in one launch.  x [T, K] with
// leading dimension ldx, wg and wu [F, K] with ldw, g and u with ldgu, a with lda.  F % 8 == 0.
int launch_gemm_swiglu(const void* x, int64_t ldx, const void* wg, const void* wu, int64_t ldw, int64_t T, int64_t K,
                       int64_t F, void* g, void* u, int64_t ldgu, void* a, int64_t lda, hipStream_t st);
// da = dy W^T for dy [T, K] (lddy) and W stored [F, K] (w_kmajor) or [K, F] with ldw, then (dg, du) = gradient of silu(g) * u for
// the fp32 da, which is never stored.  g, u with ldgu; dg, du with ldd.  a (or null): silu(g) * u, written again, with ldd, as
// launch_swiglu_fwd_rows does.
int launch_gemm_swiglu_grad(const void* dy, int64_t lddy, const void* w, bool w_kmajor, int64_t ldw, int64_t T, int64_t K, int64_t F,
                            const void* g, const void* u, int64_t ldgu, void* dg, void* du, int64_t ldd,
                            void* a, hipStream_t st);

// Which kernels a product, or a group, of these sizes runs on: see gemm_route in dlayer.h.  Nothing is launched.
enum { GEMM_ROUTE_K_K = 0, GEMM_ROUTE_K_MN = 1, GEMM_ROUTE_MN_MN = 2 };
enum { GEMM_ROUTE_PLAIN = 0, GEMM_ROUTE_GATED_PAIR = 1, GEMM_ROUTE_GATED_GRADIENT = 2, GEMM_ROUTE_ROTARY_SPLIT = 3, GEMM_ROUTE_ROTARY_ADJACENT = 4,
       GEMM_ROUTE_ACCUMULATE = 5 };
void query_gemm_route(int operands, int epilogue, int head_dim, int cus, int n, const int64_t* M, const int64_t* N, const int64_t* K,
                      int32_t* route);

// ---- attention.hip
// workgroups that share the work of 128 keys in the dK/dV pass, on a device of `cus` compute units
int attention_bwd_pieces(int64_t B, int64_t S, int64_t Hq, int64_t Hkv, int64_t dh, int cus);
int launch_attention_fwd(const void* q, const void* k, const void* v, int64_t B, int64_t S,
                         int64_t Hq, int64_t Hkv, int64_t dh, void* o, float* lse, hipStream_t st);
size_t attention_bwd_workspace(int64_t B, int64_t S, int64_t Hq, int64_t Hkv, int64_t dh);
// the row statistics of the backward lie at the start of its workspace: delta, then lse2, [B, Hq, S] each
inline float* attention_bwd_delta(void* workspace) { return static_cast<float*>(workspace); }
inline float* attention_bwd_lse2(void* workspace, int64_t B, int64_t S, int64_t Hq) { return attention_bwd_delta(workspace) + B * Hq * S; }
int launch_attention_bwd(const void* q, const void* k, const void* v, const void* o, const void* d_o,
                         const float* lse, int64_t B, int64_t S, int64_t Hq, int64_t Hkv, int64_t dh,
                         void* dq, void* dk, void* dv, void* workspace, hipStream_t st);

// The same for q and k that were rotated (rotary embedding) after their projections: dq and dk are
// the gradients of the UNROTATED q and k, the inverse rotation being applied to the fp32 sums before
// they are rounded.  rope_cos, rope_sin: [S][dh / 2] fp32 (launch_rope_table), or null for no rotation.  stats_done: the row
// statistics are in the workspace already (launch_gemm_delta).
int launch_attention_bwd_rope(const void* q, const void* k, const void* v, const void* o, const void* d_o,
                              const float* lse, int64_t B, int64_t S, int64_t Hq, int64_t Hkv, int64_t dh,
                              void* dq, void* dk, void* dv, void* workspace, const float* rope_cos,
                              const float* rope_sin, int rope_layout, bool stats_done, hipStream_t st);

// ---- ce.hip
size_t ce_workspace(int64_t T, int64_t V);
int launch_ce(const void* logits, const int64_t* targets, int64_t T, int64_t V, float grad_scale,
              float* loss, void* dlogits, void* workspace, hipStream_t st);
// the two halves of launch_ce, for callers that walk the rows in chunks
int launch_ce_rows(const void* logits, const int64_t* targets, int64_t rows, int64_t V, float scale, float* row_loss,
                   void* dlogits, hipStream_t st);
int launch_ce_mean(const float* row_loss, int64_t T, float* loss, hipStream_t st);
// launch_ce for at most ce_static_max_rows() rows, with the per-row losses in a static device array
int64_t ce_static_max_rows();
int launch_ce_static(const void* logits, const int64_t* targets, int64_t T, int64_t V, float grad_scale,
                     float* loss, void* dlogits, hipStream_t st);

// ---- optimizer.hip
constexpr int kOptMaxTensors = 16;
// number of 16384-element chunks the tensors of a call split into (= floats of workspace the norm needs)
int64_t opt_chunks(int n, const int64_t* numel);
// *sq_norm (+)= sum over all elements of all n gradient tensors of g^2 (fp32, fixed summation order)
int launch_grad_sq_norm(int n, const void* const* g, const int64_t* numel, float* sq_norm, float* partial,
                        int accumulate, hipStream_t st);
// AdamW on n tensors; sq_norm (device, may be null): gradients are scaled by min(1, max_norm / (sqrt(*sq_norm) + 1e-6))
int launch_adamw(int n, void* const* p, const void* const* g, float* const* m, float* const* v, const int64_t* numel,
                 int64_t step, float lr, float beta1, float beta2, float eps, float weight_decay, float max_norm,
                 const float* sq_norm, hipStream_t st);

// probes.hip: synthetic issue-rate measurements (see the file's header for families and variants);
// result[4] = cycles per block per SIMD, milliseconds, shader clock in GHz, second role's cycles per op
int launch_probe(int family, int variant, int waves_per_simd, double* result, hipStream_t st);

}  // namespace dl
