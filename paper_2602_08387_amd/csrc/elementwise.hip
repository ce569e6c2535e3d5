// Memory-bound kernels of the decoder layer: RMSNorm forward/backward, rotary embedding,
// SwiGLU forward/backward, bf16 matrix transpose, embedding gather and its gradient.
// All of them move 16 bytes per lane per access (8 bf16) with consecutive lanes on
// consecutive addresses, keep a row in registers between the reduction and the write, and
// reduce with wavefront shuffles.
#include "common.h"
#include "gain_sums.h"
#include "kernels.h"

namespace dl {

// ------------------------------------------------------------------------------------------
// RMSNorm forward: one wavefront per token row, the row stays in registers.  A launch may carry the rotary table (the
// angles as cos and sin for the kernels that rotate inside another pass, the q/k projection epilogue and the attention
// backward stores) on workgroups of its own behind the rows: for small layers a launch costs more than its work (5 us
// for the table at T = 1920).
// ------------------------------------------------------------------------------------------
struct RopeTableJob { float *cs, *sn; int seq, half; double log2_base; };

// angle p * base^(-i / half) of (position p, pair i) in fp64, stored as fp32 [seq][half]
__device__ __forceinline__ void rope_table_entry(const RopeTableJob& r, int idx) {
  if (idx >= r.seq * r.half) return;
  const int p = idx / r.half, i = idx % r.half;
  const double theta = exp2(-(double)i / (double)r.half * r.log2_base);
  double s, c;
  sincos((double)p * theta, &s, &c);
  r.cs[idx] = (float)c;
  r.sn[idx] = (float)s;
}

template <int NV, bool ROPE>
__global__ __launch_bounds__(256) void rmsnorm_fwd_kernel(const bf16_t* x, const bf16_t* gamma, bf16_t* h, float* rstd,
                                                          int blocks, int64_t T, int D, float eps, const RopeTableJob rope) {
  const int b = blockIdx.x;
  if constexpr (ROPE) {
    if (b >= blocks) {
      rope_table_entry(rope, (b - blocks) * 256 + (int)threadIdx.x);
      return;
    }
  }
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)b * 4 + (threadIdx.x >> 6);
  if (row >= T) return;
  const int nvec = D >> 3;
  const bf16x8* xr = reinterpret_cast<const bf16x8*>(x + row * D);
  bf16x8 v[NV];
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = i * 64 + lane;
    if (c < nvec) {
      v[i] = xr[c];
#pragma unroll
      for (int e = 0; e < 8; ++e) { float f = (float)v[i][e]; ss += f * f; }
    }
  }
  ss = wave_sum(ss);
  const float r = 1.0f / sqrtf(ss / (float)D + eps);
  if (lane == 0) rstd[row] = r;
  bf16x8* hr = reinterpret_cast<bf16x8*>(h + row * D);
  const bf16x8* gr = reinterpret_cast<const bf16x8*>(gamma);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = i * 64 + lane;
    if (c < nvec) {
      bf16x8 g = gr[c], o;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = (bf16_t)((float)v[i][e] * r * (float)g[e]);
      hr[c] = o;
    }
  }
}

template <bool ROPE>
static int launch_rms_fwd(const void* x, const void* gamma, int64_t T, int64_t D, float eps, void* h, float* rstd,
                          const RopeTableJob& rope, hipStream_t st) {
  const int nv = (int)((D / 8 + 63) / 64);
  const int64_t blocks = (T + 3) / 4, table = ROPE ? ((int64_t)rope.seq * rope.half + 255) / 256 : 0;
  dim3 grid((unsigned)(blocks + table)), block(256);
#define RMS_FWD(NV)                                                                                               \
  hipLaunchKernelGGL((rmsnorm_fwd_kernel<NV, ROPE>), grid, block, 0, st, (const bf16_t*)x, (const bf16_t*)gamma, \
                     (bf16_t*)h, rstd, (int)blocks, T, (int)D, eps, rope)
  if (nv <= 1) RMS_FWD(1);
  else if (nv <= 2) RMS_FWD(2);
  else if (nv <= 4) RMS_FWD(4);
  else if (nv <= 8) RMS_FWD(8);
  else if (nv <= 16) RMS_FWD(16);
  else RMS_FWD(32);
#undef RMS_FWD
  return check_launch("rmsnorm_forward");
}

int launch_rmsnorm_fwd(const void* x, const void* gamma, int64_t T, int64_t D, float eps, void* h,
                       float* rstd, hipStream_t st) {
  return launch_rms_fwd<false>(x, gamma, T, D, eps, h, rstd, RopeTableJob{}, st);
}
int launch_rmsnorm_fwd_rope_table(const void* x, const void* gamma, int64_t T, int64_t D, float eps, void* h, float* rstd, float* cos,
                                  float* sin, int64_t seq, int64_t head_dim, float base, hipStream_t st) {
  return launch_rms_fwd<true>(x, gamma, T, D, eps, h, rstd, RopeTableJob{cos, sin, (int)seq, (int)(head_dim / 2), log2((double)base)}, st);
}

// ------------------------------------------------------------------------------------------
// RMSNorm backward.  TPR threads share a row, one 16-byte vector each (two beyond 8192 columns); a workgroup of RG such
// groups walks rows with a grid stride, two at a time (one beyond 8192 columns), writes dx and keeps the gain-gradient sums of its columns in
// registers, folds its groups through LDS and writes one fp32 partial row; a second kernel sums the partial
// rows.  Bound by HBM (8 bytes per element with the residual gradient).  A thread holds one vector of a row where a wave
// held the whole row, in 100 to 128 registers for its two rows, and the residual row is asked for together with the
// others; rows of any width are read once.  h, if asked for, is the forward's output again (the same bits: the same three
// factors in the same order), at the cost of its stores, where a pass of its own reads x again (5.8 us and a launch for the
// two norms of 1920 x 1152).
// ------------------------------------------------------------------------------------------
template <int TPR, int NV, int RG>
__global__ __launch_bounds__(TPR * RG) void rmsnorm_bwd_kernel(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ gamma, const float* __restrict__ rstd,
    const bf16_t* __restrict__ dh, const bf16_t* dres, bf16_t* dx, bf16_t* __restrict__ h, float* __restrict__ partial,
    int64_t T, int D) {
  constexpr int WPR = TPR / 64, U = NV == 1 ? 2 : 1;
  __shared__ float red[2][RG][U][WPR];
  __shared__ float fold[RG > 1 ? RG * TPR * NV * 8 : 1];
  const int rg = threadIdx.x / TPR, tr = threadIdx.x % TPR, lane = threadIdx.x & 63, wave = tr >> 6;
  const int nvec = D >> 3;
  float dg[NV][8], gv[NV][8];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = i * TPR + tr;
    bf16x8 g = {0, 0, 0, 0, 0, 0, 0, 0};
    if (c < nvec) g = reinterpret_cast<const bf16x8*>(gamma)[c];
    unpack8(g, gv[i]);
#pragma unroll
    for (int e = 0; e < 8; ++e) dg[i][e] = 0.f;
  }
  const float inv_d = 1.0f / (float)D;
  const int64_t stride = (int64_t)gridDim.x * RG;
  int par = 0;
  for (int64_t base = (int64_t)blockIdx.x * RG; base < T; base += U * stride, par ^= 1) {
    bf16x8 xv[U][NV], dv[U][NV], rv[U][NV];
    float r[U], dot[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t row = base + u * stride + rg;
      const bool row_ok = row < T;
      r[u] = row_ok ? rstd[row] : 0.f;
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int c = i * TPR + tr;
        const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
        xv[u][i] = dv[u][i] = rv[u][i] = zero;
        if (row_ok && c < nvec) {
          xv[u][i] = reinterpret_cast<const bf16x8*>(x + row * D)[c];
          dv[u][i] = reinterpret_cast<const bf16x8*>(dh + row * D)[c];
          if (dres) rv[u][i] = reinterpret_cast<const bf16x8*>(dres + row * D)[c];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      dot[u] = 0.f;
#pragma unroll
      for (int i = 0; i < NV; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float xh = (float)xv[u][i][e] * r[u], d = (float)dv[u][i][e];
          dg[i][e] += d * xh;
          dot[u] += d * gv[i][e] * xh;
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
      for (int u = 0; u < U; ++u) dot[u] += __shfl_xor(dot[u], o, 64);
    if constexpr (WPR > 1) {
      // two sets of slots in turn: a wave writes a set again only after a barrier that every reader of it has passed
      if (lane == 0) {
#pragma unroll
        for (int u = 0; u < U; ++u) red[par][rg][u][wave] = dot[u];
      }
      __syncthreads();
#pragma unroll
      for (int u = 0; u < U; ++u) {
        dot[u] = red[par][rg][u][0];
#pragma unroll
        for (int w = 1; w < WPR; ++w) dot[u] += red[par][rg][u][w];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t row = base + u * stride + rg;
      if (row >= T) continue;
      const float mean = dot[u] * inv_d;
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int c = i * TPR + tr;
        if (c < nvec) {
          bf16x8 o;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float xh = (float)xv[u][i][e] * r[u];
            o[e] = (bf16_t)(r[u] * ((float)dv[u][i][e] * gv[i][e] - xh * mean) + (float)rv[u][i][e]);
          }
          reinterpret_cast<bf16x8*>(dx + row * D)[c] = o;
          if (h) {
#pragma unroll
            for (int e = 0; e < 8; ++e) o[e] = (bf16_t)((float)xv[u][i][e] * r[u] * gv[i][e]);
            reinterpret_cast<bf16x8*>(h + row * D)[c] = o;
          }
        }
      }
    }
  }
  if constexpr (RG > 1) {
#pragma unroll
    for (int i = 0; i < NV; ++i)
#pragma unroll
      for (int e = 0; e < 8; ++e) fold[(rg * NV + i) * TPR * 8 + tr * 8 + e] = dg[i][e];
    __syncthreads();
    for (int c = threadIdx.x; c < D; c += RG * TPR) {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < RG; ++w) s += fold[w * NV * TPR * 8 + c];
      partial[(int64_t)blockIdx.x * D + c] = s;
    }
  } else {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = i * TPR + tr;
      if (c < nvec) {
        f32x4* p = reinterpret_cast<f32x4*>(partial + (int64_t)blockIdx.x * D) + c * 2;
        p[0] = f32x4{dg[i][0], dg[i][1], dg[i][2], dg[i][3]};
        p[1] = f32x4{dg[i][4], dg[i][5], dg[i][6], dg[i][7]};
      }
    }
  }
}

__global__ __launch_bounds__(1024) void colsum_partials_kernel(const GainSums s) {
  __shared__ float red[32 * 33];
  gain_sums<1024>(s, (int)blockIdx.x, red);
}

// Workgroups, i.e. partial rows: one per eight rows and at most 512, which is what the size query asks room for.
static int rms_bwd_blocks(int64_t T) {
  const int64_t b = (T + 7) / 8;
  return (int)(b < 512 ? b : 512);
}
size_t rmsnorm_bwd_workspace(int64_t T, int64_t D) { return (size_t)rms_bwd_blocks(T) * D * sizeof(float); }

// Threads per row by the width.  512 threads to a workgroup, so that two are resident on a compute unit - but 1024, two
// rows side by side, for rows of 2056 to 4096 columns while every compute unit has at most one (D 4096, us, 512 / 1024
// threads: T 2048 17.7 / 16.2, T 4096 25.3 / 27.6).  With 256 threads and up to 1024 partial rows: D 2048 T 8192 27.7
// against 24.8, D 768 T 8192 14.3 against 13.0.
int launch_rmsnorm_bwd_rows(const void* x, const void* gamma, const float* rstd, const void* dh,
                            const void* dres, int64_t T, int64_t D, void* dx, void* h, void* workspace, hipStream_t st) {
  const int nb = rms_bwd_blocks(T);
  float* partial = (float*)workspace;
#define RMS_BWD(TPR, NV, RG)                                                                                   \
  hipLaunchKernelGGL((rmsnorm_bwd_kernel<TPR, NV, RG>), dim3(nb), dim3(TPR * RG), 0, st, (const bf16_t*)x,      \
                     (const bf16_t*)gamma, rstd, (const bf16_t*)dh, (const bf16_t*)dres, (bf16_t*)dx, (bf16_t*)h, partial, T, (int)D)
  if (D <= 512) RMS_BWD(64, 1, 8);
  else if (D <= 1024) RMS_BWD(128, 1, 4);
  else if (D <= 2048) RMS_BWD(256, 1, 2);
  else if (D <= 4096 && nb <= 256) RMS_BWD(512, 1, 2);
  else if (D <= 4096) RMS_BWD(512, 1, 1);
  else if (D <= 8192) RMS_BWD(1024, 1, 1);
  else RMS_BWD(1024, 2, 1);
#undef RMS_BWD
  return check_launch("rmsnorm_backward");
}

GainSums rmsnorm_bwd_gain_sums(const void* ws_a, void* dgamma_a, const void* ws_b, void* dgamma_b, int64_t T, int64_t D, int accumulate) {
  return {(const float*)ws_a, (const float*)ws_b, dgamma_a, dgamma_b, rms_bwd_blocks(T), (int)D, accumulate};
}
int launch_gain_sums(const GainSums& s, hipStream_t st) {
  hipLaunchKernelGGL(colsum_partials_kernel, dim3((unsigned)gain_sum_blocks(s)), dim3(1024), 0, st, s);
  return check_launch("rmsnorm_backward(dgamma)");
}
int launch_rmsnorm_bwd_gain(const void* ws_a, void* dgamma_a, const void* ws_b, void* dgamma_b, int64_t T, int64_t D,
                            int accumulate, hipStream_t st) {
  return launch_gain_sums(rmsnorm_bwd_gain_sums(ws_a, dgamma_a, ws_b, dgamma_b, T, D, accumulate), st);
}

int launch_rmsnorm_bwd(const void* x, const void* gamma, const float* rstd, const void* dh,
                       const void* dres, int64_t T, int64_t D, void* dx, void* dgamma,
                       int accumulate, void* workspace, hipStream_t st) {
  if (int rc = launch_rmsnorm_bwd_rows(x, gamma, rstd, dh, dres, T, D, dx, nullptr, workspace, st)) return rc;
  return launch_rmsnorm_bwd_gain(workspace, dgamma, nullptr, nullptr, T, D, accumulate, st);
}

// ------------------------------------------------------------------------------------------
// Rotary embedding, in place.  One block per token: the first head_dim/2 threads evaluate the
// angle p * base^(-2i/dh) and its sine/cosine in fp64 (positions reach 8191 rad, where fp32
// range reduction is not accurate enough), park them in LDS as fp32, then every thread rotates
// pairs of all heads of that token.
// ------------------------------------------------------------------------------------------
// rotates all heads of one token row zt ([n_heads, head_dim]) with the angles parked in cs / sn
__device__ __forceinline__ void rope_rotate_row(bf16_t* zt, const float* cs, const float* sn, int n_heads,
                                                int head_dim, int layout) {
  const int half = head_dim >> 1;
  if (layout == 0) {
    // pairs (i, i + half): handle 8 consecutive i per thread
    const int groups = half >> 3;  // per head
    for (int w = threadIdx.x; w < n_heads * groups; w += blockDim.x) {
      const int hd = w / groups, i0 = (w % groups) << 3;
      bf16x8* pa = reinterpret_cast<bf16x8*>(zt + hd * head_dim + i0);
      bf16x8* pb = reinterpret_cast<bf16x8*>(zt + hd * head_dim + half + i0);
      bf16x8 a = *pa, b = *pb, oa, ob;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float c = cs[i0 + e], s = sn[i0 + e], fa = (float)a[e], fb = (float)b[e];
        oa[e] = (bf16_t)(fa * c - fb * s);
        ob[e] = (bf16_t)(fa * s + fb * c);
      }
      *pa = oa;
      *pb = ob;
    }
  } else {
    const int groups = head_dim >> 3;
    for (int w = threadIdx.x; w < n_heads * groups; w += blockDim.x) {
      const int hd = w / groups, e0 = (w % groups) << 3;
      bf16x8* pz = reinterpret_cast<bf16x8*>(zt + hd * head_dim + e0);
      bf16x8 v = *pz, o;
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const int i = (e0 + e) >> 1;
        const float c = cs[i], s = sn[i], fa = (float)v[e], fb = (float)v[e + 1];
        o[e] = (bf16_t)(fa * c - fb * s);
        o[e + 1] = (bf16_t)(fa * s + fb * c);
      }
      *pz = o;
    }
  }
}

__global__ __launch_bounds__(256) void rope_kernel(bf16_t* z, int seq, int n_heads, int head_dim, double log2_base, int layout,
                                                   int inverse) {
  __shared__ float cs[64], sn[64];
  const int64_t tok = blockIdx.x;
  const int p = (int)(tok % seq);
  const int half = head_dim >> 1;
  if ((int)threadIdx.x < half) {
    const double theta = exp2(-2.0 * (double)threadIdx.x / (double)head_dim * log2_base);
    double s, c;
    sincos((double)p * theta, &s, &c);
    cs[threadIdx.x] = (float)c;
    sn[threadIdx.x] = inverse ? -(float)s : (float)s;
  }
  __syncthreads();
  rope_rotate_row(z + tok * (int64_t)n_heads * head_dim, cs, sn, n_heads, head_dim, layout);
}

int launch_rope(void* z, int64_t batch, int64_t seq, int64_t n_heads, int64_t head_dim,
                float base, int layout, int inverse, hipStream_t st) {
  hipLaunchKernelGGL(rope_kernel, dim3((unsigned)(batch * seq)), dim3(256), 0, st, (bf16_t*)z, (int)seq,
                     (int)n_heads, (int)head_dim, log2((double)base), layout, inverse);
  return check_launch("rope_apply");
}

// The angles as a table, one thread per (position, pair).
__global__ __launch_bounds__(256) void rope_table_kernel(const RopeTableJob r) { rope_table_entry(r, blockIdx.x * 256 + threadIdx.x); }

int launch_rope_table(float* cos, float* sin, int64_t seq, int64_t head_dim, float base, hipStream_t st) {
  const int64_t n = seq * (head_dim / 2);
  hipLaunchKernelGGL(rope_table_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st,
                     (RopeTableJob{cos, sin, (int)seq, (int)(head_dim / 2), log2((double)base)}));
  return check_launch("rope table");
}

// ------------------------------------------------------------------------------------------
// SwiGLU
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void swiglu_fwd_kernel(const bf16x8* __restrict__ g,
                                                         const bf16x8* __restrict__ u,
                                                         bf16x8* __restrict__ a, int64_t nvec) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nvec;
       i += (int64_t)gridDim.x * blockDim.x) {
    bf16x8 gv = g[i], uv = u[i], o;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float z = (float)gv[e];
      o[e] = (bf16_t)(z * logistic(z) * (float)uv[e]);
    }
    a[i] = o;
  }
}

__global__ __launch_bounds__(256) void swiglu_bwd_kernel(const bf16x8* g, const bf16x8* u,
                                                         const bf16x8* __restrict__ da, bf16x8* dg,
                                                         bf16x8* du, int64_t nvec) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nvec;
       i += (int64_t)gridDim.x * blockDim.x) {
    bf16x8 gv = g[i], uv = u[i], dv = da[i], og, ou;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float z = (float)gv[e], d = (float)dv[e];
      const float s = logistic(z);
      og[e] = (bf16_t)(d * (float)uv[e] * s * (1.0f + z * (1.0f - s)));
      ou[e] = (bf16_t)(d * z * s);
    }
    dg[i] = og;
    du[i] = ou;
  }
}

// Row variant: g, u are [rows, cols] with leading dimension ld_gu, a with ld_p (the layer keeps it with padded
// rows).  One row per workgroup at a time.
constexpr int SW_U = 4;   // 16-byte vectors per thread in flight
__device__ __forceinline__ bf16x8 swiglu_vec(bf16x8 gv, bf16x8 uv) {
  bf16x8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float z = (float)gv[e];
    o[e] = (bf16_t)(z * logistic(z) * (float)uv[e]);
  }
  return o;
}
__global__ __launch_bounds__(256) void swiglu_fwd_rows_kernel(const bf16_t* __restrict__ g, const bf16_t* __restrict__ u,
                                                              bf16_t* __restrict__ a, int rows, int cols_vec,
                                                              int64_t ld_gu, int64_t ld_p) {
  for (int r = blockIdx.x; r < rows; r += gridDim.x) {
    const bf16x8* gr = reinterpret_cast<const bf16x8*>(g + r * ld_gu);
    const bf16x8* ur = reinterpret_cast<const bf16x8*>(u + r * ld_gu);
    bf16x8* ar = reinterpret_cast<bf16x8*>(a + r * ld_p);
    for (int i0 = threadIdx.x; i0 < cols_vec; i0 += 256 * SW_U) {
      bf16x8 gv[SW_U], uv[SW_U];
#pragma unroll
      for (int q = 0; q < SW_U; ++q) {
        const int i = i0 + q * 256;
        if (i < cols_vec) { gv[q] = __builtin_nontemporal_load(gr + i); uv[q] = __builtin_nontemporal_load(ur + i); }
      }
#pragma unroll
      for (int q = 0; q < SW_U; ++q) {
        const int i = i0 + q * 256;
        if (i < cols_vec) ar[i] = swiglu_vec(gv[q], uv[q]);
      }
    }
  }
}

static unsigned ew_blocks(int64_t nvec) {
  int64_t b = (nvec + 255) / 256;
  return (unsigned)(b < 256 * 16 ? (b > 0 ? b : 1) : 256 * 16);
}

int launch_swiglu_fwd(const void* g, const void* u, int64_t n, void* a, hipStream_t st) {
  hipLaunchKernelGGL(swiglu_fwd_kernel, dim3(ew_blocks(n / 8)), dim3(256), 0, st, (const bf16x8*)g,
                     (const bf16x8*)u, (bf16x8*)a, n / 8);
  return check_launch("swiglu_forward");
}
int launch_swiglu_bwd(const void* g, const void* u, const void* da, int64_t n, void* dg, void* du,
                      hipStream_t st) {
  hipLaunchKernelGGL(swiglu_bwd_kernel, dim3(ew_blocks(n / 8)), dim3(256), 0, st, (const bf16x8*)g,
                     (const bf16x8*)u, (const bf16x8*)da, (bf16x8*)dg, (bf16x8*)du, n / 8);
  return check_launch("swiglu_backward");
}

int launch_swiglu_fwd_rows(const void* g, const void* u, int64_t rows, int64_t cols, int64_t ld_gu, void* a,
                           int64_t ld_a, hipStream_t st) {
  hipLaunchKernelGGL(swiglu_fwd_rows_kernel, dim3((unsigned)(rows < 8192 ? rows : 8192)), dim3(256), 0, st,
                     (const bf16_t*)g, (const bf16_t*)u, (bf16_t*)a, (int)rows, (int)(cols / 8), ld_gu, ld_a);
  return check_launch("swiglu_forward(rows)");
}
// ------------------------------------------------------------------------------------------
// bf16 transpose: out[c][r] = in[r][c], 64x64 tiles through LDS (16-byte global accesses on
// both sides).  R and C are multiples of 64.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ void transpose_tile(const bf16_t* __restrict__ in, bf16_t* __restrict__ out, int64_t C,
                                               int64_t ld_out, int64_t r0, int64_t c0) {
  __shared__ bf16_t tile[64][66];
  const int t = threadIdx.x;
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const int idx = it * 256 + t;         // 512 vectors of 8
    const int r = idx >> 3, cv = (idx & 7) << 3;
    bf16x8 v = *reinterpret_cast<const bf16x8*>(in + (r0 + r) * C + c0 + cv);
#pragma unroll
    for (int e = 0; e < 8; ++e) tile[r][cv + e] = v[e];
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const int idx = it * 256 + t;
    const int c = idx >> 3, rv = (idx & 7) << 3;
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = tile[rv + e][c];
    *reinterpret_cast<bf16x8*>(out + (c0 + c) * ld_out + r0 + rv) = v;
  }
}

__global__ __launch_bounds__(256) void transpose_kernel(const bf16_t* __restrict__ in,
                                                        bf16_t* __restrict__ out, int64_t R,
                                                        int64_t C, int64_t ld_out) {
  transpose_tile(in, out, C, ld_out, (int64_t)blockIdx.y * 64, (int64_t)blockIdx.x * 64);
}

// Several transposes in one launch (the seven weights of a layer: for small layers each launch costs
// more than its copy).  The argument block is only read with compile-time indices.
struct TransposeGroup {
  const bf16_t* in[kMaxTransposeGroup];
  bf16_t* out[kMaxTransposeGroup];
  int R[kMaxTransposeGroup], C[kMaxTransposeGroup];
  int64_t ld_out[kMaxTransposeGroup];
  int tile_start[kMaxTransposeGroup + 1];
  int n;
};
__global__ __launch_bounds__(256) void transpose_group_kernel(const TransposeGroup g) {
  const int id = blockIdx.x;
  const bf16_t* in = g.in[0];
  bf16_t* out = g.out[0];
  int C = g.C[0], start = 0;
  int64_t ld_out = g.ld_out[0];
#pragma unroll
  for (int i = 1; i < kMaxTransposeGroup; ++i)
    if (i < g.n && id >= g.tile_start[i]) { in = g.in[i]; out = g.out[i]; C = g.C[i]; ld_out = g.ld_out[i]; start = g.tile_start[i]; }
  const int tiles_x = C / 64, tl = id - start;
  transpose_tile(in, out, C, ld_out, (int64_t)(tl / tiles_x) * 64, (int64_t)(tl % tiles_x) * 64);
}

int launch_transpose_group(const TransposeJob* jobs, int n, hipStream_t st) {
  if (n < 1 || n > kMaxTransposeGroup) return fail(-1, "transpose group: 1..%d matrices, got %d", kMaxTransposeGroup, n);
  TransposeGroup g{};
  g.n = n;
  for (int i = 0; i < n; ++i) {
    g.in[i] = (const bf16_t*)jobs[i].in;
    g.out[i] = (bf16_t*)jobs[i].out;
    g.R[i] = (int)jobs[i].R;
    g.C[i] = (int)jobs[i].C;
    g.ld_out[i] = jobs[i].ld_out;
    g.tile_start[i + 1] = g.tile_start[i] + (int)((jobs[i].R / 64) * (jobs[i].C / 64));
  }
  hipLaunchKernelGGL(transpose_group_kernel, dim3((unsigned)g.tile_start[n]), dim3(256), 0, st, g);
  return check_launch("transpose group");
}

int launch_transpose(const void* in, void* out, int64_t R, int64_t C, int64_t ld_out, hipStream_t st) {
  hipLaunchKernelGGL(transpose_kernel, dim3((unsigned)(C / 64), (unsigned)(R / 64)), dim3(256), 0,
                     st, (const bf16_t*)in, (bf16_t*)out, R, C, ld_out);
  return check_launch("transpose");
}

// ------------------------------------------------------------------------------------------
// Embedding gather and its gradient.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void embed_fwd_kernel(const bf16_t* __restrict__ table,
                                                        const int64_t* __restrict__ ids,
                                                        bf16_t* __restrict__ x0, int64_t V, int D) {
  const int64_t t = blockIdx.x;
  int64_t id = ids[t];
  const bool ok = id >= 0 && id < V;
  const bf16x8* src = reinterpret_cast<const bf16x8*>(table + (ok ? id : 0) * D);
  bf16x8* dst = reinterpret_cast<bf16x8*>(x0 + t * D);
  bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int c = threadIdx.x; c < (D >> 3); c += blockDim.x) dst[c] = ok ? src[c] : zero;
}

int launch_embed_fwd(const void* table, const int64_t* ids, int64_t T, int64_t V, int64_t D,
                     void* x0, hipStream_t st) {
  hipLaunchKernelGGL(embed_fwd_kernel, dim3((unsigned)T), dim3(256), 0, st, (const bf16_t*)table,
                     ids, (bf16_t*)x0, V, (int)D);
  return check_launch("embed_forward");
}

// ------------------------------------------------------------------------------------------
// Embedding gradient dtable[v] = sum of the rows dx0[t] with ids[t] == v, deterministic and without
// floating-point atomics.  The tokens of every id are gathered into a list (integer atomics: which slot
// a token gets depends on scheduling, the SET of tokens in a list does not), the list is sorted, and
// the rows are summed by a fixed assignment of ranks to partial sums.  So the result is bitwise
// reproducible.
//   count[v]   tokens with id v; slot[t] = the token's place among them      (embed_count_kernel)
//   start[v]   first slot of id v's segment of list                          (embed_segments_kernel)
//   list[...]  token indices grouped by id, slot[t] = position of t in list  (embed_fill_kernel)
//   the segments of more than 512 tokens brought into order, beyond 131072 tokens only  (embed_sort_kernel)
// Then one launch sums the rows with tokens, ids with few, with some and with many of them on workgroups of their own
// (T = 8192, V = 128256, D = 4096, Zipf ids: 53 us where three launches took 109), and another zeroes the rows
// without (0.97 of 1.05 GB, 165 us, 6.3 TB/s: the floor of the whole; both in one launch, side by side, take longer
// than one after the other).  The hot counters - the commonest word's, the cursor - take one atomic per wavefront or
// workgroup, not one per token: same-address atomics are served one after the other and cost 16 to 20 us in each of
// three kernels at that shape, 5 us now.
// ------------------------------------------------------------------------------------------
constexpr int kEmbThreads = 512;
constexpr int kEmbVecs = 16;        // 16-byte column vectors per workgroup (128 columns) of a heavy id
constexpr int kEmbGroups = kEmbThreads / kEmbVecs;   // partial sums of a heavy id: the row of rank r goes to sum r % 32
constexpr int kEmbLight = 4;        // ids with at most this many tokens: one wavefront sums the row, tokens sorted in registers
constexpr int kEmbMedium = 64;      // up to here one workgroup sums the row; beyond, one per 128 columns
constexpr int kEmbListMax = 4096;   // sorted tokens held in LDS at a time
constexpr int kEmbWordsMax = 4096;  // 32-bit words of the sorting bitmap: 131072 tokens at a time
constexpr int kEmbBitmapTokens = kEmbWordsMax * 32;
constexpr int kEmbSegIds = 4096;    // ids per workgroup of embed_segments_kernel

__global__ __launch_bounds__(256) void embed_zero_ints_kernel(int* p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = 0;
}

// One atomic per distinct id of a wavefront: its first lane with the id adds their number, the others take their
// place behind its answer.
__global__ __launch_bounds__(256) void embed_count_kernel(const int64_t* __restrict__ ids, int T, int64_t V, int* count,
                                                          int* __restrict__ slot) {
  const int t = blockIdx.x * 256 + threadIdx.x, lane = threadIdx.x & 63;
  const int64_t id64 = t < T ? ids[t] : -1;
  const bool ok = id64 >= 0 && id64 < V;
  const int id = ok ? (int)id64 : -1;
  unsigned long long left = __ballot(ok);
  unsigned long long mine = 0;
  while (left) {
    const int first = __builtin_ctzll(left);
    const unsigned long long same = __ballot(ok && id == __builtin_amdgcn_readlane(id, first));
    if ((same >> lane) & 1) mine = same;
    left &= ~same;
  }
  // all leaders' atomics go out together
  const int leader = mine ? __builtin_ctzll(mine) : lane;
  int base = 0;
  if (ok && lane == leader) base = atomicAdd(&count[id], __builtin_popcountll(mine));
  base = __shfl(base, leader, 64);
  if (t < T) slot[t] = ok ? base + __builtin_popcountll(mine & ((1ull << lane) - 1)) : -1;
}

// Sum of v over the lanes before this one; total of the wavefront in `total`.
__device__ __forceinline__ int wave_prefix(int v, int lane, int& total) {
  int incl = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int x = __shfl_up(incl, off, 64);
    if (lane >= off) incl += x;
  }
  total = __shfl(incl, 63, 64);
  return incl - v;
}

// start[v] = first slot of id v's segment of `list`.  The segments only have to be disjoint, not in id
// order, so they are handed out from a running cursor: one atomic per workgroup.  Where a segment lands depends on
// scheduling; what it holds does not.
__global__ __launch_bounds__(1024) void embed_segments_kernel(const int* __restrict__ count, int* __restrict__ start, int V,
                                                              int* cursor) {
  __shared__ int wsum[16], wbase[16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int v0 = blockIdx.x * kEmbSegIds + threadIdx.x * 4;
  int c[4], mine = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) { c[i] = v0 + i < V ? count[v0 + i] : 0; mine += c[i]; }
  int total;
  int off = wave_prefix(mine, lane, total);
  if (lane == 0) wsum[wave] = total;
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int w = 0; w < 16; ++w) { wbase[w] = run; run += wsum[w]; }
    const int base = run > 0 ? atomicAdd(cursor, run) : 0;
    for (int w = 0; w < 16; ++w) wbase[w] += base;
  }
  __syncthreads();
  off += wbase[wave];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (v0 + i < V) start[v0 + i] = off;
    off += c[i];
  }
}

__global__ __launch_bounds__(256) void embed_fill_kernel(const int64_t* __restrict__ ids, int T, const int* __restrict__ count,
                                                         const int* __restrict__ start, int* __restrict__ list,
                                                         int* __restrict__ slot, int* __restrict__ many, int most, int* n_many) {
  const int t = blockIdx.x * 256 + threadIdx.x, lane = threadIdx.x & 63;
  const int place = t < T ? slot[t] : -1;   // -1: an id outside the table
  int cls = -1, id = 0;
  if (place >= 0) {
    id = (int)ids[t];
    const int s = start[id] + place;
    list[s] = t;
    slot[t] = s;
    if (place == 0) cls = count[id] > kEmbMedium ? 1 : count[id] > kEmbLight ? 0 : -1;
  }
  // ids with more than kEmbLight tokens: the medium ones from the front of `many`, the heavy ones from its back; the order
  // does not matter (the entries are independent)
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const unsigned long long m = __ballot(cls == k);
    if (!m) continue;
    int base = 0;
    if (lane == __builtin_ctzll(m)) base = atomicAdd(n_many + k, __builtin_popcountll(m));
    base = __shfl(base, __builtin_ctzll(m), 64) + __builtin_popcountll(m & ((1ull << lane) - 1));
    if (cls == k) many[k == 0 ? base : most - 1 - base] = id;
  }
}

// Bits of the tokens [lo, lo + 32 words) with this id, from the ids themselves; eight loads per thread in flight.  Every
// thread of the workgroup calls it.
template <int NT>
__device__ __forceinline__ void embed_mark_tokens(const int64_t* __restrict__ ids, int64_t id, int lo, int T, int words, unsigned* bits) {
  const int lane = threadIdx.x & 63;
  for (int i0 = 0; i0 < words * 32; i0 += 8 * NT) {
    int64_t v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int t = lo + i0 + q * NT + (int)threadIdx.x;
      v[q] = t < T ? ids[t] : -1;   // an id that is looked for is never negative
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int i = i0 + q * NT + (int)threadIdx.x;
      const unsigned long long m = __ballot(v[q] == id);
      if ((lane & 31) == 0 && i < words * 32) bits[i >> 5] = (unsigned)(lane ? m >> 32 : m);
    }
  }
}

// Writes base + the index of every set bit, in ascending order, to out; returns their number.  The bits and, at the return,
// the list are the workgroup's: the caller puts a barrier on either side.  wsum: a word per wavefront.
template <int NT>
__device__ __forceinline__ int embed_list_bits(const unsigned* bits, int words, int base, int* out, int* wsum) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int per = (words + NT - 1) / NT, w0 = tid * per, w1 = w0 + per < words ? w0 + per : words;
  int mine = 0, total, n = 0;
  for (int w = w0; w < w1; ++w) mine += __builtin_popcount(bits[w]);
  int o = wave_prefix(mine, lane, total);
  if (lane == 0) wsum[wave] = total;
  __syncthreads();
  for (int w = 0; w < NT / 64; ++w) { if (w < wave) o += wsum[w]; n += wsum[w]; }
  for (int w = w0; w < w1; ++w) {
    unsigned m = bits[w];
    while (m) { out[o++] = base + w * 32 + __builtin_ctz(m); m &= m - 1; }
  }
  return n;
}

// Brings the token lists of more than kEmbThreads tokens into ascending order, in place, one workgroup per id, so that the
// column splits of the summing kernel need not each sort them.  Only for batches that one bitmap does not span: up to there
// the summing kernel's own bitmap costs less than this launch.  Lists of up to kEmbSortMax tokens go through a bitonic
// network in LDS, whatever the number of tokens in the batch; a longer one is rebuilt from one walk over the ids.
constexpr int kEmbSortMax = 8192;
__global__ __launch_bounds__(1024) void embed_sort_kernel(const int64_t* __restrict__ ids, const int* __restrict__ count,
                                                          const int* __restrict__ start, int* list, const int* __restrict__ many,
                                                          int most, const int* __restrict__ n_many, int T) {
  __shared__ int lst[kEmbSortMax];
  __shared__ int wsum[16];
  const int nh = n_many[1], tid = threadIdx.x;
  for (int hi = blockIdx.x; hi < nh; hi += gridDim.x) {
    const int64_t id = many[most - 1 - hi];
    const int first = start[id], L = count[id];
    if (L <= kEmbThreads) continue;
    __syncthreads();   // the list of the id before has been read
    if (L <= kEmbSortMax) {
      int n2 = 1;
      while (n2 < L) n2 <<= 1;
      for (int i = tid; i < n2; i += 1024) lst[i] = i < L ? list[first + i] : T;
      __syncthreads();
      for (int k = 2; k <= n2; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
          for (int i = tid; i < n2; i += 1024) {
            const int p = i ^ j;
            if (p > i) {
              const int x = lst[i], y = lst[p];
              if ((x > y) == ((i & k) == 0)) { lst[i] = y; lst[p] = x; }
            }
          }
          __syncthreads();
        }
      for (int i = tid; i < L; i += 1024) list[first + i] = lst[i];
    } else {
      unsigned* bits = reinterpret_cast<unsigned*>(lst);
      static_assert(kEmbWordsMax <= kEmbSortMax, "the bitmap takes the list's place");
      int done = 0;
      for (int lo = 0; lo < T; lo += kEmbBitmapTokens) {
        const int left = T - lo, words = (left < kEmbBitmapTokens ? left + 31 : kEmbBitmapTokens) >> 5;
        embed_mark_tokens<1024>(ids, id, lo, T, words, bits);
        __syncthreads();
        done += embed_list_bits<1024>(bits, words, lo, list + first + done, wsum);
        __syncthreads();   // the bits and the wavefronts' sums have been read
      }
    }
  }
}

// Rows of an id with more than kEmbMedium tokens, 128 columns per workgroup: the row of rank r in ascending token order goes
// to partial sum r % 32, whichever way the order is found.  Up to 512 tokens are ranked in LDS by counting the smaller ones.
// More come from a bitmap of the batch where one spans it: filled from the id's list, or, where there are more of them
// than the list in LDS holds, from the ids, a piece of 4096 tokens at a time (scanning the id's list anew for every
// piece took time that grew with the square of T; half of the batch one id, V 128256, us, that way and this: T 65536
// D 4096 972 / 828).  Beyond that size embed_sort_kernel has sorted the list (T 262144 D 1024 4706 / 2471; Zipf ids 1094 / 688).
__device__ __forceinline__ void embed_sum_heavy(const bf16_t* __restrict__ dx0, const int64_t* __restrict__ ids,
                                                const int* __restrict__ count, const int* __restrict__ start,
                                                const int* __restrict__ list, int64_t id, int split, bf16_t* __restrict__ dtable, int T,
                                                int D, char* lds) {
  int* lst = reinterpret_cast<int*>(lds);
  unsigned* bits = reinterpret_cast<unsigned*>(lst + kEmbListMax);
  float(*part)[kEmbVecs][8] = reinterpret_cast<float(*)[kEmbVecs][8]>(bits);   // after the last use of the bitmap
  __shared__ int wsum[kEmbThreads / 64];
  const int tid = threadIdx.x;
  const int vec = tid % kEmbVecs, grp = tid / kEmbVecs;
  const int cvec = split * kEmbVecs + vec;
  const bool col_ok = cvec < (D >> 3);
  const bf16_t* col = dx0 + (col_ok ? cvec * 8 : 0);
  const int first = start[id], L = count[id];
  const bool few = L <= kEmbThreads, sorted = !few && T > kEmbBitmapTokens;
  // the walk: over ranks of a sorted list, else over tokens
  const int end = few ? 1 : sorted ? L : T, step = few ? 1 : sorted || L > kEmbListMax ? kEmbListMax : T;
  float a[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) a[e] = 0.f;
  int done = 0;      // rows of the steps before
  for (int lo = 0; lo < end; lo += step) {
    int n = 0;
    __syncthreads();   // the list and the partial sums of the step or id before have been read
    if (few) {
      const int mine = tid < L ? list[first + tid] : 0;
      if (tid < L) reinterpret_cast<int*>(bits)[tid] = mine;
      __syncthreads();
      if (tid < L) {
        int rank = 0;
        for (int j = 0; j < L; ++j) rank += reinterpret_cast<const int*>(bits)[j] < mine;
        lst[rank] = mine;
      }
      n = L;
    } else if (sorted) {
      n = L - lo < kEmbListMax ? L - lo : kEmbListMax;
      for (int i = tid; i < n; i += kEmbThreads) lst[i] = list[first + lo + i];
    } else {
      const int left = T - lo, words = (left < step ? left + 31 : step + 31) >> 5;
      if (L > kEmbListMax) {
        embed_mark_tokens<kEmbThreads>(ids, id, lo, T, words, bits);
      } else {
        for (int w = tid; w < words; w += kEmbThreads) bits[w] = 0u;
        __syncthreads();
        for (int i = tid; i < L; i += kEmbThreads) {
          const int t = list[first + i];
          atomicOr(&bits[t >> 5], 1u << (t & 31));
        }
      }
      __syncthreads();
      n = embed_list_bits<kEmbThreads>(bits, words, lo, lst, wsum);
    }
    __syncthreads();
    if (col_ok) {
      int j = (grp - done) & (kEmbGroups - 1);
      for (; j + 7 * kEmbGroups < n; j += 8 * kEmbGroups) {   // eight rows in flight
        bf16x8 r[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) r[q] = *reinterpret_cast<const bf16x8*>(col + (int64_t)lst[j + q * kEmbGroups] * D);
#pragma unroll
        for (int q = 0; q < 8; ++q)
#pragma unroll
          for (int e = 0; e < 8; ++e) a[e] += (float)r[q][e];
      }
      for (; j < n; j += kEmbGroups) {
        const bf16x8 r0 = *reinterpret_cast<const bf16x8*>(col + (int64_t)lst[j] * D);
#pragma unroll
        for (int e = 0; e < 8; ++e) a[e] += (float)r0[e];
      }
    }
    done += n;
  }
  __syncthreads();   // the bitmap (or the unsorted list in its place) has been read
#pragma unroll
  for (int e = 0; e < 8; ++e) part[grp][vec][e] = a[e];
  __syncthreads();
  // pairwise in a fixed order, one thread per column
  if (tid < kEmbVecs * 8 && split * kEmbVecs * 8 + tid < D) {
    float q[kEmbGroups];
#pragma unroll
    for (int g = 0; g < kEmbGroups; ++g) q[g] = part[g][tid >> 3][tid & 7];
#pragma unroll
    for (int w = 1; w < kEmbGroups; w <<= 1)
#pragma unroll
      for (int g = 0; g < kEmbGroups; g += 2 * w) q[g] += q[g + w];
    dtable[id * D + split * kEmbVecs * 8 + tid] = (bf16_t)q[0];
  }
}

// rows of dtable no token points at
__global__ __launch_bounds__(256) void embed_zero_rows_kernel(const int* __restrict__ count, u32x4* __restrict__ dtable, int64_t V,
                                                              int row_vec) {
  const u32x4 z = {0, 0, 0, 0};
  for (int64_t v = blockIdx.x; v < V; v += gridDim.x) {
    if (count[v] != 0) continue;
    u32x4* row = dtable + v * row_vec;
    for (int c = threadIdx.x; c < row_vec; c += 256) row[c] = z;
  }
}

// The rows with tokens.  Workgroups [0, n_hb * n_cs): the heavy ids, column split by column split; n_mb: the medium ids;
// the rest: ids of up to kEmbLight tokens, a wavefront per token (the first of its id does the work).
__global__ __launch_bounds__(kEmbThreads, 8) void embed_grad_kernel(
    const bf16_t* __restrict__ dx0, const int64_t* __restrict__ ids, const int* __restrict__ count,
    const int* __restrict__ start, const int* __restrict__ list, const int* __restrict__ slot, const int* __restrict__ many,
    int most, const int* __restrict__ n_many, bf16_t* __restrict__ dtable, int T, int D, int n_hb, int n_cs, int n_mb) {
  extern __shared__ __attribute__((aligned(16))) char lds[];
  const int nvec = D >> 3, tid = threadIdx.x;
  int b = blockIdx.x;
  if (b < n_hb * n_cs) {
    const int nh = n_many[1];
    for (int hi = b / n_cs; hi < nh; hi += n_hb) embed_sum_heavy(dx0, ids, count, start, list, many[most - 1 - hi], b % n_cs, dtable, T, D, lds);
    return;
  }
  b -= n_hb * n_cs;
  if (b < n_mb) {
    int* tmp = reinterpret_cast<int*>(lds);
    int* lst = tmp + kEmbMedium;
    const int nm = n_many[0];
    for (int mi = b; mi < nm; mi += n_mb) {
      const int64_t id = many[mi];
      const int first = start[id], L = count[id];
      __syncthreads();   // the list of the id before has been read
      const int mine = tid < L ? list[first + tid] : 0;
      if (tid < L) tmp[tid] = mine;
      __syncthreads();
      if (tid < L) {
        int rank = 0;
        for (int j = 0; j < L; ++j) rank += tmp[j] < mine;
        lst[rank] = mine;
      }
      __syncthreads();
      for (int c = tid; c < nvec; c += kEmbThreads) {
        const bf16_t* col = dx0 + c * 8;
        float a[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) a[e] = 0.f;
        int j = 0;
        for (; j + 8 <= L; j += 8) {
          bf16x8 r[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) r[q] = *reinterpret_cast<const bf16x8*>(col + (int64_t)lst[j + q] * D);
#pragma unroll
          for (int q = 0; q < 8; ++q)
#pragma unroll
            for (int e = 0; e < 8; ++e) a[e] += (float)r[q][e];
        }
        for (; j < L; ++j) {
          const bf16x8 r0 = *reinterpret_cast<const bf16x8*>(col + (int64_t)lst[j] * D);
#pragma unroll
          for (int e = 0; e < 8; ++e) a[e] += (float)r0[e];
        }
        *reinterpret_cast<bf16x8*>(dtable + id * D + c * 8) = pack8(a);
      }
    }
    return;
  }
  b -= n_mb;
  constexpr int WPB = kEmbThreads / 64;
  const int t = b * WPB + __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  if (t >= T) return;
  // The tokens, sorted in registers, go to partial sum rank % 4, then (s0 + s1) + (s2 + s3).
  const int s = slot[t];
  if (s < 0) return;
  const int64_t id = ids[t];
  const int L = count[id];
  if (L > kEmbLight || s != start[id]) return;
  int r[kEmbLight];
#pragma unroll
  for (int i = 0; i < kEmbLight; ++i) r[i] = i < L ? list[s + i] : T;
#pragma unroll
  for (int i = 0; i < kEmbLight; ++i)       // sorting network for four keys (padding sorts last)
#pragma unroll
    for (int j = 0; j + 1 < kEmbLight - i; ++j)
      if (r[j] > r[j + 1]) { const int x = r[j]; r[j] = r[j + 1]; r[j + 1] = x; }
  static_assert(kEmbLight == 4, "one row per partial sum");
#pragma unroll 2
  for (int c = lane; c < nvec; c += 64) {
    bf16x8 v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
      v[i] = zero;
      if (i < L) v[i] = *reinterpret_cast<const bf16x8*>(dx0 + (int64_t)r[i] * D + c * 8);
    }
    bf16x8 o;
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (bf16_t)(((float)v[0][e] + (float)v[1][e]) + ((float)v[2][e] + (float)v[3][e]));
    *reinterpret_cast<bf16x8*>(dtable + id * D + c * 8) = o;
  }
}

// count[V], the counters of medium and heavy ids and the segment cursor (padded to 4 ints), start[V], list[T], slot[T],
// many[T / 5 + 1]
size_t embed_bwd_workspace(int64_t T, int64_t V) { return (size_t)(2 * V + 4 + 2 * T + T / (kEmbLight + 1) + 1) * sizeof(int); }

int launch_embed_bwd(const void* dx0, const int64_t* ids, int64_t T, int64_t V, int64_t D,
                     void* dtable, void* workspace, hipStream_t st) {
  int* count = (int*)workspace;
  int* n_many = count + V;
  int* start = n_many + 4;
  int* list = start + V;
  int* slot = list + T;
  int* many = slot + T;
  const int64_t most = T / (kEmbLight + 1) + 1;
  const unsigned tb = (unsigned)((T + 255) / 256);
  const int64_t zn = V + 4, zb = (zn + 255) / 256;
  hipLaunchKernelGGL(embed_zero_ints_kernel, dim3((unsigned)(zb < 2048 ? zb : 2048)), dim3(256), 0, st, count, zn);
  if (int rc = check_launch("embed_backward(clear)")) return rc;
  hipLaunchKernelGGL(embed_count_kernel, dim3(tb), dim3(256), 0, st, ids, (int)T, V, count, slot);
  if (int rc = check_launch("embed_backward(count)")) return rc;
  hipLaunchKernelGGL(embed_segments_kernel, dim3((unsigned)((V + kEmbSegIds - 1) / kEmbSegIds)), dim3(1024), 0, st, (const int*)count,
                     start, (int)V, n_many + 2);
  if (int rc = check_launch("embed_backward(segments)")) return rc;
  hipLaunchKernelGGL(embed_fill_kernel, dim3(tb), dim3(256), 0, st, ids, (int)T, (const int*)count, (const int*)start, list, slot,
                     many, (int)most, n_many);
  if (int rc = check_launch("embed_backward(fill)")) return rc;
  if (T > kEmbBitmapTokens) {
    const int64_t lists = T / (kEmbThreads + 1);
    hipLaunchKernelGGL(embed_sort_kernel, dim3((unsigned)(lists < 1024 ? lists : 1024)), dim3(1024), 0, st, ids, (const int*)count,
                       (const int*)start, list, (const int*)many, (int)most, (const int*)n_many, (int)T);
    if (int rc = check_launch("embed_backward(sort)")) return rc;
  }
  // Half of the chip's 1024 workgroup slots for the heavy ids, as many for the medium ones; a workgroup that finds no id
  // ends at once.
  const int64_t cs = (D / 8 + kEmbVecs - 1) / kEmbVecs, max_heavy = T / (kEmbMedium + 1);
  int64_t hb = 512 / cs > 0 ? 512 / cs : 1, mb = most < 512 ? most : 512;
  if (hb > max_heavy) hb = max_heavy;
  const int64_t lb = (T + kEmbThreads / 64 - 1) / (kEmbThreads / 64);
  constexpr size_t lds = kEmbListMax * sizeof(int) + (kEmbWordsMax > kEmbThreads * 8 ? kEmbWordsMax : kEmbThreads * 8) * 4;
  static std::atomic<unsigned long long> lds_done{0};
  if (int rc = reserve_lds(embed_grad_kernel, lds, lds_done, "embed_backward")) return rc;
  hipLaunchKernelGGL(embed_grad_kernel, dim3((unsigned)(hb * cs + mb + lb)), dim3(kEmbThreads), lds, st, (const bf16_t*)dx0, ids,
                     (const int*)count, (const int*)start, (const int*)list, (const int*)slot, (const int*)many, (int)most,
                     (const int*)n_many, (bf16_t*)dtable, (int)T, (int)D, (int)hb, (int)cs, (int)mb);
  if (int rc = check_launch("embed_backward")) return rc;
  hipLaunchKernelGGL(embed_zero_rows_kernel, dim3((unsigned)(V < 16384 ? V : 16384)), dim3(256), 0, st, (const int*)count,
                     (u32x4*)dtable, V, (int)(D / 8));
  return check_launch("embed_backward(zero)");
}

}  // namespace dl
