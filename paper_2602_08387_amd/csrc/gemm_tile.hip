// bf16 GEMM for problems that do not fill the chip with 256 x 256 tiles: one 128 x 256, 128 x 128 or 64 x 64 tile per
// workgroup.  Same operand layouts, same MFMA, same order of summation as the persistent kernel (gemm.hip): a
// product has the same bits on either.
//
// What bounds it: a CU works on one or two tiles, so nothing covers what a K-step serialises.  With four waves, a
// two-stage ring and its loads and fragment reads in bunches around the barrier a 128 x 128 tile paid 0.77 us per K-step
// of 64 (T = 1920, K = 6272, N = 1152: 68 us), of which its MFMAs are 0.21 us and its loads, 16 cycles each at the
// address unit, 0.22.  Measured on the way: a four-stage ring alone changes nothing; eight waves of 64 x 32 0.48;
// reads and loads between the rows of MFMAs, half a K-step ahead, 0.40 (44 us).  A 64 x 64 tile takes 0.25 us, four
// times the tiles to fill the chip with (T = 1000, K = 2048, N = 1024: 25 -> 9 us); a 128 x 256 tile 0.62 to 0.75
// (T = 8192, K = 4096, N = 768: 64 -> 50 us).  Full rounds of 256 x 256 tiles stay on the persistent kernel: a quarter
// fewer loads per flop, and its epilogue under the next tile's main loop.
//
// The epilogue passes the fp32 sums through LDS (the ring is free by then), so every fused epilogue is an
// element-wise function of rows: residual or accumulation, rotary embedding (both members of a pair lie in the
// tile), gated pair, activation gradient.
#include "gemm_core.h"

namespace dl {

// Operand fragments of one wave from an LDS tile: F blocks of 16 rows (the M/N index) from row0 on, k-substep kk.
// The reads are assembly (for the builtins the compiler waits for the loads in flight, which it cannot tell from what is read)
// and not counted by the compiler: consumers sit behind wait_reads().
template <int R, bool KMAJOR, int F>
struct FragReader {
  uint32_t at[KMAJOR ? 2 : F];
  __device__ __forceinline__ void init(const char* tile, int row0, int lane) {
    const uint32_t base = (uint32_t)(uintptr_t)(LDS_PTR(char))(const_cast<char*>(tile));
    if constexpr (KMAJOR) {
      const int row = row0 + (lane & 15);
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) at[kk] = base + row * (BK * 2) + (((kk * 4 + (lane >> 4)) ^ ((row >> 1) & 7)) << 4);
    } else {
      const int grp = lane >> 4, e = (lane & 15) >> 2, g = lane & 3, krow = (grp << 3) + e;
      const int f = TileLoader<R, false, 1>::mn_swz(krow);   // same for krow + 4 and krow + 32
#pragma unroll
      for (int j = 0; j < F; ++j) {
        const int col = row0 + j * 16 + (g << 2);
        at[j] = base + krow * (R * 2) + ((((col >> 3) ^ f) << 4) | ((col & 7) << 1));
      }
    }
  }
  template <int KKS, int J>
  __device__ __forceinline__ void read(bf16x8 (&v)[F], uint32_t stage) const {
    if constexpr (KMAJOR) {
      asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v[J]) : "v"(at[KKS] + stage), "n"(J * 16 * BK * 2));
    } else {
      bf16x4 lo, hi;
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(at[J] + stage), "n"(KKS * 32 * R * 2));
      asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(at[J] + stage), "n"(KKS * 32 * R * 2 + 4 * R * 2));
      v[J].lo = lo;
      v[J].hi = hi;
    }
  }
};

// waits for this wave's LDS reads and ties the fragments to that wait
template <int FA, int FB>
__device__ __forceinline__ void wait_reads(bf16x8 (&a)[FA], bf16x8 (&b)[FB]) {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
  for (int j = 0; j < FA; ++j) asm volatile("" : "+v"(a[j]));
#pragma unroll
  for (int j = 0; j < FB; ++j) asm volatile("" : "+v"(b[j]));
}

enum { TILE_PLAIN = 0, TILE_SWIGLU = 1, TILE_SWIGLU_GRAD = 2, TILE_ROPE = 3 };

// NST: ring stages.  EPI as the persistent kernel's epilogues.
template <bool GROUPED, int BM, int BN, int WM, int WN, bool AK, bool BKM, int NST, int EPI>
__device__ __forceinline__ void gemm_tile(const GemmGroupKArgs& grp, const GemmKArgs& one) {
  constexpr int NW = WM * WN, NT = NW * 64;
  constexpr int TM = BM / WM, TN = BN / WN, FM = TM / 16, FN = TN / 16;
  constexpr int A_BYTES = BM * BK * 2, STAGE = A_BYTES + BN * BK * 2;
  constexpr bool PAIR = EPI == TILE_SWIGLU;
  static_assert(BK == 64 && MI == 16 && KSTEP == 32, "two k-substeps per stage");
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave_m = wave % WM, wave_n = wave / WM;

  int ntiles;
  if constexpr (GROUPED) {
    ntiles = grp.tile_start[1];
#pragma unroll
    for (int i = 2; i <= MAX_GROUP; ++i) if (i <= grp.n) ntiles = grp.tile_start[i];
  } else {
    ntiles = one.tiles_m * one.tiles_n;
  }
  int pid = xcd_contiguous(blockIdx.x, ntiles);
  int tiles_m, tiles_n, K0, GM, M, N, m_base, accumulate, rope, start = 0;
  const bf16_t *a0, *b0, *res;
  bf16_t* cmat;
  int64_t lda0, ldb0, ldc;
  auto take = [&](const auto& q) {
    tiles_m = q.tiles_m; tiles_n = q.tiles_n; K0 = q.K[0]; GM = q.band_rows;
    a0 = q.a[0]; b0 = q.b[0]; lda0 = q.lda[0]; ldb0 = q.ldb[0];
    M = q.M; N = q.N; m_base = q.m_base; accumulate = q.accumulate; cmat = q.c; res = q.r; ldc = q.ldc; rope = q.rope;
  };
  LoadCursor<BM, BN, NW, AK, BKM, PAIR> cur;
  constexpr int LPW = TileLoader<BM, AK, NW>::PER_WAVE + TileLoader<BN, BKM, NW>::PER_WAVE;
  int total = 0;
  if constexpr (GROUPED) {
    int pi = 0;
#pragma unroll
    for (int i = 1; i < MAX_GROUP; ++i)
      if (i < grp.n && pid >= grp.tile_start[i]) { pi = i; start = grp.tile_start[i]; }
    take(group_problem(pi));
    pid -= start;
    cur.nseg = 1;
    total = K0 / BK;
  } else {
    take(one);
    cur.nseg = one.nseg;
    for (int s = 0; s < one.nseg; ++s) total += one.K[s] / BK;
  }
  int m0, n0;
  {
    const int band = pid / (GM * tiles_n), first_m = band * GM, band_h = min(tiles_m - first_m, GM), in_band = pid - band * GM * tiles_n;
    m0 = (first_m + in_band % band_h) * BM;
    n0 = (in_band / band_h) * BN;
    cur.left = total;
    int first = k_start(m0 + m_base, total);
    cur.seg = 0;
    if constexpr (!GROUPED) {
      for (int s = 0; s + 1 < one.nseg; ++s)
        if (cur.seg == s && first >= one.K[s] / BK) { first -= one.K[s] / BK; cur.seg = s + 1; }
    }
    cur.k = first * BK;
    if (cur.seg == 0) {
      if constexpr (PAIR) cur.open_pair(a0, b0, one.b2, lda0, ldb0, K0, M, N, m0, n0, lane);
      else cur.open_raw(a0, b0, lda0, ldb0, K0, M, N, m0, n0, lane);
    } else {
      cur.open(one, cur.seg, m0, n0, lane);
    }
  }

  FragReader<BM, AK, FM> ra;
  FragReader<BN, BKM, FN> rb;
  ra.init(smem, wave_m * TM, lane);
  rb.init(smem + A_BYTES, wave_n * TN, lane);
  f32x4 acc[FN][FM];
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

#pragma unroll
  for (int s = 0; s < NST; ++s) cur.issue_next(one, smem + s * STAGE, wave, m0, n0, lane);
  if (total >= NST) wait_vmcnt<(NST - 1) * LPW>(); else wait_vmcnt<0>();
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  // Fragments run half a K-step ahead of the MFMAs.  The MFMAs of a k-substep go out in rows (one fragment of the side
  // with more of them against all of the other side); the reads of the next substep go between its first rows and
  // half of a K-step's loads behind one of them.  In a bunch in front of the MFMAs the reads of all waves, and still
  // more the loads (16 cycles each at the address unit), queue with every wave's MFMAs behind them.
  constexpr int NF = FM + FN, ROWS = FM > FN ? FM : FN;
  bf16x8 fa[2][FM], fb[2][FN];
  auto read_one = [&](auto KS, auto F, uint32_t stage) {
    constexpr int ks = decltype(KS)::value, f = decltype(F)::value;
    if constexpr (f < FM) ra.template read<ks, f>(fa[ks], stage);
    else rb.template read<ks, f - FM>(fb[ks], stage);
  };
  auto mfma_row = [&](auto KS, auto RW) {
    constexpr int ks = decltype(KS)::value, r = decltype(RW)::value;
    if constexpr (FM > FN) {
#pragma unroll
      for (int i = 0; i < FN; ++i) acc[i][r] = mfma(fb[ks][i], fa[ks][r], acc[i][r]);
    } else {
#pragma unroll
      for (int j = 0; j < FM; ++j) acc[r][j] = mfma(fb[ks][r], fa[ks][j], acc[r][j]);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  constexpr std::integral_constant<int, 0> S0{};
  constexpr std::integral_constant<int, 1> S1{};
  static_for<0, NF>([&](auto f) { read_one(S0, f, 0u); });
  wait_reads(fa[0], fb[0]);
  uint32_t st = 0, prev = 0;             // byte offsets of the stages of K-steps t and t - 1
  for (int t = 0; t < total; ++t) {
    constexpr int RD0 = ROWS >= 4 ? 2 : 1;              // rows the reads are spread over
    static_for<0, ROWS>([&](auto r) {
      constexpr int i = decltype(r)::value;
      if constexpr (i < RD0) static_for<i * NF / RD0, (i + 1) * NF / RD0>([&](auto f) { read_one(S1, f, st); });
      mfma_row(S0, r);
      if constexpr (i == ROWS / 2 - 1) {
        if (t > 0) cur.template issue_piece<1, 2>(one, smem + prev, wave, m0, n0, lane);
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    wait_reads(fa[1], fb[1]);
    const uint32_t nx = st + STAGE == NST * STAGE ? 0 : st + STAGE;
    mfma_row(S1, S0);
    if (t + 1 < total) {
      // K-step t + 1 has landed once at most the NST - 2 younger ones are in flight; past the barrier every wave has its
      // last fragments of K-step t in registers, and its stage takes K-step t + NST
      if (t + NST <= total) wait_vmcnt<(NST - 2) * LPW>(); else wait_vmcnt<0>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    }
    // the reads go out after the last K-step too (of a stage nobody fills any more; nobody uses them)
    constexpr int RD1 = ROWS >= 4 ? 2 : 1;
    static_for<1, ROWS>([&](auto r) {
      constexpr int i = decltype(r)::value;
      if constexpr (i <= RD1) static_for<(i - 1) * NF / RD1, i * NF / RD1>([&](auto f) { read_one(S0, f, nx); });
      mfma_row(S1, r);
      if constexpr (i == (ROWS > 2 ? ROWS - 2 : 1)) {
        if (t + 1 < total) cur.template issue_piece<0, 2>(one, smem + st, wave, m0, n0, lane);
        __builtin_amdgcn_sched_barrier(0);
      }
    });
    wait_reads(fa[0], fb[0]);
    prev = st;
    st = nx;
  }

  // Epilogue.  fp32 sums to LDS, rows of BN + 4 floats (the 16 bytes more put the 16 rows a store instruction touches in
  // different banks), then 8 consecutive columns per thread along rows.
  constexpr int SP = BN + 4;
  constexpr int OC = PAIR ? BN / 2 : BN;               // output columns of the tile
  constexpr int VPR = OC / 8, NV = BM * VPR / NT;      // 8-column vectors per row and per thread
  static_assert(BM * VPR % NT == 0, "vectors deal evenly");
  float* stg = reinterpret_cast<float*>(smem);
  const int on0 = PAIR ? n0 / 2 : n0, ON = PAIR ? N / 2 : N;
  bf16x8 pre[EPI == TILE_PLAIN ? NV : 1];
  if constexpr (EPI == TILE_PLAIN) {
    const bf16_t* src = res ? res : accumulate ? cmat : nullptr;
    if (src) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int id = v * NT + (int)threadIdx.x, m = m0 + id / VPR, n = on0 + id % VPR * 8;
        const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
        pre[v] = zero;
        if (m < M && n < ON) pre[v] = *reinterpret_cast<const bf16x8*>(src + (int64_t)m * ldc + n);
      }
    }
  }
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();   // every wave is done reading the ring
  asm volatile("" ::: "memory");
#pragma unroll
  for (int i = 0; i < FN; ++i)
#pragma unroll
    for (int j = 0; j < FM; ++j)
      *reinterpret_cast<f32x4*>(stg + (wave_m * TM + j * 16 + (lane & 15)) * SP + wave_n * TN + i * 16 + (lane >> 4) * 4) = acc[i][j];
  __syncthreads();
  auto row8 = [&](int row, int col, float (&f)[8]) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(stg + row * SP + col), b = *reinterpret_cast<const f32x4*>(stg + row * SP + col + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) { f[e] = a[e]; f[e + 4] = b[e]; }
  };
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    const int id = v * NT + (int)threadIdx.x, row = id / VPR, col = id % VPR * 8;
    const int m = m0 + row, n = on0 + col;
    if (m >= M || n >= ON) continue;
    if constexpr (EPI == TILE_SWIGLU) {
      // of every 64 tile columns the first 32 are g, the next 32 u (LoadCursor PAIR)
      float g[8], u[8], a[8];
      const int gc = (col >> 5) * 64 + (col & 31);
      row8(row, gc, g);
      row8(row, gc + 32, u);
#pragma unroll
      for (int e = 0; e < 8; ++e) a[e] = g[e] * logistic(g[e]) * u[e];
      *reinterpret_cast<bf16x8*>(cmat + (int64_t)m * ldc + n) = pack8(g);
      *reinterpret_cast<bf16x8*>(one.c2 + (int64_t)m * ldc + n) = pack8(u);
      *reinterpret_cast<bf16x8*>(one.c3 + (int64_t)m * one.ldc3 + n) = pack8(a);
    } else if constexpr (EPI == TILE_SWIGLU_GRAD) {
      float d[8], z[8], u[8];
      row8(row, col, d);
      unpack8(*reinterpret_cast<const bf16x8*>(one.e1 + (int64_t)m * one.lde + n), z);
      unpack8(*reinterpret_cast<const bf16x8*>(one.e2 + (int64_t)m * one.lde + n), u);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float sg = logistic(z[e]), dz = d[e] * u[e] * sg * (1.0f + z[e] * (1.0f - sg));
        u[e] = d[e] * z[e] * sg;
        d[e] = dz;
      }
      *reinterpret_cast<bf16x8*>(cmat + (int64_t)m * ldc + n) = pack8(d);
      *reinterpret_cast<bf16x8*>(one.c2 + (int64_t)m * ldc + n) = pack8(u);
    } else {
      float f[8];
      row8(row, col, f);
      if constexpr (EPI == TILE_ROPE) {
        if (rope) {
          const int dh = grp.rope_dh, hd2 = dh >> 1, pos = (m + m_base) % grp.rope_seq, o = n % dh;
          const float* cr = grp.rope_cos + (int64_t)pos * hd2;
          const float* sr = grp.rope_sin + (int64_t)pos * hd2;
          if (grp.rope_layout == 0) {
            const bool lowh = o < hd2;
            const int idx = lowh ? o : o - hd2;
            float p[8];
            row8(row, lowh ? col + hd2 : col - hd2, p);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float c = cr[idx + e], s = sr[idx + e];
              f[e] = lowh ? rotated_first(f[e], p[e], c, s) : rotated_second(p[e], f[e], c, s);
            }
          } else {
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
              const float c = cr[(o + e) >> 1], s = sr[(o + e) >> 1], x = f[e], y = f[e + 1];
              f[e] = rotated_first(x, y, c, s);
              f[e + 1] = rotated_second(x, y, c, s);
            }
          }
        }
      } else if (res || accumulate) {
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] += (float)pre[v][e];
      }
      *reinterpret_cast<bf16x8*>(cmat + (int64_t)m * ldc + n) = pack8(f);
    }
  }
}

template <int BM, int BN, int WM, int WN, bool AK, bool BKM, int NST, int EPI>
__global__ __launch_bounds__(WM* WN * 64) void gemm_tile_kernel(const GemmKArgs p) {
  gemm_tile<false, BM, BN, WM, WN, AK, BKM, NST, EPI>(GemmGroupKArgs{}, p);
}
template <int BM, int BN, int WM, int WN, bool AK, bool BKM, int NST, int EPI>
__global__ __launch_bounds__(WM* WN * 64) void gemm_tile_group_kernel(const GemmGroupKArgs g) {
  gemm_tile<true, BM, BN, WM, WN, AK, BKM, NST, EPI>(g, g.prob[0]);
}

template <int BM, int BN, int WM, int WN, int NST, bool AK, bool BKM, int EPI>
static int launch_tiles(const GemmKArgs* ks, int n, const RopeEpilogue* rope, hipStream_t st) {
  constexpr size_t ring = (size_t)NST * (BM + BN) * BK * 2, staging = (size_t)BM * (BN + 4) * sizeof(float);
  constexpr size_t lds = ring > staging ? ring : staging;
  auto tiled = [](GemmKArgs k) {
    k.tiles_m = (k.M + BM - 1) / BM;
    k.tiles_n = (k.N + BN - 1) / BN;
    k.band_rows = 8;
    return k;
  };
  const dim3 block(WM * WN * 64);
  static std::atomic<unsigned long long> lds_done{0};
  if constexpr (EPI != TILE_ROPE) {
    if (n == 1) {
      auto kern = gemm_tile_kernel<BM, BN, WM, WN, AK, BKM, NST, EPI>;
      if (int rc = reserve_lds(kern, lds, lds_done, "gemm tile")) return rc;
      const GemmKArgs k = tiled(ks[0]);
      hipLaunchKernelGGL(kern, dim3((unsigned)(k.tiles_m * k.tiles_n)), block, lds, st, k);
      return check_launch("gemm tile");
    }
  }
  // several products: the weight gradients (both operands mn-major) and the head projections
  if constexpr (EPI == TILE_ROPE || (EPI == TILE_PLAIN && !AK && !BKM)) {
    auto kern = gemm_tile_group_kernel<BM, BN, WM, WN, AK, BKM, NST, EPI>;
    static std::atomic<unsigned long long> lds_done_group{0};
    if (int rc = reserve_lds(kern, lds, lds_done_group, "gemm tile group")) return rc;
    GemmGroupKArgs g{};
    g.n = n;
    for (int i = 0; i < n; ++i) {
      g.prob[i] = tiled(ks[i]);
      g.tile_start[i + 1] = g.tile_start[i] + g.prob[i].tiles_m * g.prob[i].tiles_n;
    }
    if (rope) {
      g.rope_cos = rope->cos; g.rope_sin = rope->sin;
      g.rope_seq = rope->seq; g.rope_dh = rope->head_dim; g.rope_layout = rope->layout;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)g.tile_start[n]), block, lds, st, g);
    return check_launch("gemm tile group");
  }
  return fail(-1, "gemm tile: no grouped launch of this kind");
}

// T128x256: 144 KB of LDS, T128: 96 KB, one workgroup of eight waves per CU; T64: 64 KB, two of four waves.
template <bool AK, bool BKM, int EPI>
static int launch_size(TileSize size, const GemmKArgs* ks, int n, const RopeEpilogue* rope, hipStream_t st) {
  switch (size) {
    case TileSize::T128x256: return launch_tiles<128, 256, 2, 4, 3, AK, BKM, EPI>(ks, n, rope, st);
    case TileSize::T128: return launch_tiles<128, 128, 2, 4, 3, AK, BKM, EPI>(ks, n, rope, st);
    case TileSize::T64: return launch_tiles<64, 64, 2, 2, 4, AK, BKM, EPI>(ks, n, rope, st);
  }
  return fail(-1, "gemm tile: unknown size");
}

int launch_gemm_tile(TileSize size, const GemmKArgs* ks, int n, bool ak, bool bk, TileEpilogue epi, const RopeEpilogue* rope,
                     hipStream_t st) {
  if (rope) return launch_size<true, true, TILE_ROPE>(size, ks, n, rope, st);
  if (epi == TileEpilogue::SWIGLU) return launch_size<true, true, TILE_SWIGLU>(size, ks, n, nullptr, st);
  if (epi == TileEpilogue::SWIGLU_GRAD)
    return bk ? launch_size<true, true, TILE_SWIGLU_GRAD>(size, ks, n, nullptr, st) : launch_size<true, false, TILE_SWIGLU_GRAD>(size, ks, n, nullptr, st);
  if (ak && bk) return launch_size<true, true, TILE_PLAIN>(size, ks, n, nullptr, st);
  if (!ak && !bk) return launch_size<false, false, TILE_PLAIN>(size, ks, n, nullptr, st);
  if (ak && !bk) return launch_size<true, false, TILE_PLAIN>(size, ks, n, nullptr, st);
  return fail(-1, "gemm tile: operand layout not built");
}

}  // namespace dl
