// bf16 GEMM for problems that do not fill the chip with 256 x 256 tiles: one 128 x 256, 128 x 128 or 64 x 64 tile per
// workgroup.  Same operand layouts, same MFMA, same order of summation as the persistent kernel (gemm.hip): a
// product has the same bits on either.
//
// What bounds it: the smaller the tile, the more bytes per flop have to reach a CU, and some 100 GB/s per CU is what the
// global -> LDS loads bring (128 x 128: 92, 64 x 64: 100, one tile per CU; T = 8192, N = 768 on 128 x 256 tiles 75, next to its
// fragment reads: without either of the two it runs at the MFMAs' rate).  And a wave that loads stands still: the address unit
// takes 16 cycles per wave-wide load, of all waves in turn.  So four waves of a workgroup do nothing but load, and the others
// never wait for the address unit.  Microseconds per K-step of 64 (K from 2048 to 4096 or 3136 to 6272), all waves loading
// and now: 64 x 64 (T = 1000, N = 1024: 256 tiles) 0.25, 0.16; 128 x 128 (T = 1920, N = 1152: 135 tiles) 0.39, 0.35; 128 x 256 (192
// tiles) 0.66, 0.61.  Whole products: T 1000, K 2048, N 1024 10.9 -> 9.0 us; T 1920, K 6272, N 1152 42.7 -> 38.8; T 8192, K 4096, N 768
// 54 -> 49.5; weight gradient 1024 x 1024 of 2048 tokens 12.4 -> 9.8.  Measured on the way: deeper rings (five stages, eight)
// change nothing; fragments requested a whole K-step ahead: 128 x 128 10 % slower; tiles through registers and ds_write instead of
// straight to LDS 20 to 50 % slower; two wave groups a slot apart, as in the persistent kernel, on the 128 x 256 tile as fast as this.
// Full rounds of 256 x 256 tiles stay on the persistent kernel: a quarter fewer loads per flop, its epilogue under the next
// tile's main loop, and accumulators that leave no registers for a third wave per SIMD.
//
// The epilogue passes the fp32 sums through LDS (the ring is free by then), so every fused epilogue is an
// element-wise function of rows: residual or accumulation, rotary embedding (both members of a pair lie in the
// tile), gated pair, activation gradient.
#include "gain_sums.h"
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

// TILE_DELTA: plain, and of every head's columns -rowsum(dO * O) of the values stored, and lse * log2(e), as
// attn_delta_kernel writes them (same order of summation).
enum { TILE_PLAIN = 0, TILE_SWIGLU = 1, TILE_SWIGLU_GRAD = 2, TILE_ROPE = 3, TILE_DELTA = 4 };

// A workgroup's tile: its problem's fields and where it lies.
struct TileOf {
  int m0, n0, K0, M, N, m_base, accumulate, rope, total;
  const bf16_t *a0, *b0, *res;
  bf16_t* c;
  int64_t lda0, ldb0, ldc;
};
template <bool GROUPED, int BM, int BN>
__device__ __forceinline__ TileOf find_tile(const GemmGroupKArgs& grp, const GemmKArgs& one) {
  int ntiles;
  if constexpr (GROUPED) {
    ntiles = grp.tile_start[1];
#pragma unroll
    for (int i = 2; i <= MAX_GROUP; ++i) if (i <= grp.n) ntiles = grp.tile_start[i];
  } else {
    ntiles = one.tiles_m * one.tiles_n;
  }
  int pid = xcd_contiguous(blockIdx.x, ntiles);
  int tiles_m, tiles_n, GM, start = 0;
  TileOf t;
  auto take = [&](const auto& q) {
    tiles_m = q.tiles_m; tiles_n = q.tiles_n; GM = q.band_rows; t.K0 = q.K[0];
    t.a0 = q.a[0]; t.b0 = q.b[0]; t.lda0 = q.lda[0]; t.ldb0 = q.ldb[0];
    t.M = q.M; t.N = q.N; t.m_base = q.m_base; t.accumulate = q.accumulate; t.c = q.c; t.res = q.r; t.ldc = q.ldc; t.rope = q.rope;
  };
  t.total = 0;
  if constexpr (GROUPED) {
    int pi = 0;
#pragma unroll
    for (int i = 1; i < MAX_GROUP; ++i)
      if (i < grp.n && pid >= grp.tile_start[i]) { pi = i; start = grp.tile_start[i]; }
    take(group_problem(pi));
    pid -= start;
    t.total = t.K0 / BK;
  } else {
    take(one);
    for (int s = 0; s < one.nseg; ++s) t.total += one.K[s] / BK;
  }
  const int band = pid / (GM * tiles_n), first_m = band * GM, band_h = min(tiles_m - first_m, GM), in_band = pid - band * GM * tiles_n;
  t.m0 = (first_m + in_band % band_h) * BM;
  t.n0 = (in_band / band_h) * BN;
  return t;
}

// The tile's results: `to_staging` writes a wave's fp32 sums to [BM][BN + 4] floats in LDS (the ring is free by then), from where
// every fused epilogue is an element-wise function of rows.
template <int BM, int BN, int NT, int EPI, typename F>
__device__ __forceinline__ void tile_epilogue(const GemmGroupKArgs& grp, const GemmKArgs& one, const DeltaEpilogue& da, const TileOf& t, char* smem, F&& to_staging) {
  constexpr bool PAIR = EPI == TILE_SWIGLU;
  // Epilogue.  fp32 sums to LDS, rows of BN + 4 floats (the 16 bytes more put the 16 rows a store instruction touches in
  // different banks), then 8 consecutive columns per thread along rows.
  constexpr int SP = BN + 4;
  constexpr int OC = PAIR ? BN / 2 : BN;               // output columns of the tile
  constexpr int VPR = OC / 8, NV = (BM * VPR + NT - 1) / NT;   // 8-column vectors per row and per thread
  float* stg = reinterpret_cast<float*>(smem);
  const int M = t.M, N = t.N, m0 = t.m0, n0 = t.n0, accumulate = t.accumulate;
  const int64_t ldc = t.ldc;
  const bf16_t* res = t.res;
  bf16_t* cmat = t.c;
  const int on0 = PAIR ? n0 / 2 : n0, ON = PAIR ? N / 2 : N;
  // Residual or old value, asked for before the staging.  Not as bf16x8: the compiler takes those apart between two loads, each time behind a
  // wait (T 1600, K 448, N 12608 32.1 us, 29.5 without; T 8192, K 768, N 768 14.5, 13.7).
  u32x4 pre[EPI == TILE_PLAIN ? NV : 1];
  if constexpr (EPI == TILE_PLAIN) {
    const bf16_t* src = res ? res : accumulate ? cmat : nullptr;
    if (src) {
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        const int id = v * NT + (int)threadIdx.x, m = m0 + id / VPR, n = on0 + id % VPR * 8;
        const u32x4 zero = {0, 0, 0, 0};
        pre[v] = zero;
        if ((BM * VPR % NT == 0 || id < BM * VPR) && m < M && n < ON) pre[v] = *reinterpret_cast<const u32x4*>(src + (int64_t)m * ldc + n);
      }
    }
  }
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();   // every wave is done reading the ring
  asm volatile("" ::: "memory");
  to_staging(stg);
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
    if ((BM * VPR % NT != 0 && id >= BM * VPR) || m >= M || n >= ON) continue;
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
        const float sg = logistic(z[e]), dz = d[e] * u[e] * sg * (1.0f + z[e] * (1.0f - sg)), a = z[e] * sg * u[e];
        u[e] = d[e] * z[e] * sg;
        d[e] = dz;
        z[e] = a;
      }
      if (one.c3) *reinterpret_cast<bf16x8*>(one.c3 + (int64_t)m * ldc + n) = pack8(z);
      *reinterpret_cast<bf16x8*>(cmat + (int64_t)m * ldc + n) = pack8(d);
      *reinterpret_cast<bf16x8*>(one.c2 + (int64_t)m * ldc + n) = pack8(u);
    } else {
      float f[8];
      row8(row, col, f);
      if constexpr (EPI == TILE_ROPE) {
        if (t.rope) {
          const int dh = grp.rope_dh, hd2 = dh >> 1, pos = (m + t.m_base) % grp.rope_seq, o = n % dh;
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
      } else if (EPI == TILE_PLAIN && (res || accumulate)) {
        const bf16x8 old = __builtin_bit_cast(bf16x8, pre[v]);
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] += (float)old[e];
      }
      const bf16x8 out = pack8(f);
      *reinterpret_cast<bf16x8*>(cmat + (int64_t)m * ldc + n) = out;
      if constexpr (EPI == TILE_DELTA) {
        const bf16x8 o = *reinterpret_cast<const bf16x8*>(static_cast<const bf16_t*>(da.o) + (int64_t)m * ldc + n);
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) s += (float)o[e] * (float)out[e];
        for (int off = da.head_dim >> 4; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        if (n % da.head_dim == 0) {
          const int b = m / da.seq;
          const int64_t at = ((int64_t)b * da.heads + n / da.head_dim) * da.seq + (m - b * da.seq);
          da.delta[at] = -s;
          da.lse2[at] = da.lse[at] * kLog2e;
        }
      }
    }
  }
}

constexpr int LOADERS = 4;   // waves that load; two are slower (T 512, K = N = 2048 input gradient 9.1 -> 10.2 us)
constexpr int FEW = 2;       // ring stages of the kernels for contractions of at most as many K-steps
constexpr int tile_threads(int bm, int nst) { return ((bm == 64 ? 4 : 8) + (nst == FEW ? 0 : LOADERS)) * 64; }

// NST: ring stages.  FEW: nothing is left to load in the loop, so all K-steps go out at the start, by the waves that multiply, and are waited
// for together.  EPI as the persistent kernel's epilogues.
template <bool GROUPED, int BM, int BN, bool AK, bool BKM, int NST, int EPI>
__device__ __forceinline__ void gemm_tile(const GemmGroupKArgs& grp, const GemmKArgs& one, const DeltaEpilogue& da) {
  constexpr int WM = 2, WN = BM == 64 ? 2 : 4, NW = WM * WN, NL = NST == FEW ? NW : LOADERS, NT = tile_threads(BM, NST);   // waves that multiply, load
  constexpr int TM = BM / WM, TN = BN / WN, FM = TM / 16, FN = TN / 16;
  constexpr int A_BYTES = BM * BK * 2, STAGE = A_BYTES + BN * BK * 2;
  constexpr bool PAIR = EPI == TILE_SWIGLU;
  static_assert(BK == 64 && MI == 16 && KSTEP == 32, "two k-substeps per stage");
  extern __shared__ __attribute__((aligned(1024))) char smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave_m = wave % WM, wave_n = wave / WM;

  const TileOf t = find_tile<GROUPED, BM, BN>(grp, one);
  const int M = t.M, N = t.N, m0 = t.m0, n0 = t.n0, total = t.total;
  constexpr int LPW = TileLoader<BM, AK, NL>::PER_WAVE + TileLoader<BN, BKM, NL>::PER_WAVE;
  f32x4 acc[FN][FM];
  LoadCursor<BM, BN, NL, AK, BKM, PAIR> cur;
  const int lwave = NST == FEW ? wave : wave - NW;
  auto first_loads = [&] {
    cur.nseg = GROUPED ? 1 : one.nseg;
    cur.left = total;
    int first = k_start(m0 + t.m_base, total);
    cur.seg = 0;
    if constexpr (!GROUPED) {
      for (int s = 0; s + 1 < one.nseg; ++s)
        if (cur.seg == s && first >= one.K[s] / BK) { first -= one.K[s] / BK; cur.seg = s + 1; }
    }
    cur.k = first * BK;
    if (cur.seg == 0) {
      if constexpr (PAIR) cur.open_pair(t.a0, t.b0, one.b2, t.lda0, t.ldb0, t.K0, M, N, m0, n0, lane);
      else cur.open_raw(t.a0, t.b0, t.lda0, t.ldb0, t.K0, M, N, m0, n0, lane);
    } else {
      cur.open(one, cur.seg, m0, n0, lane);
    }
#pragma unroll
    for (int s = 0; s < NST; ++s) cur.issue_next(one, smem + s * STAGE, lwave, m0, n0, lane);
  };
  if (NST != FEW && wave >= NW) {
    first_loads();
    if (total >= NST) wait_vmcnt<(NST - 1) * LPW>(); else wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    uint32_t st = 0;
    for (int k = 0; k + 1 < total; ++k) {
      // K-step k + 1 has landed once at most the NST - 2 younger ones are in flight; past the barrier every wave has its
      // last fragments of K-step k in registers, and its stage takes K-step k + NST
      if (k + NST <= total) wait_vmcnt<(NST - 2) * LPW>(); else wait_vmcnt<0>();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      cur.issue_next(one, smem + st, lwave, m0, n0, lane);
      st = st + STAGE == NST * STAGE ? 0 : st + STAGE;
    }
  } else {
    if constexpr (NST == FEW) first_loads();
    FragReader<BM, AK, FM> ra;
    FragReader<BN, BKM, FN> rb;
    ra.init(smem, wave_m * TM, lane);
    rb.init(smem + A_BYTES, wave_n * TN, lane);
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
      for (int j = 0; j < FM; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

    if constexpr (NST == FEW) wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    // Fragments run half a K-step ahead of the MFMAs.  The MFMAs of a k-substep go out in rows (one fragment of the side
    // with more of them against all of the other side); the reads of the next substep go between its first rows: in a bunch in
    // front of the MFMAs the reads of all waves queue with every wave's MFMAs behind them.
    constexpr int NF = FM + FN, ROWS = FM > FN ? FM : FN;
    bf16x8 fa[2][FM], fb[2][FN];
    auto read_one = [&](auto KS, auto F, uint32_t stage) {
      constexpr int ks = decltype(KS)::value, f = decltype(F)::value;
      if constexpr (f < FM) ra.template read<ks, f>(fa[ks], stage);
      else rb.template read<ks, f - FM>(fb[ks], stage);
    };
    auto mfma_row = [&](auto KS, auto RW) {
      constexpr int ks = decltype(KS)::value, r = decltype(RW)::value;
      if constexpr (FM >= FN) {   // the B operand stays (see mfma_quadrant)
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
    uint32_t st = 0;                       // byte offset of the stage
    for (int k = 0; k < total; ++k) {
      constexpr int RD0 = ROWS >= 4 ? 2 : 1;              // rows the reads are spread over
      static_for<0, ROWS>([&](auto r) {
        constexpr int i = decltype(r)::value;
        if constexpr (i < RD0) static_for<i * NF / RD0, (i + 1) * NF / RD0>([&](auto f) { read_one(S1, f, st); });
        mfma_row(S0, r);
      });
      wait_reads(fa[1], fb[1]);
      const uint32_t nx = st + STAGE == NST * STAGE ? 0 : st + STAGE;
      mfma_row(S1, S0);
      if (NST != FEW && k + 1 < total) {   // K-step k + 1 has landed, see above
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
      }
      // the reads go out after the last K-step too (of a stage nobody fills any more; nobody uses them)
      constexpr int RD1 = ROWS >= 4 ? 2 : 1;
      static_for<1, ROWS>([&](auto r) {
        constexpr int i = decltype(r)::value;
        if constexpr (i <= RD1) static_for<(i - 1) * NF / RD1, i * NF / RD1>([&](auto f) { read_one(S0, f, nx); });
        mfma_row(S1, r);
      });
      wait_reads(fa[0], fb[0]);
      st = nx;
    }
  }
  tile_epilogue<BM, BN, NT, EPI>(grp, one, da, t, smem, [&](float* stg) {
    if (NST != FEW && wave >= NW) return;
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
      for (int j = 0; j < FM; ++j)
        *reinterpret_cast<f32x4*>(stg + (wave_m * TM + j * 16 + (lane & 15)) * (BN + 4) + wave_n * TN + i * 16 + (lane >> 4) * 4) = acc[i][j];
  });
}

template <int BM, int BN, bool AK, bool BKM, int NST, int EPI>
__global__ __launch_bounds__(tile_threads(BM, NST)) void gemm_tile_kernel(const GemmKArgs p) {
  gemm_tile<false, BM, BN, AK, BKM, NST, EPI>(GemmGroupKArgs{}, p, DeltaEpilogue{});
}
template <int BM, int BN, bool AK, bool BKM, int NST, int EPI>
__global__ __launch_bounds__(tile_threads(BM, NST)) void gemm_tile_group_kernel(const GemmGroupKArgs g, const GainSums gains, int first_gain) {
  // Weight gradients of a layer: the gain sums of its norms ride behind the tiles (a launch of their own takes 2.5 to 5 us)
  if constexpr (EPI == TILE_PLAIN) {
    if ((int)blockIdx.x >= first_gain) {
      extern __shared__ __attribute__((aligned(1024))) char smem[];
      gain_sums<tile_threads(BM, NST)>(gains, (int)blockIdx.x - first_gain, reinterpret_cast<float*>(smem));
      return;
    }
  }
  gemm_tile<true, BM, BN, AK, BKM, NST, EPI>(g, g.prob[0], DeltaEpilogue{});
}

template <int BM, int BN, bool BKM, int NST>
__global__ __launch_bounds__(tile_threads(BM, NST)) void gemm_tile_delta_kernel(const GemmKArgs p, const DeltaEpilogue d) {
  gemm_tile<false, BM, BN, true, BKM, NST, TILE_DELTA>(GemmGroupKArgs{}, p, d);
}

template <int BM, int BN, int NST, bool AK, bool BKM, int EPI>
static int launch_tiles(const GemmKArgs* ks, int n, const RopeEpilogue* rope, const DeltaEpilogue* delta, const GainSums* gains, hipStream_t st) {
  constexpr size_t ring = (size_t)NST * (BM + BN) * BK * 2, staging = (size_t)BM * (BN + 4) * sizeof(float);
  constexpr size_t lds = ring > staging ? ring : staging;
  auto tiled = [](GemmKArgs k) {
    k.tiles_m = (k.M + BM - 1) / BM;
    k.tiles_n = (k.N + BN - 1) / BN;
    k.band_rows = 8;
    return k;
  };
  const dim3 block(tile_threads(BM, NST));
  static std::atomic<unsigned long long> lds_done{0};
  if constexpr (EPI == TILE_DELTA) {
    auto kern = gemm_tile_delta_kernel<BM, BN, BKM, NST>;
    if (int rc = reserve_lds(kern, lds, lds_done, "gemm tile (row statistics)")) return rc;
    const GemmKArgs k = tiled(ks[0]);
    hipLaunchKernelGGL(kern, dim3((unsigned)(k.tiles_m * k.tiles_n)), block, lds, st, k, *delta);
    return check_launch("gemm tile (row statistics)");
  } else if constexpr (EPI != TILE_ROPE) {
    if (n == 1 && !gains) {
      auto kern = gemm_tile_kernel<BM, BN, AK, BKM, NST, EPI>;
      if (int rc = reserve_lds(kern, lds, lds_done, "gemm tile")) return rc;
      const GemmKArgs k = tiled(ks[0]);
      hipLaunchKernelGGL(kern, dim3((unsigned)(k.tiles_m * k.tiles_n)), block, lds, st, k);
      return check_launch("gemm tile");
    }
  }
  // several products: the weight gradients (both operands mn-major) and the head projections
  if constexpr (EPI == TILE_ROPE || (EPI == TILE_PLAIN && !AK && !BKM)) {
    auto kern = gemm_tile_group_kernel<BM, BN, AK, BKM, NST, EPI>;
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
    const int tiles = g.tile_start[n];
    hipLaunchKernelGGL(kern, dim3((unsigned)(tiles + (gains ? gain_sum_blocks(*gains) : 0))), block, lds, st, g, gains ? *gains : GainSums{}, tiles);
    return check_launch("gemm tile group");
  }
  return fail(-1, "gemm tile: no grouped launch of this kind");
}

// T128x256: 144 KB of LDS, T128: 96 KB, one workgroup of eight waves and four that load per CU; T64: 64 KB, two of four and four.
// FEW: 133, 67 and 32 KB.
template <bool AK, bool BKM, int EPI>
static int launch_size(TileSize size, const GemmKArgs* ks, int n, const RopeEpilogue* rope, hipStream_t st, const DeltaEpilogue* delta = nullptr,
                       const GainSums* gains = nullptr) {
  // One or two K-steps: four waves fewer to start, for which such a launch waits longer than for its loads.  us, with loading waves / without:
  // T 1792, K 64, N 960 4.5 / 4.2; gated pair T 768, K 64, F 832 4.7 / 4.3; T 11520, K 128, N 512 8.2 / 7.8.  Over 162 products 1.026 (K 64)
  // and 1.016 (K 128), with residual 1.015 and 1.014, gated pairs 1.035 and 1.025; three K-steps 0.998, four 0.97; the activation's
  // gradient 0.97, head projections and weight gradients no faster.
  if constexpr (AK && BKM && (EPI == TILE_PLAIN || EPI == TILE_SWIGLU)) {
    int64_t k = 0;
    for (int s = 0; s < ks[0].nseg; ++s) k += ks[0].K[s];
    if (n == 1 && k <= FEW * BK) {
      switch (size) {
        case TileSize::T128x256: return launch_tiles<128, 256, FEW, AK, BKM, EPI>(ks, n, rope, delta, gains, st);
        case TileSize::T128: return launch_tiles<128, 128, FEW, AK, BKM, EPI>(ks, n, rope, delta, gains, st);
        case TileSize::T64: return launch_tiles<64, 64, FEW, AK, BKM, EPI>(ks, n, rope, delta, gains, st);
      }
    }
  }
  switch (size) {
    case TileSize::T128x256: return launch_tiles<128, 256, 3, AK, BKM, EPI>(ks, n, rope, delta, gains, st);
    case TileSize::T128: return launch_tiles<128, 128, 3, AK, BKM, EPI>(ks, n, rope, delta, gains, st);
    case TileSize::T64: return launch_tiles<64, 64, 4, AK, BKM, EPI>(ks, n, rope, delta, gains, st);
  }
  return fail(-1, "gemm tile: unknown size");
}

int launch_gemm_tile_delta(TileSize size, const GemmKArgs& k, bool bk, const DeltaEpilogue& d, hipStream_t st) {
  return bk ? launch_size<true, true, TILE_DELTA>(size, &k, 1, nullptr, st, &d) : launch_size<true, false, TILE_DELTA>(size, &k, 1, nullptr, st, &d);
}

int launch_gemm_tile(TileSize size, const GemmKArgs* ks, int n, bool ak, bool bk, TileEpilogue epi, const RopeEpilogue* rope,
                     hipStream_t st, const GainSums* gains) {
  if (rope) return launch_size<true, true, TILE_ROPE>(size, ks, n, rope, st);
  if (epi == TileEpilogue::SWIGLU) return launch_size<true, true, TILE_SWIGLU>(size, ks, n, nullptr, st);
  if (epi == TileEpilogue::SWIGLU_GRAD)
    return bk ? launch_size<true, true, TILE_SWIGLU_GRAD>(size, ks, n, nullptr, st) : launch_size<true, false, TILE_SWIGLU_GRAD>(size, ks, n, nullptr, st);
  if (ak && bk) return launch_size<true, true, TILE_PLAIN>(size, ks, n, nullptr, st);
  if (!ak && !bk) return launch_size<false, false, TILE_PLAIN>(size, ks, n, nullptr, st, nullptr, gains);
  if (ak && !bk) return launch_size<true, false, TILE_PLAIN>(size, ks, n, nullptr, st);
  return fail(-1, "gemm tile: operand layout not built");
}

}  // namespace dl
