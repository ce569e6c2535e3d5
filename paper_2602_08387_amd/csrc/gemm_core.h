// Pieces shared by the GEMM kernels (gemm.hip, gemm_tile.hip): kernel arguments, the asynchronous global -> LDS
// tile loads, operand fragments and the load cursor.  The layouts are described at the top of gemm.hip.
#pragma once
#include "common.h"
#include "kernels.h"
#include <atomic>
#include <type_traits>

namespace dl {

constexpr int BK = 64;   // k-values per pipeline stage
constexpr int MI = 16;               // MFMA block edge: 16x16x32 holds 2.2 PFLOP/s under the power limit, 32x32x16 1.95
constexpr int KSTEP = 32;            // k per MFMA
__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

struct GemmKArgs {
  const bf16_t* a[3];
  const bf16_t* b[3];
  int64_t lda[3], ldb[3];
  int K[3];
  int nseg;
  int M, N;
  int m_base;      // rows of the whole product above this part of it (the second launch of a product in two parts)
  bf16_t* c;
  int64_t ldc;
  const bf16_t* r;
  int accumulate;
  int tiles_m, tiles_n;
  int band_rows;   // tile rows per band of the tile sequence (see band_rows_for)
  // persistent kernels: tiles of a band, 2^32 / that rounded up, K-steps of all segments
  int band_tiles;
  uint32_t band_recip;
  int ksteps;
  // gated-pair products only (see gemm_swiglu_kernel): second weight, second and third output
  const bf16_t* b2;
  bf16_t *c2, *c3;
  int64_t ldc3;
  // activation-gradient epilogue only (see EPI_SWIGLU_GRAD); the one-tile kernels write silu(e1) * e2 to c3 unless it is null
  const bf16_t *e1, *e2;
  int64_t lde;
  // rotary epilogue only (see EPI_ROPE): rotate this problem's output
  int rope;
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, (int)bytes, 0x00020000);
}

// Loads one operand tile (R rows of the M/N index, BK of k) for K-step origin k0 into LDS.
template <int R, bool KMAJOR, int NW>
struct TileLoader {
  static constexpr int NINSTR = R * BK * 2 / 1024;  // wave-wide 1 KiB loads per tile
  static constexpr int PER_WAVE = NINSTR / NW;
  static_assert(NINSTR % NW == 0 && PER_WAVE >= 1, "tile loads must divide across waves");
  static constexpr int CPRK = BK / 8;               // chunks per row of a k-major tile
  static constexpr int RPW = 16 / CPRK;             // k-major rows per 256-byte bank window
  static constexpr int CPR = R / 8;                 // chunks per k-row (mn-major)
  static constexpr int RPI = KMAJOR ? 1024 / (BK * 2) : 1024 / (R * 2);  // tile rows per instruction
  // k-major: swizzle variants a lane needs across its instructions (precomputed offsets);
  // mn-major: the chunk swizzle is applied per instruction from (row part, chunk, k-row in instr).
  static constexpr int NVAR = KMAJOR ? (RPI >= 16 ? 1 : 16 / RPI) : 1;
  static_assert(PER_WAVE % NVAR == 0, "swizzle variant must not depend on the wave index");
  uint32_t voff[NVAR];
  int pc, kq;

  // chunk XOR of k-row k of an mn-major tile: the rows k..k+3 (bits 2-3) and k+8.. (bit 1) that a
  // 32-lane transposed read touches fall in 8 different 32-byte bank groups.
  // A 64-wide tile has 128-byte rows: two rows share a bank window, rows k, k + 2 are told apart by bit 2.
  static __device__ __forceinline__ int mn_swz(int k) {
    if constexpr (CPR == 8) return (((k >> 1) & 1) << 2) | (((k >> 3) & 1) << 1);
    return (((k & 3) << 2) | (((k >> 3) & 1) << 1)) & (CPR - 1);
  }

  __device__ __forceinline__ void init(int lane, int64_t ld) {
    if constexpr (KMAJOR) {
      // instruction j covers rows RPI*j ..; the swizzle depends on (row / RPW) & (CPRK - 1)
#pragma unroll
      for (int v = 0; v < NVAR; ++v) {
        const int row = v * RPI + lane / CPRK;   // row modulo 16
        const int c = (lane % CPRK) ^ ((row / RPW) & (CPRK - 1));
        voff[v] = (uint32_t)((lane / CPRK) * ld * 2 + (c << 4));
      }
    } else {
      kq = lane / CPR;
      pc = lane % CPR;
      voff[0] = (uint32_t)(kq * ld * 2);
    }
  }

  __device__ __forceinline__ void issue(__amdgpu_buffer_rsrc_t rs, char* lds_tile, int wave, int64_t ld,
                                        int k0) const {
    issue_range<0, PER_WAVE>(rs, lds_tile, wave, ld, k0);
  }
  // this wave's loads I0 .. I1-1 of the tile
  template <int I0, int I1>
  __device__ __forceinline__ void issue_range(__amdgpu_buffer_rsrc_t rs, char* lds_tile, int wave, int64_t ld,
                                              int k0) const {
#pragma unroll
    for (int i = I0; i < I1; ++i) {
      const int j = wave * PER_WAVE + i;
      const uint32_t soff = KMAJOR ? (uint32_t)(((int64_t)RPI * j * ld + k0) * 2)
                                   : (uint32_t)(((int64_t)(k0 + j * RPI) * ld) * 2);
      uint32_t vo;
      if constexpr (KMAJOR) vo = voff[i % NVAR];
      else vo = voff[0] + (uint32_t)((pc ^ mn_swz(j * RPI + kq)) << 4);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (LDS_PTR(void))(lds_tile + j * 1024), 16, vo, soff, 0, 0);
    }
  }
  // Tile of a PAIR of k-major matrices: of every 64 tile rows the first 32 are rows of the first
  // matrix and the next 32 the SAME rows of the second (tile row r <- matrix (r / 32) & 1, row
  // (r / 64) * 32 + r % 32), so that a wave whose MFMA tile spans 64 of these rows holds both values
  // of a column pair.  LDS placement and swizzle are those of the plain tile.
  template <int I0, int I1>
  __device__ __forceinline__ void issue_pair_range(__amdgpu_buffer_rsrc_t rs0, __amdgpu_buffer_rsrc_t rs1,
                                                   char* lds_tile, int wave, int64_t ld, int k0) const {
    static_assert(KMAJOR && 32 % RPI == 0, "an instruction's rows must lie in one matrix");
#pragma unroll
    for (int i = I0; i < I1; ++i) {
      const int j = wave * PER_WAVE + i;
      const int r0 = j * RPI;
      const int row = (r0 >> 6) * 32 + (r0 & 31);
      const uint32_t soff = (uint32_t)(((int64_t)row * ld + k0) * 2);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(((r0 >> 5) & 1) ? rs1 : rs0, (LDS_PTR(void))(lds_tile + j * 1024), 16,
                                               voff[i % NVAR], soff, 0, 0);
    }
  }
};

// Rotation of the pair (a, b) by the angle with cosine c and sine s.  The fused operations are written out: left to the
// compiler, every kernel rounds another one of the two products, and a head has other bits on another tile.
__device__ __forceinline__ float rotated_first(float a, float b, float c, float s) { return __builtin_fmaf(a, c, -(b * s)); }
__device__ __forceinline__ float rotated_second(float a, float b, float c, float s) { return __builtin_fmaf(b, c, a * s); }

// f(integral_constant<int, I>) for I = I0 .. N-1: a loop whose index is a compile-time constant
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// Start of a tile's contraction, in K-steps: (g mod 8) eighths of the way through K (the walk wraps around),
// g = the tile's group of 2048 rows, whatever the tile height.  Tiles that run at the same time belong to
// different groups, and without this all of them stream the same k-range of their operands at once: the requests
// then crowd the same memory channels (worst with rows a multiple of 4 KiB apart).  The start depends on the
// row group only - not on the workgroup, the launch, the tile size or the band height - so a product gives the
// same bits in whatever launch it is computed.
__device__ __forceinline__ int k_start(int m0, int total) { return (((m0 >> 11) & 7) * total) >> 3; }

// acc[i][j] += A[i] B[j] over two k-substeps, for 2 x 4 blocks: cIJ is block (i, j), aKI and bKJ the operands of substep K.
// As assembly, in place: left to itself the compiler lets accumulators wander from one set of registers to another and
// runs out of them.  The B operand stays for two MFMAs and the blocks are taken four at a time: the fewer operand bits
// change from one MFMA to the next, the less power it draws (16384 x 4096 x 14336: A held for four MFMAs while B changes
// 1288 us, this order 1268; B held for four gains no more).  The s_nop covers a VALU write of an operand right in front; the
// accumulators may not be read otherwise before mfma_drain().
__device__ __forceinline__ void mfma_quadrant(f32x4& c00, f32x4& c10, f32x4& c01, f32x4& c11, f32x4& c02, f32x4& c12, f32x4& c03, f32x4& c13,
                                              bf16x8 a00, bf16x8 a01, bf16x8 a10, bf16x8 a11, bf16x8 b00, bf16x8 b01, bf16x8 b02, bf16x8 b03,
                                              bf16x8 b10, bf16x8 b11, bf16x8 b12, bf16x8 b13) {
#define MFMA(C, A, B) "v_mfma_f32_16x16x32_bf16 %" #C ", %" #A ", %" #B ", %" #C "\n\t"
  asm volatile("s_nop 1\n\t"
               MFMA(0, 8, 12) MFMA(1, 9, 12) MFMA(2, 8, 13) MFMA(3, 9, 13) MFMA(0, 10, 16) MFMA(1, 11, 16) MFMA(2, 10, 17) MFMA(3, 11, 17)
               MFMA(4, 8, 14) MFMA(5, 9, 14) MFMA(6, 8, 15) MFMA(7, 9, 15) MFMA(4, 10, 18) MFMA(5, 11, 18) MFMA(6, 10, 19) MFMA(7, 11, 19)
               : "+v"(c00), "+v"(c10), "+v"(c01), "+v"(c11), "+v"(c02), "+v"(c12), "+v"(c03), "+v"(c13)
               : "v"(a00), "v"(a01), "v"(a10), "v"(a11), "v"(b00), "v"(b01), "v"(b02), "v"(b03), "v"(b10), "v"(b11), "v"(b12), "v"(b13));
#undef MFMA
}
// Waits until the last MFMA has written its block, and makes the accumulators depend on the wait: the compiler, which sees no
// MFMA and no hazard, may otherwise put a read of them in front of it.
template <int N, int M>
__device__ __forceinline__ void mfma_drain(f32x4 (&acc)[N][M]) {
  asm volatile("s_nop 15\n\ts_nop 3" ::: "memory");
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = 0; j < M; ++j) asm volatile("" : "+v"(acc[i][j]));
}

// 16 bytes per lane from LDS address `at` + OFF, or transposed 2 x 8 of k-rows r and r + 4, HI bytes apart.  As
// assembly: for the builtins the compiler cannot tell that a read stays clear of the stage the asynchronous loads are filling
// and waits for those in front of it.  It does not count these reads either, so every fragment passes through a wait that names it.
template <int OFF>
__device__ __forceinline__ void lds_read(bf16x8& v, uint32_t at) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(at), "n"(OFF));
}
template <int OFF, int HI>
__device__ __forceinline__ void lds_read_tr(bf16x8& v, uint32_t at) {
  bf16x4 lo, hi;
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo) : "v"(at), "n"(OFF));
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(hi) : "v"(at), "n"(OFF + HI));
  v.lo = lo;
  v.hi = hi;
}

// Position of the next tile pair to fetch: segment, k offset, and that segment's descriptors.
// PAIR: the B tile interleaves two weight matrices (TileLoader::issue_pair_range); n0 and N then
// count columns of the interleaved product, twice the rows of either matrix.
template <int BM, int BN, int NW, bool AK, bool BKM, bool PAIR = false>
struct LoadCursor {
  TileLoader<BM, AK, NW> la;
  TileLoader<BN, BKM, NW> lb;
  __amdgpu_buffer_rsrc_t ra, rb, rb2;
  int64_t lda, ldb;
  int seg = 0, k = 0, kend = 0, nseg = 1;   // kend: K of the open segment (kept in a register: no kernarg read per K-step)
  int left = 0;                             // K-steps of the tile still to fetch; the walk may start anywhere and wraps

  __device__ __forceinline__ void open_raw(const bf16_t* a, const bf16_t* b, int64_t lda_, int64_t ldb_, int K, int M,
                                           int N, int m0, int n0, int lane) {
    kend = K;
    lda = lda_;
    ldb = ldb_;
    const bf16_t* ab = AK ? a + (int64_t)m0 * lda : a + m0;
    const bf16_t* bb = BKM ? b + (int64_t)n0 * ldb : b + n0;
    const uint32_t a_bytes = AK ? (uint32_t)((((int64_t)(M - m0 - 1)) * lda + K) * 2)
                                : (uint32_t)((((int64_t)(K - 1)) * lda + (M - m0)) * 2);
    const uint32_t b_bytes = BKM ? (uint32_t)((((int64_t)(N - n0 - 1)) * ldb + K) * 2)
                                 : (uint32_t)((((int64_t)(K - 1)) * ldb + (N - n0)) * 2);
    ra = make_rsrc(ab, a_bytes);
    rb = make_rsrc(bb, b_bytes);
    la.init(lane, lda);
    lb.init(lane, ldb);
  }
  __device__ __forceinline__ void open_pair(const bf16_t* a, const bf16_t* b, const bf16_t* b2, int64_t lda_,
                                            int64_t ldb_, int K, int M, int N, int m0, int n0, int lane) {
    static_assert(!PAIR || (AK && BKM), "paired weights are k-major");
    open_raw(a, b, lda_, ldb_, K, M, N / 2, m0, n0 / 2, lane);
    rb2 = make_rsrc(b2 + (int64_t)(n0 / 2) * ldb_, (uint32_t)((((int64_t)(N / 2 - n0 / 2 - 1)) * ldb_ + K) * 2));
  }
  __device__ __forceinline__ void open(const GemmKArgs& p, int s, int m0, int n0, int lane) {
    open_raw(p.a[s], p.b[s], p.lda[s], p.ldb[s], p.K[s], p.M, p.N, m0, n0, lane);
  }
  // `segs`: the problem whose further K-segments follow (only read when nseg > 1)
  __device__ __forceinline__ void issue_next(const GemmKArgs& segs, char* stage, int wave, int m0, int n0, int lane) {
    if (left > 0) {
      la.issue(ra, stage, wave, lda, k);
      if constexpr (PAIR)
        lb.template issue_pair_range<0, TileLoader<BN, BKM, NW>::PER_WAVE>(rb, rb2, stage + BM * BK * 2, wave, ldb, k);
      else
        lb.issue(rb, stage + BM * BK * 2, wave, ldb, k);
      advance(segs, m0, n0, lane);
    }
  }
  // one K-step on: past the end of a segment the walk goes on in the next one, past the last in the first
  __device__ __forceinline__ void advance(const GemmKArgs& segs, int m0, int n0, int lane) {
    --left;
    k += BK;
    if (k == kend) {
      k = 0;
      if (nseg > 1 && left > 0) {
        seg = seg + 1 == nseg ? 0 : seg + 1;
        open(segs, seg, m0, n0, lane);
      }
    }
  }
};

// Workgroups are dealt round-robin to the 8 XCDs, each with its own L2: give every XCD a contiguous
// range of the tile sequence.
__device__ __forceinline__ int xcd_contiguous(int id, int ntiles) {
  const int per_xcd = ntiles >> 3;
  return id < (per_xcd << 3) ? (id & 7) * per_xcd + (id >> 3) : id;
}

// Several independent problems of one operand layout in one grid: their tile sequences are laid end
// to end, so the last, partly filled round of one problem runs alongside the first of the next.
constexpr int MAX_GROUP = 8;
struct GemmGroupKArgs {
  GemmKArgs prob[MAX_GROUP];
  int tile_start[MAX_GROUP + 1];
  int n;
  // rotary epilogue only (see EPI_ROPE): cos and sin of the angle of (position, pair), [seq][head_dim/2]
  const float *rope_cos, *rope_sin;
  int rope_seq, rope_dh, rope_layout;
};
// Problem i of a grouped launch, whose GemmGroupKArgs is the kernel's first argument: a reference into the constant
// kernel-argument segment, so that a wave-uniform run-time index becomes scalar loads of the one problem (selecting
// among all of them by compile-time index held eight problems in scalar registers and spilled two hundred).
typedef const __attribute__((address_space(4))) GemmGroupKArgs ConstGroupKArgs;
__device__ __forceinline__ const __attribute__((address_space(4))) GemmKArgs& group_problem(int i) {
  static_assert(std::is_trivially_copyable<GemmGroupKArgs>::value, "read in place");
  return ((ConstGroupKArgs*)__builtin_amdgcn_kernarg_segment_ptr())->prob[__builtin_amdgcn_readfirstlane(i)];
}

// Kernels of gemm_tile.hip: one tile per workgroup.
enum class TileSize { T128x256, T128, T64 };
enum class TileEpilogue { PLAIN, SWIGLU, SWIGLU_GRAD };
// one product with the row statistics of the attention backward in its epilogue; the tile holds whole heads
int launch_gemm_tile_delta(TileSize size, const GemmKArgs& k, bool b_kmajor, const DeltaEpilogue& d, hipStream_t st);
// gains: weight gradients only, summed by further workgroups of the launch
int launch_gemm_tile(TileSize size, const GemmKArgs* ks, int n, bool a_kmajor, bool b_kmajor, TileEpilogue epi, const RopeEpilogue* rope,
                     hipStream_t st, const GainSums* gains = nullptr);

}  // namespace dl
