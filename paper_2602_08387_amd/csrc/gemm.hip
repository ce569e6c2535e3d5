// bf16 GEMM for gfx950 (products that fill the chip; gemm_tile.hip has the others): C[M,N] = sum_s opA_s[M,K_s] * opB_s[K_s,N] (+R) with fp32 accumulation
// on v_mfma_f32_16x16x32_bf16.  One kernel template serves the three products of a linear
// layer (y = x W^T, dx = dy W, dW = dy^T x): each operand may be stored with the contraction
// index contiguous ("k-major") or with its M/N index contiguous ("mn-major").
//
// Data path: global --buffer_load ... lds (16 B per lane, no VGPR staging)--> LDS ring of two
// stages of 64 k --ds_read_b128 (k-major) or ds_read_b64_tr_b16 (mn-major)--> MFMA operands.  The
// buffer descriptor's range check zero-fills rows past the end of a matrix, so M and N need not be
// tile multiples; K_s must be a multiple of 64.
//
// What bounds it: the power limit.  At 8192 x 8192 x 8192 the matrix pipes are busy 83 % of the cycles, at 1.8 GHz, and the
// two trade against each other: what a kernel gains is what it saves in energy per product.  Measured on working copies,
// as busy share x GHz: this loop 1.47; without its global loads 1.68; without its LDS reads 1.73; with all loads hitting the L2
// 1.50.  Hence: few instructions beside the MFMAs, and MFMAs in an order that changes few operand bits (mfma_quadrant).
// One loop of both waves of a SIMD in step, half a K-step of loads by four of the eight waves, as it was before:
// 8192 x 8192 x 8192 729 us, now 714; 16384 x 14336 x 4096 (streams an operand of 470 MB) 1436, now 1256; weight gradients of
// 16384 tokens, 14336 x 4096 1465, now 1378; of 8192 tokens, 2048 x 5632 171, now 157; gated pair at T 8192, K 2048, F 5632 303, now 296.
//
// LDS layouts (the async load puts lane l's 16 bytes at chunk l of a 1 KiB span, so swizzles
// are applied on the global-address side).  The LDS serves 256 B of banks per clock: a 16-byte
// read is done 16 lanes at a time, an 8-byte transposed read 32 lanes at a time.
//   k-major tile  [256 rows][64 k]  : 128 bytes per row = 8 chunks; chunk c of row r sits at c ^ ((r / 2) & 7), so 16
//                                     consecutive rows reading one logical chunk touch 16 different 16-byte bank groups.
//   mn-major half [64 k][128 mn]    : 16 chunks per k-row; chunk c of k-row k sits at c ^ (((k & 3) << 2) | (((k >> 3) & 1) << 1)):
//                                     the 8 k-rows x 32 B that 32 lanes of a transposed read touch fall in 8 different
//                                     32-byte bank groups.
// MFMA roles: the N-side operand feeds MFMA "A" (row index i), the M-side operand feeds MFMA
// "B" (column index j), so a lane ends up with 4 consecutive n for one m.  The epilogue passes
// the tile through LDS so that global stores (and residual loads) are 16 bytes per lane along
// rows of C.
#include "gemm_core.h"
#include "gemm_schedule.h"

namespace dl {

// Persistent workgroup: one per CU (the ring and the staging take the whole LDS), walking the tile sequence with stride
// gridDim.x; wave w owns 128 rows (M) x 64 columns (N) of the 256 x 256 tile.  Main loop: see kstep below.  Between two
// tiles the first two K-steps of the next tile are already on their way into the LDS ring while the
// epilogue of the current one drains the accumulators through a staging region of its own, and the
// C stores of a tile complete under the next tile's main loop.  Vector memory operations complete in order, so
// nothing between two tiles should wait for a load of its own (a spilled register, a table) behind the tile's loads:
// the gated pair took 346 us instead of 296 with twenty registers spilled around its epilogue.  The epilogues that read
// (residual, accumulation, rotary table, g and u) do wait: for the next tile's loads, and since their range checks are branches,
// behind which the compiler counts no store, each part of one for the stores of the part before.
//
// The kernel arguments are only read with compile-time offsets: a run-time index into the argument block
// would make the compiler copy the whole block to scratch memory and read it back through vector loads.  A
// grouped launch reads its problem through group_problem().
//
// SINGLE: every tile has one K-step.  A path of its own in the common kernel costs that 130 to 260 spilled registers, a branch in its
// loop 1 to 2 % of short contractions.
//
// Short contractions: the two wave groups take 1 to 4 thousand cycles more for a tile's fill and drain than waves in step did and
// 80 fewer for each K-step, and a short launch is not at the power limit.  us, in step / now: 4096 x K -> 4096, K = 128
// 12.4 / 12.8, 256 14.4 / 15.1, 512 19.6 / 20.2, 1024 30.2 / 30.3, 4096 95.3 / 93.8.  Not in the stores of the last tile (counted
// in the waits behind them: no change), nor in the loads of zeros behind the last one (left out: no change).
//
// EPI_SWIGLU: the gated pair of the MLP in one pass.  B interleaves the rows of two weight matrices
// (LoadStream PAIR) so that every wave holds g = x Wg^T and u = x Wu^T for the same 32 columns; the
// epilogue stores g to c, u to c2 and silu(g) * u, taken from the fp32 sums, to c3.  M x N is the interleaved
// product: N = twice the columns of g.
//
// EPI_SWIGLU_GRAD: the product is da, the gradient arriving at a = silu(g) * u; the epilogue reads the
// g and u tiles (e1, e2, leading dimension lde) and stores dg to c and du to c2, from the fp32 sums of da, instead
// of da.
//
// EPI_ROPE (grouped launch of head projections): problems flagged `rope` have the rotary embedding
// applied to their output in the epilogue, on the fp32 accumulators, so that q and k are rounded to
// bf16 once.  Rows of C are tokens (position = row % rope_seq), columns are [head][head_dim].  A wave
// owns 64 columns and needs both members of a pair: with adjacent pairs (2i, 2i+1) a lane holds them
// already; with split pairs (i, i + head_dim/2) a 64-wide head is one wave's strip, a 32-wide head half
// of one, and for 128-wide heads the B tile is loaded in partner order (PERM, every problem of the
// launch) and the epilogue stores the two 32-column runs of a wave where they belong.
enum { EPI_PLAIN = 0, EPI_SWIGLU = 1, EPI_SWIGLU_GRAD = 2, EPI_ROPE = 3 };

constexpr int PM = 256, PN = 256, PWM = 2, PWN = 4;   // tile and waves
constexpr int STAGE = (PM + PN) * BK * 2, HALF = STAGE / 4, NS = 2;
static_assert(HALF == LOADS_PER_HALF * PWM * PWN * 1024, "a half tile is sent by all waves, 1 KiB per load");

// The lane number, anew.  What the compiler computes from one that it knows is lifted out of the tile loop and spilled across the
// main loop, and its reload (counted in order behind the next tile's loads) then waits for all of those.
__device__ __forceinline__ int lane_anew() {
  int l;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
  return l;
}

// Where a tile's loads begin: prepared while the tile before it is being stored, taken up by LoadStream::begin.
struct StreamStart {
  const bf16_t *a, *b, *b2;
  uint32_t a_bytes, b_bytes, b2_bytes, lda2, ldb2;   // sizes from the tile's first element on, bytes of a row
  int k, kend, seg, m0, n0;                          // where in K, end of the segment, segment; the tile
  bool pad;                                          // one K-step, walked as two: the second is all zeros
};

// Load cursor.  A K-step is fetched in four halves of 16 KiB, two loads per wave each: A half h is 64 of the 128 rows (M index)
// of either wave row, B half h 32 of the 64 columns (N index) of each wave column.  Next to a load stands no more than
// an addition: the instructions of a load phase are on the critical path of the wave group that loads.
//   KM (both k-major): eight rows of 64 k per load, swizzled as TileLoader's tiles.  PAIR: the B halves are rows of two matrices,
//      the same rows of either.  PERM: the rows of a B half lie as the rotary partners of 128-wide heads do, half 1 holding the
//      features 64 beyond those of half 0.
//   else (both mn-major): four k-rows of 128 M (N) values per load.  A half h: columns 64 h .. of either wave row's 128; B half h: columns
//      128 h .. of the tile, so that a load reads 256 contiguous bytes (and a wave owns columns 32 w .. and 128 + 32 w ..).
template <bool KM, bool PAIR, bool PERM, bool SEGS>
struct LoadStream {
  __amdgpu_buffer_rsrc_t ra, rb, rb2;
  uint32_t va, vb;                          // lane offsets
  uint32_t sa, sb, sa0, sb0, lda2, ldb2;    // wave's offset at the present k and at k = 0; bytes of a row
  int k, kend, seg, left, m0, n0;
  bool pad;

  __device__ __forceinline__ void begin(const StreamStart& s, int total, int wave) {
    const int lane = lane_anew();
    ra = make_rsrc(s.a, s.a_bytes);
    rb = make_rsrc(s.b, s.b_bytes);
    if constexpr (PAIR) rb2 = make_rsrc(s.b2, s.b2_bytes);
    k = s.k; kend = s.kend; seg = s.seg; left = total; pad = s.pad;
    if constexpr (SEGS) { m0 = s.m0; n0 = s.n0; }
    lda2 = s.lda2;
    ldb2 = s.ldb2;
    if constexpr (KM) {
      const int row = lane >> 3, c = (lane & 7) ^ (((wave & 1) * 4 + (row >> 1)) & 7);
      va = row * lda2 + (c << 4);
      vb = row * ldb2 + (c << 4);
      const int w = wave >> 1, rows = PAIR ? w * 32 : PERM ? (w >> 1) * 128 + (w & 1) * 32 : w * 64;
      sa0 = ((wave >> 2) * 128 + (wave & 3) * 8) * lda2;
      sb0 = (rows + (wave & 1) * 8) * ldb2;
      sa = sa0 + k * 2;
      sb = sb0 + k * 2;
    } else {
      const int row = lane >> 4, c = (lane & 15) ^ ((row << 2) | (((wave >> 1) & 1) << 1));
      va = row * lda2 + (c >> 3) * 256 + (c & 7) * 16;
      vb = row * ldb2 + c * 16;
      sa0 = wave * 4 * lda2;
      sb0 = wave * 4 * ldb2;
      sa = sa0 + k * lda2;
      sb = sb0 + k * ldb2;
    }
  }
  // nothing more to fetch: loads go on and bring zeros, so that the main loop counts them as ever
  __device__ __forceinline__ void close() {
    ra = rb = make_rsrc(nullptr, 0);
    if constexpr (PAIR) rb2 = ra;
    left = LEFT_CLOSED;
    pad = false;
  }
  static __device__ __forceinline__ int a_part(int wave) { return KM ? (wave >> 2) * 16384 + (wave & 3) * 1024 : wave * 1024; }
  static __device__ __forceinline__ int b_part(int wave) { return 2 * HALF + (KM ? (wave >> 1) * 8192 + (wave & 1) * 1024 : wave * 1024); }
  // half H of A or B; `dst`: this wave's part of the stage
  template <bool A, int H>
  __device__ __forceinline__ void issue(char* dst) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const __amdgpu_buffer_rsrc_t rs = A ? ra : PAIR && H ? rb2 : rb;
      uint32_t so;
      int at;
      if constexpr (KM) {
        at = A ? H * 8192 + i * 4096 : H * 4096 + i * 2048;
        so = A ? sa + (H * 64 + i * 32) * lda2 : sb + ((PAIR ? 0 : PERM ? H * 64 : H * 32) + i * 16) * ldb2;
      } else {
        at = H * HALF + i * 8192;
        so = A ? sa + H * 128 + i * 32 * lda2 : sb + H * 256 + i * 32 * ldb2;
      }
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (LDS_PTR(void))(dst + at), 16, A ? va : vb, so, 0, 0);
    }
  }
  // One K-step on.  The walk may start anywhere in K; past the end of a segment it goes on in the next one, past the last in the first.
  __device__ __forceinline__ void advance(const GemmKArgs& p, int wave) {
    --left;
    k += BK;
    sa += KM ? BK * 2 : BK * lda2;
    sb += KM ? BK * 2 : BK * ldb2;
    if (k == kend) {
      k = 0;
      sa = sa0;
      sb = sb0;
      if constexpr (SEGS) {
        if (p.nseg > 1 && opens_segment(left)) {
          StreamStart s;
          s.seg = seg + 1 == p.nseg ? 0 : seg + 1;
          open_segment(s, p, m0, n0);
          begin(s, left, wave);
        }
      }
      if (pad) {
        ra = rb = make_rsrc(nullptr, 0);
        if constexpr (PAIR) rb2 = ra;
      }
    }
  }
  // s from its segment's beginning
  static __device__ __forceinline__ void open_segment(StreamStart& s, const GemmKArgs& p, int m0, int n0) {
    open(s, p.a[s.seg], p.b[s.seg], p.lda[s.seg], p.ldb[s.seg], p.K[s.seg], p.M, p.N, m0, n0);
    s.k = 0;
    s.pad = false;
  }
  static __device__ __forceinline__ void open(StreamStart& s, const bf16_t* a, const bf16_t* b, int64_t lda, int64_t ldb, int K, int M, int N,
                                              int m0, int n0) {
    s.kend = K;
    s.m0 = m0;
    s.n0 = n0;
    s.lda2 = (uint32_t)(lda * 2);
    s.ldb2 = (uint32_t)(ldb * 2);
    // byte offsets and sizes below 4 GiB, as every tensor is
    s.a = KM ? reinterpret_cast<const bf16_t*>(reinterpret_cast<const char*>(a) + (uint32_t)m0 * s.lda2) : a + m0;
    s.b = KM ? reinterpret_cast<const bf16_t*>(reinterpret_cast<const char*>(b) + (uint32_t)n0 * s.ldb2) : b + n0;
    s.a_bytes = KM ? (uint32_t)(M - m0 - 1) * s.lda2 + K * 2 : (uint32_t)(K - 1) * s.lda2 + (M - m0) * 2;
    s.b_bytes = KM ? (uint32_t)(N - n0 - 1) * s.ldb2 + K * 2 : (uint32_t)(K - 1) * s.ldb2 + (N - n0) * 2;
  }
};

template <bool GROUPED, bool KM, int EPI = EPI_PLAIN, bool PERM = false, bool SINGLE = false>
__device__ __forceinline__ void gemm_persistent(const GemmGroupKArgs& grp, const GemmKArgs& one) {
  constexpr int TM = PM / PWM, TN = PN / PWN, FM = TM / MI, FN = TN / MI;
  constexpr bool SWIGLU = EPI == EPI_SWIGLU;
  static_assert(TM == 128 && TN == 64, "halves, quadrants and staging are laid out for 128 x 64 per wave");
  static_assert(EPI == EPI_PLAIN || KM, "fused epilogues: k-major operands");
  static_assert(EPI == EPI_PLAIN || GROUPED == (EPI == EPI_ROPE), "the rotary epilogue is the grouped launch's, the others are not");
  static_assert(!PERM || EPI == EPI_ROPE, "partner-order tiles: rotary epilogue only");
  extern __shared__ __attribute__((aligned(1024))) char smem[];

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave_m = wave % PWM, wave_n = wave / PWM;
  int ntiles;
  if constexpr (GROUPED) {
    ntiles = grp.tile_start[1];
#pragma unroll
    for (int i = 2; i <= MAX_GROUP; ++i) if (i <= grp.n) ntiles = grp.tile_start[i];
  } else {
    ntiles = one.tiles_m * one.tiles_n;
  }

  // What the epilogue needs of a tile's problem, by value.
  struct Tile { int m0, n0, total, M, N, accumulate, rope; bf16_t* c; const bf16_t* r; int64_t ldc; };
  constexpr bool SEGS = KM && !GROUPED && EPI == EPI_PLAIN && !SINGLE;   // fused input gradients: several K-segments
  using Stream = LoadStream<KM, SWIGLU, PERM, SEGS>;
  Stream cur;

  // tile id -> tile, and where its loads begin.  The tile sequence of a problem runs in bands of 2^band_shift (8 or 4) tile
  // rows, so that the ~32 consecutive tiles an XCD holds at a time share A and B panels.
  auto locate = [&](int id, StreamStart& s) {
    int pid = xcd_contiguous(id, ntiles);
    int tiles_m, K0, shift, band_tiles, start = 0;
    uint32_t recip;
    const bf16_t *a0, *b0;
    int64_t lda0, ldb0;
    Tile t;
    auto take = [&](const auto& q) {
      tiles_m = q.tiles_m; band_tiles = q.band_tiles; recip = q.band_recip; K0 = q.K[0]; shift = q.band_rows == 4 ? 2 : 3;
      t.total = q.ksteps;
      a0 = q.a[0]; b0 = q.b[0]; lda0 = q.lda[0]; ldb0 = q.ldb[0];
      t.M = q.M; t.N = q.N; t.accumulate = q.accumulate; t.c = q.c; t.r = q.r; t.ldc = q.ldc;
      t.rope = EPI == EPI_ROPE ? q.rope : 0;
    };
    if constexpr (GROUPED) {
      // problem index: the number of problems whose first tile is not after pid
      int pi = 0;
#pragma unroll
      for (int i = 1; i < MAX_GROUP; ++i)
        if (i < grp.n && pid >= grp.tile_start[i]) { pi = i; start = grp.tile_start[i]; }
      take(group_problem(pi));   // a single K-segment (checked on the host)
      pid -= start;
    } else {
      take(one);
    }
    int band = (int)__umulhi((uint32_t)pid, recip);   // at most one too many
    if (band * band_tiles > pid) --band;
    const int first_m = band << shift, in_band = pid - band * band_tiles;
    const int band_h = tiles_m - first_m;
    if (band_h >> shift) {
      t.m0 = (first_m + (in_band & ((1 << shift) - 1))) * PM;
      t.n0 = (in_band >> shift) * PN;
    } else {   // the last band, of fewer rows
      t.m0 = (first_m + in_band % band_h) * PM;
      t.n0 = (in_band / band_h) * PN;
    }
    int first = k_start(t.m0, t.total);   // in K-steps from the start of segment 0
    s.seg = 0;
    if constexpr (SEGS) {
      for (int s2 = 0; s2 + 1 < one.nseg; ++s2)
        if (s.seg == s2 && first >= one.K[s2] / BK) { first -= one.K[s2] / BK; s.seg = s2 + 1; }
    }
    if (!SEGS || s.seg == 0) {
      Stream::open(s, a0, b0, lda0, ldb0, K0, t.M, SWIGLU ? t.N / 2 : t.N, t.m0, SWIGLU ? t.n0 / 2 : t.n0);
      if constexpr (SWIGLU) {
        s.b2 = one.b2 + (int64_t)(t.n0 / 2) * ldb0;
        s.b2_bytes = s.b_bytes;
      }
    } else {
      Stream::open_segment(s, one, t.m0, t.n0);
    }
    s.k = first * BK;
    s.pad = t.total == 1;
    t.total = max(t.total, 2);
    return t;
  };

  const int step = (int)gridDim.x;
  int id = blockIdx.x;
  if (id >= ntiles) return;
  StreamStart start;
  Tile tl = locate(id, start), next = tl;
  cur.begin(start, tl.total, wave);
  const int pa = Stream::a_part(wave), pb = Stream::b_part(wave);
  first_loads(
      tl.total & 1,
      [&](auto T, auto H) {
        constexpr int h = decltype(H)::value;
        cur.template issue<(h < HALF_B0), h & 1>(smem + decltype(T)::value * STAGE + (h < HALF_B0 ? pa : pb));
      },
      [&] { cur.advance(one, wave); });
  bool more = id + step < ntiles;
  if (more) next = locate(id + step, start);

  // Wait for the next tile's first loads (in_flight_landed).  AFTER: stores that went out behind them.
  auto landed = [&](int total, auto after) {
    constexpr int AFTER = decltype(after)::value;
    if (total & 1) wait_vmcnt<in_flight_landed(true) + AFTER>(); else wait_vmcnt<in_flight_landed(false) + AFTER>();
  };
  constexpr Int<0> C0{};
  constexpr Int<EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_GRAD ? 32 : 16> STORES{};   // of a wave, of a whole tile
  wait_vmcnt<IN_FLIGHT_FIRST>();
  int waits_from = 0;   // see tile_k_steps

  // Waves 4 to 7, the other wave of each SIMD, run one slot behind waves 0 to 3.
  const bool behind = wave >= 4;
  uint32_t cs = 0;   // the ring stage of the K-step: the K-steps of successive tiles form one stream through the ring
  while (true) {
    const Tile p = tl;
    const int m0 = p.m0, n0 = p.n0, total = p.total;
    f32x4 acc[FN][FM];
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
      for (int j = 0; j < FM; ++j) {
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;
        asm volatile("" : "+v"(acc[i][j]));   // zeroed here, not in front of the first MFMA (see mfma_quadrant)
      }
    // Lane's place in a fragment.  k-major: rows of 128 bytes, the second 32 k at this ^ 64.  mn-major: rows of 256 bytes (one k),
    // block f of 16 at this ^ 32 f.
    uint32_t lane_a, lane_b;
    const int lane0 = lane_anew();
    const uint32_t lds0 = (uint32_t)(uintptr_t)(LDS_PTR(char))(smem);
    if constexpr (KM) {
      const uint32_t l = (lane0 & 15) * (BK * 2) + (((lane0 >> 4) ^ ((lane0 >> 1) & 7)) << 4);
      lane_a = l + lds0 + wave_m * TM * BK * 2;
      lane_b = l + lds0 + 2 * HALF + wave_n * TN * BK * 2;
    } else {
      const int grp = lane0 >> 4, e = (lane0 >> 2) & 3, g = lane0 & 3;
      const uint32_t l = (grp * 8 + e) * 256 + (((g >> 1) ^ (e << 2) ^ ((grp & 1) << 1)) << 4) + (g & 1) * 8;
      lane_a = (l ^ (wave_m * 128)) + lds0;
      lane_b = (l ^ (wave_n * 64)) + lds0 + 2 * HALF;
    }
    bf16x8 fa[2][FM], fb[2][FN];
    // the wave's A or B fragments of half H
    auto read = [&](auto H, auto NEXT) {
      constexpr int h = decltype(H)::value & 1;
      constexpr bool A = decltype(H)::value < HALF_B0;
      constexpr int F = A ? FM : FN;
      auto& a = fa;
      auto& b = fb;
      const uint32_t at = (A ? lane_a : lane_b) + (decltype(NEXT)::value ? STAGE - cs : cs);
      static_for<0, 2>([&](auto kk_c) {
        constexpr int kk = decltype(kk_c)::value;
        static_for<0, F / 2>([&](auto f_c) {
          constexpr int f = decltype(f_c)::value;
          bf16x8& v = A ? a[kk][(h * F / 2 + f) % FM] : b[kk][(h * F / 2 + f) % FN];
          if constexpr (KM) lds_read<(h * F / 2 + f) * MI * BK * 2>(v, kk ? at ^ 64 : at);
          else lds_read_tr<h * HALF + kk * 8192, 1024>(v, at ^ (f * 32));
        });
      });
    };
    // waits for this wave's LDS reads and makes the half's fragments depend on it
    auto arrived = [&](auto H) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      constexpr int h = decltype(H)::value & 1;
      constexpr bool A = decltype(H)::value < HALF_B0;
      constexpr int F = A ? FM : FN;
      auto& a = fa;
      auto& b = fb;
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int f = h * F / 2; f < (h + 1) * F / 2; ++f) {
          bf16x8& v = A ? a[kk][f % FM] : b[kk][f % FN];
          asm volatile("" : "+v"(v));
        }
    };
    auto send = [&](auto H) {
      constexpr int h = decltype(H)::value;
      cur.template issue<(h < HALF_B0), h & 1>(smem + cs + (h < HALF_B0 ? pa : pb));
    };
    auto barrier = [&] {
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    };
    auto multiply = [&](auto Q, auto PHASE) {
      constexpr int q = decltype(Q)::value, ph = decltype(PHASE)::value;
      constexpr int i = (ph == 0 || ph == 3 ? q : 1 - q) * FN / 2, j = ph < 2 ? 0 : FM / 2;
      __builtin_amdgcn_sched_barrier(0);
      mfma_quadrant(acc[i][j], acc[i + 1][j], acc[i][j + 1], acc[i + 1][j + 1], acc[i][j + 2], acc[i + 1][j + 2], acc[i][j + 3],
                    acc[i + 1][j + 3], fb[0][i], fb[0][i + 1], fb[1][i], fb[1][i + 1], fa[0][j], fa[0][j + 1], fa[0][j + 2], fa[0][j + 3],
                    fa[1][j], fa[1][j + 1], fa[1][j + 2], fa[1][j + 3]);
      __builtin_amdgcn_sched_barrier(0);
    };
    // One wave group feeds the matrix pipes while the other, a slot apart, reads and loads.
    auto ops = wave_ops(read, arrived, send, [&] { wait_vmcnt<IN_FLIGHT_PHASE>(); }, barrier, multiply,
                        [&] { if (more) cur.begin(start, next.total, wave); else cur.close(); },
                        [&] { cur.advance(one, wave); }, [&] { cs = STAGE - cs; });
    if constexpr (SINGLE) tile_of_one_k_step(ops, behind, waits_from);
    else tile_k_steps(ops, total, behind, waits_from);
    mfma_drain(acc);

    // Waiting for the next tile's loads behind the epilogue's stores takes a known number of them: where the tile lies inside C.
    const bool inside = m0 + PM <= p.M && n0 + PN <= p.N;
    // Epilogue through LDS (a region behind the ring): each wave owns a [TM/4][64] bf16 staging area
    // (128 bytes per row, chunk c of row m stored at c ^ ((m >> 1) & 7)), filled from the accumulator
    // layout (8 bytes per lane) and drained row-contiguously (16 bytes per lane, 8 lanes per row); a
    // wave's tile goes through it in 4 * TN/64 pieces.
    constexpr int HM = TM / 4, HF = FM / 4;
    char* stg = smem + NS * STAGE + wave * (HM * 128);
    const int lane = lane_anew();
    const int lm = lane & (MI - 1), lq = lane / MI;
    const int rrow = lane >> 3, rpc = lane & 7;
    constexpr int TPB = 64 / MI;      // MFMA blocks per 64 staged columns
    // this lane's 4 columns of block i (within the 64 staged ones); jj: block row in the quarter
    auto stg_off = [&](int jj, int i) {
      const int row = jj * MI + lm;
      const int n = i * MI + lq * 4;
      return row * 128 + ((((n >> 3) ^ ((row >> 1) & 7)) << 4) | ((n & 4) << 1));
    };
    if constexpr (EPI == EPI_SWIGLU_GRAD) {
      // In steps of one MFMA block row (MI rows x 64 columns per wave), which keeps the registers the
      // step needs next to the accumulators few: a whole row quarter at a time made the compiler
      // spill values the main loop uses.
      const int nbase = n0 + wave_n * TN;
      constexpr int NT = MI / 8;
      // block rows whose g and u are in flight ahead of the one being worked on.  Two or three ahead
      // measure the same (three spills registers of the main loop): all workgroups reach their
      // epilogues together, and what the reads then wait for is HBM bandwidth, not latency.
      constexpr int PF = 1;
      bf16x8 gv[PF + 1][NT], uv[PF + 1][NT];
      // g and u of block row s, 16 bytes per lane along rows (the layout of the drain below)
      auto fetch = [&](int s, bf16x8 (&g8)[NT], bf16x8 (&u8)[NT]) {
        const int mbase = m0 + wave_m * TM + s * MI;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const int row = t * 8 + rrow;
          const int m = mbase + row;
          const int n = nbase + ((rpc ^ ((row >> 1) & 7)) << 3);
          const bf16x8 zero = {0, 0, 0, 0, 0, 0, 0, 0};
          g8[t] = zero;
          u8[t] = zero;
          if (m < p.M && n < p.N) {
            g8[t] = *reinterpret_cast<const bf16x8*>(one.e1 + (int64_t)m * one.lde + n);
            u8[t] = *reinterpret_cast<const bf16x8*>(one.e2 + (int64_t)m * one.lde + n);
          }
        }
      };
      // rows -> accumulator layout through the staging area
      auto to_acc_layout = [&](const bf16x8 (&v8)[NT], bf16x4 (&q)[TPB]) {
#pragma unroll
        for (int t = 0; t < NT; ++t) *reinterpret_cast<bf16x8*>(stg + (t * 8 + rrow) * 128 + (rpc << 4)) = v8[t];
#pragma unroll
        for (int i = 0; i < TPB; ++i) q[i] = *reinterpret_cast<const bf16x4*>(stg + stg_off(0, i));
      };
      auto drain = [&](int s, const bf16x4 (&q)[TPB], bf16_t* dst) {
#pragma unroll
        for (int i = 0; i < TPB; ++i) *reinterpret_cast<bf16x4*>(stg + stg_off(0, i)) = q[i];
        const int mbase = m0 + wave_m * TM + s * MI;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const int row = t * 8 + rrow;
          const int m = mbase + row;
          const int n = nbase + ((rpc ^ ((row >> 1) & 7)) << 3);
          const bf16x8 v = *reinterpret_cast<const bf16x8*>(stg + row * 128 + (rpc << 4));
          if (m < p.M && n < p.N) *reinterpret_cast<bf16x8*>(dst + (int64_t)m * p.ldc + n) = v;
        }
      };
      static_for<0, PF>([&](auto s_c) {
        constexpr int s = decltype(s_c)::value;
        fetch(s, gv[s], uv[s]);
      });
      static_for<0, FM>([&](auto s_c) {
        constexpr int s = decltype(s_c)::value;
        bf16x4 gq[TPB], uq[TPB];
        to_acc_layout(gv[s % (PF + 1)], gq);
        to_acc_layout(uv[s % (PF + 1)], uq);
        // issued before this row's stores; those sit behind branches, so the compiler's wait for it is one for them too
        if constexpr (s + PF < FM) fetch(s + PF, gv[(s + PF) % (PF + 1)], uv[(s + PF) % (PF + 1)]);
#pragma unroll
        for (int i = 0; i < TPB; ++i)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float z = (float)gq[i][e], d = acc[i][s][e];
            const float sg = logistic(z);
            gq[i][e] = (bf16_t)(d * (float)uq[i][e] * sg * (1.0f + z * (1.0f - sg)));
            uq[i][e] = (bf16_t)(d * z * sg);
          }
        if (s == 0 && more && !inside) landed(next.total, C0);
        drain(s, gq, p.c);
        drain(s, uq, one.c2);
      });
    } else if constexpr (SWIGLU) {
      // staged columns 0..31 are g, 32..63 are u, both for columns nh .. nh+31 of their matrices
      const int nh = n0 / 2 + wave_n * 32, NH = p.N / 2;
#pragma unroll
      for (int hf = 0; hf < 4; ++hf) {
        const int mbase = m0 + wave_m * TM + hf * HM;
#pragma unroll
        for (int jj = 0; jj < HF; ++jj)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16_t)acc[i][hf * HF + jj][e];
            *reinterpret_cast<bf16x4*>(stg + stg_off(jj, i)) = o;
          }
        if (hf == 0 && more && !inside) landed(next.total, C0);
#pragma unroll
        for (int t = 0; t < HM / 8; ++t) {
          const int row = t * 8 + rrow;
          const int m = mbase + row;
          const int cl = (rpc ^ ((row >> 1) & 7)) << 3;
          const int n = nh + (cl & 31);
          const bf16x8 v = *reinterpret_cast<const bf16x8*>(stg + row * 128 + (rpc << 4));
          bf16_t* dst = cl >= 32 ? one.c2 : p.c;
          if (m < p.M && n < NH) *reinterpret_cast<bf16x8*>(dst + (int64_t)m * p.ldc + n) = v;
        }
#pragma unroll
        for (int jj = 0; jj < HF; ++jj)
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float z = acc[i][hf * HF + jj][e];
              o[e] = (bf16_t)(z * logistic(z) * acc[i + 2][hf * HF + jj][e]);
            }
            *reinterpret_cast<bf16x4*>(stg + stg_off(jj, i)) = o;
          }
#pragma unroll
        for (int t = 0; t < HM / 8; ++t) {
          const int row = t * 8 + rrow;
          const int m = mbase + row;
          const int cl = (rpc ^ ((row >> 1) & 7)) << 3;
          const int n = nh + cl;
          const bf16x8 v = *reinterpret_cast<const bf16x8*>(stg + row * 128 + (rpc << 4));
          if (cl < 32 && m < p.M && n < NH) *reinterpret_cast<bf16x8*>(one.c3 + (int64_t)m * one.ldc3 + n) = v;
        }
      }
    } else {
      const int nbase = n0 + wave_n * TN;
      // Column of C of staged column cl.  Partner-order tiles: staged columns 0..31 are features (wave_n & 1) * 32 + .. of head wave_n / 2
      // of the tile, 32..63 the same features 64 further on.  mn-major B: the wave's 32 columns of either half of the tile.
      auto column = [&](int cl) {
        if constexpr (PERM) return n0 + (wave_n >> 1) * 128 + (wave_n & 1) * 32 + (cl & 31) + ((cl >> 5) << 6);
        else if constexpr (!KM) return n0 + wave_n * 32 + (cl & 31) + ((cl >> 5) << 7);
        else return nbase + cl;
      };
#pragma unroll
      for (int hf = 0; hf < 4; ++hf) {
        const int mbase = m0 + wave_m * TM + hf * HM;
        if (p.r || p.accumulate) {
          const bf16_t* src = p.r ? p.r : p.c;
#pragma unroll
          for (int t = 0; t < HM / 8; ++t) {
            const int row = t * 8 + rrow;
            const int m = mbase + row;
            const int n = column((rpc ^ ((row >> 1) & 7)) << 3);
            bf16x8 v = {0, 0, 0, 0, 0, 0, 0, 0};
            if (m < p.M && n < p.N) v = *reinterpret_cast<const bf16x8*>(src + (int64_t)m * p.ldc + n);
            *reinterpret_cast<bf16x8*>(stg + row * 128 + (rpc << 4)) = v;
          }
#pragma unroll
          for (int jj = 0; jj < HF; ++jj)
#pragma unroll
            for (int i = 0; i < TPB; ++i) {
              const bf16x4 v = *reinterpret_cast<const bf16x4*>(stg + stg_off(jj, i));
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[i][hf * HF + jj][e] += (float)v[e];
            }
        }
        if constexpr (EPI == EPI_ROPE) {
          if (p.rope) {
            const int hd2 = grp.rope_dh >> 1;
#pragma unroll
            for (int jj = 0; jj < HF; ++jj) {
              const int j = hf * HF + jj;
              const int pos = (mbase + jj * MI + lm) % grp.rope_seq;
              const float* cr = grp.rope_cos + (int64_t)pos * hd2;
              const float* sr = grp.rope_sin + (int64_t)pos * hd2;
              if (grp.rope_layout == 0) {
                // block ib holds first-half features idx .. idx+3 of a head for this lane, block pb their partners
                const bool narrow = grp.rope_dh == 32;
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                  const int idx = narrow ? lq * 4 : (PERM ? (wave_n & 1) * 32 : 0) + t * 16 + lq * 4;
                  const f32x4 c4 = *reinterpret_cast<const f32x4*>(cr + idx);
                  const f32x4 s4 = *reinterpret_cast<const f32x4*>(sr + idx);
                  auto rot = [&](f32x4& a, f32x4& b) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                      const float fa = a[e], fb = b[e];
                      a[e] = rotated_first(fa, fb, c4[e], s4[e]);
                      b[e] = rotated_second(fa, fb, c4[e], s4[e]);
                    }
                  };
                  if (narrow) rot(acc[2 * t][j], acc[2 * t + 1][j]);
                  else rot(acc[t][j], acc[t + 2][j]);
                }
              } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                  const int idx = ((nbase + i * MI + lq * 4) % grp.rope_dh) >> 1;
                  const f32x2 c2 = *reinterpret_cast<const f32x2*>(cr + idx);
                  const f32x2 s2 = *reinterpret_cast<const f32x2*>(sr + idx);
#pragma unroll
                  for (int e = 0; e < 4; e += 2) {
                    const float fa = acc[i][j][e], fb = acc[i][j][e + 1];
                    acc[i][j][e] = rotated_first(fa, fb, c2[e >> 1], s2[e >> 1]);
                    acc[i][j][e + 1] = rotated_second(fa, fb, c2[e >> 1], s2[e >> 1]);
                  }
                }
              }
            }
          }
        }
#pragma unroll
        for (int jj = 0; jj < HF; ++jj)
#pragma unroll
          for (int i = 0; i < TPB; ++i) {
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (bf16_t)acc[i][hf * HF + jj][e];
            *reinterpret_cast<bf16x4*>(stg + stg_off(jj, i)) = o;
          }
        if (hf == 0 && more && !inside) landed(next.total, C0);
#pragma unroll
        for (int t = 0; t < HM / 8; ++t) {
          const int row = t * 8 + rrow;
          const int m = mbase + row;
          const int n = column((rpc ^ ((row >> 1) & 7)) << 3);
          const bf16x8 v = *reinterpret_cast<const bf16x8*>(stg + row * 128 + (rpc << 4));
          if (m < p.M && n < p.N) *reinterpret_cast<bf16x8*>(p.c + (int64_t)m * p.ldc + n) = v;
        }
      }
    }
    if (!more) break;
    waits_from = 1;
    tl = next;
    id += step;
    more = id + step < ntiles;
    if (more) next = locate(id + step, start);   // while the stores and the loads behind them are on their way
    if (inside) landed(tl.total, STORES);
  }
  wait_vmcnt<0>();   // a closed stream's loads still write to LDS
}

template <bool KM, bool SINGLE>
__global__ __launch_bounds__(512) void gemm_kernel(const GemmKArgs p) {
  gemm_persistent<false, KM, EPI_PLAIN, false, SINGLE>(GemmGroupKArgs{}, p);
}

template <int EPI, bool SINGLE>
__global__ __launch_bounds__(512) void gemm_swiglu_kernel(const GemmKArgs p) {
  gemm_persistent<false, true, EPI, false, SINGLE>(GemmGroupKArgs{}, p);
}

template <bool KM, bool SINGLE>
__global__ __launch_bounds__(512) void gemm_group_kernel(const GemmGroupKArgs g) {
  gemm_persistent<true, KM, EPI_PLAIN, false, SINGLE>(g, g.prob[0]);
}

template <bool PERM, bool SINGLE>
__global__ __launch_bounds__(512) void gemm_group_rope_kernel(const GemmGroupKArgs g) {
  gemm_persistent<true, true, EPI_ROPE, PERM, SINGLE>(g, g.prob[0]);
}

// Tile rows per band of the tile sequence.  An XCD runs some 32 consecutive tiles at a time: 8 rows x 4
// columns of tiles with bands of 8, 4 x 8 with bands of 4 - twelve operand panels either way, but the
// wider arrangement touches longer runs of every C row (and of the g, u rows the activation-gradient
// epilogue reads).  us, bands of 8 / 4, T = 16384: K = 4096, N = 14336 1280 / 1289, N = 4096 381 / 383, gated pair 2652 / 2663;
// K = 14336, N = 4096 1316 / 1280, K = 28672 2729 / 2661; activation gradient 1590 / 1577; weight gradient 14336 x 4096
// 1427 / 1398, of T = 8192 128256 x 2048 3240 / 3147.  (On an earlier loop bands of 2 or 16 lost everywhere.)
static int band_rows_for(bool both_kmajor, int64_t k_total, bool epilogue_reads_tiles) {
  return both_kmajor && !epilogue_reads_tiles && k_total <= 4096 ? 8 : 4;
}

int compute_units() {
  static std::atomic<int> cu_count[64];   // per device; 0 = not asked yet
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev > 63) return 256;
  int cus = cu_count[dev].load(std::memory_order_relaxed);
  if (cus == 0) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 256;
    cus = n > 0 ? n : 256;
    cu_count[dev].store(cus, std::memory_order_relaxed);
  }
  return cus;
}
// One workgroup per CU (the tile's ring and staging take all of the LDS), fewer if there are fewer tiles.
static int persistent_grid(int ntiles) {
  const int cus = compute_units();
  return ntiles < cus ? ntiles : cus;
}

constexpr size_t kPersistentLds = (size_t)NS * STAGE + (size_t)PWM * PWN * (PM / PWM / 4) * 128;

static int64_t k_total(const GemmKArgs& k) {
  int64_t t = 0;
  for (int s = 0; s < k.nseg; ++s) t += k.K[s];
  return t;
}
static GemmKArgs persistent_tiling(GemmKArgs k, bool both_kmajor, bool epilogue_reads_tiles) {
  k.tiles_m = (k.M + PM - 1) / PM;
  k.tiles_n = (k.N + PN - 1) / PN;
  k.band_rows = band_rows_for(both_kmajor, k_total(k), epilogue_reads_tiles);
  k.band_tiles = k.band_rows * k.tiles_n;
  k.band_recip = (uint32_t)((((uint64_t)1 << 32) + k.band_tiles - 1) / k.band_tiles);
  k.ksteps = (int)(k_total(k) / BK);
  return k;
}

#define GEMM_LAUNCH(KERN, NTILES, ARGS, WHAT)                                                                   \
  do {                                                                                                          \
    auto kern_ = KERN;                                                                                          \
    static std::atomic<unsigned long long> lds_done{0};                                                         \
    if (int rc_ = reserve_lds(kern_, kPersistentLds, lds_done, WHAT)) return rc_;                               \
    hipLaunchKernelGGL(kern_, dim3((unsigned)persistent_grid(NTILES)), dim3(512), kPersistentLds, st, ARGS); \
    return check_launch(WHAT);                                                                                  \
  } while (0)
// The instance for products of one K-step, or the common one.  us, common (walked as two K-steps) and own instance: 4096 x 64 -> 4096 12.9,
// 11.3; 16384 x 64 -> 4096 31.0, 29.2; weight gradient 14336 x 4096 of 64 tokens 31.3, 26.5.
#define GEMM_LAUNCH_STEPS(SINGLE, NTILES, ARGS, WHAT, KERN, ...)                        \
  do {                                                                                  \
    if (SINGLE) GEMM_LAUNCH((KERN<__VA_ARGS__, true>), NTILES, ARGS, WHAT);             \
    GEMM_LAUNCH((KERN<__VA_ARGS__, false>), NTILES, ARGS, WHAT);                        \
  } while (0)

static int launch_persistent_group(const GemmKArgs* ks, int n, bool ak, bool bk, const RopeEpilogue* rope, hipStream_t st) {
  GemmGroupKArgs g{};
  g.n = n;
  bool single = true;
  for (int i = 0; i < n; ++i) {
    g.prob[i] = persistent_tiling(ks[i], ak && bk, false);
    g.tile_start[i + 1] = g.tile_start[i] + g.prob[i].tiles_m * g.prob[i].tiles_n;
    single = single && g.prob[i].ksteps == 1;
  }
  if (rope) {
    g.rope_cos = rope->cos; g.rope_sin = rope->sin;
    g.rope_seq = rope->seq; g.rope_dh = rope->head_dim; g.rope_layout = rope->layout;
    for (int i = 0; i < n; ++i) g.prob[i].rope = ks[i].rope;
    if (rope->layout == 0 && rope->head_dim == 128)
      GEMM_LAUNCH_STEPS(single, g.tile_start[n], g, "gemm group (rotary epilogue)", gemm_group_rope_kernel, true);
    GEMM_LAUNCH_STEPS(single, g.tile_start[n], g, "gemm group (rotary epilogue)", gemm_group_rope_kernel, false);
  }
  // only the layout in use is instantiated: the weight-gradient products (both operands mn-major)
  if (!ak && !bk) GEMM_LAUNCH_STEPS(single, g.tile_start[n], g, "gemm group", gemm_group_kernel, false);
  return fail(-1, "gemm group: operand layout not built");
}

static int launch_persistent(const GemmKArgs& k, bool ak, bool bk, TileEpilogue epi, hipStream_t st) {
  const GemmKArgs a = persistent_tiling(k, ak && bk, epi == TileEpilogue::SWIGLU_GRAD);
  const int ntiles = a.tiles_m * a.tiles_n;
  const bool single = a.ksteps == 1;
  if (epi == TileEpilogue::SWIGLU) GEMM_LAUNCH_STEPS(single, ntiles, a, "gemm swiglu", gemm_swiglu_kernel, EPI_SWIGLU);
  if (epi == TileEpilogue::SWIGLU_GRAD) GEMM_LAUNCH_STEPS(single, ntiles, a, "gemm swiglu grad", gemm_swiglu_kernel, EPI_SWIGLU_GRAD);
  if (ak && bk) GEMM_LAUNCH_STEPS(single, ntiles, a, "gemm", gemm_kernel, true);
  if (!ak && !bk) GEMM_LAUNCH_STEPS(single, ntiles, a, "gemm", gemm_kernel, false);
  return fail(-1, "gemm: operand layout not built");
}
#undef GEMM_LAUNCH_STEPS
#undef GEMM_LAUNCH

// ------------------------------------------------------------------------------------------
// Which kernel a product runs on.  A 256 x 256 tile has the cheapest K-step per flop, but a launch costs whole rounds
// of 256 tiles: 289 tiles take two.  So the time of every candidate is estimated from its rounds -
//   time = launch + rounds x (K-steps x step) + tile + (rounds - 1) x again, a last round that is filled to f taking step
//   lo + f (hi - lo)
// (a CU runs faster while others idle: clock, L2) - and the cheapest runs: the persistent kernel, one of the three
// tile sizes of gemm_tile.hip, or the persistent kernel for its full rounds and a smaller tile, in a second
// launch, for the rows left over.  All give the same bits.  Microseconds, from sweeps on MI355X
// (both operands k-major / an operand mn-major); per_cu: tiles of a compute unit in flight.  The constants, and the launches
// beside them, were taken before the wave groups and the loading waves, but for the fixed parts of full mn-major tiles; now
// most launches are up to 25 % quicker.  Over 115 products (256 compute units) the choice was on average 0.5 % (k-major) and 0.4 %
// (mixed) behind the best kernel, and 1.4 % (mn-major) before those fixed parts were taken again.
// ------------------------------------------------------------------------------------------
struct KernelCost { int bm, bn, per_cu; double lo, hi, tile, again; };   // again: fixed part of a workgroup's later tiles
constexpr int kPersistent = 3;
static const KernelCost kCostKK[4] = {
    {128, 256, 1, 0.62, 0.75, 4.0, 4.0},   // T = 8192, K = 4096, N = 768 (192 tiles): 50 us against 71 on 96 tiles of 256 x 256
    {128, 128, 1, 0.38, 0.48, 3.0, 3.0},   // T = 1920, K = 6272, N = 1152 (135 tiles): 44 us; 67 as 75 tiles of 128 x 256
    {64, 64, 2, 0.25, 0.33, 2.0, 2.0},     // T = 2048, K = 2816, N = 1024 (512 tiles): 20 us; 23 as 128 tiles of 128 x 128
    {256, 256, 1, 0.98, 1.39, 5.0, 5.0}};  // T = 8192, K = 5632, N = 2048 (256 tiles): 132 us
// The fixed part per tile counts where the contraction is short (a weight gradient over few tokens), and there the 256 x 256
// tile's is large: its two-stage ring starts and its accumulators drain with nothing beside them.  Less so since its wave
// groups run a slot apart: with 8.0 for 8.5 weight gradients over 128 to 384 tokens go to it, us, 128 x 256 or 128 x 128 tiles
// before: 128 tokens, 8192 x 8192 47.7, now 33.7; 192, 4096 x 4096 16.9, now 14.1; 320, 4096 x 3072 17.5, now 14.5; 512,
// 14336 x 4096 (in two launches) 79, now 69.5.  Thirty-six of 170 that changed were measured: 8 to 30 % faster, all of them.
// A workgroup's later tiles cost less, their fill and drain lie beside other tiles' K-steps, and so does a product of one K-step, which
// has its own kernel.  128 x 256 tiles before the wave groups, with them, and now: 64 tokens, 4096 x 4096 13.5, 14.1, 11.7;
// 14336 x 4096 34.2, 36.1, 26.5; 128 tokens, 14336 x 4096 41.8, 43.9, 30.9; 192 tokens 46.0, 47.6, 35.3; 256 tokens 52, 52.4,
// 40.7.  Of a grid of 6800 sizes and groups the 222 that changed were measured: 6 to 58 % faster, all of them.
static const KernelCost kCostMN[4] = {
    {128, 256, 1, 0.70, 0.85, 3.8, 3.8},   // 4096 x 4096, K = 64 (512 tiles): 13.2 us; 768 x 768, K = 8192 (18 tiles): 94 us
    {128, 128, 1, 0.48, 0.56, 2.2, 2.2},   // the first as 1024 tiles: 14.8 us; the second as 36: 63 us
    {64, 64, 2, 0.28, 0.39, 1.3, 1.3},     // as 4096 tiles: 17.2 us; as 144: 39 us
    {256, 256, 1, 1.20, 1.45, 8.0, 5.0}};  // as 9 tiles: 157 us
static const KernelCost kCostOneStep = {256, 256, 1, 1.20, 1.45, 5.5, 4.5};   // a mn-major product of one K-step: the first as 256 tiles: 11.7 us
// The persistent kernels' epilogue fetches the old value of a weight gradient 16 bytes at a time and waits for each, 5 to 6 us per tile
// where the contraction is short; the one-tile kernels ask for all of it at once.  Without this constant accumulation over few tokens ran
// on full tiles; us, 128 x 256 tiles / full ones: 64 tokens, 4160 x 5120 20.3 / 27.7; 128, 1344 x 9216 14.6 / 17.5; 192, 3584 x 10304
// 40.6 / 46.6; 256, 4160 x 13568 59.8 / 66.0; 512, 5440 x 1792 21.1 (128 x 128) / 23.8.  Not above 512 tokens, where the constants overrate the
// full tile by as much (1024, 2560 x 6400 and the like 0 to 8 % slower with it).
constexpr double kOldValueUs = 4.0;
constexpr double kLaunchUs = 3.5;

static double kernel_us(const KernelCost& c, int cus, const GemmKArgs* ks, int n) {
  int64_t tiles = 0, steps = 0;
  for (int i = 0; i < n; ++i) {
    tiles += (int64_t)((ks[i].M + c.bm - 1) / c.bm) * ((ks[i].N + c.bn - 1) / c.bn);
    const int64_t s = k_total(ks[i]) / BK;
    steps = s > steps ? s : steps;
  }
  const int64_t slots = (int64_t)c.per_cu * cus, full = tiles / slots, rem = tiles % slots;
  double us = kLaunchUs + full * steps * c.hi + c.tile + (full + (rem ? 1 : 0) - 1) * c.again;
  if (rem) us += steps * (c.lo + (c.hi - c.lo) * rem / slots);
  return us;
}

// rows [r0, r0 + rows) of a product
static GemmKArgs row_part(GemmKArgs k, int r0, int rows, bool a_kmajor) {
  for (int s = 0; s < k.nseg; ++s) k.a[s] += a_kmajor ? (int64_t)r0 * k.lda[s] : r0;
  k.c += (int64_t)r0 * k.ldc;
  if (k.c2) k.c2 += (int64_t)r0 * k.ldc;
  if (k.c3) k.c3 += (int64_t)r0 * k.ldc3;
  if (k.r) k.r += (int64_t)r0 * k.ldc;
  if (k.e1) { k.e1 += (int64_t)r0 * k.lde; k.e2 += (int64_t)r0 * k.lde; }
  k.M = rows;
  k.m_base += r0;
  return k;
}

// What a product, or a group of them, runs as: `first` takes all of it, or rows of it that `second`, in a launch of its own,
// does not (head and tail: the products, or their rows, of the two).
struct GemmPlan {
  int first, second = -1;   // index into the cost tables
  const GemmKArgs *head, *tail;   // the caller's products, or parts
  int nh = 0, nt = 0;
  GemmKArgs parts[2][MAX_GROUP];
};

static void plan_gemm(GemmPlan& p, const GemmKArgs* ks, int n, bool ak, bool bk, TileEpilogue epi, const RopeEpilogue* rope, int cus) {
  const KernelCost* cost = ak && bk ? kCostKK : kCostMN;
  int64_t longest = 0;
  for (int i = 0; i < n; ++i) longest = k_total(ks[i]) > longest ? k_total(ks[i]) : longest;
  const bool one_step = !ak && !bk && longest == BK;
  KernelCost full_tile = one_step ? kCostOneStep : cost[kPersistent];
  if (!ak && !bk && ks[0].accumulate && longest <= 512) {
    full_tile.tile += kOldValueUs;
    full_tile.again += kOldValueUs;
  }
  // a 64-column tile does not hold both members of a split pair of a 128-wide head; the persistent kernels are not built
  // for one k-major and one mn-major operand
  const bool no64 = rope && rope->layout == 0 && rope->head_dim == 128, persistent = ak == bk;
  auto best_tile = [&](const GemmKArgs* ps, int m, double& us) {
    int best = 0;
    us = kernel_us(cost[0], cus, ps, m);
    for (int c = 1; c < (no64 ? 2 : 3); ++c) {
      const double u = kernel_us(cost[c], cus, ps, m);
      if (u < us) { us = u; best = c; }
    }
    return best;
  };
  double tile_us;
  const int tile = best_tile(ks, n, tile_us);
  const double whole_us = persistent ? kernel_us(full_tile, cus, ks, n) : 1e30;
  // full rounds of the persistent kernel, the rows behind them on a smaller tile
  int64_t tiles = 0;
  for (int i = 0; i < n; ++i) tiles += (int64_t)((ks[i].M + PM - 1) / PM) * ((ks[i].N + PN - 1) / PN);
  if (persistent && tiles > cus && tiles % cus != 0) {
    int64_t room = tiles / cus * cus;
    for (int i = 0; i < n; ++i) {
      const int tn = (ks[i].N + PN - 1) / PN;
      const int64_t fit = room / tn * PM;   // rows that still fit
      const int rows = fit < ks[i].M ? (int)fit : ks[i].M;
      if (rows > 0) p.parts[0][p.nh++] = row_part(ks[i], 0, rows, ak);
      if (rows < ks[i].M) p.parts[1][p.nt++] = row_part(ks[i], rows, ks[i].M - rows, ak);
      room -= (int64_t)((rows + PM - 1) / PM) * tn;
    }
    p.head = p.parts[0];
    p.tail = p.parts[1];
    if (p.nh > 0 && p.nt > 0) {
      double tail_us;
      const int tail_tile = best_tile(p.tail, p.nt, tail_us);
      // The cut is judged with the whole fixed part for every tile: with the lower one 24 products of mn-major operands went back to
      // one launch, between 5 % faster and 1.5 % slower (1024 tokens, 10240 x 10240: 182.1 us in two launches, 184.9 in one).
      KernelCost every_tile = full_tile;
      every_tile.again = every_tile.tile;
      const double split_us = kernel_us(every_tile, cus, p.head, p.nh) + tail_us;
      // The second launch drains the chip once more, which the estimate of a launch leaves out: 3 %, and 10 % for the gated
      // pair, whose three outputs the persistent kernel stores under its next main loop (T = 2048, K = 4096,
      // F = 14336: 413 us in two launches, 406 in one, 7 % apart the other way in the estimate).
      const double margin = epi == TileEpilogue::SWIGLU ? 0.9 : 0.97;
      if (split_us < margin * kernel_us(every_tile, cus, ks, n) && split_us < tile_us) {
        p.first = kPersistent;
        p.second = tail_tile;
        return;
      }
    }
  }
  p.head = ks;
  p.nh = n;
  p.nt = 0;
  p.first = whole_us <= tile_us ? kPersistent : tile;
}

static int run_gemm(const GemmKArgs* ks, int n, bool ak, bool bk, TileEpilogue epi, const RopeEpilogue* rope, hipStream_t st,
                    const GainSums* gains = nullptr) {
  GemmPlan p;
  plan_gemm(p, ks, n, ak, bk, epi, rope, compute_units());
  if (p.first != kPersistent) return launch_gemm_tile((TileSize)p.first, p.head, p.nh, ak, bk, epi, rope, st, gains);
  if (gains)
    if (int rc = launch_gain_sums(*gains, st)) return rc;
  const int rc = p.nh > 1 || rope ? launch_persistent_group(p.head, p.nh, ak, bk, rope, st) : launch_persistent(p.head[0], ak, bk, epi, st);
  if (rc || p.second < 0) return rc;
  return launch_gemm_tile((TileSize)p.second, p.tail, p.nt, ak, bk, epi, rope, st);
}

void query_gemm_route(int operands, int epilogue, int head_dim, int cus, int n, const int64_t* M, const int64_t* N, const int64_t* K,
                      int32_t* route) {
  GemmKArgs ks[MAX_GROUP] = {};
  for (int i = 0; i < n; ++i) {
    ks[i].nseg = 1;
    ks[i].M = (int)M[i];
    ks[i].N = (int)(epilogue == GEMM_ROUTE_GATED_PAIR ? 2 * N[i] : N[i]);
    ks[i].K[0] = (int)K[i];
    ks[i].accumulate = epilogue == GEMM_ROUTE_ACCUMULATE;
  }
  RopeEpilogue rope{};
  rope.head_dim = head_dim;
  rope.layout = epilogue == GEMM_ROUTE_ROTARY_ADJACENT;
  const bool rotary = epilogue == GEMM_ROUTE_ROTARY_SPLIT || epilogue == GEMM_ROUTE_ROTARY_ADJACENT;
  const TileEpilogue epi = epilogue == GEMM_ROUTE_GATED_PAIR      ? TileEpilogue::SWIGLU
                           : epilogue == GEMM_ROUTE_GATED_GRADIENT ? TileEpilogue::SWIGLU_GRAD
                                                                   : TileEpilogue::PLAIN;
  GemmPlan p;
  plan_gemm(p, ks, n, operands != GEMM_ROUTE_MN_MN, operands == GEMM_ROUTE_K_K, epi, rotary ? &rope : nullptr,
            cus > 0 ? cus : compute_units());
  int64_t rows = 0;
  for (int i = 0; i < p.nh; ++i) rows += p.head[i].M;
  route[0] = p.first;
  route[1] = p.second;
  route[2] = (int32_t)rows;
}

static GemmKArgs kernel_args(const GemmArgs& g) {
  GemmKArgs k{};
  k.nseg = g.nseg;
  for (int s = 0; s < g.nseg; ++s) {
    k.a[s] = (const bf16_t*)g.seg[s].a;
    k.b[s] = (const bf16_t*)g.seg[s].b;
    k.lda[s] = g.seg[s].lda;
    k.ldb[s] = g.seg[s].ldb;
    k.K[s] = g.seg[s].K;
  }
  k.M = g.M;
  k.N = g.N;
  k.c = (bf16_t*)g.c;
  k.ldc = g.ldc;
  k.r = (const bf16_t*)g.r;
  k.accumulate = g.accumulate;
  return k;
}

int launch_gemm(const GemmArgs& g, hipStream_t st) {
  const GemmKArgs k = kernel_args(g);
  return run_gemm(&k, 1, g.a_kmajor, g.b_kmajor, TileEpilogue::PLAIN, nullptr, st);
}

int launch_gemm_delta(const GemmArgs& g, const DeltaEpilogue& d, bool* done, hipStream_t st) {
  const GemmKArgs k = kernel_args(g);
  GemmPlan p;
  plan_gemm(p, &k, 1, g.a_kmajor, g.b_kmajor, TileEpilogue::PLAIN, nullptr, compute_units());
  // a launch of its own costs 2 to 9 us; on the persistent kernel a wave holds half of a 128-wide head, and the
  // statistics are a hundredth of the attention backward that follows
  *done = p.first != kPersistent && g.a_kmajor && !(p.first == (int)TileSize::T64 && d.head_dim == 128);
  return *done ? launch_gemm_tile_delta((TileSize)p.first, k, g.b_kmajor, d, st)
               : run_gemm(&k, 1, g.a_kmajor, g.b_kmajor, TileEpilogue::PLAIN, nullptr, st);
}

int launch_gemm_swiglu(const void* x, int64_t ldx, const void* wg, const void* wu, int64_t ldw, int64_t T, int64_t K,
                       int64_t F, void* g, void* u, int64_t ldgu, void* a, int64_t lda, hipStream_t st) {
  GemmKArgs k{};
  k.nseg = 1;
  k.a[0] = (const bf16_t*)x;
  k.b[0] = (const bf16_t*)wg;
  k.b2 = (const bf16_t*)wu;
  k.lda[0] = ldx;
  k.ldb[0] = ldw;
  k.K[0] = (int)K;
  k.M = (int)T;
  k.N = (int)(2 * F);
  k.c = (bf16_t*)g;
  k.c2 = (bf16_t*)u;
  k.ldc = ldgu;
  k.c3 = (bf16_t*)a;
  k.ldc3 = lda;
  return run_gemm(&k, 1, true, true, TileEpilogue::SWIGLU, nullptr, st);
}

int launch_gemm_swiglu_grad(const void* dy, int64_t lddy, const void* w, bool w_kmajor, int64_t ldw, int64_t T, int64_t K, int64_t F,
                            const void* g, const void* u, int64_t ldgu, void* dg, void* du, int64_t ldd,
                            void* a, hipStream_t st) {
  GemmKArgs k{};
  k.nseg = 1;
  k.a[0] = (const bf16_t*)dy;
  k.b[0] = (const bf16_t*)w;
  k.lda[0] = lddy;
  k.ldb[0] = ldw;
  k.K[0] = (int)K;
  k.M = (int)T;
  k.N = (int)F;
  k.c = (bf16_t*)dg;
  k.c2 = (bf16_t*)du;
  k.ldc = ldd;
  k.e1 = (const bf16_t*)g;
  k.e2 = (const bf16_t*)u;
  k.lde = ldgu;
  if (!a) return run_gemm(&k, 1, true, w_kmajor, TileEpilogue::SWIGLU_GRAD, nullptr, st);
  GemmPlan p;
  plan_gemm(p, &k, 1, true, w_kmajor, TileEpilogue::SWIGLU_GRAD, nullptr, compute_units());
  // The one-tile kernels' epilogue has g and u at hand and writes a as well; with the norms' outputs from their backward
  // that takes a layer of 1920 tokens, D 1152, F 3136, two micro-batches, from 664 to 641 us.  On the persistent kernel
  // (not tried) a third run of stores would lie in an epilogue that waits for each of them, and a launch of its own is a hundredth of
  // the step.
  if (p.first != kPersistent) {
    k.c3 = (bf16_t*)a;
    return launch_gemm_tile((TileSize)p.first, &k, 1, true, w_kmajor, TileEpilogue::SWIGLU_GRAD, nullptr, st);
  }
  if (int rc = launch_swiglu_fwd_rows(g, u, T, F, ldgu, a, ldd, st)) return rc;
  return run_gemm(&k, 1, true, w_kmajor, TileEpilogue::SWIGLU_GRAD, nullptr, st);
}

static int run_group(const GemmArgs* gs, int n, const RopeEpilogue* rope, const GainSums* gains, hipStream_t st) {
  if (n < 1 || n > MAX_GROUP) return fail(-1, "gemm group: 1..%d problems, got %d", MAX_GROUP, n);
  GemmKArgs ks[MAX_GROUP];
  for (int i = 0; i < n; ++i) {
    if (gs[i].a_kmajor != gs[0].a_kmajor || gs[i].b_kmajor != gs[0].b_kmajor)
      return fail(-1, "gemm group: all problems must share one operand layout");
    if (gs[i].nseg != 1) return fail(-1, "gemm group: problems must have a single K-segment");
    ks[i] = kernel_args(gs[i]);
    if (rope) ks[i].rope = (rope->rotate_mask >> i) & 1;
  }
  if (rope) {
    if (!gs[0].a_kmajor || !gs[0].b_kmajor) return fail(-1, "gemm group: the rotary epilogue needs k-major operands");
    if (rope->head_dim != 32 && rope->head_dim != 64 && rope->head_dim != 128) return fail(-1, "gemm group: head_dim %d", rope->head_dim);
    for (int i = 0; i < n; ++i)
      if (gs[i].r || gs[i].accumulate || gs[i].N % rope->head_dim || gs[i].ldc % 8)
        return fail(-1, "gemm group: rotary epilogue on a product with residual, accumulation or partial heads");
  }
  return run_gemm(ks, n, gs[0].a_kmajor, gs[0].b_kmajor, TileEpilogue::PLAIN, rope, st, gains);
}
int launch_gemm_group(const GemmArgs* gs, int n, hipStream_t st) { return run_group(gs, n, nullptr, nullptr, st); }
int launch_gemm_group_rope(const GemmArgs* gs, int n, const RopeEpilogue* rope, hipStream_t st) { return run_group(gs, n, rope, nullptr, st); }
int launch_gemm_group_gains(const GemmArgs* gs, int n, const GainSums& gains, hipStream_t st) { return run_group(gs, n, nullptr, &gains, st); }

}  // namespace dl
