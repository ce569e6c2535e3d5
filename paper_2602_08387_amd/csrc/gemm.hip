// bf16 GEMM for gfx950 (products that fill the chip; gemm_tile.hip has the others): C[M,N] = sum_s opA_s[M,K_s] * opB_s[K_s,N] (+R) with fp32 accumulation
// on v_mfma_f32_16x16x32_bf16.  One kernel template serves the three products of a linear
// layer (y = x W^T, dx = dy W, dW = dy^T x): each operand may be stored with the contraction
// index contiguous ("k-major") or with its M/N index contiguous ("mn-major").
//
// Data path: global --buffer_load ... lds (16 B per lane, no VGPR staging)--> LDS ring of NS
// stages, BK k-values each --ds_read_b128 (k-major) or ds_read_b64_tr_b16 (mn-major)--> MFMA
// operands.  Loads run NS-1 K-steps ahead of the MFMAs.  The buffer descriptor's range check
// zero-fills rows past the end of a matrix, so M and N need not be tile multiples; K_s must be a
// multiple of 64.
//
// LDS layouts (the async load puts lane l's 16 bytes at chunk l of a 1 KiB span, so swizzles
// are applied on the global-address side).  The LDS serves 256 B of banks per clock: a 16-byte
// read is done 16 lanes at a time, an 8-byte transposed read 32 lanes at a time.
//   k-major tile  [rows][BK k]   : BK*2 bytes per row = CPR chunks; chunk c of row r sits at
//                                  c ^ ((r / (16/CPR)) & (CPR-1)), so 16 consecutive rows reading
//                                  one logical chunk touch 16 different 16-byte bank groups.
//   mn-major tile [BK k][R mn]   : R/8 chunks per k-row; chunk c of k-row k sits at
//                                  c ^ ((((k & 3) << 2) | (((k >> 3) & 1) << 1)) & (R/8 - 1)): the
//                                  8 k-rows x 32 B that 32 lanes of a transposed read touch fall in
//                                  8 different 32-byte bank groups.
// MFMA roles: the N-side operand feeds MFMA "A" (row index i), the M-side operand feeds MFMA
// "B" (column index j), so a lane ends up with 4 consecutive n for one m.  The epilogue passes
// the tile through LDS so that global stores (and residual loads) are 16 bytes per lane along
// rows of C.
#include "gemm_core.h"

namespace dl {

// Persistent workgroup: one per CU, walking the tile sequence with stride gridDim.x.  Between two
// tiles the first two K-steps of the next tile are already on their way into the LDS ring while the
// epilogue of the current one drains the accumulators through a staging region of its own, and the
// C stores of a tile complete under the next tile's main loop.
//
// The kernel arguments are only read with compile-time offsets: a run-time index into the argument block
// would make the compiler copy the whole block to scratch memory and read it back through vector loads.  A
// grouped launch reads its problem through group_problem().
//
// EPI_SWIGLU: the gated pair of the MLP in one pass.  B interleaves the rows of two weight matrices
// (LoadCursor PAIR) so that every wave holds g = x Wg^T and u = x Wu^T for the same 32 columns; the
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
template <bool GROUPED, int BM, int BN, int WM, int WN, bool AK, bool BKM, int EPI = EPI_PLAIN, bool PERM = false>
__device__ __forceinline__ void gemm_persistent(const GemmGroupKArgs& grp, const GemmKArgs& one) {
  constexpr int NW = WM * WN;
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr int FM = TM / MI, FN = TN / MI;
  constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2, STAGE = A_BYTES + B_BYTES;
  // Only one wave per SIMD issues the global -> LDS loads.  The address unit takes 16 cycles per
  // wave-wide 16-byte load (1024 cycles per K-step for a 256x256x64 tile pair) and a wave blocks
  // while its loads queue up; if both waves of a SIMD do that at the same time the matrix pipe
  // starves, whereas a loading wave next to a computing wave keeps it fed (+3..6 % measured).
  constexpr int NL = NW < 4 ? NW : 4;
  using LoadA = TileLoader<BM, AK, NL>;
  using LoadB = TileLoader<BN, BKM, NL>;
  constexpr int LPW = LoadA::PER_WAVE + LoadB::PER_WAVE;   // loads per wave per stage
  static_assert(NS == 2, "the stage hand-over below is written for a two-stage ring");
  static_assert(TN % 64 == 0 && FM % 4 == 0, "staging layout: 128-byte rows, four row quarters");
  extern __shared__ __attribute__((aligned(1024))) char smem[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave_m = wave % WM, wave_n = wave / WM;
  const bool loader = wave < NL;
  int ntiles;
  if constexpr (GROUPED) {
    ntiles = grp.tile_start[1];
#pragma unroll
    for (int i = 2; i <= MAX_GROUP; ++i) if (i <= grp.n) ntiles = grp.tile_start[i];
  } else {
    ntiles = one.tiles_m * one.tiles_n;
  }

  // What the epilogue needs of a tile's problem, by value (the next tile's cursor is opened before the
  // current tile's epilogue runs).
  struct Tile { int m0, n0, total, M, N, accumulate, rope; bf16_t* c; const bf16_t* r; int64_t ldc; };
  constexpr bool SWIGLU = EPI == EPI_SWIGLU;
  LoadCursor<BM, BN, NL, AK, BKM, SWIGLU, PERM> cur;
  static_assert(EPI == EPI_PLAIN || (TN == 64 && MI == 16), "fused epilogues: one 64-column strip per wave");
  static_assert(EPI == EPI_PLAIN || GROUPED == (EPI == EPI_ROPE), "the rotary epilogue is the grouped launch's, the others are not");
  static_assert(!PERM || (EPI == EPI_ROPE && AK && BKM && BN % 128 == 0), "partner-order tiles: rotary epilogue only");

  // tile id -> tile origin, and the load cursor opened on the tile's first K-segment.  The tile
  // sequence of a problem runs in bands of band_rows (8 or 4) tile-rows, so that the ~32 consecutive
  // tiles an XCD holds at a time share A and B panels.
  auto locate = [&](int id) {
    int pid = xcd_contiguous(id, ntiles);
    int tiles_m, tiles_n, K0, GM, start = 0;
    const bf16_t *a0, *b0;
    int64_t lda0, ldb0;
    Tile t;
    auto take = [&](const auto& q) {
      tiles_m = q.tiles_m; tiles_n = q.tiles_n; K0 = q.K[0]; GM = q.band_rows > 0 ? q.band_rows : 8;
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
      take(group_problem(pi));
      pid -= start;
      cur.nseg = 1;   // grouped problems have a single K-segment (checked on the host)
      t.total = K0 / BK;
    } else {
      take(one);
      cur.nseg = one.nseg;
      t.total = 0;
      for (int s2 = 0; s2 < one.nseg; ++s2) t.total += one.K[s2] / BK;
    }
    const int band = pid / (GM * tiles_n);
    const int first_m = band * GM;
    const int band_h = min(tiles_m - first_m, GM);
    const int in_band = pid - band * GM * tiles_n;
    t.m0 = (first_m + in_band % band_h) * BM;
    t.n0 = (in_band / band_h) * BN;
    cur.left = t.total;
    int first = k_start(t.m0, t.total);   // in K-steps from the start of segment 0
    cur.seg = 0;
    if constexpr (!GROUPED) {
      for (int s2 = 0; s2 + 1 < one.nseg; ++s2)
        if (cur.seg == s2 && first >= one.K[s2] / BK) { first -= one.K[s2] / BK; cur.seg = s2 + 1; }
    }
    cur.k = first * BK;
    if (cur.seg == 0) {
      if constexpr (SWIGLU) cur.open_pair(a0, b0, one.b2, lda0, ldb0, K0, t.M, t.N, t.m0, t.n0, lane);
      else cur.open_raw(a0, b0, lda0, ldb0, K0, t.M, t.N, t.m0, t.n0, lane);
    } else {
      cur.open(one, cur.seg, t.m0, t.n0, lane);
    }
    return t;
  };

  // Load cursor: runs two K-steps ahead of the compute cursor, across segment boundaries.
  int id = blockIdx.x;
  if (id >= ntiles) return;
  Tile tl = locate(id);
  if (loader) {
    cur.issue_next(one, smem, wave, tl.m0, tl.n0, lane);
    cur.issue_next(one, smem + STAGE, wave, tl.m0, tl.n0, lane);
  }
  if (tl.total >= 2) wait_vmcnt<LPW>(); else wait_vmcnt<0>();

  // K-step s of a tile lives in ring stage (s + par) & 1: the K-steps of successive tiles form one
  // stream through the ring, so `par` moves on by the tile's number of K-steps.
  int par = 0;
  while (true) {
    const Tile p = tl;   // this tile; `tl` moves on to the next one during its last K-steps
    const int m0 = tl.m0, n0 = tl.n0, total = tl.total;
    bool early = false;
    acc_t acc[FN][FM];
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
      for (int j = 0; j < FM; ++j)
#pragma unroll
        for (int e = 0; e < NACC; ++e) acc[i][j][e] = 0.f;

    // K-step 0 has landed in every loading wave's share (waited for before the first tile, or in the
    // previous tile's epilogue); the barrier makes it visible to all waves
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");

    // Software-pipelined K loop: operand fragments are double-buffered in registers; the barrier that
    // hands over to the next stage sits before the last MFMA group of the current one, so the matrix
    // pipe stays busy while the first fragments of the next stage are fetched from LDS.
    constexpr int KK = BK / KSTEP;
    bf16x8 fa[2][FM], fb[2][FN];
    {
      const char* ta = smem + par * STAGE;
      const char* tb = ta + A_BYTES;
#pragma unroll
      for (int j = 0; j < FM; ++j) fa[0][j] = read_frag<BM, AK>(ta, wave_m * TM + j * MI, 0, lane);
#pragma unroll
      for (int i = 0; i < FN; ++i) fb[0][i] = read_frag<BN, BKM>(tb, wave_n * TN + i * MI, 0, lane);
    }
    if constexpr (!(AK && BKM)) wait_frags(fa[0], fb[0]);
    for (int t = 0; t < total; ++t) {
      // Every load of this tile is out once its last but one K-step begins.  The cursor moves on to the
      // workgroup's next tile there, and that tile's first two K-steps go out at this tile's last two
      // hand-overs like any other refill: by the time the epilogue runs they have had a K-step to land.
      if (t == total - 2 && id + (int)gridDim.x < ntiles) {
        tl = locate(id + gridDim.x);
        early = true;
      }
      char* st_cur = smem + ((t + par) & 1) * STAGE;
      const char* ta = st_cur;
      const char* tb = ta + A_BYTES;
      static_for<0, KK>([&](auto kk_c) {
        constexpr int kk = decltype(kk_c)::value;
        constexpr int cb = kk & 1, nb = cb ^ 1;
        if constexpr (AK && BKM) {
          if (kk + 1 < KK) {
#pragma unroll
            for (int j = 0; j < FM; ++j) fa[nb][j] = read_frag<BM, AK>(ta, wave_m * TM + j * MI, kk + 1, lane);
#pragma unroll
            for (int i = 0; i < FN; ++i) fb[nb][i] = read_frag<BN, BKM>(tb, wave_n * TN + i * MI, kk + 1, lane);
          } else {
            // all of this wave's reads of stage t are in registers; stage t+1 must have landed
            wait_vmcnt<0>();   // the only loads in flight are those of stage t+1, issued one K-step ago
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            // every wave now holds its last fragments of stage t in registers: refill that stage with
            // step t+2 right away, so the loads get a whole K-step to land (about 2800 cycles at 1.9 GHz
            // under sustained load; cycle counters put the wait for the slowest of them, those that
            // miss the L2, at some 300 cycles per K-step on top of that)
            if (loader) cur.issue_next(one, st_cur, wave, tl.m0, tl.n0, lane);
            // the reads go out unconditionally (after the last K-step they fetch stale bytes nobody
            // uses), which keeps them in one block with this group's MFMAs so that the scheduler
            // interleaves them (+2 %)
            const char* na = smem + ((t + 1 + par) & 1) * STAGE;
            const char* nbp = na + A_BYTES;
#pragma unroll
            for (int j = 0; j < FM; ++j) fa[nb][j] = read_frag<BM, AK>(na, wave_m * TM + j * MI, 0, lane);
#pragma unroll
            for (int i = 0; i < FN; ++i) fb[nb][i] = read_frag<BN, BKM>(nbp, wave_n * TN + i * MI, 0, lane);
          }
#pragma unroll
          for (int i = 0; i < FN; ++i)
#pragma unroll
            for (int j = 0; j < FM; ++j)
              acc[i][j] = mfma(fb[cb][i], fa[cb][j], acc[i][j]);
#pragma unroll
          for (int q = 0; q < FM + FN; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, (FM * FN) / (FM + FN), 0);  // MFMA
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                      // DS read
          }
        } else {
          // With a transposed operand the fragment reads are inline assembly (see read_frag), which the
          // scheduler neither counts nor places, so the order is fixed by hand: the group's FN rows of
          // MFMAs, each preceded by its share of the next fragments.  In the last group of a K-step the
          // first row runs before the hand-over (it only needs registers), so the matrix pipe has
          // work while the wave sits at the barrier.
          constexpr bool last = kk + 1 == KK;
          // the refill of the drained stage is spread over the rows after the hand-over: a wave is held
          // for some 27 cycles per load instruction, which its own queued MFMAs then cover (-0.15 ms)
          constexpr bool GEMM_SPREAD_LOADS = true;
          constexpr int NF = FM + FN;                       // fragments to fetch: A 0..FM-1, then B
          constexpr int NCH = last ? FN - 1 : FN;           // chunks they are spread over
          const char* ra_ = last ? smem + ((t + 1 + par) & 1) * STAGE : ta;
          const char* rb_ = ra_ + A_BYTES;
          const bool do_reads = !last || t + 1 < total;
          static_for<0, FN>([&](auto i_c) {
            constexpr int i = decltype(i_c)::value;
            if (last && i == 1) {
              wait_vmcnt<0>();   // stage t+1 has landed (loads issued one K-step ago)
              asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
              __builtin_amdgcn_s_barrier();
              asm volatile("" ::: "memory");
              if (!GEMM_SPREAD_LOADS && loader) cur.issue_next(one, st_cur, wave, tl.m0, tl.n0, lane);   // step t+2 into the drained stage
            }
            if constexpr (GEMM_SPREAD_LOADS && last && i >= 1) {
              if (loader) cur.template issue_piece<i - 1, FN - 1>(one, st_cur, wave, tl.m0, tl.n0, lane);
            }
              const int ch = last ? i - 1 : i;
            if (ch >= 0 && do_reads) {
#pragma unroll
              for (int f = ch * NF / NCH; f < (ch + 1) * NF / NCH; ++f) {
                if (f < FM) fa[nb][f] = read_frag<BM, AK>(ra_, wave_m * TM + f * MI, last ? 0 : kk + 1, lane);
                else fb[nb][f - FM] = read_frag<BN, BKM>(rb_, wave_n * TN + (f - FM) * MI, last ? 0 : kk + 1, lane);
              }
            }
#pragma unroll
            for (int j = 0; j < FM; ++j) acc[i][j] = mfma(fb[cb][i], fa[cb][j], acc[i][j]);
            __builtin_amdgcn_sched_barrier(0);
          });
          // the fragments fetched above are complete once this wait has passed; the next group's MFMAs
          // depend on it
          wait_frags(fa[nb], fb[nb]);
        }
      });
    }
    // Next tile.  Normally its cursor was opened and its first two K-steps sent during the last two
    // K-steps above; a tile of a single K-step sends them here (the last hand-over waited for every
    // load and passed a barrier after every wave's last LDS read: the whole ring is free).
    id += gridDim.x;
    const bool more = id < ntiles;
    par = (par + total) & 1;
    if (more && !early) {
      tl = locate(id);
      if (loader) {
        cur.issue_next(one, smem + par * STAGE, wave, tl.m0, tl.n0, lane);
        cur.issue_next(one, smem + (par ^ 1) * STAGE, wave, tl.m0, tl.n0, lane);
      }
    }

    // Epilogue through LDS (a region behind the ring): each wave owns a [TM/4][64] bf16 staging area
    // (128 bytes per row, chunk c of row m stored at c ^ ((m >> 1) & 7)), filled from the accumulator
    // layout (8 bytes per lane) and drained row-contiguously (16 bytes per lane, 8 lanes per row); a
    // wave's tile goes through it in 4 * TN/64 pieces.
    constexpr int HM = TM / 4, HF = FM / 4;
    char* stg = smem + NS * STAGE + wave * (HM * 128);
    const int lm = lane & (MI - 1), lq = lane / MI;
    const int rrow = lane >> 3, rpc = lane & 7;
    constexpr int TPB = 64 / MI;      // MFMA blocks per 64 staged columns
    constexpr int NG = NACC / 4;      // 4-column groups a lane holds per MFMA block
    // column (within the 64 staged ones) of group g of block i for this lane; jj: block row in the half
    auto stg_off = [&](int jj, int i, int g) {
      const int row = jj * MI + lm;
      const int n = i * MI + (MI == 32 ? g * 8 + lq * 4 : lq * 4);
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
        for (int i = 0; i < TPB; ++i) q[i] = *reinterpret_cast<const bf16x4*>(stg + stg_off(0, i, 0));
      };
      auto drain = [&](int s, const bf16x4 (&q)[TPB], bf16_t* dst) {
#pragma unroll
        for (int i = 0; i < TPB; ++i) *reinterpret_cast<bf16x4*>(stg + stg_off(0, i, 0)) = q[i];
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
        // each fetch is issued before this row's stores, so waiting for it does not wait for the stores
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
        if (s == 0 && more) {
          if (tl.total >= 2) wait_vmcnt<LPW>(); else wait_vmcnt<0>();
        }
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
            *reinterpret_cast<bf16x4*>(stg + stg_off(jj, i, 0)) = o;
          }
        if (hf == 0 && more) {
          if (tl.total >= 2) wait_vmcnt<LPW>(); else wait_vmcnt<0>();
        }
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
            *reinterpret_cast<bf16x4*>(stg + stg_off(jj, i, 0)) = o;
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
#pragma unroll
    for (int nb = 0; nb < TN / 64; ++nb) {
      const int nbase = n0 + wave_n * TN + nb * 64;
#pragma unroll
      for (int hf = 0; hf < 4; ++hf) {
        const int mbase = m0 + wave_m * TM + hf * HM;
        if (p.r || p.accumulate) {
          const bf16_t* src = p.r ? p.r : p.c;
#pragma unroll
          for (int t = 0; t < HM / 8; ++t) {
            const int row = t * 8 + rrow;
            const int m = mbase + row;
            const int n = nbase + ((rpc ^ ((row >> 1) & 7)) << 3);
            bf16x8 v = {0, 0, 0, 0, 0, 0, 0, 0};
            if (m < p.M && n < p.N) v = *reinterpret_cast<const bf16x8*>(src + (int64_t)m * p.ldc + n);
            *reinterpret_cast<bf16x8*>(stg + row * 128 + (rpc << 4)) = v;
          }
#pragma unroll
          for (int jj = 0; jj < HF; ++jj)
#pragma unroll
            for (int i = 0; i < TPB; ++i)
#pragma unroll
              for (int g = 0; g < NG; ++g) {
                const bf16x4 v = *reinterpret_cast<const bf16x4*>(stg + stg_off(jj, i, g));
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[nb * TPB + i][hf * HF + jj][g * 4 + e] += (float)v[e];
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
                  auto rot = [&](acc_t& a, acc_t& b) {
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
          for (int i = 0; i < TPB; ++i)
#pragma unroll
            for (int g = 0; g < NG; ++g) {
              bf16x4 o;
#pragma unroll
              for (int e = 0; e < 4; ++e) o[e] = (bf16_t)acc[nb * TPB + i][hf * HF + jj][g * 4 + e];
              *reinterpret_cast<bf16x4*>(stg + stg_off(jj, i, g)) = o;
            }
        // Before this tile's first store: the next tile's K-step 0 must have landed, and waiting for
        // it here (nothing younger than K-step 1 is in flight) keeps the stores out of that wait, so
        // they complete under the next main loop.
        if (nb == 0 && hf == 0 && more) {
          if (tl.total >= 2) wait_vmcnt<LPW>(); else wait_vmcnt<0>();
        }
#pragma unroll
        for (int t = 0; t < HM / 8; ++t) {
          const int row = t * 8 + rrow;
          const int m = mbase + row;
          const int cl = (rpc ^ ((row >> 1) & 7)) << 3;   // column among the wave's 64
          // partner-order tiles: staged columns 0..31 are features (wave_n & 1) * 32 + .. of head wave_n / 2 of
          // the tile, columns 32..63 the same features 64 further on
          const int n = PERM ? n0 + (wave_n >> 1) * 128 + (wave_n & 1) * 32 + (cl & 31) + ((cl >> 5) << 6) : nbase + cl;
          const bf16x8 v = *reinterpret_cast<const bf16x8*>(stg + row * 128 + (rpc << 4));
          if (m < p.M && n < p.N) *reinterpret_cast<bf16x8*>(p.c + (int64_t)m * p.ldc + n) = v;
        }
      }
    }
    }
    if (!more) break;
  }
}

template <int BM, int BN, int WM, int WN, bool AK, bool BKM>
__global__ __launch_bounds__(WM* WN * 64) void gemm_kernel(const GemmKArgs p) {
  gemm_persistent<false, BM, BN, WM, WN, AK, BKM>(GemmGroupKArgs{}, p);
}

template <int BM, int BN, int WM, int WN, int EPI>
__global__ __launch_bounds__(WM* WN * 64) void gemm_swiglu_kernel(const GemmKArgs p) {
  gemm_persistent<false, BM, BN, WM, WN, true, true, EPI>(GemmGroupKArgs{}, p);
}

template <int BM, int BN, int WM, int WN, bool AK, bool BKM>
__global__ __launch_bounds__(WM* WN * 64) void gemm_group_kernel(const GemmGroupKArgs g) {
  gemm_persistent<true, BM, BN, WM, WN, AK, BKM>(g, g.prob[0]);
}

template <int BM, int BN, int WM, int WN, bool PERM>
__global__ __launch_bounds__(WM* WN * 64) void gemm_group_rope_kernel(const GemmGroupKArgs g) {
  gemm_persistent<true, BM, BN, WM, WN, true, true, EPI_ROPE, PERM>(g, g.prob[0]);
}

// Tile rows per band of the tile sequence.  An XCD runs some 32 consecutive tiles at a time: 8 rows x 4
// columns of tiles with bands of 8, 4 x 8 with bands of 4 - twelve operand panels either way, but the
// wider arrangement touches longer runs of every C row (and of the g, u rows the activation-gradient
// epilogue reads).  Measured at the 8B shape, per launch: bands of 8 are 1-2.5 % faster for k-major
// products with K <= 4096 (q/k/v, o, gate/up forward, o input gradient), bands of 4 are 1-4 % faster for
// the long contractions (down projection, fused input gradients: +6-8 % at K = 8192), the
// activation-gradient epilogue and the weight gradients; bands of 2 or 16 lose everywhere.
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

constexpr int PM = 256, PN = 256, PWM = 2, PWN = 4;   // the persistent kernels' tile and waves
constexpr size_t kPersistentLds = (size_t)NS * (PM + PN) * BK * 2 + (size_t)PWM * PWN * (PM / PWM / 4) * 128;

static int64_t k_total(const GemmKArgs& k) {
  int64_t t = 0;
  for (int s = 0; s < k.nseg; ++s) t += k.K[s];
  return t;
}
static GemmKArgs persistent_tiling(GemmKArgs k, bool both_kmajor, bool epilogue_reads_tiles) {
  k.tiles_m = (k.M + PM - 1) / PM;
  k.tiles_n = (k.N + PN - 1) / PN;
  k.band_rows = band_rows_for(both_kmajor, k_total(k), epilogue_reads_tiles);
  return k;
}

#define GEMM_LAUNCH(KERN, NTILES, ARGS, WHAT)                                                                   \
  do {                                                                                                          \
    auto kern_ = KERN;                                                                                          \
    static std::atomic<unsigned long long> lds_done{0};                                                         \
    if (int rc_ = reserve_lds(kern_, kPersistentLds, lds_done, WHAT)) return rc_;                               \
    hipLaunchKernelGGL(kern_, dim3((unsigned)persistent_grid(NTILES)), dim3(PWM * PWN * 64), kPersistentLds, st, ARGS); \
    return check_launch(WHAT);                                                                                  \
  } while (0)

static int launch_persistent_group(const GemmKArgs* ks, int n, bool ak, bool bk, const RopeEpilogue* rope, hipStream_t st) {
  GemmGroupKArgs g{};
  g.n = n;
  for (int i = 0; i < n; ++i) {
    g.prob[i] = persistent_tiling(ks[i], ak && bk, false);
    g.tile_start[i + 1] = g.tile_start[i] + g.prob[i].tiles_m * g.prob[i].tiles_n;
  }
  if (rope) {
    g.rope_cos = rope->cos; g.rope_sin = rope->sin;
    g.rope_seq = rope->seq; g.rope_dh = rope->head_dim; g.rope_layout = rope->layout;
    for (int i = 0; i < n; ++i) g.prob[i].rope = ks[i].rope;
    if (rope->layout == 0 && rope->head_dim == 128)
      GEMM_LAUNCH((gemm_group_rope_kernel<PM, PN, PWM, PWN, true>), g.tile_start[n], g, "gemm group (rotary epilogue)");
    GEMM_LAUNCH((gemm_group_rope_kernel<PM, PN, PWM, PWN, false>), g.tile_start[n], g, "gemm group (rotary epilogue)");
  }
  // only the layout in use is instantiated: the weight-gradient products (both operands mn-major)
  if (!ak && !bk) GEMM_LAUNCH((gemm_group_kernel<PM, PN, PWM, PWN, false, false>), g.tile_start[n], g, "gemm group");
  return fail(-1, "gemm group: operand layout not built");
}

static int launch_persistent(const GemmKArgs& k, bool ak, bool bk, TileEpilogue epi, hipStream_t st) {
  const GemmKArgs a = persistent_tiling(k, ak && bk, epi == TileEpilogue::SWIGLU_GRAD);
  const int ntiles = a.tiles_m * a.tiles_n;
  if (epi == TileEpilogue::SWIGLU) GEMM_LAUNCH((gemm_swiglu_kernel<PM, PN, PWM, PWN, EPI_SWIGLU>), ntiles, a, "gemm swiglu");
  if (epi == TileEpilogue::SWIGLU_GRAD) GEMM_LAUNCH((gemm_swiglu_kernel<PM, PN, PWM, PWN, EPI_SWIGLU_GRAD>), ntiles, a, "gemm swiglu grad");
  if (ak && bk) GEMM_LAUNCH((gemm_kernel<PM, PN, PWM, PWN, true, true>), ntiles, a, "gemm");
  if (!ak && !bk) GEMM_LAUNCH((gemm_kernel<PM, PN, PWM, PWN, false, false>), ntiles, a, "gemm");
  return fail(-1, "gemm: operand layout not built");
}
#undef GEMM_LAUNCH

// ------------------------------------------------------------------------------------------
// Which kernel a product runs on.  A 256 x 256 tile has the cheapest K-step per flop, but a launch costs whole rounds
// of 256 tiles: 289 tiles take two.  So the time of every candidate is estimated from its rounds -
//   time = launch + rounds x (K-steps x step + tile), a last round that is filled to f taking step lo + f (hi - lo)
// (a CU runs faster while others idle: clock, L2) - and the cheapest runs: the persistent kernel, one of the three
// tile sizes of gemm_tile.hip, or the persistent kernel for its full rounds and a smaller tile, in a second
// launch, for the rows left over.  All give the same bits.  Microseconds, from sweeps on MI355X
// (both operands k-major / an operand mn-major); per_cu: tiles of a compute unit in flight.  The estimates are within 10 % of
// the measured launches from 15 us up (256 compute units).
// ------------------------------------------------------------------------------------------
struct KernelCost { int bm, bn, per_cu; double lo, hi, tile; };
constexpr int kPersistent = 3;
static const KernelCost kCostKK[4] = {
    {128, 256, 1, 0.62, 0.75, 4.0},   // T = 8192, K = 4096, N = 768 (192 tiles): 50 us against 71 on 96 tiles of 256 x 256
    {128, 128, 1, 0.38, 0.48, 3.0},   // T = 1920, K = 6272, N = 1152 (135 tiles): 44 us; 67 as 75 tiles of 128 x 256
    {64, 64, 2, 0.25, 0.33, 2.0},     // T = 2048, K = 2816, N = 1024 (512 tiles): 20 us; 23 as 128 tiles of 128 x 128
    {256, 256, 1, 0.98, 1.39, 5.0}};  // T = 8192, K = 5632, N = 2048 (256 tiles): 132 us
// The fixed part per tile counts where the contraction is short (a weight gradient over few tokens), and there the 256 x 256
// tile's is large: its two-stage ring starts and its accumulators drain with nothing beside them.
static const KernelCost kCostMN[4] = {
    {128, 256, 1, 0.70, 0.85, 3.8},   // 4096 x 4096, K = 64 (512 tiles): 13.2 us; 768 x 768, K = 8192 (18 tiles): 94 us
    {128, 128, 1, 0.48, 0.56, 2.2},   // the first as 1024 tiles: 14.8 us; the second as 36: 63 us
    {64, 64, 2, 0.28, 0.39, 1.3},     // as 4096 tiles: 17.2 us; as 144: 39 us
    {256, 256, 1, 1.20, 1.45, 8.5}};  // as 256 tiles: 15.6 us; as 9: 157 us
constexpr double kLaunchUs = 3.5;

static double kernel_us(const KernelCost& c, int cus, const GemmKArgs* ks, int n) {
  int64_t tiles = 0, steps = 0;
  for (int i = 0; i < n; ++i) {
    tiles += (int64_t)((ks[i].M + c.bm - 1) / c.bm) * ((ks[i].N + c.bn - 1) / c.bn);
    const int64_t s = k_total(ks[i]) / BK;
    steps = s > steps ? s : steps;
  }
  const int64_t slots = (int64_t)c.per_cu * cus, full = tiles / slots, rem = tiles % slots;
  double us = kLaunchUs + full * (steps * c.hi + c.tile);
  if (rem) us += steps * (c.lo + (c.hi - c.lo) * rem / slots) + c.tile;
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
  const double whole_us = persistent ? kernel_us(cost[kPersistent], cus, ks, n) : 1e30;
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
      const double split_us = kernel_us(cost[kPersistent], cus, p.head, p.nh) + tail_us;
      // The second launch drains the chip once more, which the estimate of a launch leaves out: 3 %, and 10 % for the gated
      // pair, whose three outputs the persistent kernel stores under its next main loop (T = 2048, K = 4096,
      // F = 14336: 413 us in two launches, 406 in one, 7 % apart the other way in the estimate).
      const double margin = epi == TileEpilogue::SWIGLU ? 0.9 : 0.97;
      if (split_us < margin * whole_us && split_us < tile_us) {
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

static int run_gemm(const GemmKArgs* ks, int n, bool ak, bool bk, TileEpilogue epi, const RopeEpilogue* rope, hipStream_t st) {
  GemmPlan p;
  plan_gemm(p, ks, n, ak, bk, epi, rope, compute_units());
  if (p.first != kPersistent) return launch_gemm_tile((TileSize)p.first, p.head, p.nh, ak, bk, epi, rope, st);
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
                            hipStream_t st) {
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
  return run_gemm(&k, 1, true, w_kmajor, TileEpilogue::SWIGLU_GRAD, nullptr, st);
}

int launch_gemm_group(const GemmArgs* gs, int n, hipStream_t st) { return launch_gemm_group_rope(gs, n, nullptr, st); }

int launch_gemm_group_rope(const GemmArgs* gs, int n, const RopeEpilogue* rope, hipStream_t st) {
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
  return run_gemm(ks, n, gs[0].a_kmajor, gs[0].b_kmajor, TileEpilogue::PLAIN, rope, st);
}

}  // namespace dl
