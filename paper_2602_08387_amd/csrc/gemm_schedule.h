// Order of the loads, waits, barriers and LDS reads of the persistent GEMM (gemm.hip), apart from what each of them does: the kernel
// runs these functions with its own operations, and a host program replays them with a model of the wait counter and of the
// two wave groups (tests/gemm_schedule_driver.cpp).  Nothing else orders the asynchronous global -> LDS loads against
// the reads, and a read that no wait covers finds the right data nearly always, so running the kernel does not tell.
#pragma once
#include <type_traits>

#if defined(__HIP__)
#define DL_SCHEDULE __device__ inline __attribute__((always_inline))
#else
#define DL_SCHEDULE inline
#endif

namespace dl {

template <int V> using Int = std::integral_constant<int, V>;

// The halves of a K-step's two tiles, each sent by all waves together, LOADS_PER_HALF loads each.
enum { HALF_A0 = 0, HALF_A1 = 1, HALF_B0 = 2, HALF_B1 = 3 };
constexpr int LOADS_PER_HALF = 2;

// A K-step has four phases, one quadrant of the wave's tile each: A0 Bq, A0 Bq', A1 Bq', A1 Bq (q' = 1 - q).  q = 1 for the last
// K-step of a tile and every other before it, so that the next K-step's first B half can be read before this one's last is
// done with.  The half that is read for the next phase (from phase 2 on one of the next K-step), and the half of the K-step after
// next that is sent, into what every wave has read since two phases:
constexpr int half_read(int q, int phase) { return phase == 1 ? HALF_A1 : phase == 2 ? HALF_A0 : HALF_B1 - q; }
constexpr int half_sent(int q, int phase) { return phase == 0 ? HALF_A0 : phase == 1 ? HALF_B0 + q : phase == 2 ? HALF_B1 - q : HALF_A1; }

// Loads that may still be in flight, of this wave (they land in the order in which they went out).
// A phase: the half that the next phase reads went out six phases ago, five halves are younger.
constexpr int IN_FLIGHT_PHASE = 5 * LOADS_PER_HALF;
// A workgroup's first tile: A half 0 and the B halves of K-step 0 have landed.
constexpr int IN_FLIGHT_FIRST = 5 * LOADS_PER_HALF;
// Another tile: K-step 0 has landed, and of K-step 1 what the first three phases are not going to wait for, its first two
// halves (three where K-step 0 has q = 1).
constexpr int in_flight_landed(bool odd) { return (odd ? 1 : 2) * LOADS_PER_HALF; }

// K-steps that a stream of loads has left.  Past the end of a K-segment it opens the next one, but not behind the workgroup's last tile, where
// loads go on and bring zeros so that the main loop counts them as ever.
constexpr int LEFT_CLOSED = 0;
constexpr bool opens_segment(int left) { return left > 0; }

// What one wave does in the main loop.  read(H, NEXT): the fragments of half H from this K-step's stage of the ring or the next
// one's; arrived(H): waits for them; send(H): half H into this stage; wait(): until at most IN_FLIGHT_PHASE loads are in flight; barrier():
// all waves; multiply(Q, PHASE); next_tile(): the loads go on with the workgroup's next tile; next_k(): they go on to the
// next K-step; next_stage(): the ring turns.
template <class Read, class Arrived, class Send, class Wait, class Barrier, class Multiply, class NextTile, class NextK, class NextStage>
struct WaveOps {
  Read read; Arrived arrived; Send send; Wait wait; Barrier barrier; Multiply multiply; NextTile next_tile; NextK next_k; NextStage next_stage;
};
template <class... F>
DL_SCHEDULE WaveOps<F...> wave_ops(F... f) { return {f...}; }

// The first two K-steps of a workgroup's first tile, to stages 0 and 1: send(STAGE, H).  The B halves of K-step 1 go in the order
// in which it wants them, as all later ones do, since IN_FLIGHT_PHASE counts on it; both of K-step 0 are waited for.
template <class Send, class NextK>
DL_SCHEDULE void first_loads(bool odd, Send&& send, NextK&& next_k) {
  send(Int<0>{}, Int<HALF_A0>{});
  send(Int<0>{}, Int<HALF_B0>{});
  send(Int<0>{}, Int<HALF_B1>{});
  send(Int<0>{}, Int<HALF_A1>{});
  next_k();
  send(Int<1>{}, Int<HALF_A0>{});
  if (odd) {
    send(Int<1>{}, Int<HALF_B0>{});
    send(Int<1>{}, Int<HALF_B1>{});
  } else {
    send(Int<1>{}, Int<HALF_B1>{});
    send(Int<1>{}, Int<HALF_B0>{});
  }
  send(Int<1>{}, Int<HALF_A1>{});
  next_k();
}

template <int Q, int PHASE, class W>
DL_SCHEDULE void k_step_from(W& w, bool waits) {
  if constexpr (PHASE < 4) {
    constexpr Int<half_read(Q, PHASE)> H{};
    // a slot of memory work
    w.read(H, Int<PHASE / 2>{});
    w.send(Int<half_sent(Q, PHASE)>{});
    if (PHASE == 3 || waits) w.wait();
    w.barrier();
    // a slot of MFMAs
    w.multiply(Int<Q>{}, Int<PHASE>{});
    w.arrived(H);
    w.barrier();
    if constexpr (PHASE == 3) w.next_k();
    k_step_from<Q, PHASE + 1>(w, waits);
  }
}

// A tile's first fragments; `odd`: an odd number of K-steps.
template <class W>
DL_SCHEDULE void open_tile(W& w, bool odd, bool behind) {
  w.barrier();   // K-step 0 has landed in every wave's share: visible to all waves
  w.read(Int<HALF_A0>{}, Int<0>{});
  if (odd) w.read(Int<HALF_B1>{}, Int<0>{}); else w.read(Int<HALF_B0>{}, Int<0>{});
  w.arrived(Int<HALF_A0>{});
  w.arrived(Int<HALF_B0>{});
  w.arrived(Int<HALF_B1>{});
  w.barrier();   // before the first load into this stage
  if (behind) w.barrier();
}

// The K-steps of one tile, at least two.  `behind`: the wave belongs to the group that runs one slot behind the other.  waits_from: K-step from
// which on the first three phases wait for loads; 1 in a workgroup's later tiles, where what they read in K-step 0 has landed
// (waiting there would be for the last tile's stores).
template <class W>
DL_SCHEDULE void tile_k_steps(W& w, int total, bool behind, int waits_from) {
  const bool odd = total & 1;
  open_tile(w, odd, behind);
  if (odd) {
    k_step_from<1, 0>(w, waits_from == 0);
    w.next_stage();
  }
  for (int t = odd; t < total; t += 2) {
    if (t == total - 2) w.next_tile();   // every load of this tile is out
    k_step_from<0, 0>(w, t >= waits_from);
    w.next_stage();
    k_step_from<1, 0>(w, t + 1 >= waits_from);
    w.next_stage();
  }
  if (!behind) w.barrier();
}

// A tile of one K-step, where all tiles are such: loaded as two, of which the second brings zeros that nothing reads; its place
// takes the second of the next tile, in the order in which phases would send it.
template <class W>
DL_SCHEDULE void tile_of_one_k_step(W& w, bool behind, int waits_from) {
  open_tile(w, false, behind);
  w.next_tile();
  k_step_from<0, 0>(w, waits_from == 0);
  w.next_stage();
  w.send(Int<half_sent(1, 0)>{});
  w.send(Int<half_sent(1, 1)>{});
  w.send(Int<half_sent(1, 2)>{});
  w.send(Int<half_sent(1, 3)>{});
  w.next_k();
  w.next_stage();
  if (!behind) w.barrier();
}

}  // namespace dl
