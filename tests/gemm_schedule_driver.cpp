// Replays the persistent GEMM's order of loads, waits, barriers and LDS reads (csrc/gemm_schedule.h) over tiles of even and odd
// numbers of K-steps, and checks every read of a half tile: each wave's part of the right K-step is known to have landed, by a
// wait that a barrier separates from the read, and no wave sends the next content of that place before a barrier past the
// arrival of the read.  A load counts as landed only once a wait says so: at most n in flight means all but the youngest n.
#include <cstdio>
#include <cstdlib>
#include <tuple>
#include <utility>
#include <vector>

#include "../paper_2602_08387_amd/csrc/gemm_schedule.h"

using namespace dl;

struct Tile { int total; bool inside; };   // K-steps; stores waited for by their number
struct Send { int tile, step, stage, half, epoch, landed; };
struct Read { int tile, step, stage, half, epoch, arrived; };
constexpr int NEVER = 1 << 30;

// A wave of either group; `epoch`: barriers passed.
struct Wave {
  const std::vector<Tile>& tiles;
  int epoch = 0, cs = 0, tile = 0, step = 0;   // the tile and K-step that it works on
  int to_tile = 0, to_step = 0;                // that its loads are at
  std::vector<Send> sends;
  std::vector<Read> reads;
  std::vector<int> in_flight;                  // in order: index of a send, or -1 for a store
  bool single;                                 // products of one K-step

  Wave(const std::vector<Tile>& t, bool s) : tiles(t), single(s) {}

  void send_to(int stage, int half) {
    sends.push_back({to_tile, to_step, stage, half, epoch, NEVER});
    for (int i = 0; i < LOADS_PER_HALF; ++i) in_flight.push_back((int)sends.size() - 1);
  }
  void wait_for(int n) {
    while ((int)in_flight.size() > n) {
      const int s = in_flight.front();
      in_flight.erase(in_flight.begin());
      bool last = s >= 0;
      for (int o : in_flight) last = last && o != s;
      if (last) sends[s].landed = epoch;
    }
  }
  void stores(int n) { in_flight.insert(in_flight.end(), n, -1); }

  template <class H, class Next>
  void read(H, Next) {
    const int next = Next::value;
    // behind a tile's last K-step the next tile's first is read once more, by its own first reads
    const bool over = step + next >= (single ? 1 : tiles[tile].total);
    if (!over) reads.push_back({tile, step + next, next ? 1 - cs : cs, H::value, epoch, NEVER});
  }
  template <class H>
  void arrived(H) { for (Read& r : reads) if (r.arrived == NEVER) r.arrived = epoch; }
  template <class H>
  void send(H) { send_to(cs, H::value); }
  void wait() { wait_for(IN_FLIGHT_PHASE); }
  void barrier() { ++epoch; }
  template <class Q, class P>
  void multiply(Q, P) {}
  void next_tile() {
    if (to_tile != tile || to_step != tiles[tile].total) { std::printf("loads of tile %d end at K-step %d\n", to_tile, to_step); std::exit(2); }
    ++to_tile;
    to_step = 0;
  }
  void next_k() { ++to_step; }
  void next_stage() { cs = 1 - cs; ++step; }
};

// `single`: the loop of products of one K-step, whose tiles are loaded as two
static Wave run(const std::vector<Tile>& tiles, bool single, bool behind, int store_count, int edge_stores) {
  Wave w(tiles, single);
  first_loads(
      tiles[0].total & 1, [&](auto stage, auto half) { w.send_to(decltype(stage)::value, decltype(half)::value); }, [&] { w.next_k(); });
  w.wait_for(IN_FLIGHT_FIRST);
  int waits_from = 0;
  for (w.tile = 0; w.tile < (int)tiles.size(); ++w.tile) {
    w.step = 0;
    if (single) tile_of_one_k_step(w, behind, waits_from);
    else tile_k_steps(w, tiles[w.tile].total, behind, waits_from);
    const bool more = w.tile + 1 < (int)tiles.size();
    const int landed = more ? in_flight_landed(tiles[w.tile + 1].total & 1) : 0;
    if (more && !tiles[w.tile].inside) w.wait_for(landed);
    w.stores(tiles[w.tile].inside ? store_count : edge_stores);
    waits_from = 1;
    if (more && tiles[w.tile].inside) w.wait_for(landed + store_count);
  }
  w.wait_for(0);
  return w;
}

static int check(const std::vector<Tile>& tiles, int store_count, int edge_stores, bool single = false) {
  const Wave waves[2] = {run(tiles, single, false, store_count, edge_stores), run(tiles, single, true, store_count, edge_stores)};
  int bad = 0;
  auto complain = [&](const Read& r, int reader, const char* what) {
    ++bad;
    std::printf("tiles of");
    for (const Tile& t : tiles) std::printf(" %d%s", t.total, t.inside ? "" : " (edge)");
    std::printf(" K-steps: group %d reads %s%d of tile %d, K-step %d: %s\n", reader, r.half < HALF_B0 ? "A" : "B", r.half & 1, r.tile, r.step, what);
  };
  if (waves[0].epoch != waves[1].epoch) { std::printf("barriers: %d and %d\n", waves[0].epoch, waves[1].epoch); return 1; }
  for (int reader = 0; reader < 2; ++reader)
    for (const Read& r : waves[reader].reads)
      for (const Wave& w : waves) {
        const Send* at = nullptr;     // this read's content
        const Send* next = nullptr;   // what comes to the same place after it
        for (const Send& s : w.sends) {
          if (s.stage != r.stage || s.half != r.half) continue;
          if (s.tile == r.tile && s.step == r.step) at = &s;
          else if (at && !next) next = &s;
        }
        if (!at) complain(r, reader, "never sent there");
        else if (at->landed >= r.epoch) complain(r, reader, "no wait covers it");
        if (next && next->epoch <= r.arrived) complain(r, reader, "overwritten");
      }
  return bad;
}

// A closed stream opens no segment during the two K-steps of loads that a workgroup's last tile still sends; an open one does until its
// last K-step is out.
static int check_close() {
  int left = LEFT_CLOSED, bad = 0;
  for (int i = 0; i < 2; ++i)
    if (opens_segment(--left)) ++bad, std::printf("a closed stream opens a segment\n");
  for (left = 3; left > 0;) {
    --left;
    if (opens_segment(left) != (left != 0)) ++bad, std::printf("an open stream, %d K-steps left\n", left);
  }
  return bad;
}

int main() {
  int bad = check_close(), runs = 0;
  for (int stores : {16, 32})
    for (int edge_stores : {0, 5, stores})
      for (int a = 2; a <= 7; ++a)
        for (int b = 2; b <= 7; ++b)
          for (int c = 2; c <= 7; ++c)
            for (int in = 0; in < 4; ++in, ++runs) bad += check({{a, (in & 1) != 0}, {b, (in & 2) != 0}, {c, true}}, stores, edge_stores);
  for (int edge_stores : {0, 5, 16})
    for (int in = 0; in < 4; ++in, ++runs) bad += check({{2, (in & 1) != 0}, {2, (in & 2) != 0}, {2, true}}, 16, edge_stores, true);
  bad += check({{2, true}}, 16, 0, true), ++runs;
  for (int total : {2, 3, 64, 65}) bad += check({{total, true}}, 16, 0), ++runs;
  std::printf("%d runs, %d reads not covered\n", runs, bad);
  return bad != 0;
}
