// scan.hpp built for the CPU (hip_cpu/): the tile numbers, the prefixes of
// both walks on either side of the line between them, and a wait that runs
// out.  Prints "ok".
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <numeric>
#include <random>
#include <thread>

#include "scan.hpp"

#define CHECK(c)                                                            \
  do {                                                                      \
    if (!(c)) {                                                             \
      std::fprintf(stderr, "check failed at line %d: %s\n", __LINE__, #c); \
      std::exit(1);                                                         \
    }                                                                       \
  } while (0)

// Whatever workgroups have started, in whatever order, their tiles are the
// first ones: a tile whose workgroup has not started (kept out, for instance,
// by other kernels' waiting workgroups on the CUs it would run on) has no
// successor that waits for it.
static void tickets_follow_the_start_order() {
  constexpr int kBlocks = 96;
  std::mt19937 rng(7);
  for (int trial = 0; trial < 12; ++trial) {
    std::vector<unsigned> order(kBlocks);
    std::iota(order.begin(), order.end(), 0u);
    if (trial > 0) std::shuffle(order.begin(), order.end(), rng);
    if (trial > 6)   // the workgroups of one XCD start last
      std::stable_partition(order.begin(), order.end(), [&](unsigned b) { return b % 8 != unsigned(trial) % 8; });
    std::vector<uint32_t> counters(1024, 0);   // at least what a scan's ticket takes
    int last = -1;
    for (int started = 1; started <= kBlocks; ++started) {
      int tile = -1, s_tile = -1;
      cpu::run_block(order[started - 1], 64, [&] {
        const int t = gmb::claim_tile(counters.data(), &s_tile);
        if (threadIdx.x == 0) tile = t;
      });
      last = std::max(last, tile);
      CHECK(last + 1 == started);
    }
  }
}

// One workgroup of BLOCK threads takes all tiles in turn.
template <int BLOCK, int NV>
static void prefixes(int tiles) {
  std::mt19937 rng(tiles);
  std::vector<int32_t> agg(static_cast<size_t>(tiles) * NV);
  for (auto& a : agg) a = static_cast<int32_t>(rng() % 4097);
  std::vector<uint64_t> words(static_cast<size_t>(tiles) * NV, 0);
  std::vector<int32_t> smem(NV * (BLOCK / 64)), want(NV, 0);
  cpu::run_block(0, BLOCK, [&] {
    for (int t = 0; t < tiles; ++t) {
      int32_t a[NV], ex[NV];
      for (int v = 0; v < NV; ++v) a[v] = agg[t * NV + v];
      CHECK((gmb::tile_prefix<BLOCK, NV>(words.data(), tiles, t, tiles, a, ex, smem.data())));
      for (int v = 0; v < NV; ++v) CHECK(ex[v] == want[v]);
      __syncthreads();
      if (threadIdx.x == 0)
        for (int v = 0; v < NV; ++v) want[v] += a[v];
      __syncthreads();
    }
  });
}

// Three workgroups take tiles by ticket, side by side.
static void prefixes_side_by_side(int tiles) {
  constexpr int BLOCK = 64;
  std::vector<uint64_t> words(tiles, 0);
  std::vector<uint32_t> counters(1024, 0);
  std::vector<std::thread> groups;
  for (unsigned b = 0; b < 3; ++b)
    groups.emplace_back([&, b] {
      int s_tile = 0;
      int32_t smem[BLOCK / 64];
      cpu::run_block(b, BLOCK, [&] {
        for (;;) {
          const int t = gmb::claim_tile(counters.data(), &s_tile);
          __syncthreads();
          if (t >= tiles) break;
          int32_t a[1] = {t + 1}, ex[1];
          CHECK((gmb::tile_prefix<BLOCK, 1>(words.data(), 0, t, tiles, a, ex, smem)));
          CHECK(ex[0] == t * (t + 1) / 2);
          __syncthreads();
        }
      });
    });
  for (auto& g : groups) g.join();
}

// The predecessor never publishes: the wait ends, every thread hears of it,
// and the tile has published something for its own successors.
static void a_wait_that_runs_out(int tiles) {
  constexpr int BLOCK = 128;
  std::vector<uint64_t> words(tiles, 0);
  int32_t smem[BLOCK / 64];
  cpu::run_block(0, BLOCK, [&] {
    int32_t a[1] = {5}, ex[1];
    CHECK(!(gmb::tile_prefix<BLOCK, 1>(words.data(), 0, 1, tiles, a, ex, smem, 20)));
  });
  CHECK(words[1] != 0);
}

int main() {
  tickets_follow_the_start_order();
  for (int tiles : {1, 2, 65, gmb::kFlatTiles, gmb::kFlatTiles + 1}) {
    prefixes<64, 1>(tiles);
    if (tiles <= 65) prefixes<256, 3>(tiles);
  }
  prefixes<128, 2>(gmb::kFlatTiles + 77);
  prefixes_side_by_side(200);
  prefixes_side_by_side(gmb::kFlatTiles + 40);
  a_wait_that_runs_out(2);
  a_wait_that_runs_out(gmb::kFlatTiles + 1);
  std::puts("ok");
}
