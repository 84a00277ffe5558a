// hb_tile_shape.h -- launch shapes of the tile kernel (hb_tile.hip) and the
// arithmetic of its leaf-id staging: plain C++, so that a program without a
// GPU can check them.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

#ifdef __HIP__
#define HB_HOST_DEVICE __host__ __device__
#else
#define HB_HOST_DEVICE
#endif

namespace hb {

constexpr int kTileThreads = 1024;
constexpr int kTileStage = 4;  // 16-byte pieces of a chunk per thread: chunks of up to 64 KiB
constexpr int kTileChunkMax = kTileStage * kTileThreads * 16;
constexpr int kTileChunkTrees = 64;  // trees per chunk at most
// Trees that the tables hold past the last one, for the last chunk: as many as
// a chunk may hold (64 of any size made the tables of 20 depth-11 trees four times
// as large as the trees, and took 1.2 of the 3.1 ms of their compile).
constexpr int tile_pad_trees(int tree_bytes) {
  return tree_bytes * kTileChunkTrees <= kTileChunkMax ? kTileChunkTrees : kTileChunkMax / tree_bytes;
}

// What a shape depends on besides the batch: the model's sizes and one of its
// tile tables (fp32 tile, or the rank tile with its thresholds).
struct TileSpec {
  int32_t n_trees, n_cols, n_outputs, levels, tree_bytes;
  bool rank;
  int32_t n_thr, search_steps;
};

// A launch shape: R rows per workgroup, nt trees per chunk, ilp trees a wave
// walks together (nt is a multiple of ilp for every wave group).
struct TileShape {
  int rows = 0;  // 0: does not fit
  int split = 0, parts = 1;  // chunks per workgroup of a tree split (0: all), workgroups per row tile
  int nt = 0, ilp = 0, bufs = 0, st_chunks = 0, buf_off = 0, stage_off = 0, lds = 0;
  double cost = 0;
  int tried = 0;  // estimates made to find it
};

// Leaf ids pass through LDS as 16-bit slots: st trees' columns of the
// workgroup's rows, two such buffers from stage_off on. A lane writes out four
// consecutive trees of a row.
HB_HOST_DEVICE constexpr uint32_t tile_slot_stride(int rows) { return 2u * (uint32_t)rows + 4u; }
// The staged tree read for place k of a flush of st trees: the places a lane
// has beyond the last tree read that tree's slot again (and store nothing).
HB_HOST_DEVICE constexpr int tile_flush_tree(int k, int st) { return k < st ? k : st - 1; }
// A flush starts at a multiple of nt trees, which need not be one of four: the
// 16-byte stores are declared with the alignment of an id (the hardware takes
// global stores of any size at four bytes).
constexpr int kTileIdStoreAlign = 4;

// The shape of the least estimated time in clocks: rounds of workgroups over
// the CUs, each of
//   walk    a wave-level step (node and feature read, four vector
//           instructions) every 7 clocks or a little more where enough are in
//           flight, else the 260 clocks of the dependent reads over the
//           16 ilp in flight;
//   chunks  1,300 clocks to hand a chunk over, and its bytes at 40 a clock;
//   ranks   0.22 clocks per threshold staged, 11 per search step of 64 rows.
// The constants are fitted to forced shapes on 28 to 300 columns, 60K to 1M
// rows; the shapes it takes are the fastest measured or within 10% of it.
//
// With ws_bytes a batch too small to give every CU a row tile may also divide
// the chunks of a tile among workgroups; each adds a tile load (2,000 clocks and
// 3 per value of 64 rows), and the second kernel that adds the parts takes
// about 10,000.
//
// The search runs on every call, so its cost must not grow with the trees:
//   * a split of k rounds of workgroups is cheapest with the fewest chunks per
//     workgroup that k rounds hold, so only those are tried, round by round,
//     until the rounds' loads alone exceed what is gained;
//   * a chunk size is left out where its chunks, or with a split their least
//     share, already cost more than the best shape.
// Both leave the result as trying everything gives it (time on one host core: 500
// depth-8 trees with 2-vectors, 10,000 rows 55 us, now 2.0; 3,500 trees of 31
// leaves, 7 classes, 4,000 rows 503, now 3.3).
inline TileShape best_shape(const TileSpec &t, int64_t n_rows, bool ids, int64_t ws_bytes, int lds_max, int cus) {
  TileShape best;
  const bool rank = t.rank;
  const int max_parts = (int)std::min<int64_t>(ws_bytes / (n_rows * t.n_outputs * 8), 1 << 20);
  for (int lg = rank ? 7 : 6; lg <= 10; ++lg) {
    const int R = 1 << lg, G = kTileThreads / R;
    const int64_t buf = ((int64_t)t.n_cols * R * (rank ? 2 : 4) + 15) / 16 * 16;
    const int64_t row_tiles = (n_rows + R - 1) / R;
    const double tiles = (double)row_tiles, rounds = std::ceil(tiles / cus), share = tiles / cus;
    const bool may_split = max_parts > 1 && row_tiles < cus;
    const int few_tiles = (int)std::min<int64_t>(row_tiles, cus);
    const double ranks = rank ? 0.22 * t.n_thr + 11.0 * t.search_steps * (R / 64) : 0.0;
    const double load = ws_bytes ? 2000.0 + 3.0 * t.n_cols * (R / 64) + ranks : ranks;
    // LDS of a tree's id slots: ids are written for up to 32 trees at a time (a 128-byte line per row)
    const int64_t slot = ids ? 2LL * tile_slot_stride(R) : 0;
    for (int bufs = 2; bufs >= 1; --bufs) {
      const int64_t room = buf <= lds_max ? (lds_max - buf) / (bufs * (int64_t)t.tree_bytes + slot) : 0;
      const int nt_max = (int)std::min({(int64_t)(ids ? 32 : kTileChunkTrees), room, (int64_t)kTileChunkMax / t.tree_bytes});
      for (int ilp : {1, 2, 3, 4, 8}) {
        const double step = std::max(7.0 + 1.0 / ilp, 260.0 / (16 * ilp));
        const double tree = t.levels * (R / 64) * step + t.tree_bytes / 40.0 + (bufs == 1 ? t.tree_bytes / 64.0 : 0.0);
        const double hand0 = bufs == 1 ? 2000.0 : 1300.0;
        for (int nt = G * ilp; nt <= nt_max; nt += G * ilp) {
          const int n_chunks = (t.n_trees + nt - 1) / nt;
          const double chunks = (double)n_chunks, chunk = nt * tree + hand0;
          // (a split takes at least its share of the walks, or one chunk)
          const double bound = may_split ? load + std::min(chunks * chunk, std::max(share * chunks, 1.0) * chunk + 10000.0)
                                         : rounds * (chunks * chunk + load);
          if (best.rows && bound >= best.cost) continue;  // (a shape is taken for 0.1% less, far above rounding)
          ++best.tried;
          const int64_t slots = nt * slot, stage = buf + (int64_t)bufs * nt * t.tree_bytes;
          int m = 1;
          while (ids && 2 * m * nt <= 32 && stage + 2 * m * slots <= lds_max) m *= 2;
          const double bytes = (double)nt * t.tree_bytes;
          const double walk = (double)nt * t.levels * (R / 64) * step;
          const double hand = 1300.0 + bytes / 40.0 + (bufs == 1 ? 700.0 + bytes / 64.0 : 0.0);
          double cost = rounds * (chunks * (walk + hand) + load);
          int split = 0, parts = 1;
          if (may_split) {
            const int least_per = (n_chunks + max_parts - 1) / max_parts;
            for (int k = 1;; ++k) {
              const int most = k * cus / few_tiles;  // parts that k rounds hold
              const int per = std::max((n_chunks + most - 1) / most, least_per);
              if (per < n_chunks) {
                ++best.tried;
                const int p = (n_chunks + per - 1) / per;
                const double c = std::ceil(tiles * p / cus) * (per * (walk + hand) + load) + 10000.0;
                if (c < cost || (c == cost && per < split)) {
                  cost = c;
                  split = per;
                  parts = p;
                }
              }
              // later rounds: the walks' share, and one more load each
              const double later = share * chunks * (walk + hand) + (k + 1) * load + 10000.0;
              if (per == 1 || per == least_per || later > (best.rows ? std::min(cost, best.cost) : cost)) break;
            }
          }
          if (best.rows && cost >= best.cost * 0.999) continue;
          best.cost = cost;
          best.split = split;
          best.parts = parts;
          best.rows = R;
          best.nt = nt;
          best.ilp = ilp;
          best.bufs = bufs;
          best.st_chunks = m;
          best.buf_off = (int)buf;
          best.stage_off = (int)stage;
          // (thresholds pass through all of the LDS the tile leaves; the group sums take 8 K bytes per thread)
          best.lds = rank ? lds_max : (int)std::max<int64_t>(stage + m * slots, (int64_t)kTileThreads * t.n_outputs * 8);
        }
      }
    }
  }
  return best;
}

}  // namespace hb
