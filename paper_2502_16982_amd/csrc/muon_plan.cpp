// Host-side launch planner of the Muon step (see muon_plan.h).  Plain C++: no HIP header, no device call.
#include "muon_plan.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>

namespace muon {

namespace {

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
inline int round_up_i(int64_t v, int a) { return (int)((v + a - 1) / a * a); }

// Iterate-sized buffers per matrix: X and Xt[0] always; Xt[1] on the fp32 path (transpose ping-pong) and, on the
// bf16 path, only for matrices iterated on their transpose (it receives O in W's orientation).
int x_buffers(const MatPlan& q, int ns_dtype) { return (!on_matrix_cores(ns_dtype) || q.transposed) ? 3 : 2; }

// Workgroups are handed to the 8 accelerator dies (XCDs, each with a private L2) round-robin by workgroup index:
// entry b of a tile table runs on XCD b % 8.  Tiles that share operand panels are therefore dealt to the same
// XCD: when a launch holds many problems, each goes whole to the least-loaded XCD; otherwise every problem is
// cut into 8 contiguous runs of its tile list.  Problems arrive longest-first, so the tail of a launch is made of
// short tiles.
constexpr int kXcds = 8;

GemmTile make_tile(int32_t prob, int row0, int col0, int shape, int flags) {
  GemmTile t{};
  t.prob = prob;
  t.r0 = (uint16_t)(row0 / kTileUnit);
  t.c0 = (uint16_t)(col0 / kTileUnit);
  t.shape = (uint8_t)shape;
  t.flags = (uint8_t)flags;
  t.pad_ = 0;
  return t;
}

// Square tiles of `size` elements over a tm x tn grid, in an order whose consecutive runs of 32 (one tile per compute
// unit of an XCD) form BH x BW blocks of the grid: the 32 tiles running together on an XCD then share BH row panels
// and BW column panels, which they sweep along k in step, instead of 1 + 32 panels for a row-major run.
// Tiles (i, j) with i < skip_m and j < skip_n are left out (a coarser shape covers them), as is column skip_col
// (covered by strip tiles; -1: none).  upper_only: tiles on or above the diagonal; those on it get kTileDiagonal and,
// when diag_shape >= 0, that shape.
// `cuts` receives the list positions at which a block ends.
void blocked_tiles(int32_t prob, int size, int shape, int tm, int tn, bool upper_only, int skip_m, int skip_n, int skip_col,
                   std::vector<GemmTile>& out, std::vector<int>& cuts, int BH = 4, int BW = 8, int diag_shape = -1) {
  for (int bi = 0; bi < tm; bi += BH)
    for (int bj = 0; bj < tn; bj += BW) {
      for (int i = bi; i < std::min(bi + BH, tm); ++i)
        for (int j = bj; j < std::min(bj + BW, tn); ++j)
          if ((!upper_only || j >= i) && !(i < skip_m && j < skip_n) && j != skip_col) {
            const bool diag = upper_only && i == j;
            out.push_back(make_tile(prob, i * size, j * size, diag && diag_shape >= 0 ? diag_shape : shape, diag ? kTileDiagonal : 0));
          }
      if (!out.empty() && (cuts.empty() || cuts.back() != (int)out.size())) cuts.push_back((int)out.size());
    }
}

// 512 x 128 tiles over the 128-wide column strip [0, rows) x [col0, col0 + 128) of an output (rows >= 512, a multiple
// of 128).  The last tile is shifted up to end at `rows`; where it overlaps its neighbour both compute the same
// values from the same operands in the same order.
void strip_tiles(int32_t prob, int rows, int col0, std::vector<GemmTile>& out, std::vector<int>& cuts) {
  const int H = kShapeRows[kShape512x128];
  for (int r0 = 0; r0 < rows; r0 += H) out.push_back(make_tile(prob, std::min(r0, rows - H), col0, kShape512x128, 0));
  cuts.push_back((int)out.size());
}

// A persistent launch (one block per compute unit striding through the table) gives every block the same number of
// tiles only if the table length is a multiple of the number of blocks; the r tiles beyond that cost the launch a whole
// extra round.  When r is small they are taken out of the coarse lists - plain 256 x 256 tiles from the end of the
// problems that come last in the launch order - and handed to the fine launch, four 128 x 128 tiles each, where they
// run side by side, one per compute unit.  With several planes no launch is persistent, and what the moved tiles gain is that
// they run as 64 x 64 blocks: `most` is then what a launch in quarters holds (2 of 4096^2, 16 tiles, 7590 / 7510 us without / with
// the move, three planes 13550 / 13300; apply product of 2 of 2560 x 3328, 4 tiles, 2585 / 2504 and 4374 / 4260; but 16 of 2048 x
// 8192, whose 64 would run 128 wide again, 24910 / 25350).
// `moved` receives them per problem; returns how many were moved.
constexpr int kMaxMovedTiles = 64;
size_t move_tail_to_fine(const std::vector<int>& order, std::vector<std::vector<GemmTile>>& lists,
                         std::vector<std::vector<int>>& cuts, int blocks, int most, std::vector<std::vector<GemmTile>>& moved) {
  size_t total = 0;
  for (const auto& l : lists) total += l.size();
  if (blocks <= 0 || total <= (size_t)blocks) return 0;
  const size_t r = total % (size_t)blocks;
  if (r == 0 || r > (size_t)most) return 0;
  size_t plain = 0;
  for (const auto& l : lists)
    for (const GemmTile& t : l) plain += (t.shape == kShape256 && !(t.flags & kTileDiagonal)) ? 1 : 0;
  if (plain < r) return 0;
  size_t left = r;
  for (size_t oi = order.size(); oi-- > 0 && left > 0;) {
    std::vector<GemmTile>& l = lists[order[oi]];
    for (size_t i = l.size(); i-- > 0 && left > 0;)
      if (l[i].shape == kShape256 && !(l[i].flags & kTileDiagonal)) {
        moved[order[oi]].push_back(l[i]);
        l.erase(l.begin() + (std::ptrdiff_t)i);
        --left;
      }
    // block boundaries are list positions: those past the shortened list go
    std::vector<int>& c = cuts[order[oi]];
    while (!c.empty() && c.back() > (int)l.size()) c.pop_back();
  }
  return r;
}

// `slots` > 0 (coarse tables; the compute units of a die): a persistent launch gives the block in slot c of a die the
// entries c, c + slots, c + 2 slots, ... of that die's sequence.  Tiles differ in cost (a diagonal tile issues 9/16
// of the MFMAs of a full one), so within every run of `slots` entries - the tiles the die runs at the same time,
// whose set stays as it is - the tiles are handed to the slots most expensive first, each to the slot that has
// accumulated least so far.
// `join_equal` (fine tables): problems with K loops of one length are cut into the 8 runs together, not one by one, so that
// a die works on an eighth of the problems instead of an eighth of each: with few tiles per problem every die fetched
// nearly every operand (layer of 4 x 1024^2 and 3 x 1024 x 4096: fine launches -4 to -8 %, with two planes -4 to -17 %).
size_t deal_tiles(const std::vector<int>& order, const std::vector<std::vector<GemmTile>>& per_problem,
                  const std::vector<std::vector<int>>& per_problem_cuts, const std::vector<int64_t>& weight, GemmTile* out,
                  int slots = 0, bool join_equal = false) {
  std::vector<std::vector<GemmTile>> seq(kXcds);
  std::vector<int64_t> load(kXcds, 0);
  int rr = 0;
  size_t nonempty = 0;
  for (const auto& t : per_problem) nonempty += t.empty() ? 0 : 1;
  const bool whole = nonempty >= 4 * (size_t)kXcds;
  for (size_t oi = 0; oi < order.size(); ++oi) {
    const int pi = order[oi];
    if (per_problem[pi].empty()) continue;
    if (whole) {
      // least-loaded XCD (tiles weighted by the length of their K loop), ties broken round-robin
      const std::vector<GemmTile>& tiles = per_problem[pi];
      int best = rr;
      for (int x = 0; x < kXcds; ++x)
        if (load[(rr + x) % kXcds] < load[best]) best = (rr + x) % kXcds;
      seq[best].insert(seq[best].end(), tiles.begin(), tiles.end());
      load[best] += weight[pi] * (int64_t)tiles.size();
      rr = (rr + 1) % kXcds;
    } else {
      // 8 contiguous runs of equal length (so that entry b of the dealt table still lands on die b % 8).  A run
      // starts and ends inside blocks; its whole blocks go first, so that the tiles a die runs together come from
      // one block, and the two partial blocks at its ends follow.
      std::vector<GemmTile> tiles = per_problem[pi];
      std::vector<int> cuts = per_problem_cuts[pi];
      while (join_equal && oi + 1 < order.size() && weight[order[oi + 1]] == weight[pi]) {
        const int pj = order[++oi];
        for (int c : per_problem_cuts[pj]) cuts.push_back(c + (int)tiles.size());
        tiles.insert(tiles.end(), per_problem[pj].begin(), per_problem[pj].end());
      }
      const size_t n = tiles.size();
      for (int x = 0; x < kXcds; ++x) {
        const size_t lo = n * x / kXcds, hi = n * (x + 1) / kXcds;
        size_t c0 = lo, c1 = lo;                   // first and last block boundary inside [lo, hi] (none: c0 = c1 = lo)
        bool found = false;
        for (int c : cuts)
          if ((size_t)c >= lo && (size_t)c <= hi) {
            if (!found) c0 = (size_t)c;
            c1 = (size_t)c;
            found = true;
          }
        seq[x].insert(seq[x].end(), tiles.begin() + c0, tiles.begin() + c1);
        seq[x].insert(seq[x].end(), tiles.begin() + lo, tiles.begin() + c0);
        seq[x].insert(seq[x].end(), tiles.begin() + c1, tiles.begin() + hi);
      }
    }
  }
  if (slots > 0) {
    // cost in units of K: the MFMA work of the main loop plus a fixed part for the first slabs and the epilogue; a
    // 512 x 128 tile counts a quarter more than a 256 x 256 one (640 operand rows per K slab instead of 512; measured:
    // factors 1.15 to 1.3 do equally well, the fixed part hardly matters)
    auto cost = [&](const GemmTile& t) {
      int64_t blocks = t.shape == kShape256Diag ? 36 : (int64_t)kShapeRows[t.shape] * kShapeCols[t.shape] / 1024;
      if (t.shape == kShape512x128) blocks += blocks / 4;
      return (int64_t)512 + weight[t.prob] * blocks / 64;
    };
    for (auto& q : seq) {
      std::vector<int64_t> acc((size_t)slots, 0);
      for (size_t r0 = 0; r0 < q.size(); r0 += (size_t)slots) {
        const size_t cnt = std::min((size_t)slots, q.size() - r0);
        std::vector<GemmTile> round(q.begin() + (std::ptrdiff_t)r0, q.begin() + (std::ptrdiff_t)(r0 + cnt));
        std::stable_sort(round.begin(), round.end(), [&](const GemmTile& a, const GemmTile& b) { return cost(a) > cost(b); });
        std::vector<size_t> slot(cnt);
        std::iota(slot.begin(), slot.end(), (size_t)0);
        std::stable_sort(slot.begin(), slot.end(), [&](size_t a, size_t b) { return acc[a] < acc[b]; });
        for (size_t i = 0; i < cnt; ++i) {
          q[r0 + slot[i]] = round[i];
          acc[slot[i]] += cost(round[i]);
        }
      }
    }
  }
  size_t o = 0;
  for (size_t s = 0;; ++s) {
    bool any = false;
    for (int x = 0; x < kXcds; ++x)
      if (s < seq[x].size()) {
        out[o++] = seq[x][s];
        any = true;
      }
    if (!any) break;
  }
  return o;
}

// Tiles per work item of the elementwise passes: one after the other in a block, each pays the latency of a chain of
// loads, so a list is given at least 2048 blocks (eight per compute unit, all resident) before they take more.  Measured, us
// with runs of 4 / by this rule: momentum pass of four of 512^2 10.8 / 7.2, of 1000 x 3001 37 / 14 (with the wide accesses at
// odd widths); long lists are within 3 % of runs of one, whose table would be four times as long.
int ew_run(size_t tiles) { return (int)std::min<size_t>((size_t)kEwRun, std::max<size_t>(1, tiles / 2048)); }

// The coarse tiles (256 x 256, strips among them) a product's outputs hold, and what their matrices are like on average,
// each tile counted once: sides and area.
struct CoarseLoad {
  size_t tiles = 0;
  double m = 0.0, n = 0.0, area = 0.0, mm = 0.0, nn = 0.0;     // mm, nn: averages of the squares
  void add(size_t t, double rows, double cols) {
    if (t == 0) return;
    tiles += t;
    const double w = (double)t / (double)tiles;
    m += w * (rows - m);
    n += w * (cols - n);
    area += w * (rows * cols - area);
    mm += w * (rows * rows - mm);
    nn += w * (cols * cols - nn);
  }
  // standard deviation over a fifth of the average: about where the longest K is 1.5 times the shortest
  bool mixed_m() const { return mm - m * m > 0.04 * m * m; }
  bool mixed_n() const { return nn - n * n > 0.04 * n * n; }
  bool one_m() const { return mm - m * m < 0.0025 * m * m; }
  // share of the blocks that have a tile, over the rounds of `blocks` tiles
  double fill(int blocks) const {
    const size_t b = (size_t)std::max(blocks, 1);
    return (double)tiles / (double)((tiles + b - 1) / b * b);
  }
  // tiles for every 256 blocks (the numbers below were measured on 256 compute units)
  size_t per_256(int blocks) const { return tiles * 256 / (size_t)std::max(blocks, 1); }
};

// Whether a product goes to the fine launch altogether: its coarse tiles (one block per compute unit, `blocks` at a time)
// are too few, or cannot pay for their epilogue.  Averages over the tiles, not extremes of the list: one large or long
// matrix more does not move all the others.  Measured, us per launch, coarse / fine (128 x 128, or their quarters).
// Plain bf16, Gram and polynomial: 2048^2 (36 tiles) 45 / 24, 3584^2 (105) 69 / 56, 4096^2 (136) 83 / 102.  Up to one full
// round small matrices stay fine a little longer: 16 of 1024^2 (160) 35 / 33 and 39 / 34, 25 of 1024^2 (250) 46 / 43 and 49
// / 43, 12 of 2048 x 1408 (216) 68 / 67 and 56 / 51; but 8 of 2048 x 1536 (168) 53 / 56 and 48 / 46, 4 of 2048^2 (144) 50 /
// 56 and 53 / 58, 7 of 2048^2 (252) 67 / 73 and 70 / 75.
// Several planes: both launches run 128 x 128 tiles (gemm_planes.h).  A coarse entry's four run on one die in the order of
// coarse blocks; with two planes the symmetric ones have three accumulators, a compute unit each and the shorter polynomial.  A
// fine launch mixes in whatever else is fine, runs in quarters where it is short, and folds the norm there.  Measured, Gram and
// polynomial together, us per launch pair, coarse / fine.  Two planes: 48 of 1024^2 434 / 412, 24 of 1024 x 4096 491 / 444, 40 of
// 1408 x 2048 976 / 940, 24 of 1536^2 663 / 613, 12 of 1536 x 6144 689 / 684, 12 of 1536 x 8192 826 / 847, 4 of 2048 x 8192
// 563 / 675, 16 1939 / 2083, 11 of 2304 x 3840 1129 / 1153, 4 of 2560 x 5120 635 / 655, 4 of 2816 x 11008 (264 tiles) 1335 / 1251, 2 of
// 3072^2 369 / 421, 3 of 3200^2 572 / 612, 7 of 4096^2 2636 / 3034; the line errs, by the old tile's leave, at 4 of 2048^2 258 /
// 277, 4 of 2048 x 4096 357 / 400, 7 of 2688 x 3200 912 / 993.  Three planes: 48 of 1024^2 711 / 663, 25 of 1024 x 8192 1390 / 1358,
// 16 of 1408 x 2048 702 / 677, 12 of 1536 x 6144 1177 / 1171, 7 of 2048^2 678 / 664, 7 of 2048 x 4096 961 / 964, 4 of 2560 x 5120
// 1100 / 1398, 4 of 2816^2 (264 tiles) 1025 / 909, 2 of 3072^2 654 / 703, 4096^2 822 / 831; it errs at 24 of 1024 x 4096 805 / 865.
// Lists that mix K (or m): two planes 7 of 2048 x 8192 and 4 of 1024^2 991 / 944, 48 of 1024^2 beside one 3072^2 955 / 943; three
// planes of one large m: 4 of 2560 x 10240 and of 2560^2 2393 / 2372.
bool few_coarse_sym(const CoarseLoad& c, int planes, int blocks) {
  if (c.per_256(blocks) < 112) return true;
  if (planes == 1) return c.per_256(blocks) < 256 && c.n <= 2048 && c.area <= 3.0 * (1 << 20);
  if (c.m >= 3072) return false;
  const double fill = c.fill(blocks);
  if (c.mixed_m() || (c.mixed_n() && !(planes == 3 && c.m >= 2560 && c.one_m()))) return true;
  if (planes == 3 && fill >= 0.9 && c.m >= 2048) return false;
  return fill < 0.55 || fill * c.area < (planes == 2 ? 8.0 : 5.0) * (1 << 20);
}
// Apply product, plain bf16: 2048^2 (64 tiles) 44 / 26, two of 1024 x 4096 (128: a full round of fine tiles) 31 / 24, 8 of
// 1024^2 (128) 31 / 23, 4 of 512 x 4096 23 / 16; with a short K (m) a little beyond it: 5 of 256 x 8192 (160) 21 / 15, 5 of
// 512 x 4096 (160) 23 / 20, 3 of 640 x 5120 (150) 27 / 24, 4 of 768 x 3072 (144) 27 / 26, 10 of 1024^2 (160) 31 / 32, 4 of
// 1000 x 2500 (160) 31 / 31; but 3 of 1280 x 2560 (150) 36 / 38, 4 of 1536^2 (144) 39 / 43, 3072^2 (144) 63 / 78, four of
// 1024 x 4096 (256) 38 / 41.
// Several planes, as above, coarse / fine.  Two planes: 48 of 1024^2 302 / 307, 24 of 1024 x 4096 598 / 584, 40 of 1408 x 2048 899 /
// 887, 24 of 1536^2 481 / 483, 12 of 1536 x 8192 1241 / 1234, 7 of 2048 x 4096 626 / 638, 16 of 2048 x 8192 2847 / 2887, 8 of 2560^2
// 704 / 750, 4 of 2816 x 11008 1780 / 1823, 7 of 4096^2 2409 / 2496; where strips take many of the tiles it errs: 3 of 3200^2 577 /
// 527.  Three planes: 24 of 1024 x 4096 1139 / 1124, 24 of 1536^2 905 / 895, 7 of 2048^2 593 / 591, 4 of 2560^2 670 / 695, 4 of
// 2560 x 5120 1289 / 1320, 6 of 3072^2 1656 / 1666, 3 of 3200^2 1035 / 979.
bool few_coarse_apply(const CoarseLoad& c, int planes, int blocks) {
  if (c.per_256(blocks) <= 128 || (c.per_256(blocks) < 176 && c.m <= 1024)) return true;
  if (planes == 1 || c.m > 1536) return false;
  return c.m <= 1280 || c.area < (planes == 2 ? 10.0 : 8.0) * (1 << 20) || c.fill(blocks) < 0.95;
}

// Whether a fine launch runs each entry as four blocks, one per quarter.  bf16: 64 x 64 blocks of a 128 x 128 entry, which
// are quicker through one tile (0.35 against 0.6 us per 64 of K) but need more of the compute unit for the same work: while
// the launch holds less work than about 176 tiles of its longest K.  Measured, us per launch, 128 / 64: Gram product of
// 1024^2 (36 tiles) 16.2 / 10.4, four of 1024 x 4096 (144) 42 / 39, four of 2048 x 1408 (264) 31 / 34; apply product of
// 1024^2 (64) 14.6 / 9.9, of 32 of 256 x 384 (192) 8.4 / 8.0, of four of 1024^2 (256) 16.3 / 18.2.
// fp32 launches run their 64 x 64 entries as four blocks of 32 x 32 up to about 180 entries' work, and again where there is a
// little more than one entry for each of `blocks` compute units, so that whole entries would need a second round for a few.
// Measured, us per step, quarters / whole for the launches of that many entries: 144 (products of 4 of 512^2) 207 / 221, 180 (5)
// 242 / 261, 196 (apply product of 896^2) 245 / 236, 200 (2 of 640^2) 204 / 195, 216 (6 of 512^2) 278 / 260, 252 (7) 286 / 262,
// 256 (apply products of 1024^2, of 4 of 512^2) 327 / 314, 215 / 207, 288 (8 of 512^2) 315 / 351; earlier, us per launch, apply
// product of 64 of 128 x 256 (512) 17.7 / 13.6, Gram product of 16 of 512^2 (576) 34.4 / 34.1.
constexpr int kFewFine = 176, kFewF32 = 180, kLittleOverF32 = 64;
// Planes: 64-wide blocks pay while all of them have a place at the same time (three on a compute unit with two planes, two
// with three), and again where 128-wide ones would leave their last round badly filled, the sooner the shorter K.  us per
// launch, 128 / 64, entries (work) of the longest K.
// Two planes, up to 192 and from 257 to 320 with K up to 2048, with K = 256 and less all the way; mixed lists whose count (above
// K = 512) or work with a block's fixed cost stays near that, too: 90 of 256 15.6 / 10.8, 144 of 1024
// 33.8 / 29.9, 156 of 6144 136 / 123, 180 of 512 19.8 / 19.2, of 4096 126 / 100, 189 of 768 25.9 / 23.2; 213 of 128 12.0 / 11.1, 240 of 256 18.5 /
// 18.8, 251 of 128 12.4 / 11.4, 316 (210) of 256 16.5 / 15.8; 260 of 2048 72.5 / 68.1, 272 of 128 14.0 / 12.7, 288 of 1024 54.1 / 47.4, 300 of
// 512 34.7 / 29.2, of 1408 56.0 / 50.9, of 2048 82.3 / 81.9, 320 of 512 27.8 / 26.2; but 195 of 640 26.7 / 27.2, of 1408 38.9 / 42.2, 200 of 512
// 20.0 / 22.0, of 2048 52.6 / 56.7, 240 of 512 20.8 / 23.5, 323 (232) of 640 25.9 / 29.0; 288 of 4096 136 / 143, 312 of 6144 204 / 258; 324 of
// 768 36.4 / 38.3, 360 of 256 20.7 / 21.4, 384 of 1024 45.9 / 49.3, 481 (343) of 384 21.9 / 26.2.  Mixed, (work, with 512 of fixed
// cost): 348 (296, 325) of 384 22.1 / 20.7, 333 (276, 308) of 384 25.1 / 24.1; but 477 (310, 393) of 512 a step of 529 / 536, 335 (300) of
// 768 34.2 / 36.6, 408 (274) of 640 a step of 346 / 367.
// Three planes: 72 of 256 20.9 / 12.4, 108 of 4096 121 / 88, 120 of 512 26.3 / 20.3, 126 of 3072 97 / 72; 144 of 1024 41.8 / 39.9, 168 of 768
// 36.2 / 32.7, 195 of 384 26.4 / 25.8, 204 of 128 17.1 / 14.7, 251 of 128 17.1 / 15.5, 512 of 128 30.1 / 25.2, 626 (583) of 256 58.2 / 45.1, 875 (837)
// of 256 72.7 / 56.8; but 140 of 4096 131 / 137, 156 of 1536 55.8 / 61.5, 180 of 1024 44.1 / 45.9, 200 of 512 30.7 / 30.3, 255 of 384 26.5 / 27.2.
// Beyond one round, by its fill: 272 of 512 50.5 / 38.3, 600 of 512 (0.78) 78 / 76, 420 of 768 (0.82) 74 / 67; 360 of 1024 (0.70) 84 / 77, 576
// of 1024 (0.75) 127 / 115; 272 of 2048 (0.53) 135 / 113, 312 of 1536 (0.61) 108 / 96; 288 of 4096 (0.56) 256 / 238, 272 of 8192 490 / 474; but 432
// of 1024 (0.84) 85 / 90, 840 of 768 (0.82) 136 / 145, 360 of 2048 (0.70) 139 / 145, 420 of 2560 (0.82) 177 / 211, 390 of 6144 (0.76) 407 / 537,
// 324 of 8192 (0.63) 506 / 578, 300 of 4096 (0.59) 264 / 275; 1080 of 1024 (0.84) 204 / 230, of 384 (0.84) 114 / 121, 1300 of 512 (0.85) 147 / 166.
// Where K is mixed a round is also counted with what a block costs beside its K, about 512 of it: 323 entries, the work of 232 of 640,
// 272 so, 48.6 / 42.4; 333 (247, 281) of 768 52.8 / 45.7; but 260 (223, 237) of 768 38.0 / 42.3.
constexpr int64_t kLongKPlanes2 = 2048, kShortKPlanes2 = 256, kMixedKPlanes2 = 512, kMostFine3 = 1024, kBlockK = 512;
struct Fine3 {
  int64_t k;        // longest K
  int entries;      // of a launch in quarters within one round of 256 compute units
  int fill;         // per cent of the last round
};
constexpr Fine3 kFine3[] = {{256, (int)kMostFine3, 100}, {768, 200, 85}, {1024, 150, 80}, {2048, 128, 65}, {INT64_MAX, 128, 57}};
// entries whose 64-wide blocks all have a place at the same time
int lone_entries(int planes, int blocks) { return planes == 2 ? 3 * blocks / 4 : blocks / 2; }
// What a fine launch holds: entries of one K after the other.
struct Load {
  int64_t entries, k;
};
std::vector<Load> load_of(const std::vector<std::vector<GemmTile>>& tiles, const std::vector<int64_t>& k) {
  std::vector<Load> out;
  for (size_t i = 0; i < tiles.size(); ++i) {
    if (tiles[i].empty()) continue;
    if (!out.empty() && out.back().k == k[i]) out.back().entries += (int64_t)tiles[i].size();
    else out.push_back({(int64_t)tiles[i].size(), k[i]});
  }
  return out;
}
// a launch's work in entries of its longest K; `fixed`: what an entry costs beside its K
int64_t entries_of_work(const std::vector<Load>& load, int64_t fixed = 0) {
  int64_t longest = 1, total = 0;
  for (const Load& l : load) {
    longest = std::max(longest, l.k + fixed);
    total += (l.k + fixed) * l.entries;
  }
  return (total + longest - 1) / longest;
}
// Plain bf16: 128-wide blocks with a ring of four slabs (gemm_ring128.h) where every entry has a compute unit to itself, from where
// 64-wide ones stop paying.  us per launch, 64-wide / 128-wide with two stages / with the ring, polynomial products (K, entries):
//   256  180 9.5 / 9.7 / 10.0, 240 9.2 / 9.0 / 8.9;  384  180 11.2 / 11.7 / 11.6, 243 11.2 / 10.7 / 10.3
//   512  150 11.9 / 12.4 / 11.8, 180 12.1 / 12.6 / 12.0, 240 13.8 / 12.7 / 12.3;  768  126 11.5 / 15.2 / 13.3, 147 13.8 / 15.0 / 13.1, 252 16.9 / 15.4 / 14.3
//   1024  108 12.0 / 16.0 / 13.7, 144 15.0 / 16.3 / 14.0, 252 19.3 / 17.4 / 15.2
//   1408  66 12.6 / 19.3 / 15.2, 132 17.4 / 20.0 / 16.1, 198 22.0 / 20.9 / 16.8;  2048  136 22.7 / 25.3 / 18.9;  2816  253 40.1 / 33.9 / 27.6
// apply products:
//   512  144 9.6 / 10.5 / 9.8, 176 9.9 / 10.8 / 10.1, 208 11.6 / 10.8 / 10.3;  768  144 11.6 / 13.1 / 11.8, 180 12.2 / 13.7 / 11.9
//   1024  192 14.0 / 15.4 / 13.0;  1408  242 21.2 / 20.1 / 15.9
// with more entries than compute units: 512  260 15.6 / 14.2 / 18.2;  1408  264 24.9 / 22.8 / 27.8
constexpr int64_t kRingK = 256, kRingFewK = 768;   // shortest K of a launch; longest K from which fewer entries do
bool runs_on_ring128(const std::vector<Load>& load, int blocks) {
  int64_t count = 0, longest = 0;
  for (const Load& l : load) {
    if (l.k < kRingK) return false;
    count += l.entries;
    longest = std::max(longest, l.k);
  }
  const int64_t work = entries_of_work(load), b = std::max(blocks, 1);
  if (count > b) return false;
  return longest >= kRingFewK ? work > b / 2 + 8 : longest > kRingK && work > kFewFine;
}
bool runs_in_quarters(const std::vector<Load>& load, bool mc, int planes, int blocks) {
  const int64_t entries = entries_of_work(load);
  int64_t longest = 0, count = 0;
  for (const Load& l : load) {
    longest = std::max(longest, l.k);
    count += l.entries;
  }
  const int64_t b = std::max(blocks, 1);
  if (mc && planes == 2) {
    if (entries <= lone_entries(2, blocks)) return true;
    if (4 * entries > 5 * b || longest > (entries > b ? kLongKPlanes2 : kShortKPlanes2)) return false;
    return longest <= kMixedKPlanes2 ? 3 * entries_of_work(load, kBlockK) <= 4 * b : 4 * count <= 5 * b;
  }
  if (mc && planes == 3) {
    const Fine3* f = kFine3;
    while (longest > f->k) ++f;
    if (entries <= f->entries * b / 256) return true;
    for (int64_t e : {entries, entries_of_work(load, kBlockK)}) {
      const int64_t rounds = (e + b - 1) / b;
      if (rounds > 1 && e <= kMostFine3 && 100 * e < f->fill * rounds * b) return true;
    }
    return false;
  }
  if (mc) return entries <= kFewFine && !runs_on_ring128(load, blocks);
  return entries <= kFewF32 || (entries > blocks && entries <= blocks + kLittleOverF32);
}

// fp32: entries beyond full rounds of whole ones (three to a compute unit) that run in quarters in a launch of their own, where they
// are few and the round they would add is long.  us per apply product, with that round / with the second launch: 832 entries of K = 512
// 43.3 / 40.8, 800 of 640 55.0 / 51.0, 832 of 1024 77.4 / 69.2; but 896 of 512 43.8 / 44.3, 900 of 640 53.3 / 57.3, 832 of 256 27.4 / 27.8.
// us per step of other lists: 784 of 512 410 / 398, 800 of 512 394 / 394; beyond the line nothing is sure: 864 of 512 431 / 427, 837 of 576 475 / 476, 840
// of 640 497 / 494, but 834 of 384 317 / 322, 868 of 448 394 / 398.
constexpr int64_t kTailK = 512;
int tail_in_quarters(const std::vector<Load>& load, bool whole, bool long_k, int blocks) {
  int64_t count = 0;
  for (const Load& l : load) {
    if (l.k < kTailK) return 0;
    count += l.entries;
  }
  const int64_t places = (long_k ? 2 : 3) * (int64_t)std::max(blocks, 1), tail = count % places;
  return whole && count > places && 4 * tail <= blocks ? (int)tail : 0;
}

// 3: 128-wide blocks with a ring of four slabs (runs_on_ring128).  Launches in quarters that leave most compute units with one block or none: 2 = each 32 x 32 as one wave of its
// own (shortest chain of slabs; twice the operand traffic), 1 = 64 x 64 blocks with a ring of four slabs (two blocks on a
// compute unit instead of three), 0 = with a ring of three.
// Plain bf16, waves for the fewest entries, with K up to 1024 a few more, us per step, 0 / 1 / 2: 256^2 (3 and 4 entries) 58.5 / 57.4 /
// 51.8, 512^2 (10, 16) 78.0 / 73.4 / 68.3, 2 of 512^2 (20, 32) 81.4 / 78.7 / 77.1, 63 x 4097 (1, 33) 135.7 / 115.4 / 112.9; per launch 27
// entries of K = 384 6.6 / 6.6 / 6.4, 25 of 768 (the work of 22) a step of 143.9 / 142.1 for 1 / 2, 36 of 1024 9.9 / 9.4 / 9.7 (even in the
// step: 112.5 / 112.9), of 4096 21.7 / 18.4 / 21.9, 40 of 512 7.0 / 7.1 / 7.9.
// The longer ring goes by the work: entries that have a compute unit to themselves, or a few long ones among short ones.  us per launch,
// 0 / 1: 60 entries of 512 8.3 / 8.0, 63 of 768 9.9 / 9.6; 72 of 1024 11.0 / 11.3, 80 of 512 8.0 / 8.5, 100 8.8 / 9.1, 140 11.3 / 11.9; lists
// that mix K, work in brackets: 130 (67) 24.4 / 23.3, 133 (66) 25.9 / 22.7, 128 (61) 24.7 / 22.4, 112 (50) 23.0 / 20.6, 100 (62) 95.7 /
// 72.8, 96 (42) 26.2 / 21.4, 80 (26) 22.1 / 18.5, 45 (14) 36.2 / 26.6.
// Planes, 0 / 1, two and three: 40 of 512 9.8 / 9.8 and 12.3 / 11.8, 36 of 4096 36.6 / 30.1 and 50.8 / 45.7, 63 of 768 12.8 / 12.2 and 17.1 /
// 16.8; 70 of 512 12.8 / 12.6 and 17.6 / 18.1, 72 of 1024 17.4 / 17.8 and 25.5 / 26.4, 100 of 512 13.5 / 13.7 and 18.7 / 19.1; mixed 80 (22)
// 36.6 / 30.9 and 51.6 / 46.3, 66 (40) 37.0 / 33.0 and 52.3 / 48.8, 70 (44) 18.0 / 17.3 and 24.9 / 25.7, 66 (46) 29.0 / 26.8 and 40.4 / 41.9
// (two planes up to 51, three up to 40).
constexpr size_t kFewest = 24, kFewestShort = 36;
constexpr int64_t kShortK = 1024;
int few_blocks(const std::vector<Load>& load, int planes, int blocks) {
  size_t n = 0;
  int64_t longest = 0;
  for (const Load& l : load) {
    n += (size_t)l.entries;
    longest = std::max(longest, l.k);
  }
  if (planes == 1 && runs_on_ring128(load, blocks)) return 3;
  if (planes == 1 && (n <= kFewest || (n <= kFewestShort && longest <= kShortK))) return 2;
  const int64_t work = entries_of_work(load), b = std::max(blocks, 1);
  if (planes > 1) return 4 * (int64_t)n <= b || (planes == 2 ? 5 * work <= b : 32 * work <= 5 * b) ? 1 : 0;
  return 4 * work <= b + b / 16 ? 1 : 0;
}

// What a group brings to the fine level of paired launches, by PairProduct, and the shortest and longest K of each product.
struct PairSide {
  std::vector<Load> load[4];
  std::vector<std::vector<GemmTile>> coarse_sym;       // and the coarse tiles of its symmetric products
  std::vector<std::vector<int>> coarse_cuts;
  std::vector<std::vector<GemmTile>> coarse_app;       // of its apply product, where that is not all fine tiles
  std::vector<std::vector<int>> app_cuts;
  std::vector<int64_t> w_n, w_m;
  std::vector<Load> lone;                               // its lone table
  int64_t lo[4] = {kMaxDim, kMaxDim, kMaxDim, kMaxDim}, hi[4] = {};
};
PairForm fine_form(std::vector<Load> load, const std::vector<Load>& more, int blocks) {
  load.insert(load.end(), more.begin(), more.end());
  PairForm f;
  f.quarters = runs_in_quarters(load, true, 1, blocks);
  f.few = few_blocks(load, 1, blocks);
  return f;
}
PairForm pair_form(const PairSide& x, int px, const PairSide& y, int py, int blocks) {
  PairForm f = fine_form(x.load[px], y.load[py], blocks);
  f.persistent = 2 * std::max(x.hi[px], y.hi[py]) <= 3 * std::min(x.lo[px], y.lo[py]);
  return f;
}

// In a table of both groups: problems from n0 on are the second's.
void mark_second(GemmTile* tiles, int count, int n0) {
  for (int t = 0; t < count; ++t)
    if (tiles[t].prob >= n0) {
      tiles[t].prob -= n0;
      tiles[t].flags |= kTileSecond;
    }
}

// Whether a product in 128-wide blocks shares a launch with an apply product in coarse tiles (`g`'s): where the compute units that the
// last round of those leaves idle can take it.  A coarse tile takes about 1.65 us per slab and 8, a block 0.3 and 5.  Step, in parts of the
// one without the Gram route, alone / beside: 3000^2 with one of 1024 x 4096 (144 tiles; 36 and 256 blocks) 1.085 / 1.030, 4 of 1536^2 with
// one of 640 x 5000 (144; 15 and 200) 1.048 / 1.031, 4 of 1024^2 with 3 of 1024 x 4096 (192; 256) 0.999 / 0.994;
// but 48 of 1024^2 with 4 of 1024 x 4096 (768, full rounds; 144) 1.011 / 1.026, 8 of 2048^2 with 2 (512; 72) 1.010 / 1.032.
bool fits_beside(const Group& g, const std::vector<Load>& load, int blocks) {
  const int64_t b = std::max(blocks, 1), rest = g.coarse.n_apply % b;
  double need = 0.0;
  int64_t entries = 0;
  for (const Load& l : load) {
    entries += l.entries;
    need += (double)l.entries * (0.3 * (double)l.k / 64.0 + 5.0);
  }
  return rest > 0 && entries > 0 && entries <= b && need <= 1.25 * (double)(b - rest) * (1.65 * (double)g.longest_m / 64.0 + 8.0);
}

// Whether the apply products of both groups, where they come together, take one table of coarse tiles: where that saves a round.  An
// all-fine one counts as a round.  us per step of three iterations, where all of them meet, without the route / two launches or beside / one
// table: 4 of 1024^2 with 3 of 1024 x 4096 (64 tiles and 192) 306 / 325 / 311, 3000^2 with one (144, 64) 526 / 542 / 530, 4 of 1536^2 with one of 640 x 5000
// (144, 50) 339 / 359 / 345, 10 of 1536^2 with 6 of 1024 x 4096 (360, 384) 1063 / 1171 / 1085.
bool saves_a_round(size_t tiles0, bool fine0, size_t tiles1, bool fine1, int blocks) {
  const size_t b = (size_t)std::max(blocks, 1);
  auto rounds = [b](size_t t) { return (t + b - 1) / b; };
  return rounds(tiles0 + tiles1) < (fine0 ? 1 : rounds(tiles0)) + (fine1 ? 1 : rounds(tiles1));
}

void plan_matrices(const muon_param* p, int n, int ns_dtype, std::vector<MatPlan>& out, size_t& total_partials) {
  out.resize(n);
  total_partials = 0;
  const size_t es = on_matrix_cores(ns_dtype) ? 2 : 4;
  for (int i = 0; i < n; ++i) {
    MatPlan& q = out[i];
    q.rows = p[i].rows;
    q.cols = p[i].cols;
    q.transposed = q.rows > q.cols;
    q.m = (int)std::min(q.rows, q.cols);
    q.n = (int)std::max(q.rows, q.cols);
    q.w_dtype = p[i].w_dtype;
    q.g_dtype = p[i].g_dtype;
    q.tile = on_matrix_cores(ns_dtype) ? kShapeRows[kShape128] : kF32Tile;
    q.mp = round_up_i(q.m, q.tile);
    q.np = round_up_i(q.n, q.tile);
    const int ap = q.transposed ? q.np : q.mp, bp = q.transposed ? q.mp : q.np;
    q.ew_tr = ap / kEwTile;
    q.ew_tc = bp / kEwTile;
    q.ns_bytes = (align_up(es * (size_t)q.mp * q.np, 256) * x_buffers(q, ns_dtype) + align_up(es * (size_t)q.mp * q.mp, 256) * 2) *
                 (size_t)planes_of(ns_dtype);
    q.part_off = total_partials;
    total_partials += (size_t)q.ew_tr * q.ew_tc;
    q.chunk = 0;
    q.coarse = false;
    q.gram = gram_route(q, ns_dtype);
  }
}

// Size of everything that is not Newton-Schulz temporaries.
struct TableLayout {
  size_t mats, ptrs, scal, partials, ew_tiles, gemm, total;
};

// No tile shape is smaller than the fine tile, so the fine-tile counts bound the table sizes.  (An upper bound: there is one
// apply table, not two, but callers' workspaces are sized by this.)
// (The tables of the Gram route have their place in the second apply table's and in the slack.)
constexpr size_t kTableAlign = 128;
size_t gemm_tables_bytes_for(const MatPlan& q) {
  const int tm = q.mp / q.tile, tn = q.np / q.tile;
  const size_t sym = (size_t)tm * (tm + 1) / 2 + 1, app = (size_t)tm * tn + 1;
  return 7 * sizeof(GemmProblem) + (2 * sym + 2 * app) * sizeof(GemmTile);
}

TableLayout table_layout(const std::vector<MatPlan>& mp, size_t total_partials) {
  TableLayout t{};
  const size_t n = mp.size();
  size_t gemm = 0;
  for (const MatPlan& q : mp) gemm += gemm_tables_bytes_for(q);
  // every table start is aligned to 256 B; chunks x groups x 13 tables bounds the slack
  t.mats = align_up(n * sizeof(MatDesc), 256);
  t.ptrs = align_up(n * sizeof(MatPtrs), 256);
  t.scal = align_up(n * 4 * sizeof(float), 256);
  t.partials = align_up(total_partials * sizeof(float), 256);
  t.ew_tiles = align_up(total_partials * sizeof(EwTile), 256) + 256 * n;  // per-chunk alignment slack
  t.gemm = align_up(gemm, 256) + (size_t)n * 16 * 256;
  t.total = t.mats + t.ptrs + t.scal + t.partials + t.ew_tiles + t.gemm;
  return t;
}

// Consecutive matrices per chunk, never more than `cap` bytes of temporaries in one (a single matrix always fits).
int count_chunks(const std::vector<MatPlan>& mats, size_t cap) {
  int chunks = 1;
  size_t used = 0;
  for (const MatPlan& q : mats) {
    if (used > 0 && used + q.ns_bytes > cap) {
      ++chunks;
      used = 0;
    }
    used += q.ns_bytes;
  }
  return chunks;
}

}  // namespace

bool on_matrix_cores(int ns_dtype) { return ns_dtype != MUON_F32; }
int planes_of(int ns_dtype) { return ns_dtype == MUON_BF16X2 ? 2 : ns_dtype == MUON_BF16X3 ? 3 : 1; }
// bf16 path, m >= 64: the a*X term of Eq. 2 is folded into the polynomial, B' = b A + c A A + a I, so that the apply
// product X' = B' X needs no addend (a third of its epilogue's memory traffic).  B's diagonal is rounded to bf16
// once either way; for tiny matrices, where the diagonal carries most of the product, the explicit addend is kept.
// The split forms keep the explicit addend: folded into B's diagonal it would be rounded at the diagonal's magnitude
// (a = 3.44), not the iterate's.
bool folds_identity(const MatPlan& q, int ns_dtype) { return ns_dtype == MUON_BF16 && q.m >= 64; }

// Whether a matrix takes the Gram route: from its own sides, so that its result does not depend on the list.  A group of two iterations
// then has one Gram and one apply product instead of two of each, and 5 products of m x m instead of 2: with five iterations three
// Gram and three apply products against six more of m x m.  Where a launch is a chain of slabs and little else that pays from a
// ratio n / m on that falls with m (the chain of the Gram product is n long, that of the six m); in lists that fill the chip sooner, so
// the line is where a matrix alone does not lose.  us per step, all products of Eq. 2 / Gram route, one matrix and several:
//   384 x 1536 84 / 87, 24 282 / 260; x 2304 96.5 / 94.7; x 3072 116 / 108, 24 496 / 421
//   512 x 2048 101.6 / 103.2, 8 198 / 186; x 3072 124 / 119; x 4096 141 / 129, 24 791 / 676
//   640 x 1664 106 / 112, 24 618 / 565; x 2560 123.8 / 124.4, 8 316 / 279; x 5120 173 / 155;  768 x 3072 147.5 / 147.2, 8 446 / 406
//   768 x 2304 133 / 136, x 2688 136 / 141;  1024 x 2816 158 / 169, 3 333 / 304; x 3072 166 / 173, 3 341 / 311; x 3584 182 / 186, 3 363 / 329; x 3840
//   189 / 190; x 4096 195.1 / 196.5, 3 383 / 341, 12 1307 / 1034;  1152 x 4096 222 / 214
//   1408 x 2816 240 / 253, 8 1142 / 1102; x 3840 304 / 292, 8 1478 / 1320;  2048 x 4096 530 / 523, 8 2588 / 2788; x 5632 663 / 619, 4 1819 / 1636
//   2560 x 5120 693 / 667;  3072 x 4608 960 / 985; x 6144 1219 / 1165;  4096 x 8192 2363 / 2164; x 11008 3057 / 2610;  2 of 4096 x 6144 3407 / 4072
// Fewer rows than 384 gain alone (256 x 4096 122 / 108) and lose beside anything longer.  Beside other matrices: 4 of 512^2 and 2 of 512 x
// 4096 173 / 164, 4 of 1024^2 and 3 of 1024 x 4096 472 / 453, 8 and 6 1065 / 978, 48 and 36 4622 / 4276, 4 of 4096^2 and 3 of 4096 x 11008 12992 / 11960;
// a few beside much more of the other kind pay for the longer chain of launches: 3000^2 and one of 1024 x 4096 827 / 866 (on a slower card
// 850 / 905), 4 of 1536^2 and one of 640 x 5000 528 / 544, 8 of 2048^2 and 2 of 1024 x 4096 1931 / 1957, 48 of 1024^2 and 4 1934 / 1965.  (Three iterations, which no
// matrix takes on its Gram matrix, but in two groups all the same: 4 of 1024^2 and 3 of 1024 x 4096 306 / 311, 3000^2 and one 526 / 530, alone even.)
bool gram_route(const MatPlan& q, int ns_dtype) {
  if (ns_dtype != MUON_BF16 || q.mp < 384) return false;
  const double least = q.mp >= 2560 ? 2.0 : q.mp >= 1280 ? 2.6 : q.mp >= 640 ? 4.0 : 8.0;
  return q.np >= least * q.mp;
}

bool gram_coefficients_fit(const double* coeff, int steps, double* gain) {
  // An element is at most its matrix's spectral norm.  s: bound on X's, which is 1 at the start (the Frobenius norm); the maximum of
  // |a x + b x^3 + c x^5| over [0, s] is at an end or where the derivative vanishes.  A quarter is added for rounding.
  const double slack = 1.25, most = 65504.0 / slack;
  double s = 1.0, shrunk = 1.0;
  *gain = slack;
  for (int k = 0; k < steps;) {
    const int group = gram_group(k, steps);
    const bool first = k == 0;                   // of the first, which is in bf16, X alone
    double q = 1.0;
    for (int j = 0; j < group; ++j, ++k) {
      const double a = coeff[3 * k], b = coeff[3 * k + 1], c = coeff[3 * k + 2], t = s * s;
      auto f = [&](double x) { return std::fabs(x * (a + x * x * (b + c * x * x))); };
      double next = f(s), p = std::max(std::fabs(a), std::fabs(a + t * (b + c * t)));
      if (c != 0.0) {
        const double v = -b / (2.0 * c), disc = 9.0 * b * b - 20.0 * a * c;
        if (v > 0.0 && v < t) p = std::max(p, std::fabs(a + v * (b + c * v)));
        if (disc >= 0.0)
          for (double root : {(-3.0 * b + std::sqrt(disc)) / (10.0 * c), (-3.0 * b - std::sqrt(disc)) / (10.0 * c)})
            if (root > 0.0 && root < t) next = std::max(next, f(std::sqrt(root)));
      } else if (b != 0.0) {
        const double root = -a / (3.0 * b);
        if (root > 0.0 && root < t) next = std::max(next, f(std::sqrt(root)));
      }
      q *= std::max(p, 1.0);
      // A and T = P A; D = P - a I and Q; the next X
      const double worst = std::max(first ? 0.0 : std::max(kGramScaleA * t * std::max(1.0, p), kGramScaleP * std::max(p + std::fabs(a), q)),
                                    kGramScaleX * next);
      if (!(worst <= most)) return false;        // not a number, too
      s = next;
      *gain *= std::max(p, 1.0);
      // What f16 holds as well as bf16 would: small singular values, which follow a, must not shrink much, and an X that eps leaves small must
      // not grow so far (store_norm keeps one scale for all iterations).  The paper's coefficients: up to ten iterations.
      shrunk *= std::min(std::fabs(a), 1.0);
      if (!(shrunk >= 1.0 / 64.0 && *gain <= (double)(1 << 19))) return false;
    }
  }
  return true;
}

int validate_shapes(const muon_param* p, int32_t n, int32_t ns_dtype) {
  if (!p || n <= 0) return MUON_E_INVALID_ARG;
  if (ns_dtype != MUON_F32 && ns_dtype != MUON_BF16 && ns_dtype != MUON_BF16X2 && ns_dtype != MUON_BF16X3)
    return MUON_E_UNSUPPORTED_DTYPE;
  for (int i = 0; i < n; ++i) {
    if (p[i].rows < 1 || p[i].cols < 1 || p[i].rows > kMaxDim || p[i].cols > kMaxDim) return MUON_E_INVALID_ARG;
    if ((p[i].w_dtype != MUON_F32 && p[i].w_dtype != MUON_BF16) || (p[i].g_dtype != MUON_F32 && p[i].g_dtype != MUON_BF16))
      return MUON_E_UNSUPPORTED_DTYPE;
  }
  return MUON_OK;
}

int plan_workspace_bytes(const muon_param* shapes, int32_t n, int32_t ns_dtype, size_t max_bytes, size_t* out) {
  if (!out) return MUON_E_INVALID_ARG;
  int st = validate_shapes(shapes, n, ns_dtype);
  if (st != MUON_OK) return st;
  std::vector<MatPlan> mp;
  size_t total_partials = 0;
  plan_matrices(shapes, n, ns_dtype, mp, total_partials);
  const TableLayout tl = table_layout(mp, total_partials);
  size_t all = 0, biggest = 0;
  for (const MatPlan& q : mp) {
    all += q.ns_bytes;
    biggest = std::max(biggest, q.ns_bytes);
  }
  size_t want = tl.total + all;
  const size_t least = tl.total + biggest;
  if (max_bytes != 0 && want > max_bytes) want = std::max(max_bytes, least);
  *out = align_up(want, 256);
  return MUON_OK;
}

int plan_build(Plan& plan, const muon_param* shapes, int32_t n, int32_t ns_dtype, uintptr_t ws_base, size_t workspace_bytes) {
  int st = validate_shapes(shapes, n, ns_dtype);
  if (st != MUON_OK) return st;
  const int coarse_blocks = plan.coarse_blocks;
  plan = Plan{};
  plan.coarse_blocks = coarse_blocks;
  plan.n = n;
  plan.ns_dtype = ns_dtype;
  size_t total_partials = 0;
  plan_matrices(shapes, n, ns_dtype, plan.mats, total_partials);
  const TableLayout tl = table_layout(plan.mats, total_partials);

  size_t biggest = 0;
  for (const MatPlan& q : plan.mats) biggest = std::max(biggest, q.ns_bytes);
  if (workspace_bytes < tl.total + biggest) return MUON_E_WORKSPACE_TOO_SMALL;
  const size_t ns_budget = workspace_bytes - tl.total;

  // ---- chunking: consecutive matrices while their temporaries fit.  The number of chunks is what the budget
  // forces; the cut positions then come from the smallest cap that still gives that number, so that the chunks carry
  // about equal work instead of leaving a short last one (every chunk's launches end in a tail). ----
  {
    const int want = count_chunks(plan.mats, ns_budget);
    size_t lo = biggest, hi = ns_budget;     // count_chunks(hi) == want; find the smallest cap with that property
    while (lo < hi) {
      const size_t mid = lo + (hi - lo) / 2;
      if (count_chunks(plan.mats, mid) <= want) hi = mid;
      else lo = mid + 1;
    }
    const size_t cap = hi;
    size_t used = 0;
    Chunk cur{};
    for (int i = 0; i < n; ++i) {
      if (cur.count > 0 && used + plan.mats[i].ns_bytes > cap) {
        plan.chunks.push_back(cur);
        cur = Chunk{};
        cur.first = i;
        used = 0;
      }
      plan.mats[i].chunk = (int)plan.chunks.size();
      used += plan.mats[i].ns_bytes;
      cur.count++;
    }
    plan.chunks.push_back(cur);
  }

  // ---- host image of the table region ----
  std::vector<unsigned char> img(tl.total, 0);
  size_t off = 0;
  const size_t off_mats = off; off += tl.mats;
  const size_t off_ptrs = off; off += tl.ptrs;
  const size_t off_scal = off; off += tl.scal;
  const size_t off_part = off; off += tl.partials;
  size_t cursor = off;   // ew tiles and gemm tables are appended from here
  unsigned char* const ws = reinterpret_cast<unsigned char*>(ws_base);   // address arithmetic only, never dereferenced
  unsigned char* ns_base = ws + tl.total;
  const bool mc = on_matrix_cores(ns_dtype);
  const size_t es = mc ? 2 : 4;
  const size_t planes = (size_t)planes_of(ns_dtype);

  MatDesc* h_mats = reinterpret_cast<MatDesc*>(img.data() + off_mats);
  auto dev = [&](size_t o) { return ws + o; };

  for (Chunk& ch : plan.chunks) {
    size_t ns_off = 0;
    for (int i = ch.first; i < ch.first + ch.count; ++i) {
      const MatPlan& q = plan.mats[i];
      MatDesc& d = h_mats[i];
      const size_t xb = align_up(es * (size_t)q.mp * q.np, 256), ab = align_up(es * (size_t)q.mp * q.mp, 256);
      d.X = ns_base + ns_off; ns_off += xb * planes;
      d.Xt[0] = ns_base + ns_off; ns_off += xb * planes;
      d.Xt[1] = nullptr;
      if (x_buffers(q, ns_dtype) == 3) { d.Xt[1] = ns_base + ns_off; ns_off += xb * planes; }
      d.Ag = ns_base + ns_off; ns_off += ab * planes;
      d.Bp = ns_base + ns_off; ns_off += ab * planes;
      d.x_plane = planes > 1 ? (int64_t)(xb / es) : 0;
      d.gram_route = q.gram;
      d.partials = reinterpret_cast<float*>(dev(off_part)) + q.part_off;
      d.scal = reinterpret_cast<float*>(dev(off_scal)) + 4 * (size_t)i;
      d.rows = (int)q.rows; d.cols = (int)q.cols;
      d.m = q.m; d.n = q.n; d.mp = q.mp; d.np = q.np;
      d.transposed = q.transposed;
      d.w_dtype = q.w_dtype; d.g_dtype = q.g_dtype;
      d.n_part = q.ew_tr * q.ew_tc;
      d.ew_tiles_c = q.ew_tc;
      d.sqrt_max = (float)std::sqrt((double)q.n);
    }

    size_t whole = 0, ragged = 0;
    for (int i = ch.first; i < ch.first + ch.count; ++i)
      if (plan.mats[i].w_dtype == MUON_BF16) (plan.mats[i].cols % 64 ? ragged : whole) += (size_t)(plan.mats[i].rows * plan.mats[i].cols);
    // (what the caches hold anyway does not mind: 4 of 1000 x 3001, 20 of 333 x 200 and 30 of 100 x 1002 0 to 1 % slower without)
    constexpr size_t kManyRagged = (size_t)64 << 20;
    ch.stream_w = whole >= ragged || ragged < kManyRagged;

    // elementwise tiles of the chunk
    cursor = align_up(cursor, 256);
    ch.ew_tiles_off = cursor;
    ch.n_ew_tiles = 0;
    {
      EwTile* t = reinterpret_cast<EwTile*>(img.data() + cursor);
      size_t all = 0;
      for (int i = ch.first; i < ch.first + ch.count; ++i) all += (size_t)plan.mats[i].ew_tr * plan.mats[i].ew_tc;
      const int run = ew_run(all);
      for (int i = ch.first; i < ch.first + ch.count; ++i) {
        const MatPlan& q = plan.mats[i];
        for (int r = 0; r < q.ew_tr; ++r)
          for (int c = 0; c < q.ew_tc; c += run) {
            t[ch.n_ew_tiles].mat = i;
            t[ch.n_ew_tiles].tr = (int16_t)r;
            t[ch.n_ew_tiles].tc = (int16_t)c;
            t[ch.n_ew_tiles].count = (int16_t)std::min(run, q.ew_tc - c);
            t[ch.n_ew_tiles].pad_ = 0;
            ch.n_ew_tiles++;
          }
      }
      cursor += (size_t)ch.n_ew_tiles * sizeof(EwTile);
    }

    // Whether the products go to the fine launch altogether is decided for the chunk, not for a group.
    // (Apply products: for a group where there are two, whose apply products never meet in a launch.)
    CoarseLoad coarse_sym, coarse_sym_of[2], coarse_app[2], coarse_app_all;
    std::vector<int> members_of[2];              // Eq. 2 as it is written, Gram route
    for (int i = ch.first; i < ch.first + ch.count; ++i) {
      const MatPlan& q = plan.mats[i];
      members_of[q.gram].push_back(i);
      if (!mc) continue;
      const size_t cm = (size_t)(q.mp / kCoarse), cn = (size_t)(q.np / kCoarse);
      const int strip_h = kShapeRows[kShape512x128];
      const bool odd_m = (q.mp % kCoarse) != 0;
      const size_t sym_tiles = cm * (cm + 1) / 2 + (odd_m && q.mp >= strip_h ? (size_t)((q.mp + strip_h - 1) / strip_h) : 0);
      coarse_sym.add(sym_tiles, q.mp, q.np);
      coarse_sym_of[q.gram].add(sym_tiles, q.mp, q.np);
      const size_t app_tiles = cm * cn + (odd_m && q.np >= strip_h ? (size_t)((q.np + strip_h - 1) / strip_h) : 0);
      coarse_app[q.gram].add(app_tiles, q.mp, q.np);
      coarse_app_all.add(app_tiles, q.mp, q.np);
    }
    const bool few_sym = few_coarse_sym(coarse_sym, (int)planes, plan.coarse_blocks);
    ch.paired = !members_of[1].empty();
    PairSide pair_sides[2];

    // GEMM groups of the chunk
    for (int route = 0; route < 2; ++route) {
      const std::vector<int>& members = members_of[route];
      if (members.empty()) {
        if (route == 0) ch.groups.push_back(Group{});        // groups[1] is the Gram route's
        continue;
      }
      const bool few_app = few_coarse_apply(coarse_app[route], (int)planes, plan.coarse_blocks);
      const CoarseLoad& coarse_own = coarse_sym_of[route];
      Group g{};
      g.gram = route == 1;
      g.n_prob = (int)members.size();
      g.members = members;
      const size_t np_ = members.size();
      auto take = [&](size_t bytes) {
        cursor = align_up(cursor, kTableAlign);
        const size_t o = cursor;
        cursor += bytes;
        return o;
      };
      for (int v = 0; v < 2; ++v) g.prob_gram[v] = take(sizeof(GemmProblem) * np_);
      g.prob_poly = take(sizeof(GemmProblem) * np_);
      for (int v = 0; v < 4; ++v) g.prob_apply[v] = take(sizeof(GemmProblem) * np_);
      if (g.gram) g.prob_ops = take(sizeof(GemmProblem) * np_ * kGramOps);
      for (size_t k = 0; k < np_; ++k) {
        const MatPlan& q = plan.mats[members[k]];
        const MatDesc& d = h_mats[members[k]];
        GemmProblem gp{};
        gp.scal = d.scal;
        const size_t xb = align_up(es * (size_t)q.mp * q.np, 256), ab = align_up(es * (size_t)q.mp * q.mp, 256);
        const int64_t xpl = planes > 1 ? (int64_t)(xb / es) : 0, apl = planes > 1 ? (int64_t)(ab / es) : 0;
        // bf16 path: ONE layout of the iterate, ping-ponging between X and Xt[0] (both m_pad x n_pad); fp32 path: X
        // updated in place plus its transpose ping-ponging between Xt[0] and Xt[1].
        void* const xbuf[2] = {d.X, mc ? d.Xt[0] : d.X};
        // Gram: A = X X^T
        for (int par = 0; par < 2; ++par) {
          gp.L = xbuf[par]; gp.R = xbuf[par]; gp.partials = d.partials; gp.Et = nullptr; gp.C = d.Ag; gp.Ct = nullptr;
          gp.K = q.np; gp.ldl = q.np; gp.ldr = q.np; gp.n_part = d.n_part; gp.ldet = 0; gp.ldc = q.mp; gp.ldct = q.mp; gp.symmetric = 1;
          gp.l_plane = xpl; gp.r_plane = xpl; gp.et_plane = 0; gp.c_plane = apl; gp.ct_plane = apl;
          reinterpret_cast<GemmProblem*>(img.data() + g.prob_gram[par])[k] = gp;
        }
        // polynomial: B = b A + c A A  (A is symmetric, so it is its own transposed addend)
        gp.partials = nullptr; gp.n_part = 0;
        gp.L = d.Ag; gp.R = d.Ag; gp.Et = d.Ag; gp.C = d.Bp; gp.Ct = nullptr;
        gp.K = q.mp; gp.ldl = q.mp; gp.ldr = q.mp; gp.ldet = q.mp; gp.ldc = q.mp; gp.ldct = q.mp; gp.symmetric = 1;
        gp.l_plane = apl; gp.r_plane = apl; gp.et_plane = apl; gp.c_plane = apl; gp.ct_plane = apl;
        gp.diag_add = folds_identity(q, ns_dtype) ? 1 : 0;
        reinterpret_cast<GemmProblem*>(img.data() + g.prob_poly)[k] = gp;
        gp.diag_add = 0;
        for (int par = 0; par < 2; ++par)
          for (int last = 0; last < 2; ++last) {
            gp.symmetric = 0;
            if (mc) {
              // apply, bf16: the product is posed transposed, T = X'^T = X^T B, with its L operand X^T read K-major
              // straight from the row-major X; the kernel's cheap transposed store of T is then X' itself, row-major.
              // Only the last iteration of a matrix iterated on its transpose needs T as it is (O in W's
              // orientation), through the kernel's other output, into Xt[1].
              gp.L = xbuf[par]; gp.R = d.Bp; gp.K = q.mp; gp.ldl = q.np; gp.ldr = q.mp;
              gp.Et = folds_identity(q, ns_dtype) ? nullptr : xbuf[par]; gp.ldet = q.np;
              gp.C = nullptr; gp.ldc = 0; gp.Ct = xbuf[par ^ 1]; gp.ldct = q.np;
              if (last && q.transposed) { gp.C = d.Xt[1]; gp.ldc = q.mp; gp.Ct = nullptr; gp.ldct = 0; }
              gp.l_plane = xpl; gp.r_plane = apl; gp.et_plane = xpl; gp.c_plane = xpl; gp.ct_plane = xpl;
            } else {
              // apply, fp32: X' = a X + B X, reading X^T from Xt[p], writing X in place and X'^T to Xt[p^1]; the last
              // iteration writes only the layout W needs.
              gp.L = d.Bp; gp.R = d.Xt[par]; gp.Et = d.Xt[par]; gp.C = d.X; gp.Ct = d.Xt[par ^ 1];
              gp.K = q.mp; gp.ldl = q.mp; gp.ldr = q.mp; gp.ldet = q.mp; gp.ldc = q.np; gp.ldct = q.mp;
              if (last) {
                if (q.transposed) gp.C = nullptr;
                else gp.Ct = nullptr;
              }
            }
            reinterpret_cast<GemmProblem*>(img.data() + g.prob_apply[par * 2 + last])[k] = gp;
            if (g.gram) {                        // the same with Q
              gp.R = d.Ag;
              reinterpret_cast<GemmProblem*>(img.data() + g.prob_ops)[(kGramApply + par * 2 + last) * np_ + k] = gp;
            }
          }
        if (g.gram) {
          for (int par = 0; par < 2; ++par) {
            void* const U = xbuf[par ^ 1];
            struct { void *l, *r, *e, *c; } const ops[kGramParityOps] = {
                {d.Bp, d.Ag, nullptr, U}, {U, d.Bp, nullptr, d.Ag}, {d.Ag, d.Ag, d.Ag, U}, {U, d.Bp, d.Bp, d.Ag}};
            for (int op = 0; op < kGramParityOps; ++op) {
              GemmProblem s = reinterpret_cast<const GemmProblem*>(img.data() + g.prob_poly)[k];
              s.L = ops[op].l; s.R = ops[op].r; s.Et = ops[op].e; s.C = ops[op].c;
              s.diag_add = 0;
              if (op != kGramD) s.symmetric = kMirrored;     // (D is a polynomial of one matrix, symmetric to the bit)
              reinterpret_cast<GemmProblem*>(img.data() + g.prob_ops)[(par * kGramParityOps + op) * np_ + k] = s;
            }
          }
        }
      }
      // Launch order of the problems, longest K loop first (the tail of a launch is then made of short tiles):
      // the Gram product runs over n, the other two over m.
      std::vector<int> by_n(np_), by_m(np_);
      std::iota(by_n.begin(), by_n.end(), 0);
      std::iota(by_m.begin(), by_m.end(), 0);
      std::stable_sort(by_n.begin(), by_n.end(), [&](int x, int y) {
        const MatPlan &a = plan.mats[members[x]], &b = plan.mats[members[y]];
        return a.np != b.np ? a.np > b.np : a.mp > b.mp;
      });
      std::stable_sort(by_m.begin(), by_m.end(), [&](int x, int y) {
        const MatPlan &a = plan.mats[members[x]], &b = plan.mats[members[y]];
        return a.mp != b.mp ? a.mp > b.mp : a.np > b.np;
      });
      std::vector<int64_t> w_n(np_), w_m(np_);
      for (size_t k = 0; k < np_; ++k) {
        w_n[k] = plan.mats[members[k]].np;
        w_m[k] = plan.mats[members[k]].mp;
      }
      // tile tables: level 1 = 256 x 256 tiles and 512 x 128 strip tiles (matrix cores only), level 0 = what they
      // leave uncovered, in fine tiles
      // uniform: every tile of the Gram product (n) / of the other two products (m) runs the same K.  steady: the
      // longest K is at most 1.5 times the shortest - such launches run persistent blocks with the planner's static,
      // cost-balanced assignment (measured: 27-layer MoE list, K = 1408 and 2048 mixed, polynomial launches -7 %);
      // with a wider spread the hardware's dynamic dispatch of one block per tile does better (K = 4096 and 11008
      // mixed: persistent +7 %).
      bool uniform_n = true, uniform_m = true;
      int64_t lo_n = w_n[0], hi_n = w_n[0], lo_m = w_m[0], hi_m = w_m[0];
      for (size_t k = 0; k < np_; ++k) {
        if (w_n[k] != w_n[0]) uniform_n = false;
        if (w_m[k] != w_m[0]) uniform_m = false;
        lo_n = std::min(lo_n, w_n[k]); hi_n = std::max(hi_n, w_n[k]);
        lo_m = std::min(lo_m, w_m[k]); hi_m = std::max(hi_m, w_m[k]);
      }
      g.longest_n = hi_n;
      g.longest_m = hi_m;
      const bool steady_n = 2 * hi_n <= 3 * lo_n, steady_m = 2 * hi_m <= 3 * lo_m;
      std::vector<std::vector<GemmTile>> moved_sym(np_), moved_app(np_);   // coarse tiles handed to the fine level
      for (int level = 1; level >= 0; --level) {
        if (level == 1 && !mc) continue;
        std::vector<std::vector<GemmTile>> sym(np_), app(np_);
        std::vector<std::vector<int>> sym_cuts(np_), app_cuts(np_);
        size_t n_sym = 0, n_app = 0;
        bool strips = false;
        for (size_t k = 0; k < np_; ++k) {
          const MatPlan& q = plan.mats[members[k]];
          const int cm_sym = mc && !few_sym ? q.mp / kCoarse : 0;            // coarse tiles along a side
          const int cm = mc && !few_app ? q.mp / kCoarse : 0, cn = mc && !few_app ? q.np / kCoarse : 0;
          const int tm = q.mp / q.tile, tn = q.np / q.tile, r = kCoarse / q.tile;
          const int strip_h = kShapeRows[kShape512x128];
          // the 128 columns an odd multiple of 128 leaves beside the 256-tiles go to 512 x 128 tiles where the
          // output is at least 512 rows high
          const bool odd_m = mc && (q.mp % kCoarse) != 0;
          const bool sym_strip = odd_m && !few_sym && q.mp >= strip_h, app_strip = odd_m && !few_app && q.np >= strip_h;
          if (level == 1) {
            // plain bf16: a diagonal tile is computed from its upper triangle of 32 x 32 blocks (9/16 of the MFMAs)
            blocked_tiles((int32_t)k, kCoarse, kShape256, cm_sym, cm_sym, true, 0, 0, -1, sym[k], sym_cuts[k], 4, 8,
                          ns_dtype == MUON_BF16 ? (int)kShape256Diag : -1);
            if (sym_strip) strip_tiles((int32_t)k, q.mp, q.mp - q.tile, sym[k], sym_cuts[k]);
            // tiles of X'^T in 8 x 2 blocks: measured against 8 x 4, 4 x 8, 16 x 2 and whole-width blocks, 0.7 % (4096-wide
            // block) to 1.5 % (MoE shapes) faster than 8 x 4, the next best (the K-major panels are the strided ones)
            blocked_tiles((int32_t)k, kCoarse, kShape256, cn, cm, false, 0, 0, -1, app[k], app_cuts[k], 8, 2);
            if (app_strip) strip_tiles((int32_t)k, q.np, q.mp - q.tile, app[k], app_cuts[k]);
            strips = strips || sym_strip || app_strip;
          } else {
            const int fine_shape = mc ? (int)kShape128 : 0;
            blocked_tiles((int32_t)k, q.tile, fine_shape, tm, tm, true, cm_sym * r, cm_sym * r, sym_strip ? tm - 1 : -1, sym[k], sym_cuts[k]);
            if (mc) blocked_tiles((int32_t)k, q.tile, fine_shape, tn, tm, false, cn * r, cm * r, app_strip ? tm - 1 : -1, app[k], app_cuts[k], 8, 4);
            else blocked_tiles((int32_t)k, q.tile, fine_shape, tm, tn, false, 0, 0, -1, app[k], app_cuts[k]);
            // the coarse tiles moved here: four fine tiles each (never a diagonal tile, so none of the four is one)
            for (int which = 0; which < 2; ++which) {
              const std::vector<GemmTile>& mv = which ? moved_app[k] : moved_sym[k];
              std::vector<GemmTile>& dst = which ? app[k] : sym[k];
              std::vector<int>& dcuts = which ? app_cuts[k] : sym_cuts[k];
              for (const GemmTile& t : mv) {
                for (int dr = 0; dr < r; ++dr)
                  for (int dc = 0; dc < r; ++dc)
                    dst.push_back(make_tile((int32_t)k, t.r0 * kTileUnit + dr * q.tile, t.c0 * kTileUnit + dc * q.tile, fine_shape, 0));
                dcuts.push_back((int)dst.size());
              }
            }
          }
        }
        if (level == 1) {
          // launches whose tiles all run the same K: even out their last round (paired symmetric launches have the other
          // group's tiles there)
          const int most = planes == 1 ? kMaxMovedTiles : lone_entries((int)planes, plan.coarse_blocks) / 4;
          if (uniform_n && uniform_m && !ch.paired) move_tail_to_fine(by_n, sym, sym_cuts, plan.coarse_blocks, most, moved_sym);
          if (uniform_m) move_tail_to_fine(by_m, app, app_cuts, plan.coarse_blocks, most, moved_app);
        }
        for (size_t k = 0; k < np_; ++k) {
          n_sym += sym[k].size();
          n_app += app[k].size();
          if (level == 1) plan.mats[members[k]].coarse = !sym[k].empty() || !app[k].empty();
        }
        TileSet& ts = level ? g.coarse : g.fine;
        ts.strips = strips;
        if (ch.paired) {
          PairSide& side = pair_sides[route];
          side.lo[kPairGram] = lo_n; side.hi[kPairGram] = hi_n;
          side.lo[kPairSym] = side.lo[kPairApply] = lo_m; side.hi[kPairSym] = side.hi[kPairApply] = hi_m;
          if (level == 1) {
            side.coarse_sym = sym, side.coarse_cuts = sym_cuts, side.w_n = w_n, side.w_m = w_m;
            side.coarse_app = app, side.app_cuts = app_cuts;
          }
          if (level == 0) {
            side.load[kPairGram] = load_of(sym, w_n);
            side.load[kPairSym] = load_of(sym, w_m);
            side.load[kPairApply] = load_of(app, w_m);
          }
        }
        if (level == 0) {
          const std::vector<Load> l_sym = load_of(sym, w_n), l_poly = load_of(sym, w_m), l_app = load_of(app, w_m);
          ts.quarter_sym = runs_in_quarters(l_sym, mc, (int)planes, plan.coarse_blocks);
          ts.quarter_poly = runs_in_quarters(l_poly, mc, (int)planes, plan.coarse_blocks);
          ts.quarter_apply = runs_in_quarters(l_app, mc, (int)planes, plan.coarse_blocks);
          if (!mc) {
            ts.tail_sym = tail_in_quarters(l_sym, !ts.quarter_sym, hi_n > kF32LongK, plan.coarse_blocks);
            ts.tail_poly = tail_in_quarters(l_poly, !ts.quarter_poly, hi_m > kF32LongK, plan.coarse_blocks);
            ts.tail_apply = tail_in_quarters(l_app, !ts.quarter_apply, hi_m > kF32LongK, plan.coarse_blocks);
          }
          if (mc) {
            ts.few_sym = few_blocks(l_sym, (int)planes, plan.coarse_blocks);
            ts.few_poly = few_blocks(l_poly, (int)planes, plan.coarse_blocks);
            ts.few_apply = few_blocks(l_app, (int)planes, plan.coarse_blocks);
          }
        }
        ts.long_n = !mc && hi_n > kF32LongK;
        ts.long_m = !mc && hi_m > kF32LongK;
        ts.persistent_n = planes == 1 && steady_n;
        ts.persistent_m = planes == 1 && steady_m;
        ts.sym = take(n_sym * sizeof(GemmTile));
        ts.poly = take(n_sym * sizeof(GemmTile));
        ts.apply = take(n_app * sizeof(GemmTile));      // the last iteration runs the same tiles: only its outputs differ
        // The two symmetric products run the same tiles but not the same K (n for the Gram product, m for the
        // polynomial), so each gets its own table: dealt longest K first and weighted by its own K, and with the costs
        // evened out over a die's blocks where its launch is persistent (where the hardware hands out the blocks, with several
        // planes always, the plain order measured better).
        const int slots = level == 1 && planes == 1 ? plan.coarse_blocks / kXcds : 0;
        ts.n_sym = (int)deal_tiles(by_n, sym, sym_cuts, w_n, reinterpret_cast<GemmTile*>(img.data() + ts.sym), steady_n ? slots : 0, level == 0);
        ts.n_poly = (int)deal_tiles(by_m, sym, sym_cuts, w_m, reinterpret_cast<GemmTile*>(img.data() + ts.poly), steady_m ? slots : 0, level == 0);
        ts.n_apply = (int)deal_tiles(by_m, app, app_cuts, w_m, reinterpret_cast<GemmTile*>(img.data() + ts.apply), steady_m ? slots : 0, level == 0);
      }
      // Where the other group has no symmetric product to share a launch with, a group's coarse tiles may be too few, or leave their rounds badly filled with a K that
      // two-stage tiles handle well: all of them in a fine launch.  us per step, coarse / fine: 30 of 1024^2 with 3 of 1024 x 4096 (30
      // tiles) 1613 / 1465, 12 of 1024 x 4096 (120) 1971 / 1905, 48 with 36 (360 tiles on 256 compute units) 4062 / 4036, 30 with 18 of 1408 x
      // 3840 (324) 3607 / 3442; beside an apply product in fine tiles, 8 of 1024^2 with 6 (60 tiles, 31 us, then the 22 of the apply product) 1057 / 960.
      constexpr double kLoneFill = 0.75, kLoneM = 1536;
      if (g.gram && g.coarse.n_sym > 0 && (few_coarse_sym(coarse_own, (int)planes, plan.coarse_blocks) ||
                                           (coarse_own.m <= kLoneM && coarse_own.fill(plan.coarse_blocks) < kLoneFill))) {
        std::vector<std::vector<GemmTile>> sym(np_);
        std::vector<std::vector<int>> sym_cuts(np_);
        size_t count = 0;
        for (size_t k = 0; k < np_; ++k) {
          const MatPlan& q = plan.mats[members[k]];
          blocked_tiles((int32_t)k, q.tile, kShape128, q.mp / q.tile, q.mp / q.tile, true, 0, 0, -1, sym[k], sym_cuts[k]);
          count += sym[k].size();
        }
        g.lone = take(count * sizeof(GemmTile));
        g.n_lone = (int)deal_tiles(by_m, sym, sym_cuts, w_m, reinterpret_cast<GemmTile*>(img.data() + g.lone), 0, true);
        pair_sides[1].lone = load_of(sym, w_m);
      }
      ch.groups.push_back(g);
    }
    if (ch.paired && ch.groups[0].coarse.n_sym > 0 && ch.groups[1].coarse.n_sym > 0) {
      // one list of both groups' coarse symmetric tiles, dealt as one for every pair of products
      std::vector<std::vector<GemmTile>> tiles = pair_sides[0].coarse_sym;
      std::vector<std::vector<int>> cuts = pair_sides[0].coarse_cuts;
      const int n0 = (int)tiles.size();
      for (size_t k = 0; k < pair_sides[1].coarse_sym.size(); ++k) {
        tiles.push_back(pair_sides[1].coarse_sym[k]);
        for (GemmTile& t : tiles.back()) t.prob += n0;
        cuts.push_back(pair_sides[1].coarse_cuts[k]);
      }
      ch.n_shared_sym = ch.groups[0].coarse.n_sym + ch.groups[1].coarse.n_sym;
      for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2; ++j) {
          if (i && pair_sides[0].w_m == pair_sides[0].w_n) {      // (square matrices: the same K)
            ch.shared_sym[i][j] = ch.shared_sym[0][j];
            continue;
          }
          std::vector<int64_t> w = i ? pair_sides[0].w_m : pair_sides[0].w_n;
          const std::vector<int64_t>& w1 = j ? pair_sides[1].w_m : pair_sides[1].w_n;
          w.insert(w.end(), w1.begin(), w1.end());
          std::vector<int> order(w.size());
          std::iota(order.begin(), order.end(), 0);
          std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return w[x] > w[y]; });
          const int64_t lo = *std::min_element(w.begin(), w.end()), hi = *std::max_element(w.begin(), w.end());
          cursor = align_up(cursor, kTableAlign);
          ch.shared_sym[i][j] = cursor;
          GemmTile* const out = reinterpret_cast<GemmTile*>(img.data() + cursor);
          deal_tiles(order, tiles, cuts, w, out, 2 * hi <= 3 * lo ? plan.coarse_blocks / kXcds : 0, false);
          mark_second(out, ch.n_shared_sym, n0);
          cursor += (size_t)ch.n_shared_sym * sizeof(GemmTile);
        }
    }
    if (ch.paired && !members_of[0].empty() && !few_coarse_apply(coarse_app_all, (int)planes, plan.coarse_blocks)) {
      // one list of both groups' coarse tiles of the apply products
      std::vector<std::vector<GemmTile>> tiles;
      std::vector<std::vector<int>> cuts;
      std::vector<int64_t> w;
      size_t count[2] = {0, 0};
      bool fits = true;                          // all-fine products: nothing may be left beside the coarse tiles
      const int n0 = (int)members_of[0].size();
      for (int r = 0; r < 2; ++r) {
        const bool fine = ch.groups[r].coarse.n_apply == 0;
        for (size_t k = 0; k < members_of[r].size(); ++k) {
          const MatPlan& q = plan.mats[members_of[r][k]];
          std::vector<GemmTile> own;
          std::vector<int> own_cuts;
          if (!fine) {
            own = pair_sides[r].coarse_app[k];
            own_cuts = pair_sides[r].app_cuts[k];
          } else {
            const bool strip = q.mp % kCoarse != 0;
            fits = fits && q.np % kCoarse == 0 && (!strip || q.np >= kShapeRows[kShape512x128]);
            if (!fits) break;
            blocked_tiles((int32_t)k, kCoarse, kShape256, q.np / kCoarse, q.mp / kCoarse, false, 0, 0, -1, own, own_cuts, 8, 2);
            if (strip) strip_tiles((int32_t)k, q.np, q.mp - q.tile, own, own_cuts);
            ch.shared_app_strips = ch.shared_app_strips || strip;
          }
          count[r] += own.size();
          for (GemmTile& t : own) t.prob += r * n0;
          tiles.push_back(std::move(own));
          cuts.push_back(std::move(own_cuts));
        }
        ch.shared_app_strips = ch.shared_app_strips || (!fine && ch.groups[r].coarse.strips);
        w.insert(w.end(), pair_sides[r].w_m.begin(), pair_sides[r].w_m.end());
      }
      const size_t start = align_up(cursor, kTableAlign), bytes = (count[0] + count[1]) * sizeof(GemmTile);
      if (fits && start + bytes <= tl.total &&
          saves_a_round(count[0], ch.groups[0].coarse.n_apply == 0, count[1], ch.groups[1].coarse.n_apply == 0, plan.coarse_blocks)) {
        std::vector<int> order(w.size());
        std::iota(order.begin(), order.end(), 0);
        std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return w[x] > w[y]; });
        ch.shared_app_steady = 2 * *std::max_element(w.begin(), w.end()) <= 3 * *std::min_element(w.begin(), w.end());
        ch.shared_app = start;
        ch.n_shared_app = (int)(count[0] + count[1]);
        GemmTile* const out = reinterpret_cast<GemmTile*>(img.data() + start);
        deal_tiles(order, tiles, cuts, w, out, ch.shared_app_steady ? plan.coarse_blocks / kXcds : 0, false);
        mark_second(out, ch.n_shared_app, n0);
        cursor = start + bytes;
      }
    }
    if (ch.paired) {
      for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 4; ++j) ch.pair[i][j] = pair_form(pair_sides[0], i, pair_sides[1], j, plan.coarse_blocks);
      for (int i = 0; i < 2; ++i)
        for (int p : {kPairGram, kPairSym, kPairApply}) {
          const Group& g = ch.groups[i];
          const bool lone = p == kPairSym && g.n_lone > 0;
          ch.beside[i][p] = (lone || (p == kPairApply ? g.coarse.n_apply : g.coarse.n_sym) == 0) && pair_sides[i].lo[p] >= kRingK &&
                            fits_beside(ch.groups[i ^ 1], lone ? pair_sides[i].lone : pair_sides[i].load[p], plan.coarse_blocks);
        }
      ch.groups[1].lone_form[0] = fine_form(pair_sides[1].lone, {}, plan.coarse_blocks);
      ch.groups[1].lone_form[1] = fine_form(pair_sides[1].lone, pair_sides[0].load[kPairApply], plan.coarse_blocks);
    }
    {
      // Lists short enough for quarter blocks or the 128-wide ring save the norm's own launch (about 4 us): every block adds up its matrix's
      // partials while its first operands are on their way, at most four per thread, or per lane where it is a wave.  With
      // waves the norm's launch / the fold, us per step: 64 x 4000 (126 partials) 110.0 / 109.2, 64 x 8000 (252) 170.0 / 170.4, 256 x
      // 8000 (504) 185.0 / 186.1, 128 x 16000 (500) 279.6 / 281.6, 64 x 32000 (1000) 508.8 / 510.0.
      constexpr int kFoldedPerThread = 4;
      const PairForm& first = ch.pair[ch.groups[0].n_prob > 0 ? kPairGram : kPairNone][kPairGram];
      const int few = ch.paired ? first.few : ch.groups[0].fine.few_sym;
      const int most_folded = kFoldedPerThread * (few == 2 ? 64 : 256);
      int most_parts = 0;
      for (int i = ch.first; i < ch.first + ch.count; ++i) most_parts = std::max(most_parts, h_mats[i].n_part);
      bool coarse = false;
      for (const Group& g : ch.groups) coarse = coarse || g.coarse.n_sym > 0;
      ch.fold_norm = !coarse && (ch.paired ? first.quarters || first.few == 3 : ch.groups[0].fine.quarter_sym || few == 3) && most_parts <= most_folded;
    }
  }
  if (cursor > tl.total) return MUON_E_WORKSPACE_TOO_SMALL;   // the layout bound is conservative; this cannot happen
  img.resize(cursor);
  plan.image.swap(img);
  plan.off_mats = off_mats;
  plan.off_ptrs = off_ptrs;
  return MUON_OK;
}

int64_t plan_tiles(const Plan& plan, int chunk, int product, int level, int32_t* out, int32_t cap_records) {
  int64_t total = 0;
  const bool mc = on_matrix_cores(plan.ns_dtype);
  for (const Group& g : plan.chunks[chunk].groups) {
    const TileSet& ts = level ? g.coarse : g.fine;
    const size_t off = product == 0 ? ts.sym : product == 1 ? ts.poly : ts.apply;
    const int count = product == 0 ? ts.n_sym : product == 1 ? ts.n_poly : ts.n_apply;
    const GemmTile* t = reinterpret_cast<const GemmTile*>(plan.image.data() + off);
    for (int i = 0; i < count; ++i, ++total) {
      if (total >= cap_records) continue;
      int32_t* r = out + 6 * total;
      r[0] = g.members[t[i].prob];
      r[1] = t[i].r0 * kTileUnit;
      r[2] = t[i].c0 * kTileUnit;
      r[3] = mc ? kShapeRows[t[i].shape] : kF32Tile;
      r[4] = mc ? kShapeCols[t[i].shape] : kF32Tile;
      // 32 x 32 blocks of the tile that are computed: all of them, except for the diagonal shape (upper triangle)
      r[5] = mc && t[i].shape == kShape256Diag ? 36 : r[3] / 32 * (r[4] / 32);
    }
  }
  return total;
}

}  // namespace muon
