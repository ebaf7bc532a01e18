// The prefill kernel's tiles and the work plan of a call, for the kernel
// (prefill.hip) and for the entry points and their workspace (jfkv_host.cpp).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "jfkv_internal.h"

namespace jfkv {
namespace prefill {

// Keys per tile (a page holds whole tiles): 64, or 32 at d = 256, where the
// double-buffered K and two V tiles of 64 keys would not fit in LDS.
template <int D>
constexpr int keys_per_tile() { return D > 128 ? 32 : 64; }
constexpr int kWaves = 8;          // waves per block: two per SIMD
// 16-row MFMA tiles of query rows per wave (the registers of d = 256 hold one)
template <int D>
constexpr int row_tiles() { return D > 128 ? 1 : 2; }

// fp32 words of a part of a row block in the workspace: per wave the output
// accumulators ([dim tile][row tile][lane] of four), then (maximum, sum)
// ([row tile][lane])
template <int D>
constexpr int part_floats() { return kWaves * row_tiles<D>() * 64 * (D / 4 + 2); }

// Key tiles of the row blocks of one KV head in turn: block rb (rows rb * rows
// .. of (position, query head) rows) has the prefix's n_pre tiles and those of
// the chunk up to its last position.  Its last row over gq * kt is carried as
// quotient and remainder, so stepping needs no division.
struct RowBlockTiles {
  int n_pre, last, q, r, dq, dr, u;
  __host__ __device__ RowBlockTiles(int rows, int T, int gq, int n_pre_, int kt)
      : n_pre(n_pre_), last((T - 1) / kt), u(gq * kt) {
    q = (rows - 1) / u;
    r = (rows - 1) % u;
    dq = rows / u;
    dr = rows % u;
  }
  __host__ __device__ int tiles() const { return n_pre + 1 + (q < last ? q : last); }
  __host__ __device__ void next() {
    q += dq;
    r += dr;
    if (r >= u) {
      r -= u;
      ++q;
    }
  }
};

// How a call's work is laid over the chip: n_blk blocks per KV head share the
// head's `tiles` key tiles (over all its row blocks) evenly, or n_blk = 0: one
// block per row block.  A block fills a CU, so row blocks that do not fill the
// chip, or leave its last turn nearly empty, cost as much as if they did.
// Row blocks are started in turn, later ones have more tiles, and a CU takes
// the next when it is done, so its chain is row blocks i, i + CUs, ...; the
// longest chain is the time of whole row blocks.
// Shares of one tile pay while half the chip takes them, otherwise two tiles
// and more (without a prefix, where tiles are shorter, four).  An even share
// takes its tiles and, in tiles too (SplitCost), a query load, a pipeline fill
// and a state to store for each further row block that it touches, and (with a
// prefix, where chunk rows are not fetched ahead) more for chunk tiles; the
// call takes its longest share, the combine's launch, and the states' traffic in
// proportion to the blocks.
// Fitted at 1,830 shapes of 16..8,192 rows, a third of them without a prefix,
// the others over 1..200,000 positions, with 4 to 64 query heads of 64, 128 and
// 256 dims, each laid out both ways (a tile takes 3.0, 1.8 and 2.1 us at
// head_dim 128, 64 and 256 with a prefix, 2.3, 1.3 and 1.4 without): the rule's
// choices cost 0.06 % more than the faster layout of each shape, 4 us at most
// below 35 us and 6 % at most above.
// Measured, even shares against whole row blocks: 256 rows over 196,608 (24/4
// heads, 256) 2.50 against 13.1 ms; 1,000 over 7,000 (32/8, 128) 218 against
// 392 us; 100 over 20,000 (4/1, 128) 37 against 1,010 us; 72 over 162 (4/1,
// 128) 17 against 23 us; and where row blocks stay whole: 16 over 162 (4/1,
// 128) 18.1 against 17.4 us; without a prefix, 4,096 of 32/8 heads, 128, 260
// against 230, 2,509 of 64/8 256 against 183, 5,981 of 16/2, 64, 214 against 174.
struct SplitCost {
  double combine;  // per call
  double part;     // per further row block that a share touches
  double full;     // of the states, when the blocks fill the chip
  double chunk;    // more per chunk tile of a share
};
template <int D, bool PRE>
constexpr SplitCost kSplitCost = D == 128  ? (PRE ? SplitCost{1, 2.3, 3, 0.06} : SplitCost{0.2, 3.8, 6.3, 0})
                                 : D == 64 ? (PRE ? SplitCost{4.7, 2, 0.8, 0.36} : SplitCost{0.9, 4.5, 7.1, 0})
                                           : (PRE ? SplitCost{2.5, 3.6, 2, 0.37} : SplitCost{7.6, 7.6, 0.7, 0});
// A split has to gain what its scratch, its second launch and the estimate's own
// error are worth.  2,048 rows of 32/8 heads (two full turns): over 16,384
// positions estimated at 2.7 % less, 874 against 897 us; over 32,768 1.4 % less,
// 1,647 against 1,669; over 65,536 0.7 % less, 3,189 against 3,206; over 131,072
// 0.4 % less, 6,291 against 6,283.
constexpr double kWorthwhile = 0.98;
constexpr int64_t kMaxTurns = 16;  // row blocks per CU above which the last turn hardly counts

template <int D>
PrefillPlan plan_t(const jf_kv_layout& L, int32_t T, int32_t Hq, int32_t prefix_len, bool split) {
  constexpr int kRows = 16 * row_tiles<D>() * kWaves;
  constexpr int KT = keys_per_tile<D>();
  PrefillPlan p;
  const int gq = Hq / L.num_kv_heads;
  const int n_pre = (int)(((int64_t)prefix_len + KT - 1) / KT);
  p.n_rb = ((int64_t)T * gq + kRows - 1) / kRows;
  if (!split) return p;
  const int64_t per_head = std::max(1, num_cus() / L.num_kv_heads);
  if (p.n_rb > kMaxTurns * per_head) return p;
  // tiles of the two longest chains of row blocks on one CU: the last of those
  // without and of those with a row block in the last turn
  int64_t chain[2] = {0, 0};
  const int64_t last = (p.n_rb - 1) % per_head;
  RowBlockTiles rbt(kRows, T, gq, n_pre, KT);
  for (int64_t rb = 0, cu = 0; rb < p.n_rb; ++rb, rbt.next()) {
    const int t = rbt.tiles();
    p.tiles += t;
    if (cu == last) chain[1] += t;
    if (++cu == per_head) {
      cu = 0;
      chain[0] += t;
    }
  }
  const int64_t whole = std::max(chain[0], chain[1]);
  const int64_t n_blk =
      n_pre ? std::max(std::min(p.tiles, per_head / 2), std::min(p.tiles / 2, per_head))
            : std::min(p.tiles / 4, per_head);
  if (n_blk <= 1) return p;
  const SplitCost c = n_pre ? kSplitCost<D, true> : kSplitCost<D, false>;
  const double tile = 1 + c.chunk * (p.tiles - p.n_rb * n_pre) / p.tiles;
  const double fixed = c.combine + c.full * n_blk / per_head, limit = kWorthwhile * whole;
  const int64_t share = p.tiles / n_blk, rest = p.tiles % n_blk;
  if (share * tile + fixed >= limit) return p;
  // share j is tiles j * tiles / n_blk .. (j + 1) * tiles / n_blk - 1
  double longest = 0;
  rbt = RowBlockTiles(kRows, T, gq, n_pre, KT);
  int64_t end = rbt.tiles();  // of the row blocks up to rbt's
  for (int64_t j = 0, to = 0, part = 0; j < n_blk; ++j) {
    const int64_t from = to;
    to += share;
    if ((part += rest) >= n_blk) {
      part -= n_blk;
      ++to;
    }
    int more = 0;
    while (end < to) {
      more += end > from;  // (or the share begins with the next row block)
      rbt.next();
      end += rbt.tiles();
    }
    longest = std::max(longest, (to - from) * tile + c.part * more);
  }
  if (longest + fixed < limit && (n_blk + 1) * p.tiles <= INT32_MAX)  // (the kernels' products)
    p.n_blk = (int)n_blk;
  return p;
}

// split false: whole row blocks, as without a workspace.
inline PrefillPlan make_plan(const jf_kv_layout& L, int32_t T, int32_t Hq, int32_t prefix_len,
                             bool split) {
  return L.head_dim == 64    ? plan_t<64>(L, T, Hq, prefix_len, split)
         : L.head_dim == 128 ? plan_t<128>(L, T, Hq, prefix_len, split)
                             : plan_t<256>(L, T, Hq, prefix_len, split);
}

inline size_t plan_bytes(const jf_kv_layout& L, const PrefillPlan& p) {
  const size_t part = L.head_dim == 64 ? part_floats<64>() : L.head_dim == 128 ? part_floats<128>() : part_floats<256>();
  return 2 * (size_t)p.n_blk * L.num_kv_heads * part * sizeof(float);
}

}  // namespace prefill
}  // namespace jfkv
