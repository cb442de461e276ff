// The plan of a partial call: row tile, splits and what they keep in the
// split-K workspace.  Host arithmetic only.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "mla_kernels.h"

namespace mla {

// What the plan is made from: jobs, query rows and heads of a job, logical
// blocks and slots of a selection, its kind, the caller's options (0: the
// library's choice) and the compute units of the device.
struct PlanArgs {
  int64_t R, Mq, H, NB, K;
  bool tokens, per_row, fp8;
  int32_t n_splits, row_tile;
  int64_t cus;
};

struct Plan {
  int row_groups;          // of 64 rows a tile: 1 or 2
  int64_t row_tiles;       // tiles of a job
  int64_t S, sps;          // splits of a tile's slots, slots of a split
  bool by_id;              // splits by logical block instead of slot range
  bool long_lists;         // 64-row tiles: lists too long for the eight-wave kernel
  double us;               // what the call should take
};

// Bytes of split rows that a plan stays within where any plan does: what the
// allocation-free entry's scratch array holds.
constexpr uint64_t kPlanScratch = 64ull << 20;

struct Planner {
  PlanArgs a;
  int64_t rows, Kb;        // of a job; slots in 64-token blocks
  int64_t tile_qrows = 1;  // per-row selections: query rows a tile spans (one mask bit each)
  int row_groups = 0;      // of every plan, or 0: either
  const char* refused = nullptr;
  Plan cover{};            // the fewest splits that give every compute unit a workgroup
  bool keep32 = false;     // split rows are held in fp32, whatever their number

  explicit Planner(const PlanArgs& args) : a(args), rows(a.Mq * a.H) {
    Kb = a.tokens ? (a.K + 63) / 64 : a.K;  // a token selection's slots fill K / 64 blocks
    // the row groups of the covering plan: the caller's; 1 where a job has no
    // more rows; 2 where splits are long (8 blocks and more).  Per-row selections
    // keep to them, for a tile of twice the rows shares more loads; elsewhere the
    // cheaper is taken
    int groups = 1;
    if (a.row_tile) {
      groups = a.row_tile / 64;
    } else if (rows > 64) {
      const int64_t units2 = a.R * row_tiles_of(2);
      const int64_t s2 = std::min<int64_t>((a.cus + units2 - 1) / units2, std::max<int64_t>(Kb / 2, 1));
      groups = Kb < 8 * s2 ? 1 : 2;
    }
    if (a.per_row) {
      if (groups == 2 && tile_query_rows(2) > kPerRowMaxRows) {
        if (a.row_tile == 128) {
          refused = "per-row selections: too many query rows per 128-row tile";
          return;
        }
        groups = 1;
      }
      tile_qrows = tile_query_rows(groups);
      if (tile_qrows > kPerRowMaxRows) refused = "per-row selections: too many query rows per tile";
      else if (a.NB * tile_qrows * 2 > kPerRowCounterBytes)
        refused = "per-row selections: NB x query rows per tile too large";
      if (refused) return;
    }
    row_groups = a.row_tile || rows <= 64 || a.per_row ? groups : 0;
    // at least two blocks a split: one block costs less than its split's fixed
    // part.  Two splits of at most two blocks save at most two blocks' time and
    // add the combine's launch: one split does better (4 blocks of one 16-row
    // job: 12.4 us in one split against 14.9 in two)
    const int64_t units = std::max<int64_t>(a.R * row_tiles_of(groups), 1);
    int64_t S = std::min<int64_t>((a.cus + units - 1) / units, std::max<int64_t>(most_blocks() / 2, 1));
    if (S == 2 && !by_id() && Kb <= 5) S = 1;
    cover = plan_of(groups, std::max<int64_t>(S, 1));
    // Sums that the covering plan holds in fp32 (in registers from the first
    // block to the last, or in a few split rows) are held so in any other.
    keep32 = a.n_splits == 0 && (cover.S == 1 || !ws_half(cover.S));
  }

  int64_t row_tiles_of(int rg) const { return (rows + 64 * rg - 1) / (64 * rg); }

  int64_t tile_query_rows(int rg) const {
    const int64_t rw = 64 * rg;
    int64_t most = 0;
    for (int64_t r0 = 0; r0 < rows; r0 += rw) {
      const int64_t last = std::min<int64_t>(r0 + rw, rows) - 1;
      most = std::max<int64_t>(most, last / a.H - r0 / a.H + 1);
    }
    return most;
  }

  // Split rows in the workspace, then their scales (fp16 rows only), then their
  // lse values and maxima.  fp16 rows halve the workspace round trip, which pays
  // from about a megabyte of split rows on; tiny workspaces keep fp32 rows,
  // whose epilogue is a little shorter, and so do plans of more splits than the
  // covering one where that holds fp32: 300 jobs of 16 rows x 64 blocks, one
  // split to cover the chip, take 256 us in that, 242 in three with fp32 rows
  // (240 with fp16 ones).
  uint64_t split_rows(int64_t S) const { return (uint64_t)a.R * S * rows; }
  bool ws_half(int64_t S) const { return !keep32 && split_rows(S) * kDLat * 4 >= kWsHalfMinBytes; }
  uint64_t ws_rows_bytes(int64_t S) const { return split_rows(S) * kDLat * (ws_half(S) ? 2 : 4); }
  uint64_t ws_size(int64_t S) const { return ws_rows_bytes(S) + 3 * split_rows(S) * 4; }
  bool fits(const Plan& q) const { return q.S <= 1 || ws_size(q.S) <= kPlanScratch; }

  // entries one split's list holds (per-row selections with an fp8 cache: a
  // shorter one, see the kernel's LDS layout)
  int64_t list_cap() const { return a.per_row && a.fp8 ? kPerRowListShort : kMaxSlotsPerSplit; }
  // per-row selections whose tile slots all fit one list split by logical
  // block: every split then scans all slots and the rows that chose a block
  // in different slots still share its load
  bool by_id() const { return a.per_row && tile_qrows > 1 && a.K * tile_qrows <= list_cap(); }
  // the most blocks a tile can visit
  int64_t most_blocks() const { return by_id() ? std::min<int64_t>(a.NB, a.K * tile_qrows) : Kb; }

  // the plan of about S splits with tiles of rg row groups, and its time
  Plan plan_of(int rg, int64_t S) const {
    Plan q{rg, row_tiles_of(rg), S, a.K, by_id(), false, 0.0};
    // a split's block list holds at most so many entries: its slots, or for
    // per-row selections its slots of every query row of the tile
    const int64_t cap = list_cap();
    if (a.tokens) {
      // whole virtual blocks per split, at most one list of tokens
      S = std::max<int64_t>(S, (a.K + kMaxSlotsPerSplit - 1) / kMaxSlotsPerSplit);
      q.sps = std::max<int64_t>(64, ((a.K + S - 1) / S + 63) / 64 * 64);
      q.sps = std::min<int64_t>(q.sps, kMaxSlotsPerSplit);
      q.S = std::max<int64_t>(1, (a.K + q.sps - 1) / q.sps);
    } else if (!q.by_id) {
      S = std::max<int64_t>(S, (a.K * tile_qrows + cap - 1) / cap);
      q.sps = std::max<int64_t>(1, (a.K + S - 1) / S);
      if (a.per_row) q.sps = std::min<int64_t>(q.sps, std::max<int64_t>(1, cap / tile_qrows));
      q.S = std::max<int64_t>(1, (a.K + q.sps - 1) / q.sps);
    }
    q.long_lists = a.per_row && !a.fp8 && rg == 1 && q.sps * tile_qrows > kPerRowListShort;
    // What a call takes, microseconds.  A workgroup fills its CU, so that a
    // grid goes in waves of one a CU.  A wave takes as long as one of its work
    // items, a fixed part (its prologue, query rows and epilogue) and its blocks'
    // time, or as the bytes of all its blocks take from memory: a last wave of a
    // few workgroups is bound by the former, a full one often by the latter.
    // Splits add the combine, by the bytes of the rows it reads.  The rows' own
    // bytes are left out.  Fitted to 140000 timed plans of 28000 calls of 1..700
    // jobs of 8..256 rows x 1..1500 blocks or 16..6000 tokens (9 % rms in 128-row
    // tiles, 9 to 17 % in 64-row ones).
    const double blocks = q.by_id ? (double)((most_blocks() + q.S - 1) / q.S)
                        : a.tokens ? (double)((q.sps + 63) / 64)
                        : a.per_row ? (double)std::min<int64_t>(std::max<int64_t>(a.NB, 1), q.sps * tile_qrows)
                        : (double)q.sps;
    struct Rate {
      double fixed, block, bytes;  // us, us, bytes a us
    };
    // by selection, cache and tile: half of a 64-row tile, one for all rows,
    // one of several, 128 rows
    static constexpr Rate kRate[2][2][4] = {
        {{{5.5, 1.62, 6.3e6}, {7.9, 1.83, 5.9e6}, {8.2, 1.85, 7.5e6}, {14.0, 3.27, 4.8e6}},
         {{6.6, 1.87, 5.5e6}, {9.4, 2.32, 5.5e6}, {9.4, 2.30, 5.5e6}, {14.1, 4.16, 5.5e6}}},
        {{{5.0, 1.99, 6.6e6}, {7.8, 2.19, 6.1e6}, {8.5, 2.17, 8.7e6}, {14.2, 3.78, 5.0e6}},
         {{5.7, 2.38, 5.5e6}, {8.4, 2.64, 5.5e6}, {9.2, 2.49, 5.5e6}, {14.5, 4.89, 5.5e6}}}};
    const Rate& rate = kRate[a.tokens][a.fp8][rg == 2 ? 3 : rows <= 32 ? 0 : rows <= 64 ? 1 : 2];
    // (rows with selections of their own share blocks, nobody here knows which)
    const double item_bytes = a.per_row ? 0.0 : blocks * kBlock * (kDLat + kDPe) * (a.fp8 ? 1 : 2);
    auto wave_us = [&](int64_t items) {
      return rate.fixed + std::max(blocks * rate.block, (double)items * item_bytes / rate.bytes);
    };
    const int64_t items = a.R * q.row_tiles * q.S, rest = items % a.cus;
    q.us = (double)(items / a.cus) * wave_us(a.cus) + (rest ? wave_us(rest) : 0.0);
    if (q.S > 1) q.us += 1.8 + 0.4e-6 * (double)ws_rows_bytes(q.S);
    return q;
  }

  Plan choose() const {
    Plan plan{};
    if (a.n_splits > 0) {
      for (int rg = 2; rg >= 1; --rg) {
        if (row_groups && rg != row_groups) continue;
        const Plan q = plan_of(rg, std::min<int64_t>(a.n_splits, std::max<int64_t>(by_id() ? a.NB : a.K, 1)));
        if (!plan.row_groups || q.us < plan.us) plan = q;
      }
      return plan;
    }
    // The covering plan, one split, or as many as one, two or three waves of
    // workgroups hold.  A grid just past a whole number of waves costs a wave
    // more: 20 jobs of 128 rows x 200 blocks take 122 us in 13 splits (260
    // workgroups) and 85 in 12, 40 x 600 blocks 622 and 420 (fp8 708 and 446), 24
    // of 2048 tokens 67 and 39.  Several waves of shorter splits where one wave
    // leaves CUs idle: 281 jobs of 8 rows x 86 fp8 blocks 327 us in one split,
    // 241 in three.  A plan has to promise 3 % over the covering one, about what
    // the prices are off between plans of one call: of the timed calls one in
    // 4000 then takes 2 % more than in the covering plan, and the mean is 9.3 %
    // less (9.5 with the best plan of each call; a fourth wave adds nothing).
    // A plan whose split rows fit the allocation-free entry's scratch (64 MiB)
    // goes before one whose rows do not, for every entry; where a list's limit
    // leaves none that fits, the cheapest is taken: 256 jobs of 128 rows x 2048
    // tokens, two splits at least, take 395 us in 64-row tiles and 211 in 128-row
    // ones, and their split rows are the same 65 MiB.
    // Per-row selections in ranges of slots keep the covering plan: a block that
    // rows chose in different slots is loaded once a range, so that other ranges
    // mean other loads, which only the ids tell (28 jobs of 10 x 16 rows with 144
    // blocks each: 268 us in four ranges, priced cheaper, 241 in the covering
    // five).
    plan = cover;
    if (a.per_row && tile_qrows > 1 && !by_id()) return plan;
    double best = 0.97 * cover.us;
    for (int rg = 1; rg <= 2; ++rg) {
      if (row_groups && rg != row_groups) continue;
      const int64_t units = std::max<int64_t>(a.R * row_tiles_of(rg), 1);
      const int64_t most = std::max<int64_t>(most_blocks() / 2, 1);
      int64_t last = 0;
      for (int waves = 0; waves <= 3; ++waves) {
        const int64_t S = std::max<int64_t>(1, std::min<int64_t>(waves * a.cus / units, most));
        if (S == last || (S == 2 && !by_id() && Kb <= 5)) continue;
        last = S;
        const Plan q = plan_of(rg, S);
        if (fits(plan) && !fits(q)) continue;
        if ((fits(q) && !fits(plan)) || q.us < best) {
          plan = q;
          best = q.us;
        }
      }
    }
    return plan;
  }
};

}  // namespace mla
