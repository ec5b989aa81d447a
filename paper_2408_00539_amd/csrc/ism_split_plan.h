// Host part of the split-key launches (plain C++, no HIP): which kernel a
// cached prefill takes, the columns and key tiles of its workgroups, and how
// many units the device plan (ism_plan.h) may make of the dialogues' keys.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace ism {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// How a cached prefill runs: kOneWave when the (row, query head) pairs of the
// longest new segment that share a KV head fill at most one 32-column block,
// so that the cache is streamed once (two blocks would stream it twice: the
// row-tiled forward kernel shares its K/V tiles among four waves); else the
// forward kernel, its key ranges split into about 448 units when its
// workgroups leave most of the 512 that fit the chip unused. Measured
// unsplit against split (us), by workgroups: 32 (8 ragged dialogues up to
// 12000 keys, 16 rows, 32/2 heads) 172, 43; 32 (1 x 4000, 100 rows, 32/8) 64,
// 31; 160 (10 x 3000, 50 rows, 32/8) 61, 55; 236 (8 ragged up to 3000, 200
// rows, 32/2) 83, 114; 320 (20 ragged up to 4000, 60 rows, 32/8) 95, 120: the
// partials of that many rows cost more than the idle workgroups.
enum PrefillKind { kRowTiles, kRowTilesSplit, kOneWave };
inline PrefillKind prefill_kind(int32_t batch, int64_t total_new, int32_t max_new, int32_t hq,
                                int32_t hkv) {
  const int64_t g = hq / hkv;
  if (max_new * g <= 32) return kOneWave;
  const int64_t wgs = hkv * (total_new * g / 128 + batch);
  return wgs < 192 ? kRowTilesSplit : kRowTiles;
}

// The columns of a workgroup and how many units to make. The kernel decides
// the shape: one-wave workgroups of 32 columns and 32-key tiles (kOneWave,
// and every decode step: ism_split.hip, where the unit counts are measured),
// or the forward kernel's of 128 columns and 64-key tiles. A chunk is cut for
// at least min_tiles tiles (the chunks of a dialogue are then evened out, so
// a short dialogue's may hold fewer); at most 64 chunks.
struct SplitPlan {
  int32_t colw, col_groups, col_stride, budget, max_units, max_splits, tile_shift, min_tiles;
  // workspace of the partials and the plan (0: one chunk per dialogue)
  size_t part_bytes, ml_bytes, plan_bytes;
  size_t bytes() const { return part_bytes + ml_bytes + plan_bytes; }
};

constexpr int kSplitUnits = 640, kSplitUnits64 = 960, kSplitUnits128 = 448;
// From this many (dialogue, KV head, column group) workgroups on (1280 one-wave
// workgroups fit the chip), a one-wave launch keeps every dialogue whole and
// needs no plan, whose scans over many dialogues every workgroup would repeat.
// Measured with the plan and without (us): decode, 32/8 heads, 256 ragged
// dialogues up to 1000 keys 106.3, 101.6; 1000: 404, 347; 2000: 1080, 845; 8
// drafted rows over 300 ragged up to 800 keys 128, 114; 64/8 heads, d 64, 256
// x 300 keys 34.9, 28.1. Below it, splitting the long dialogues of a ragged
// batch is worth the plan.
constexpr int kSplitDirect = 2048;
inline SplitPlan split_plan(PrefillKind kind, int32_t batch, int64_t total_rows, int32_t max_rows,
                            int32_t hq, int32_t hkv, int32_t d, int64_t max_len, int32_t fixed,
                            bool limited, size_t ws_bytes) {
  SplitPlan p{};
  const int64_t cols = (int64_t)max_rows * (hq / hkv);
  const bool one_wave = kind == kOneWave;
  p.colw = one_wave ? 32 : 128;
  p.tile_shift = one_wave ? 5 : 6;
  p.min_tiles = 4;
  p.col_groups = (int32_t)((cols + p.colw - 1) / p.colw);
  p.col_stride = (int32_t)(cols < p.colw ? cols : p.colw);
  const int target = !one_wave ? kSplitUnits128 : d == 64 ? kSplitUnits64 : kSplitUnits;
  p.budget = (target + hkv - 1) / hkv;
  const int64_t tiles = (max_len + (1 << p.tile_shift) - 1) >> p.tile_shift;
  const int64_t most = fixed > 0 ? fixed : (tiles + p.min_tiles - 1) / p.min_tiles;
  p.max_splits = (int32_t)(most < 1 ? 1 : fixed <= 0 && most > 64 ? 64 : most);
  if (one_wave && fixed <= 0 && (int64_t)batch * hkv * p.col_groups >= kSplitDirect)
    p.max_splits = 1;
  // column groups of all dialogues together, partials of one unit over all
  // KV heads
  const int64_t by_rows = total_rows * (hq / hkv) / p.colw + batch, groups = p.col_groups;
  const int64_t all_groups = by_rows < (int64_t)batch * groups ? by_rows : (int64_t)batch * groups;
  const int64_t per = (int64_t)hkv * p.col_stride * (d + 2) * 4;
  int64_t units = all_groups * p.max_splits;
  if (fixed <= 0 && units > (int64_t)p.budget + all_groups) units = (int64_t)p.budget + all_groups;
  auto layout = [&](int64_t n) {
    p.max_units = (int32_t)n;
    p.part_bytes = align_up((size_t)n * hkv * p.col_stride * d * 4);
    p.ml_bytes = align_up((size_t)n * hkv * p.col_stride * 2 * 4);
    p.plan_bytes = align_up((size_t)batch * 2 * 4);
  };
  layout(units);
  if (limited && p.max_splits > 1 && p.bytes() > ws_bytes) {
    // a smaller workspace: fewer units, down to one chunk per dialogue (the
    // two partial buffers are rounded up, by less than kAlign each)
    const int64_t fit = ((int64_t)ws_bytes - (int64_t)p.plan_bytes - 2 * (int64_t)kAlign) / per;
    if (fixed > 0 && fit >= all_groups) {
      p.max_splits = (int32_t)(fit / all_groups);
      layout(all_groups * p.max_splits);
    } else if (fixed <= 0 && fit > all_groups) {
      p.budget = (int32_t)(fit - all_groups);
      layout(fit);
    } else {
      p.max_splits = 1;
    }
  }
  if (p.max_splits == 1) {
    p.max_units = (int32_t)all_groups;
    p.part_bytes = p.ml_bytes = p.plan_bytes = 0;
  }
  return p;
}

}  // namespace ism
