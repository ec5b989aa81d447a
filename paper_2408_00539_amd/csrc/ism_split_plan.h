// Host part of the split-key launches (plain C++, no HIP): which kernel a
// cached prefill takes, the columns and key tiles of its workgroups, and how
// many units the device plan (ism_plan.h) may make of the dialogues' keys.
#pragma once

#include <stddef.h>
#include <stdint.h>

namespace ism {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// How a call over the cache runs. A decode step: the split-key kernel. A
// cached prefill: the same kernel (kOneWave) when the (row, query head) pairs
// of the longest new segment that share a KV head fill at most one 32-column
// block, so that the cache is streamed once (two blocks would stream it
// twice: the row-tiled forward kernel shares its K/V tiles among four waves);
// else the forward kernel, its key ranges split when its workgroups leave
// most of the 512 that fit the chip unused and the cache is longer than two
// chunks. Measured unsplit against split (us), by workgroups: 32 (8 dialogues
// of 2000 to 12000 keys, 16 rows, 32/2 heads) 170, 37; 32 (1 x 4000, 100 rows,
// 32/8) 63, 33; 160 (10 x 3000, 50 rows, 32/8) 61, 55; 236 (8 ragged up to
// 3000, 200 rows, 32/2) 83, 114; 320 (20 ragged up to 4000, 60 rows, 32/8) 95,
// 120: the partials of that many rows cost more than the idle workgroups. By
// capacity: 768 (1 x 600, 100 rows, 32/8) 19.3, 21.0; 1024 (3 x 700, 64 rows)
// 20.7, 24.7; 1280 (12 x 1000, 33 rows) 27.5, 26.7; 2304 (8 x 2000, 12 rows,
// 64/8, d 64) 34.5, 23.5.
enum SplitKind { kRowTiles, kRowTilesSplit, kOneWave, kDecodeStep };
inline SplitKind prefill_kind(int32_t batch, int64_t total_new, int32_t max_new, int32_t hq,
                              int32_t hkv, int32_t cache_cap) {
  const int64_t g = hq / hkv;
  if (max_new * g <= 32) return kOneWave;
  const int64_t wgs = hkv * (total_new * g / 128 + batch);
  return wgs < 192 && cache_cap > 1024 ? kRowTilesSplit : kRowTiles;
}

// The columns of a workgroup and how many units to make. The kernel decides
// the shape: one-wave workgroups of 32 columns and 32-key tiles (ism_split.hip)
// or the forward kernel's of 128 columns and 64-key tiles. A chunk is cut for
// at least min_tiles tiles, 128 or 256 keys (the chunks of a dialogue are then
// evened out, so those of a short dialogue can be smaller); at most 64 chunks.
// Row-tiled dialogues of up to 512 keys stay whole, as their rows' partials
// cost more than the second chunk saves (cache of 8192, 4 x 300 keys, 40 rows,
// 32 heads 19.4 whole, 21.1 us cut; 1 x 300, 200 rows, 32/8 20.4, 22.6).
struct SplitPlan {
  int32_t colw, col_groups, col_stride, budget, max_units, max_splits, tile_shift, min_tiles;
  int32_t whole_tiles;
  // workspace of the partials and the plan (0: one chunk per dialogue)
  size_t part_bytes, ml_bytes, plan_bytes;
  size_t bytes() const { return part_bytes + ml_bytes + plan_bytes; }
};

// Units of all KV heads at most, which is also the grid: the one-wave
// workgroups that the chip holds at once at d = 128 (four to a CU by their
// LDS), so that the last chunks don't start when the first end, and no
// surplus workgroups pass through the CUs (a surplus left some SIMDs with two
// of a call's waves, which then end last: 800 units with 640 surplus workgroups
// 589 us, without 544). With 768, 1024, 1152 units (us): decode, 32/8 heads, 40
// ragged dialogues up to 4000 keys 61.4, 60.4, 68.6; 64 ragged up to 4000
// 107, 103, 119; 64 x 4000 169, 165, 175; 100 x 8192 (800 units whole) 611,
// 561, 606. Partials of 17 columns and more weigh more (8 rows, 32/8 heads, 8 x
// 3000 29.5, 31.9, 32.1; decode, 32/1 heads, 16 x 8192 26.5, 29.3, -), so those
// take 768 while dialogues need cutting, and so do calls of few slabs, whose
// chunks are short (12 x 4000, 16/4 heads 22.9, 24.1; 20 ragged up to 5000, d 64
// 24.4, 25.8; but 24 ragged up to 6000, 32/8 67.1, 65.1). A call that fills the chip with whole
// dialogues has an eighth of them and 256 more for the long ones. Row-tiled
// launches, whose partials weigh most, cut for 448 units (two to a CU).
constexpr int kSplitUnits = 1024, kSplitUnitsFew = 768, kSplitUnits128 = 448;
// From this many (dialogue, KV head, column group) workgroups on, a one-wave
// launch keeps every dialogue whole and needs no plan, whose scans over many
// dialogues every workgroup would repeat. Measured with the plan and without
// (us): decode, 32/8 heads, 256 x 1000 keys 175, 170; 1000 x 300 276, 204; 2000
// ragged up to 500 682, 355; 64/8 heads, d 64, 256 x 300 34.6, 28.1; 8 drafted
// rows, 32/8 heads, 256 ragged up to 1000 136, 123; 500 x 300 150, 125. One wave
// then streams a dialogue's keys at 45 per us, which decides the call when one
// dialogue is many times the mean, and for drafted rows the forward kernel's
// four waves, which served them before, had 63: one of 32000 keys among 255 of
// 300 119 planned, 705 whole, 508 before. Prefills whose cache has room for
// such a dialogue (90 us and more) therefore keep the plan up to the 256
// dialogues that it holds in registers.
constexpr int kSplitDirect = 2048, kSplitDirectKeys = 4096;
inline SplitPlan split_plan(SplitKind kind, int32_t batch, int64_t total_rows, int32_t max_rows,
                            int32_t hq, int32_t hkv, int32_t d, int64_t max_len, int32_t fixed,
                            bool limited, size_t ws_bytes) {
  SplitPlan p{};
  const int64_t cols = (int64_t)max_rows * (hq / hkv);
  const bool one_wave = kind == kOneWave || kind == kDecodeStep;
  p.colw = one_wave ? 32 : 128;
  p.tile_shift = one_wave ? 5 : 6;
  p.min_tiles = 4;
  p.whole_tiles = one_wave ? 0 : 8;
  p.col_groups = (int32_t)((cols + p.colw - 1) / p.colw);
  p.col_stride = (int32_t)(cols < p.colw ? cols : p.colw);
  const int64_t tiles = (max_len + (1 << p.tile_shift) - 1) >> p.tile_shift;
  const int64_t most = fixed > 0 ? fixed : (tiles + p.min_tiles - 1) / p.min_tiles;
  p.max_splits = (int32_t)(most < 1 ? 1 : fixed <= 0 && most > 64 ? 64 : most);
  if (one_wave && fixed <= 0 && (int64_t)batch * hkv * p.col_groups >= kSplitDirect &&
      (kind == kDecodeStep || batch > 256 || max_len <= kSplitDirectKeys))
    p.max_splits = 1;
  // column groups of all dialogues together, partials of one unit over all
  // KV heads
  const int64_t by_rows = total_rows * (hq / hkv) / p.colw + batch, groups = p.col_groups;
  const int64_t all_groups = by_rows < (int64_t)batch * groups ? by_rows : (int64_t)batch * groups;
  const int64_t per = (int64_t)hkv * p.col_stride * (d + 2) * 4;
  const int64_t whole = all_groups * hkv;  // units if no dialogue is cut
  const bool few = whole <= 160 || (p.col_stride > 16 && whole <= 512);
  int64_t target = few ? kSplitUnitsFew : kSplitUnits;
  if (whole >= target) target = whole + whole / 8 + 256;
  // (row-tiled: the units aimed at, to which rounding up adds one per group)
  p.budget = (int32_t)(one_wave ? target / hkv : (kSplitUnits128 + hkv - 1) / hkv);
  const int64_t bound = one_wave ? p.budget : p.budget + all_groups;
  int64_t units = all_groups * p.max_splits;
  if (fixed <= 0 && units > bound) units = bound;
  else if (one_wave) p.budget = 0;
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
      p.budget = (int32_t)fit;
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
