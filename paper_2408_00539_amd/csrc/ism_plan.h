// Device plan of a split-key launch (ism_split.hip): how the dialogues' key
// ranges are cut into units. Every workgroup derives the same plan from the
// length arrays: lane l of a wave holds dialogue l (and l + 64, ... in turn),
// and two wave scans on DPP lane moves find its unit.
#pragma once

#include "ism_common.h"
#include "ism_kernels.h"

namespace ism {

typedef int32_t i32x2 __attribute__((ext_vector_type(2)));

// A dialogue's extent. For an out-of-contract length (oob) the new rows that
// fall inside the cache are appended all the same, and the outputs become
// NaN.
struct Extent {
  int r0, rows;  // its rows of q / o
  int cached;    // key t >= cached is new row t - cached
  int keys;      // keys that some row sees, at most the cache's capacity
  bool oob;      // the cache cannot hold the new rows
};

__device__ __forceinline__ Extent extent_from(const SplitArgs &a, int r0, int rows, int cached) {
  Extent x;
  x.r0 = r0;
  x.rows = min(max(rows, 0), a.max_rows);
  x.cached = cached;
  const int64_t end = (int64_t)cached + x.rows;
  x.oob = cached < 0 || end > a.cap;
  x.keys = (int)min(max(end, (int64_t)1), (int64_t)a.cap);
  if (end <= 0) x.cached = 1;
  return x;
}

// The length arrays' entries of dialogue b.
struct RawLen {
  int r0, rows, cached;
};
__device__ __forceinline__ RawLen raw_len(const SplitArgs &a, int b) {
  RawLen r{b, 1, a.cache_len[b]};
  if (a.cu_new) {
    r.r0 = a.cu_new[b];
    r.rows = a.cu_new[b + 1] - r.r0;
  }
  return r;
}

__device__ __forceinline__ int tiles_of(const SplitArgs &a, const Extent &x) {
  return x.rows > 0 ? ((x.keys - 1) >> a.tile_shift) + 1 : 0;
}

// Column groups (workgroups per chunk and KV head) of `rows` new rows.
__device__ __forceinline__ int groups_of(const SplitArgs &a, int rows) {
  return min((int)(((int64_t)rows * a.group + a.colw - 1) >> (a.colw == 32 ? 5 : 7)), a.col_groups);
}

// a / b (a >= 0, b >= 1) through the hardware reciprocal, exact: the first
// estimate is at most a >> 21 (or one) off, so that what remains over b is
// below 2^22 and the second is at most one off. (The plan is a serial chain at
// the start of every workgroup; an integer division is 40 instructions.)
__device__ __forceinline__ int quot(int a, int b) {
  const float inv = __builtin_amdgcn_rcpf((float)b);
  int q = (int)((float)a * inv);
  q += (int)((float)(a - q * b) * inv);
  const int r = a - q * b;
  return q + (r >= b ? 1 : r < 0 ? -1 : 0);
}

// Tiles per chunk of a dialogue of t tiles, when chunks hold at most lc tiles
// (or fixed_splits is set) and the chunks are as equal as whole tiles allow;
// up to whole_tiles tiles are one chunk.
__device__ __forceinline__ int chunk_len(const SplitArgs &a, int t, int lc) {
  if (t <= a.whole_tiles) return max(t, 1);
  const int n = min(a.fixed_splits ? a.fixed_splits : quot(t + lc - 1, lc), a.max_splits);
  return n <= 1 ? max(t, 1) : quot(t + n - 1, n);
}
// Chunks of that length (none is empty; 0 for a dialogue without new rows).
__device__ __forceinline__ int chunks_of(const SplitArgs &a, int t, int lc) {
  const int per = chunk_len(a, t, lc);
  return quot(t + per - 1, per);
}

// Inclusive sum over the wave's lanes: row shifts, then row broadcasts.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_or_zero(int x) {
  return __builtin_amdgcn_update_dpp(0, x, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ int wave_scan(int x) {
  x += dpp_or_zero<0x111, 0xf>(x);  // row_shr 1
  x += dpp_or_zero<0x112, 0xf>(x);  // row_shr 2
  x += dpp_or_zero<0x114, 0xf>(x);  // row_shr 4
  x += dpp_or_zero<0x118, 0xf>(x);  // row_shr 8
  x += dpp_or_zero<0x142, 0xa>(x);  // row_bcast 15
  x += dpp_or_zero<0x143, 0xc>(x);  // row_bcast 31
  return x;
}
__device__ __forceinline__ float wave_total(float x) {
  auto f = [](int i) { return __builtin_bit_cast(float, i); };
  auto i = [](float v) { return __builtin_bit_cast(int, v); };
  x += f(dpp_or_zero<0x111, 0xf>(i(x)));
  x += f(dpp_or_zero<0x112, 0xf>(i(x)));
  x += f(dpp_or_zero<0x114, 0xf>(i(x)));
  x += f(dpp_or_zero<0x118, 0xf>(i(x)));
  x += f(dpp_or_zero<0x142, 0xa>(i(x)));
  x += f(dpp_or_zero<0x143, 0xc>(i(x)));
  return f(__builtin_amdgcn_readlane(i(x), 63));
}

// One workgroup's work: chunk `split` of the n chunks of dialogue b, column
// group cg of KV head kvh, and its slot among the partials.
struct Unit {
  int b, split, n, kvh, cg, slot;
  int tile0, tiles;  // the chunk
  Extent x;
};

// Dialogue b's lengths, tiles and column groups (none past the batch).
struct Entry {
  RawLen r;
  int t, g;
};
__device__ __forceinline__ Entry load_entry(const SplitArgs &a, int b) {
  Entry x;
  x.r = raw_len(a, min(b, a.batch - 1));
  const Extent e = extent_from(a, x.r.r0, x.r.rows, x.r.cached);
  x.t = b < a.batch ? tiles_of(a, e) : 0;
  x.g = b < a.batch ? groups_of(a, e.rows) : 0;
  return x;
}
// Up to 64 kWaves dialogues are held in registers, `lane`, `lane` + 64, ...
constexpr int kWaves = 4;
__device__ __forceinline__ int units_of(const SplitArgs &a, const Entry &x, int lc) {
  return chunks_of(a, x.t, lc) * x.g;
}

// Tiles per chunk at most: a length for which the chunks of all dialogues,
// sum n_b groups_b, are at most the grid's units per KV head, which the host
// bounds: `budget`, or budget + sum groups_b for the row-tiled kernel (one
// chunk per dialogue always fits; the same sums in every workgroup). A
// one-wave launch with its dialogues in registers counts the chunks of each
// length tried: first the one that fills the budget if every dialogue's last
// chunk is half full (equal dialogues then get as many chunks as the budget
// holds), then lengths that make room for what rounding up did add. Others
// take the length whose bound, sum t_b groups_b / lc + sum groups_b, fits.
__device__ __forceinline__ int chunk_limit(const SplitArgs &a, int lane, const Entry (&w)[kWaves]) {
  constexpr int kLongest = 1 << 26;  // tiles: any dialogue is one chunk
  float sum = (float)w[0].t * (float)w[0].g, groups = (float)w[0].g;
  if (a.batch > 64)
#pragma unroll
    for (int i = 1; i < kWaves; ++i) {
      sum += (float)w[i].t * (float)w[i].g;
      groups += (float)w[i].g;
    }
  for (int b0 = 64 * kWaves; b0 < a.batch; b0 += 64) {
    const Entry x = load_entry(a, b0 + lane);
    sum += (float)x.t * (float)x.g;
    groups += (float)x.g;
  }
  sum = wave_total(sum);
  groups = wave_total(groups);
  const float budget = (float)a.budget;
  const bool count = a.colw == 32 && a.batch <= 64 * kWaves;
  float units = a.colw != 32 ? budget : budget - (count ? 0.5f : 1.f) * groups;
  for (int lc = 0;;) {
    // sum / units, rounded up
    const float l = units >= 1.f ? sum * __builtin_amdgcn_rcpf(units) * 1.0001f : 1e9f;
    const int next = __builtin_amdgcn_readfirstlane((int)fminf(l, (float)kLongest) + 1);
    lc = max(max(next, a.min_tiles), lc ? lc + (lc >> 4) + 1 : 0);
    if (!count) return lc;
    auto most = [&](const Entry &x) __attribute__((always_inline)) {
      return min(quot(x.t + lc - 1, lc), a.max_splits) * x.g;
    };
    int c = most(w[0]);
    if (a.batch > 64)
#pragma unroll
      for (int i = 1; i < kWaves; ++i) c += most(w[i]);
    c = __builtin_amdgcn_readlane(wave_scan(c), 63);
    if (c <= a.budget || lc > kLongest) return lc;
    units = budget - ((float)c - sum * __builtin_amdgcn_rcpf((float)lc));
  }
}

// The unit of workgroup `bid` (false: none). Workgroups go round-robin to the
// 8 XCDs, so XCD x takes a contiguous eighth of the units and the column
// groups that read the same chunk share its L2.
__device__ __forceinline__ bool find_unit(const SplitArgs &a, int bid, int lane, Unit &u) {
  if (a.max_splits == 1 && a.colw == 32) {
    // One chunk per dialogue and the same column groups in each (a one-wave
    // launch has several only with one row per dialogue): no plan is needed.
    const int units = a.batch * a.col_groups * a.hkv, per_xcd = (units + 7) >> 3;
    const int i = bid >> 3, flat = (bid & 7) * per_xcd + i;
    if (i >= per_xcd || flat >= units) return false;
    u.b = __builtin_amdgcn_readfirstlane(quot(flat, a.col_groups * a.hkv));
    const int k = flat - u.b * a.col_groups * a.hkv;
    u.kvh = __builtin_amdgcn_readfirstlane(quot(k, a.col_groups));
    u.cg = k - u.kvh * a.col_groups;
    const RawLen r = raw_len(a, u.b);
    u.x = extent_from(a, r.r0, r.rows, r.cached);
    u.x.keys = __builtin_amdgcn_readfirstlane(u.x.keys);
    u.split = u.tile0 = 0;
    u.n = 1;
    u.slot = flat;
    u.tiles = __builtin_amdgcn_readfirstlane(tiles_of(a, u.x));
    return u.tiles > 0;
  }
  Entry w[kWaves] = {load_entry(a, lane)};
  if (a.batch > 64)
#pragma unroll
    for (int i = 1; i < kWaves; ++i) w[i] = load_entry(a, 64 * i + lane);
  const int lc = a.fixed_splits || a.max_splits == 1 ? 1
                 : a.budget                          ? chunk_limit(a, lane, w)
                                                     : a.min_tiles;
  // the units of all dialogues (per KV head), then this workgroup's among
  // them: by wave of 64 dialogues, then one scan
  int cnt[kWaves], inc[kWaves], all = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i)
    if (i == 0 || a.batch > 64) {
      cnt[i] = units_of(a, w[i], lc);
      inc[i] = wave_scan(cnt[i]);
      all += __builtin_amdgcn_readlane(inc[i], 63);
    }
  for (int b0 = 64 * kWaves; b0 < a.batch; b0 += 64)
    all += __builtin_amdgcn_readlane(wave_scan(units_of(a, load_entry(a, b0 + lane), lc)), 63);
  // (never more than the host made room for, whatever the length arrays say)
  const int units = min(all, a.max_units) * a.hkv, per_xcd = (units + 7) >> 3;
  const int i = bid >> 3, flat = (bid & 7) * per_xcd + i;
  if (i >= per_xcd || flat >= units) return false;
  int base = 0, b0 = 0, n = cnt[0], up = inc[0];
  Entry e = w[0];
  if (a.batch > 64) {
#pragma unroll
    for (int j = 1; j < kWaves; ++j) {
      const int next = base + __builtin_amdgcn_readlane(up, 63);
      if (b0 == 64 * (j - 1) && flat >= next * a.hkv && 64 * j < a.batch) {
        base = next;
        b0 = 64 * j;
        n = cnt[j];
        up = inc[j];
        e = w[j];
      }
    }
    for (int b = 64 * kWaves; b < a.batch; b += 64) {
      const int next = base + __builtin_amdgcn_readlane(up, 63);
      if (b0 != b - 64 || flat < next * a.hkv) break;
      base = next;
      b0 = b;
      e = load_entry(a, b + lane);
      n = units_of(a, e, lc);
      up = wave_scan(n);
    }
  }
  const int src = __builtin_ctzll(__builtin_amdgcn_ballot_w64((base + up) * a.hkv > flat));
  const int first = base + __builtin_amdgcn_readlane(up - n, src);
  const int gs = __builtin_amdgcn_readlane(e.g, src);
  u.b = __builtin_amdgcn_readfirstlane(b0 + src);
  u.n = __builtin_amdgcn_readfirstlane(quot(__builtin_amdgcn_readlane(n, src), gs));
  const int j = flat - first * a.hkv;  // chunk-major, then KV head, column group
  u.split = __builtin_amdgcn_readfirstlane(quot(j, gs * a.hkv));
  const int k = j - u.split * gs * a.hkv;
  u.kvh = __builtin_amdgcn_readfirstlane(quot(k, gs));
  u.cg = k - u.kvh * gs;
  u.slot = flat;
  u.x = extent_from(a, __builtin_amdgcn_readlane(e.r.r0, src),
                    __builtin_amdgcn_readlane(e.r.rows, src),
                    __builtin_amdgcn_readlane(e.r.cached, src));
  u.x.keys = __builtin_amdgcn_readfirstlane(u.x.keys);  // (formed with vector instructions)
  const int t_all = __builtin_amdgcn_readlane(e.t, src);
  const int per = __builtin_amdgcn_readfirstlane(chunk_len(a, t_all, lc));
  u.tile0 = u.split * per;
  u.tiles = min(per, t_all - u.tile0);
  // the combine reads the dialogue's chunks and first slot here
  if (j == 0 && a.plan && lane == 0) *(i32x2 *)(a.plan + 2 * u.b) = i32x2{u.n, first * a.hkv};
  return true;
}

}  // namespace ism
