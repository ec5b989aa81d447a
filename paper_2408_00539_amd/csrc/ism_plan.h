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

// a / b (a >= 0, b >= 1) through the hardware reciprocal: exact for
// a < 2^22, where the estimate is at most one off, else the long division.
// (The plan is a serial chain at the start of every workgroup.)
__device__ __forceinline__ int quot(int a, int b) {
  if (a >= 1 << 22) return a / b;
  int q = (int)((float)a * __builtin_amdgcn_rcpf((float)b));
  const int r = a - q * b;
  q += r >= b ? 1 : r < 0 ? -1 : 0;
  return q;
}

// Tiles per chunk of a dialogue of t tiles, when chunks hold at most lc tiles
// (or fixed_splits is set) and the chunks are as equal as whole tiles allow.
__device__ __forceinline__ int chunk_len(const SplitArgs &a, int t, int lc) {
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

// The unit of workgroup `bid` (false: none). Chunk length: at least min_tiles,
// and such that sum n_b groups_b <= budget + sum groups_b, which bounds the
// grid on the host (the sum in fp32 and rounded up, the same in every
// workgroup). Workgroups go round-robin to the 8 XCDs, so XCD x takes a
// contiguous eighth of the units and the column groups that read the same
// chunk share its L2.
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
  RawLen r{0, 0, 0};  // dialogue `lane` (kept: most batches fit one wave)
  int t = 0, g = 0;
  auto load = [&](int b) __attribute__((always_inline)) {
    t = 0;
    g = 0;
    if (b < a.batch) {
      r = raw_len(a, b);
      const Extent x = extent_from(a, r.r0, r.rows, r.cached);
      t = tiles_of(a, x);
      g = groups_of(a, x.rows);
    }
  };
  load(lane);
  int lc = 1;
  if (!a.fixed_splits && a.max_splits > 1) {
    float sum = (float)t * (float)g;
    if (a.batch > 64) {
      for (int b0 = 64; b0 < a.batch; b0 += 64) {
        load(b0 + lane);
        sum += (float)t * (float)g;
      }
      load(lane);
    }
    const float per = wave_total(sum) * a.inv_budget;
    lc = __builtin_amdgcn_readfirstlane(max((int)fminf(per, 1e9f) + 1, a.min_tiles));
  }
  // the units of all dialogues (per KV head), then this workgroup's among
  // them: one scan when the batch fits one wave
  int cnt = chunks_of(a, t, lc) * g, inc = wave_scan(cnt);
  int all = __builtin_amdgcn_readlane(inc, 63);
  for (int b0 = 64; b0 < a.batch; b0 += 64) {
    load(b0 + lane);
    all += __builtin_amdgcn_readlane(wave_scan(chunks_of(a, t, lc) * g), 63);
  }
  // (never more than the host made room for, whatever the length arrays say)
  const int units = min(all, a.max_units) * a.hkv, per_xcd = (units + 7) >> 3;
  const int i = bid >> 3, flat = (bid & 7) * per_xcd + i;
  if (i >= per_xcd || flat >= units) return false;
  int base = 0, b0 = 0;
  if (a.batch > 64) {  // the wave of dialogues that holds it
    for (;; b0 += 64) {
      load(b0 + lane);
      cnt = chunks_of(a, t, lc) * g;
      inc = wave_scan(cnt);
      const int here = __builtin_amdgcn_readlane(inc, 63);
      if (flat < (base + here) * a.hkv || b0 + 64 >= a.batch) break;
      base += here;
    }
  }
  const int src = __builtin_ctzll(__builtin_amdgcn_ballot_w64((base + inc) * a.hkv > flat));
  const int first = base + __builtin_amdgcn_readlane(inc - cnt, src);
  const int gs = __builtin_amdgcn_readlane(g, src);
  u.b = __builtin_amdgcn_readfirstlane(b0 + src);
  u.n = __builtin_amdgcn_readfirstlane(quot(__builtin_amdgcn_readlane(cnt, src), gs));
  const int j = flat - first * a.hkv;  // chunk-major, then KV head, column group
  u.split = __builtin_amdgcn_readfirstlane(quot(j, gs * a.hkv));
  const int k = j - u.split * gs * a.hkv;
  u.kvh = __builtin_amdgcn_readfirstlane(quot(k, gs));
  u.cg = k - u.kvh * gs;
  u.slot = flat;
  u.x = extent_from(a, __builtin_amdgcn_readlane(r.r0, src), __builtin_amdgcn_readlane(r.rows, src),
                    __builtin_amdgcn_readlane(r.cached, src));
  u.x.keys = __builtin_amdgcn_readfirstlane(u.x.keys);  // (formed with vector instructions)
  const int t_all = __builtin_amdgcn_readlane(t, src);
  const int per = __builtin_amdgcn_readfirstlane(chunk_len(a, t_all, lc));
  u.tile0 = u.split * per;
  u.tiles = min(per, t_all - u.tile0);
  // the combine reads the dialogue's chunks and first slot here
  if (j == 0 && a.plan && lane == 0) *(i32x2 *)(a.plan + 2 * u.b) = i32x2{u.n, first * a.hkv};
  return true;
}

}  // namespace ism
