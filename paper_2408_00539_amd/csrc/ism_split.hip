// Attention of a few new rows per dialogue over its KV cache, with the key
// range split over workgroups: answer-token decode steps and short drafted
// answer chunks or query segments (Sec. 2.3 of the paper; Eq. 5 through the
// cache).
//
// The calls are HBM streams: the cache is read once for at most 32 columns (per 32,
// for a decode step with more query heads per KV head).
//  * columns: the (row, query head) pairs of a dialogue that share a KV head
//    are the columns of S^T = K Q^T, row-major (head innermost), 32 to a
//    one-wave workgroup. 8 drafted rows with 4 query heads per KV head fill it
//    exactly (the row-tiled forward kernel spends four half-empty waves on
//    them); a decode step with fewer columns leaves the others unused.
//  * units (ism_plan.h): a dialogue's keys are cut into chunks of whole 32-key
//    tiles at about the same length in every dialogue, so that ragged
//    dialogues load the chip evenly; equal chunk counts per dialogue left the
//    longest dialogue's chunks running alone (a step of 40 dialogues of 200 to
//    4000 keys, 32 / 8 heads, pages of 64: 79.6 us, now 66.4; 24 dialogues of
//    1500 to 6000 keys, 8 drafted rows, pages of 256: 117.4 us in the forward
//    kernel, now 82.7; d = 64, 64 / 8 heads, 40 dialogues of 400 to 9000 keys
//    104 us, now 67; equal dialogues were and are at the same rate).
//  * a dialogue cut into one chunk writes its output directly; otherwise
//    each unit writes unnormalised fp32 partials (m, l, o), merged exactly by
//    split_combine_kernel.
// A wave streams its chunk through a ring of two K/V tiles in LDS (direct
// global->LDS transfers; at d = 128 a third stage measured the same at the
// same number of workgroups and leaves room for fewer). How many units a call
// is cut into: ism_split_plan.h.
// The new rows' keys and values are read from the input, and the unit whose
// tile holds them stores them into the cache, so that no append launch runs
// first (the rotating append of 2-D positions does).
#include "ism_common.h"
#include "ism_kernels.h"
#include "ism_plan.h"

namespace ism {

namespace {

constexpr int kT = 32;  // keys per tile
constexpr int R = 2;    // ring of K/V tiles
template <int D>
struct SplitSmem {
  bf16_t kv[R][2][kT * D];
};

template <int D, bool PAGED>
__global__ void __launch_bounds__(64)
split_attn_kernel(SplitArgs a) {
  constexpr int NKS = D / 16, NDB = D / 32, RB = 2 * D, CPR = D / 8, LA = 4;
  using Dma = DmaTile<D, kT, 1, true>;  // the cache is read once
  constexpr int NI = Dma::NI;           // transfers per tile and tensor
  __shared__ __attribute__((aligned(1024))) SplitSmem<D> sm;

  const int lane = threadIdx.x, l32 = lane & 31, hf = lane >> 5;
  Unit u;
  if (!find_unit(a, (int)blockIdx.x, lane, u)) return;
  const Extent x = u.x;
  const int b = u.b, kvh = u.kvh;
  const int ncol = x.rows * a.group, col0 = u.cg * 32;
  const int tile0 = u.tile0, nt = u.tiles;
  // keys [0, from_cache) come from the cache, later ones from the input
  const int from_cache = a.append ? min(x.cached, x.keys) : x.keys;

  // this lane's column: row `row` of the dialogue, query head `head`
  const int idc = min(col0 + l32, ncol - 1);
  const int row = idc / a.group, head = kvh * a.group + (idc - row * a.group);
  const int last =
      a.causal ? (int)min((int64_t)x.cached + row, (int64_t)x.keys - 1) : x.keys - 1;
  // keys below it are seen by every row
  const int unmasked = a.causal ? min(x.cached, x.keys - 1) + 1 : x.keys;
  const float sl2 = a.scale * kLog2e;

  const int64_t slab = ((int64_t)b * a.hkv + kvh) * a.cap * D;
  auto tile_row = [&](int c) -> int64_t {  // element offset of key c's row (c % 32 == 0)
    if (PAGED)
      return paged_offset_uniform(a.block_table, a.max_pages, a.num_pages, a.page_size, a.hkv,
                                  D, b, kvh, c);
    return slab + (int64_t)c * D;
  };
  Dma dma;
  dma.init(lane, D);
  auto issue = [&](int t, int st) __attribute__((always_inline)) {
    const int c = __builtin_amdgcn_readfirstlane((tile0 + t) * kT);
    const int64_t off = tile_row(c);
    const bf16_t *ks = (const bf16_t *)a.k_cache + off, *vs = (const bf16_t *)a.v_cache + off;
    if (c + kT <= from_cache) {
      dma.issue(ks, D, kT, sm.kv[st][0]);
      dma.issue(vs, D, kT, sm.kv[st][1]);
    } else {  // the last tiles: rows of the input, and repeats of the last key
      const uint32_t lk = lds_addr(sm.kv[st][0]), lv = lds_addr(sm.kv[st][1]);
#pragma unroll
      for (int j = 0; j < NI; ++j) {
        const int r = j * Dma::RPI + lane / CPR;
        const int key = min(c + r, x.keys - 1);
        const bool isnew = key >= from_cache;
        const int64_t o = (isnew ? ((int64_t)(x.r0 + key - x.cached) * a.hkv + kvh) * D
                                 : (int64_t)(key - c) * D) +
                          ((lane % CPR) ^ swz<D>(r)) * 8;
        dma_x4((isnew ? (const bf16_t *)a.k_new : ks) + o, lk + j * 1024);
        dma_x4((isnew ? (const bf16_t *)a.v_new : vs) + o, lv + j * 1024);
      }
    }
  };
  // the first tiles' transfers start before the queries arrive
#pragma unroll
  for (int t = 0; t < R - 1; ++t)
    if (t < nt) issue(t, t);
  bf16x8 qf[NKS];
  {
    const bf16_t *qp = (const bf16_t *)a.q + ((int64_t)(x.r0 + row) * a.hq + head) * D + hf * 8;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qf[ks] = *(const bf16x8 *)(qp + ks * 16);
  }
  if (a.rope_pos1)
    rope_queries<D>(qf, hf, a.rope_pos1[x.r0 + row], a.rope_pos2[x.r0 + row], a.rope_log2_base);
  wait_loads();  // the queries (and, in order before them, the first tile)
  SwzBases<D> so;
  so.init(lane);

  f32x16 oacc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db) oacc[db] = f32x16{};
  float m_run = -INFINITY, l_run = 0.f;
  const float tau = 8.f / sl2;  // lazy rescale threshold: 2^8 in probability units
  for (int t = 0; t < nt; ++t) {
    const int c0 = (tile0 + t) * kT, st = t % R;
    // Tile t + R - 1 goes into the stage of tile t - 1 (its products consumed
    // the reads); then wait for tile t only. (Near the end of the chunk, where
    // fewer tiles are in flight and stores into the cache are in the queue,
    // which is counted in order, everything is waited for.)
    const bool more = t + R - 1 < nt;
    if (more) issue(t + R - 1, (t + R - 1) % R);
    if (more && c0 + kT <= from_cache) wait_vmem_but<(R - 1) * 2 * NI>();
    else wait_vmem();
    const bf16_t *kt = sm.kv[st][0], *vt = sm.kv[st][1];
    if (a.append && u.cg == 0 && c0 + kT > from_cache) {  // store the tile's new rows
      const int64_t off = tile_row(c0);
      for (int e = lane; e < kT * CPR; e += 64) {
        const int r = e / CPR, ch = e % CPR;
        if (c0 + r >= from_cache && c0 + r < x.keys) {
          const int s = r * D + ((ch ^ swz<D>(r)) << 3);
          *(u32x4 *)((bf16_t *)a.k_cache + off + r * D + ch * 8) = *(const u32x4 *)(kt + s);
          *(u32x4 *)((bf16_t *)a.v_cache + off + r * D + ch * 8) = *(const u32x4 *)(vt + s);
        }
      }
    }
    // Operand addresses: a tile's base is a multiple of its size, so the
    // swizzle's XOR applies to base + row offset. (The empty asm keeps the 16
    // XORed addresses from being kept in registers across the loop.)
    uint32_t ka = lds_addr(kt) + so.rowb, va0 = lds_addr(vt) + so.trb[0],
             va1 = lds_addr(vt) + so.trb[1];
    asm volatile("" : "+v"(ka), "+v"(va0), "+v"(va1));
    // S^T = K Q^T, the softmax of the tile, O^T += V^T P^T: every product's LDS
    // operand is read LA products ahead, the first V operands before the
    // softmax (left to itself the compiler waits for each read in turn)
    f32x16 sc;
    bf16x8 pf[2];
    auto rd = [&](auto nc) __attribute__((always_inline)) -> bf16x8 {
      constexpr int n = decltype(nc)::value;
      if constexpr (n < NKS) {
        return lds_row_operand(ka ^ (uint32_t)(n << 5));
      } else {
        constexpr int bt = (n - NKS) / NDB, db = (n - NKS) % NDB;
        return lds_tr_operand<16 * bt * RB>(va0 ^ (uint32_t)(db << 6), va1 ^ (uint32_t)(db << 6));
      }
    };
    auto mm = [&](auto nc, bf16x8 o) __attribute__((always_inline)) {
      constexpr int n = decltype(nc)::value;
      if constexpr (n < NKS) {
        sc = mfma32x32x16(o, qf[n], n == 0 ? f32x16{} : sc);
      } else {
        constexpr int bt = (n - NKS) / NDB, db = (n - NKS) % NDB;
        oacc[db] = mfma32x32x16(o, pf[bt], oacc[db]);
      }
    };
    auto softmax = [&](auto nc) __attribute__((always_inline)) {
      if constexpr (decltype(nc)::value == NKS) {
        if (c0 + kT > unmasked) {
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (c0 + (r >> 2) * 8 + hf * 4 + (r & 3) > last) sc[r] = -INFINITY;
        }
        float mx[2] = {-INFINITY, -INFINITY};
#pragma unroll
        for (int r = 0; r < 16; r += 4) {
          mx[0] = vmax(mx[0], vmax(sc[r], sc[r + 1]));
          mx[1] = vmax(mx[1], vmax(sc[r + 2], sc[r + 3]));
        }
        const float mt = pair_max(vmax(mx[0], mx[1]));
        if (__builtin_amdgcn_ballot_w64(mt > m_run + tau) != 0) {
          const float mnew = vmax(m_run, mt);
          // a row that has seen no key yet (an answer row before its first
          // visible tile) keeps m = -inf, l = 0
          const float alpha = mnew == -INFINITY ? 1.f : fast_exp2((m_run - mnew) * sl2);
          m_run = mnew;
          l_run *= alpha;
#pragma unroll
          for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
        }
        const float moff = m_run == -INFINITY ? 0.f : m_run * sl2;
        float sum[2] = {0.f, 0.f};
#pragma unroll
        for (int bt = 0; bt < 2; ++bt) {
          u32x4 w;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            f32x2 pr;
            pr[0] = fast_exp2(fmaf(sc[8 * bt + 2 * v], sl2, -moff));
            pr[1] = fast_exp2(fmaf(sc[8 * bt + 2 * v + 1], sl2, -moff));
            sum[bt] += pr[0] + pr[1];
            w[v] = cvt_bf16x2(pr);
          }
          pf[bt] = __builtin_bit_cast(bf16x8, w);
        }
        l_run += sum[0] + sum[1];
      }
    };
    auto none = [](auto) __attribute__((always_inline)) {};
    product_slots<NKS + 2 * NDB, LA>(rd, mm, softmax, none);
  }

  const float lt = pair_sum(l_run);
  if (col0 + l32 >= ncol) return;
  if (u.n == 1) {
    const float inv = x.oob ? __builtin_nanf("") : 1.f / lt;
    const int64_t orow = x.r0 + row;
    bf16_t *op = (bf16_t *)a.o + (orow * a.hq + head) * D + hf * 4;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        u32x2 w;
        w[0] = pack_bf16x2(oacc[db][4 * j + 0] * inv, oacc[db][4 * j + 1] * inv);
        w[1] = pack_bf16x2(oacc[db][4 * j + 2] * inv, oacc[db][4 * j + 3] * inv);
        *(u32x2 *)(op + db * 32 + 8 * j) = w;
      }
    if (a.lse && hf == 0)
      a.lse[(int64_t)head * a.total_q + orow] =
          x.oob ? __builtin_nanf("") : m_run * a.scale + logf(lt);
    return;
  }
  // partials of this column (a row that sees no key of the chunk: m = -inf,
  // l = 0, o = 0)
  const int64_t pi = (int64_t)u.slot * a.col_stride + l32;
  float *po = a.part_o + pi * D + hf * 4;
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *(f32x4 *)(po + db * 32 + 8 * j) =
          f32x4{oacc[db][4 * j], oacc[db][4 * j + 1], oacc[db][4 * j + 2], oacc[db][4 * j + 3]};
  if (hf == 0) {
    a.part_ml[pi * 2] = m_run * sl2;
    a.part_ml[pi * 2 + 1] = lt;
  }
}

// Exact merge of a dialogue's chunk partials, one (row, head) per wave:
// M = max m_s, L = sum l_s 2^(m_s - M), O = sum o_s 2^(m_s - M) / L (scores
// in log2 units). Dialogues of one chunk were written by their unit. Bound by
// the latency of its dependent loads (plan, then m and l, then o), so up to
// 16 chunks' o are in flight at once.
template <int D>
__global__ void __launch_bounds__(256)
split_combine_kernel(SplitArgs a) {
  constexpr int E = D / 64, U = 16, F = 8;  // values per lane, chunks in flight
  typedef float vecE __attribute__((ext_vector_type(E)));
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = blockIdx.y;
  const i32x2 pl = *(const i32x2 *)(a.plan + 2 * b);
  const RawLen r = raw_len(a, b);
  const Extent x = extent_from(a, r.r0, r.rows, r.cached);
  const int ncol = x.rows * a.hq, n = pl[0], groups = groups_of(a, x.rows);
  if (ncol == 0 || n <= 1) return;
  // (out-of-contract row ranges can ask for more units than the host made room
  // for: the dialogues past it left no entry, and nothing is read for them)
  if (n > a.max_splits ||
      (uint32_t)pl[1] + (int64_t)n * a.hkv * groups > (int64_t)a.max_units * a.hkv)
    return;
  const int64_t step = (int64_t)a.hkv * groups * a.col_stride;  // between chunks
  for (int col = (int)blockIdx.x * 4 + wave; col < ncol; col += (int)gridDim.x * 4) {
    const int row = col / a.hq, head = col - row * a.hq, kvh = head / a.group;
    const int idx = row * a.group + (head - kvh * a.group);
    const int cg = idx >> (a.colw == 32 ? 5 : 7);
    const int64_t p0 =
        ((int64_t)pl[1] + kvh * groups + cg) * a.col_stride + (idx - cg * a.colw);
    float mx = -INFINITY, lt = 0.f, acc[E];
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = 0.f;
    if (n <= F) {  // every lane forms the weights itself: one round of loads
      f32x2 ml[F];
      vecE v[F];
#pragma unroll
      for (int s = 0; s < F; ++s) {
        ml[s] = s < n ? *(const f32x2 *)(a.part_ml + (p0 + s * step) * 2) : f32x2{-INFINITY, 0.f};
        v[s] = s < n ? *(const vecE *)(a.part_o + (p0 + s * step) * D + lane * E) : vecE{};
      }
#pragma unroll
      for (int s = 0; s < F; ++s) mx = fmaxf(mx, ml[s][0]);
      const float mref = mx == -INFINITY ? 0.f : mx;
#pragma unroll
      for (int s = 0; s < F; ++s) {
        const float w = fast_exp2(ml[s][0] - mref);
        lt = fmaf(ml[s][1], w, lt);
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e] = fmaf(v[s][e], w, acc[e]);
      }
    }
    for (int s0 = 0; s0 < n && n > F; s0 += 64) {
      // (more than 64 chunks: rescale what the earlier ones gave)
      const int nn = min(64, n - s0);
      f32x2 ml = f32x2{-INFINITY, 0.f};
      if (lane < nn) ml = *(const f32x2 *)(a.part_ml + (p0 + (s0 + lane) * step) * 2);
      float mn = fmaxf(mx, ml[0]);
#pragma unroll
      for (int s = 32; s >= 1; s >>= 1) mn = fmaxf(mn, __shfl_xor(mn, s));
      const float mref = mn == -INFINITY ? 0.f : mn;
      const float old = fast_exp2(mx - mref), w = fast_exp2(ml[0] - mref);
      mx = mn;
      lt = lt * old + ml[1] * w;
#pragma unroll
      for (int e = 0; e < E; ++e) acc[e] *= old;
      const float *po = a.part_o + (p0 + s0 * step) * D + lane * E;
      for (int s1 = 0; s1 < nn; s1 += U) {
        vecE v[U];
#pragma unroll
        for (int s = 0; s < U; ++s)
          v[s] = s1 + s < nn ? *(const vecE *)(po + (s1 + s) * step * D) : vecE{};
#pragma unroll
        for (int s = 0; s < U; ++s) {
          const float ws = __builtin_bit_cast(
              float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, w), (s1 + s) & 63));
#pragma unroll
          for (int e = 0; e < E; ++e) acc[e] = fmaf(v[s][e], ws, acc[e]);
        }
      }
    }
    if (n > F) {
#pragma unroll
      for (int s = 32; s >= 1; s >>= 1) lt += __shfl_xor(lt, s);
    }
    bf16_t *op = (bf16_t *)a.o + ((int64_t)(x.r0 + row) * a.hq + head) * D + lane * E;
    if (x.oob) lt = __builtin_nanf("");
    if constexpr (E == 2) *(uint32_t *)op = pack_bf16x2(acc[0] / lt, acc[1] / lt);
    else op[0] = (bf16_t)(acc[0] / lt);
    if (a.lse && lane == 0)
      a.lse[(int64_t)head * a.total_q + x.r0 + row] = (mx + log2f(lt)) * kLn2;
  }
}

template <int D, bool PAGED>
hipError_t launch_split_p(const SplitArgs &a, hipStream_t stream) {
  const dim3 grid((unsigned)(((int64_t)a.max_units * a.hkv + 7) / 8 * 8));
  hipLaunchKernelGGL((split_attn_kernel<D, PAGED>), grid, dim3(64), 0, stream, a);
  const hipError_t err = hipGetLastError();
  return err == hipSuccess && a.max_splits > 1 ? launch_split_combine(a, D, stream) : err;
}

}  // namespace

hipError_t launch_split_combine(const SplitArgs &a, int d, hipStream_t stream) {
  const int64_t wgs = ((int64_t)a.max_rows * a.hq + 3) / 4;
  const dim3 grid((unsigned)(wgs < 1024 ? wgs : 1024), a.batch);
  if (d == 128) hipLaunchKernelGGL(split_combine_kernel<128>, grid, dim3(256), 0, stream, a);
  else hipLaunchKernelGGL(split_combine_kernel<64>, grid, dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_split(const SplitArgs &a, int d, hipStream_t stream) {
  if (a.colw != 32 || 1 << a.tile_shift != kT) return hipErrorInvalidValue;
  if (d == 128) return a.block_table ? launch_split_p<128, true>(a, stream)
                                     : launch_split_p<128, false>(a, stream);
  if (d == 64) return a.block_table ? launch_split_p<64, true>(a, stream)
                                    : launch_split_p<64, false>(a, stream);
  return hipErrorInvalidValue;
}

}  // namespace ism
