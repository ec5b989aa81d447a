// Forward ISM attention on gfx950: per-token visibility bounds (Eq. 5) and a
// flash-style online-softmax kernel on bf16 MFMA 32x32x16 with fp32
// accumulation. The same kernel serves the cached prefill of a new query
// segment (Sec. 2.3), where every key of the concatenated cache is visible.
//
// Work decomposition. The (row, query head) pairs of a dialogue and a set of
// query heads that share a KV head are the columns of S^T = K Q^T, row-major
// (head innermost). A workgroup of four waves owns 128 consecutive columns, 32
// to a wave, so that the K/V tile staged in LDS serves every head
// of the set, and a short segment fills whole waves (40 new rows with 4 heads
// per KV head are 5 waves, where 32-row blocks per head took 8: 40 dialogues
// of 2000 cached keys 119 -> 109 us). Each wave
// computes S^T for a 64-key tile (lane <-> column, so the softmax statistics
// of a row live in one lane pair), then O^T += V^T P^T.
//
// Mask handling. lim(j) is non-decreasing inside a dialogue, so a wave's
// bounds are lim(first row) and lim(last row): key tiles past lim(last row)
// are never visited, tiles ending at or before lim(first row) run with no
// mask instructions, and only the remaining tiles compare key <= lim(row)
// in registers. No N x N mask exists anywhere.
#include "ism_common.h"
#include "ism_kernels.h"
#include "ism_plan.h"

namespace ism {

// lim[j] = inclusive last visible key of token j (Eq. 5, 0-indexed):
// end-1 of its segment for a query segment, j itself for an answer segment.
__global__ void __launch_bounds__(256)
prep_lim_kernel(const int32_t *__restrict__ cu_segs,
                const uint8_t *__restrict__ seg_is_query, int32_t num_segs,
                int32_t total, int32_t *__restrict__ lim) {
  const int j = blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= total) return;
  int lo = 0, hi = num_segs - 1;  // largest g with cu_segs[g] <= j
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (cu_segs[mid] <= j) lo = mid; else hi = mid - 1;
  }
  lim[j] = seg_is_query[lo] ? cu_segs[lo + 1] - 1 : j;
}

hipError_t launch_prep_lim(const int32_t *cu_segs, const uint8_t *seg_is_query,
                           int32_t num_segs, int32_t total, int32_t *lim,
                           hipStream_t stream) {
  if (total <= 0) return hipSuccess;
  hipLaunchKernelGGL(prep_lim_kernel, dim3((total + 255) / 256), dim3(256), 0,
                     stream, cu_segs, seg_is_query, num_segs, total, lim);
  return hipGetLastError();
}

namespace {

constexpr int kBN = 64;  // keys per tile
constexpr int kQW = 32;  // query rows per wave
// Four-wave workgroups, two (three at d = 64) to a CU, so that one's prologue
// and last steps run beside another's products. Eight-wave workgroups stage
// each K/V tile for twice the columns, half the transfers per product, but are
// alone on their CU. Four waves against eight (us): packed, 32/8 heads, 8 x 3000
// 560, 570; 4 x 9000 2243, 2257; 3 x 12000 2945, 2941; 2 x 16384 3625, 3614; but 4
// ragged up to 16384 5662, 6101; 6 up to 12000 3501, 3851; 16/4 heads, d 64, 2 x
// 16384 1095, 1143. Cached, 32/8 heads, new rows: 64 over 40 x 2000 keys 126, 135;
// 2048 over 4 x 16384 2096, 2086; 1000 over 4000 93, 115. (Eight would win where
// equal dialogues of 129 to 256 columns leave no second round: 40 over 40 x
// 2000 111, 103; 40 over 20 x 8000 206, 178.)
constexpr int NWV = 4;
// Capacity from which a paged cache's transfers are spread over a step's
// products like the dense cache's, instead of all starting with it. On long
// key loops the burst costs four-wave workgroups more than eight-wave ones
// paid (2048 new rows over 4 x 16384 keys, 32/8 heads, pages of 64 2468 us,
// spread 2320, eight waves 2312; pages of 256 2260, 2142, 2209; 40 over 20 x
// 8000, pages of 64 272, 235, 229); on short ones, where a tile's latency is
// hidden by little else, an early start wins (64 over 40 x 2000, pages of 64
// 133, spread 156).
constexpr int kSpreadKeys = 8192;

// Waves per SIMD, which bounds registers: d = 64 fits a third wave (4 x 8000
// tokens, 16 heads: 420 -> 398 us; not the paged cache, which would spill).
constexpr int fwd_occupancy(int d, bool paged) { return d == 64 && !paged ? 3 : 2; }

// K and V tiles of 64 keys, row-major, unpadded rows of D bf16 with the
// swz<D>() chunk swizzle, double-buffered; filled by direct global->LDS
// transfers. K is read as MFMA rows (ds_read_b128), V through transposing
// reads (ds_read_b64_tr_b16) as the V^T operand.
template <int D>
struct FwdSmem {
  bf16_t k[2][kBN * D];
  bf16_t v[2][kBN * D];
};

// S^T[key][row] = K Q^T for one 64-key tile: two 32-key blocks, D/16 steps.
template <int D>
__device__ __forceinline__ void tile_scores(const char *kl, const SwzOffsets<D> &so,
                                            const bf16x8 (&qf)[D / 16], f32x16 (&s)[2]) {
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
      const bf16x8 kf = *(const bf16x8 *)(kl + kb * 32 * D * 2 + so.rowk[ks]);
      s[kb] = mfma32x32x16(kf, qf[ks], ks == 0 ? f32x16{} : s[kb]);
    }
}

// Keys past the row's bound lim get score -inf.
__device__ __forceinline__ void tile_mask(f32x16 (&s)[2], int c0, int hf, int lim) {
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = c0 + kb * 32 + (r >> 2) * 8 + hf * 4 + (r & 3);
      if (key > lim) s[kb][r] = -INFINITY;
    }
}

// Row max of a tile, combined over the lane pair that holds the row.
__device__ __forceinline__ float tile_max(const f32x16 (&s)[2]) {
  float x[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int r = 0; r < 16; r += 2) x[r & 3] = vmax(x[r & 3], vmax(s[kb][r], s[kb][r + 1]));
  return pair_max(vmax(vmax(x[0], x[2]), vmax(x[1], x[3])));
}

// The reference max in log2 units. SPLIT: a row that has seen no key yet (an
// answer row whose keys end before the chunk) has m = -inf and keeps l = 0.
template <bool SPLIT>
__device__ __forceinline__ float log2_max(float m, float sl2) {
  return SPLIT && m == -INFINITY ? 0.f : m * sl2;
}

// Lazy online-softmax update: the reference max is only raised when a row's
// tile max exceeds it by more than tau (2^8 in probability units); exact
// either way since numerator and denominator share the reference max.
template <bool SPLIT, int NDB>
__device__ __forceinline__ void raise_max(float mt, float sl2, float tau, float &m_run,
                                          float &l_run, f32x16 (&oacc)[NDB]) {
  if (__builtin_amdgcn_ballot_w64(mt > m_run + tau) != 0) {
    const float mnew = vmax(m_run, mt);
    const float alpha = SPLIT && mnew == -INFINITY ? 1.f : fast_exp2((m_run - mnew) * sl2);
    m_run = mnew;
    l_run *= alpha;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
  }
}

// Probabilities 2^(s sl2 - moff) of one tile as bf16 B operands of the P V
// product, and their fp32 row sum.
__device__ __forceinline__ float tile_probs(const f32x16 (&s)[2], float sl2, float moff,
                                            bf16x8 (&pf)[2][2]) {
  float sum[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kb = 0; kb < 2; ++kb)
#pragma unroll
    for (int bt = 0; bt < 2; ++bt) {
      u32x4 w;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        f32x2 p;
        p[0] = fast_exp2(fmaf(s[kb][8 * bt + 2 * u], sl2, -moff));
        p[1] = fast_exp2(fmaf(s[kb][8 * bt + 2 * u + 1], sl2, -moff));
        sum[u] += p[0] + p[1];
        w[u] = cvt_bf16x2(p);
      }
      pf[kb][bt] = __builtin_bit_cast(bf16x8, w);
    }
  return (sum[0] + sum[1]) + (sum[2] + sum[3]);
}

// O^T[d][row] += V^T[d][key] P^T[key][row] for one 64-key tile.
template <int D>
__device__ __forceinline__ void tile_pv(const char *vl, const SwzOffsets<D> &so,
                                        const bf16x8 (&pf)[2][2], f32x16 (&oacc)[D / 32]) {
#pragma unroll
  for (int db = 0; db < D / 32; ++db) {
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int bt = 0; bt < 2; ++bt) {
        const uint32_t o = (kb * 32 + 16 * bt) * D * 2;
        const bf16x8 vf = tr_operand_at(vl, o + so.trk[db][0], o + so.trk[db][1]);
        oacc[db] = mfma32x32x16(vf, pf[kb][bt], oacc[db]);
      }
  }
}

// One pipelined step in a fixed instruction order: the D/8 products of
// S(t+1) = K(t+1) Q^T (its two 32-key blocks alternating), then the D/8
// products of O^T += V(t)^T P(t)^T (64-key chunks outermost), so that
// consecutive products always use different accumulators. Each product is
// followed by the LDS read of the operand LA = 2 products ahead (K rows, then
// transposed V; a third operand in flight measured ~1 % slower, one only
// ~7 % slower) and by its share of the vector work: during
// the S products the exponentials, row sums and bf16 packing of tile t,
// during the P V products the row max of S(t+1). The order is pinned with
// scheduling barriers so that the matrix core and the vector ALU of a wave
// are busy at the same time. Returns the fp32 row sum of P(t); mt receives
// the (unmasked) row max of S(t+1). With LAST (a wave's last tile) there is
// no S(t+1): the exponentials run alone, then the P V products.
// With PRIO the wave raises its issue priority for the first half (the S
// products and the exponentials, the vector-heavy half) and drops it for the
// P V products, so that of the two waves on a SIMD the one in its
// exponentials issues first and the other one's products fill the matrix
// core around it (about 2 % faster on the packed forward; steps whose
// transfers all start at the step start measured ~1 % slower with it).
template <int D, bool LAST, bool PRIO, class Hook>
__device__ __forceinline__ float step_block(const char *kl, const char *vl,
                                            const SwzOffsets<D> &so, const bf16x8 (&qf)[D / 16],
                                            const f32x16 (&cur)[2], f32x16 (&nxt)[2],
                                            f32x16 (&oacc)[D / 32], float sl2, float moff,
                                            float &mt, Hook &&hook) {
  constexpr int NKS = D / 16, NDB = D / 32;
  constexpr int NS = 2 * NKS, NP = 4 * NDB, N = NS + NP, LA = 2;
  constexpr int PPS = 16 / NS;  // probability pairs per S product
  constexpr int MPP = 32 / NP;  // max elements per P V product
  auto read = [&](int n) -> bf16x8 {
    if (n < NS) {
      const int kb = n & 1, ks = n >> 1;
      return *(const bf16x8 *)(kl + kb * 32 * D * 2 + so.rowk[ks]);
    }
    const int j = n - NS, kc = j / NDB, db = j % NDB;
    const uint32_t o = ((kc >> 1) * 32 + 16 * (kc & 1)) * D * 2;
    return tr_operand_at(vl, o + so.trk[db][0], o + so.trk[db][1]);
  };
  constexpr int F = LAST ? NS : 0;  // first product that runs
  bf16x8 op[N];
#pragma unroll
  for (int n = F; n < F + LA; ++n) op[n] = read(n);
  u32x4 w[2][2];
  float sum[2] = {0.f, 0.f}, mx[2] = {-INFINITY, -INFINITY};
#pragma unroll
  for (int n = 0; n < N; ++n) {
    if (PRIO && n == 0) __builtin_amdgcn_s_setprio(1);
    if (PRIO && n == NS) __builtin_amdgcn_s_setprio(0);
    if (n < NS) {
      if (!LAST) {
        const int kb = n & 1, ks = n >> 1;
        nxt[kb] = mfma32x32x16(op[n], qf[ks], ks == 0 ? f32x16{} : nxt[kb]);
      }
    } else {
      const int j = n - NS, kc = j / NDB, db = j % NDB;
      oacc[db] = mfma32x32x16(op[n], __builtin_bit_cast(bf16x8, w[kc >> 1][kc & 1]), oacc[db]);
    }
    hook(n);  // n is a constant once the loop is unrolled
    if (n >= F && n + LA < N) op[n + LA] = read(n + LA);
    if (n < NS) {
#pragma unroll
      for (int c = 0; c < PPS; ++c) {
        const int i = n * PPS + c, kb = i >> 3, bt = (i >> 2) & 1, u = i & 3;
        f32x2 p;
        p[0] = fast_exp2(fmaf(cur[kb][8 * bt + 2 * u], sl2, -moff));
        p[1] = fast_exp2(fmaf(cur[kb][8 * bt + 2 * u + 1], sl2, -moff));
        sum[i & 1] += p[0] + p[1];
        w[kb][bt][u] = cvt_bf16x2(p);
        asm volatile("" : "+v"(sum[i & 1]));  // keep the add in this slot
      }
    } else if (!LAST) {
#pragma unroll
      for (int c = 0; c < MPP; c += 2) {
        const int e = (n - NS) * MPP + c, m = (e >> 1) & 1;
        mx[m] = vmax(mx[m], vmax(nxt[e >> 4][e & 15], nxt[e >> 4][(e & 15) + 1]));
        asm volatile("" : "+v"(mx[m]));
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  mt = LAST ? -INFINITY : pair_max(vmax(mx[0], mx[1]));
  return sum[0] + sum[1];
}

// NT: non-temporal tile transfers, for a cache-mode launch in which every
// (dialogue, head set) group has a single row tile, so that no other
// workgroup reads its K/V (verifying 8 drafted tokens per dialogue through
// the cache ran 11 % faster; with several row tiles per group the same bit
// cost the L2 sharing between them: the workload-3 prefill ran 22 % slower).
template <int D, bool CACHE, bool PAGED, bool NT, bool SPLIT>
__global__ void __launch_bounds__(NWV * 64)
__attribute__((amdgpu_waves_per_eu(fwd_occupancy(D, PAGED), fwd_occupancy(D, PAGED))))
fwd_kernel(FwdArgs a, int fold, int tiles, int chunk, SplitArgs sp) {
  constexpr int NDB = D / 32;      // 32-wide d blocks of the output
  constexpr int NKS = D / 16;      // 16-deep k steps of Q K^T
  __shared__ FwdSmem<D> sm;
  __shared__ uint32_t tab[CACHE ? 1 : kMaxTableSegs + 1];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int l32 = lane & 31, hf = lane >> 5;

  // Work item: (dialogue, set of `fold` heads) groups in XCD-aware chunks,
  // longest column tile first inside each chunk.
  int b, head0, tile, kvh;
  Unit u;  // SPLIT: the chunk of keys
  if constexpr (SPLIT) {
    if (!find_unit(sp, (int)blockIdx.x, lane, u)) return;
    b = u.b;
    kvh = u.kvh;
    head0 = kvh * fold;
    tile = __builtin_amdgcn_readfirstlane(u.cg);
  } else {
    const int hsets = a.hq / fold;
    int group;
    if (!xcd_work_item((int)blockIdx.x, a.batch * hsets, tiles, chunk, true, group, tile)) return;
    b = group / hsets;
    head0 = (group % hsets) * fold;
    kvh = head0 / (a.hq / a.hkv);
  }
  const int s = a.cu_q[b];
  const int e = SPLIT ? min(a.cu_q[b + 1], s + sp.max_rows) : a.cu_q[b + 1];
  const uint32_t G = fold, ncol = (uint32_t)max(e - s, 0) * G;
  const uint32_t c0 = (uint32_t)tile * (NWV * kQW), wc0 = c0 + wave * kQW;
  if (c0 >= ncol) return;
  const bool active = wc0 < ncol;
  // rows of the workgroup's last column and of the wave's first and last
  const int wg_last = s + (int)((min(c0 + NWV * kQW, ncol) - 1) / G);
  const int wrow0 = s + (int)(min(wc0, ncol - 1) / G);
  const int wrow1 = s + (int)((min(wc0 + kQW, ncol) - 1) / G);

  int key_begin, key_hi, wave_lo, wave_hi, cache_c = 0;
  bool oob = false;  // cache mode: C_b + L_b outside the cache (out of contract)
  const bf16_t *kbase, *vbase;
  if (CACHE) {
    key_begin = 0;
    cache_c = a.cache_len[b];
    // keys [0, C_b + L_b) (query segment) or [0, C_b + r] for row r (answer
    // segment); clamped to the slab for out-of-contract lengths, whose rows
    // get NaN
    const int slab_rows = PAGED ? a.max_pages * a.page_size : (int)(a.kv_head_stride / D);
    oob = cache_c < 0 || cache_c + (e - s) > slab_rows;
    if (a.cache_causal) {
      key_hi = max(min(cache_c + (wg_last - s) + 1, slab_rows) - 1, 0);
      wave_lo = min(cache_c + (wrow0 - s), key_hi);
      wave_hi = active ? min(cache_c + (wrow1 - s), key_hi) : -1;
    } else {
      key_hi = max(min(cache_c + (e - s), slab_rows) - 1, 0);
      wave_lo = key_hi;
      wave_hi = active ? key_hi : -1;
    }
    if constexpr (SPLIT) {
      // The chunk's keys. An answer segment's early rows may end before it:
      // then one key, which exists, is staged and no wave uses it.
      key_begin = __builtin_amdgcn_readfirstlane(u.tile0) * kBN;
      key_hi = min(key_hi, key_begin + __builtin_amdgcn_readfirstlane(u.tiles) * kBN - 1);
      key_hi = max(key_hi, key_begin);
      wave_lo = min(wave_lo, key_hi);
      wave_hi = min(wave_hi, key_hi);
    }
    const int64_t off =
        PAGED ? 0 : (int64_t)b * a.kv_seq_stride + (int64_t)kvh * a.kv_head_stride;
    kbase = (const bf16_t *)a.k + off;
    vbase = (const bf16_t *)a.v + off;
  } else {
    key_begin = s;
    if (a.lim) {
      key_hi = a.lim[wg_last];
      wave_lo = a.lim[wrow0];
      wave_hi = active ? a.lim[wrow1] : s - 1;
    } else {  // below, once the first transfers are on their way
      load_seg_table(tab, a.cu_segs, a.seg_is_query, a.num_segs, tid, NWV * 64);
      key_hi = wave_lo = wave_hi = s;
    }
    kbase = (const bf16_t *)a.k + (int64_t)kvh * a.kv_head_stride;
    vbase = (const bf16_t *)a.v + (int64_t)kvh * a.kv_head_stride;
  }
  const int64_t rs = a.kv_row_stride;
  const float sl2 = a.scale * kLog2e;
  // first key of tile t of the workgroup's key range (t < its tile count);
  // in the paged cache a 64-key tile lies inside one page
  const int32_t *btab = a.block_table;
  const int pg_max = a.max_pages, pg_num = a.num_pages, pg_size = a.page_size, nkv = a.hkv;
  auto tile_src = [&](const bf16_t *base, int t) __attribute__((always_inline)) {
    if constexpr (PAGED)
      return base + paged_offset_uniform(btab, pg_max, pg_num, pg_size, nkv, D, b, kvh,
                                         (SPLIT ? key_begin : 0) + t * kBN);
    else
      return base + (int64_t)key_begin * rs + (int64_t)t * (kBN * rs);
  };
  // lazy rescale threshold: 2^8 in probability units
  const float tau = 8.f / sl2;

  // Prologue, with its memory latencies overlapped: the transfers of K(0),
  // V(0) and K(1) need only the dialogue's key range in memory (packed mode:
  // keys past the workgroup's bound are real keys of the dialogue, masked
  // like any other invisible key), so they start before the bounds and Q.
  DmaTile<D, kBN, NWV, NT> dma;
  dma.init(tid, rs);
  {
    const int mem_rows = CACHE ? key_hi - key_begin + 1 : e - key_begin;
    const bf16_t *k0 = tile_src(kbase, 0);
    dma.issue(k0, rs, mem_rows, sm.k[0]);
    dma.issue(tile_src(vbase, 0), rs, mem_rows, sm.v[0]);
    if (mem_rows > kBN)
      dma.issue(PAGED ? tile_src(kbase, 1) : k0 + (int64_t)kBN * rs, rs, mem_rows - kBN,
                sm.k[1]);
  }
  // Per-lane column (columns past the last are computed as copies of it and
  // never stored).
  const uint32_t col = min(wc0 + l32, ncol - 1), crow = col / G;
  const int rc = s + (int)crow, head = head0 + (int)(col - crow * G);
  int lim_r;
  if (CACHE) {
    lim_r = a.cache_causal ? min(cache_c + (rc - s), key_hi) : key_hi;
  } else if (a.lim) {
    lim_r = a.lim[rc];
  } else {
    lds_barrier();  // the table
    lim_r = seg_lim(tab, a.num_segs, rc);
    key_hi = __builtin_amdgcn_readfirstlane(seg_lim(tab, a.num_segs, wg_last));
    wave_lo = __builtin_amdgcn_readfirstlane(lim_r);  // lane 0: the wave's first column
    wave_hi = active ? __builtin_amdgcn_readlane(lim_r, 31) : s - 1;  // lane 31: its last
  }
  bf16x8 qf[NKS];
  {
    const bf16_t *qp = (const bf16_t *)a.q + ((int64_t)rc * a.hq + head) * D + hf * 8;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qf[ks] = *(const bf16x8 *)(qp + ks * 16);
  }
  if constexpr (CACHE) {
    if (a.rope_pos1) rope_queries<D>(qf, hf, a.rope_pos1[rc], a.rope_pos2[rc], a.rope_log2_base);
  }
  wait_loads();  // Q, lim and the transfers above
  __syncthreads();

  f32x16 oacc[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;

  // Software pipeline over key tiles. Tile t's scores S(t) are complete (and
  // masked, the running max raised) when step t starts; step t then issues
  // S(t+1) = K(t+1) Q^T and the P(t) V(t) product in the same basic block as
  // the exponentials of tile t, so matrix and vector work of one wave
  // overlap. LDS holds K(t+1) and V(t) during step t while K(t+2) and V(t+1)
  // are in flight into the other halves of the double buffers.
  const int ntiles = (key_hi - key_begin) / kBN + 1;  // for the workgroup
  const int nw =  // this wave's (none if its rows end before a split chunk)
      active && (!SPLIT || wave_hi >= key_begin) ? (wave_hi - key_begin) / kBN + 1 : 0;
  const int64_t tile_elems = (int64_t)kBN * rs;
  const bf16_t *kt = kbase + (int64_t)key_begin * rs;
  const bf16_t *vt = vbase + (int64_t)key_begin * rs;
  // paged cache: sources of K(t+2) and V(t+1) for step t
  const bf16_t *pk2 = PAGED ? tile_src(kbase, min(2, ntiles - 1)) : kt;
  const bf16_t *pv1 = PAGED ? tile_src(vbase, min(1, ntiles - 1)) : vt;
  // its tiles per page, and those left in the pages of K(t+2) and V(t+1)
  const int tpp = PAGED ? pg_size / kBN : 1, first = SPLIT ? key_begin / kBN : 0;
  int kleft = PAGED ? tpp - (first + 2) % tpp : 0, vleft = PAGED ? tpp - (first + 1) % tpp : 0;
  SwzOffsets<D> so;
  so.init(lane);

  f32x16 sa[2], sb[2];
  if (nw > 0) {
    tile_scores<D>((const char *)sm.k[0], so, qf, sa);
    if (key_begin + kBN - 1 > wave_lo) tile_mask(sa, key_begin, hf, lim_r);
    raise_max<SPLIT>(tile_max(sa), sl2, tau, m_run, l_run, oacc);
  }
  lds_barrier();  // every wave is done with K(0) before K(2) overwrites it

  // Step t. MODE 0: K(t+2) and V(t+1) are full tiles, transferred one
  // transfer every third product from the first (a burst of transfers
  // stalls the waves that issue them; one every fourth product, the last
  // near the step end, measured 1.5-3 % slower with the phase priority of
  // step_block); MODE 1: the transfers at once (partial tiles near the end
  // of the key range); MODE 2: the workgroup's last tile, which has no
  // S(t+1) and no transfers, so the waves whose last tile it is run the
  // exponentials and P V only. (A wave whose last tile comes earlier
  // computes an unused S(t+1) there, which keeps one code path per loop.)
  auto step = [&](f32x16 (&cur)[2], f32x16 (&nxt)[2], int t, auto modec) {
    constexpr int MODE = decltype(modec)::value;
    constexpr bool LAST = MODE == 2;
    constexpr int NI = decltype(dma)::NI;
    static_assert(3 * (2 * NI - 1) < 2 * (D / 16) + 4 * (D / 32),
                  "every full-tile transfer falls inside the step's products");
    const int c0 = key_begin + t * kBN;
    const bf16_t *ksrc = PAGED ? pk2 : kt + 2 * tile_elems;
    const bf16_t *vsrc = PAGED ? pv1 : vt + tile_elems;
    if (MODE == 1 || (MODE == 0 && t >= nw)) {
      if (t + 2 < ntiles)
        dma.issue(ksrc, rs, key_hi - (c0 + 2 * kBN) + 1, sm.k[t & 1]);
      dma.issue(vsrc, rs, key_hi - (c0 + kBN) + 1, sm.v[(t + 1) & 1]);
    }
    const char *kl = (const char *)sm.k[(t + 1) & 1];
    const char *vl = (const char *)sm.v[t & 1];
    auto hook = [&](int n) __attribute__((always_inline)) {
      if (MODE == 0 && n % 3 == 0 && n / 3 < 2 * NI) {
        if (n / 3 < NI) dma.issue_one(ksrc, n / 3, sm.k[t & 1]);
        else dma.issue_one(vsrc, n / 3 - NI, sm.v[(t + 1) & 1]);
      }
    };
    if (t < nw) {
      float mt;
      l_run += step_block<D, LAST, !PAGED || MODE == 0>(kl, vl, so, qf, cur, nxt, oacc, sl2,
                                           log2_max<SPLIT>(m_run, sl2), mt, hook);
      if (!LAST && t + 1 < nw) {
        if (c0 + 2 * kBN - 1 > wave_lo) {  // S(t+1) crosses some row's bound
          tile_mask(nxt, c0 + kBN, hf, lim_r);
          mt = tile_max(nxt);
        }
        raise_max<SPLIT>(mt, sl2, tau, m_run, l_run, oacc);
      }
    }
    if (!LAST) {
      kt += tile_elems;
      vt += tile_elems;
      if constexpr (PAGED) {  // K(t+3) and V(t+2), re-based at page starts
        const bool knew = --kleft == 0, vnew = --vleft == 0;
        pk2 = knew ? tile_src(kbase, min(t + 3, ntiles - 1)) : pk2 + tile_elems;
        pv1 = vnew ? tile_src(vbase, min(t + 2, ntiles - 1)) : pv1 + tile_elems;
        if (knew) kleft = tpp;
        if (vnew) vleft = tpp;
      }
    }
    wait_vmem();
    __syncthreads();
  };
  // steps whose K(t+2) and V(t+1) are full tiles, an even count of them
  int t = 0;
  if (!PAGED || a.max_pages * pg_size >= kSpreadKeys) {
    const int nfull = max((key_hi - key_begin + 1) / kBN - 2, 0) & ~1;
    for (; t < nfull; t += 2) {
      step(sa, sb, t, std::integral_constant<int, 0>{});
      step(sb, sa, t + 1, std::integral_constant<int, 0>{});
    }
  }
  for (; t + 1 < ntiles; t += 2) {
    step(sa, sb, t, std::integral_constant<int, 1>{});
    if (t + 2 < ntiles) step(sb, sa, t + 1, std::integral_constant<int, 1>{});
  }
  if ((ntiles - 1) & 1) step(sb, sa, ntiles - 1, std::integral_constant<int, 2>{});
  else step(sa, sb, ntiles - 1, std::integral_constant<int, 2>{});

  if (!active) return;
  const float lt = pair_sum(l_run);
  // the lane's row and head again (kept over the loop they would cost
  // registers that d = 64 at three waves per SIMD does not have)
  int ln;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(ln));
  const uint32_t ocol = wc0 + (ln & 31), orow = ocol / G;
  if (ocol >= ncol) return;
  const int row = s + (int)orow, ohead = head0 + (int)(ocol - orow * G);
  if constexpr (SPLIT) {
    if (u.n > 1) {  // partials, merged by the split-key kernel's combine
      const int64_t pi = (int64_t)u.slot * sp.col_stride + (ocol - c0);
      float *po = sp.part_o + pi * D + hf * 4;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          *(f32x4 *)(po + db * 32 + 8 * i) = f32x4{oacc[db][4 * i], oacc[db][4 * i + 1],
                                                   oacc[db][4 * i + 2], oacc[db][4 * i + 3]};
      if (hf == 0) *(f32x2 *)(sp.part_ml + pi * 2) = f32x2{m_run * sl2, lt};
      return;
    }
  }
  const float inv = oob ? __builtin_nanf("") : 1.f / lt;
  bf16_t *op = (bf16_t *)a.o + ((int64_t)row * a.hq + ohead) * D + hf * 4;
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      u32x2 w;
      w[0] = pack_bf16x2(oacc[db][4 * i + 0] * inv, oacc[db][4 * i + 1] * inv);
      w[1] = pack_bf16x2(oacc[db][4 * i + 2] * inv, oacc[db][4 * i + 3] * inv);
      *(u32x2 *)(op + db * 32 + 8 * i) = w;
    }
  if (a.lse && hf == 0)
    a.lse[(int64_t)ohead * a.total_q + row] = oob ? __builtin_nanf("") : m_run * a.scale + logf(lt);
}

int gcd_int(int x, int y) {
  while (y) { const int t = x % y; x = y; y = t; }
  return x;
}

// Query heads folded into a workgroup's columns. Packed: the part of the group
// that fills whole waves (a group of 3 as one set ran 12 ragged dialogues up to
// 900 tokens, 24/8 heads, in 67 us instead of 60). In cache mode, where rows are
// few, the whole group; but a group's workgroups share an XCD, so when fewer
// than 32 groups would load the 8 XCDs unevenly, sets of 8 heads and more that
// still fill workgroups. Whole group, sets of 8 (us): 200 rows over 8 ragged
// dialogues up to 3000 keys, 32/2 heads 80, 66 (four other layouts 77-85,
// 65-71); 800 rows over 4 ragged up to 8000, 64/2 810, 603; 300 over 8 x 3000,
// 64/2 247, 248; but 14 over 40 x 2000, 32/2 40, 49 and 30 x 3000, 64/4 56, 78.
int fold_of(const FwdArgs &a, bool cache) {
  const int g = a.hq / a.hkv;
  if (!cache) return gcd_int(g, NWV);
  int fold = g;
  while (fold >= 16 && fold % 2 == 0 && (int64_t)a.batch * (a.hq / fold) < 32 &&
         (int64_t)a.max_rows * (fold / 2) >= NWV * kQW)
    fold /= 2;
  return fold;
}

int64_t column_tiles(const FwdArgs &a, int fold) {
  const int64_t w = NWV * kQW;
  return ((int64_t)a.max_rows * fold + w - 1) / w;
}

template <int D, bool CACHE, bool PAGED>
hipError_t launch_fwd_p(const FwdArgs &a, hipStream_t stream) {
  const int fold = fold_of(a, CACHE);
  const int tiles = (int)column_tiles(a, fold);
  const int64_t groups = (int64_t)a.batch * (a.hq / fold);
  if (groups * tiles == 0) return hipSuccess;
  const dim3 grid((unsigned)xcd_grid(groups, tiles));
  if constexpr (CACHE) {
    if (tiles == 1) {
      hipLaunchKernelGGL((fwd_kernel<D, true, PAGED, true, false>), grid, dim3(NWV * 64), 0,
                         stream, a, fold, tiles, ISM_SCHED_CHUNK, SplitArgs{});
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((fwd_kernel<D, CACHE, PAGED, false, false>), grid, dim3(NWV * 64), 0,
                     stream, a, fold, tiles, ISM_SCHED_CHUNK, SplitArgs{});
  return hipGetLastError();
}

template <int D, bool CACHE>
hipError_t launch_fwd_t(const FwdArgs &a, hipStream_t stream) {
  if (CACHE && a.block_table) return launch_fwd_p<D, true, true>(a, stream);
  return launch_fwd_p<D, CACHE, false>(a, stream);
}

template <int D, bool PAGED>
hipError_t launch_fwd_split_p(const FwdArgs &a, const SplitArgs &sp, hipStream_t stream) {
  const dim3 grid((unsigned)(((int64_t)sp.max_units * a.hkv + 7) / 8 * 8));
  if (sp.col_groups == 1)
    hipLaunchKernelGGL((fwd_kernel<D, true, PAGED, true, true>), grid, dim3(NWV * 64), 0, stream,
                       a, a.hq / a.hkv, 0, 0, sp);
  else
    hipLaunchKernelGGL((fwd_kernel<D, true, PAGED, false, true>), grid, dim3(NWV * 64), 0, stream,
                       a, a.hq / a.hkv, 0, 0, sp);
  const hipError_t err = hipGetLastError();
  return err == hipSuccess && sp.max_splits > 1 ? launch_split_combine(sp, D, stream) : err;
}

}  // namespace

hipError_t launch_fwd_split(const FwdArgs &a, const SplitArgs &sp, int d, hipStream_t stream) {
  if (sp.colw != NWV * kQW || 1 << sp.tile_shift != kBN) return hipErrorInvalidValue;
  if (d == 128) return a.block_table ? launch_fwd_split_p<128, true>(a, sp, stream)
                                     : launch_fwd_split_p<128, false>(a, sp, stream);
  if (d == 64) return a.block_table ? launch_fwd_split_p<64, true>(a, sp, stream)
                                    : launch_fwd_split_p<64, false>(a, sp, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_fwd(const FwdArgs &a, int d, bool cache_mode,
                      hipStream_t stream) {
  if (d == 128) return cache_mode ? launch_fwd_t<128, true>(a, stream)
                                  : launch_fwd_t<128, false>(a, stream);
  if (d == 64) return cache_mode ? launch_fwd_t<64, true>(a, stream)
                                 : launch_fwd_t<64, false>(a, stream);
  return hipErrorInvalidValue;
}

}  // namespace ism
