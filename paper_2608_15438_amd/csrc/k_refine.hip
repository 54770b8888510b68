// Step 5: exact refinement of C(q) in the original space (Sec. 3.4 intro,
// Sec. 3.5) -- the HBM-bound part of the search.
//
//  plan   (one wave per query)  row prefix over the query's clusters, total
//         rows R_q, tile size T_q = max(smallest, ceil(R_q / 64)) and the
//         (query, row range) tiles;
//  refine (persistent waves)    each wave takes tiles (its own number's, or
//         from one of a few atomic counters) and walks the tile's virtual rows; 8 lanes cover one 128-byte row
//         segment with one 16-byte load each, so a wave instruction reads 8
//         full cache lines; U rows per lane group are in flight;
//         uint8:  |x - q|^2 = x.x - 2 x.q + q.q with packed u8 dot products,
//                 exact in int32;   fp32: fmaf((x-q), (x-q), acc);
//         the 8 partial sums are combined with xor shuffles; a sorted top-k
//         of (distance, original id) lives in lanes 0..k-1 and a candidate
//         reads its original id only when it can enter it.  Rows past 1 KB
//         are summed per 1 KB slab (reduced over the 8 lanes, added in slab
//         order) against the query row in LDS, and an fp32 row stops being
//         read once its sum passes the list's k-th key;
//  merge  (one wave per query)  the tiles' partial top-k lists are merged.
#include "nr_internal.h"

// launch shape of the refinement (tuned on MI355X)
#ifndef NR_REFINE_BLOCKS_PER_CU
#define NR_REFINE_BLOCKS_PER_CU 8
#endif
#ifndef NR_REFINE_U1
#define NR_REFINE_U1 8          // rows in flight per lane group for 128-byte rows
#endif
#ifndef NR_REFINE_NT
#define NR_REFINE_NT 1          // non-temporal payload loads (+3% on MI355X)
#endif

namespace nr {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ uint4 load_payload(const uint4 *p) {
#if NR_REFINE_NT
  const u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
#else
  return *p;
#endif
}

// ------------------------------------------------------------------ plan
// cluster counts come from the caller in nr_refine: keep them in [0, cap]
__device__ __forceinline__ int clamp_count(int32_t n, int64_t cap) {
  return n < 0 ? 0 : (n > cap ? (int)cap : n);
}

// One wave per query: the rows before each of its clusters, its tile size, its
// tiles (numbered from one atomic per block, so in any order: the merge orders
// the results) and each tile's first cluster.  (As three kernels -- rows, a
// scan over the queries, tiles -- 12 us for one query, 35 for 10,000.)
constexpr int PLAN_WAVES = 16;
__global__ void __launch_bounds__(PLAN_WAVES * WAVE) k_plan(PlanArgs a) {
  __shared__ int32_t s_nt[PLAN_WAVES];
  __shared__ int32_t s_base;
  const int lane = lane_id(), wv = threadIdx.x / WAVE;
  const int64_t q = (int64_t)blockIdx.x * PLAN_WAVES + wv;
  const bool live = q < a.nq && !(a.qmask && !a.qmask[q]);
  uint32_t *pre = a.rowpre + (live ? q : 0) * (a.cap + 1);
  uint32_t tot = 0, t = TILE_MIN_ROWS;
  int nt = 0, ncl = 0;
  if (live) {
    const int n = clamp_count(a.nclus[q], a.cap);
    const uint32_t *cl = a.clus + q * a.cap;
    uint64_t run = 0;
    const int own0 = a.own_cseed ? a.own_cseed[q] : 0;
    // own (seed) pass of the shared schedule: only the leading clusters, compacted
    uint32_t *co = a.clus_out ? a.clus_out + q * a.cap : nullptr;
    int nout = 0;
    if (lane == 0) pre[0] = 0;
    // the compacted seed pass needs only the leading clusters
    const int nw = co && a.own_cseed && own0 < n ? own0 : n;
    for (int i0 = 0; i0 < nw; i0 += WAVE) {
      const int i = i0 + lane;
      uint32_t c = 0;
      uint64_t sz = 0;
      if (i < nw) {
        c = cl[i];
        if (c < a.n_clusters) {
          sz = a.cl_off[(uint64_t)c + 1] - a.cl_off[c];
          // the seed pass leaves every later cluster to the scan
          if (a.own_cseed && i >= own0) sz = 0;
        }
      }
      const uint64_t incl = wave_incl_scan_u64(sz);
      if (co) {
        const uint64_t keep = ballot(sz > 0);
        const int pos = nout + popc64(keep & lanemask_lt());
        if (sz > 0) {
          co[pos] = c;
          pre[pos + 1] = (uint32_t)(run + incl);
        }
        nout += popc64(keep);
      } else if (i < n) {
        pre[i + 1] = (uint32_t)(run + incl);
      }
      run += bcast_u64(incl, WAVE - 1);
    }
    ncl = co ? nout : n;
    // a list of more than 2^32 - 1 rows (only possible with repeated clusters
    // given to nr_refine) is refused: it returns no candidates
    tot = run > 0xffffffffull ? 0u : (uint32_t)run;
    const uint32_t tmin = a.tile_min ? a.tile_min : TILE_MIN_ROWS;
    t = (tot + MAX_TILES_PER_QUERY - 1) / MAX_TILES_PER_QUERY;
    if (t < tmin) t = tmin;
    nt = (int)(((uint64_t)tot + t - 1) / t);
    if (lane == 0) {
      if (a.rfull) a.rfull[q] = tot;
      if (co) a.nclus_out[q] = nout;
    }
  }
  if (lane == 0) s_nt[wv] = nt;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t sum = 0;
    for (int i = 0; i < PLAN_WAVES; ++i) sum += s_nt[i];
    s_base = sum > 0 ? atomicAdd(&a.tile_off[a.nq], sum) : 0;
  }
  __syncthreads();
  if (q >= a.nq) return;
  int32_t off = s_base;
  for (int i = 0; i < wv; ++i) off += s_nt[i];
  if (lane == 0) {
    a.rtot[q] = tot;
    a.tsize[q] = t;
    a.ntile[q] = nt;
    a.tile_off[q] = off;
  }
  __threadfence_block();  // the wave reads back the row prefix it wrote
  for (int x = lane; x < nt; x += WAVE) {
    const uint32_t v0 = (uint32_t)x * t;
    // last cluster i with pre[i] <= v0 (clusters of zero rows are skipped)
    int lo = 0, hi = ncl - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (pre[mid] <= v0) lo = mid; else hi = mid - 1;
    }
    a.tile_q[off + x] = (int32_t)q;
    a.tile_c0[off + x] = lo;
  }
}

hipError_t launch_plan(const PlanArgs &a, hipStream_t s) {
  if (a.nq <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_plan, dim3((unsigned)((a.nq + PLAN_WAVES - 1) / PLAN_WAVES)),
                     dim3(PLAN_WAVES * WAVE), 0, s, a);
  return hipGetLastError();
}

// ------------------------------------------------------------------ top-k in lanes
// The refinement's running top-k: lanes 0..k-1 hold a list sorted by (key,
// id), kth_key is the last entry's key when full.  An entry's original id is
// read only when it decides something -- a candidate whose key equals a key in
// the list (ids order equal keys) -- or when the tile's list is written out,
// so the row loop does not wait for id loads.  Entries keep their payload row
// (phys) until then; id is UNREAD.  Rows and ids are below 2^32 - 1.
constexpr uint32_t UNREAD = 0xffffffffu;
struct LazyTopK {
  uint32_t key, id, phys;
  int cnt;
  uint32_t kth_key;
};

__device__ __forceinline__ void ltopk_init(LazyTopK &t) {
  t.key = 0xffffffffu;
  t.id = UNREAD;
  t.phys = 0;
  t.cnt = 0;
  t.kth_key = 0xffffffffu;
}

// the value of the lane below (lane 0 keeps its own)
__device__ __forceinline__ uint32_t lane_up1(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x138, 0xF, 0xF, false);
}

// insert the payload row cp with key ck if (ck, its id) ranks among the k best
// (wave-uniform arguments)
__device__ __forceinline__ void ltopk_insert(LazyTopK &t, int k, uint32_t ck, uint32_t cp,
                                             const int64_t *row_ids) {
  const int lane = lane_id();
  if (t.cnt == k && ck > t.kth_key) return;
  // ids matter only among equal keys: read the candidate's and those of the
  // listed entries with its key (one round of loads, rare)
  const bool eq = lane < t.cnt && t.key == ck;
  uint32_t cid = UNREAD;
  if (ballot(eq)) {
    cid = (uint32_t)row_ids[cp];
    if (eq && t.id == UNREAD) t.id = (uint32_t)row_ids[t.phys];
    // a tie with the k-th entry: the candidate enters only below its id
    if (t.cnt == k && ck == t.kth_key && cid >= bcast_u32(t.id, k - 1)) return;
  }
  const bool less = lane < t.cnt && (t.key < ck || (t.key == ck && t.id < cid));
  const int pos = popc64(ballot(less));
  const uint32_t up_key = lane_up1(t.key), up_id = lane_up1(t.id), up_phys = lane_up1(t.phys);
  if (lane == pos) {
    t.key = ck;
    t.id = cid;
    t.phys = cp;
  } else if (lane > pos && lane < k) {
    t.key = up_key;
    t.id = up_id;
    t.phys = up_phys;
  }
  t.cnt = t.cnt + 1 < k ? t.cnt + 1 : k;
  if (t.cnt == k) t.kth_key = bcast_u32(t.key, k - 1);
}

// Candidates of one step (one per lane of `m`, payload row cp), all at once:
// their ids and the list's unread ones are loaded, the candidates sorted by
// (key, id) -- ids are below 2^32 -- and merged with the list.  While a list
// fills, a step of 64 rows holds tens of entrants, each an insertion otherwise.
constexpr int BATCH_MIN = 5;   // entrants of a step from which they go together (3 to 12 alike)
__device__ __forceinline__ void ltopk_batch(LazyTopK &t, int k, uint64_t m, uint32_t ck,
                                            uint32_t cp, const int64_t *row_ids) {
  const int lane = lane_id();
  const bool in = (m >> lane) & 1ull;
  uint32_t cid = 0;
  if (in) cid = (uint32_t)row_ids[cp];
  if (lane < t.cnt && t.id == UNREAD) t.id = (uint32_t)row_ids[t.phys];
  const uint64_t cand = wave_sort_u64(in ? ((uint64_t)ck << 32) | cid : ~0ull);
  const uint64_t list = lane < t.cnt ? ((uint64_t)t.key << 32) | t.id : ~0ull;
  const uint64_t v = wave_merge_least_u64(list, cand);
  const int n = t.cnt + popc64(m);
  t.cnt = n < k ? n : k;
  t.key = lane < t.cnt ? (uint32_t)(v >> 32) : 0xffffffffu;
  t.id = (uint32_t)v;
  if (t.cnt == k) t.kth_key = bcast_u32(t.key, k - 1);
}

// The rows of one step into the list.  Row 8 u + g of the step has its key in
// every lane of group g; lane (g, gl) takes that of u = gl.  phys_of() gives
// the payload row of the lane's own row (called only when a row may enter).
template <int U, class Phys>
__device__ __forceinline__ void ltopk_step(LazyTopK &t, int k, const uint32_t (&key)[U],
                                           uint32_t rows_left, const int64_t *row_ids,
                                           Phys phys_of) {
  const int lane = lane_id(), g = lane >> 3, gl = lane & 7;
  uint32_t kk = key[0];
#pragma unroll
  for (int u = 1; u < U; ++u) kk = gl == u ? key[u] : kk;
  const bool in = gl < U && (uint32_t)(8 * gl + g) < rows_left;
  uint64_t m = ballot(in && kk <= t.kth_key);
  if (!m) return;
  const uint32_t phys = phys_of();
  if (popc64(m) >= BATCH_MIN) {
    ltopk_batch(t, k, m, kk, phys, row_ids);
    return;
  }
  while (m) {
    const int src = __ffsll((unsigned long long)m) - 1;
    m &= m - 1;
    const uint32_t ck = bcast_u32(kk, src);
    if (t.cnt == k && ck > t.kth_key) continue;
    ltopk_insert(t, k, ck, bcast_u32(phys, src), row_ids);
  }
}

// ------------------------------------------------------------------ refine
#ifndef NR_REFINE_WAVES1
#define NR_REFINE_WAVES1 1      // waves per SIMD the registers are sized for (128-byte rows; 1: free)
#endif

template <int IS_U8, int NSEG, int U>
__global__ void __launch_bounds__(256, NSEG <= 1 ? NR_REFINE_WAVES1 : 1) k_refine(RefineArgs a) {
  __shared__ uint32_t s_vs[4][STAGE_CLUSTERS + 1];
  __shared__ uint64_t s_ps[4][STAGE_CLUSTERS];
  // rows longer than 8 segments: the wave's copy of the query row (slot gl of
  // segment s at s * 8 + gl), read a chunk at a time
  constexpr int SC = 8;
  __shared__ uint4 s_qrow[4][NSEG > SC ? NSEG * 8 : 1];
  const int lane = lane_id();
  const int w = threadIdx.x >> 6;
  const int g = lane >> 3;      // lane group: one row at a time
  const int gl = lane & 7;      // 16-byte slot inside a 128-byte row segment
  uint32_t *vs = s_vs[w];
  uint64_t *ps = s_ps[w];
  const int total = a.tile_off[a.nq];
  const int rb = a.row_bytes;
  const int k = a.k;
  unsigned long long nbytes = 0;  // row bytes this lane (group) read

  // the wave's tiles: its own number where there are no more tiles than waves
  // (a wave that has none then ends without an atomic), else those congruent
  // to it modulo TILE_COUNTERS, in turn
  const int nwaves = (int)gridDim.x * 4;
  const int wid = __builtin_amdgcn_readfirstlane((int)blockIdx.x * 4 + w);
  const int cg = wid % TILE_COUNTERS;
  auto next_tile = [&]() __attribute__((always_inline)) {
    int x = 0;
    if (lane == 0) x = atomicAdd(&a.counter[cg * TILE_COUNTER_STRIDE], 1);
    return __builtin_amdgcn_readfirstlane(x) * TILE_COUNTERS + cg;
  };
  for (int t = total <= nwaves ? wid : next_tile(); t < total;) {
    const int64_t q = a.tile_q[t];
    const uint32_t T = a.tsize[q];
    const uint32_t R = a.rtot[q];
    const uint32_t v0 = (uint32_t)(t - a.tile_off[q]) * T;
    const uint32_t v1 = v0 + T < R ? v0 + T : R;
    const uint32_t *pre = a.rowpre + q * (a.cap + 1);
    const uint32_t *cl = a.clus + q * a.cap;
    const int n_cl = clamp_count(a.nclus[q], a.cap);
    int c = a.tile_c0[t];

    // this lane's slices of the query: in registers for rows of up to 8
    // segments, from the wave's LDS copy for longer ones
    uint4 qv[NSEG <= SC ? NSEG : 1];
    uint4 *qrow = s_qrow[w];
    const unsigned char *qb = (const unsigned char *)a.queries + q * (int64_t)rb;
    if constexpr (NSEG <= SC) {
#pragma unroll
      for (int s = 0; s < NSEG; ++s) {
        const int off = 128 * s + 16 * gl;
        qv[s] = off < rb ? *(const uint4 *)(qb + off) : make_uint4(0, 0, 0, 0);
      }
    } else {
      __builtin_amdgcn_wave_barrier();  // the previous tile is done with the copy
      for (int i = lane; i < NSEG * 8; i += WAVE)
        qrow[i] = 16 * i < rb ? *(const uint4 *)(qb + 16 * i) : make_uint4(0, 0, 0, 0);
      __builtin_amdgcn_wave_barrier();
    }
    int32_t qq = 0;
    if (IS_U8) {
#pragma unroll
      for (int s = 0; s < NSEG; ++s) {
        const uint4 qs4 = NSEG <= SC ? qv[NSEG <= SC ? s : 0] : qrow[s * 8 + gl];
        uint32_t acc = (uint32_t)qq;
        acc = __builtin_amdgcn_udot4(qs4.x, qs4.x, acc, false);
        acc = __builtin_amdgcn_udot4(qs4.y, qs4.y, acc, false);
        acc = __builtin_amdgcn_udot4(qs4.z, qs4.z, acc, false);
        acc = __builtin_amdgcn_udot4(qs4.w, qs4.w, acc, false);
        qq = (int32_t)acc;
      }
      qq += __shfl_xor(qq, 1);
      qq += __shfl_xor(qq, 2);
      qq += __shfl_xor(qq, 4);
    }
    LazyTopK tk;
    ltopk_init(tk);

    uint32_t v = v0;
    while (v < v1) {
      // stage clusters c .. c+ns-1: virtual and physical first rows
      const int ns = n_cl - c < STAGE_CLUSTERS ? n_cl - c : STAGE_CLUSTERS;
      for (int j = lane; j < ns; j += WAVE) {
        vs[j] = pre[c + j];
        const uint32_t cj = cl[c + j];
        ps[j] = cj < a.n_clusters ? a.cl_off[cj] : 0;
      }
      if (lane == 0) vs[ns] = pre[c + ns];
      __builtin_amdgcn_wave_barrier();
      const uint32_t vend = v1 < vs[ns] ? v1 : vs[ns];
      // per lane group (rows of a group only increase): the staged cluster
      // holding its rows, its first virtual row and physical row, and the
      // next cluster's first virtual row, kept in registers so that a row
      // costs an LDS read only where it crosses into the next cluster
      int cur = 0;
      uint32_t vcur = vs[0], vnext = vs[1];
      uint64_t pcur = ps[0];
      if constexpr (NSEG == 1) {
        // rows of one 128-byte segment: a two-stage pipeline, the rows of the
        // next step loading while those of this one are scored (two register
        // buffers, the loop unrolled by two).  A row's payload index is kept
        // only until its load is issued; an entrant's is found again from
        // the staged clusters.
        uint4 xa[U], xb[U];
        auto issue = [&](uint32_t vb, uint4(&x)[U]) __attribute__((always_inline)) {
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const uint32_t rv = vb + 8 * u + g;
            const bool ok = rv < vend;
            uint64_t phys = 0;
            if (ok) {
              if (vnext <= rv) {
                do {
                  ++cur;
                  vnext = vs[cur + 1];
                } while (vnext <= rv);
                vcur = vs[cur];
                pcur = ps[cur];
              }
              phys = pcur + (rv - vcur);
            }
            x[u] = (ok && 16 * gl < rb) ? load_payload(a.ra.seg(phys, 16 * gl))
                                        : make_uint4(0, 0, 0, 0);
          }
        };
        auto score = [&](uint32_t vb, const uint4(&x)[U]) __attribute__((always_inline)) {
          uint32_t key[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            if (IS_U8) {
              uint32_t xx = 0, xq = 0;
              xx = __builtin_amdgcn_udot4(x[u].x, x[u].x, xx, false);
              xx = __builtin_amdgcn_udot4(x[u].y, x[u].y, xx, false);
              xx = __builtin_amdgcn_udot4(x[u].z, x[u].z, xx, false);
              xx = __builtin_amdgcn_udot4(x[u].w, x[u].w, xx, false);
              xq = __builtin_amdgcn_udot4(x[u].x, qv[0].x, xq, false);
              xq = __builtin_amdgcn_udot4(x[u].y, qv[0].y, xq, false);
              xq = __builtin_amdgcn_udot4(x[u].z, qv[0].z, xq, false);
              xq = __builtin_amdgcn_udot4(x[u].w, qv[0].w, xq, false);
              int32_t part = (int32_t)xx - 2 * (int32_t)xq;
              part += __shfl_xor(part, 1);
              part += __shfl_xor(part, 2);
              part += __shfl_xor(part, 4);
              key[u] = (uint32_t)(part + qq);
            } else {
              float acc = 0.0f;
              const float t0 = __uint_as_float(x[u].x) - __uint_as_float(qv[0].x);
              const float t1 = __uint_as_float(x[u].y) - __uint_as_float(qv[0].y);
              const float t2 = __uint_as_float(x[u].z) - __uint_as_float(qv[0].z);
              const float t3 = __uint_as_float(x[u].w) - __uint_as_float(qv[0].w);
              acc = fmaf(t0, t0, acc);
              acc = fmaf(t1, t1, acc);
              acc = fmaf(t2, t2, acc);
              acc = fmaf(t3, t3, acc);
              acc += __shfl_xor(acc, 1);
              acc += __shfl_xor(acc, 2);
              acc += __shfl_xor(acc, 4);
              key[u] = __float_as_uint(acc);
            }
          }
          // a row's payload index: the last staged cluster starting at or
          // before its virtual row
          const uint32_t left = vend - vb;
          if (lane == 0) nbytes += (unsigned long long)(left < 8 * U ? left : 8 * U) * (uint32_t)rb;
          ltopk_step<U>(tk, k, key, left, a.row_ids, [&]() -> uint32_t {
            const uint32_t rv = vb + 8 * gl + g;
            int lo = 0, hi = ns - 1;
            while (lo < hi) {
              const int mid = (lo + hi + 1) >> 1;
              if (vs[mid] <= rv) lo = mid; else hi = mid - 1;
            }
            return (uint32_t)ps[lo] + (rv - vs[lo]);
          });
        };
        uint32_t vb = v;
        issue(vb, xa);
        for (;;) {
          const uint32_t vn = vb + 8 * U;
          if (vn < vend) issue(vn, xb);
          score(vb, xa);
          if (vn >= vend) break;
          const uint32_t vn2 = vn + 8 * U;
          if (vn2 < vend) issue(vn2, xa);
          score(vn, xb);
          if (vn2 >= vend) break;
          vb = vn2;
        }
      } else
      for (uint32_t vb = v; vb < vend; vb += 8 * U) {
        uint64_t phys[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const uint32_t rv = vb + 8 * u + g;
          ok[u] = rv < vend;
          phys[u] = 0;
          if (ok[u]) {
            if (vnext <= rv) {
              do {
                ++cur;
                vnext = vs[cur + 1];
              } while (vnext <= rv);
              vcur = vs[cur];
              pcur = ps[cur];
            }
            phys[u] = pcur + (rv - vcur);
          }
        }
        uint32_t key[U];
        if constexpr (NSEG > SC) {
          // long rows: slabs of SC segments (1 KB).  Each slab is accumulated
          // in segment order per lane, reduced over the row's 8 lanes, and
          // added to the row's running sum in slab order: the arithmetic the
          // batch-shared scan uses for rows this long
          uint32_t xx[U], xq[U];
          float fs[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            xx[u] = 0;
            xq[u] = 0;
            fs[u] = 0.0f;
          }
          const int nsl = (rb + 128 * SC - 1) / (128 * SC);
          // fp32: the running sum only grows (non-negative terms rounded to
          // nearest), so a row whose sum is already past the list's k-th key
          // cannot enter it and reads no further slabs
          const uint32_t bound = tk.kth_key;
#pragma unroll 1
          for (int sl = 0; sl < nsl; ++sl) {
            const int s0 = sl * SC;
            if (!IS_U8 && sl > 0) {
              bool any = false;
#pragma unroll
              for (int u = 0; u < U; ++u) {
                ok[u] = ok[u] && __float_as_uint(fs[u]) <= bound;
                any |= ok[u];
              }
              if (!ballot(any)) break;
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
              if (ok[u] && gl == 0) nbytes += (uint32_t)(rb - 128 * s0 < 128 * SC ? rb - 128 * s0 : 128 * SC);
            uint4 xc[U][SC];
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
              for (int s = 0; s < SC; ++s) {
                const int off = 128 * (s0 + s) + 16 * gl;
                xc[u][s] = (ok[u] && off < rb) ? load_payload(a.ra.seg(phys[u], off))
                                               : make_uint4(0, 0, 0, 0);
              }
            }
            uint4 qc[SC];
#pragma unroll
            for (int s = 0; s < SC; ++s) qc[s] = qrow[(s0 + s) * 8 + gl];
#pragma unroll
            for (int u = 0; u < U; ++u) {
              float fa = 0.0f;
#pragma unroll
              for (int s = 0; s < SC; ++s) {
                if (IS_U8) {
                  xx[u] = __builtin_amdgcn_udot4(xc[u][s].x, xc[u][s].x, xx[u], false);
                  xx[u] = __builtin_amdgcn_udot4(xc[u][s].y, xc[u][s].y, xx[u], false);
                  xx[u] = __builtin_amdgcn_udot4(xc[u][s].z, xc[u][s].z, xx[u], false);
                  xx[u] = __builtin_amdgcn_udot4(xc[u][s].w, xc[u][s].w, xx[u], false);
                  xq[u] = __builtin_amdgcn_udot4(xc[u][s].x, qc[s].x, xq[u], false);
                  xq[u] = __builtin_amdgcn_udot4(xc[u][s].y, qc[s].y, xq[u], false);
                  xq[u] = __builtin_amdgcn_udot4(xc[u][s].z, qc[s].z, xq[u], false);
                  xq[u] = __builtin_amdgcn_udot4(xc[u][s].w, qc[s].w, xq[u], false);
                } else {
                  const float t0 = __uint_as_float(xc[u][s].x) - __uint_as_float(qc[s].x);
                  const float t1 = __uint_as_float(xc[u][s].y) - __uint_as_float(qc[s].y);
                  const float t2 = __uint_as_float(xc[u][s].z) - __uint_as_float(qc[s].z);
                  const float t3 = __uint_as_float(xc[u][s].w) - __uint_as_float(qc[s].w);
                  fa = fmaf(t0, t0, fa);
                  fa = fmaf(t1, t1, fa);
                  fa = fmaf(t2, t2, fa);
                  fa = fmaf(t3, t3, fa);
                }
              }
              if (!IS_U8) {
                fa += __shfl_xor(fa, 1);
                fa += __shfl_xor(fa, 2);
                fa += __shfl_xor(fa, 4);
                fs[u] = sl == 0 ? fa : fs[u] + fa;
              }
            }
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            if (IS_U8) {
              // integer sums: the slab order does not matter
              int32_t part = (int32_t)xx[u] - 2 * (int32_t)xq[u];
              part += __shfl_xor(part, 1);
              part += __shfl_xor(part, 2);
              part += __shfl_xor(part, 4);
              key[u] = (uint32_t)(part + qq);
            } else {
              key[u] = __float_as_uint(fs[u]);
            }
          }
        } else {
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (ok[u] && gl == 0) nbytes += (uint32_t)rb;
        uint4 xv[U][NSEG];
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
          for (int s = 0; s < NSEG; ++s) {
            const int off = 128 * s + 16 * gl;
            xv[u][s] = (ok[u] && off < rb) ? load_payload(a.ra.seg(phys[u], off))
                                           : make_uint4(0, 0, 0, 0);
          }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
          if (IS_U8) {
            uint32_t xx = 0, xq = 0;
#pragma unroll
            for (int s = 0; s < NSEG; ++s) {
              xx = __builtin_amdgcn_udot4(xv[u][s].x, xv[u][s].x, xx, false);
              xx = __builtin_amdgcn_udot4(xv[u][s].y, xv[u][s].y, xx, false);
              xx = __builtin_amdgcn_udot4(xv[u][s].z, xv[u][s].z, xx, false);
              xx = __builtin_amdgcn_udot4(xv[u][s].w, xv[u][s].w, xx, false);
              xq = __builtin_amdgcn_udot4(xv[u][s].x, qv[s].x, xq, false);
              xq = __builtin_amdgcn_udot4(xv[u][s].y, qv[s].y, xq, false);
              xq = __builtin_amdgcn_udot4(xv[u][s].z, qv[s].z, xq, false);
              xq = __builtin_amdgcn_udot4(xv[u][s].w, qv[s].w, xq, false);
            }
            int32_t part = (int32_t)xx - 2 * (int32_t)xq;
            part += __shfl_xor(part, 1);
            part += __shfl_xor(part, 2);
            part += __shfl_xor(part, 4);
            key[u] = (uint32_t)(part + qq);
          } else {
            float acc = 0.0f;
#pragma unroll
            for (int s = 0; s < NSEG; ++s) {
              float t0 = __uint_as_float(xv[u][s].x) - __uint_as_float(qv[s].x);
              float t1 = __uint_as_float(xv[u][s].y) - __uint_as_float(qv[s].y);
              float t2 = __uint_as_float(xv[u][s].z) - __uint_as_float(qv[s].z);
              float t3 = __uint_as_float(xv[u][s].w) - __uint_as_float(qv[s].w);
              acc = fmaf(t0, t0, acc);
              acc = fmaf(t1, t1, acc);
              acc = fmaf(t2, t2, acc);
              acc = fmaf(t3, t3, acc);
            }
            acc += __shfl_xor(acc, 1);
            acc += __shfl_xor(acc, 2);
            acc += __shfl_xor(acc, 4);
            key[u] = __float_as_uint(acc);
          }
        }
        }
        // rows that may enter the top-k
        const uint32_t left = vend - vb;
        ltopk_step<U>(tk, k, key, left, a.row_ids, [&]() -> uint32_t {
          uint32_t p = (uint32_t)phys[0];
#pragma unroll
          for (int u = 1; u < U; ++u) p = gl == u ? (uint32_t)phys[u] : p;
          return p;
        });
      }
      v = vend;
      c += ns;
      __builtin_amdgcn_wave_barrier();
    }
    // partial result of this tile: the ids not read yet, all at once
    if (lane < tk.cnt && tk.id == UNREAD) tk.id = (uint32_t)a.row_ids[tk.phys];
    if (lane < k) {
      a.pkey[(int64_t)t * k + lane] = lane < tk.cnt ? tk.key : 0xffffffffu;
      a.pid[(int64_t)t * k + lane] = lane < tk.cnt ? (int64_t)tk.id : -1;
    }
    if (total <= nwaves) break;
    t = next_tile();
  }
  if (a.rbytes) {
    for (int m = 1; m < WAVE; m <<= 1) nbytes += shfl_xor_u64(nbytes, m);
    if (lane == 0 && nbytes) atomicAdd(a.rbytes, nbytes);
  }
}

template <int IS_U8>
static hipError_t launch_refine_t(const RefineArgs &a, int nseg, int grid, hipStream_t s) {
#define NR_REFINE_CASE(NS, UU)                                                     \
  if (nseg <= NS) {                                                                \
    hipLaunchKernelGGL((k_refine<IS_U8, NS, UU>), dim3(grid), dim3(256), 0, s, a); \
    return hipGetLastError();                                                      \
  }
  NR_REFINE_CASE(1, NR_REFINE_U1)
  NR_REFINE_CASE(2, 4)
  NR_REFINE_CASE(3, 4)
  NR_REFINE_CASE(4, 2)
  NR_REFINE_CASE(8, 1)
  NR_REFINE_CASE(16, 2)
  NR_REFINE_CASE(48, 2)
#undef NR_REFINE_CASE
  return hipErrorInvalidValue;
}

hipError_t launch_refine(const RefineArgs &a, int dtype, int n_cu, int blocks_per_cu,
                         hipStream_t s) {
  if (a.nq <= 0) return hipSuccess;
  const int nseg = (a.row_bytes + 127) / 128;
  const int grid = n_cu * (blocks_per_cu > 0 ? blocks_per_cu : NR_REFINE_BLOCKS_PER_CU);
  return dtype == NR_U8 ? launch_refine_t<1>(a, nseg, grid, s) : launch_refine_t<0>(a, nseg, grid, s);
}

// ------------------------------------------------------------------ merge
__global__ void __launch_bounds__(256) k_merge(MergeArgs a) {
  const int lane = lane_id();
  const int64_t q = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (q >= a.nq) return;
  if (a.qmask && !a.qmask[q]) return;
  const int k = a.k;
  const int64_t e0 = (int64_t)a.tile_off[q] * k, e1 = e0 + (int64_t)a.ntile[q] * k;
  // (key, id) in one word (ids are below 2^32, -1 is an empty entry).  The
  // tiles' lists are sorted; those of as many tiles as fit 64 lanes are sorted
  // together, then merged with the best so far
  uint64_t best = ~0ull;
  const int64_t step = (int64_t)(WAVE / k) * k;
  for (int64_t i0 = e0; i0 < e1; i0 += step) {
    const int64_t i = i0 + lane;
    uint64_t v = ~0ull;
    if (lane < step && i < e1) {
      const int64_t id = a.pid[i];
      if (id >= 0) v = ((uint64_t)a.pkey[i] << 32) | (uint32_t)id;
    }
    if (step > k) v = wave_sort_u64(v);
    best = i0 == e0 ? v : wave_merge_least_u64(best, v);
  }
  if (lane < k) {
    const bool have = best != ~0ull;
    const uint32_t key = (uint32_t)(best >> 32);
    a.out_ids[q * k + lane] = have ? (int64_t)(uint32_t)best : -1;
    // (the shared schedule's seed keeps its keys: a uint8 row's is exact, fp32 is not past 2^24)
    a.out_dists[q * k + lane] =
        have ? (a.is_u8 && !a.qrec ? (float)key : __uint_as_float(key)) : INFINITY;
  }
  // The scan's record of the query: its bound (the k-th key of the seed pass,
  // or all ones while that list is short), the bound the head test compares
  // with, and |q|^2 for uint8 rows.  uint8 keys are integers, so the head bound
  // is the key minus |q head|^2 (a row's head part of the distance is |x_h|^2 -
  // 2 x_h.q_h + |q_h|^2); fp32 rows keep a relative margin of 1e-4 over the key
  // for the rounding of the head's partial sum.
  if (a.qrec && lane == k - 1) {
    const uint32_t bound = (uint32_t)(best >> 32);   // an empty entry's is all ones
    uint4 r = make_uint4(bound, 0u, 0u, 0u);
    if (a.is_u8) {
      const uint2 qn = a.qnorm[q];
      r.y = (uint32_t)(bound == 0xffffffffu ? INT32_MAX
                                            : (int32_t)((int64_t)bound - (int64_t)qn.y));
      r.z = qn.x;
    } else {
      r.y = bound == 0xffffffffu ? __float_as_uint(INFINITY)
                                 : __float_as_uint(__uint_as_float(bound) * 1.0001f);
    }
    a.qrec[q] = r;
  }
  if (lane == 0 && a.qstats) {
    a.qstats[q * NR_QSTATS + NR_QS_ROWS] = (int32_t)a.rtot[q];
    a.qstats[q * NR_QSTATS + NR_QS_TILES] = a.ntile[q];
  }
}

hipError_t launch_merge(const MergeArgs &a, hipStream_t s) {
  if (a.nq <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_merge, dim3((unsigned)((a.nq + 3) / 4)), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace nr
