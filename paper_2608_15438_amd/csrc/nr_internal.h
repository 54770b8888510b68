// Internal declarations of the gfx950 search library: kernel argument
// structs, launch wrappers and wave64 helpers.  Not part of the ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "neuroute.h"

namespace nr {

constexpr int WAVE = 64;
#ifndef NR_MAX_TILES_PER_QUERY
#define NR_MAX_TILES_PER_QUERY 64
#endif
constexpr int MAX_TILES_PER_QUERY = NR_MAX_TILES_PER_QUERY;  // refinement tiles per query
#ifndef NR_TILE_MIN_ROWS
#define NR_TILE_MIN_ROWS 512
#endif
constexpr int TILE_MIN_ROWS = NR_TILE_MIN_ROWS;  // smallest refinement tile
constexpr int STAGE_CLUSTERS = 128;       // clusters staged in LDS per refinement wave
constexpr int64_t QUERY_CHUNK = 16384;    // queries per internal launch sequence
// rows per launch of an encoder that holds no activations: a one-layer encoder
// takes 8 threads a row, and a launch fewer than 2^32
constexpr int64_t ENCODE_ROWS = (int64_t)1 << 26;
#ifndef NR_OWN_TILE_MIN_ROWS
#define NR_OWN_TILE_MIN_ROWS 2048
#endif
constexpr uint32_t OWN_TILE_MIN_ROWS = NR_OWN_TILE_MIN_ROWS;  // smallest tile of the own pass
// Rows of a query's first clusters that it refines on its own before the
// shared scan: about 1 / div of the rows its list holds (estimated from the
// mean size of its first 64 clusters), within [lo, hi].  More seed rows give
// tighter bounds (fewer survivors of the scan, and for uint8 rows fewer rows
// that pass the head test) but are read once per query instead of once per
// batch, and the rows that the bound acts on grow with the list.  fp32 heads
// drop few rows, so fp32 seeds are the smaller; uint8 rows past 1 KB keep 1024.
// The bound is the seed's k-th key, so a large k needs SEED_ROWS_PER_K rows per
// neighbour: with 8, the survivors of k = 64 flooded their lists.  Whole searches
// on MI355X with seeds of 256 / 512 / 1024 / 2048 / 4096 rows, ms:
//   fp32, k = 10:   25M x 96 (11k rows a list) 3.62 / 3.51 / 3.65 / 4.2 / 4.89, 1M x 200 (9k)
//                   2.07 / 2.15 / 2.39 / 2.98 / 4.10, 500k x 768 (9k) 14.8 / 3.26 / 3.00 /
//                   3.68 / 5.46, 500k x 1536 (4k) 1.16 / 1.27 / 1.63 / - / -
//   uint8, k = 10:  4M x 256 (14k) 1.56 / 1.47 / 1.46 / 1.62 / 1.92, 32M x 128 (23k) 5.41 /
//                   3.16 / 2.86 / 2.97 / 3.12, 256M x 128 (56k) 8.5 / 6.3 / 5.5 / 5.17 / 5.04
//   k = 64:         1M x 100 fp32 2.91 / 2.01 / 1.96 / 2.15 / 2.65, 4M x 256 uint8 7.85 /
//                   2.63 / 1.82 / 1.88 / 2.15, 500k x 1536 fp32 20 / 18 / 4.75 / 4.29 / 5.89
// Short lists: a scan costs some 150 us however little it is left, so a batch of
// short lists goes best without one.  Where the lists of rows of at most 1 KB
// (probe budget x mean bucket) come to at most SEED_WHOLE bytes, a query reads up
// to 4096 rows of its own; past that, uint8 lists estimated at most `brief` rows
// long take 2 lo (1M x 128 in clusters of three, 725 rows a list: 0.78 ms, but 0.95
// ms with the few lists past 1024 rows in the scan).  1M rows in 8192 buckets, us:
//   fp32, seeds of 512 / 4096 rows:
//     d = 96:  3,000 queries of 1.0k rows (0.8 GB) 514 / 338, 1.5k (1.3 GB) 566 / 440, 2.7k
//              (2.2 GB) 638 / 754; 10,000 of 1.0k (2.8 GB) 831 / 781, 1.5k (4.2 GB) 925 / 1087;
//              700 of 1.5k (0.3 GB) 355 / 221, 5.3k (1.1 GB) 494 / 466
//     d = 32:  3,000 of 1.4k (0.3 GB) 786 / 344, 5.2k (1.2 GB) 829 / 783; 10,000 of 1.4k
//              (0.9 GB) 970 / 632, 2.7k (1.9 GB) 1026 / 1086
//     d = 256: 512 of 1.3k (0.6 GB) 356 / 407, 2.8k (1.3 GB) 453 / 511; 3,000 of 0.9k (2.3 GB)
//              619 / 630
//   uint8, seeds by div and brief / of 4096 rows:
//     d = 128: 10,000 of 2.7k (1.9 GB) 920 / 853, 4.7k (3.7 GB) 1044 / 1191; 1,000 of 9.7k
//              (0.9 GB) 510 / 378, 19k (1.9 GB) 436 / 428
//     d = 256: 512 of 7.1k (0.6 GB) 570 / 567; 700 of 12k (1.6 GB) 636 / 648
//   Longer rows gain nothing from it (500k x 768, 512 queries of 1.1k rows 542 / 688).
struct SeedRule {
  uint32_t lo, hi, div, brief;  // div 0: lo rows whatever the list
};
constexpr uint32_t SEED_ROWS_PER_K = 32;
constexpr double SEED_WHOLE = 1.5e9;
// list_bytes: the bytes of all lists' rows together, about
inline SeedRule seed_rule(bool is_u8, int row_bytes, int k, double list_bytes) {
  SeedRule r{512, 4096, 24, 0};
  if (row_bytes <= 1024 && list_bytes <= SEED_WHOLE) r = SeedRule{4096, 4096, 0, 0};
  else if (is_u8) r = row_bytes > 1024 ? SeedRule{1024, 1024, 0, 0} : SeedRule{1024, 4096, 12, 8192};
  const uint32_t by_k = SEED_ROWS_PER_K * (uint32_t)k;
  if (r.lo < by_k) r.lo = by_k;
  if (r.hi < r.lo) r.hi = r.lo;
  return r;
}
#ifndef NR_SURVIVOR_CAP
#define NR_SURVIVOR_CAP 2048
#endif
constexpr int SURVIVOR_CAP = NR_SURVIVOR_CAP;  // survivors a query keeps in its own slots
#ifndef NR_SURVIVOR_POOL
#define NR_SURVIVOR_POOL (1u << 22)
#endif
constexpr uint32_t SURVIVOR_POOL = NR_SURVIVOR_POOL;  // survivors past SURVIVOR_CAP, all queries
#ifndef NR_OPEN_PAIRS
#define NR_OPEN_PAIRS (1u << 22)
#endif
constexpr uint32_t OPEN_PAIRS = NR_OPEN_PAIRS;  // fp32 rows past 1 KB: pairs open after slab 0
// The persistent kernels take their tiles from TILE_COUNTERS counters, each in
// a 128-byte line of its own, a wave always from the same one.  One counter
// answers an atomic in 12 ns: 8192 waves asking it once took 100 us, however
// little there was to do.
constexpr int TILE_COUNTERS = 16, TILE_COUNTER_STRIDE = 32;
constexpr int SHARED_G = 8;               // queries scored per shared work unit (at most)
constexpr int SHARED_MAX_NSEG = 48;       // rows of at most 48 x 128 bytes use the shared scan
constexpr uint32_t SHARED_ROWS = 2048;    // rows per shared work unit (at most)
constexpr int MAX_KC = 16384;             // top-K_c heap held in LDS
// the shared schedule's scan-list build: LIST_WPT words of 32 pair counts per
// thread; the counts array is hist_words long (whole words, and at least
// n_clusters + 1 counts)
constexpr int LIST_WPT = 1;
constexpr int LIST_THREADS = 256;
__host__ __device__ inline int64_t list_words(int64_t n_clusters) { return (n_clusters + 31) / 32; }
__host__ __device__ inline int64_t hist_words(int64_t n_clusters) {
  return (list_words(n_clusters) + 1) * 32;
}
__host__ __device__ inline int64_t list_blocks(int64_t n_clusters) {
  const int64_t per = (int64_t)LIST_WPT * LIST_THREADS;
  const int64_t b = (list_words(n_clusters) + per - 1) / per;
  return b > 0 ? b : 1;
}

// ---------------------------------------------------------------- kernels
// Addressing of the permuted payload: bytes [0, h) of row r at hb + r * hs,
// bytes [h, row_bytes) at tb + r * ts.  Row-major: hb = tb - h = rows,
// hs = ts = row_bytes.  Split layout: a head plane then a tail plane.
struct RowAddr {
  const unsigned char *hb;
  const unsigned char *tb;
  uint64_t hs, ts;
  int h;
  __device__ __forceinline__ const uint4 *seg(uint64_t r, int off) const {
    return off < h ? reinterpret_cast<const uint4 *>(hb + r * hs + off)
                   : reinterpret_cast<const uint4 *>(tb + r * ts + (off - h));
  }
};

struct EncodeLayerArgs {
  const void *in;        // [M x K]: uint8 or fp32 (layer 0) / fp32 activations
  int in_u8;
  float *out;            // [M x N] fp32
  const float *W;        // [N x K] row-major
  const float *bias;     // [N]
  const float *bn_scale; // [N] or null
  const float *bn_shift; // [N] or null
  float in_scale;
  int relu;
  int64_t M;
  int N, K;
};

// words that a search sets to zero before its first use of them: the probe
// kernel, which runs before every other kernel of the search but the encoder,
// clears them on its way (seven fills took 5 us each)
struct ZeroArgs {
  int32_t *per_query[2];  // [nq] each, may be null
  int32_t *p[6];
  int n[6];               // words at p[i]
};

struct ProbeArgs {
  ZeroArgs zero;
  const float *logits;   // [nq x b]
  const float *tau;      // [b]
  int64_t nq;
  int b, l_sel, r_max, P, n_bins, finite;
  float s_max, bin_scale;
  uint32_t *codes;       // [nq x P]
  float *costs;
  int32_t *bins;
  int32_t *counts;       // [nq]
  // optional, for the search: each probe's bucket looked up in the directory
  // (lk[q x P + i] = [bc_off[code], bc_off[code + 1])) and each query's route
  // pass (see route_tiers; tier[q] = the first pass whose heap holds the
  // summed sizes of its multi-cluster buckets)
  const uint32_t *bc_off;
  uint2 *lk;             // [nq x P] (NULL: no lookup)
  int32_t *tier;         // [nq] (NULL: no tiers)
  int tier_n, tier_h0, tier_h1;
};

// calibration (k_calib.hip): bucket scores of the targets and margin points
struct CalibArgs {
  const float *logits;          // [nq x b]
  const float *tau;             // [b]
  int64_t nq, n;
  int b, l_sel, r_max, K;
  const int64_t *targets;       // [nq x K] original ids, < 0: none
  const uint32_t *row_of_id;    // [n] permuted row of each original id
  const uint64_t *cl_off;       // [n_clusters + 1]
  int64_t n_clusters, n_codes;  // n_codes = 2^b
  const uint32_t *bc_off;       // [n_codes + 1]
  const float *centroids;       // [n_clusters x b]
  float *scores;                // [nq x K]
  float *xy;                    // [nq x 2]
};

// per-query pair counting of the shared schedule (see pair_hist_wave)
struct PairHistArgs {
  uint32_t *hist;               // [n_clusters + 1] pairs per cluster past the leading clusters
  const uint64_t *cl_off;
  int64_t n_clusters;
  SeedRule seed;                // rows the leading clusters cover at least
  int32_t *cseed;               // [nq] leading clusters
  uint32_t *rfull;              // [nq] rows of the leading clusters (whole list: eager_rows)
  uint2 *qnorm;                 // [nq] uint8 rows: |q|^2 and its head part
  const unsigned char *queries;
  int row_bytes, scan_head, is_u8, eager_rows;
  uint32_t *pair_rank;          // [nq x cap] each counted pair's rank among its cluster's pairs
  int64_t cap;
};

struct RouteArgs {
  const float *logits;
  int64_t nq;
  int b, P;
  const int32_t *bins;
  const int32_t *counts;
  uint2 *lk;             // [nq x P] cluster range of each probe's bucket (written by k_probe)
  int pst;               // probes per query whose ranges are staged in LDS (set per pass)
  int hcap, pass;        // heap slots in LDS and pass number (set by launch_route)
  int tiered;            // redo[q] holds the pass that routes query q
  int32_t *redo;         // [nq] the pass of each query (written by k_probe when tiered)
  const float *centroids;
  int k_c, b_batch, b_min, t_low, u_heap, u_front;
  float alpha_front;
  int gate_on, early_stop_on, lowq_or, finite;
  int m_knots;
  float m_x[NR_MAX_KNOTS], m_y[NR_MAX_KNOTS], m_slope[NR_MAX_KNOTS];
  uint32_t *clus;        // [nq x cap]
  int32_t *nclus;        // [nq]
  int64_t cap;
  int32_t *qstats;       // [nq x NR_QSTATS] or null
  int unordered;         // the order of H's clusters in the list does not matter
  PairHistArgs ph;       // with ph_on: each query's pairs are counted once its list is final
  int ph_on;
};

struct PlanArgs {
  int64_t nq;
  const uint32_t *clus;
  const int32_t *nclus;
  int64_t cap;
  const uint64_t *cl_off;
  int64_t n_clusters;    // cluster ids >= n_clusters count as empty
  uint32_t *rowpre;      // [nq x (cap + 1)]
  uint32_t *rtot;        // [nq]
  uint32_t *tsize;       // [nq]
  int32_t *ntile;        // [nq]
  int32_t *tile_off;     // [nq + 1] first tile of each query; [nq]: tiles (zero before)
  int32_t *tile_q;       // [nq x MAX_TILES_PER_QUERY]
  int32_t *tile_c0;
  uint32_t *rfull;       // [nq] rows of the whole list, may be null
  const int32_t *qmask;  // [nq] only queries with qmask[q] != 0 get tiles, may be null
  const int32_t *own_cseed;  // [nq] may be null; else only list positions i < own_cseed[q] count
  uint32_t *clus_out;        // with own_cseed: [nq x cap] the clusters that count, compacted
  int32_t *nclus_out;        // [nq]
  uint32_t tile_min;         // smallest tile (rows); 0: TILE_MIN_ROWS
};

struct RefineArgs {
  RowAddr ra;            // permuted payload
  const int64_t *row_ids;
  const uint64_t *cl_off;
  int64_t n_clusters;
  const void *queries;   // [nq x d]
  int64_t nq;
  int d, row_bytes, k;
  const uint32_t *clus;
  const int32_t *nclus;
  int64_t cap;
  const uint32_t *rowpre;
  const uint32_t *rtot;
  const uint32_t *tsize;
  const int32_t *tile_off;
  const int32_t *tile_q;
  const int32_t *tile_c0;
  int32_t *counter;
  uint32_t *pkey;        // [nq x MAX_TILES_PER_QUERY x k]
  int64_t *pid;
  unsigned long long *rbytes;  // row bytes the kernel read (added to)
};

struct MergeArgs {
  int64_t nq;
  int k, is_u8;
  const int32_t *tile_off, *ntile;
  const uint32_t *pkey;
  const int64_t *pid;
  const uint32_t *rtot;
  int64_t *out_ids;
  float *out_dists;
  int32_t *qstats;
  const int32_t *qmask;  // only queries with qmask[q] != 0 are written, may be null
  uint4 *qrec;           // [nq] the shared scan's record of each query, may be null; with it,
                         // out_dists gets the keys' bits
  const uint2 *qnorm;    // [nq] uint8 rows, with qrec
};

// batch-shared refinement: a candidate row listed by several queries of the
// batch is read once and scored for all of them
struct SharedArgs {
  int64_t nq;
  int k, is_u8, row_bytes;
  int g;                      // queries per work unit (SHARED_G)
  SeedRule seed;              // rows the leading clusters of a list cover at least
  int64_t n_clusters;
  RowAddr ra;                 // permuted payload
  int scan_head;              // bytes of each row the scan's filter reads (its head)
  const unsigned char *scan_hb;  // head of row r at scan_hb + r * scan_hs
  uint64_t scan_hs;
  const int64_t *row_ids;
  const uint64_t *cl_off;
  const void *queries;
  const uint32_t *clus;
  const int32_t *nclus;
  int64_t cap;
  int32_t *cseed;             // [nq] leading clusters, scored by the query's own (seed) pass
  uint32_t *rfull;            // [nq] rows of the whole list
  const uint32_t *rtot;       // [nq] rows of the own pass
  int32_t *tile_off;          // [nq + 1] tiles of the own pass ([nq]: how many)
  int32_t *own_counter;       // [TILE_COUNTERS x TILE_COUNTER_STRIDE] of the own pass
  const int64_t *own_ids;     // [nq x k] top-k of the own pass (sorted)
  const float *own_dists;     // its keys (fp32 distances, or the bits of uint8 rows' whole ones)
  uint32_t *own_rows;         // [nq] copy of rtot kept for diagnostics
  uint32_t *hist;             // [n_clusters + 1] pairs per cluster past the leading clusters
  uint32_t *pair_rank;        // [nq x cap] rank of each counted pair among its cluster's pairs
  uint32_t *hpos;             // [n_clusters] start of cluster c's pairs in pair_q (clusters
                              // with pairs only)
  uint32_t *slist;            // [n_clusters] the scan list: clusters with pairs, in order
  uint32_t *lpair, *lpm;      // [list] start in pair_q and number of pairs of entry i
  uint64_t *lbase;            // [list] first payload row of entry i's cluster
  uint32_t *lsz;              // [list] rows of entry i's cluster
  uint64_t *swork_off;        // [list + 1] start of entry i in the work space
  uint64_t *lmeta;            // [4] list length, pairs, work
  uint32_t *thr_n, *thr_h;    // [list_blocks x LIST_THREADS] per-thread sums of the prep
  uint64_t *thr_w;
  uint32_t *blk_n, *blk_h;    // [list_blocks] per-block sums, then their offsets
  uint64_t *blk_w;
  int eager_rows;             // 1: rfull gets the rows of the whole list (else the leading ones)
  uint32_t *pair_q;           // [pairs] query of each scanned pair, grouped by cluster
  uint2 *qnorm;               // [nq] uint8 rows: (|q|^2, |q head|^2 over scan_head bytes)
  uint4 *qrec;                // [nq] the scan's record of a query, written after the seed
                              // merge: (bound key, head threshold, |q|^2, 0)
  int32_t *scnt;              // [nq] survivors appended
  uint32_t *skey;             // [nq x SURVIVOR_CAP]
  int64_t *sid;
  int32_t *flag;              // [nq] 1: survivors lost (pool full), recompute per query
  unsigned long long *pool_cnt;  // survivors appended to the pool
  uint32_t *pool_q, *pool_key;   // [SURVIVOR_POOL] query and key of pooled survivors
  int64_t *pool_id;
  uint32_t *poff;             // [nq + 1] per-query start of its pooled survivors in pool2
  uint32_t *pcur;             // [nq] scatter cursors
  uint32_t *pool2_key;        // [SURVIVOR_POOL] pooled survivors grouped by query
  int64_t *pool2_id;
  unsigned long long *open_cnt;  // fp32 rows past 1 KB: (query, row) pairs still at or
  uint32_t *open_q, *open_key;   // before the bound after the first 1 KB slab, their
  uint64_t *open_row;            // running sum and payload row [OPEN_PAIRS]
  uint32_t *counter;  // [TILE_COUNTERS x TILE_COUNTER_STRIDE] tile counters
  int64_t *wstats;            // [7] scanned rows, seed tiles, scanned pair rows, rows read
                              // past their heads, bytes the scan read from them, row
                              // bytes of the open-pair pass, row bytes of k_refine
  int64_t *out_ids;
  float *out_dists;
  int32_t *qstats;
};


hipError_t launch_encode_layer(const EncodeLayerArgs &a, hipStream_t s);
// layers a (hidden, K -> N) and z (codes, N -> NZ) in one kernel: whether M
// rows should go there, and the launch
bool encode_pair(int64_t M, int K, int N, int NZ, bool u8);
hipError_t launch_encode_pair(const EncodeLayerArgs &a, const EncodeLayerArgs &z, hipStream_t s);
hipError_t launch_probe(const ProbeArgs &a, hipStream_t s);
constexpr int ROUTE_LIGHT_HEAP = 512;  // heap slots of the route's first pass
constexpr int ROUTE_MID_HEAP = 2048;   // and of its second when K_c is larger still
// the heap sizes of the route's passes for K_c: one pass of K_c keys up to
// ROUTE_LIGHT_HEAP, else ROUTE_LIGHT_HEAP, ROUTE_MID_HEAP (when K_c is larger
// still) and K_c; returns the number of passes
inline int route_tiers(int k_c, int tiers[3]) {
  if (k_c <= ROUTE_LIGHT_HEAP) {
    tiers[0] = k_c;
    return 1;
  }
  int nt = 0;
  tiers[nt++] = ROUTE_LIGHT_HEAP;
  if (k_c > ROUTE_MID_HEAP) tiers[nt++] = ROUTE_MID_HEAP;
  tiers[nt++] = k_c;
  return nt;
}
size_t route_lds_bytes(int k_c, int pst);
// aux, fork, join (may be null): a second stream and two events, on which the
// passes with larger heaps run beside the first
hipError_t launch_route(const RouteArgs &a, hipStream_t s, hipStream_t aux = nullptr,
                        hipEvent_t fork = nullptr, hipEvent_t join = nullptr);
hipError_t launch_plan(const PlanArgs &a, hipStream_t s);
// blocks_per_cu: 0 for the tuned default; fewer leave room on every CU for
// work on another stream (the scan's preparation beside the seed pass)
hipError_t launch_refine(const RefineArgs &a, int dtype, int n_cu, int blocks_per_cu,
                         hipStream_t s);
hipError_t launch_merge(const MergeArgs &a, hipStream_t s);
// fresh: the workspace is new, so clear the pair counts
hipError_t launch_shared_hist(const SharedArgs &a, bool fresh, hipStream_t s);
PairHistArgs pair_hist_args(const SharedArgs &a);
hipError_t launch_shared_prep(const SharedArgs &a, hipStream_t s);
hipError_t launch_shared_refine(const SharedArgs &a, int dtype, int n_cu, hipStream_t s);
// the open pairs' remaining slabs (fp32 rows past 1 KB; a no-op otherwise)
hipError_t launch_scan_open(const SharedArgs &a, int dtype, int n_cu, hipStream_t s);
hipError_t launch_shared_merge(const SharedArgs &a, hipStream_t s);
hipError_t launch_unique_rows(const uint32_t *slist, const uint32_t *lpm, const uint64_t *lmeta,
                              const uint64_t *cl_off, int64_t *out, hipStream_t s);
hipError_t launch_list_rows(const uint32_t *clus, const int32_t *nclus, int64_t cap, int64_t nq,
                            const uint64_t *cl_off, int64_t n_clusters, uint32_t *rows,
                            hipStream_t s);
hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t s);

hipError_t launch_inverse_perm(const int64_t *row_ids, int64_t n, uint32_t *row_of_id,
                               hipStream_t s);
hipError_t launch_calib(const CalibArgs &a, hipStream_t s);
// index construction (k_build.hip)
struct BuildArgs {
  int64_t n;
  int b;
  const float *lg;            // [n x b] latents by original id
  const uint32_t *codes;      // [n]
  const uint32_t *sizes;      // [2^b]
  int rule;
  uint32_t t;
  uint32_t *kb, *multi, *mpos, *mlist;   // [2^b] (+1 for the scans)
  unsigned long long *stats;  // [3] sum kb, multi buckets, max kb
  uint64_t *blk;              // scan scratch [build_scan_blocks(max items)]
  uint64_t *kbpre, *boff;     // [2^b + 1]
  uint32_t *cursor, *nkept, *ncl;        // [2^b] (+1)
  uint32_t *ids, *ids_tmp, *label;       // [n]
  uint64_t *skey, *skey_tmp;  // [n]
  double *d2;                 // [n]
  int64_t n_multi;
  const double *U;            // [n_multi x kmax]
  int kmax;
  uint32_t seed;
  int lloyd, spc;
  int64_t slots;              // max_clusters: cluster slots of all buckets
  double *cent;               // [slots x build_pad(b)]
  uint32_t *ccnt;             // [slots]
  uint4 *slot;                // [slots]
  uint32_t *changed;          // [2^b]
  uint32_t *list_mid, *list_big;  // [n / 64 + 1], [n / 256 + 1] buckets by size
  uint32_t *counts;           // [5] the lists' lengths and the number of tiles
  uint2 *tile;                // [n / 64 + n_multi + 1]
  uint32_t *bc_off;           // [2^b + 1] out
  int64_t *row_ids;           // [n] out
  uint64_t *csize;            // [max_clusters]
  float *centroids;           // [max_clusters x b] out
};
size_t build_scan_blocks(int64_t n);
int build_pad(int b);  // doubles per centre: b rounded up to a multiple of 4
size_t build_tau_ws(int64_t ns, int b);
hipError_t launch_build_tau(const float *lg, int64_t ns, int b, float *tau, void *ws,
                            hipStream_t s);
hipError_t launch_build_codes(const float *lg, int64_t m, int b, const float *tau, uint32_t *codes,
                              uint32_t *sizes, hipStream_t s);
hipError_t launch_build_nonempty(const uint32_t *sizes, int64_t nb, unsigned long long *out,
                                 hipStream_t s);
hipError_t run_build_plan(const BuildArgs &a, hipStream_t s);
hipError_t run_build_index(const BuildArgs &a, hipStream_t s);
hipError_t launch_build_cl_off(const uint64_t *csize, int64_t n_clusters, uint64_t *cl_off,
                               uint64_t *blk, hipStream_t s);

// L_sim training (k_lsim.hip)
size_t pair_sqdist_ws_floats(int64_t B, int D);
hipError_t launch_pair_sqdist(const float *x, int64_t B, int D, float *ws, float *out,
                              hipStream_t s);
hipError_t launch_lsim_grad(const float *d2, const float *lat, int64_t B, int L, float gr,
                            float tau, const double *tau2, double *num_cnt, float *grad,
                            hipStream_t s);
size_t pair_quantile_ws_bytes();
hipError_t launch_pair_quantile(const float *d2, int64_t B, int64_t n, float q, void *ws,
                                double *out, hipStream_t s);

hipError_t launch_stream_read(const void *buf, int64_t bytes, uint32_t *sink, int n_cu,
                              hipStream_t s);

// index validation at upload; flags[0] |= error bits
hipError_t launch_validate(const uint32_t *bc_off, int64_t n_codes, const uint64_t *cl_off,
                           int64_t n_clusters, const int64_t *row_ids, int64_t n,
                           uint32_t *bitmap, int32_t *flags, hipStream_t s);

// ---------------------------------------------------------------- wave64 helpers
__device__ __forceinline__ int lane_id() { return __lane_id(); }

__device__ __forceinline__ uint32_t bcast_u32(uint32_t v, int src) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, src);
}
__device__ __forceinline__ float bcast_f32(float v, int src) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src));
}
__device__ __forceinline__ uint64_t bcast_u64(uint64_t v, int src) {
  uint32_t lo = bcast_u32((uint32_t)v, src), hi = bcast_u32((uint32_t)(v >> 32), src);
  return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m) {
  uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, m);
  uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), m);
  return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t shfl_u64(uint64_t v, int src) {
  uint32_t lo = (uint32_t)__shfl((int)(uint32_t)v, src);
  uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(v >> 32), src);
  return ((uint64_t)hi << 32) | lo;
}
__device__ __forceinline__ uint64_t ballot(bool p) { return __ballot(p); }
__device__ __forceinline__ int popc64(uint64_t m) { return __popcll(m); }
__device__ __forceinline__ uint64_t lanemask_lt() {
  int l = lane_id();
  return l == 0 ? 0ull : (~0ull >> (64 - l));
}
__device__ __forceinline__ float wave_min_f32(float v) {
  for (int m = 32; m >= 1; m >>= 1) v = fminf(v, __shfl_xor(v, m));
  return v;
}
// inclusive scans over the wave by DPP moves (shifts inside rows of 16 lanes,
// then row totals onto the rows after them; lanes a move leaves out add 0):
// six dependent VALU steps where shuffles wait for the LDS crossbar six times
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_incl_scan_u32(uint32_t v) {
  v += dpp_or_zero<0x111, 0xF>(v);  // row_shr:1, 2, 4, 8
  v += dpp_or_zero<0x112, 0xF>(v);
  v += dpp_or_zero<0x114, 0xF>(v);
  v += dpp_or_zero<0x118, 0xF>(v);
  v += dpp_or_zero<0x142, 0xA>(v);  // row_bcast:15 onto rows 1 and 3
  v += dpp_or_zero<0x143, 0xC>(v);  // row_bcast:31 onto rows 2 and 3
  return v;
}
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp_or_zero_u64(uint64_t v) {
  return ((uint64_t)dpp_or_zero<CTRL, ROWS>((uint32_t)(v >> 32)) << 32) |
         dpp_or_zero<CTRL, ROWS>((uint32_t)v);
}
__device__ __forceinline__ uint64_t wave_incl_scan_u64(uint64_t v) {
  v += dpp_or_zero_u64<0x111, 0xF>(v);
  v += dpp_or_zero_u64<0x112, 0xF>(v);
  v += dpp_or_zero_u64<0x114, 0xF>(v);
  v += dpp_or_zero_u64<0x118, 0xF>(v);
  v += dpp_or_zero_u64<0x142, 0xA>(v);
  v += dpp_or_zero_u64<0x143, 0xC>(v);
  return v;
}
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
  return bcast_u32(wave_incl_scan_u32(v), WAVE - 1);
}
// the value of lane l ^ M, by VALU moves (DPP inside a row of 16 lanes, row
// swaps across rows) rather than through the LDS crossbar, whose latency is
// most of a sorting network's
template <int M>
__device__ __forceinline__ uint32_t xor_lane(uint32_t v) {
  if constexpr (M == 1)
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xB1, 0xF, 0xF, false);
  else if constexpr (M == 2)
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4E, 0xF, 0xF, false);
  else if constexpr (M == 4) {  // mirror the half row, then each quad: l -> 7 - l -> l ^ 4
    const int h = __builtin_amdgcn_update_dpp((int)v, (int)v, 0x141, 0xF, 0xF, false);
    return (uint32_t)__builtin_amdgcn_update_dpp(h, h, 0x1B, 0xF, 0xF, false);
  } else if constexpr (M == 8)
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x128, 0xF, 0xF, false);
  else if constexpr (M == 16) {
    const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    return (lane_id() & 16) ? r[0] : r[1];
  } else {
    static_assert(M == 32, "a power of two below 64");
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (lane_id() & 32) ? r[0] : r[1];
  }
}
template <int M>
__device__ __forceinline__ uint64_t xor_lane_u64(uint64_t v) {
  return ((uint64_t)xor_lane<M>((uint32_t)(v >> 32)) << 32) | xor_lane<M>((uint32_t)v);
}
// compare-exchange with lane l ^ J: ascending inside blocks of K lanes whose
// bit K is clear
template <int K, int J>
__device__ __forceinline__ uint64_t sort_step(uint64_t key) {
  const int l = lane_id();
  const uint64_t o = xor_lane_u64<J>(key);
  return (((l & J) == 0) == ((l & K) == 0)) == (key < o) ? key : o;
}
template <int K, int J = K / 2>
__device__ __forceinline__ uint64_t sort_stage(uint64_t key) {
  key = sort_step<K, J>(key);
  if constexpr (J > 1) key = sort_stage<K, J / 2>(key);
  return key;
}
// ascending bitonic sort of one u64 key per lane, where every lane from n on
// holds ~0: only the first power of two >= n lanes need the network
__device__ __forceinline__ uint64_t wave_sort_u64(uint64_t key, int n = WAVE) {
  key = sort_stage<2>(key);
  if (n > 2) key = sort_stage<4>(key);
  if (n > 4) key = sort_stage<8>(key);
  if (n > 8) key = sort_stage<16>(key);
  if (n > 16) key = sort_stage<32>(key);
  if (n > 32) key = sort_stage<64>(key);
  return key;
}
// the 64 least of two ascending lists of 64 keys, ascending
__device__ __forceinline__ uint64_t wave_merge_least_u64(uint64_t a, uint64_t b) {
  // b reversed: rows mirrored (l -> l ^ 15), then l ^ 16, l ^ 32
  uint32_t lo = (uint32_t)b, hi = (uint32_t)(b >> 32);
  lo = (uint32_t)__builtin_amdgcn_update_dpp((int)lo, (int)lo, 0x140, 0xF, 0xF, false);
  hi = (uint32_t)__builtin_amdgcn_update_dpp((int)hi, (int)hi, 0x140, 0xF, 0xF, false);
  lo = xor_lane<32>(xor_lane<16>(lo));
  hi = xor_lane<32>(xor_lane<16>(hi));
  const uint64_t r = ((uint64_t)hi << 32) | lo;
  return sort_stage<64>(a < r ? a : r);
}
// number of entries of sorted a[0..n) strictly below key
__device__ __forceinline__ int lower_bound_u64(const uint64_t *a, int n, uint64_t key) {
  int lo = 0, hi = n;
  while (lo < hi) {
    int mid = (lo + hi) >> 1;
    if (a[mid] < key) lo = mid + 1; else hi = mid;
  }
  return lo;
}

// One wave, query q with list cl[0..n): the leading clusters covering at
// least the seed's rows stay with the query (cseed[q]); every later (cluster,
// query) pair is counted in hist (its rank among the cluster's pairs goes to
// pair_rank); rfull[q] gets the rows of the leading
// clusters (of the whole list with eager_rows); for uint8 rows qnorm[q] gets
// |q|^2 and the part of it over the scan's head.
__device__ inline void pair_hist_wave(const PairHistArgs &h, int64_t q, const uint32_t *cl, int n) {
  const int lane = lane_id();
  // rows of the leading clusters, and of the whole list when eager_rows is
  // set (otherwise the sizes of the later clusters are not needed here)
  const bool all = h.eager_rows != 0;
  uint64_t run = 0;
  int cs = -1;
  // the seed: sizes of the leading clusters until they cover its rows
  uint32_t seed_min = 0;
  for (int i0 = 0; i0 < n && (cs < 0 || all); i0 += WAVE) {
    const int i = i0 + lane;
    uint64_t sz = 0;
    if (i < n) {
      const uint32_t c = cl[i];
      if (c < h.n_clusters) sz = h.cl_off[(uint64_t)c + 1] - h.cl_off[c];
    }
    const uint64_t incl = wave_incl_scan_u64(sz);
    if (i0 == 0) {
      // the list's rows, from the mean size of its first clusters
      const uint64_t est = bcast_u64(incl, WAVE - 1) * (uint64_t)n / (uint64_t)(n < WAVE ? n : WAVE);
      const uint64_t want = h.seed.div > 0 ? est / h.seed.div : 0;
      seed_min = want > h.seed.hi ? h.seed.hi : (want < h.seed.lo ? h.seed.lo : (uint32_t)want);
      if (est <= h.seed.brief) seed_min = 2 * h.seed.lo;
    }
    int upto = WAVE - 1;
    if (cs < 0) {
      const uint64_t hit = ballot(i < n && run + incl >= seed_min);
      if (hit) {
        cs = i0 + __ffsll((unsigned long long)hit);  // first position past the seed
        if (!all) upto = cs - 1 - i0;
      }
    }
    run += bcast_u64(incl, upto);
  }
  // the pairs past the seed, four per lane at a time: their cluster ids are
  // all loaded, then all counted, so each group costs two memory round trips
  if (cs >= 0) {
    for (int i0 = cs; i0 < n; i0 += 4 * WAVE) {
      uint32_t c[4], r[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + u * WAVE + lane;
        c[u] = i < n ? cl[i] : 0xffffffffu;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) r[u] = c[u] < h.n_clusters ? atomicAdd(&h.hist[c[u]], 1u) : 0u;
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (c[u] < h.n_clusters) h.pair_rank[q * h.cap + i0 + u * WAVE + lane] = r[u];
    }
  }
  if (lane == 0) {
    h.cseed[q] = cs < 0 ? n : cs;
    h.rfull[q] = run > 0xffffffffull ? 0u : (uint32_t)run;
  }
  // uint8 rows: |q|^2 and the part of it over the scan's head (at most 128
  // bytes, so within lanes 0..7's first chunks), lane c taking the 16-byte
  // chunks c, c + 64, ...; integer sums, so the order of the additions does
  // not matter
  if (h.is_u8) {
    uint32_t p = 0, ph = 0;
    for (int c = lane; 16 * c < h.row_bytes; c += WAVE) {
      const uint4 v = *reinterpret_cast<const uint4 *>(h.queries +
                                                       (uint64_t)q * h.row_bytes + 16 * c);
      uint32_t t = 0;
      t = __builtin_amdgcn_udot4(v.x, v.x, t, false);
      t = __builtin_amdgcn_udot4(v.y, v.y, t, false);
      t = __builtin_amdgcn_udot4(v.z, v.z, t, false);
      t = __builtin_amdgcn_udot4(v.w, v.w, t, false);
      p += t;
      if (16 * c < h.scan_head) ph += t;
    }
    const uint32_t full = wave_sum_u32(p);
    const uint32_t head = wave_sum_u32(ph);
    if (lane == 0) h.qnorm[q] = make_uint2(full, head);
  }
}

}  // namespace nr
