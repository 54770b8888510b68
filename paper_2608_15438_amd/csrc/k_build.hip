// Index construction on the GPU (Sec. 3.3 "Bucket allocation" and
// "In-bucket clustering"; binarisation thresholds, Sec. 3.2.3), from the
// latents the encoder kernel gives the base rows:
//   tau      per latent dimension, the lower median of a sample of rows
//            (radix select on order-preserving keys);
//   codes    bit j of a row's code = [l_j >= tau_j] (Eq. 10) and the bucket
//            sizes (atomic counts);
//   buckets  exclusive scan of the sizes, an atomic scatter of the row ids into
//            bucket order, then every bucket's ids sorted ascending;
//   k-means  of the buckets with K_B >= 2 clusters: k-means++ on a sample (a
//            wave per small bucket, a block per larger one), then Lloyd passes
//            over the whole bucket (a wave per 64 members, then a wave per
//            cluster), in fp64 and in a fixed order of summation (below);
//   layout   clusters kept per bucket -> bc_off (scan), every bucket's rows in
//            (cluster, id) order -> row_ids, cluster sizes -> cl_off (scan),
//            centroids = fp64 means of the member latents (in id order),
//            rounded to fp32.
// The k-means follows the reading of "a limited number of k-means
// iterations" that the reference builder takes: the sample is the first
// min(|B|, spc K_B) members ordered by (mix32(id, seed), id); the first centre
// is its first member; each further centre is drawn with probability
// proportional to the integer weight floor(D^2 2^20) (capped at 2^30), by the
// bucket's pre-drawn uniform U: the first sample member whose running weight
// exceeds floor(U * total); squared distances add the dimensions in order;
// centroid sums add the members in id order.  Integer weights make the draws
// independent of summation order, so the result is the reference builder's.
#include "nr_internal.h"

namespace nr {

constexpr int BT = 256;               // threads per block of the build kernels
constexpr int SCAN_PER_THREAD = 16;   // items per thread of the scans
constexpr int64_t SCAN_BLOCK = (int64_t)BT * SCAN_PER_THREAD;
constexpr int SORT_LDS = 4096;        // keys sorted in LDS by one block
constexpr int64_t TAU_SMALL = 8192;   // sample rows from which the whole chip selects tau

// ------------------------------------------------------------------ helpers
__device__ __forceinline__ uint32_t mix32_dev(uint64_t x, uint32_t seed) {
  uint64_t h = (x ^ (uint64_t)seed) & 0xFFFFFFFFull;
  h = (((h >> 16) ^ h) * 0x45D9F3Bull) & 0xFFFFFFFFull;
  h = (((h >> 16) ^ h) * 0x45D9F3Bull) & 0xFFFFFFFFull;
  return (uint32_t)((h >> 16) ^ h);
}

__device__ __forceinline__ int64_t d2_weight(double d2) {
  double w = floor(d2 * 1048576.0);           // 2^20
  if (w > 1073741824.0) w = 1073741824.0;     // 2^30
  return (int64_t)w;
}

// block-wide exclusive scan of one value per thread (any integral T);
// *total gets the block's sum.  Uses `sh` (NT / WAVE entries).
template <class T, int NT = BT>
__device__ __forceinline__ T block_excl_scan(T v, T *sh, T *total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  T incl = v;
  for (int o = 1; o < WAVE; o <<= 1) {
    const T t = __shfl_up(incl, o);
    if (lane >= o) incl += t;
  }
  __syncthreads();
  if (lane == WAVE - 1) sh[w] = incl;
  __syncthreads();
  T before = 0, all = 0;
  for (int i = 0; i < NT / WAVE; ++i) {
    if (i < w) before += sh[i];
    all += sh[i];
  }
  *total = all;
  return before + incl - v;
}

// ------------------------------------------------------------------ scans
// out[i] = sum of in[0..i), out[n] = total, for n up to ~2^40 items.
template <class In>
__global__ void __launch_bounds__(BT) k_scan_sums(const In *in, int64_t n, uint64_t *blk) {
  __shared__ uint64_t sh[BT / WAVE];
  const int64_t base = (int64_t)blockIdx.x * SCAN_BLOCK + (int64_t)threadIdx.x * SCAN_PER_THREAD;
  uint64_t s = 0;
  for (int u = 0; u < SCAN_PER_THREAD; ++u)
    if (base + u < n) s += (uint64_t)in[base + u];
  uint64_t tot;
  (void)block_excl_scan<uint64_t>(s, sh, &tot);
  if (threadIdx.x == 0) blk[blockIdx.x] = tot;
}

__global__ void __launch_bounds__(BT) k_scan_top(uint64_t *blk, int64_t nblk) {
  __shared__ uint64_t sh[BT / WAVE];
  const int64_t per = (nblk + BT - 1) / BT;
  const int64_t b0 = (int64_t)threadIdx.x * per;
  const int64_t b1 = b0 + per < nblk ? b0 + per : nblk;
  uint64_t s = 0;
  for (int64_t b = b0; b < b1; ++b) s += blk[b];
  uint64_t tot;
  uint64_t run = block_excl_scan<uint64_t>(s, sh, &tot);
  for (int64_t b = b0; b < b1; ++b) {
    const uint64_t x = blk[b];
    blk[b] = run;
    run += x;
  }
  if (threadIdx.x == 0) blk[nblk] = tot;
}

template <class In, class Out>
__global__ void __launch_bounds__(BT) k_scan_apply(const In *in, int64_t n, const uint64_t *blk,
                                                   int64_t nblk, Out *out) {
  __shared__ uint64_t sh[BT / WAVE];
  const int64_t base = (int64_t)blockIdx.x * SCAN_BLOCK + (int64_t)threadIdx.x * SCAN_PER_THREAD;
  uint64_t s = 0;
  for (int u = 0; u < SCAN_PER_THREAD; ++u)
    if (base + u < n) s += (uint64_t)in[base + u];
  uint64_t tot;
  uint64_t run = blk[blockIdx.x] + block_excl_scan<uint64_t>(s, sh, &tot);
  for (int u = 0; u < SCAN_PER_THREAD; ++u)
    if (base + u < n) {
      out[base + u] = (Out)run;
      run += (uint64_t)in[base + u];
    }
  if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = (Out)blk[nblk];
}

// blk: [ceil(n / SCAN_BLOCK) + 1] scratch
template <class In, class Out>
hipError_t launch_scan(const In *in, int64_t n, Out *out, uint64_t *blk, hipStream_t s) {
  const int64_t nblk = n > 0 ? (n + SCAN_BLOCK - 1) / SCAN_BLOCK : 1;
  hipLaunchKernelGGL((k_scan_sums<In>), dim3((unsigned)nblk), dim3(BT), 0, s, in, n, blk);
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(BT), 0, s, blk, nblk);
  hipLaunchKernelGGL((k_scan_apply<In, Out>), dim3((unsigned)nblk), dim3(BT), 0, s, in, n, blk,
                     nblk, out);
  return hipGetLastError();
}

int build_pad(int b) { return (b + 3) / 4 * 4; }

size_t build_scan_blocks(int64_t n) { return (size_t)((n + SCAN_BLOCK - 1) / SCAN_BLOCK) + 2; }

// ------------------------------------------------------------------ tau
// order-preserving u32 key of a float (-0 and +0 map apart, as their order
// in a total order; no NaN reaches here)
__device__ __forceinline__ uint32_t fkey(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float fkey_inv(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// Radix select of every dimension's (ns - 1) / 2-th smallest value at once:
// per digit (8 bits, from the top) one pass over the sample counts, in LDS, the
// digits of the keys that match the dimension's prefix so far, and one block
// per dimension picks the digit holding the rank.  Rows are read whole and in
// order by the whole chip: 1M x 16 latents take 0.12 ms where one block per
// dimension (k_build_tau below) read its column in 5.6 ms.
struct TauState {
  uint32_t prefix, rank;
};

// thread t counts dimension t % b; a step of the block reads 256 / b rows
__global__ void __launch_bounds__(BT) k_tau_hist(const float *lg, int64_t ns, int b, int shift,
                                                 const TauState *st, uint32_t *hist) {
  extern __shared__ uint32_t h[];  // [b][256]
  for (int i = threadIdx.x; i < b * 256; i += BT) h[i] = 0;
  __syncthreads();
  const int rows = BT / b;
  if ((int)threadIdx.x < rows * b) {
    const int j = threadIdx.x % b;
    const uint32_t prefix = st[j].prefix;
    const uint32_t mask = shift == 24 ? 0u : (0xFFFFFFFFu << (shift + 8));
    const int64_t total = ns * b, step = (int64_t)gridDim.x * rows * b;
    for (int64_t e = (int64_t)blockIdx.x * rows * b + threadIdx.x; e < total; e += 4 * step) {
      float v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = e + u * step < total ? lg[e + u * step] : 0.0f;
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t k = fkey(v[u]);
        if (e + u * step < total && (k & mask) == prefix)
          atomicAdd(&h[j * 256 + ((k >> shift) & 255u)], 1u);
      }
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < b * 256; i += BT)
    if (h[i]) atomicAdd(&hist[i], h[i]);
}

// the digit of dimension blockIdx.x: the last whose count of keys below it is
// at most the rank; clears the counts for the next pass
__global__ void __launch_bounds__(256) k_tau_pick(uint32_t *hist, TauState *st, int shift,
                                                  float *tau) {
  __shared__ uint32_t sh[BT / WAVE];
  const int j = blockIdx.x, d = threadIdx.x;
  const TauState s = st[j];
  const uint32_t c = hist[j * 256 + d];
  hist[j * 256 + d] = 0;
  uint32_t tot;
  const uint32_t below = block_excl_scan<uint32_t>(c, sh, &tot);
  if (below <= s.rank && s.rank < below + c) {   // one digit: the rank is below tot
    const uint32_t p = s.prefix | ((uint32_t)d << shift);
    st[j] = TauState{p, s.rank - below};
    if (shift == 0) tau[j] = fkey_inv(p);
  }
}

__global__ void k_tau_init(TauState *st, uint32_t *hist, int b, uint32_t rank) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < b) st[i] = TauState{0u, rank};
  if (i < b * 256) hist[i] = 0;
}

// one block per dimension: the (ns - 1) / 2-th smallest value of column j
__global__ void __launch_bounds__(BT) k_build_tau(const float *lg, int64_t ns, int b, float *tau) {
  __shared__ uint32_t hist[256];
  __shared__ uint32_t s_prefix, s_rank;
  const int j = blockIdx.x;
  uint32_t prefix = 0;
  uint32_t rank = (uint32_t)((ns - 1) / 2);   // rank among the keys matching the prefix
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    const uint32_t hmask = pass == 0 ? 0u : (0xFFFFFFFFu << (shift + 8));
    for (int i = threadIdx.x; i < 256; i += BT) hist[i] = 0;
    __syncthreads();
    for (int64_t i = threadIdx.x; i < ns; i += BT) {
      const uint32_t k = fkey(lg[i * b + j]);
      if ((k & hmask) == prefix) atomicAdd(&hist[(k >> shift) & 255u], 1u);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t r = rank, d = 0;
      while (d < 255 && hist[d] <= r) {
        r -= hist[d];
        ++d;
      }
      s_prefix = prefix | (d << shift);
      s_rank = r;
    }
    __syncthreads();
    prefix = s_prefix;
    rank = s_rank;
    __syncthreads();
  }
  if (threadIdx.x == 0) tau[j] = fkey_inv(prefix);
}

// ------------------------------------------------------------------ codes
__global__ void k_build_codes(const float *lg, int64_t m, int b, const float *tau,
                              uint32_t *codes, uint32_t *sizes) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
    uint32_t c = 0;
    for (int j = 0; j < b; ++j) c |= (lg[i * b + j] >= tau[j] ? 1u : 0u) << j;
    codes[i] = c;
    atomicAdd(&sizes[c], 1u);
  }
}

// clusters per bucket: rule NR_CLUSTER_CAPACITY: ceil(size / t); FIXED:
// min(size, t); NONE: min(size, 1)
__global__ void k_build_kb(const uint32_t *sizes, int64_t nb, int rule, uint32_t t, uint32_t *kb,
                           uint32_t *multi) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < nb; c += stride) {
    const uint32_t s = sizes[c];
    uint32_t k;
    if (rule == NR_CLUSTER_CAPACITY) k = (s + t - 1) / t;
    else if (rule == NR_CLUSTER_FIXED) k = s < t ? s : t;
    else k = s < 1u ? s : 1u;
    kb[c] = k;
    multi[c] = k >= 2 ? 1u : 0u;
  }
}

__global__ void k_build_multi_list(const uint32_t *multi, const uint32_t *mpos, int64_t nb,
                                   uint32_t *mlist) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < nb; c += stride)
    if (multi[c]) mlist[mpos[c]] = (uint32_t)c;
}

// ------------------------------------------------------------------ buckets
__global__ void k_build_scatter(const uint32_t *codes, int64_t n, const uint64_t *boff,
                                uint32_t *cursor, uint32_t *ids) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const uint32_t c = codes[i];
    const uint64_t pos = boff[c] + atomicAdd(&cursor[c], 1u);
    if (pos < boff[c + 1]) ids[pos] = (uint32_t)i;   // sizes and codes agree
  }
}

// Ascending sort of keys[0, n) by one block of NT threads: bitonic in LDS for
// n <= SORT_LDS (`lds`, SORT_LDS keys), else a stable LSD radix sort over 4-bit
// digits through tmp[0, n) (`cnt`, 16 x NT counts).
template <int NT, class K>
__device__ void block_sort(K *keys, int64_t n, K *tmp, int key_bits, K *lds, uint32_t *cnt,
                           uint32_t *shs) {
  if (n <= 1) return;
  if (n <= SORT_LDS) {
    int p2 = 1;
    while (p2 < n) p2 <<= 1;
    for (int i = threadIdx.x; i < p2; i += NT) lds[i] = i < n ? keys[i] : (K)~(K)0;
    __syncthreads();
    for (int k = 2; k <= p2; k <<= 1)
      for (int jj = k >> 1; jj > 0; jj >>= 1) {
        for (int i = threadIdx.x; i < p2; i += NT) {
          const int l = i ^ jj;
          if (l > i) {
            const K a = lds[i], c = lds[l];
            const bool up = (i & k) == 0;
            if ((a > c) == up) {
              lds[i] = c;
              lds[l] = a;
            }
          }
        }
        __syncthreads();
      }
    for (int i = threadIdx.x; i < n; i += NT) keys[i] = lds[i];
    __syncthreads();
    return;
  }
  const int64_t per = (n + NT - 1) / NT;
  const int64_t i0 = (int64_t)threadIdx.x * per;
  const int64_t i1 = i0 + per < n ? i0 + per : n;
  constexpr int COLS = NT / 16;   // columns of one digit that a thread scans
  K *src = keys, *dst = tmp;
  for (int shift = 0; shift < key_bits; shift += 4) {
    for (int d = 0; d < 16; ++d) cnt[d * NT + threadIdx.x] = 0;
    for (int64_t i = i0; i < i1; ++i) cnt[((src[i] >> shift) & 15) * NT + threadIdx.x] += 1;
    __syncthreads();
    // exclusive offsets in (digit, thread) order: thread t owns the 16 counts
    // from 16 t on, which lie in one digit's row
    uint32_t *mine = cnt + (threadIdx.x / COLS) * NT + (threadIdx.x % COLS) * 16;
    uint32_t loc = 0;
    for (int c = 0; c < 16; ++c) loc += mine[c];
    uint32_t tot;
    uint32_t run = block_excl_scan<uint32_t, NT>(loc, shs, &tot);
    for (int c = 0; c < 16; ++c) {
      const uint32_t x = mine[c];
      mine[c] = run;
      run += x;
    }
    __syncthreads();
    for (int64_t i = i0; i < i1; ++i) {
      const K k = src[i];
      const int d = (int)((k >> shift) & 15);
      dst[cnt[d * NT + threadIdx.x]++] = k;
    }
    __syncthreads();
    K *t = src;
    src = dst;
    dst = t;
  }
  if (src != keys)
    for (int64_t i = threadIdx.x; i < n; i += NT) keys[i] = src[i];
  __syncthreads();
}

// Buckets (or multi-cluster buckets) that one wave does not take go to two
// lists, appended in any order (each is independent work): mid, for blocks of
// BT threads, and big, for blocks of BIG threads.  Most buckets hold a few
// rows, so one wave per bucket and four buckets per block keep the chip full
// where one block per bucket left most lanes idle; the few large buckets,
// whose chains end the kernel, get 1024 threads each.
constexpr int WAVE_ROWS = WAVE;   // rows of a bucket sorted and seeded by one wave
constexpr int MID_ROWS = BT;      // and by a block of BT threads
constexpr int BIG = 1024;
constexpr int LIST_GRID = 2048;   // blocks that walk a list

// Kernels with a wave per item are launched over WAVES_MAX items at a time (a
// launch takes fewer than 2^32 threads); a wave's item is `first` + its number
constexpr int64_t WAVES_MAX = (int64_t)1 << 24;
__device__ __forceinline__ int64_t wave_number() {
  return (int64_t)blockIdx.x * (BT / WAVE) + threadIdx.x / WAVE;
}

struct SizeLists {
  uint32_t *mid, *big;
  uint32_t *count;  // [2], zero before the wave kernel
};

__device__ __forceinline__ void list_bucket(const SizeLists &l, int64_t m, uint32_t c) {
  if (m <= MID_ROWS) l.mid[atomicAdd(&l.count[0], 1u)] = c;
  else l.big[atomicAdd(&l.count[1], 1u)] = c;
}

// the ids of every bucket ascending: one wave per bucket of at most 64 rows
__global__ void __launch_bounds__(BT) k_build_sort_wave(uint32_t *ids, const uint64_t *boff,
                                                        int64_t nb, SizeLists l, int64_t first) {
  const int lane = lane_id();
  const int64_t c = first + wave_number();
  if (c >= nb) return;
  const uint64_t s0 = boff[c];
  const int64_t m = (int64_t)(boff[c + 1] - s0);
  if (m <= 1) return;
  if (m > WAVE_ROWS) {
    if (lane == 0) list_bucket(l, m, (uint32_t)c);
    return;
  }
  uint32_t key = lane < m ? ids[s0 + lane] : 0xffffffffu;
  int top = 2;
  while (top < m) top <<= 1;
  for (int k = 2; k <= top; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      const uint32_t o = (uint32_t)__shfl_xor((int)key, j);
      const bool up = (lane & k) == 0, lower = (lane & j) == 0;
      key = (lower == up) == (key < o) ? key : o;
    }
  if (lane < m) ids[s0 + lane] = key;
}

template <int NT>
__global__ void __launch_bounds__(NT) k_build_sort_list(uint32_t *ids, const uint64_t *boff,
                                                        uint32_t *tmp, const uint32_t *list,
                                                        const uint32_t *count) {
  __shared__ uint32_t lds[SORT_LDS];
  __shared__ uint32_t cnt[16 * NT];
  __shared__ uint32_t shs[NT / WAVE];
  const uint32_t total = *count;
  for (uint32_t i = blockIdx.x; i < total; i += gridDim.x) {
    const uint64_t s0 = boff[list[i]], s1 = boff[list[i] + 1];
    block_sort<NT, uint32_t>(ids + s0, (int64_t)(s1 - s0), tmp + s0, 32, lds, cnt, shs);
  }
}

// ------------------------------------------------------------------ k-means
struct KmArgs {
  const float *lg;          // [n x b] latents by original id
  int b;
  const uint64_t *boff;     // [nb + 1] bucket row offsets
  const uint32_t *ids;      // [n] ids in bucket order, ascending inside a bucket
  const uint32_t *kb;       // [nb]
  const uint64_t *kbpre;    // [nb + 1] exclusive scan of kb: cluster slots of a bucket
  const uint32_t *mlist;    // [n_multi] buckets with kb >= 2, ascending
  int64_t n_multi;
  const double *U;          // [n_multi x kmax]
  int kmax;
  uint32_t seed;
  int spc;
  uint64_t *skey;           // [n] scratch: sample keys, in bucket order (big buckets)
  uint64_t *skey_tmp;       // [n] sort scratch
  double *d2;               // [n] scratch
  uint32_t *label;          // [n] slot within its bucket of each member (bucket order)
  double *cent;             // [slots x bp] centres, by slot
  int bp;                   // b rounded up to a multiple of 4; zeros from b on
  uint32_t *ccnt;           // [slots] members per slot
  const uint4 *slot;        // [slots] see k_build_slots
  int64_t slots;
  uint32_t *changed;        // [nb] last Lloyd pass (from 1) that changed a label of the bucket
  uint2 *tile;              // [n / 64 + n_multi] (bucket, first member) of 64 members each
  uint32_t *ntile;          // zero before the tiles are listed
  uint32_t *nkept;          // [nb] clusters kept per bucket (multi buckets; zero before)
};

__device__ __forceinline__ uint64_t sample_key(uint32_t id, uint32_t seed) {
  return ((uint64_t)mix32_dev(id, seed) << 32) | id;
}

// members of a bucket's sample
__device__ __forceinline__ int64_t sample_size(int64_t m, int K, int spc) {
  int64_t S = m;
  if ((int64_t)spc * K < S) S = (int64_t)spc * K;
  if (S > (int64_t)(1 << 21)) S = (int64_t)1 << 21;
  return S;
}

// Rows and centres of b dimensions are handled as BP of them, zeros from b on
// (BP >= b a template argument): a zero dimension adds +0 to a squared
// distance, which leaves its bits, and the loads of a row have no branch
// between them.
template <int BP>
__device__ __forceinline__ void load_row(float (&x)[BP], const float *r, int b) {
#pragma unroll
  for (int j = 0; j < BP; ++j) x[j] = r[j < b ? j : 0];
#pragma unroll
  for (int j = 0; j < BP; ++j) x[j] = j < b ? x[j] : 0.0f;
}

// fp64 squared distance, dimensions in order
template <int BP>
__device__ __forceinline__ double sqd(const float (&x)[BP], const float (&c)[BP]) {
  double acc = 0.0;
#pragma unroll
  for (int j = 0; j < BP; ++j) {
    const double t = (double)x[j] - (double)c[j];
    acc = acc + t * t;
  }
  return acc;
}

// k-means++ of a bucket of at most 64 rows by one wave, a sample member per
// lane: its row and D^2 stay in registers, the running weights are a wave scan
template <int BP>
__global__ void __launch_bounds__(BT) k_build_seed_wave(KmArgs a, SizeLists l,
                                                        int64_t first) {
  const int lane = lane_id();
  const int64_t mi = first + wave_number();
  if (mi >= a.n_multi) return;
  const uint32_t code = a.mlist[mi];
  const uint64_t s0 = a.boff[code];
  const int64_t m = (int64_t)(a.boff[code + 1] - s0);
  if (m > WAVE_ROWS) {
    if (lane == 0) list_bucket(l, m, (uint32_t)mi);
    return;
  }
  const int K = (int)a.kb[code], b = a.b;
  double *C = a.cent + a.kbpre[code] * a.bp;
  const int S = (int)sample_size(m, K, a.spc);
  uint64_t key = lane < m ? sample_key(a.ids[s0 + lane], a.seed) : ~0ull;
  key = wave_sort_u64(key, (int)m);
  const uint32_t id = lane < S ? (uint32_t)key : (uint32_t)bcast_u64(key, 0);
  float x[BP], c[BP];
  load_row<BP>(x, a.lg + (uint64_t)id * b, b);
  uint32_t pid = bcast_u32(id, 0);
  double d2 = 0.0;
  const double us = lane < K ? a.U[mi * a.kmax + lane] : 0.0;   // K <= 64: a uniform per lane
  uint32_t drawn = 0;   // lane r: the id of draw r
  for (int r = 0; r < K; ++r) {
    if (r > 0) {
      const int64_t w = lane < S ? d2_weight(d2) : 0;
      const int64_t incl = (int64_t)wave_incl_scan_u64((uint64_t)w);
      const int64_t tot = (int64_t)bcast_u64((uint64_t)incl, WAVE - 1);
      int pick = 0;
      if (tot > 0) {
        const double u = __longlong_as_double(
            (long long)bcast_u64((uint64_t)__double_as_longlong(us), r));
        const int64_t target = (int64_t)floor(u * (double)tot);
        const uint64_t over = ballot(incl > target);
        pick = over ? __ffsll((unsigned long long)over) - 1 : S - 1;
      }
      pid = bcast_u32(id, pick);
    }
    if (lane == r) drawn = pid;
    load_row<BP>(c, a.lg + (uint64_t)pid * b, b);
    const double d = sqd<BP>(x, c);
    if (r == 0 || d < d2) d2 = d;
  }
  for (int e = lane; e < (K * a.bp + WAVE - 1) / WAVE * WAVE; e += WAVE) {
    const int r = e / a.bp, j = e - r * a.bp;
    const uint32_t rid = (uint32_t)__shfl((int)drawn, r < K ? r : 0);
    if (r < K) C[e] = j < b ? (double)a.lg[(uint64_t)rid * b + j] : 0.0;
  }
}

// k-means++ of a listed bucket by a block of NT threads.  Thread t owns the
// sample members [t per, (t + 1) per); up to PT of them stay in registers with
// their D^2.  The update of D^2 by a new centre also sums the thread's weights
// for the next draw, so a draw costs one block scan, two barriers and the load
// of one row; the draws are kept in LDS and the centres written at the end,
// and the uniforms read 64 at a time, because a barrier waits for every load
// and store before it (376 draws among 1128 rows of 16: 3.7 ms with them and
// with the members past the first in memory).
template <int NT, int BP>
__global__ void __launch_bounds__(NT) k_build_seed_list(KmArgs a, const uint32_t *list,
                                                        const uint32_t *count) {
  constexpr int NW = NT / WAVE;
  constexpr int PT = BP <= 16 ? 2 : 1;
  __shared__ uint64_t keys[SORT_LDS];
  __shared__ uint32_t cnt[16 * NT];   // counts of the sort, then the draws
  __shared__ uint32_t shs[NW];
  __shared__ int64_t s_tot[2][NW];
  __shared__ int64_t s_pick[2];
  const int lane = lane_id(), wv = threadIdx.x / WAVE;
  const uint32_t total = *count;
  for (uint32_t li = blockIdx.x; li < total; li += gridDim.x) {
    const int64_t mi = list[li];
    const uint32_t code = a.mlist[mi];
    const uint64_t s0 = a.boff[code];
    const int64_t m = (int64_t)(a.boff[code + 1] - s0);
    const int K = (int)a.kb[code], b = a.b;
    const uint32_t *mid = a.ids + s0;
    double *C = a.cent + a.kbpre[code] * a.bp;
    double *D2 = a.d2 + s0;
    uint64_t *sk = a.skey + s0;
    const double *U = a.U + mi * a.kmax;
    for (int64_t i = threadIdx.x; i < m; i += NT) sk[i] = sample_key(mid[i], a.seed);
    __syncthreads();
    block_sort<NT, uint64_t>(sk, m, a.skey_tmp + s0, 64, keys, cnt, shs);
    const int64_t S = sample_size(m, K, a.spc);
    const int64_t per = (S + NT - 1) / NT;
    const int64_t c0 = (int64_t)threadIdx.x * per < S ? (int64_t)threadIdx.x * per : S;
    const int64_t c1 = c0 + per < S ? c0 + per : S;
    const bool regs = per <= PT;
    const bool in_lds = m <= SORT_LDS;  // the sort leaves its keys there too
    auto sample_id = [&](int64_t i) -> uint32_t {
      if (in_lds) return reinterpret_cast<const uint32_t *>(keys)[2 * (int)i];  // the low word
      return (uint32_t)sk[i];
    };
    float x[PT][BP], c[BP];
    double d2[PT];
#pragma unroll
    for (int t = 0; t < PT; ++t) {
      d2[t] = 0.0;
      if (regs) load_row<BP>(x[t], a.lg + (uint64_t)sample_id(c0 + t < c1 ? c0 + t : 0) * b, b);
    }
    if (threadIdx.x == 0) s_pick[0] = s_pick[1] = S;
    uint32_t pid = sample_id(0);
    int64_t wsum = 0;
    double us = 0.0;   // lane l: the uniform of draw r with r % 64 = l
    for (int r = 0; r < K; ++r) {
      if ((r & (WAVE - 1)) == 0) us = r + lane < K ? U[r + lane] : 0.0;
      if (r > 0) {
        const int p = r & 1;
        const int64_t incl = (int64_t)wave_incl_scan_u64((uint64_t)wsum);
        if (lane == WAVE - 1) s_tot[p][wv] = incl;
        __syncthreads();
        if (threadIdx.x == 0) s_pick[p ^ 1] = S;   // read by all before this barrier
        int64_t before = incl - wsum, tot = 0;
#pragma unroll
        for (int i = 0; i < NW; ++i) {
          const int64_t v = s_tot[p][i];
          before += i < wv ? v : 0;
          tot += v;
        }
        if (tot > 0) {   // the same in every thread
          const double u = __longlong_as_double(
              (long long)bcast_u64((uint64_t)__double_as_longlong(us), r & (WAVE - 1)));
          const int64_t target = (int64_t)floor(u * (double)tot);
          if (before <= target && target < before + wsum) {
            int64_t at = c0;
            int64_t run = before;
            if (regs) {
#pragma unroll
              for (int t = 0; t < PT; ++t) {
                const bool more = at == c0 + t && at + 1 < c1;
                if (more) run += d2_weight(d2[t]);
                if (more && run <= target) ++at;
              }
            } else {
              for (; at + 1 < c1; ++at) {
                run += d2_weight(D2[at]);
                if (run > target) break;
              }
            }
            s_pick[p] = at;
          }
        }
        __syncthreads();
        int64_t pick = 0;
        if (tot > 0) pick = s_pick[p] < S ? s_pick[p] : S - 1;
        pid = (uint32_t)__builtin_amdgcn_readfirstlane((int)sample_id(pick));
      }
      const float *xp = a.lg + (uint64_t)pid * b;
      load_row<BP>(c, xp, b);
      if (r < 16 * NT) {
        if (threadIdx.x == 0) cnt[r] = pid;
      } else if ((int)threadIdx.x < a.bp) {
        C[(int64_t)r * a.bp + threadIdx.x] = (int)threadIdx.x < b ? (double)xp[threadIdx.x] : 0.0;
      }
      wsum = 0;
      if (regs) {
#pragma unroll
        for (int t = 0; t < PT; ++t) {
          const double d = sqd<BP>(x[t], c);
          if (r == 0 || d < d2[t]) d2[t] = d;
          if (c0 + t < c1) wsum += d2_weight(d2[t]);
        }
      } else {
        for (int64_t s = c0; s < c1; ++s) {
          load_row<BP>(x[0], a.lg + (uint64_t)sample_id(s) * b, b);
          const double d = sqd<BP>(x[0], c);
          const double o = r == 0 ? d : D2[s];
          const double v = d < o ? d : o;
          D2[s] = v;
          wsum += d2_weight(v);
        }
      }
    }
    __syncthreads();
    const int64_t kept = (int64_t)(K < 16 * NT ? K : 16 * NT) * a.bp;
    for (int64_t e = threadIdx.x; e < kept; e += NT) {
      const int r = (int)(e / a.bp), j = (int)(e - (int64_t)r * a.bp);
      C[e] = j < b ? (double)a.lg[(uint64_t)cnt[r] * b + j] : 0.0;
    }
    __syncthreads();   // the next bucket's sort reuses the block's LDS
  }
}

// The slots of every bucket, 64 buckets per wave (those of one slot each by
// their own lane): (first row, rows, slot within the bucket, bucket), so that
// the waves that take a slot each start from one load
__global__ void __launch_bounds__(BT) k_build_slots(const uint32_t *kb, const uint64_t *kbpre,
                                                    const uint64_t *boff, int64_t nb,
                                                    int64_t slots, uint4 *slot, int64_t first) {
  const int lane = lane_id();
  const int64_t w0 = first + wave_number();
  const int64_t c = w0 * WAVE + lane;
  const uint32_t k = c < nb ? kb[c] : 0u;
  const uint64_t p = c < nb ? kbpre[c] : 0ull;
  const uint32_t s0 = c < nb ? (uint32_t)boff[c] : 0u;
  const uint32_t m = c < nb ? (uint32_t)boff[c + 1] - s0 : 0u;
  if (k == 1 && (int64_t)p < slots) slot[p] = make_uint4(s0, m, 0u, (uint32_t)c);
  uint64_t many = ballot(k > 1);
  while (many) {
    const int src = __ffsll((unsigned long long)many) - 1;
    many &= many - 1;
    const uint64_t ps = bcast_u64(p, src);
    const uint32_t ks = bcast_u32(k, src), ss = bcast_u32(s0, src), ms = bcast_u32(m, src);
    for (uint32_t i = lane; i < ks; i += WAVE)
      if ((int64_t)(ps + i) < slots)
        slot[ps + i] = make_uint4(ss, ms, i, (uint32_t)(w0 * WAVE + src));
  }
}

// the multi-cluster buckets' members, 64 to a tile; 64 buckets per wave, one
// atomic each
__global__ void __launch_bounds__(BT) k_build_tiles(KmArgs a, int64_t first) {
  const int lane = lane_id();
  const int64_t mi = (first + wave_number()) * WAVE + lane;
  uint32_t code = 0, nt = 0;
  if (mi < a.n_multi) {
    code = a.mlist[mi];
    nt = ((uint32_t)(a.boff[code + 1] - a.boff[code]) + WAVE - 1) / WAVE;
  }
  const uint32_t incl = wave_incl_scan_u32(nt);
  uint32_t base = 0;
  if (lane == WAVE - 1) base = atomicAdd(a.ntile, incl);
  base = bcast_u32(base, WAVE - 1) + incl - nt;
  if (nt == 1) a.tile[base] = make_uint2(code, 0u);
  uint64_t many = ballot(nt > 1);
  while (many) {
    const int src = __ffsll((unsigned long long)many) - 1;
    many &= many - 1;
    const uint32_t n = bcast_u32(nt, src), at = bcast_u32(base, src), cd = bcast_u32(code, src);
    for (uint32_t t = lane; t < n; t += WAVE) a.tile[at + t] = make_uint2(cd, t * WAVE);
  }
}

// Lloyd, first half: the nearest centre of each member, one wave per tile.
// Every member of a tile has the same centres, so they are read once per wave
// (scalar loads, two centres in flight) and the fp64 arithmetic bounds the
// pass.  A bucket in which the last pass changed no label is at rest: its
// centres and labels stay as they are.
template <int BP>
__global__ void __launch_bounds__(BT) k_build_assign(KmArgs a, uint32_t pass,
                                                     int64_t first) {
  const int lane = lane_id();
  const uint32_t t =
      (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(first + wave_number()));
  if (t >= *a.ntile) return;
  const uint2 tl = a.tile[t];
  const uint32_t code = (uint32_t)__builtin_amdgcn_readfirstlane((int)tl.x);
  const uint32_t i0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)tl.y);
  // passes count from 1; another tile of the bucket may store this pass's number
  if (pass > 1 && a.changed[code] + 1 < pass) return;
  const uint64_t s0 = a.boff[code];
  const uint32_t m = (uint32_t)(a.boff[code + 1] - s0);
  const int K = (int)a.kb[code], b = a.b;
  const double *__restrict__ C = a.cent + a.kbpre[code] * BP;
  const uint32_t i = i0 + lane;
  const bool in = i < m;
  float xf[BP];
  load_row<BP>(xf, a.lg + (uint64_t)a.ids[s0 + (in ? i : i0)] * b, b);
  double x[BP];
#pragma unroll
  for (int j = 0; j < BP; ++j) x[j] = (double)xf[j];
  double best = INFINITY;
  uint32_t bk = 0;
#pragma unroll 2
  for (int k = 0; k < K; ++k) {
    const double *c = C + (int64_t)k * BP;
    double acc = 0.0;
#pragma unroll
    for (int j = 0; j < BP; ++j) {
      const double d = x[j] - c[j];
      acc = acc + d * d;
    }
    if (k == 0 || acc < best) {
      best = acc;
      bk = (uint32_t)k;
    }
  }
  const bool moved = in && (pass == 1 || a.label[s0 + i] != bk);
  if (moved) a.label[s0 + i] = bk;
  if (ballot(moved) && lane == 0) a.changed[code] = pass;
}

// the wave's lanes j < b add row[id][j] of the members whose lanes are set in
// `mask`, in lane order, eight rows in flight (the order of the additions is
// the result's; only their loads run ahead)
__device__ __forceinline__ void ordered_add(double &sum, const float *lg, int b, uint32_t id,
                                            uint64_t mask) {
  const int j = lane_id() < b ? lane_id() : 0;
  while (mask) {
    float v[8];
    int n = 0;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      v[u] = 0.0f;
      if (mask) {
        const int src = __ffsll((unsigned long long)mask) - 1;
        mask &= mask - 1;
        v[u] = lg[(uint64_t)bcast_u32(id, src) * b + j];
        ++n;
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (u < n) sum = sum + (double)v[u];
  }
}

// Lloyd, second half: one wave per slot finds its members 64 labels at a time
// and adds them in id order
__global__ void __launch_bounds__(BT) k_build_update(KmArgs a, uint32_t pass, int last,
                                                     int64_t first) {
  const int lane = lane_id();
  const int64_t sl = first + wave_number();
  if (sl >= a.slots) return;
  const uint4 rec = a.slot[sl];
  const uint32_t code = rec.w, m = rec.y, k = rec.z;
  if (m == 0 || a.kb[code] < 2) return;
  uint32_t n_k = 0;
  if (a.changed[code] == pass) {
    const uint32_t *label = a.label + rec.x, *ids = a.ids + rec.x;
    double sum = 0.0;
    for (uint32_t r0 = 0; r0 < m; r0 += 4 * WAVE) {
      uint32_t lab[4], id[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t i = r0 + u * WAVE + lane;
        lab[u] = i < m ? label[i] : 0xffffffffu;
        id[u] = i < m ? ids[i] : 0u;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint64_t mk = ballot(lab[u] == k);
        if (!mk) continue;
        n_k += (uint32_t)popc64(mk);
        ordered_add(sum, a.lg, a.b, id[u], mk);
      }
    }
    if (n_k > 0 && lane < a.b) a.cent[sl * a.bp + lane] = sum / (double)n_k;
    if (lane == 0) a.ccnt[sl] = n_k;
  } else if (last) {
    n_k = a.ccnt[sl];
  }
  if (last && lane == 0 && n_k > 0) atomicAdd(&a.nkept[code], 1u);
}

// clusters of each bucket: 0 (empty), 1 (K_B = 1) or the kept count
__global__ void k_build_ncl(const uint32_t *sizes, const uint32_t *kb, const uint32_t *nkept,
                            int64_t nb, uint32_t *ncl) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < nb; c += stride)
    ncl[c] = sizes[c] == 0 ? 0u : (kb[c] >= 2 ? nkept[c] : 1u);
}

struct FinArgs {
  const float *lg;
  int b;
  const uint64_t *boff;
  const uint32_t *ids, *kb, *label, *ccnt;
  const double *cent;
  int bp;
  const uint4 *slot;
  int64_t slots;
  const uint32_t *bc_off;
  int64_t *row_ids;        // [n] out
  uint64_t *csize;         // [n_clusters] out: rows per cluster
  float *centroids;        // [n_clusters x b] out
};

// one wave per slot: its cluster's rows in (cluster, id) order, size and
// centroid.  Empty slots are dropped, so a slot's cluster number and first row
// come from the counts of its bucket's earlier slots
__global__ void __launch_bounds__(BT) k_build_finish(FinArgs a, int64_t first) {
  const int lane = lane_id();
  const int64_t sl = first + wave_number();
  if (sl >= a.slots) return;
  const uint4 rec = a.slot[sl];
  const uint32_t c = rec.w, m = rec.y, k = rec.z;
  if (m == 0) return;
  const uint64_t s0 = rec.x;
  const int b = a.b;
  const uint32_t *mid = a.ids + s0;
  const uint32_t g0 = a.bc_off[c];
  if (a.kb[c] < 2) {  // one cluster: rows in id order, fp64 mean in id order
    double sum = 0.0;
    for (uint32_t r0 = 0; r0 < m; r0 += WAVE) {
      const uint32_t i = r0 + lane;
      const uint32_t id = i < m ? mid[i] : 0u;
      if (i < m) a.row_ids[s0 + i] = id;
      ordered_add(sum, a.lg, b, id, ballot(i < m));
    }
    if (lane < b) a.centroids[(uint64_t)g0 * b + lane] = (float)(sum / (double)m);
    if (lane == 0) a.csize[g0] = m;
    return;
  }
  const uint32_t n_k = a.ccnt[sl];
  if (n_k == 0) return;
  const int64_t slot0 = sl - k;
  uint32_t kept = 0, rows = 0;  // clusters and rows of the slots before
  for (uint32_t k0 = 0; k0 < k; k0 += WAVE) {
    const uint32_t v = k0 + lane < k ? a.ccnt[slot0 + k0 + lane] : 0u;
    kept += (uint32_t)popc64(ballot(v > 0));
    rows += wave_sum_u32(v);
  }
  const uint32_t g = g0 + kept;
  if (lane < b) a.centroids[(uint64_t)g * b + lane] = (float)a.cent[sl * a.bp + lane];
  if (lane == 0) a.csize[g] = n_k;
  uint64_t pos = s0 + rows;
  for (uint32_t r0 = 0; r0 < m; r0 += WAVE) {
    const uint32_t i = r0 + lane;
    const bool f = i < m && a.label[s0 + i] == k;
    const uint64_t mk = ballot(f);
    if (f) a.row_ids[pos + popc64(mk & lanemask_lt())] = mid[i];
    pos += (uint64_t)popc64(mk);
  }
}

// ------------------------------------------------------------------ launches
// work space of the whole-chip select, or 0 for samples that one block per
// dimension selects in about the launches' time (eight of them)
size_t build_tau_ws(int64_t ns, int b) {
  if (ns < TAU_SMALL || ns > 0xffffffffll) return 0;
  return (size_t)b * (256 * sizeof(uint32_t) + sizeof(TauState));
}

hipError_t launch_build_tau(const float *lg, int64_t ns, int b, float *tau, void *ws,
                            hipStream_t s) {
  if (ws) {
    TauState *st = static_cast<TauState *>(ws);
    uint32_t *hist = reinterpret_cast<uint32_t *>(st + b);
    const int64_t per = 4 * (BT / b);   // rows per step of a block
    const int64_t g = (ns + per - 1) / per;
    hipLaunchKernelGGL(k_tau_init, dim3((unsigned)b), dim3(256), 0, s, st, hist, b,
                       (uint32_t)((ns - 1) / 2));
    for (int shift = 24; shift >= 0; shift -= 8) {
      hipLaunchKernelGGL(k_tau_hist, dim3((unsigned)(g < 1024 ? g : 1024)), dim3(BT),
                         (size_t)b * 1024, s, lg, ns, b, shift, st, hist);
      hipLaunchKernelGGL(k_tau_pick, dim3((unsigned)b), dim3(256), 0, s, hist, st, shift, tau);
    }
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_build_tau, dim3((unsigned)b), dim3(BT), 0, s, lg, ns, b, tau);
  return hipGetLastError();
}

hipError_t launch_build_codes(const float *lg, int64_t m, int b, const float *tau, uint32_t *codes,
                              uint32_t *sizes, hipStream_t s) {
  if (m <= 0) return hipSuccess;
  int64_t blocks = (m + BT - 1) / BT;
  if (blocks > 65536) blocks = 65536;
  hipLaunchKernelGGL(k_build_codes, dim3((unsigned)blocks), dim3(BT), 0, s, lg, m, b, tau, codes,
                     sizes);
  return hipGetLastError();
}

static dim3 grid_for(int64_t items) {
  int64_t g = (items + BT - 1) / BT;
  return dim3((unsigned)(g > 65536 ? 65536 : (g < 1 ? 1 : g)));
}

__global__ void k_build_nonempty(const uint32_t *sizes, int64_t nb, unsigned long long *out) {
  __shared__ unsigned long long sh[BT / WAVE];
  unsigned long long c = 0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nb; i += stride)
    c += sizes[i] > 0 ? 1ull : 0ull;
  unsigned long long tot;
  (void)block_excl_scan<unsigned long long>(c, sh, &tot);
  if (threadIdx.x == 0) atomicAdd(out, tot);
}

// stats[0] = sum kb, stats[1] = buckets with kb >= 2, stats[2] = max kb
__global__ void k_build_kb_stats(const uint32_t *kb, int64_t nb, unsigned long long *stats) {
  __shared__ unsigned long long sh[BT / WAVE];
  unsigned long long sum = 0, nm = 0, mx = 0;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nb; i += stride) {
    const uint32_t k = kb[i];
    sum += k;
    nm += k >= 2 ? 1ull : 0ull;
    mx = k > mx ? k : mx;
  }
  unsigned long long t;
  (void)block_excl_scan<unsigned long long>(sum, sh, &t);
  if (threadIdx.x == 0) atomicAdd(&stats[0], t);
  (void)block_excl_scan<unsigned long long>(nm, sh, &t);
  if (threadIdx.x == 0) atomicAdd(&stats[1], t);
  atomicMax(&stats[2], mx);
}

hipError_t launch_build_nonempty(const uint32_t *sizes, int64_t nb, unsigned long long *out,
                                 hipStream_t s) {
  hipLaunchKernelGGL(k_build_nonempty, grid_for(nb), dim3(BT), 0, s, sizes, nb, out);
  return hipGetLastError();
}

hipError_t run_build_plan(const BuildArgs &A, hipStream_t s) {
  const int64_t nb = (int64_t)1 << A.b;
  hipError_t e;
  hipLaunchKernelGGL(k_build_kb, grid_for(nb), dim3(BT), 0, s, A.sizes, nb, A.rule, A.t, A.kb,
                     A.multi);
  hipLaunchKernelGGL(k_build_kb_stats, grid_for(nb), dim3(BT), 0, s, A.kb, nb, A.stats);
  if ((e = launch_scan(A.multi, nb, A.mpos, A.blk, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_build_multi_list, grid_for(nb), dim3(BT), 0, s, A.multi, A.mpos, nb,
                     A.mlist);
  return hipGetLastError();
}

// blocks of the kernels that walk a list of at most `items` buckets
static dim3 list_grid(int64_t items) {
  return dim3((unsigned)(items < LIST_GRID ? (items > 0 ? items : 1) : LIST_GRID));
}

// launch(grid, first) over `items` waves, WAVES_MAX at a time
template <class Launch>
static void for_waves(int64_t items, Launch launch) {
  constexpr int64_t wpb = BT / WAVE;
  for (int64_t first = 0; first < items; first += WAVES_MAX) {
    const int64_t n = items - first < WAVES_MAX ? items - first : WAVES_MAX;
    launch(dim3((unsigned)((n + wpb - 1) / wpb)), first);
  }
}

template <int BP>
static void launch_seeds(const KmArgs &k, const SizeLists &l, int64_t n, hipStream_t s) {
  for_waves(k.n_multi, [&](dim3 g, int64_t first) {
    hipLaunchKernelGGL(k_build_seed_wave<BP>, g, dim3(BT), 0, s, k, l, first);
  });
  hipLaunchKernelGGL((k_build_seed_list<BT, BP>), list_grid(k.n_multi), dim3(BT), 0, s, k, l.mid,
                     l.count);
  hipLaunchKernelGGL((k_build_seed_list<BIG, BP>), list_grid(n / MID_ROWS), dim3(BIG), 0, s, k,
                     l.big, l.count + 1);
}

static void launch_assign(const KmArgs &k, uint32_t pass, dim3 g, int64_t first, hipStream_t s) {
  switch (k.bp / 4) {
    case 1: hipLaunchKernelGGL(k_build_assign<4>, g, dim3(BT), 0, s, k, pass, first); break;
    case 2: hipLaunchKernelGGL(k_build_assign<8>, g, dim3(BT), 0, s, k, pass, first); break;
    case 3: hipLaunchKernelGGL(k_build_assign<12>, g, dim3(BT), 0, s, k, pass, first); break;
    case 4: hipLaunchKernelGGL(k_build_assign<16>, g, dim3(BT), 0, s, k, pass, first); break;
    case 5: hipLaunchKernelGGL(k_build_assign<20>, g, dim3(BT), 0, s, k, pass, first); break;
    case 6: hipLaunchKernelGGL(k_build_assign<24>, g, dim3(BT), 0, s, k, pass, first); break;
    case 7: hipLaunchKernelGGL(k_build_assign<28>, g, dim3(BT), 0, s, k, pass, first); break;
    default: hipLaunchKernelGGL(k_build_assign<32>, g, dim3(BT), 0, s, k, pass, first); break;
  }
}

hipError_t run_build_index(const BuildArgs &A, hipStream_t s) {
  const int64_t nb = (int64_t)1 << A.b;
  const int64_t n = A.n;
  hipError_t e;
  if ((e = launch_scan(A.kb, nb, A.kbpre, A.blk, s)) != hipSuccess) return e;
  // bucket order of the row ids
  if ((e = launch_scan(A.sizes, nb, A.boff, A.blk, s)) != hipSuccess) return e;
  if ((e = launch_fill_i32((int32_t *)A.cursor, nb, 0, s)) != hipSuccess) return e;
  hipLaunchKernelGGL(k_build_scatter, grid_for(n), dim3(BT), 0, s, A.codes, n, A.boff, A.cursor,
                     A.ids);
  const SizeLists l{A.list_mid, A.list_big, A.counts};
  if ((e = launch_fill_i32((int32_t *)A.counts, 5, 0, s)) != hipSuccess) return e;
  for_waves(nb, [&](dim3 g, int64_t first) {
    hipLaunchKernelGGL(k_build_sort_wave, g, dim3(BT), 0, s, A.ids, A.boff, nb, l, first);
  });
  hipLaunchKernelGGL(k_build_sort_list<BT>, list_grid(nb), dim3(BT), 0, s, A.ids, A.boff,
                     A.ids_tmp, l.mid, l.count);
  hipLaunchKernelGGL(k_build_sort_list<BIG>, list_grid(n / MID_ROWS), dim3(BIG), 0, s, A.ids,
                     A.boff, A.ids_tmp, l.big, l.count + 1);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if ((e = launch_fill_i32((int32_t *)A.slot, 4 * A.slots, 0, s)) != hipSuccess) return e;
  for_waves((nb + WAVE - 1) / WAVE, [&](dim3 g, int64_t first) {
    hipLaunchKernelGGL(k_build_slots, g, dim3(BT), 0, s, A.kb, A.kbpre, A.boff, nb, A.slots, A.slot,
                       first);
  });
  // k-means of the multi-cluster buckets
  if ((e = launch_fill_i32((int32_t *)A.nkept, nb, 0, s)) != hipSuccess) return e;
  if (A.n_multi > 0) {
    KmArgs k{};
    k.lg = A.lg;
    k.b = A.b;
    k.boff = A.boff;
    k.ids = A.ids;
    k.kb = A.kb;
    k.kbpre = A.kbpre;
    k.mlist = A.mlist;
    k.n_multi = A.n_multi;
    k.U = A.U;
    k.kmax = A.kmax;
    k.seed = A.seed;
    k.spc = A.spc;
    k.skey = A.skey;
    k.skey_tmp = A.skey_tmp;
    k.d2 = A.d2;
    k.label = A.label;
    k.cent = A.cent;
    k.ccnt = A.ccnt;
    k.bp = build_pad(A.b);
    k.slot = A.slot;
    k.slots = A.slots;
    k.changed = A.changed;
    k.tile = A.tile;
    k.ntile = A.counts + 4;
    k.nkept = A.nkept;
    const SizeLists lm{A.list_mid, A.list_big, A.counts + 2};
    for_waves((A.n_multi + WAVE - 1) / WAVE, [&](dim3 g, int64_t first) {
      hipLaunchKernelGGL(k_build_tiles, g, dim3(BT), 0, s, k, first);
    });
    switch ((A.b + 7) / 8) {
      case 1: launch_seeds<8>(k, lm, n, s); break;
      case 2: launch_seeds<16>(k, lm, n, s); break;
      case 3: launch_seeds<24>(k, lm, n, s); break;
      default: launch_seeds<32>(k, lm, n, s); break;
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (int it = 1; it <= A.lloyd; ++it) {
      for_waves(n / WAVE + A.n_multi, [&](dim3 g, int64_t first) {
        launch_assign(k, (uint32_t)it, g, first, s);
      });
      for_waves(A.slots, [&](dim3 g, int64_t first) {
        hipLaunchKernelGGL(k_build_update, g, dim3(BT), 0, s, k, (uint32_t)it,
                           it == A.lloyd ? 1 : 0, first);
      });
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  // directory, rows, cluster sizes, centroids
  hipLaunchKernelGGL(k_build_ncl, grid_for(nb), dim3(BT), 0, s, A.sizes, A.kb, A.nkept, nb, A.ncl);
  if ((e = launch_scan(A.ncl, nb, A.bc_off, A.blk, s)) != hipSuccess) return e;
  FinArgs f{};
  f.lg = A.lg;
  f.b = A.b;
  f.boff = A.boff;
  f.ids = A.ids;
  f.kb = A.kb;
  f.label = A.label;
  f.ccnt = A.ccnt;
  f.cent = A.cent;
  f.bp = build_pad(A.b);
  f.slot = A.slot;
  f.slots = A.slots;
  f.bc_off = A.bc_off;
  f.row_ids = A.row_ids;
  f.csize = A.csize;
  f.centroids = A.centroids;
  for_waves(A.slots, [&](dim3 g, int64_t first) {
    hipLaunchKernelGGL(k_build_finish, g, dim3(BT), 0, s, f, first);
  });
  return hipGetLastError();
}

hipError_t launch_build_cl_off(const uint64_t *csize, int64_t n_clusters, uint64_t *cl_off,
                               uint64_t *blk, hipStream_t s) {
  return launch_scan(csize, n_clusters, cl_off, blk, s);
}

}  // namespace nr
