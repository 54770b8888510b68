// Encoder training with the selective similarity loss L_sim (Sec. 3.2.2, the
// loss of Eq. "similarityconfig" with the dual-threshold mask of Eq. 8) for a
// mini-batch of B rows: inputs x [B x E] (scaled as the encoder sees them)
// and latents l [B x L], rho = sqrt(L / E),
//   S_emb(i, j) = ||x_i - x_j||,   S_lat(i, j) = ||l_i - l_j||,
//   m(i, j) = [i != j and (S_emb <= tau_emb or S_lat <= gamma rho tau_emb)],
//   L_sim = sum m (S_lat - gamma rho S_emb)^2 / sum m.
//
// k_pair_sqdist: all B x B squared input distances, |x_i|^2 + |x_j|^2 -
// 2 x_i . x_j with the dot products on the fp32 matrix cores
// (v_mfma_f32_16x16x4f32, one 64 x 64 tile per 256-thread block).  The rows
// are centred on the batch mean first (distances do not change), which keeps
// the norms, and so the cancellation in the expansion, small; k_center writes
// them in rows of whole 64-byte groups, so the tiles load 16 bytes at a time
// without bounds checks.  Norms and the expansion are taken in fp64: what
// rounds is the fp32 chain of the dot products, two chains of every other
// K-tile.
//
// k_pair_quantile: an order statistic of the off-diagonal distances (tau_emb
// of a batch) by radix select over their bits.
//
// k_lsim_grad: one pass over the pairs that yields the loss's numerator and
// mask count and the gradient with respect to the latents.  The mask is a
// constant of the step (as in the paper's formulation, the thresholds select
// pairs) and the distances are symmetric, so for row j
//   dL/dl_j = (1 / sum m) sum_i 4 m_ij d_ij (l_j - l_i) / S_lat(i, j),
// d_ij = S_lat(i, j) - gamma rho S_emb(i, j); the kernel writes the sum
// without the 1 / sum m factor.  Latent distances are taken directly from the
// coordinate differences (L <= 32).  The sums are added in a fixed order, so
// the gradient is the same bit for bit on every run.  Only the numerator's
// block sums meet in a double-precision atomic (its last bits may vary; the
// mask count is exact).
#include "nr_internal.h"

namespace nr {

typedef float v4f_l __attribute__((ext_vector_type(4)));

constexpr int LS_M = 64, LS_K = 16;

// Column sums of x over blocks of LS_ROWS rows (partial[blk][c]) and the
// column's range inside each block (range[blk][c]), then the shifts of the
// columns from the partials, added in block order.  4096 x 128 rows: 62 us
// with 256 rows per block (16 blocks, one long chain each), 4 us with 32.
constexpr int LS_ROWS = 32;

__global__ void __launch_bounds__(128) k_col_partial(const float *x, int64_t B, int D,
                                                     float *partial, float *range) {
  const int64_t r0 = (int64_t)blockIdx.x * LS_ROWS;
  const int nr = (int)(B - r0 < LS_ROWS ? B - r0 : LS_ROWS);
  for (int c = threadIdx.x; c < D; c += 128) {
    float s = 0.0f, lo = INFINITY, hi = -INFINITY;
#pragma unroll 8
    for (int i = 0; i < nr; ++i) {
      const float v = x[(r0 + i) * D + c];
      s += v;
      lo = fminf(lo, v);
      hi = fmaxf(hi, v);
    }
    partial[(int64_t)blockIdx.x * D + c] = s;
    range[(int64_t)blockIdx.x * D + c] = hi - lo;
  }
}

// The shift of a column: its mean, cut to 12 bits where that costs nothing.  Cut,
// it leaves the rows up to 2^-11 of the mean off centre, against which the
// products cancel (at a mean of 1e5 times the spread the distances were off by 2e-4
// of their scale).  So it is cut only where that is at most 1/64 of the column's
// range in every whole block of 32 rows, about 1/16 of the spread, less than half
// a percent of the norms.  The distances' error is the same then (3.5e-8 of their
// norm for 4096 uint8 rows of 128 either way, 1.3e-7 with fp32 norms and one
// chain), and the bits stay what they were, which decide the pairs at the mask's
// thresholds and so the trained weights.
// Two waves per 64 columns: sums, ranges; sixteen loads of each in flight.
__global__ void __launch_bounds__(128) k_col_mean(const float *partial, const float *range,
                                                  int64_t nblk, int64_t B, int D, float *mean) {
  __shared__ float s_least[64];
  const int lane = lane_id();
  const bool sums = threadIdx.x < WAVE;
  const int64_t c = (int64_t)blockIdx.x * 64 + lane;
  const int64_t n = sums || B < LS_ROWS ? nblk : B / LS_ROWS;   // ranges: of whole blocks
  const float *col = (sums ? partial : range) + (c < D ? c : D - 1);
  double s = 0.0;
  float least = INFINITY;
  for (int64_t b0 = 0; b0 < n; b0 += 16) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = col[(b0 + u < n ? b0 + u : n - 1) * D];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      s += b0 + u < n ? v[u] : 0.0f;
      least = fminf(least, v[u]);
    }
  }
  if (!sums) s_least[lane] = least;
  __syncthreads();
  if (!sums || c >= D) return;
  const float m = (float)(s / (double)B);
  const float cut = __uint_as_float(__float_as_uint(m) & 0xfffff000u);
  mean[c] = 64.0f * fabsf(m - cut) <= s_least[lane] ? cut : m;
}

// centred rows xc [B][DP], zeros from D on, and their squared norms; one wave
// per row
__global__ void __launch_bounds__(256) k_center(const float *x, int64_t B, int D, int DP,
                                                const float *mean, float *xc, double *norm) {
  const int lane = lane_id();
  const int64_t i = (int64_t)blockIdx.x * 4 + threadIdx.x / WAVE;
  if (i >= B) return;
  double s = 0.0;
  for (int c = lane; c < DP; c += WAVE) {
    const float v = c < D ? x[i * D + c] - mean[c] : 0.0f;
    xc[i * DP + c] = v;
    s += (double)v * (double)v;
  }
  for (int m = 1; m < WAVE; m <<= 1) s += __shfl_xor(s, m);
  if (lane == 0) norm[i] = s;
}

// Tiles on and above the diagonal only; each writes its mirror too, so the
// matrix is symmetric bit for bit.  The next K-tile is loaded while this one
// is multiplied (two LDS buffers).  4096 rows of 128: 69 us with element-wise
// loads and stores of the mirror, 43 us with 16-byte ones and two chains (which
// with fp64 norms bring the distances' error against 64 bits from 1.3e-7 of
// their norm to 3.5e-8; 39 us with one chain).
__global__ void __launch_bounds__(256) k_pair_sqdist(const float *xc, int64_t B, int DP,
                                                      const double *norm, float *out, int vec) {
  __shared__ float As[2][LS_K][LS_M + 4];
  __shared__ float Bs[2][LS_K][LS_M + 4];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  // block t -> tile (bi, bj), bi <= bj: t = bj (bj + 1) / 2 + bi
  const uint32_t t = blockIdx.x;
  uint32_t bj = (uint32_t)((sqrtf(8.0f * (float)t + 1.0f) - 1.0f) * 0.5f);
  while ((uint64_t)bj * (bj + 1) / 2 > t) --bj;
  while ((uint64_t)(bj + 1) * (bj + 2) / 2 <= t) ++bj;
  const uint32_t bi = t - (uint32_t)((uint64_t)bj * (bj + 1) / 2);
  const int64_t i0 = (int64_t)bi * LS_M, j0 = (int64_t)bj * LS_M;
  const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32;
  v4f_l acc[2][2][2];   // [K-tile parity]
  for (int p = 0; p < 2; ++p)
    for (int i = 0; i < 2; ++i)
      for (int j = 0; j < 2; ++j) acc[p][i][j] = v4f_l{0.f, 0.f, 0.f, 0.f};
  // thread -> row tid / 4, four columns from 4 (tid % 4) (rows past B repeat
  // the last one and are not written)
  const int lr = tid >> 2, lk = (tid & 3) * 4;
  const float *pa = xc + (i0 + lr < B ? i0 + lr : B - 1) * DP + lk;
  const float *pb = xc + (j0 + lr < B ? j0 + lr : B - 1) * DP + lk;
  float4 ra = *reinterpret_cast<const float4 *>(pa), rb = *reinterpret_cast<const float4 *>(pb);
  auto stash = [&](int buf) {
    As[buf][lk][lr] = ra.x;
    As[buf][lk + 1][lr] = ra.y;
    As[buf][lk + 2][lr] = ra.z;
    As[buf][lk + 3][lr] = ra.w;
    Bs[buf][lk][lr] = rb.x;
    Bs[buf][lk + 1][lr] = rb.y;
    Bs[buf][lk + 2][lr] = rb.z;
    Bs[buf][lk + 3][lr] = rb.w;
  };
  stash(0);
  __syncthreads();
  auto tile = [&](int k0, int buf) __attribute__((always_inline)) {   // buf: a constant
    const bool more = k0 + LS_K < DP;
    if (more) {
      ra = *reinterpret_cast<const float4 *>(pa + k0 + LS_K);
      rb = *reinterpret_cast<const float4 *>(pb + k0 + LS_K);
    }
#pragma unroll
    for (int kk = 0; kk < LS_K; kk += 4) {
      const int kr = kk + (lane >> 4), c = lane & 15;
      float av[2], bv[2];
      av[0] = As[buf][kr][wm + c];
      av[1] = As[buf][kr][wm + 16 + c];
      bv[0] = Bs[buf][kr][wn + c];
      bv[1] = Bs[buf][kr][wn + 16 + c];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[buf][i][j] =
              __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bv[j], acc[buf][i][j], 0, 0, 0);
    }
    if (more) stash(buf ^ 1);
    __syncthreads();
  };
  for (int k0 = 0; k0 < DP; k0 += 2 * LS_K) {
    tile(k0, 0);
    if (k0 + LS_K < DP) tile(k0 + LS_K, 1);
  }
  // D layout of a 16x16 block: lane l, register r -> row 4*(l/16) + r, column l%16
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int64_t cj = j0 + wn + 16 * j + (lane & 15);
      const int64_t r0 = i0 + wm + 16 * i + 4 * (lane >> 4);
      if (cj >= B) continue;
      const double nj = norm[cj];
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t ri = r0 + r;
        const double ni = norm[ri < B ? ri : B - 1];
        v[r] = (float)((ni + nj) - 2.0 * ((double)acc[0][i][j][r] + (double)acc[1][i][j][r]));
        v[r] = v[r] > 0.f ? v[r] : 0.f;
        if (ri == cj) v[r] = 0.f;
        if (ri < B) out[ri * B + cj] = v[r];
      }
      if (vec && r0 + 3 < B) {  // B a multiple of 4: the four are one aligned group
        *reinterpret_cast<float4 *>(out + cj * B + r0) = make_float4(v[0], v[1], v[2], v[3]);
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (r0 + r < B) out[cj * B + r0 + r] = v[r];
      }
    }
}

// ------------------------------------------------------------------ quantile
// The linear-interpolation quantile of the first n off-diagonal elements of
// d2 in row order (n: all of them or a limit), from the two order statistics
// around its rank.  Values are not negative, so their bits order like them:
// three passes over the matrix count digits of 11, 10 and 10 bits in LDS (a
// copy per wave: the leading digit of distances takes few values), and one
// block after each picks the digit that holds the rank.  (A pick by the last
// block of a pass needs a device-scope release by every block, which writes
// its L2 back: 90 us a pass.)  The sort that a general quantile runs moved the whole batch (4096 rows: 64 MB)
// twice per digit, 0.9 ms; this reads it three times, 0.09 ms.
constexpr int QB0 = 2048, QB1 = 1024;   // bins of the first and the later digits

struct QuantState {
  uint32_t hist[3][QB0];
  uint32_t prefix;     // digits picked so far
  uint32_t rank;       // rank among the keys of that prefix
  uint32_t above;      // least key past the prefix's range (last pass)
  uint32_t nan;        // whether an element is NaN (first pass): then so is the quantile
};

__global__ void __launch_bounds__(256) k_quant_init(QuantState *st, uint32_t rank) {
  uint32_t *h = &st->hist[0][0];
  for (int i = blockIdx.x * 256 + threadIdx.x; i < 3 * QB0; i += gridDim.x * 256) h[i] = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    st->prefix = 0;
    st->rank = rank;
    st->above = 0xffffffffu;
    st->nan = 0;
  }
}

__device__ __forceinline__ uint32_t agent_load(const uint32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int PASS>
__global__ void __launch_bounds__(256) k_pair_quantile(const float *d2, int64_t B, int64_t n,
                                                       QuantState *st, int vec) {
  constexpr int BINS = PASS == 0 ? QB0 : QB1;
  constexpr int SHIFT = PASS == 0 ? 20 : (PASS == 1 ? 10 : 0);
  __shared__ uint32_t h[4][BINS];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  for (int i = tid; i < 4 * BINS; i += 256) (&h[0][0])[i] = 0;
  __syncthreads();
  const uint32_t prefix = st->prefix;
  uint32_t above = 0xffffffffu;
  bool nan = false;
  auto count = [&](uint32_t k, bool in) {
    if (PASS == 0) {
      if (in) atomicAdd(&h[wv][k >> SHIFT], 1u);
      nan |= in && k > 0x7f800000u;
    } else {
      const uint32_t top = k >> (SHIFT + 10);
      if (in && top == prefix) atomicAdd(&h[wv][(k >> SHIFT) & 1023u], 1u);
      if (PASS == 2 && in && top > prefix && k < above) above = k;
    }
  };
  const int64_t rows = (n + B - 2) / (B - 1);   // B >= 2
  for (int64_t i = blockIdx.x; i < rows; i += gridDim.x) {
    const float *row = d2 + i * B;
    // the row's elements j < jn are among the first n, the diagonal aside
    const int64_t left = n - i * (B - 1);
    const int diag = (int)i;
    const int jn = (int)(left >= B - 1 ? B : (left > i ? left + 1 : left));
    for (int j0 = 0; j0 < jn; j0 += 16 * 256) {
      // sixteen elements per thread in flight
      float v[16];
      if (vec) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int j = j0 + (u * 256 + tid) * 4;
          const float4 x = j < (int)B ? *reinterpret_cast<const float4 *>(row + j)
                                      : make_float4(0.f, 0.f, 0.f, 0.f);
          v[4 * u] = x.x;
          v[4 * u + 1] = x.y;
          v[4 * u + 2] = x.z;
          v[4 * u + 3] = x.w;
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          const int j = j0 + ((u >> 2) * 256 + tid) * 4 + (u & 3);
          count(__float_as_uint(v[u]) & 0x7fffffffu, j < jn && j != diag);
        }
      } else {
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          const int j = j0 + u * 256 + tid;
          v[u] = j < jn ? row[j] : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          const int j = j0 + u * 256 + tid;
          count(__float_as_uint(v[u]) & 0x7fffffffu, j < jn && j != diag);
        }
      }
    }
  }
  __syncthreads();
  for (int i = tid; i < BINS; i += 256) {
    const uint32_t c = h[0][i] + h[1][i] + h[2][i] + h[3][i];
    if (c) atomicAdd(&st->hist[PASS][i], c);
  }
  if (PASS == 0 && ballot(nan) && lane == 0) atomicOr(&st->nan, 1u);
  if (PASS == 2) {
    for (int m = 1; m < WAVE; m <<= 1) {
      const uint32_t o = (uint32_t)__shfl_xor((int)above, m);
      above = o < above ? o : above;
    }
    // (most waves see a value no less than another's)
    if (lane == 0 && above < agent_load(&st->above)) atomicMin(&st->above, above);
  }
}

// the digit that holds the rank, by one block; after the last, the quantile
template <int PASS>
__global__ void __launch_bounds__(256) k_quant_pick(QuantState *st, float w, int between,
                                                    double *out) {
  constexpr int BINS = PASS == 0 ? QB0 : QB1;
  __shared__ uint32_t wsum[4];
  __shared__ uint32_t s_next;
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const uint32_t prefix = st->prefix;
  constexpr int PER = BINS / 256;
  uint32_t c[PER], sum = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    c[u] = st->hist[PASS][tid * PER + u];
    sum += c[u];
  }
  const uint32_t incl = wave_incl_scan_u32(sum);
  if (lane == WAVE - 1) wsum[wv] = incl;
  if (tid == 0) s_next = 0xffffffffu;
  __syncthreads();
  uint32_t run = incl - sum;
  for (int i = 0; i < wv; ++i) run += wsum[i];
  const uint32_t rank = st->rank;
  int at = -1;
  uint32_t below = 0, cnt = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    if (at < 0 && run <= rank && rank < run + c[u]) {
      at = tid * PER + u;
      below = run;
      cnt = c[u];
    }
    run += c[u];
  }
  __syncthreads();   // every thread has read the state
  if (PASS < 2) {
    if (at >= 0) {
      st->prefix = PASS == 0 ? (uint32_t)at : (prefix << 10) | (uint32_t)at;
      st->rank = rank - below;
    }
    return;
  }
  // the value of the rank, and the one after it: in the same bin, in the next
  // occupied bin of the prefix, or the least key past the prefix
  __shared__ uint32_t s_at, s_same;
  if (at >= 0) {
    s_at = (uint32_t)at;
    s_same = rank - below + 1 < cnt;
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const uint32_t b = (uint32_t)(tid * PER + u);
    if (c[u] && b > s_at) atomicMin(&s_next, b);
  }
  __syncthreads();
  if (tid == 0) {
    const uint32_t lo = (prefix << 10) | s_at;
    uint32_t hi = lo;
    if (between && !s_same)
      hi = s_next != 0xffffffffu ? (prefix << 10) | s_next : st->above;
    const float a = __uint_as_float(lo), b = __uint_as_float(hi);
    // the interpolation of torch.quantile (its lerp)
    const float d = b - a;
    *out = st->nan ? (double)NAN : (double)(w < 0.5f ? fmaf(w, d, a) : fmaf(-d, 1.0f - w, b));
  }
}

size_t pair_quantile_ws_bytes() { return sizeof(QuantState); }

hipError_t launch_pair_quantile(const float *d2, int64_t B, int64_t n, float q, void *ws,
                                double *out, hipStream_t s) {
  QuantState *st = static_cast<QuantState *>(ws);
  // the rank in fp32, as torch.quantile takes it for fp32 input
  const float r = q * (float)(n - 1);
  const float f = floorf(r);
  const float w = r - f;
  const int between = ceilf(r) > f ? 1 : 0;
  hipLaunchKernelGGL(k_quant_init, dim3(8), dim3(256), 0, s, st, (uint32_t)f);
  const int64_t rows = (n + B - 2) / (B - 1);
  const dim3 grid((unsigned)(rows < 1024 ? rows : 1024));
  // 16-byte loads where every row starts on a 16-byte boundary
  const int vec = B % 4 == 0 && (reinterpret_cast<uintptr_t>(d2) & 15) == 0;
  hipLaunchKernelGGL(k_pair_quantile<0>, grid, dim3(256), 0, s, d2, B, n, st, vec);
  hipLaunchKernelGGL(k_quant_pick<0>, dim3(1), dim3(256), 0, s, st, w, between, out);
  hipLaunchKernelGGL(k_pair_quantile<1>, grid, dim3(256), 0, s, d2, B, n, st, vec);
  hipLaunchKernelGGL(k_quant_pick<1>, dim3(1), dim3(256), 0, s, st, w, between, out);
  hipLaunchKernelGGL(k_pair_quantile<2>, grid, dim3(256), 0, s, d2, B, n, st, vec);
  hipLaunchKernelGGL(k_quant_pick<2>, dim3(1), dim3(256), 0, s, st, w, between, out);
  return hipGetLastError();
}

// ------------------------------------------------------------------ loss and gradient
// A block owns LG_COLS rows of the gradient: lane l of a wave holds row
// j = LG_COLS blockIdx + l % 16 and its running gradient in registers, and the
// block's 64 (wave, l / 16) subsets share the other rows i, whose latents are
// staged in LDS LG_TILE at a time (four rows per wave read at once, the same
// for 16 lanes).  Nothing crosses lanes until the end.  4096 rows of 24: 305 us
// with a wave per gradient row (48 LDS reads per pair and a butterfly over 24
// gradients), 72 us so.
constexpr int LG_COLS = 16, LG_TILE = 256, LG_WAVES = 16, LG_SUB = 4 * LG_WAVES;

// the largest x with sqrtf(x) <= thr (negative: none), so that the mask's
// comparisons need no square root
__device__ __forceinline__ float sqrt_bound(float thr) {
  if (!(thr >= 0.0f)) return -1.0f;
  if (thr == INFINITY) return INFINITY;
  float x = thr * thr;
  while (sqrtf(x) > thr) x = __uint_as_float(__float_as_uint(x) - 1u);
  for (;;) {
    const float y = __uint_as_float(__float_as_uint(x) + 1u);
    if (!(sqrtf(y) <= thr)) break;
    x = y;
  }
  return x;
}

template <int L>
__global__ void __launch_bounds__(64 * LG_WAVES) k_lsim_grad(const float *d2, const float *lat,
                                                              int64_t B, float gr, float tau,
                                                              const double *tau2, double *num_cnt,
                                                              float *grad) {
  // rows of whole 16-byte groups, an odd number of them, so that four rows
  // start in different banks
  constexpr int LP = ((L + 3) / 4 * 4) | 4;
  __shared__ __attribute__((aligned(16))) float li_s[LG_TILE * LP];
  __shared__ double red[LG_WAVES];
  __shared__ uint32_t redc[LG_WAVES];
  const int tid = threadIdx.x;
  const int lane = tid & (WAVE - 1), wv = tid / WAVE;
  const int sub = wv * 4 + (lane >> 4);
  const int64_t j = (int64_t)blockIdx.x * LG_COLS + (lane & 15);
  const bool col_ok = j < B;
  if (tau2) tau = (float)sqrt(*tau2);
  const float emb_max = sqrt_bound(tau), lat_max = sqrt_bound(gr * tau);
  float lj[L], g[L];
#pragma unroll
  for (int c = 0; c < L; ++c) {
    lj[c] = lat[(col_ok ? j : 0) * L + c];
    g[c] = 0.f;
  }
  double num = 0.0;
  uint32_t cnt = 0;
  for (int64_t i0 = 0; i0 < B; i0 += LG_TILE) {
    __syncthreads();
    const int rows = (int)(B - i0 < LG_TILE ? B - i0 : LG_TILE);
    for (int e = tid; e < rows * L; e += 64 * LG_WAVES) {
      const int r = e / L;
      li_s[r * LP + (e - r * L)] = lat[i0 * L + e];
    }
    float dv[LG_TILE / LG_SUB];
#pragma unroll
    for (int u = 0; u < LG_TILE / LG_SUB; ++u) {
      const int64_t i = i0 + sub + u * LG_SUB;
      dv[u] = col_ok && i < B ? d2[i * B + j] : INFINITY;
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < LG_TILE / LG_SUB; ++u) {
      const int r = sub + u * LG_SUB;
      const bool ok = col_ok && r < rows && i0 + r != j;
      const float4 *row = reinterpret_cast<const float4 *>(li_s + (r < rows ? r : 0) * LP);
      float t[L];
      float sl2 = 0.f;
#pragma unroll
      for (int c4 = 0; c4 < (L + 3) / 4; ++c4) {
        const float4 v = row[c4];
        const float vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int x = 0; x < 4; ++x)
          if (4 * c4 + x < L) {
            t[4 * c4 + x] = lj[4 * c4 + x] - vv[x];
            sl2 = fmaf(t[4 * c4 + x], t[4 * c4 + x], sl2);
          }
      }
      if (!(ok && (dv[u] <= emb_max || sl2 <= lat_max))) continue;
      const float sl = sqrtf(sl2);
      const float dd = sl - gr * sqrtf(dv[u]);
      num += (double)dd * (double)dd;
      cnt += 1;
      // the pairs (i, j) and (j, i) contribute alike
      const float coef = 4.0f * dd;
      if (coef != 0.f && sl > 0.f) {
        const float s = coef / sl;
#pragma unroll
        for (int c = 0; c < L; ++c) g[c] = fmaf(s, t[c], g[c]);
      }
    }
  }
  // the gradient: a wave's four subsets, then the waves, in a fixed order
  __syncthreads();
  float *gs = li_s;   // [wave][column][L]
#pragma unroll
  for (int c = 0; c < L; ++c) {
    float v = g[c];
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    if (lane < 16) gs[(wv * LG_COLS + lane) * L + c] = v;
  }
  for (int m = 1; m < WAVE; m <<= 1) {
    num += __shfl_xor(num, m);
    cnt += (uint32_t)__shfl_xor((int)cnt, m);
  }
  if (lane == 0) {
    red[wv] = num;
    redc[wv] = cnt;
  }
  __syncthreads();
  for (int e = tid; e < LG_COLS * L; e += 64 * LG_WAVES) {
    float v = 0.f;
    for (int k = 0; k < LG_WAVES; ++k) v += gs[k * LG_COLS * L + e];
    const int64_t jj = (int64_t)blockIdx.x * LG_COLS + e / L;
    if (jj < B) grad[jj * L + e % L] = v;
  }
  if (tid == 0) {
    double tn = 0.0, tc = 0.0;
    for (int k = 0; k < LG_WAVES; ++k) {
      tn += red[k];
      tc += (double)redc[k];
    }
    atomicAdd(&num_cnt[0], tn);
    atomicAdd(&num_cnt[1], tc);
  }
}

static int center_stride(int D) { return (D + LS_K - 1) / LS_K * LS_K; }

size_t pair_sqdist_ws_floats(int64_t B, int D) {
  // the centred rows from a 16-byte boundary on, then norms, partial sums, ranges, means
  return 4 + (size_t)B * center_stride(D) +
         (size_t)(2 * ((B + LS_ROWS - 1) / LS_ROWS) + 1) * (size_t)D + 2 * (size_t)B;
}

hipError_t launch_pair_sqdist(const float *x, int64_t B, int D, float *ws, float *out,
                              hipStream_t s) {
  if (B <= 0) return hipSuccess;
  const int64_t nblk = (B + LS_ROWS - 1) / LS_ROWS;
  const int DP = center_stride(D);
  float *xc = reinterpret_cast<float *>((reinterpret_cast<uintptr_t>(ws) + 15) & ~(uintptr_t)15);
  double *norm = reinterpret_cast<double *>(xc + B * DP);   // DP: whole 64-byte groups
  float *partial = reinterpret_cast<float *>(norm + B), *range = partial + nblk * D;
  float *mean = range + nblk * D;
  hipLaunchKernelGGL(k_col_partial, dim3((unsigned)nblk), dim3(128), 0, s, x, B, D, partial, range);
  hipLaunchKernelGGL(k_col_mean, dim3((unsigned)((D + 63) / 64)), dim3(128), 0, s, partial, range,
                     nblk, B, D, mean);
  hipLaunchKernelGGL(k_center, dim3((unsigned)((B + 3) / 4)), dim3(256), 0, s, x, B, D, DP, mean,
                     xc, norm);
  const int64_t gb = (B + LS_M - 1) / LS_M;
  const int vec = B % 4 == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0;
  hipLaunchKernelGGL(k_pair_sqdist, dim3((unsigned)(gb * (gb + 1) / 2)), dim3(256), 0, s, xc, B,
                     DP, norm, out, vec);
  return hipGetLastError();
}

template <int L>
static void launch_lsim_l(const float *d2, const float *lat, int64_t B, int l, float gr, float tau,
                          const double *tau2, double *num_cnt, float *grad, hipStream_t s) {
  if (l == L) {
    hipLaunchKernelGGL(k_lsim_grad<L>, dim3((unsigned)((B + LG_COLS - 1) / LG_COLS)),
                       dim3(64 * LG_WAVES), 0, s, d2, lat, B, gr, tau, tau2, num_cnt, grad);
  } else if constexpr (L < 32) {
    launch_lsim_l<L + 1>(d2, lat, B, l, gr, tau, tau2, num_cnt, grad, s);
  }
}

// tau2 (may be NULL): a device copy of tau_emb's square, used instead of tau
hipError_t launch_lsim_grad(const float *d2, const float *lat, int64_t B, int L, float gr,
                            float tau, const double *tau2, double *num_cnt, float *grad,
                            hipStream_t s) {
  if (B <= 0) return hipSuccess;
  hipError_t e = launch_fill_i32((int32_t *)num_cnt, 4, 0, s);
  if (e != hipSuccess) return e;
  launch_lsim_l<1>(d2, lat, B, L, gr, tau, tau2, num_cnt, grad, s);
  return hipGetLastError();
}

}  // namespace nr
