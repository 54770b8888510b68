// Step 1: encoder forward pass (Sec. 3.2.1; architecture Sec. 4.5, App. A),
// one launch per linear layer, or one for the last two (k_encode_pair).  Each layer is a dense contraction
//   out[m][n] = act( in_scale * sum_k in[m][k] * W[n][k] + bias[n] )
// on the fp32 matrix cores (v_mfma_f32_16x16x4f32).  A 256-thread block owns a
// BM x BN output tile and each of its four waves a (BM/2) x (BN/2) quarter, as
// (BM/32) x (BN/32) blocks of 16 x 16.  K is staged through LDS BK at a time in
// two buffers (the next tile is read into registers while the current one is
// multiplied; one barrier per tile); uint8 inputs are widened while staging,
// and rows whose length is a multiple of 4 are read 4 elements per load.
// Every output is one MFMA chain over k in increasing order, 4 at a time,
// whatever the tile shape, so the logits do not depend on it.
// Hidden layers fold eval-mode BatchNorm (per-channel scale and shift) and
// ReLU into the epilogue; the last layer writes the logits.
#include "nr_internal.h"

namespace nr {

typedef float v4f __attribute__((ext_vector_type(4)));


// element (m, kg) of the input, zero outside [0, M) x [0, K)
__device__ __forceinline__ float enc_load_in(const EncodeLayerArgs &a, int64_t m, int kg) {
  if (m >= a.M || kg >= a.K) return 0.f;
  return a.in_u8 ? (float)((const uint8_t *)a.in)[m * a.K + kg]
                 : ((const float *)a.in)[m * a.K + kg];
}

// elements (m, kg .. kg+3) of the input (K a multiple of 4, so the four are
// all inside or all past the row)
__device__ __forceinline__ float4 enc_load_in4(const EncodeLayerArgs &a, int64_t m, int kg) {
  if (m >= a.M || kg >= a.K) return make_float4(0.f, 0.f, 0.f, 0.f);
  if (a.in_u8) {
    const uint32_t v = *reinterpret_cast<const uint32_t *>((const uint8_t *)a.in + m * a.K + kg);
    return make_float4((float)(v & 0xffu), (float)((v >> 8) & 0xffu), (float)((v >> 16) & 0xffu),
                       (float)(v >> 24));
  }
  return *reinterpret_cast<const float4 *>((const float *)a.in + m * a.K + kg);
}

__device__ __forceinline__ float4 enc_load_w4(const EncodeLayerArgs &a, int n, int kg) {
  if (n >= a.N || kg >= a.K) return make_float4(0.f, 0.f, 0.f, 0.f);
  return *reinterpret_cast<const float4 *>(a.W + (int64_t)n * a.K + kg);
}

// Two orders of a K-tile of 16 in LDS.  By row: KS floats apart, k = 4 s + g at
// slot 4 g + s, so that the operands of lane l of a 16x16x4 block (k = l / 16 of
// each of four steps) are one 16-byte read, and reads and writes fall on
// different banks.  By k: a row of operands per k, a read per operand, up to
// three lanes on a bank, but a K-tile's reads spread over its steps.  Layers by
// row / by k, us: 32 x 64 tiles 1 to 9 % faster by row (16,384 x 256 -> 64 17.3 /
// 18.8, 32,768 uint8 rows of 1536 -> 128 185 / 199); 64 x 64 tiles, two layers K -> N
// -> 16, fp32 slower by row (16,384 rows of 512 -> 512 114 / 105, 512 -> 1024 217 / 198,
// 1536 -> 512 283 / 258), uint8 rows faster for long K and N up to 512 (8,192 of
// 1536 -> 512 155 / 166, 16,384 of 1536 -> 256 146 / 154; but 12,288 of 768 -> 1024
// 242 / 223); code layers (32 x 32) slower by row from K = 512 on (12,288 rows of 64 ->
// 1024 -> 16 69 / 66).
// Tiles of 128 x 64, 64 x 128 and 128 x 128 are no faster (5, 4 and 24 % slower
// for the 1536-d encoder)
constexpr int KS = 20;
__device__ __forceinline__ constexpr int enc_slot(int k) { return 4 * (k & 3) + (k >> 2); }

template <int MI, int NJ>
__device__ __forceinline__ void enc_ktile(v4f (&acc)[MI][NJ], const float *A, const float *W) {
  const int at = (lane_id() & 15) * KS + 4 * (lane_id() >> 4);
  float4 a4[MI], b4[NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i) a4[i] = *reinterpret_cast<const float4 *>(A + 16 * i * KS + at);
#pragma unroll
  for (int j = 0; j < NJ; ++j) b4[j] = *reinterpret_cast<const float4 *>(W + 16 * j * KS + at);
#pragma unroll
  for (int s = 0; s < 4; ++s)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const float av = s == 0 ? a4[i].x : s == 1 ? a4[i].y : s == 2 ? a4[i].z : a4[i].w;
        const float bv = s == 0 ? b4[j].x : s == 1 ? b4[j].y : s == 2 ? b4[j].z : b4[j].w;
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv, acc[i][j], 0, 0, 0);
      }
}

template <int BM, int BN, int BK, bool VEC, bool ROWS>
__global__ void __launch_bounds__(256) k_encode_layer(EncodeLayerArgs a) {
  constexpr int MI = BM / 32, NJ = BN / 32;  // 16 x 16 blocks per wave
  constexpr int VW = VEC ? 4 : 1;            // elements per load
  constexpr int LA = BM * BK / VW, LW = BN * BK / VW;  // loads per tile
  constexpr int PA = (LA + 255) / 256, PW = (LW + 255) / 256;  // per thread (at most)
  static_assert(BK == 16 && BM % 32 == 0 && BN % 32 == 0, "whole MFMA blocks");
  // two K-tiles of A (activations) and W
  __shared__ __attribute__((aligned(16))) float As[2][ROWS ? BM * KS : BK * (BM + 4)];
  __shared__ __attribute__((aligned(16))) float Ws[2][ROWS ? BN * KS : BK * (BN + 4)];
  auto at = [](int rows, int r, int k) {
    return ROWS ? r * KS + enc_slot(k) : k * (rows + 4) + r;
  };
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  // tile of this block: the column tiles of one row tile are consecutive
  // blocks on the same XCD (blocks go to XCDs in turn, block id mod 8), so
  // they share that XCD's L2 copy of the row tile's inputs
  const int64_t nb = (a.N + BN - 1) / BN;
  const int64_t t8 = (int64_t)(blockIdx.x >> 3);
  const int64_t u = (t8 / nb) * 8 + (blockIdx.x & 7);
  if (u * BM >= a.M) return;  // a slot past the last row tile
  const int64_t m0 = u * BM;
  const int n0 = (int)(t8 % nb) * BN;
  const int wm = (wave & 1) * (BM / 2), wn = (wave >> 1) * (BN / 2);
  const int K = a.K, N = a.N;
  v4f acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
  // load e of a tile: row e / (BK / VW), elements VW * (e % (BK / VW)) onwards
  // (consecutive threads read consecutive elements of a row)
  float ra[PA][VW], rw[PW][VW];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int u = 0; u < PA; ++u) {
      const int e = tid + 256 * u;
      const int r = e / (BK / VW), kk = VW * (e % (BK / VW));
      if (LA % 256 != 0 && e >= LA) continue;
      if constexpr (VEC) {
        const float4 v = enc_load_in4(a, m0 + r, k0 + kk);
        ra[u][0] = v.x;
        ra[u][VW > 1 ? 1 : 0] = v.y;
        ra[u][VW > 2 ? 2 : 0] = v.z;
        ra[u][VW > 3 ? 3 : 0] = v.w;
      } else {
        ra[u][0] = enc_load_in(a, m0 + r, k0 + kk);
      }
    }
#pragma unroll
    for (int u = 0; u < PW; ++u) {
      const int e = tid + 256 * u;
      const int r = e / (BK / VW), kk = VW * (e % (BK / VW));
      if (LW % 256 != 0 && e >= LW) continue;
      if constexpr (VEC) {
        const float4 v = enc_load_w4(a, n0 + r, k0 + kk);
        rw[u][0] = v.x;
        rw[u][VW > 1 ? 1 : 0] = v.y;
        rw[u][VW > 2 ? 2 : 0] = v.z;
        rw[u][VW > 3 ? 3 : 0] = v.w;
      } else {
        const int n = n0 + r, kg = k0 + kk;
        rw[u][0] = (n < N && kg < K) ? a.W[(int64_t)n * K + kg] : 0.f;
      }
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int u = 0; u < PA; ++u) {
      const int e = tid + 256 * u;
      const int r = e / (BK / VW), kk = VW * (e % (BK / VW));
      if (LA % 256 != 0 && e >= LA) continue;
#pragma unroll
      for (int v = 0; v < VW; ++v) As[buf][at(BM, r, kk + v)] = ra[u][v];
    }
#pragma unroll
    for (int u = 0; u < PW; ++u) {
      const int e = tid + 256 * u;
      const int r = e / (BK / VW), kk = VW * (e % (BK / VW));
      if (LW % 256 != 0 && e >= LW) continue;
#pragma unroll
      for (int v = 0; v < VW; ++v) Ws[buf][at(BN, r, kk + v)] = rw[u][v];
    }
  };
  fetch(0);
  stash(0);
  __syncthreads();
  int buf = 0;
  for (int k0 = 0; k0 < K; k0 += BK) {
    const bool more = k0 + BK < K;
    if (more) fetch(k0 + BK);
    if constexpr (ROWS) {
      enc_ktile<MI, NJ>(acc, &As[buf][wm * KS], &Ws[buf][wn * KS]);
    } else {
#pragma unroll
      for (int kk = 0; kk < BK; kk += 4) {
        // A operand of a 16x16x4 block: lane l holds row l % 16, k l / 16
        const int kr = kk + (lane >> 4), c = lane & 15;
        float av[MI], bv[NJ];
#pragma unroll
        for (int i = 0; i < MI; ++i) av[i] = As[buf][at(BM, wm + 16 * i + c, kr)];
#pragma unroll
        for (int j = 0; j < NJ; ++j) bv[j] = Ws[buf][at(BN, wn + 16 * j + c, kr)];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[i], bv[j], acc[i][j], 0, 0, 0);
      }
    }
    if (more) stash(buf ^ 1);
    __syncthreads();
    buf ^= 1;
  }
  const int64_t M = a.M;
  // D layout of a 16x16 block: lane l, register r -> row 4*(l/16) + r, column l%16
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int n = n0 + wn + 16 * j + (lane & 15);
      if (n >= N) continue;
      const float bias = a.bias ? a.bias[n] : 0.f;
      const float sc = a.bn_scale ? a.bn_scale[n] : 1.f;
      const float sh = a.bn_shift ? a.bn_shift[n] : 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t m = m0 + wm + 16 * i + 4 * (lane >> 4) + r;
        if (m >= M) continue;
        float v = acc[i][j][r] * a.in_scale + bias;
        if (a.relu) {
          v = v * sc + sh;
          v = v > 0.f ? v : 0.f;
        }
        a.out[m * N + n] = v;
      }
    }
}

// The last hidden layer and the code layer (at most 32 outputs) in one kernel:
// a block owns BM rows, computes their hidden activations 64 at a time as above
// (the next tile's first loads go out before its products), passes them through
// LDS and adds each 64's products to the code layer's accumulators.  k runs in
// increasing order in both chains, so the logits are those of the two kernels
// bit for bit; the activations (1 KB a row at 256) never reach memory, and all
// rows go in one launch.  Bound by the fp32 matrix cores.
template <int BM, bool VEC>
__global__ void __launch_bounds__(256) k_encode_pair(EncodeLayerArgs a, EncodeLayerArgs z) {
  constexpr int BN = 64, BK = 16;
  constexpr int MI = BM / 32, NJ = 2;
  constexpr int VW = VEC ? 4 : 1;
  constexpr int LA = BM * BK / VW, LW = BN * BK / VW;
  constexpr int PA = (LA + 255) / 256, PW = (LW + 255) / 256;
  __shared__ __attribute__((aligned(16))) float As[2][BM][KS];
  __shared__ __attribute__((aligned(16))) float Ws[2][BN][KS];
  __shared__ __attribute__((aligned(16))) float Hs[BN][BM + 4];  // activations, [k][row]
  __shared__ float Zs[BN][32 + 4];                               // code layer, [k][output]
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int64_t m0 = (int64_t)blockIdx.x * BM;
  const int wm = (wave & 1) * (BM / 2), wn = (wave >> 1) * (BN / 2);
  const int K = a.K, N = a.N, NZ = z.N;
  float ra[PA][VW], rw[PW][VW];
  auto fetch = [&](int n0, int k0) {
#pragma unroll
    for (int u = 0; u < PA; ++u) {
      const int e = tid + 256 * u;
      const int r = e / (BK / VW), kk = VW * (e % (BK / VW));
      if (LA % 256 != 0 && e >= LA) continue;
      if constexpr (VEC) {
        const float4 v = enc_load_in4(a, m0 + r, k0 + kk);
        ra[u][0] = v.x;
        ra[u][VW > 1 ? 1 : 0] = v.y;
        ra[u][VW > 2 ? 2 : 0] = v.z;
        ra[u][VW > 3 ? 3 : 0] = v.w;
      } else {
        ra[u][0] = enc_load_in(a, m0 + r, k0 + kk);
      }
    }
#pragma unroll
    for (int u = 0; u < PW; ++u) {
      const int e = tid + 256 * u;
      const int r = e / (BK / VW), kk = VW * (e % (BK / VW));
      if (LW % 256 != 0 && e >= LW) continue;
      if constexpr (VEC) {
        const float4 v = enc_load_w4(a, n0 + r, k0 + kk);
        rw[u][0] = v.x;
        rw[u][VW > 1 ? 1 : 0] = v.y;
        rw[u][VW > 2 ? 2 : 0] = v.z;
        rw[u][VW > 3 ? 3 : 0] = v.w;
      } else {
        const int n = n0 + r, kg = k0 + kk;
        rw[u][0] = (n < N && kg < K) ? a.W[(int64_t)n * K + kg] : 0.f;
      }
    }
  };
  auto stash = [&](int buf) {
#pragma unroll
    for (int u = 0; u < PA; ++u) {
      const int e = tid + 256 * u;
      const int r = e / (BK / VW), kk = VW * (e % (BK / VW));
      if (LA % 256 != 0 && e >= LA) continue;
#pragma unroll
      for (int v = 0; v < VW; ++v) As[buf][r][enc_slot(kk + v)] = ra[u][v];
    }
#pragma unroll
    for (int u = 0; u < PW; ++u) {
      const int e = tid + 256 * u;
      const int r = e / (BK / VW), kk = VW * (e % (BK / VW));
      if (LW % 256 != 0 && e >= LW) continue;
#pragma unroll
      for (int v = 0; v < VW; ++v) Ws[buf][r][enc_slot(kk + v)] = rw[u][v];
    }
  };
  // the wave's 16 x 16 blocks of the code layer: BM / 16 row blocks x 2
  constexpr int NZB = BM / 32;
  const int zr = BM == 64 ? wave : (wave & 1);
  v4f zacc[NZB];
#pragma unroll
  for (int i = 0; i < NZB; ++i) zacc[i] = v4f{0.f, 0.f, 0.f, 0.f};
  fetch(0, 0);
  for (int n0 = 0; n0 < N; n0 += BN) {
    // this tile's part of the code layer: thread -> k tid % 64, outputs tid / 64 + 4 i
    float rz[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int k = n0 + (tid & 63), n = (tid >> 6) + 4 * i;
      rz[i] = k < N && n < NZ ? z.W[(int64_t)n * N + k] : 0.f;
    }
    v4f acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};
    stash(0);
    __syncthreads();
    int buf = 0;
    for (int k0 = 0; k0 < K; k0 += BK) {
      const bool more = k0 + BK < K;
      if (more) fetch(n0, k0 + BK);
      enc_ktile<MI, NJ>(acc, &As[buf][wm][0], &Ws[buf][wn][0]);
      if (more) stash(buf ^ 1);
      __syncthreads();
      buf ^= 1;
    }
    if (n0 + BN < N) fetch(n0 + BN, 0);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int col = wn + 16 * j + (lane & 15), n = n0 + col;
      const bool ok = n < N;
      const float bias = ok && a.bias ? a.bias[n] : 0.f;
      const float sc = ok && a.bn_scale ? a.bn_scale[n] : 1.f;
      const float sh = ok && a.bn_shift ? a.bn_shift[n] : 0.f;
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          v[r] = acc[i][j][r] * a.in_scale + bias;
          v[r] = v[r] * sc + sh;
          v[r] = ok && v[r] > 0.f ? v[r] : 0.f;
        }
        *reinterpret_cast<float4 *>(&Hs[col][wm + 16 * i + 4 * (lane >> 4)]) =
            make_float4(v[0], v[1], v[2], v[3]);
      }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) Zs[tid & 63][(tid >> 6) + 4 * i] = rz[i];
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < BN; kk += 4) {
      const int kr = kk + (lane >> 4), c = lane & 15;
      const float av = Hs[kr][16 * zr + c];
#pragma unroll
      for (int i = 0; i < NZB; ++i) {
        const int zc = BM == 64 ? i : (wave >> 1);
        zacc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, Zs[kr][16 * zc + c], zacc[i], 0, 0, 0);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NZB; ++i) {
    const int zc = BM == 64 ? i : (wave >> 1);
    const int n = 16 * zc + (lane & 15);
    if (n >= NZ) continue;
    const float bias = z.bias ? z.bias[n] : 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int64_t m = m0 + 16 * zr + 4 * (lane >> 4) + r;
      if (m < a.M) z.out[m * NZ + n] = zacc[i][r] * z.in_scale + bias;
    }
  }
}

// A pair goes to one kernel where the rows fill the chip by themselves: a block
// walks all of the hidden layer with three blocks to a CU (LDS), so few rows end
// with few blocks' chains (65,536 rows are 1.3 rounds of the chip), and longer
// chains (K) and more of them (N) hide less of their loads than the layer kernel's
// seven blocks do.  Layers go 16,384 rows at a time, the last ones in a launch of
// their own.  Two kernels / one, us, fp32 rows (uint8 rows in brackets), K -> N -> 16:
//   16,384 rows: 128 -> 256 32 / 26, 256 -> 128 26 / 24, 512 -> 64 28 / 23, 256 -> 256 41 / 42
//     (43 / 46), 512 -> 128 40 / 42, 128 -> 1024 90 / 91 (92 / 98)
//   20,000 rows: 256 -> 256 60 / 51, 512 -> 128 60 / 49, 768 -> 64 62 / 37
//   32,768 rows: 256 -> 512 139 / 125, 256 -> 1024 252 / 239 (but 50,000 406 / 439), 512 ->
//     256 120 / 115 (but 40,000 (167 / 183))
//   65,536 rows: 512 -> 256 233 / 203, 512 -> 512 411 / 403 (422 / 494), 768 -> 256 312 / 295
//     (334 / 407), 768 -> 512 568 / 584 (100,000: 891 / 968), 1536 -> 128 373 / 313 (378 /
//     400, 80,000: 449 / 406), 256 -> 1024 492 / 439, 768 -> 1024 1076 / 1160, 1536 -> 512 1018 / 1239 (1031 / 1439)
//   131,072 rows: (512 -> 512 845 / 788), 512 -> 1024 1566 / 1461 (1591 / 1565), (768 -> 256
//     669 / 630), (768 -> 512 1146 / 1235), 1536 -> 256 1128 / 1132, 1536 -> 512 2027 / 2233
// 1M rows of 128 -> 256 -> 24: 1.96 ms in two kernels per 16,384 rows, 0.97 in
// one (84 TFLOP/s of fp32).  One query behind 128 -> 256 -> 16: a whole search 64 us
// with two kernels, 74 with one
bool encode_pair(int64_t M, int K, int N, int NZ, bool u8) {
  const int64_t KN = (int64_t)K * N;
  if (NZ > 32) return false;
  if (KN <= 32768 || (KN <= 65536 && (K <= 128 || N <= 64))) return M >= 16384;
  if (KN <= 65536 || K <= 128) return M > 16384;
  if (K <= 256) return M >= (KN <= 131072 ? 32768 : 65536);
  if (KN <= 131072 || (!u8 && (KN <= 196608 || (K <= 768 && KN <= 262144)))) return M >= 65536;
  if (KN <= 196608 && N <= 128) return M >= 73728;
  return (K <= 512 || KN <= 196608) && M >= 131072;
}

hipError_t launch_encode_pair(const EncodeLayerArgs &a, const EncodeLayerArgs &z, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if (z.N > 32 || z.K != a.N || !a.relu || z.relu) return hipErrorInvalidValue;
  const bool vec = a.K % 4 == 0 && (reinterpret_cast<uintptr_t>(a.in) & 15) == 0 &&
                   (reinterpret_cast<uintptr_t>(a.W) & 15) == 0;
  // 64 rows a block where that still gives each CU three (the LDS's share)
  const bool big = a.M >= 64 * 768;
  const dim3 grid((unsigned)(big ? (a.M + 63) / 64 : (a.M + 31) / 32));
  if (big && vec)
    hipLaunchKernelGGL((k_encode_pair<64, true>), grid, dim3(256), 0, s, a, z);
  else if (big)
    hipLaunchKernelGGL((k_encode_pair<64, false>), grid, dim3(256), 0, s, a, z);
  else if (vec)
    hipLaunchKernelGGL((k_encode_pair<32, true>), grid, dim3(256), 0, s, a, z);
  else
    hipLaunchKernelGGL((k_encode_pair<32, false>), grid, dim3(256), 0, s, a, z);
  return hipGetLastError();
}

template <int BM, int BN, int BK, bool ROWS>
static hipError_t launch_tile(const EncodeLayerArgs &a, hipStream_t s) {
  // row tiles in groups of 8 (one per XCD), each with all its column tiles
  const int64_t nm = (a.M + BM - 1) / BM, nn = (a.N + BN - 1) / BN;
  const dim3 grid((unsigned)(((nm + 7) / 8) * 8 * nn));
  // four-element loads need rows (and so every row start) 4-element aligned
  const bool vec = a.K % 4 == 0 && (reinterpret_cast<uintptr_t>(a.in) & 15) == 0 &&
                   (reinterpret_cast<uintptr_t>(a.W) & 15) == 0;
  if (vec)
    hipLaunchKernelGGL((k_encode_layer<BM, BN, BK, true, ROWS>), grid, dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((k_encode_layer<BM, BN, BK, false, ROWS>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

// Tile shapes measured on MI355X (10,000 queries): 64 x 64 where that still
// gives the chip about four blocks per CU (the 1536 -> 512 layer: 196 us for
// the whole 1536-d encoder, 255 us with 64 x 64 x 32 tiles and one load per
// element), 32 x 64 for smaller layers (128 -> 256: the 1B encoder in 22 us
// against 29 us with 64 x 64), 32 x 32 for the code layer (at most 32 outputs)
hipError_t launch_encode_layer(const EncodeLayerArgs &a, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if (a.N <= 32)
    return a.K < 512 ? launch_tile<32, 32, 16, true>(a, s) : launch_tile<32, 32, 16, false>(a, s);
  const int64_t tiles64 = ((a.M + 63) / 64) * ((a.N + 63) / 64);
  if (tiles64 >= 1024)
    return a.in_u8 && a.K >= 512 && a.N <= 512 ? launch_tile<64, 64, 16, true>(a, s)
                                               : launch_tile<64, 64, 16, false>(a, s);
  return launch_tile<32, 64, 16, true>(a, s);
}

}  // namespace nr
