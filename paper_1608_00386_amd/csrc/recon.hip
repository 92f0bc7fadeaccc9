// recon_apply: reconstructor (control matrix) times slopes, C = alpha R S^T + beta C
// (Sec. 2.6-2.7 of the paper: slopes multiplied by the control matrix give the differential
// coefficients added to the mirror).  R is [M][N] row-major FP32 and is streamed from HBM once
// per call; that stream bounds the operation (4 flop per byte of R at B = 8).
//
//   B == 1      : split-K streaming GEMV on the vector ALUs
//   2 <= B <= 8 : the same streaming order with every realisation at once (vector ALUs; R read
//                 once in 1 KB bursts per row, the slopes staged in LDS per workgroup)
//   B > 8       : split-K GEMM on the FP32 matrix cores, up to 32 realisations a pass, R and
//                 the slopes staged in LDS
// Both write per-split partial sums to a workspace; a second kernel adds the splits in a fixed
// order and applies alpha/beta, so results are deterministic.  R and S need no more than their
// natural 4-byte alignment: 16-byte loads of any row (N need not be a multiple of 4) take the
// hardware's unaligned access, the last 1-3 columns of a row element by element.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/wfs.h"
#include "wfs_common.h"

namespace wfs {

constexpr int kRB = 256;
constexpr int kBatchRW = 8;  // rows per wave of the small-batch kernel
constexpr int kBatchMax = 8;  // realisations of the small-batch kernel
constexpr bool kBatchPF = true;  // small-batch kernel: next slice's rows of R in flight

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v4fu __attribute__((ext_vector_type(4), aligned(4)));

// 16-byte streaming load of R (read once per call: non-temporal), 4-byte aligned
__device__ __forceinline__ float4 ldnt4(const float* p) {
  const v4fu v = __builtin_nontemporal_load(reinterpret_cast<const v4fu*>(p));
  return make_float4(v.x, v.y, v.z, v.w);
}

__device__ __forceinline__ float4 ld4(const float* p) {
  const v4fu v = *reinterpret_cast<const v4fu*>(p);
  return make_float4(v.x, v.y, v.z, v.w);
}

// Columns k .. k + 3 of a row below k1, zero past it.
template <bool NT>
__device__ __forceinline__ float4 ld4_below(const float* row, int k, int k1) {
  if (k + 4 <= k1) return NT ? ldnt4(row + k) : ld4(row + k);
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  if (k < k1) v.x = row[k];
  if (k + 1 < k1) v.y = row[k + 1];
  if (k + 2 < k1) v.z = row[k + 2];
  return v;
}

// Four products, added to a lane's sum at once: a quarter of the roundings of its growing sum
// (one realisation of 55,608 columns: rms 5.3 -> 2.4 in 2^-24 of the root of the sum of squares,
// for one instruction more in four).
__device__ __forceinline__ float dot4(float4 r, float4 s) {
  return fmaf(r.x, s.x, fmaf(r.y, s.y, fmaf(r.z, s.z, r.w * s.w)));
}

// ---------------------------------------------------------------------------------------
// GEMV / generic: wave per (RW rows, split); lanes stride over k.
// ---------------------------------------------------------------------------------------
template <int RW>
__global__ __launch_bounds__(kRB) void recon_valu_kernel(const float* __restrict__ R, int M,
                                                         int N, const float* __restrict__ S,
                                                         int b, int chunk, int splits,
                                                         int row_groups, float* __restrict__ ws) {
  const int wave = (blockIdx.x * kRB + threadIdx.x) >> 6;
  const int lane = threadIdx.x & 63;
  if (wave >= row_groups * splits) return;
  const int g = wave / splits, sp = wave - g * splits;
  const int row0 = g * RW;
  const int k0 = sp * chunk, k1 = min(N, k0 + chunk);
  const float* s = S + (int64_t)b * N;
  float acc[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) acc[r] = 0.0f;
  // whole float4s of the chunk; two steps of loads in flight
  const int kv = k0 + ((k1 - k0) & ~3);
  int k = k0 + 4 * lane;
  for (; k + 4 * 64 < kv; k += 2 * 4 * 64) {
    const float4 s0 = ld4(s + k), s1 = ld4(s + k + 256);
    float4 r0[RW], r1[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
      const int row = min(row0 + r, M - 1);
      r0[r] = ldnt4(R + (int64_t)row * N + k);
      r1[r] = ldnt4(R + (int64_t)row * N + k + 256);
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) acc[r] += dot4(r0[r], s0) + dot4(r1[r], s1);
  }
  for (; k < kv; k += 4 * 64) {
    const float4 sv = ld4(s + k);
#pragma unroll
    for (int r = 0; r < RW; ++r)
      acc[r] += dot4(ldnt4(R + (int64_t)min(row0 + r, M - 1) * N + k), sv);
  }
  if (kv + lane < k1) {  // the last 1-3 columns
#pragma unroll
    for (int r = 0; r < RW; ++r)
      acc[r] = fmaf(R[(int64_t)min(row0 + r, M - 1) * N + kv + lane], s[kv + lane], acc[r]);
  }
#pragma unroll
  for (int r = 0; r < RW; ++r) {
    float v = acc[r];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    acc[r] = v;
  }
  if (lane == 0) {
#pragma unroll
    for (int r = 0; r < RW; ++r)
      if (row0 + r < M) ws[((int64_t)sp * 1 + 0) * M + row0 + r] = acc[r];
  }
}

// ---------------------------------------------------------------------------------------
// Small batch (2 <= B <= 8), slopes staged in LDS: workgroup = one split (columns
// [k0, k1)) x 4 row groups of 8 rows, one per wave.  The split's columns go by in slices of
// 256: the workgroup stages the slice of every realisation's slopes in LDS (double-buffered,
// the next slice's global loads in flight while this one is used; one barrier a slice), and
// each lane streams the float4 at column k + 4 lane of its wave's 8 rows (1 KB contiguous per
// row and instruction) and forms 8 x B dot products, reduced across the wave at the end.
// Holding the slopes in LDS instead of registers halves the vector-memory instructions and
// frees the registers for a second set of R loads (PF: the next slice's rows are in flight
// while this slice is summed).
// ---------------------------------------------------------------------------------------
template <int BB, bool PF>
__global__ __launch_bounds__(kRB) void recon_batch_lds_kernel(const float* __restrict__ R,
                                                              int M, int N,
                                                              const float* __restrict__ S,
                                                              int B, int chunk, int quads,
                                                              float* __restrict__ ws) {
  constexpr int RW = kBatchRW;
  __shared__ float4 slab[2][BB][64];
  const int wg = blockIdx.x;
  const int sp = wg / quads, q = wg - sp * quads;  // consecutive workgroups: one split
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int row0 = (q * 4 + wave) * RW;
  const int k0 = sp * chunk, k1 = min(N, k0 + chunk);
  const int ns = (k1 - k0 + 255) / 256;
  const float* rrow[RW];
#pragma unroll
  for (int r = 0; r < RW; ++r) rrow[r] = R + (int64_t)min(row0 + r, M - 1) * N;
  const bool whole4 = (N & 3) == 0;  // (uniform) a float4 of a row is whole or past its end
  // slope slice loads: thread t stages float4 j = t & 63 of realisations t / 64 and 4 + t / 64
  auto load_s = [&](int s, auto whole, float4 (&v)[2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int b = (threadIdx.x >> 6) + 4 * h, k = k0 + 256 * s + 4 * (threadIdx.x & 63);
      if (b >= B || b >= BB)
        v[h] = make_float4(0.f, 0.f, 0.f, 0.f);
      else if (whole)
        v[h] = ld4(S + (int64_t)b * N + k);
      else if (whole4)
        v[h] = k < k1 ? ld4(S + (int64_t)b * N + k) : make_float4(0.f, 0.f, 0.f, 0.f);
      else
        v[h] = ld4_below<false>(S + (int64_t)b * N, k, k1);
    }
  };
  auto store_s = [&](int buf, const float4 (&v)[2]) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int b = (threadIdx.x >> 6) + 4 * h;
      if (b < BB) slab[buf][b][threadIdx.x & 63] = v[h];
    }
  };
  auto load_r = [&](int s, auto whole, float4 (&v)[RW]) {
    const int k = k0 + 256 * s + 4 * lane;
    if (whole) {
#pragma unroll
      for (int r = 0; r < RW; ++r) v[r] = ldnt4(rrow[r] + k);
    } else if (whole4) {
#pragma unroll
      for (int r = 0; r < RW; ++r)
        v[r] = k < k1 ? ldnt4(rrow[r] + k) : make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
#pragma unroll
      for (int r = 0; r < RW; ++r) v[r] = ld4_below<true>(rrow[r], k, k1);
    }
  };
  float acc[RW][BB];
#pragma unroll
  for (int r = 0; r < RW; ++r)
#pragma unroll
    for (int b = 0; b < BB; ++b) acc[r][b] = 0.0f;
  float4 sv[2], rv[RW], rn[RW];
  load_s(0, k0 + 256 <= k1, sv);
  if constexpr (PF) load_r(0, k0 + 256 <= k1, rv);
  store_s(0, sv);
  __syncthreads();
  // step s; the next slice's loads (a slice that may be short has a branch for each load)
  auto step = [&](int s, auto next, auto whole) {
    const int cur = s & 1;
    if (next) load_s(s + 1, whole, sv);
    if constexpr (PF) {
      if (next) load_r(s + 1, whole, rn);
    } else {
      load_r(s, std::false_type{}, rv);
    }
#pragma unroll
    for (int b = 0; b < BB; ++b) {
      const float4 x = slab[cur][b][lane];
#pragma unroll
      for (int r = 0; r < RW; ++r) acc[r][b] += dot4(rv[r], x);
    }
    if (next) {
      store_s(cur ^ 1, sv);
      __syncthreads();
      if constexpr (PF) {
#pragma unroll
        for (int r = 0; r < RW; ++r) rv[r] = rn[r];
      }
    }
  };
  int s = 0;
  for (; k0 + 256 * (s + 2) <= k1; ++s) step(s, std::true_type{}, std::true_type{});
  for (; s < ns; ++s) step(s, s + 1 < ns, std::false_type{});
#pragma unroll
  for (int r = 0; r < RW; ++r)
#pragma unroll
    for (int b = 0; b < BB; ++b) {
      float v = acc[r][b];
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
      acc[r][b] = v;
    }
  if (lane == 0) {
#pragma unroll
    for (int r = 0; r < RW; ++r)
#pragma unroll
      for (int b = 0; b < BB; ++b)
        if (row0 + r < M && b < B) ws[((int64_t)sp * B + b) * M + row0 + r] = acc[r][b];
  }
}

// ---------------------------------------------------------------------------------------
// MFMA GEMM, TB tiles of 16 realisations a pass.  v_mfma_f32_16x16x4f32 operand layout
// (wave64): lane l supplies A[l%16][l/16] and B[l/16][l%16]; the four accumulator registers of
// lane l hold D[4*(l/16)+i][l%16].  The K index of one MFMA is only a label shared by A and B,
// so lane (i, kq) feeds the four consecutive columns of one float4 to four MFMAs.
//
// Bound by the stream of R: each wave loads its 16 rows 512 bytes a row at a time (two rows an
// instruction) and turns them into operands through its own LDS tile, the next tile's loads in
// flight; the workgroup's four waves share the slices of the slopes, double-buffered, one
// barrier a tile.  Loading the operands straight from memory (32 bytes a lane of 16 rows)
// reached 3.9 TB/s of R: B = 16 at 5,400 x 55,608 took 321 us, this takes 224 us (5.4 TB/s),
// and up to 32 realisations read R once.  FP32 matrix instructions of 32 cycles each: 61 us of
// the device's matrix time per 16 realisations of that size.
//
// A matrix instruction adds its four products to the accumulator one after the other, so a chain
// of them rounds as often as there are products.  Eight chains a tile of realisations, ended
// after a few tiles and added to a sum, keep the error below that of one GEMV a realisation
// (rms, in 2^-24 of the root of the sum of squares; N(0, 1) operands of 5,400 rows):
//   columns   GEMV   eight chains a split   ended kFolds times     B    us before and after
//   55,607    5.28   8.5                    3.3                    16   235 -> 235
//   55,607    5.28   12.6                   4.5                    24   303 -> 318
//   5,001     2.01   3.0                    1.50 (SHORT)           16   31.4 -> 30.7
//   5,001     2.01   3.9                    1.92                   20   38.4 -> 42.7
//   1,001     1.49   2.6                    1.35 (SHORT)           20   17.5 -> 18.5
// Splits of few tiles (SHORT) end their chains twice a tile; the sum is in 64 bits there, once a
// tile or once in two (FP64 additions take 16 cycles: every tile of 32 realisations 1.2 x).
// ---------------------------------------------------------------------------------------
constexpr int kTileK = 128;           // columns of one tile
constexpr int kTileP = kTileK + 4;    // LDS pitch: 16 rows on different banks
constexpr int kTileB = 32;            // realisations of one pass at most
constexpr int kFolds = 8;             // times a split's chains end

template <int TB, bool SHORT>
__device__ __forceinline__ void recon_mfma(const float* __restrict__ R, int M, int N,
                                           const float* __restrict__ S, int B, int chunk,
                                           int row_blocks, int per_fold, float* __restrict__ ws) {
  __shared__ __align__(16) float rt[4][16][kTileP];
  __shared__ __align__(16) float sl[2][TB * 16][kTileP];
  const int sp = blockIdx.x / row_blocks, g = blockIdx.x - sp * row_blocks;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int row0 = (g * 4 + wave) * 16;
  const int k0 = sp * chunk, k1 = min(N, k0 + chunk);
  const int nt = (k1 - k0 + kTileK - 1) / kTileK;
  const int i16 = lane & 15, kq = lane >> 4;
  const int lr = lane >> 5, lc = 4 * (lane & 31);  // this lane's row of a pair, its columns
  float4 rv[8], sv[2 * TB];
  auto load_r = [&](int t) {
    const int k = k0 + t * kTileK + lc;
    if (k0 + (t + 1) * kTileK <= k1) {  // uniform; the last tile of a row may be short
#pragma unroll
      for (int i = 0; i < 8; ++i) rv[i] = ldnt4(R + (int64_t)min(row0 + 2 * i + lr, M - 1) * N + k);
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        rv[i] = ld4_below<true>(R + (int64_t)min(row0 + 2 * i + lr, M - 1) * N, k, k1);
    }
  };
  auto load_s = [&](int t) {  // thread: slope rows threadIdx.x / 32 + 8 i, the same columns
    const int k = k0 + t * kTileK + 4 * (threadIdx.x & 31);
#pragma unroll
    for (int i = 0; i < 2 * TB; ++i) {
      const int b = (threadIdx.x >> 5) + 8 * i;
      sv[i] = b < B ? ld4_below<false>(S + (int64_t)b * N, k, k1)
                    : make_float4(0.f, 0.f, 0.f, 0.f);
    }
  };
  auto store_s = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 2 * TB; ++i)
      *reinterpret_cast<float4*>(&sl[buf][(threadIdx.x >> 5) + 8 * i][4 * (threadIdx.x & 31)]) =
          sv[i];
  };
  const v4f zero = {0.0f, 0.0f, 0.0f, 0.0f};
  v4f acc[TB][8];  // chains of products
  typedef typename std::conditional<SHORT, double, float>::type sum_t;
  sum_t sum[TB][4];
  v4f even[TB];  // SHORT: the last tile of even number, where two tiles go to the sum at once
  const bool each = TB == 1 || nt <= 5;  // (uniform) every tile does
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
#pragma unroll
    for (int i = 0; i < 4; ++i) sum[tb][i] = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[tb][i] = zero;
  }
  // the chains' ends, added in pairs; the chains start again
  auto ends = [&](int tb) {
    v4f* c = acc[tb];
    const v4f e = ((c[0] + c[4]) + (c[1] + c[5])) + ((c[2] + c[6]) + (c[3] + c[7]));
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = zero;
    return e;
  };
  auto add = [&](int tb, v4f e) {
#pragma unroll
    for (int i = 0; i < 4; ++i) sum[tb][i] += (sum_t)e[i];
  };
  load_s(0);
  load_r(0);
  store_s(0);
  __syncthreads();
  for (int t0 = 0; t0 < nt; t0 += per_fold) {
    const int t1 = min(t0 + per_fold, nt);
    for (int t = t0; t < t1; ++t) {
      // the wave's tile of R (its last readers are this wave's own, in order)
#pragma unroll
      for (int i = 0; i < 8; ++i)
        *reinterpret_cast<float4*>(&rt[wave][2 * i + lr][lc]) = rv[i];
      wave_sync();
      if (t + 1 < nt) {
        load_r(t + 1);
        load_s(t + 1);
      }
      v4f half[TB];
#pragma unroll
      for (int q = 0; q < kTileK / 16; ++q) {
        const float4 a = *reinterpret_cast<const float4*>(&rt[wave][i16][16 * q + 4 * kq]);
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
          const float4 x =
              *reinterpret_cast<const float4*>(&sl[t & 1][tb * 16 + i16][16 * q + 4 * kq]);
          v4f* c = acc[tb] + 4 * (q & 1);
          c[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, x.x, c[0], 0, 0, 0);
          c[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, x.y, c[1], 0, 0, 0);
          c[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, x.z, c[2], 0, 0, 0);
          c[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, x.w, c[3], 0, 0, 0);
        }
        if (SHORT && q == kTileK / 32 - 1) {
#pragma unroll
          for (int tb = 0; tb < TB; ++tb) half[tb] = ends(tb);
          __builtin_amdgcn_sched_barrier(0);  // (both halves at once would spill)
        }
      }
      if constexpr (SHORT) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
          const v4f e = ends(tb);
          if (each) {
            add(tb, half[tb]);
            add(tb, e);
          } else if (t & 1) {
            add(tb, even[tb] + (half[tb] + e));
          } else {
            even[tb] = half[tb] + e;
          }
        }
      }
      wave_sync();
      if (t + 1 < nt) store_s((t + 1) & 1);
      __syncthreads();
    }
    if constexpr (!SHORT) {
#pragma unroll
      for (int tb = 0; tb < TB; ++tb) add(tb, ends(tb));
    }
  }
  if (SHORT && !each && (nt & 1)) {
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) add(tb, even[tb]);
  }
  // D[4*kq + i][i16]: row = row0 + 4 kq + i, realisation = 16 tb + i16
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
    const int b = 16 * tb + i16;
    if (b < B) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = row0 + 4 * kq + i;
        if (row < M) ws[((int64_t)sp * B + b) * M + row] = (float)sum[tb][i];
      }
    }
  }
}

template <int TB>
__global__ __launch_bounds__(kRB) void recon_mfma_kernel(const float* R, int M, int N,
                                                         const float* S, int B, int chunk,
                                                         int row_blocks, int per_fold, float* ws) {
  recon_mfma<TB, false>(R, M, N, S, B, chunk, row_blocks, per_fold, ws);
}

template <int TB>
__global__ __launch_bounds__(kRB) __attribute__((amdgpu_waves_per_eu(TB == 1 ? 3 : 2))) void
recon_mfma_short_kernel(const float* R, int M, int N, const float* S, int B, int chunk,
                        int row_blocks, float* ws) {
  recon_mfma<TB, true>(R, M, N, S, B, chunk, row_blocks, 1, ws);
}

// C[b][i] = alpha * sum_sp ws[sp][b][i] + beta * C[b][i]   (splits added in order)
__global__ __launch_bounds__(kRB) void recon_reduce_kernel(const float* __restrict__ ws, int M,
                                                           int B, int splits, float* C,
                                                           int64_t ldc, float alpha, float beta,
                                                           int b_first, int b_count) {
  const int64_t gid = (int64_t)blockIdx.x * kRB + threadIdx.x;
  if (gid >= (int64_t)M * b_count) return;
  const int bl = (int)(gid / M), i = (int)(gid - (int64_t)bl * M);
  // four chains of additions, each of every fourth split
  const float* w = ws + (int64_t)bl * M + i;
  const int64_t step = (int64_t)b_count * M;
  float c4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  int sp = 0;
  for (; sp + 4 <= splits; sp += 4)
#pragma unroll
    for (int k = 0; k < 4; ++k) c4[k] += w[(sp + k) * step];
#pragma unroll
  for (int k = 0; k < 3; ++k)
    if (sp + k < splits) c4[k] += w[(sp + k) * step];
  const float s = (c4[0] + c4[1]) + (c4[2] + c4[3]);
  float* c = C + (int64_t)(b_first + bl) * ldc + i;
  *c = beta == 0.0f ? alpha * s : fmaf(alpha, s, beta * *c);
}

// ---------------------------------------------------------------------------------------
// launch shape: every (row group, split) wave of a call runs in ONE round of the device's
// resident wave slots, so no wave of a second round streams its chunk after the others end
// ---------------------------------------------------------------------------------------
static std::mutex g_occ_mu;
static int g_slots[64][3];  // per device: resident waves of the MFMA, GEMV and small-batch
                            // kernels

static hipError_t resident_waves(int which, int* out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_occ_mu);
  if (g_slots[dev][which] == 0) {
    int cus = 0, blocks = 0;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    const void* k = which == 0   ? reinterpret_cast<const void*>(recon_mfma_kernel<1>)
                    : which == 1 ? reinterpret_cast<const void*>(recon_valu_kernel<2>)
                                 : reinterpret_cast<const void*>(
                                       recon_batch_lds_kernel<kBatchMax, kBatchPF>);
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, k, kRB, 0);
    if (e != hipSuccess) return e;
    g_slots[dev][which] = std::max(1, cus * std::max(1, blocks) * (kRB / 64));
  }
  *out = g_slots[dev][which];
  return hipSuccess;
}

// Splits of the N columns (chunks of a multiple of `align`) for `row_groups` waves per split:
// as many as one round of `slots` resident waves holds, at most N/256, and at most
// `max_splits` (the workspace a caller can offer).
static int choose_splits(int row_groups, int N, int align, int slots, int64_t max_splits,
                         int* chunk) {
  int64_t want = std::max<int64_t>(1, slots / row_groups);
  want = std::min<int64_t>(want, std::max(1, N / 256));
  want = std::max<int64_t>(1, std::min<int64_t>(want, max_splits));
  int c = (int)((N + want - 1) / want);
  c = (c + align - 1) / align * align;
  *chunk = c;
  return (N + c - 1) / c;  // <= want
}

enum ReconPath { kReconGemv, kReconBatch, kReconMfma };

struct ReconShape {
  ReconPath path;
  int units;   // wave row groups per split
  int align;   // columns a chunk is a multiple of
  int slots;   // resident waves
  int tile_b;  // realisations of a partial-sum tile that every call of the path can run with
};

static hipError_t recon_shape(ReconPath path, int M, int N, int B, bool aligned, ReconShape* sh) {
  sh->path = path;
  if (path == kReconBatch) {
    sh->units = ((M + kBatchRW - 1) / kBatchRW + 3) / 4 * 4;
    // (a split's last slice, if not whole, branches for each load: 8 realisations of 5,400 x
    // 8,001 took 47 us with 64 columns, 43 with 256; few columns need the even splits: rms at
    // 515 columns 1.45 with 256, 1.40 with 64, one GEMV a realisation 1.39)
    sh->align = aligned || N >= 1024 ? 256 : 64;
    sh->tile_b = std::min(B, kBatchMax);
    return resident_waves(2, &sh->slots);
  }
  if (path == kReconMfma) {
    sh->units = (M + 63) / 64 * 4;
    sh->align = kTileK;
    sh->tile_b = std::min(16, B);
    return resident_waves(0, &sh->slots);
  }
  sh->units = (M + 1) / 2;
  sh->align = aligned ? 256 : 64;
  sh->tile_b = 1;
  return resident_waves(1, &sh->slots);
}

static ReconPath recon_path(int B) {
  return B == 1 ? kReconGemv : (B <= kBatchMax ? kReconBatch : kReconMfma);
}

// Operands that were always taken however large M is: rows or vectors not 16-byte aligned run
// one GEMV per realisation where a workspace cannot hold a tile of them.
static bool recon_aligned(const float* R, int N, const float* S) {
  return N % 4 == 0 && (uintptr_t)R % 16 == 0 && (uintptr_t)S % 16 == 0;
}

// Floats of partial sums a call wants (its split count unconstrained by the workspace); `most`:
// no fewer than a call with a smaller B or the other alignment, so that a workspace grown by one
// call takes them all.
hipError_t recon_work_floats(const float* R, int M, int N, const float* S, int B, bool most,
                             int64_t* floats) {
  *floats = 0;
  const bool aligned = recon_aligned(R, N, S);
  for (int path = most ? kReconGemv : recon_path(B); path <= recon_path(B); ++path)
    for (int other = 0; other <= (most ? 1 : 0); ++other) {
      ReconShape sh;
      hipError_t e = recon_shape((ReconPath)path, M, N, B, aligned != (other != 0), &sh);
      if (e != hipSuccess) return e;
      int chunk;
      const int splits = choose_splits(sh.units, N, sh.align, sh.slots, INT32_MAX, &chunk);
      *floats = std::max(*floats, (int64_t)splits * sh.tile_b * M);
    }
  return hipSuccess;
}

static hipError_t recon_reduce(const float* ws, int M, int bc, int splits, float* C, int64_t ldc,
                               float alpha, float beta, int b0, hipStream_t st) {
  const int64_t n = (int64_t)M * bc;
  hipLaunchKernelGGL(recon_reduce_kernel, dim3((unsigned)((n + kRB - 1) / kRB)), dim3(kRB), 0, st,
                     ws, M, bc, splits, C, ldc, alpha, beta, b0, bc);
  return hipGetLastError();
}

// C = alpha R S^T + beta C with the split partial sums in ws; the split count (and the
// realisations of a matrix-core pass) shrink to what ws holds.
hipError_t recon_launch(const float* R, int M, int N, const float* S, int B, float* C,
                        int64_t ldc, float alpha, float beta, float* ws, int64_t ws_floats,
                        hipStream_t st) {
  ReconPath path = recon_path(B);
  if (path != kReconGemv && ws_floats < (int64_t)std::min(B, 16) * M) path = kReconGemv;
  const bool aligned = recon_aligned(R, N, S);
  ReconShape sh;
  hipError_t e = recon_shape(path, M, N, B, aligned, &sh);
  if (e != hipSuccess) return e;
  if (ws_floats < M) return hipErrorInvalidValue;
  int chunk;
  if (path == kReconBatch) {
    const int splits =
        choose_splits(sh.units, N, sh.align, sh.slots, ws_floats / ((int64_t)B * M), &chunk);
    const int quads = sh.units / 4, grid = quads * splits;
    if (B <= 2)
      hipLaunchKernelGGL((recon_batch_lds_kernel<2, kBatchPF>), dim3(grid), dim3(kRB), 0, st, R,
                         M, N, S, B, chunk, quads, ws);
    else if (B <= 4)
      hipLaunchKernelGGL((recon_batch_lds_kernel<4, kBatchPF>), dim3(grid), dim3(kRB), 0, st, R,
                         M, N, S, B, chunk, quads, ws);
    else
      hipLaunchKernelGGL((recon_batch_lds_kernel<kBatchMax, kBatchPF>), dim3(grid), dim3(kRB), 0,
                         st, R, M, N, S, B, chunk, quads, ws);
    e = hipGetLastError();
    return e == hipSuccess ? recon_reduce(ws, M, B, splits, C, ldc, alpha, beta, 0, st) : e;
  }
  if (path == kReconMfma) {
    // passes of up to 32 realisations, evenly wide, their partial sums in the floats that 16
    // want (half the splits then); 16 where ws holds no more
    const int most = ws_floats >= (int64_t)kTileB * M ? kTileB : 16;
    const int passes = (B + most - 1) / most;
    const int per = ((B + passes - 1) / passes + 15) / 16 * 16;
    for (int b0 = 0; b0 < B; b0 += per) {
      const int bc = std::min(per, B - b0);
      const int splits = choose_splits(sh.units, N, sh.align, bc > 16 ? sh.slots / 2 : sh.slots,
                                       ws_floats / ((int64_t)bc * M), &chunk);
      const int grid = sh.units / 4 * splits;
      // Chains ended kFolds times; with more than 16 realisations and rows of whole float4s
      // twice (rms 8.9 at 55,608 columns, 313 us for 32 realisations; once 12.6 and 308, kFolds
      // times 4.5 and 326), where nothing asks for a GEMV's exactness.  SHORT up to kFolds tiles:
      // from there on chains of one or more tiles are as exact as a GEMV's and take less (16
      // tiles, 5,400 x 8,001 and 20 realisations: rms 2.2 and 60.5 us, SHORT 1.6 and 63.7, a
      // GEMV 2.3).
      const bool exact = bc <= 16 || !aligned;
      const float* sb = S + (int64_t)b0 * N;
      const int tiles = chunk / kTileK;
      if (exact && tiles <= kFolds) {
        const auto k = bc <= 16 ? recon_mfma_short_kernel<1> : recon_mfma_short_kernel<2>;
        hipLaunchKernelGGL(k, dim3(grid), dim3(kRB), 0, st, R, M, N, sb, bc, chunk, sh.units / 4,
                           ws);
      } else {
        const auto k = bc <= 16 ? recon_mfma_kernel<1> : recon_mfma_kernel<2>;
        hipLaunchKernelGGL(k, dim3(grid), dim3(kRB), 0, st, R, M, N, sb, bc, chunk, sh.units / 4,
                           exact ? tiles / kFolds : (tiles + 1) / 2, ws);
      }
      e = hipGetLastError();
      if (e == hipSuccess) e = recon_reduce(ws, M, bc, splits, C, ldc, alpha, beta, b0, st);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  constexpr int RW = 2;
  const int splits = choose_splits(sh.units, N, sh.align, sh.slots, ws_floats / M, &chunk);
  for (int b = 0; b < B; ++b) {
    const int waves = sh.units * splits;
    hipLaunchKernelGGL((recon_valu_kernel<RW>), dim3((waves + 3) / 4), dim3(kRB), 0, st, R, M, N,
                       S, b, chunk, splits, sh.units, ws);
    e = hipGetLastError();
    if (e == hipSuccess) e = recon_reduce(ws, M, 1, splits, C, ldc, alpha, beta, b, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// ---------------------------------------------------------------------------------------
// recon_apply's workspace: one buffer per (device, stream), so calls on different streams
// never share partial sums.  A buffer is never freed while the process lives (a captured
// graph may still hold it): a larger problem allocates a larger buffer and keeps the old one.
// No buffer is allocated while the stream is capturing.
// ---------------------------------------------------------------------------------------
struct StreamWork {
  int dev;
  hipStream_t stream;
  float* ptr;
  int64_t floats;
};
static std::mutex g_ws_mu;
static std::vector<StreamWork> g_ws;       // current buffer of each (device, stream)
static std::vector<float*> g_ws_retired;   // outgrown buffers, kept for captured graphs

// The stream's buffer, grown for a call of this size and every smaller B where it holds fewer
// than `floats` (*have: what it holds).  While
// the stream is capturing it cannot grow: *capturing is set, *out and *have are the current
// buffer (or null and 0).
hipError_t recon_stream_work(hipStream_t st, const float* R, int M, int N, const float* S, int B,
                             int64_t floats, float** out, int64_t* have, bool* capturing) {
  *capturing = false;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> lk(g_ws_mu);
  StreamWork* w = nullptr;
  for (auto& x : g_ws)
    if (x.dev == dev && x.stream == st) w = &x;
  *out = w ? w->ptr : nullptr;
  *have = w ? w->floats : 0;
  if (w && w->floats >= floats) return hipSuccess;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  e = hipStreamIsCapturing(st, &cs);
  if (e != hipSuccess) return e;
  if (cs != hipStreamCaptureStatusNone) {
    *capturing = true;
    return hipErrorStreamCaptureUnsupported;
  }
  e = recon_work_floats(R, M, N, S, B, true, &floats);
  if (e != hipSuccess) return e;
  float* p = nullptr;
  e = hipMalloc((void**)&p, sizeof(float) * (size_t)floats);
  if (e != hipSuccess) return e;
  if (w) {
    g_ws_retired.push_back(w->ptr);
    w->ptr = p;
    w->floats = floats;
  } else {
    g_ws.push_back(StreamWork{dev, st, p, floats});
  }
  *out = p;
  *have = floats;
  return hipSuccess;
}

// ---------------------------------------------------------------------------------------
// Fixed workspace of recon_apply_noalloc: a file-scope device array (each GPU the library runs
// on holds its own copy until the process ends).  In host code `scratch` names a host-side
// stand-in, not device memory: kernels get its device address, fetched once per device with
// hipGetSymbolAddress on the first call there.  Every call on one GPU shares it.
// ---------------------------------------------------------------------------------------
constexpr int64_t kStaticWorkFloats = int64_t(1) << 22;  // 16 MiB of partial sums
static __device__ __align__(256) float scratch[kStaticWorkFloats];
static std::mutex g_static_mu;
static float* g_static_ptr[64];

int64_t recon_static_work_floats() { return kStaticWorkFloats; }

// Floats of partial sums a call cannot do without (M rows x the realisations of one tile; a
// single realisation's for operands that are not 16-byte aligned).
int64_t recon_min_work_floats(const float* R, int M, int N, const float* S, int B) {
  return (int64_t)(recon_aligned(R, N, S) ? std::min(B, 16) : 1) * M;
}

hipError_t recon_static_work(float** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_static_mu);
  if (!g_static_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_static_ptr[dev] = static_cast<float*>(p);
  }
  *out = g_static_ptr[dev];
  return hipSuccess;
}

}  // namespace wfs
