// Phase screens on the GPU (Sec. 2.1 of the paper: the atmosphere is a set of phase screens
// made by filtering random noise in the Fourier domain with a Kolmogorov or von Karman phase
// spectrum, parameterised by r0 and L0).
//
//   phi = Re( sum_k W_k sqrt(PSD(f_k)) df exp(+2 pi i k.x / n) ),  W = a + i b, a, b ~ N(0, 1),
//   PSD(f) = 0.023 r0^(-5/3) (f^2 + L0^-2)^(-11/6)  (L0 = infinity: Kolmogorov), f = 0 zeroed,
//
// on an n x n periodic grid of pitch dx (df = 1 / (n dx)).  The noise is Philox4x32-10 keyed by
// the seed, one block per Fourier sample (counter: sample index, stream id), Box-Muller on its
// first two words.  Only the real part is wanted, so the transform is that of the spectrum's
// Hermitian part H[k] = (S[k] + conj S[-k]) / 2, S = W sqrt(PSD) df, whose transform is real:
// the row pass forms the n / 2 + 1 rows k_y = 0 .. n / 2 (noise of k and -k, filter, an n-point
// FFT in LDS, written in C-column tiles), the column pass two real columns per complex FFT
// (Z[k_y] = G[k_y][x] + i G[k_y][x + 1], G[-k_y] = conj G[k_y]).  That is half the FFT work and
// half the tile traffic of transforming S whole (per screen, n = 1024: 20.8 -> 15.0 us, bound by
// the two launches' latency chains; 2048: 52.8 -> 31.6; 4096: 270 -> 107).  The unnormalised
// inverse DFT is the forward one of the conjugate.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "../../include/wfs.h"
#include "lds_fft.h"
#include "wfs_common.h"

namespace wfs {
int set_error(int code, const char* msg);

constexpr int kScrBlock = 512;
constexpr int kScrMaxN = 4096;

struct ScreenParams {
  float2* T;            // [n / C][n / 2 + 1][C] row transforms
  float* out;           // [n][n]
  float c_psd;          // 0.023 r0^(-5/3)
  float inv_l02;        // L0^-2 (0: Kolmogorov)
  float inv_ndx;        // df = 1 / (n dx), cycles per metre per frequency index
  uint32_t seed_lo, seed_hi, sid_lo, sid_hi;
};

// Real columns per column-pass workgroup: enough workgroups to cover the 256 CUs where n
// allows (n / C >= 256), C / 2 padded columns within the LDS.
__host__ __device__ constexpr int scr_cols(int n) {
  return n >= 4096 ? 4 : (n / 256 > 8 ? 8 : (n / 256 < 2 ? 2 : n / 256));
}
__host__ __device__ constexpr int scr_col_threads(int n) { return n >= 2048 ? 512 : 256; }

// cos and sin of 2 pi j / 4096 (the largest transform's roots), in double at compile time: the
// Taylor series on the first eighth of the circle, the rest by symmetry.
struct Roots {
  float c[kScrMaxN], s[kScrMaxN];
  constexpr Roots() : c(), s() {
    constexpr int q = kScrMaxN / 4;
    for (int j = 0; j <= q / 2; ++j) {
      const double a = 6.283185307179586476925286766559 * j / kScrMaxN, x2 = a * a;
      double sn = a, cs = 1.0, ts = a, tc = 1.0;
      for (int k = 1; k <= 9; ++k) {
        tc *= -x2 / ((2.0 * k - 1.0) * (2.0 * k));
        ts *= -x2 / ((2.0 * k) * (2.0 * k + 1.0));
        cs += tc;
        sn += ts;
      }
      const float fc = (float)cs, fs = (float)sn;
      put(j, fc, fs);
      put(q - j, fs, fc);
    }
  }

 private:
  constexpr void put(int j, float cs, float sn) {  // j in the first quarter: and the others
    constexpr int q = kScrMaxN / 4;
    c[j] = cs;
    s[j] = sn;
    if (j < q) {
      c[q + j] = -sn;
      s[q + j] = cs;
      c[2 * q + j] = -cs;
      s[2 * q + j] = -sn;
      c[3 * q + j] = sn;
      s[3 * q + j] = -cs;
    }
  }
};

// The n - 1 twiddles of lds_fft for n = 2^LOG2N (fft_tw_angle), in the library's data: no
// workgroup forms them.
template <int LOG2N>
struct ScreenTwiddles {
  alignas(16) float v[2 << LOG2N];
  constexpr explicit ScreenTwiddles(const Roots& r) : v() {
    constexpr int n = 1 << LOG2N, step = kScrMaxN / n;
    int lns = 0;
    while (lns < LOG2N) {
      const int lr = fft_stage_lr(LOG2N, lns), ns = 1 << lns;
      for (int m = 1; m < 1 << lr; ++m)
        for (int k = 0; k < ns; ++k) {
          const int at = ns - 1 + (m - 1) * ns + k;
          const int j = (((m * k) << (LOG2N - lns - lr)) & (n - 1)) * step;
          v[2 * at] = r.c[j];
          v[2 * at + 1] = -r.s[j];
        }
      lns += lr;
    }
  }
};

constexpr Roots kRoots{};
template <int LOG2N>
__device__ const ScreenTwiddles<LOG2N> kScreenTw{kRoots};

// The workgroup's copy of the twiddles in LDS: loaded before the work that precedes the
// transform, stored after it, so that no transform stage waits for memory.
template <int LOG2N, int THREADS>
struct TwiddleCopy {
  static constexpr int kN4 = (1 << LOG2N) / 2, kPer = (kN4 + THREADS - 1) / THREADS;
  float4 t[kPer];
  __device__ __forceinline__ void load() {
    const float4* src = reinterpret_cast<const float4*>(kScreenTw<LOG2N>.v);
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int k = threadIdx.x + i * THREADS;
      t[i] = src[k < kN4 ? k : 0];
    }
  }
  __device__ __forceinline__ void store(float2* tws) const {
    float4* d = reinterpret_cast<float4*>(tws);
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int k = threadIdx.x + i * THREADS;
      if (k < kN4) d[k] = t[i];
    }
  }
};

// W = a + i b of Fourier sample (ky, kx)
__device__ __forceinline__ float2 screen_normal(const ScreenParams& p, uint32_t idx) {
  const uint4 w = philox4x32_10(make_uint4(idx, 0u, p.sid_lo, p.sid_hi), p.seed_lo, p.seed_hi);
  const float r = sqrtf(-1.3862943611198906f * __builtin_amdgcn_logf(u24(w.x)));
  float sn, cs;
  sincos_rev(u24(w.y), &sn, &cs);
  return make_float2(r * cs, r * sn);
}

// Row pass: workgroup per row ky = 0 .. n / 2 of the Hermitian part.
template <int LOG2N>
__global__ __launch_bounds__(kScrBlock) void screen_rows_kernel(ScreenParams p) {
  extern __shared__ __align__(16) float2 tws[];  // the twiddles, then the row
  constexpr int n = 1 << LOG2N, C = scr_cols(n), R = n / 2 + 1;
  const int ky = blockIdx.x, tid = threadIdx.x;
  float2* sh = tws + n;
  TwiddleCopy<LOG2N, kScrBlock> tw;
  tw.load();
  const float fy = (float)ky * p.inv_ndx;
  const uint32_t row = (uint32_t)ky << LOG2N, nrow = (uint32_t)((n - ky) & (n - 1)) << LOG2N;
  const float half_c = 0.5f * sqrtf(p.c_psd);
  for (int kx = tid; kx < n; kx += kScrBlock) {
    const int ix = kx < n / 2 ? kx : kx - n;  // frequency index in [-n/2, n/2)
    const float fx = (float)ix * p.inv_ndx;
    const float f2 = fx * fx + fy * fy;
    float amp = 0.0f;
    if (kx | ky) {
      // sqrt(PSD) df / 2 = sqrt(c) (f^2 + L0^-2)^(-11/12) df / 2
      amp = half_c * exp2f(-11.0f / 12.0f * log2f(f2 + p.inv_l02)) * p.inv_ndx;
    }
    const float2 a = screen_normal(p, row + (uint32_t)kx);
    const float2 b = screen_normal(p, nrow + (uint32_t)((n - kx) & (n - 1)));
    // conj H: the forward transform of conj(H) is conj of the inverse of H
    sh[fft_pad(kx)] = make_float2((a.x + b.x) * amp, (b.y - a.y) * amp);
  }
  tw.store(tws);
  __syncthreads();
  lds_fft<LOG2N, n, kScrBlock>(sh, 1, fft_span(n), tws);
  float2* o = p.T + (int64_t)ky * C;
  for (int x = tid; x < n; x += kScrBlock)
    o[(int64_t)(x / C) * R * C + (x & (C - 1))] = sh[fft_pad(x)];
}

// Column pass: C adjacent real columns per workgroup, two per complex transform.
template <int LOG2N>
__global__ __launch_bounds__(scr_col_threads(1 << LOG2N)) void screen_cols_kernel(ScreenParams p) {
  extern __shared__ __align__(16) float2 tws[];  // the twiddles, then the columns
  constexpr int n = 1 << LOG2N, C = scr_cols(n), P = C / 2, R = n / 2 + 1;
  constexpr int T = scr_col_threads(n), ld = fft_pitch(n, P);
  const int tid = threadIdx.x;
  float2* sh = tws + n;
  TwiddleCopy<LOG2N, T> tw;
  tw.load();
  const int g = xcd_logical_block(blockIdx.x, n / C);
  const float4* src = reinterpret_cast<const float4*>(p.T + (int64_t)g * R * C);  // [R][P]
  for (int i = tid; i < R * P; i += T) {
    const int c = i & (P - 1), y = i / P;
    const float4 v = src[i];  // G[y] of columns 2 c and 2 c + 1
    sh[c * ld + fft_pad(y)] = make_float2(v.x - v.w, v.y + v.z);
    if (y > 0 && y < n / 2) sh[c * ld + fft_pad(n - y)] = make_float2(v.x + v.w, v.z - v.y);
  }
  tw.store(tws);
  __syncthreads();
  lds_fft<LOG2N, P * n, T>(sh, P, ld, tws);
  const float* z = reinterpret_cast<const float*>(sh);
  float* out = p.out + g * C;
  for (int i = tid; i < C * n; i += T) {
    const int c = i & (C - 1), y = i / C;
    out[(int64_t)y * n + c] = z[2 * ((c >> 1) * ld + fft_pad(y)) + (c & 1)];
  }
}

}  // namespace wfs

using namespace wfs;

static int scr_fail(int code, const char* msg) { return set_error(code, msg); }

// Calls f(std::integral_constant<int, log2 n>) for a screen size 16 <= n <= 4096.
template <class F>
static void scr_dispatch(int log2n, F&& f) {
  switch (log2n) {
    case 4: f(std::integral_constant<int, 4>{}); break;
    case 5: f(std::integral_constant<int, 5>{}); break;
    case 6: f(std::integral_constant<int, 6>{}); break;
    case 7: f(std::integral_constant<int, 7>{}); break;
    case 8: f(std::integral_constant<int, 8>{}); break;
    case 9: f(std::integral_constant<int, 9>{}); break;
    case 10: f(std::integral_constant<int, 10>{}); break;
    case 11: f(std::integral_constant<int, 11>{}); break;
    default: f(std::integral_constant<int, 12>{}); break;
  }
}

// Launch with LDS bytes of dynamic LDS.  The largest sizes hold more than the default 64 KB,
// which the current device's kernel is told before each launch: the limit belongs to one device,
// and a process may use several.
template <int LDS>
static hipError_t scr_launch(void (*kernel)(ScreenParams), int blocks, int threads,
                             const ScreenParams& p, hipStream_t st) {
  if constexpr (LDS > 65536) {
    const hipError_t e = hipFuncSetAttribute((const void*)kernel,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    if (e != hipSuccess) return e;
  }
  kernel<<<blocks, threads, LDS, st>>>(p);
  return hipGetLastError();
}

extern "C" {

int screen_generate(int32_t n, double pitch_m, double r0_m, double L0_m, uint64_t seed,
                    uint64_t stream_id, float* screen, float* work, int64_t work_floats,
                    void* stream) {
  if (!screen || !work) return scr_fail(WFS_EINVAL, "screen_generate: null screen or work");
  if (n < 16 || n > kScrMaxN || (n & (n - 1)))
    return scr_fail(WFS_EINVAL, "screen_generate: n must be a power of two in [16, 4096]");
  if (!(pitch_m > 0) || !std::isfinite(pitch_m) || !(r0_m > 0) || !std::isfinite(r0_m) ||
      !(L0_m > 0))
    return scr_fail(WFS_EINVAL, "screen_generate: pitch, r0 and L0 must be > 0");
  if (work_floats < 2 * (int64_t)n * n)
    return scr_fail(WFS_EINVAL, "screen_generate: work must hold 2 n^2 floats");
  int log2n = 0;
  while ((1 << log2n) < n) ++log2n;
  hipStream_t st = (hipStream_t)stream;
  ScreenParams p{};
  // 16-byte aligned inside the work buffer (n^2 + 2 n floats of its 2 n^2 are used)
  p.T = reinterpret_cast<float2*>((reinterpret_cast<uintptr_t>(work) + 15) & ~(uintptr_t)15);
  p.out = screen;
  p.c_psd = (float)(0.023 * std::pow(r0_m, -5.0 / 3.0));
  p.inv_l02 = std::isfinite(L0_m) ? (float)(1.0 / (L0_m * L0_m)) : 0.0f;
  p.inv_ndx = (float)(1.0 / (n * pitch_m));
  p.seed_lo = (uint32_t)seed;
  p.seed_hi = (uint32_t)(seed >> 32);
  p.sid_lo = (uint32_t)stream_id;
  p.sid_hi = (uint32_t)(stream_id >> 32);
  hipError_t e = hipSuccess;
  scr_dispatch(log2n, [&](auto L) {
    constexpr int LG = decltype(L)::value, N = 1 << LG;
    e = scr_launch<(N + fft_span(N)) * (int)sizeof(float2)>(screen_rows_kernel<LG>, N / 2 + 1,
                                                            kScrBlock, p, st);
  });
  if (e != hipSuccess) return scr_fail(WFS_EDEVICE, hipGetErrorString(e));
  scr_dispatch(log2n, [&](auto L) {
    constexpr int LG = decltype(L)::value, N = 1 << LG, C = scr_cols(N);
    e = scr_launch<(N + (C / 2) * fft_pitch(N, C / 2)) * (int)sizeof(float2)>(
        screen_cols_kernel<LG>, N / C, scr_col_threads(N), p, st);
  });
  if (e != hipSuccess) return scr_fail(WFS_EDEVICE, hipGetErrorString(e));
  return WFS_OK;
}

}  // extern "C"
