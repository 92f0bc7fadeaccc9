// Point-spread functions and Strehl ratios of the residual wavefront (Sec. 2.8 of the paper:
// PSFs at user wavelengths and pixel scales, on the GPU; Strehl ratio from the PSF or, by the
// Marechal approximation, from the history of the residual wavefront).
//
// Per frame, star and wavelength: residual phase on the full pupil grid (the layers and DM
// grids projected along the star's direction at infinity, bilinear, as for the sensors),
// field A exp(i kappa phi) zero-padded to N x N, its 2-D DFT, and |F|^2 / (N^2 sum A^2) added to
// a long-exposure image (unit sum per frame, zero frequency at pixel (N/2, N/2)).  Three kernels:
// the phase of every pupil pixel and star (once for all wavelengths), the y pass (a few pupil
// columns per workgroup: field and N-point FFTs in LDS; only the n_pup non-zero columns exist)
// and the x pass (a few adjacent y frequencies per workgroup, FFTs in LDS, intensity added to
// whole image rows).  Both FFTs are the Stockham radix-16 (+ one radix-2, 4 or 8 stage)
// transforms of lds_fft.h, compiled per log2 N, on bank-conflict-free padded LDS; their twiddle
// table is computed in double precision on the host (staged in LDS by the x pass).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/wfs.h"
#include "lds_fft.h"
#include "wfs_common.h"

namespace wfs {
int set_error(int code, const char* msg);

constexpr int kPsfBlock = 256;
constexpr int kPsfPoints = 4096;     // largest transform (and one row-pass workgroup's LDS)
constexpr int kPsfColPoints = 16384; // LDS points of a column-pass workgroup (C columns x N)
constexpr int kPsfColLds = 160 * 1024;  // its LDS bytes at most: C pitch + N - 1 float2
constexpr int kPsfRowLds = 96 * 1024;   // LDS bytes of a row-pass workgroup at most
constexpr int kPsfMinLog2 = 4, kPsfMaxLog2 = 12;
constexpr int kPsfMaxLambda = 16;
constexpr int kPsfMaxStars = 256;

// u = ax*i + bx0 + step*dbx (column i), v = ay*j + by0 + step*dby (row j) in layer pixels.
struct PsfAff {
  double ax, bx0, dbx, ay, by0, dby;
};

struct PsfParams {
  const float* layers;
  const DevLayer* lay;
  const PsfAff* aff;     // [n_stars][n_layers]
  const uint8_t* mask;   // [n_pup][n_pup] pupil amplitude (0 / 1), symmetric in x and y
  float* phi;            // [n_stars][n_pup x][n_pup y] pupil phase at the reference wavelength
  const float2* tw;      // the N - 1 twiddles of lds_fft, stage after stage
  float2* T;             // [n_stars][N / C][n_pup x][C] transforms along y
  double* part;          // [n_stars][n_part][2]: sums of A phi and A phi^2 of the phase's blocks
  float* psf;            // this wavelength's [n_stars][N][N]
  int64_t step;
  int32_t n_layers, n_stars, n_pup, N, log2N, cols;
  float kappa, scale;
  // the variance of the phase, by the extra workgroup a star of the y pass where write_var
  int32_t n_part, n_lambda, write_var;
  double* phase_var;  // [n_lambda][n_stars]
  double inv_lit;
  float kappa2[kPsfMaxLambda];
};

// Phase: workgroup (strip of 64 pupil columns, 4 R pupil rows, star), wave = R rows of the
// strip.  The workgroup's column and row taps (FP64) are formed once, in LDS; where the rows'
// taps are neighbouring layer rows (a layer as fine as the pupil), or few (a coarse one), each
// layer row is read and interpolated once.  The phase is kept for every wavelength, column
// after column for the y pass.
//
// Few waves (less than two a SIMD) wait for memory layer after layer: two rows a wave then,
// and the rows of D = 5 layers on their way at once (one star of 150 pixels, 13 layers: 16.5 us
// with eight rows a wave, 11.5 so).  Many waves hide it and read less with eight rows (nine
// stars of 800 pixels and 13 layers: 61 us, with four rows 71 us).
constexpr int kPhaseWaves = kPsfBlock / 64;
constexpr int phase_rows(bool few) { return few ? 2 : 8; }
// column taps, row taps of a layer
__host__ __device__ constexpr int phase_taps(int R) { return 64 + R * kPhaseWaves; }
// workgroups of a star
static int phase_tiles(int n_pup, bool few) {
  const int rows = phase_rows(few) * kPhaseWaves;
  return ((n_pup + 63) / 64) * ((n_pup + rows - 1) / rows);
}
// Few waves: eight rows a wave leave less than two waves a SIMD.
static bool phase_few(int n_pup, int n_stars, int cus) {
  return (int64_t)phase_tiles(n_pup, false) * n_stars * kPhaseWaves < 8 * (int64_t)cus;
}

// The layer rows of a wave's pupil rows: neighbours from row[0] on (tap k on k and k + 1), or up
// to kFew different ones (tap k on those at bits 4 k and 4 k + 2 of sel), or more.
constexpr int kFew = 4, kRowsMore = 0, kRowsNext = 1, kRowsFew = 2;
struct PhaseRows {
  int32_t kind, sel, row[kFew];
};

// LDS bytes of a workgroup: the taps, and the rows of each layer and wave.
static size_t psf_phase_lds(int n_layers, bool few) {
  return n_layers * (phase_taps(phase_rows(few)) * sizeof(Tap) + kPhaseWaves * sizeof(PhaseRows));
}

template <int R, int D>
__global__ __launch_bounds__(kPsfBlock) __attribute__((amdgpu_waves_per_eu(8))) void
psf_phase_kernel(PsfParams p) {
  extern __shared__ __align__(16) char smem[];
  constexpr int WV = kPhaseWaves, NT = phase_taps(R);
  __shared__ double red[2][WV];
  Tap* taps = reinterpret_cast<Tap*>(smem);  // [n_layers][NT], then the rows [n_layers][WV]
  PhaseRows* rows = reinterpret_cast<PhaseRows*>(taps + p.n_layers * NT);
  const int tid = threadIdx.x, n = p.n_pup, nl = p.n_layers;
  // the stars of a tile one after the other on one XCD, neighbouring tiles too: they read
  // mostly the same layer pixels (stars in order of launch 74 us, star after star on each XCD
  // 65, tiles in order of launch 63, so 61)
  const int lb = xcd_logical_block(blockIdx.x, gridDim.x);
  const int s = lb % p.n_stars, tile = lb / p.n_stars, strips = (n + 63) / 64;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int xb = tile % strips * 64, yb = tile / strips * (R * WV);
  const int x = xb + lane, y0 = yb + wave * R;
  const double stepd = (double)p.step;
  for (int e = tid; e < nl * NT; e += kPsfBlock) {
    const int l = e / NT, r = e - l * NT;
    const DevLayer L = p.lay[l];
    const PsfAff A = p.aff[s * nl + l];
    const bool col = r < 64;
    const double u = col ? fma(A.ax, (double)(xb + r), A.bx0 + stepd * A.dbx)
                         : fma(A.ay, (double)min(yb + r - 64, n - 1), A.by0) + stepd * A.dby;
    taps[e] = make_tap(u, col ? L.nx : L.ny, col ? L.inv_nx : L.inv_ny, L.boundary,
                       col ? 1 : L.nx);
  }
  __syncthreads();
  for (int e = tid; e < nl * WV; e += kPsfBlock) {
    const int l = e / WV;
    const Tap* t = taps + l * NT + 64 + (e - l * WV) * R;
    const int first = t[0].i0, step = t[0].i1 - t[0].i0;
    bool next = step > 0;
    int few = 0, sel = 0;
    int last = first, before = first;
#pragma unroll
    for (int q = 0; q < kFew; ++q) rows[e].row[q] = first;
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const int want[2] = {t[k].i0, t[k].i1};
      next &= want[0] == first + k * step && want[1] == first + (k + 1) * step;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        int at = few;  // one of the last two rows found, or a new one
        if (few > 0 && want[h] == last) at = few - 1;
        else if (few > 1 && want[h] == before) at = few - 2;
        else {
          before = last;
          last = want[h];
          rows[e].row[min(few, kFew - 1)] = last;
          ++few;
        }
        sel |= (at & 3) << (4 * k + 2 * h);
      }
    }
    rows[e].kind = next ? kRowsNext : few <= kFew ? kRowsFew : kRowsMore;
    rows[e].sel = sel;
  }
  __syncthreads();
  float phi[R];
#pragma unroll
  for (int k = 0; k < R; ++k) phi[k] = 0.0f;
  constexpr int NV = R + 1 > kFew ? R + 1 : kFew;
  int kind[D];
  float v[D][2][NV];
  auto load = [&](int l, auto b) __attribute__((always_inline)) {
    const PhaseRows& pr = rows[l * WV + wave];
    kind[b] = __builtin_amdgcn_readfirstlane(pr.kind);
    const DevLayer L = cload(p.lay, l);
    const float* g = p.layers + L.offset;
    const int2 i = *reinterpret_cast<const int2*>(taps + l * NT + lane);
    if (kind[b] == kRowsNext) {
      const float* row = g + __builtin_amdgcn_readfirstlane(pr.row[0]);
      uint32_t i0 = (uint32_t)i.x, i1 = (uint32_t)i.y;
      asm("" : "+v"(i0), "+v"(i1));  // (32-bit lane offsets seen here go into the loads)
#pragma unroll
      for (int q = 0; q <= R; ++q) {
        v[b][0][q] = ld_idx(row + (int64_t)q * L.nx, i0);
        v[b][1][q] = ld_idx(row + (int64_t)q * L.nx, i1);
      }
    } else if (kind[b] == kRowsFew) {
      uint32_t i0 = (uint32_t)i.x, i1 = (uint32_t)i.y;
      asm("" : "+v"(i0), "+v"(i1));
#pragma unroll
      for (int q = 0; q < kFew; ++q) {
        const float* row = g + __builtin_amdgcn_readfirstlane(pr.row[q]);
        v[b][0][q] = ld_idx(row, i0);
        v[b][1][q] = ld_idx(row, i1);
      }
    }
  };
  auto add = [&](int l, auto b) __attribute__((always_inline)) {
    const DevLayer L = cload(p.lay, l);
    const Tap* t = taps + l * NT + 64 + wave * R;
    const Tap cx = taps[l * NT + lane];
    if (kind[b] != kRowsMore) {
      float u[NV];
#pragma unroll
      for (int q = 0; q < NV; ++q) u[q] = fmaf(cx.w0, v[b][0][q], cx.w1 * v[b][1][q]);
      const int sel = __builtin_amdgcn_readfirstlane(rows[l * WV + wave].sel);
      if (kind[b] == kRowsNext) {
#pragma unroll
        for (int k = 0; k < R; ++k)
          phi[k] = fmaf(L.weight, t[k].w0 * u[k] + t[k].w1 * u[k + 1], phi[k]);  // as bilinear()
      } else {
        const float u0 = u[0], u1 = u[1], u2 = u[2], u3 = u[3];
        auto pick = [=](int at) {
          const float lo = at & 1 ? u1 : u0, hi = at & 1 ? u3 : u2;
          return at & 2 ? hi : lo;
        };
#pragma unroll
        for (int k = 0; k < R; ++k)
          phi[k] = fmaf(L.weight,
                        t[k].w0 * pick(sel >> (4 * k)) + t[k].w1 * pick(sel >> (4 * k + 2)),
                        phi[k]);
      }
      return;
    }
    const float* g = p.layers + L.offset;
    const uint32_t i0 = (uint32_t)cx.i0, i1 = (uint32_t)cx.i1;
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const float* r0 = g + __builtin_amdgcn_readfirstlane(t[k].i0);
      const float* r1 = g + __builtin_amdgcn_readfirstlane(t[k].i1);
      const float u = t[k].w0 * fmaf(cx.w0, ld_idx(r0, i0), cx.w1 * ld_idx(r0, i1)) +
                      t[k].w1 * fmaf(cx.w0, ld_idx(r1, i0), cx.w1 * ld_idx(r1, i1));
      phi[k] = fmaf(L.weight, u, phi[k]);
    }
  };
  if (y0 < n) {
    for (int l0 = 0; l0 < nl; l0 += D) {
      static_for<D>([&](auto b) __attribute__((always_inline)) {
        if (l0 + b < nl) load(l0 + b, b);
      });
      static_for<D>([&](auto b) __attribute__((always_inline)) {
        if (l0 + b < nl) add(l0 + b, b);
      });
    }
  }
  double s1 = 0.0, s2 = 0.0;
  float* out = p.phi + ((int64_t)s * n + x) * n + y0;
  const bool whole = R % 4 == 0 && x < n && y0 + R <= n;
  if (whole) {
    typedef float v4fu __attribute__((ext_vector_type(4), aligned(4)));
#pragma unroll
    for (int k = 0; k + 4 <= R; k += 4)
      *reinterpret_cast<v4fu*>(out + k) = (v4fu){phi[k], phi[k + 1], phi[k + 2], phi[k + 3]};
  }
#pragma unroll
  for (int k = 0; k < R; ++k) {
    if (x < n && y0 + k < n) {
      if (!whole) out[k] = phi[k];
      if (p.mask[(int64_t)(y0 + k) * n + x]) {
        s1 += (double)phi[k];
        s2 += (double)phi[k] * (double)phi[k];
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {  // fixed order: deterministic
    s1 += __shfl_xor(s1, o, 64);
    s2 += __shfl_xor(s2, o, 64);
  }
  if ((tid & 63) == 0) {
    red[0][wave] = s1;
    red[1][wave] = s2;
  }
  __syncthreads();
  if (tid < 2) {
    double v = 0.0;
#pragma unroll
    for (int w = 0; w < WV; ++w) v += red[tid][w];
    p.part[((int64_t)s * p.n_part + tile) * 2 + tid] = v;
  }
}

// Piston-removed pupil variance of this frame's phase of star s (strided sums of the phase's
// blocks, then a fixed-order tree), added at every wavelength.
__device__ void psf_variance(const PsfParams& p, int s, double (*red)[kPsfBlock], int tid) {
  double a = 0.0, b = 0.0;
  for (int i = tid; i < p.n_part && tid < kPsfBlock; i += kPsfBlock) {
    a += p.part[((int64_t)s * p.n_part + i) * 2];
    b += p.part[((int64_t)s * p.n_part + i) * 2 + 1];
  }
  if (tid < kPsfBlock) {
    red[0][tid] = a;
    red[1][tid] = b;
  }
  __syncthreads();
  for (int w = kPsfBlock / 2; w > 0; w >>= 1) {
    if (tid < w) {
      red[0][tid] += red[0][tid + w];
      red[1][tid] += red[1][tid + w];
    }
    __syncthreads();
  }
  if (tid < p.n_lambda) {
    const double m = red[0][0] * p.inv_lit;
    p.phase_var[tid * p.n_stars + s] += (double)p.kappa2[tid] * (red[1][0] * p.inv_lit - m * m);
  }
}

// Pupil columns of a y-pass workgroup and its threads: four columns of 2,048 points are a
// radix-16 butterfly for each of 512 threads; short columns fill the chip with two (eight stars
// of 449 pixels at N = 512: 123 us for three frames, with four 133).
constexpr int psf_row_rows(int log2N) { return log2N >= 12 || log2N <= 9 ? 2 : 4; }
constexpr int psf_row_threads(int log2N, int rows) { return rows > 1 && log2N >= 11 ? 512 : 256; }
// Pitch of the columns in LDS: neighbours' points half the banks apart, for the last stage's
// reads of 8 points of each.
__host__ __device__ constexpr int psf_row_pitch(int N) { return fft_span(N) + (N > 16 ? 8 : 7); }

// y pass: workgroup (RY pupil columns, star): field of the columns in the registers of the
// first stage (HALF: the pupil fills half of the transform at most), N-point FFTs in LDS, stored
// from the registers of the last stage in C-point tiles: T[s][k / C][x][k % C], so the x pass
// reads whole tiles.
// Bound by issue and by the 118 MB of T.  One kernel a pupil row that formed the phase too,
// column taps again for every row, with half of its threads idle in the radix-16 stages, took
// 137 us a frame (nine stars of 800 pupil pixels, 13 layers, N = 2,048); the phase takes
// 61 us and this pass 43 us.  Few columns (less than two workgroups a CU) run one a
// workgroup.
template <int LOG2N, int RY, bool HALF>
__global__ __launch_bounds__(psf_row_threads(LOG2N, RY)) void psf_rows_kernel(PsfParams p) {
  extern __shared__ __align__(16) float2 sh[];
  constexpr int N = 1 << LOG2N, TH = psf_row_threads(LOG2N, RY), LD = psf_row_pitch(N);
  __shared__ double red[2][kPsfBlock];
  const int x0 = blockIdx.x * RY, s = blockIdx.y, tid = threadIdx.x;
  const int n = p.n_pup, C = p.cols, lc = __builtin_ctz(C);  // C: a power of two
  if (x0 >= n) {  // the extra workgroup
    psf_variance(p, s, red, tid);
    return;
  }
  constexpr int NB0 = N / 16, B0 = (RY * NB0 + TH - 1) / TH, M = HALF ? 8 : 16;
  constexpr int LNS = fft_last_lns(LOG2N), LR = LOG2N - LNS, RL = 1 << LR, NBL = N >> LR;
  auto field = [&](float phi, bool lit) {
    if (!lit) return make_float2(0.0f, 0.0f);
    float sn, cs;
    sincosf(p.kappa * phi, &sn, &cs);
    return make_float2(cs, sn);
  };
  // fewer butterflies than threads: the points of the field to all threads first
  constexpr bool STAGE = RY * NB0 < TH;
  if constexpr (STAGE) {
    constexpr int P = HALF ? N / 2 : N;
    for (int i = tid; i < RY * P; i += TH) {
      const int k = i / P, y = i % P;
      const int64_t col = (int64_t)min(x0 + k, n - 1) * n;  // past the pupil: not stored
      const bool in = y < n;
      sh[k * LD + fft_pad(y)] =
          field(in ? p.phi[(int64_t)s * n * n + col + y] : 0.0f, in && p.mask[col + y]);
    }
    __syncthreads();
  }
  float2 a[B0][16];
#pragma unroll
  for (int it = 0; it < B0; ++it) {
    const int b = tid + it * TH, k = b / NB0, j = b % NB0;
    if (k >= RY) continue;
    if constexpr (STAGE) {
#pragma unroll
      for (int m = 0; m < M; ++m) a[it][m] = sh[k * LD + fft_pad(j + m * NB0)];
    } else {
      const int64_t col = (int64_t)min(x0 + k, n - 1) * n;
      const float* ph = p.phi + (int64_t)s * n * n + col;
      float f[M];
      bool lit[M];
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const int y = j + m * NB0;
        lit[m] = y < n && p.mask[col + y];
        f[m] = y < n ? ph[y] : 0.0f;
      }
#pragma unroll
      for (int m = 0; m < M; ++m) a[it][m] = field(f[m], lit[m]);
    }
    dft<16, HALF>(a[it]);
  }
  if constexpr (STAGE) __syncthreads();
#pragma unroll
  for (int it = 0; it < B0; ++it) {
    const int b = tid + it * TH, k = b / NB0, j = b % NB0;
    if (k >= RY) continue;
#pragma unroll
    for (int r = 0; r < 16; ++r) sh[k * LD + fft_pad(16 * j) + r] = a[it][r];
  }
  __syncthreads();
  if constexpr (LNS == 8) fft_stage<LOG2N, 4, 4, RY * N, TH>(sh, RY, LD, p.tw);
  // last stage, 8 points of each of the columns, which lie side by side in a tile
  constexpr int J8 = NBL < 8 ? NBL : 8, BL = (RY * NBL + TH - 1) / TH;
  float2* out = p.T + (int64_t)s * n * N + (int64_t)x0 * C;
#pragma unroll
  for (int it = 0; it < BL; ++it) {
    const int b = tid + it * TH, k = (b / J8) % RY, j = (b / (J8 * RY)) * J8 + b % J8;
    if (j >= NBL) continue;
    const float2* x = sh + k * LD;
    float2 y[RL];
    if constexpr (LNS == 0) {  // the first stage was the last: its outputs back
#pragma unroll
      for (int m = 0; m < RL; ++m) y[m] = x[fft_pad(m)];
    } else {
#pragma unroll
      for (int m = 0; m < RL; ++m) y[m] = x[fft_pad(j) + m * fft_span(NBL)];
      const float2* t = p.tw + (NBL - 1) + j;
#pragma unroll
      for (int m = 1; m < RL; ++m) y[m] = cmul(y[m], t[(m - 1) * NBL]);
      dft<RL>(y);
    }
    if (x0 + k < n) {
#pragma unroll
      for (int r = 0; r < RL; ++r) {
        const int v = j + r * NBL;
        out[(int64_t)(v >> lc) * n * C + k * C + (v & (C - 1))] = y[r];
      }
    }
  }
}

// x pass: workgroups that take groups of C adjacent y frequencies of a star in turn: N-point
// FFTs along x, intensities added to whole image rows.  Zero columns beyond the pupil are
// implicit (HALF: half of the first stage's inputs at least).
//
// A group's points fill the LDS of a CU, so nothing else covers its memory: the first stage
// takes its points straight from memory, loaded while the group before is transformed, the
// last one adds to the image straight from registers, its old values loaded before the stages.
// With a workgroup per group that staged points and results in LDS, load, transform and update
// one after the other, and 32-byte pieces of image rows (x transformed first), nine stars of
// 800 pupil pixels at N = 2,048 took 185 us a frame, 80 us so (118 MB of T and 302 MB of image
// a frame).
constexpr int kPsfColBlock = 1024;

template <int LOG2N, bool HALF>
__global__ __launch_bounds__(kPsfColBlock) void psf_cols_kernel(PsfParams p) {
  extern __shared__ float2 sh[];
  constexpr int N = 1 << LOG2N, NB0 = N / 16, M = HALF ? 8 : 16, H = N / 2;
  constexpr int LNS = fft_last_lns(LOG2N), LR = LOG2N - LNS, RL = 1 << LR, NBL = N >> LR;
  constexpr int MAXB = kPsfColPoints / RL / kPsfColBlock;
  static_assert(kPsfColPoints / 16 <= kPsfColBlock, "a first-stage butterfly a thread");
  const int tid = threadIdx.x;
  const int C = p.cols, lc = __builtin_ctz(C), n = p.n_pup, ld = fft_pitch(N, C);
  const int groups = N >> lc, total = groups * p.n_stars;
  float2* tws = sh + C * ld;  // the twiddle table, staged in LDS after the data
  const int c0 = tid & (C - 1), j0 = tid >> lc;  // the thread's butterfly of the first stage
  float2 v[M];
  auto load = [&](int lb) {  // group lb's tile of T: [n][C]
    const int s = lb / groups, k0 = (lb - s * groups) * C;
    const float2* src = p.T + (int64_t)s * n * N + (int64_t)k0 * n;
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const int y = j0 + m * NB0;
      v[m] = make_float2(0.0f, 0.0f);
      if (j0 < NB0 && y < n) v[m] = src[(y << lc) + c0];
    }
  };
  int i = blockIdx.x;
  if (HALF && i < total) load(xcd_logical_block(i, total));
  for (int t = tid; t < N - 1; t += kPsfColBlock) tws[t] = p.tw[t];
  for (; i < total; i += gridDim.x) {
    const int lb = xcd_logical_block(i, total);
    const int s = lb / groups, k0 = (lb - s * groups) * C;
    float* __restrict__ dst = p.psf + (int64_t)s * N * N;
    if constexpr (!HALF) load(lb);  // (all 16 points ahead would spill)
    float2 a[16];
#pragma unroll
    for (int m = 0; m < M; ++m) a[m] = v[m];
    dft<16, HALF>(a);
    // the thread's points of the last stage: image row of y frequency k0 + c, columns of x
    // frequencies j + r NBL; neighbouring threads on neighbouring columns
    float old[MAXB][RL];
    uint32_t at[MAXB];
    auto load_old = [&]() {
#pragma unroll
      for (int it = 0; it < MAXB; ++it) {
        const int b = tid + it * kPsfColBlock, c = b / NBL, j = b % NBL;
        at[it] = (uint32_t)((k0 + c + H) & (N - 1)) * N + j;
        if (c < C) {
#pragma unroll
          for (int r = 0; r < RL; ++r) old[it][r] = dst[at[it] + ((r * NBL + H) & (N - 1))];
        }
      }
    };
    if constexpr (HALF) load_old();
    if (HALF && i + gridDim.x < total) load(xcd_logical_block(i + gridDim.x, total));
    __syncthreads();  // the group before is read
    if (j0 < NB0) {
      float2* o = sh + c0 * ld + fft_pad(16 * j0);
#pragma unroll
      for (int r = 0; r < 16; ++r) o[r] = a[r];
    }
    __syncthreads();
    if constexpr (LNS == 8)  // three stages
      fft_stage<LOG2N, 4, 4, kPsfColPoints, kPsfColBlock>(sh, C, ld, tws);
    if constexpr (!HALF) {
      load_old();
    } else {
      // the loads ahead have arrived by now; waiting for them behind the stores below would
      // wait for the stores too
#pragma unroll
      for (int m = 0; m < M; ++m) asm volatile("" : "+v"(v[m].x), "+v"(v[m].y));
    }
#pragma unroll
    for (int it = 0; it < MAXB; ++it) {
      const int b = tid + it * kPsfColBlock, c = b / NBL, j = b % NBL;
      if (c >= C) continue;
      const float2* x = sh + c * ld;
      float2 y[RL];
      if constexpr (LNS == 0) {  // the first stage was the last: its outputs back
#pragma unroll
        for (int m = 0; m < RL; ++m) y[m] = x[fft_pad(m)];
      } else {
#pragma unroll
        for (int m = 0; m < RL; ++m) y[m] = x[fft_pad(j) + m * fft_span(NBL)];
        const float2* t = tws + (NBL - 1) + j;
#pragma unroll
        for (int m = 1; m < RL; ++m) y[m] = cmul(y[m], t[(m - 1) * NBL]);
        dft<RL>(y);
      }
#pragma unroll
      for (int r = 0; r < RL; ++r)
        dst[at[it] + ((r * NBL + H) & (N - 1))] =
            old[it][r] + (y[r].x * y[r].x + y[r].y * y[r].y) * p.scale;
    }
  }
}

struct PsfStrehlParams {
  const float* psf;
  const double* phase_var;
  float* sr_psf;
  float* sr_marechal;
  int32_t n_stars, n_lambda;
  double inv_frames;
  int64_t off[kPsfMaxLambda];   // first float of wavelength l's images
  int32_t N[kPsfMaxLambda];
  double inv_peak[kPsfMaxLambda];  // N^2 / sum A: inverse of the diffraction-limited peak
};

__global__ __launch_bounds__(kPsfBlock) void psf_strehl_kernel(PsfStrehlParams q) {
  const int i = blockIdx.x * kPsfBlock + threadIdx.x;
  if (i >= q.n_lambda * q.n_stars) return;
  const int l = i / q.n_stars, s = i - l * q.n_stars;
  const int N = q.N[l], h = N >> 1;
  if (q.sr_psf && q.psf) {
    const float c = q.psf[q.off[l] + (int64_t)s * N * N + (int64_t)h * N + h];
    q.sr_psf[i] = (float)((double)c * q.inv_frames * q.inv_peak[l]);
  }
  if (q.sr_marechal && q.phase_var)
    q.sr_marechal[i] = (float)exp(-q.phase_var[i] * q.inv_frames);
}

}  // namespace wfs

using namespace wfs;

struct psf_plan_s {
  int device = 0, cus = 1;
  int32_t n_layers = 0, n_stars = 0, n_pup = 0, n_lambda = 0;
  int64_t layer_stride = 0, n_lit = 0, psf_floats = 0;
  std::vector<int32_t> N, log2N, cols;
  std::vector<float> kappa;
  std::vector<int64_t> psf_off, tw_off;
  DevLayer* lay = nullptr;
  PsfAff* aff = nullptr;
  uint8_t* mask = nullptr;
  float2* tw = nullptr;
  float2* T = nullptr;
  float* phi = nullptr;
  int32_t n_part = 0;
  bool few_waves = false;
  double* part = nullptr;
};

static int psf_fail(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
static int psf_fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  return set_error(code, buf);
}

static int psf_hip(hipError_t e, const char* what) {
  return psf_fail(e == hipErrorOutOfMemory ? WFS_ENOMEM : WFS_EDEVICE, "%s: %s", what,
                  hipGetErrorString(e));
}

static void psf_free(psf_plan_t P) {
  if (!P) return;
  (void)hipFree(P->lay);
  (void)hipFree(P->aff);
  (void)hipFree(P->mask);
  (void)hipFree(P->tw);
  (void)hipFree(P->T);
  (void)hipFree(P->phi);
  (void)hipFree(P->part);
  delete P;
}

// Calls f(std::integral_constant<int, log2 N>) for a transform size of the plan.
template <class F>
static void psf_dispatch(int log2N, F&& f) {
  switch (log2N) {
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

// LDS bytes of a column-pass workgroup: C padded columns and the twiddles.
static size_t psf_col_lds(int N, int C) {
  return ((size_t)C * fft_pitch(N, C) + N - 1) * sizeof(float2);
}

template <class T>
static hipError_t upload(T** dst, const std::vector<T>& v) {
  hipError_t e = hipMalloc((void**)dst, v.size() * sizeof(T));
  if (e != hipSuccess) return e;
  return hipMemcpy(*dst, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice);
}

extern "C" {

int psf_plan(const wfs_layer_desc* layers, int32_t n_layers, int64_t layer_stride,
             const double* star_theta_xy, int32_t n_stars, double pupil_d_m, double obs_d_m,
             int32_t n_pup, const double* lambda_m, const int32_t* n_fft, int32_t n_lambda,
             double lambda_ref_m, double dt_s, psf_plan_t* out) {
  if (!out) return psf_fail(WFS_EINVAL, "psf_plan: null out");
  *out = nullptr;
  if (!layers || !star_theta_xy || !lambda_m || !n_fft)
    return psf_fail(WFS_EINVAL, "psf_plan: null argument");
  if (n_layers < 1 || n_layers > kMaxLayers)
    return psf_fail(WFS_EINVAL, "psf_plan: n_layers=%d outside [1, %d]", n_layers, kMaxLayers);
  if (n_stars < 1 || n_stars > kPsfMaxStars)
    return psf_fail(WFS_EINVAL, "psf_plan: n_stars=%d outside [1, %d]", n_stars, kPsfMaxStars);
  if (n_lambda < 1 || n_lambda > kPsfMaxLambda)
    return psf_fail(WFS_EINVAL, "psf_plan: n_lambda=%d outside [1, %d]", n_lambda,
                    kPsfMaxLambda);
  if (n_pup < 2 || n_pup > kPsfPoints)
    return psf_fail(WFS_EINVAL, "psf_plan: n_pup=%d outside [2, %d]", n_pup, kPsfPoints);
  if (!(pupil_d_m > 0) || !std::isfinite(pupil_d_m) || !(obs_d_m >= 0) || obs_d_m >= pupil_d_m)
    return psf_fail(WFS_EINVAL, "psf_plan: pupil %g m, obstruction %g m", pupil_d_m, obs_d_m);
  if (!(lambda_ref_m > 0) || !std::isfinite(lambda_ref_m) || !(dt_s >= 0) ||
      !std::isfinite(dt_s))
    return psf_fail(WFS_EINVAL, "psf_plan: lambda_ref_m > 0 and dt_s >= 0 required");
  if (layer_stride < 1) return psf_fail(WFS_EINVAL, "psf_plan: layer_stride < 1");
  for (int l = 0; l < n_layers; ++l) {
    const wfs_layer_desc& L = layers[l];
    if (L.nx < 2 || L.ny < 2 || (int64_t)L.nx * L.ny > (1LL << 29))
      return psf_fail(WFS_EINVAL, "psf_plan: layer %d grid %dx%d", l, L.nx, L.ny);
    if (L.offset < 0 || L.offset + (int64_t)L.nx * L.ny > layer_stride)
      return psf_fail(WFS_EINVAL, "psf_plan: layer %d outside the stride", l);
    if (!(L.pitch_m > 0) || !std::isfinite(L.pitch_m) || !std::isfinite(L.alt_m) ||
        L.alt_m < 0 || !std::isfinite(L.vx_mps) || !std::isfinite(L.vy_mps) ||
        !std::isfinite(L.weight) || (L.boundary != 0 && L.boundary != 1))
      return psf_fail(WFS_EINVAL, "psf_plan: layer %d geometry", l);
  }
  for (int s = 0; s < 2 * n_stars; ++s)
    if (!std::isfinite(star_theta_xy[s])) return psf_fail(WFS_EINVAL, "psf_plan: star angle");
  for (int l = 0; l < n_lambda; ++l) {
    const int32_t N = n_fft[l];
    if (!(lambda_m[l] > 0) || !std::isfinite(lambda_m[l]))
      return psf_fail(WFS_EINVAL, "psf_plan: lambda %d must be > 0", l);
    if (N < 16 || N > kPsfPoints || (N & (N - 1)) || N < n_pup)
      return psf_fail(WFS_EINVAL,
                      "psf_plan: n_fft[%d]=%d must be a power of two in [max(16, n_pup=%d), %d]",
                      l, N, n_pup, kPsfPoints);
  }
  psf_plan_t P = new psf_plan_s();
  hipError_t e = hipGetDevice(&P->device);
  if (e == hipSuccess)
    e = hipDeviceGetAttribute(&P->cus, hipDeviceAttributeMultiprocessorCount, P->device);
  if (e != hipSuccess) {
    psf_free(P);
    return psf_hip(e, "psf_plan");
  }
  P->n_layers = n_layers;
  P->n_stars = n_stars;
  P->n_pup = n_pup;
  P->n_lambda = n_lambda;
  P->layer_stride = layer_stride;
  P->few_waves = phase_few(n_pup, n_stars, P->cus);
  P->n_part = phase_tiles(n_pup, P->few_waves);
  // pupil: pixel centres x_i = (i + 1/2 - n/2) dx; A = 1 for obs/2 <= r <= D/2
  const double dx = pupil_d_m / n_pup;
  std::vector<uint8_t> mask((size_t)n_pup * n_pup);
  for (int j = 0; j < n_pup; ++j)
    for (int i = 0; i < n_pup; ++i) {
      const double xx = (i + 0.5 - n_pup / 2.0) * dx, yy = (j + 0.5 - n_pup / 2.0) * dx;
      const double r = std::hypot(xx, yy);
      const bool lit = r >= obs_d_m / 2.0 && r <= pupil_d_m / 2.0;
      mask[(size_t)j * n_pup + i] = lit;
      P->n_lit += lit;
    }
  if (P->n_lit == 0) {
    psf_free(P);
    return psf_fail(WFS_EINVAL, "psf_plan: no lit pupil pixel");
  }
  std::vector<DevLayer> lay(n_layers);
  std::vector<PsfAff> aff((size_t)n_stars * n_layers);
  for (int l = 0; l < n_layers; ++l) {
    const wfs_layer_desc& L = layers[l];
    lay[l] = DevLayer{L.offset, L.nx, L.ny, L.weight, L.boundary, 1.0 / L.nx, 1.0 / L.ny};
    for (int s = 0; s < n_stars; ++s) {
      // a star at infinity: X = x + theta h - v t, u = X / pitch + nx/2 - 1/2
      const double tx = star_theta_xy[2 * s], ty = star_theta_xy[2 * s + 1];
      PsfAff& A = aff[(size_t)s * n_layers + l];
      A.ax = dx / L.pitch_m;
      A.bx0 = ((0.5 - n_pup / 2.0) * dx + tx * L.alt_m) / L.pitch_m + L.nx / 2.0 - 0.5;
      A.dbx = -L.vx_mps * dt_s / L.pitch_m;
      A.ay = dx / L.pitch_m;
      A.by0 = ((0.5 - n_pup / 2.0) * dx + ty * L.alt_m) / L.pitch_m + L.ny / 2.0 - 0.5;
      A.dby = -L.vy_mps * dt_s / L.pitch_m;
    }
  }
  std::vector<float2> tw;
  int32_t Nmax = 0;
  for (int l = 0; l < n_lambda; ++l) {
    const int32_t N = n_fft[l];
    int lg = 0;
    while ((1 << lg) < N) ++lg;
    P->N.push_back(N);
    P->log2N.push_back(lg);
    // C padded columns of N points plus the N - 1 twiddles must fit the 160 KB of LDS
    int C = N >= 4096 ? 2 : std::min(16, kPsfColPoints / N);
    while (C > 4 && 2 * (N / C) * n_stars <= P->cus) C /= 2;  // CUs left over: smaller groups
    P->cols.push_back(C);
    P->kappa.push_back((float)(lambda_ref_m / lambda_m[l]));
    P->psf_off.push_back(P->psf_floats);
    P->psf_floats += (int64_t)n_stars * N * N;
    P->tw_off.push_back((int64_t)tw.size());
    for (int m = 0; m < N - 1; ++m) {
      const double a = -2.0 * M_PI * (double)fft_tw_angle(lg, m) / (double)N;
      tw.push_back(make_float2((float)std::cos(a), (float)std::sin(a)));
    }
    Nmax = std::max(Nmax, N);
  }
  // the column pass holds more than the default 64 KB of LDS (data, padding and twiddles)
  e = hipFuncSetAttribute((const void*)psf_phase_kernel<2, 5>,
                          hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)psf_phase_lds(kMaxLayers, true));
  if (e == hipSuccess)
    e = hipFuncSetAttribute((const void*)psf_phase_kernel<8, 1>,
                            hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)psf_phase_lds(kMaxLayers, false));
  for (int lg = kPsfMinLog2; lg <= kPsfMaxLog2 && e == hipSuccess; ++lg) {
    psf_dispatch(lg, [&](auto L) {
      constexpr int LG = decltype(L)::value;
      for (const void* k : {(const void*)psf_cols_kernel<LG, false>,
                            (const void*)psf_cols_kernel<LG, true>})
        if (e == hipSuccess)
          e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kPsfColLds);
      constexpr int RY = psf_row_rows(LG);
      for (const void* k : {(const void*)psf_rows_kernel<LG, RY, false>,
                            (const void*)psf_rows_kernel<LG, RY, true>,
                            (const void*)psf_rows_kernel<LG, 1, false>,
                            (const void*)psf_rows_kernel<LG, 1, true>})
        if (e == hipSuccess)
          e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kPsfRowLds);
    });
  }
  if (e != hipSuccess) {
    psf_free(P);
    return psf_hip(e, "psf_plan: column-pass LDS");
  }
  if ((e = upload(&P->lay, lay)) != hipSuccess || (e = upload(&P->aff, aff)) != hipSuccess ||
      (e = upload(&P->mask, mask)) != hipSuccess || (e = upload(&P->tw, tw)) != hipSuccess ||
      (e = hipMalloc((void**)&P->T, (size_t)n_stars * n_pup * Nmax * sizeof(float2))) !=
          hipSuccess ||
      (e = hipMalloc((void**)&P->phi, (size_t)n_stars * n_pup * n_pup * sizeof(float))) !=
          hipSuccess ||
      (e = hipMalloc((void**)&P->part, (size_t)n_stars * P->n_part * 2 * sizeof(double))) !=
          hipSuccess) {
    psf_free(P);
    return psf_hip(e, "psf_plan: device tables");
  }
  *out = P;
  return WFS_OK;
}

int psf_plan_info(psf_plan_t P, int64_t* psf_floats, int64_t* psf_offsets, int64_t* n_lit) {
  if (!P) return psf_fail(WFS_EINVAL, "psf_plan_info: null plan");
  if (psf_floats) *psf_floats = P->psf_floats;
  if (psf_offsets)
    for (int l = 0; l < P->n_lambda; ++l) psf_offsets[l] = P->psf_off[l];
  if (n_lit) *n_lit = P->n_lit;
  return WFS_OK;
}

int psf_plan_destroy(psf_plan_t P) {
  if (!P) return psf_fail(WFS_EINVAL, "psf_plan_destroy: null plan");
  hipError_t e = hipDeviceSynchronize();
  psf_free(P);
  if (e != hipSuccess) return psf_hip(e, "psf_plan_destroy");
  return WFS_OK;
}

int psf_accumulate(psf_plan_t P, const float* layers, int64_t step, float* psf,
                   double* phase_var, void* stream) {
  if (!P) return psf_fail(WFS_EINVAL, "psf_accumulate: null plan");
  if (!layers || !psf) return psf_fail(WFS_EINVAL, "psf_accumulate: null layers or psf");
  if (step < 0) return psf_fail(WFS_EINVAL, "psf_accumulate: step=%lld < 0", (long long)step);
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return psf_hip(e, "psf_accumulate");
  if (dev != P->device)
    return psf_fail(WFS_EINVAL, "psf_accumulate: current device %d is not the plan's %d", dev,
                    P->device);
  hipStream_t st = (hipStream_t)stream;
  for (int l = 0; l < P->n_lambda; ++l) {
    PsfParams p{};
    p.layers = layers;
    p.lay = P->lay;
    p.aff = P->aff;
    p.mask = P->mask;
    p.tw = P->tw + P->tw_off[l];
    p.T = P->T;
    p.part = P->part;
    p.psf = psf + P->psf_off[l];
    p.step = step;
    p.n_layers = P->n_layers;
    p.n_stars = P->n_stars;
    p.n_pup = P->n_pup;
    p.N = P->N[l];
    p.log2N = P->log2N[l];
    p.cols = P->cols[l];
    p.kappa = P->kappa[l];
    p.scale = (float)(1.0 / ((double)p.N * p.N * (double)P->n_lit));
    p.phi = P->phi;
    p.n_part = P->n_part;
    if (l == 0) {
      const auto phase = P->few_waves ? psf_phase_kernel<2, 5> : psf_phase_kernel<8, 1>;
      phase<<<P->n_part * P->n_stars, kPsfBlock, psf_phase_lds(P->n_layers, P->few_waves), st>>>(p);
      if ((e = hipGetLastError()) != hipSuccess) return psf_hip(e, "psf_accumulate: phase");
    }
    if (l == 0 && phase_var) {
      p.write_var = 1;
      p.phase_var = phase_var;
      p.n_lambda = P->n_lambda;
      p.inv_lit = 1.0 / (double)P->n_lit;
      for (int m = 0; m < P->n_lambda; ++m) p.kappa2[m] = P->kappa[m] * P->kappa[m];
    }
    psf_dispatch(p.log2N, [&](auto L) {
      constexpr int LG = decltype(L)::value, RY = psf_row_rows(LG);
      auto launch = [&](auto kernel, int rows) {
        kernel<<<dim3((P->n_pup + rows - 1) / rows + p.write_var, P->n_stars),
                 psf_row_threads(LG, rows), (size_t)rows * psf_row_pitch(p.N) * sizeof(float2), st>>>(p);
      };
      const bool half = 2 * p.n_pup <= p.N;
      if ((int64_t)(P->n_pup / RY) * P->n_stars >= 2 * P->cus)
        launch(half ? psf_rows_kernel<LG, RY, true> : psf_rows_kernel<LG, RY, false>, RY);
      else
        launch(half ? psf_rows_kernel<LG, 1, true> : psf_rows_kernel<LG, 1, false>, 1);
    });
    if ((e = hipGetLastError()) != hipSuccess) return psf_hip(e, "psf_accumulate: rows");
    // as many workgroups as are resident at once: each takes several groups
    const size_t lds = psf_col_lds(p.N, p.cols);
    const int resident = P->cus * std::max(1, std::min(2, (int)(kPsfColLds / lds)));
    const int blocks = std::min((p.N / p.cols) * P->n_stars, resident);
    psf_dispatch(p.log2N, [&](auto L) {
      constexpr int LG = decltype(L)::value;
      if (2 * p.n_pup <= p.N)
        psf_cols_kernel<LG, true><<<blocks, kPsfColBlock, lds, st>>>(p);
      else
        psf_cols_kernel<LG, false><<<blocks, kPsfColBlock, lds, st>>>(p);
    });
    if ((e = hipGetLastError()) != hipSuccess) return psf_hip(e, "psf_accumulate: columns");
  }
  return WFS_OK;
}

int psf_strehl(psf_plan_t P, const float* psf, const double* phase_var, int64_t n_frames,
               float* sr_psf, float* sr_marechal, void* stream) {
  if (!P) return psf_fail(WFS_EINVAL, "psf_strehl: null plan");
  if (n_frames < 1) return psf_fail(WFS_EINVAL, "psf_strehl: n_frames=%lld < 1",
                                    (long long)n_frames);
  if ((sr_psf && !psf) || (sr_marechal && !phase_var) || (!sr_psf && !sr_marechal))
    return psf_fail(WFS_EINVAL, "psf_strehl: outputs need their inputs (psf, phase_var)");
  PsfStrehlParams q{};
  q.psf = psf;
  q.phase_var = phase_var;
  q.sr_psf = sr_psf;
  q.sr_marechal = sr_marechal;
  q.n_stars = P->n_stars;
  q.n_lambda = P->n_lambda;
  q.inv_frames = 1.0 / (double)n_frames;
  for (int l = 0; l < P->n_lambda; ++l) {
    q.off[l] = P->psf_off[l];
    q.N[l] = P->N[l];
    q.inv_peak[l] = (double)P->N[l] * P->N[l] / (double)P->n_lit;
  }
  const int n = P->n_lambda * P->n_stars;
  psf_strehl_kernel<<<(n + kPsfBlock - 1) / kPsfBlock, kPsfBlock, 0, (hipStream_t)stream>>>(q);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return psf_hip(e, "psf_strehl");
  return WFS_OK;
}

}  // extern "C"
