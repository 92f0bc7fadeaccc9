// Adjoint of the noise-free forward sensor model (slopes -> layer screens), lag-domain path.
//
// Forward, per subaperture (see wfs_otf.h):  B[q] = c sum_k A[k] T[k] e^{2 pi i k.q / n_pix}
// over all lags k, with A[k] = sum_m E[m] conj(E[m+k]), T[k] = Kel[k] s(kx) s(ky), and the
// slopes c_x = sum (x_q) B / sum B, c_y likewise.  Given g = dL/d(c_x, c_y):
//   g_B[q] = (g_x (x_q - c_x) + g_y (y_q - c_y)) / sum B          (0 when sum B <= 0)
//   U[k]   = c T[k] ghat[k],  ghat[k] = sum_q g_B[q] e^{2 pi i k.q / n_pix}   (Hermitian in k)
//   dL     = Re sum_k U[k] dA[k],  dE[m] = i E[m] dpsi[m]
//   =>  g_psi[p] = -2 Im(E[p] V[p]),   V[p] = sum_{m'} U[m' - p] conj(E[m'])
// g_B is a plane in q, so ghat vanishes off the axes k_x = 0 and k_y = 0 modulo n_pix, and
// with S1[K] = sum_q q e^{2 pi i K q / n_pix} = n_pix / (e^{2 pi i K / n_pix} - 1):
//   ghat[0] = -n_pix^2 (g_x c_x + g_y c_y) / sum B,  ghat[K_x] = n_pix g_x S1[K_x] / sum B,
//   ghat[K_y] = n_pix g_y S1[K_y] / sum B.
// Only the lags with dy or dx a multiple of n_pix take part (n_sub = 10, 8 x 8 pixels: 105 of
// 361, and about 30 of the 100 field pixels per V[p]).  Bound by vector issue: the adjoint of
// six 80 x 80 LGS without its gather took 107 us with every lag in U and V, 42 us so.
// and the layer gradient is the transpose of the bilinear projection, kappa w_l times the
// stencil weights (subaperture fields recomputed).  Two ways to form it:
//   gather (default): g_psi (kappa applied) goes to a phase-layout buffer, then one thread per
//     layer pixel sums, sensor by sensor, the stencil weights of the pupil pixels whose
//     forward taps touch it (the same FP64 taps as the forward) -- bitwise deterministic.
//     Layers whose pupil and layer pitches are within about a factor of two read those
//     pupil pixels from per-step lists (one small kernel per call builds them, the gather
//     then needs no FP64 and no searches); the others search their candidates per tile;
//   atomic scatter: each pupil pixel adds its four weighted taps with FP32 atomics.
#include "wfs_fft.h"
#include "wfs_otf.h"

namespace wfs {

// Lag classes of one axis: the multiples of n_pix among the lags -(ns-1) .. ns-1.
__host__ __device__ inline int adj_classes(int ns, int n_pix) {
  return 1 + 2 * ((ns - 1) / n_pix);
}
// Those kept by columns: none where the rows hold every lag already.
__host__ __device__ inline int adj_col_classes(int ns, int n_pix) {
  return n_pix == 1 ? 0 : adj_classes(ns, n_pix);
}

struct AdjLds {
  int ur_off, uc_off, g_off, total;
};

// Per-wave LDS of the adjoint: the forward layout and U on the lag classes: UR [classes][2 ns -
// 1] (dy a multiple of n_pix, every dx) and UC (dx a multiple, every dy; zero where dy is one
// too, absent for one pixel), then ghat along x and y.  Once the spot (or only the field) is formed, only E and the
// lag-phase table of the forward layout are read again, so in the gather form (no stencil
// taps) these go into the dead union between them when they fit; the atomic form keeps its
// taps there and places them after the forward layout.
__host__ __device__ inline AdjLds adj_lds_layout(int ns, int n_layers, int n_pix, bool gather) {
  const OtfLds f = otf_lds_layout(ns, n_layers, n_pix);
  const int rb = adj_classes(ns, n_pix) * (2 * ns - 1) * 8;
  const int cb = adj_col_classes(ns, n_pix) * (2 * ns - 1) * 8;
  AdjLds a;
  const int e_end = (ns * ns * 8 + 15) & ~15;
  const bool in = gather && e_end + rb + cb + 2 * n_pix * 8 <= f.tw_off;
  a.ur_off = in ? e_end : f.total;
  a.uc_off = a.ur_off + rb;
  a.g_off = a.uc_off + cb;
  a.total = in ? f.total : (a.g_off + 2 * n_pix * 8 + 15) & ~15;
  return a;
}

template <int NS, bool FUSED>
__device__ void otf_adjoint_subap(const AdjParams& ap, int t, int64_t step, char* wsm) {
  const FwdParams& p = ap.f;
  const int lane = lane_id();
  int b, sid, v;
  t = __builtin_amdgcn_readfirstlane(t);
  task_of(p.otf, t, b, sid, v);
  const DevSensor S = cload(p.sen, sid);
  const DevSubap sb = cload(p.sub, S.valid_off + v);
  const int np = S.n_pix, np2 = np * np;
  const OtfLds lo = otf_lds_layout(NS, p.n_layers, np);
  const AdjLds la = adj_lds_layout(NS, p.n_layers, np, ap.gpsi != nullptr);
  const float gx = ap.grad_slopes[(int64_t)b * p.n_slopes + S.slope_off + v];
  const float gy = ap.grad_slopes[(int64_t)b * p.n_slopes + S.slope_off + S.n_valid + v];
  float s0, cx, cy;
  if (ap.fwd_slopes) {
    otf_field<NS, FUSED ? kFieldGather : kFieldPhase>(p, S, sb, sid, b, (double)step, wsm, lo);
    s0 = ap.fwd_aux[(int64_t)b * p.n_valid_total + S.aux_off + v];
    cx = ap.fwd_slopes[(int64_t)b * p.n_slopes + S.slope_off + v];
    cy = ap.fwd_slopes[(int64_t)b * p.n_slopes + S.slope_off + S.n_valid + v];
  } else {
    otf_spot<NS, FUSED ? kFieldGather : kFieldPhase>(p, S, sb, sid, b, step, wsm, lo);
    const Cog c = cog_sums(p, S, sid, b, v, step, reinterpret_cast<const float*>(wsm + lo.b_off));
    s0 = c.s0;
    cx = s0 > 0.0f ? c.sx / s0 : 0.0f;
    cy = s0 > 0.0f ? c.sy / s0 : 0.0f;
  }
  wave_sync();
  // gather mode: this subaperture's block of the sensor's pupil-frame gradient image
  float* gout = ap.gpsi ? ap.gpsi + (int64_t)b * p.pupil_per_real + S.pupil_off +
                              (int64_t)sb.a * NS * S.n_pup + sb.b * NS
                        : nullptr;
  if (!(s0 > 0.0f) || (gx == 0.0f && gy == 0.0f)) {  // wave-uniform: no gradient
    if (gout)
      for (int q = lane; q < NS * NS; q += kWave) {
        const int r = small_div<NS>(q);
        gout[r * S.n_pup + q - r * NS] = 0.0f;
      }
    return;
  }
  constexpr int NL = 2 * NS - 1;
  const int ncl = adj_classes(NS, np), hcl = ncl >> 1;
  const float inv = 1.0f / s0;
  float2* GX = reinterpret_cast<float2*>(wsm + la.g_off);  // ghat along x, then along y
  float2* GY = GX + np;
  for (int K = lane; K < np; K += kWave) {
    const float2 s1 = p.wtab[S.wtab_off + np + K];  // n_pix S1[K], 0 at K = 0
    const float fx = gx * inv, fy = gy * inv;
    float2 hx = make_float2(fx * s1.x, fx * s1.y);
    if (K == 0) hx.x = -(float)np2 * (fx * cx + fy * cy);
    GX[K] = hx;
    GY[K] = make_float2(fy * s1.x, fy * s1.y);
  }
  wave_sync();
  // U[k] = c Kel(k) s(kx) s(ky) ghat[k mod n_pix] on the lag classes
  const NaEntry el = na_entry(p, step);
  float2* UR = reinterpret_cast<float2*>(wsm + la.ur_off);
  float2* UC = reinterpret_cast<float2*>(wsm + la.uc_off);
  const float2* stab = reinterpret_cast<const float2*>(wsm + lo.stab_off);
  auto lag_u = [&](int dy, int dx, float2 g) {
    const float2 k = elong_tf(sb, el, fmaf((float)dx, sb.ex, (float)dy * sb.ey), S.flux_c);
    return cmul2(cmul2(cmul2(stab[dx + NS - 1], stab[dy + NS - 1]), k), g);
  };
  for (int t2 = lane; t2 < (ncl + adj_col_classes(NS, np)) * NL; t2 += kWave) {
    const bool col = t2 >= ncl * NL;
    const int u = col ? t2 - ncl * NL : t2;
    const int cls = small_div<NL>(u), i = u - cls * NL;
    const int d = (cls - hcl) * np, e = i - (NS - 1);  // the class's lag and the other axis'
    const int ep = e + np * NS;  // lags -> bins modulo n_pix
    const int K = ep - np * fdiv(ep, np, S.inv_npix);
    // UC leaves the lags of both classes to UR (GY[0] = 0)
    UR[t2] = lag_u(col ? e : d, col ? d : e, col ? GY[K] : GX[K]);
  }
  // taps again (the forward scratch region is free now); the gather mode needs none
  const int nlay = p.n_layers;
  Tap* taps = reinterpret_cast<Tap*>(wsm + lo.taps_off);
  const double stepd = (double)step;
  if (!gout) {
    for (int t2 = lane; t2 < 2 * NS * nlay; t2 += kWave) {
      const int l = t2 / (2 * NS), k = t2 - l * (2 * NS);
      taps[t2] = (k < NS) ? col_tap(p, sid, l, sb.b * NS + k, stepd)
                          : row_tap(p, sid, l, sb.a * NS + (k - NS), stepd);
    }
  }
  wave_sync();
  const float2* E = reinterpret_cast<const float2*>(wsm + lo.e_off);
  float* gl = ap.grad_layers + (int64_t)b * p.layer_stride;
  // lane (column c, row group): pixels (rg + slot RG, c); the field pixels of the row and
  // column classes of a pixel, n_pix apart from its own row (z: r2 = r mod n_pix + z n_pix)
  constexpr int RG = kWave / NS < NS ? kWave / NS : NS, SLOTS = (NS + RG - 1) / RG;
  const int rg = small_div<NS>(lane), c = lane - rg * NS;
  const int nz = fdiv(NS + np - 1, np, S.inv_npix);
  const int c0 = c - np * fdiv(c, np, S.inv_npix);
  int rr[SLOTS];
  float2 V[SLOTS];
#pragma unroll
  for (int k = 0; k < SLOTS; ++k) {
    rr[k] = min(rg + k * RG, NS - 1);
    V[k] = make_float2(0.0f, 0.0f);
  }
  // u conj(f)
  auto corr = [](float2 u, float2 f, float2 v) {
    return make_float2(fmaf(u.x, f.x, fmaf(u.y, f.y, v.x)),
                       fmaf(u.y, f.x, fmaf(-u.x, f.y, v.y)));
  };
  for (int z = 0; z < nz; ++z) {
#pragma unroll
    for (int k = 0; k < SLOTS; ++k) {
      const int r0 = rr[k] - np * fdiv(rr[k], np, S.inv_npix), r2 = r0 + z * np;
      if (r2 < NS) {
        const int cls = fdiv(r2 - rr[k] + np * NS, np, S.inv_npix) - NS + hcl;
        const float2* u = UR + cls * NL + (NS - 1 - c);
#pragma unroll
        for (int c2 = 0; c2 < NS; ++c2) V[k] = corr(u[c2], E[r2 * NS + c2], V[k]);
      }
    }
    const int c2 = c0 + z * np;
    if (c2 < NS && np > 1) {  // (one pixel: every lag is in UR)
      const int cls = fdiv(c2 - c + np * NS, np, S.inv_npix) - NS + hcl;
      float2 f[NS];
#pragma unroll
      for (int r2 = 0; r2 < NS; ++r2) f[r2] = E[r2 * NS + c2];
#pragma unroll
      for (int k = 0; k < SLOTS; ++k) {
        const float2* u = UC + cls * NL + (NS - 1 - rr[k]);
#pragma unroll
        for (int r2 = 0; r2 < NS; ++r2) V[k] = corr(u[r2], f[r2], V[k]);
      }
    }
  }
#pragma unroll
  for (int k = 0; k < SLOTS; ++k) {
    const int r = rg + k * RG;
    if (rg >= RG || r >= NS) continue;
    const float2 e = E[r * NS + c];
    if (!gout && e.x == 0.0f && e.y == 0.0f) continue;  // dark pixel
    const float gpsi = -2.0f * (e.x * V[k].y + e.y * V[k].x) * S.kappa;
    if (gout) {
      gout[r * S.n_pup + c] = gpsi;
      continue;
    }
    for (int l = 0; l < nlay; ++l) {
      const DevLayer& L = p.lay[l];
      const Tap cxt = taps[l * 2 * NS + c];
      const Tap ryt = taps[l * 2 * NS + NS + r];
      const float gw = gpsi * L.weight;
      float* g = gl + L.offset;
      const float w00 = ryt.w0 * cxt.w0 * gw, w01 = ryt.w0 * cxt.w1 * gw;
      const float w10 = ryt.w1 * cxt.w0 * gw, w11 = ryt.w1 * cxt.w1 * gw;
      if (w00 != 0.0f) atomicAdd(g + ryt.i0 + cxt.i0, w00);
      if (w01 != 0.0f) atomicAdd(g + ryt.i0 + cxt.i1, w01);
      if (w10 != 0.0f) atomicAdd(g + ryt.i1 + cxt.i0, w10);
      if (w11 != 0.0f) atomicAdd(g + ryt.i1 + cxt.i1, w11);
    }
  }
  wave_sync();
}

template <int NS, bool FUSED>
__global__ __launch_bounds__(kBlock) void wfs_adjoint_kernel(AdjParams ap) {
  extern __shared__ __align__(16) char smem[];
  const FwdParams& p = ap.f;
  const int64_t step = current_step(p);
  const int wave = threadIdx.x >> 6;
  char* wsm = smem + wave * p.lds_per_wave;
  const int total = p.otf.per_real * p.batch;
  const int L = p.xcd_remap ? xcd_logical_block(blockIdx.x, gridDim.x) : blockIdx.x;
  const int t = L * kWavesPerBlock + wave;  // one subaperture per wave
  if (t < total) otf_adjoint_subap<NS, FUSED>(ap, t, step, wsm);
}

// Gather tiles: kGTW layer columns x kGTH layer rows per block; wave w takes the rows
// w, w + 4, ... (kGPix rows per thread).
constexpr int kGTW = 64;
constexpr int kGPix = 4;
constexpr int kGTH = kGPix * kBlock / kGTW;
constexpr int kGCols = 128;  // candidate pupil columns per pass, the last one zero
constexpr int kGPass = kGCols - 1;
constexpr int kGRows = 32;   // candidate pupil rows per pass

// Candidate taps of a tile: pupil index k, the tap's lower index relative to the tile start
// (floor(w) - m n - tile start, w the layer coordinate, m the periodic image) and the weight
// of the upper neighbour.  The lower weight is 1 - w1, as in the forward's make_tap.
struct GTap {
  int32_t k, rel;
  float w1;
  int32_t pad;
};

// Exact forward tap of pupil index k against layer image m (see make_tap: for a periodic
// grid the fractional part of the unwrapped coordinate equals that of the wrapped one; for a
// zero boundary, candidates lie within a few pixels of the grid, where no clamping happens).
__device__ __forceinline__ GTap gather_tap(double a, double b0, double db, double stepd,
                                           int k, int64_t shift) {
  const double w = fma(a, (double)k, b0) + stepd * db;
  const double f0 = floor(w);
  GTap t;
  t.k = k;
  t.rel = (int32_t)((int64_t)f0 - shift);
  t.w1 = (float)(w - f0);
  t.pad = 0;
  return t;
}

// Pupil index range [lo, hi] whose coordinate w = a k + b (a > 0) falls in [t0 - 1, t1 + 1),
// with one index of slack on each side, clamped to [0, npup).
__device__ __forceinline__ void cand_range(double inv_a, double b, double t0, double t1,
                                           int npup, int& lo, int& hi) {
  // one index of slack on each side also covers the rounding of the reciprocal
  const double lo_d = floor((t0 - 1.0 - b) * inv_a) - 1.0;
  const double hi_d = ceil((t1 + 1.0 - b) * inv_a) + 1.0;
  lo = lo_d < 0.0 ? 0 : (lo_d > (double)npup ? npup : (int)lo_d);
  hi = hi_d < -1.0 ? -1 : (hi_d > (double)(npup - 1) ? npup - 1 : (int)hi_d);
}

// Periodic images m whose layer window [t0 - 1 + m n, t1 + 1 + m n) can meet the pupil's
// coordinate range [w(0), w(npup - 1)]; a single image for a zero boundary.
__device__ __forceinline__ void image_range(double a, double b, int n, double inv_n, int npup,
                                            int t0, int t1, int boundary, int& m_lo,
                                            int& m_hi) {
  if (boundary != 0) {
    m_lo = m_hi = 0;
    return;
  }
  const double w0 = b, w1 = fma(a, (double)(npup - 1), b);
  // floor / ceil of the bounds already include every image the rounding could move in
  m_lo = (int)floor((w0 - t1 - 1.0) * inv_n);
  m_hi = (int)ceil((w1 - t0 + 1.0) * inv_n);
}

// Layer gradient, gather form: block = (realisation, layer, kGTH x kGTW tile); thread =
// layer pixel.  For every sensor, pass by pass over the tile's candidate pupil rows and
// columns (every periodic image, kGRows x kGPass at a time): their exact forward taps and the
// rectangle of the sensor's phase-gradient image they span go to LDS (one batch of coalesced
// loads); then each wave (one layer row) walks the candidate rows, and each lane the few
// candidate columns whose taps reach its pixel, summing weight x gradient in a fixed order.
__global__ __launch_bounds__(kBlock) void wfs_adjoint_gather_kernel(GatherParams g) {
  __shared__ GTap ct[kGCols];
  __shared__ GTap rt[kGRows];
  __shared__ float gt[kGRows][kGCols];
  __shared__ float tt[kGRows][kGTW];  // column-transposed rows: sum over c of w_c g[r][c]
  __shared__ int rfirst[kGTH];        // first candidate row reaching each tile row
  const FwdParams& p = g.f;
  const int nl = p.n_layers;
  const int per_real = g.blk_start[nl];
  const int b = blockIdx.x / per_real;
  const int rb = blockIdx.x - b * per_real;
  int l = 0;
  while (l + 1 < nl && rb >= g.blk_start[l + 1]) ++l;  // block-uniform
  const DevLayer L = cload(p.lay, l);
  const int tiles_x = (L.nx + kGTW - 1) / kGTW;
  const int tile = rb - g.blk_start[l];
  const int ty0 = (tile / tiles_x) * kGTH, tx0 = (tile - (tile / tiles_x) * tiles_x) * kGTW;
  const int tid = threadIdx.x;
  const int wy = __builtin_amdgcn_readfirstlane(tid / kGTW);  // wave: tile rows wy + 4 k
  const int lx = tid - wy * kGTW;
  const int i = tx0 + lx;
  constexpr int kWavesG = kBlock / kGTW;
  const double stepd = (double)current_step(p);
  const float* gb = g.gpsi + (int64_t)b * p.pupil_per_real;
  float acc[kGPix];
#pragma unroll
  for (int k = 0; k < kGPix; ++k) acc[k] = 0.0f;
  for (int s = 0; s < p.n_sensors; ++s) {
    const DevSensor S = cload(p.sen, s);
    const DevAffine A = cload(p.aff, (int64_t)s * nl + l);
    const double bx = A.bx0 + stepd * A.dbx, by = A.by0 + stepd * A.dby;
    const int npup = S.n_pup;
    const float* gs = gb + S.pupil_off;
    int my_lo, my_hi, mx_lo, mx_hi;
    image_range(A.ay, by, L.ny, L.inv_ny, npup, ty0, ty0 + kGTH - 1, L.boundary, my_lo, my_hi);
    image_range(A.ax, bx, L.nx, L.inv_nx, npup, tx0, tx0 + kGTW - 1, L.boundary, mx_lo, mx_hi);
    for (int my = my_lo; my <= my_hi; ++my) {
      const int64_t yshift = (int64_t)my * L.ny + ty0;
      int r_lo, r_hi;
      cand_range(A.inv_ay, by, (double)yshift, (double)(yshift + kGTH - 1), npup, r_lo, r_hi);
      for (int r0 = r_lo; r0 <= r_hi; r0 += kGRows) {
        const int nr = min(kGRows, r_hi - r0 + 1);
        for (int mx = mx_lo; mx <= mx_hi; ++mx) {
          const int64_t xshift = (int64_t)mx * L.nx + tx0;
          int c_lo, c_hi;
          cand_range(A.inv_ax, bx, (double)xshift, (double)(xshift + kGTW - 1), npup, c_lo,
                     c_hi);
          for (int c0 = c_lo; c0 <= c_hi; c0 += kGPass) {
            const int nc = min(kGPass, c_hi - c0 + 1);
            __syncthreads();  // previous pass done with the tables
            if (tid < nr) rt[tid] = gather_tap(A.ay, A.by0, A.dby, stepd, r0 + tid, yshift);
            if (tid < nc) ct[tid] = gather_tap(A.ax, A.bx0, A.dbx, stepd, c0 + tid, xshift);
            {  // gradient rectangle rows r0.., columns c0.. (kGCols-pitched), loads issued first
              constexpr int kPer = kGRows * kGCols / kBlock, kStep = kBlock / kGCols;
              const int qc = tid & (kGCols - 1), qb = tid / kGCols;
              const uint32_t o0 = (uint32_t)(r0 * npup + c0 + qc);  // < pupil_per_real < 2^31
              float v[kPer];
#pragma unroll
              for (int k = 0; k < kPer; ++k) {
                const int q = qb + k * kStep;
                v[k] = (q < nr && qc < nc) ? ld_idx(gs, o0 + (uint32_t)(q * npup)) : 0.0f;
              }
#pragma unroll
              for (int k = 0; k < kPer; ++k) {
                const int q = qb + k * kStep;
                if (q < nr) gt[q][qc] = v[k];
              }
            }
            __syncthreads();
            // separable transpose, first along columns: T[r][lx] = sum over the candidate
            // columns whose taps reach lx (rel in {lx - 1, lx}, a contiguous run: rel is
            // non-decreasing) of w_c g[r][c]; up to kGC4 of them kept in registers
            int q0 = 0, q1 = nc;
            while (q0 < q1) {
              const int mid = (q0 + q1) >> 1;
              if (ct[mid].rel + 1 < lx) q0 = mid + 1;
              else q1 = mid;
            }
            constexpr int kGC4 = 4;
            int qk[kGC4];
            float wk[kGC4];
            int nk = 0;
            bool more = false;
#pragma unroll
            for (int k = 0; k < kGC4; ++k) {
              qk[k] = kGPass;  // (past the run: zero; a column beside it may hold an infinity)
              wk[k] = 0.0f;
              const int qc = q0 + k;
              if (qc < nc && ct[qc].rel <= lx) {
                const GTap tc = ct[qc];
                qk[k] = qc;
                wk[k] = (tc.rel == lx ? 1.0f - tc.w1 : 0.0f) + (tc.rel + 1 == lx ? tc.w1 : 0.0f);
                nk = k + 1;
              }
            }
            if (nk == kGC4 && q0 + kGC4 < nc && ct[q0 + kGC4].rel <= lx) more = true;
            for (int r = wy; r < nr; r += kWavesG) {
              float t = 0.0f;
#pragma unroll
              for (int k = 0; k < kGC4; ++k) t = fmaf(wk[k], gt[r][qk[k]], t);
              if (more) {  // coarse layer: more than kGC4 pupil columns per layer column
                for (int qc = q0 + kGC4; qc < nc; ++qc) {
                  const GTap tc = ct[qc];
                  if (tc.rel > lx) break;
                  const float wc =
                      (tc.rel == lx ? 1.0f - tc.w1 : 0.0f) + (tc.rel + 1 == lx ? tc.w1 : 0.0f);
                  t = fmaf(wc, gt[r][qc], t);
                }
              }
              tt[r][lx] = t;
            }
            if (tid < kGTH) {  // first candidate row whose taps reach tile row tid
              int r = 0, r1 = nr;
              while (r < r1) {
                const int mid = (r + r1) >> 1;
                if (rt[mid].rel + 1 < tid) r = mid + 1;
                else r1 = mid;
              }
              rfirst[tid] = r;
            }
            __syncthreads();
            // then along rows: G[ry][lx] += sum over the candidate rows reaching ry of w_r T
#pragma unroll
            for (int k = 0; k < kGPix; ++k) {
              const int ry = wy + k * kWavesG;  // wave-uniform
              for (int rr = rfirst[ry]; rr < nr; ++rr) {
                const GTap tr = rt[rr];
                if (tr.rel > ry) break;
                const float wr =
                    (tr.rel == ry ? 1.0f - tr.w1 : 0.0f) + (tr.rel + 1 == ry ? tr.w1 : 0.0f);
                acc[k] = fmaf(wr, tt[rr][lx], acc[k]);
              }
            }
          }
        }
      }
    }
  }
  if (i < L.nx) {
#pragma unroll
    for (int k = 0; k < kGPix; ++k) {
      const int j = ty0 + wy + k * kWavesG;
      if (j < L.ny)
        g.grad[(int64_t)b * p.layer_stride + L.offset + (int64_t)j * L.nx + i] =
            acc[k] * L.weight;
    }
  }
}

// ---------------------------------------------------------------------------------------
// Table-driven gather (layers whose inverse stencil lists are short: pupil and layer pitches
// within a factor of about two, one periodic image per layer pixel).
//
// Taps kernel, thread per (segment, index i), from the same FP64 coordinate and make_tap as the
// projection, bit for bit.  Column segments: the pupil columns whose forward taps touch layer
// column i, in increasing order, with the weight i has in their stencil.  Row segments: the
// pupil rows whose first tap row is i - 1 (a zero boundary's taps -1 .. ny - 1; a periodic
// one's last row is also its row -1), at most two as the pupil rows lie more than half a layer
// row apart, with both weights.  Candidates: for every periodic image m, the indices whose
// coordinate lies in [i - 1 + m n, i + 1 + m n), with a margin of one index.
// ---------------------------------------------------------------------------------------
constexpr int kG2R = 16;  // layer rows of a wave
constexpr int kG2TH = kG2R * kWavesPerBlock;

// Entry of the row table, base = entry - 1: the byte offset of the first pupil row in the
// sensor's image, the bytes to the second, and their weights on layer rows base (w0) and base +
// 1 (w1).  A single row stands for both with half of its weights, so the gather has no branch
// for it; n = 0: no row (offsets 0, not used).
struct RowEnt {
  int32_t off_lo, off_hi, step, n;
  float w0a, w1a, w0b, w1b;
};
static_assert(sizeof(RowEnt) == 4 * sizeof(int2), "row entries fill whole int2 entries");

__host__ __device__ inline int row_ents(int ny) { return (ny + kG2R - 1) / kG2R * kG2R + 2; }

// The table entries (int2) and threads of a (sensor, layer)'s row segment.
int adj_row_ents(int ny) { return row_ents(ny); }
int64_t adj_row_int2(int ny) { return (int64_t)row_ents(ny) * (sizeof(RowEnt) / sizeof(int2)); }

__global__ __launch_bounds__(kBlock) void wfs_adjoint_taps_kernel(GatherTabParams g) {
  const FwdParams& p = g.f;
  const AdjSeg sg = g.segs[blockIdx.y];
  int i = blockIdx.x * kBlock + threadIdx.x;
  const bool ax = sg.axis == 0;
  if (i >= (ax ? sg.n : row_ents(sg.n))) return;
  const DevLayer L = p.lay[sg.l];
  const DevAffine A = p.aff[(int64_t)sg.s * p.n_layers + sg.l];
  const int npup = p.sen[sg.s].n_pup;
  const double stepd = (double)current_step(p);
  const double a = ax ? A.ax : A.ay, b0 = ax ? A.bx0 : A.by0, db = ax ? A.dbx : A.dby;
  const double inv_a = ax ? A.inv_ax : A.inv_ay;
  const int32_t n = ax ? L.nx : L.ny;
  const double inv_n = ax ? L.inv_nx : L.inv_ny;
  const double b = b0 + stepd * db;
  RowEnt* const row_dst = reinterpret_cast<RowEnt*>(g.tab + sg.off) + i;
  if (!ax) {
    i = i == 0 ? (L.boundary == 0 ? n - 1 : -1) : i - 1;
    if (i >= n) {
      *row_dst = RowEnt{};
      return;
    }
  }
  int m_lo, m_hi;
  image_range(a, b, n, inv_n, npup, i, i, L.boundary, m_lo, m_hi);
  int2 out[kAdjKI];
#pragma unroll
  for (int k = 0; k < kAdjKI; ++k) out[k] = make_int2(-1, 0);
  RowEnt re{};
  int cnt = 0;
  for (int m = m_lo; m <= m_hi; ++m) {
    int lo, hi;
    const double base = (double)i + (double)m * (double)n;
    cand_range(inv_a, b, base, base, npup, lo, hi);
    for (int c = lo; c <= hi; ++c) {
      const double w = fma(a, (double)c, b0) + stepd * db;
      const Tap t = make_tap(w, n, inv_n, L.boundary, 1);
      if (!ax) {
        if ((L.boundary == 0 ? t.i0 : (int)floor(w)) != i || re.n == 2) continue;
        if (re.n == 0) {
          const int64_t off = 4 * (int64_t)c * npup;
          re.off_lo = (int32_t)(uint32_t)off;
          re.off_hi = (int32_t)(off >> 32);
          re.w0a = re.w0b = 0.5f * t.w0;
          re.w1a = re.w1b = 0.5f * t.w1;
        } else {
          re.step = 4 * npup;
          re.w0a *= 2.0f;
          re.w1a *= 2.0f;
          re.w0b = t.w0;
          re.w1b = t.w1;
        }
        ++re.n;
        continue;
      }
      const float wt = (t.i0 == i ? t.w0 : 0.0f) + (t.i1 == i ? t.w1 : 0.0f);
      if (wt != 0.0f && cnt < kAdjKI) {
#pragma unroll
        for (int k = 0; k < kAdjKI; ++k)
          if (k == cnt) out[k] = make_int2(c, __float_as_int(wt));
        ++cnt;
      }
    }
  }
  if (!ax) {
    *row_dst = re;
    return;
  }
  int2* dst = g.tab + sg.off + (int64_t)i * kAdjKI;
#pragma unroll
  for (int k = 0; k < kAdjKI; ++k) dst[k] = out[k];
}

// Gather kernel for tabled layers (one periodic image per layer pixel: for every sensor the
// pupil columns of one layer column are consecutive).  Block = (realisation, tabled layer,
// 64 x 64 tile); wave = 64 layer columns (one per lane) x kG2R rows, accumulated in registers.
// For every sensor in order the pupil rows are summed into the wave's layer rows first, lane =
// pupil column, and the columns of each lane's list then, through LDS: fixed order of every
// sum, bitwise deterministic.
//
// Bound by vector issue and latency (six 80 x 80 LGS and ten 1024^2 layers: 15 MB read, 42 MB
// written, 12 us at the copy rate).  Loading each lane's own columns from memory took 120 us
// however the sums were organised: 64 lanes whose addresses are not strictly consecutive go
// through the cache a quad a cycle, 16 cycles a load instead of 4.  Loading the rows as they lie
// and picking columns from LDS, with row taps from scalar loads: 53 us.

constexpr int kG2Cols = 2 * kWave;  // pupil columns of a window

// One sensor's rows over a window of pupil columns, lane holding columns col[0] and col[1]
// (window positions lane and lane + 64).  Its first tap rows -1 .. kG2R - 1 go by in pairs, the
// pupil rows of the next pair in flight while one is summed into the layer rows (over the
// window's columns), their entries a pair further ahead.  Every four finished layer rows pass
// through LDS, where a lane reads its NC columns from their positions.
template <int NC>
__device__ __forceinline__ void gather_rows(const float* gs, const RowEnt* ents,
                                            const uint32_t (&col)[2], int lane,
                                            const int (&at)[kAdjKI],
                                            const float (&wc)[kAdjKI], float4* buf,
                                            float (&acc)[kG2R]) {
  constexpr int CH = 2, NG = (kG2R + CH) / CH;
  struct Ents {
    RowEnt e[CH];
  };
  const Ents* eg = reinterpret_cast<const Ents*>(ents);
  Ents es[3];
  float v[2][CH][2][2], r[kG2R + 2][2];
  auto load = [&](auto g) __attribute__((always_inline)) {
    // (opaque: a 32-bit lane offset seen here goes with a scalar base into the load)
    uint32_t c[2] = {col[0], col[1]};
    asm("" : "+v"(c[0]), "+v"(c[1]));
    static_for<CH>([&](auto k) __attribute__((always_inline)) {
      const RowEnt& e = es[g % 3].e[k];
      const char* ga = reinterpret_cast<const char*>(gs) +
                       (int64_t)(((uint64_t)(uint32_t)e.off_hi << 32) | (uint32_t)e.off_lo);
      const char* gb = ga + (uint32_t)e.step;
      static_for<2>([&](auto h) __attribute__((always_inline)) {
        v[g & 1][k][0][h] = ld_idx(reinterpret_cast<const float*>(ga), c[h]);
        v[g & 1][k][1][h] = ld_idx(reinterpret_cast<const float*>(gb), c[h]);
      });
    });
  };
  es[0] = cload(eg, 0);
  es[1] = cload(eg, 1);
  load(std::integral_constant<int, 0>{});
  r[1][0] = r[1][1] = 0.0f;
  static_for<NG>([&](auto g) __attribute__((always_inline)) {
    if constexpr (g + 1 < NG) load(std::integral_constant<int, g + 1>{});
    if constexpr (g + 2 < NG) es[(g + 2) % 3] = cload(eg, g + 2);
    __builtin_amdgcn_sched_barrier(0);
    static_for<CH>([&](auto k) __attribute__((always_inline)) {
      constexpr int row = g * CH + k;  // r[row]: layer row y0 + row - 1
      if constexpr (row <= kG2R) {
        const RowEnt& e = es[g % 3].e[k];
        static_for<2>([&](auto h) __attribute__((always_inline)) {
          // (not a weight of zero where there is no row: the one read may hold an infinity)
          const float a = e.n ? v[g & 1][k][0][h] : 0.0f, b = e.n ? v[g & 1][k][1][h] : 0.0f;
          if constexpr (row > 0) r[row][h] = fmaf(e.w0b, b, fmaf(e.w0a, a, r[row][h]));
          r[row + 1][h] = fmaf(e.w1b, b, e.w1a * a);
        });
        if constexpr (row > 0 && row % 4 == 0) {
          buf[lane] = make_float4(r[row - 3][0], r[row - 2][0], r[row - 1][0], r[row][0]);
          buf[lane + kWave] = make_float4(r[row - 3][1], r[row - 2][1], r[row - 1][1], r[row][1]);
          wave_sync();
          float4 x[NC];
          static_for<NC>([&](auto q) __attribute__((always_inline)) { x[q] = buf[at[q]]; });
          static_for<NC>([&](auto q) __attribute__((always_inline)) {
            acc[row - 4] = fmaf(wc[q], x[q].x, acc[row - 4]);
            acc[row - 3] = fmaf(wc[q], x[q].y, acc[row - 3]);
            acc[row - 2] = fmaf(wc[q], x[q].z, acc[row - 2]);
            acc[row - 1] = fmaf(wc[q], x[q].w, acc[row - 1]);
          });
          wave_sync();
        }
      }
    });
    __builtin_amdgcn_sched_barrier(0);
  });
}

__global__ __launch_bounds__(kBlock) void wfs_adjoint_gather_tab_kernel(GatherTabParams g) {
  __shared__ float4 buf_s[kWavesPerBlock][kG2Cols + 1];  // (the last: zero)
  const FwdParams& p = g.f;
  const int nl = p.n_layers;
  const int per_real = g.blk_start[nl];
  const int b = blockIdx.x / per_real;
  const int rb = blockIdx.x - b * per_real;
  int l = 0;
  while (l + 1 < nl && rb >= g.blk_start[l + 1]) ++l;  // block-uniform
  const DevLayer L = cload(p.lay, l);
  const int tiles_x = (L.nx + kWave - 1) / kWave;
  const int tile = rb - g.blk_start[l];
  const int tyi = tile / tiles_x;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & (kWave - 1);
  const int x = (tile - tyi * tiles_x) * kWave + lane;
  const int y0 = tyi * kG2TH + wave * kG2R;
  const int nrows = min(kG2R, L.ny - y0);  // wave-uniform, may be <= 0
  if (nrows <= 0) return;                  // no block-wide barrier below
  const bool xin = x < L.nx;
  float4* buf = buf_s[wave];
  if (lane == 0) buf[kG2Cols] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  float acc[kG2R];
  static_for<kG2R>([&](auto yy) __attribute__((always_inline)) { acc[yy] = 0.0f; });
  const float* gb = g.gpsi + (int64_t)b * p.pupil_per_real;
  const int xl = xin ? x : 0;
  // of a sensor: the lane's column list (consecutive pupil columns from its first entry, with
  // their weights, 0 past the list's end), the number of pupil rows of the wave's first tap
  // row -1 + lane, where its row entries and its image are; loaded while the sensor before it
  // is summed
  int2 ce[kAdjKI];
  int en, npup;
  const RowEnt* ents;
  const float* gs;
  auto fetch = [&](int s) __attribute__((always_inline)) {
    const int2* e0 = g.tab + cload(g.tab_off, (int64_t)s * nl + l);
#pragma unroll
    for (int k = 0; k < kAdjKI; ++k) ce[k] = e0[(int64_t)xl * kAdjKI + k];
    ents = reinterpret_cast<const RowEnt*>(e0 + (int64_t)L.nx * kAdjKI) + y0;
    en = ents[min(lane, kG2R)].n;
    const DevSensor S = cload(p.sen, s);
    gs = gb + S.pupil_off;
    npup = S.n_pup;
  };
  fetch(0);
  for (int s = 0; s < p.n_sensors; ++s) {
    float wc[kAdjKI];
    int cf = 0, ncol = 0;
#pragma unroll
    for (int k = 0; k < kAdjKI; ++k) {
      const bool ok = xin && ce[k].x >= 0;
      if (k == 0) cf = ok ? ce[k].x : 0;
      wc[k] = ok ? __int_as_float(ce[k].y) : 0.0f;
      if (__builtin_amdgcn_ballot_w64(ok) != 0) ncol = k + 1;  // wave-uniform
    }
    if (__builtin_amdgcn_ballot_w64(en != 0) == 0) ncol = 0;
    const RowEnt* const ents_s = ents;
    const float* const gs_s = gs;
    const int npup_s = npup;
    if (s + 1 < p.n_sensors) fetch(s + 1);
    if (ncol == 0) continue;  // wave-uniform: no contribution
    // windows of pupil columns from the first lane's that is not done: one, or two where the
    // wave's columns hold both ends of a periodic footprint (the columns increase but there;
    // 64 layer columns touch fewer than 64 * 3 / 2 + 4 pupil columns)
    uint64_t left = __builtin_amdgcn_ballot_w64(wc[0] != 0.0f);
    while (left != 0) {
      const int c0 = __builtin_amdgcn_readlane(cf, __builtin_ctzll(left));
      const bool part = ((left >> lane) & 1) && cf >= c0 && cf + ncol <= c0 + kG2Cols;
      left &= ~__builtin_amdgcn_ballot_w64(part);
      int at[kAdjKI];  // past the lane's list: zero (a column beside it may hold an infinity)
#pragma unroll
      for (int k = 0; k < kAdjKI; ++k) at[k] = part && wc[k] != 0.0f ? cf - c0 + k : kG2Cols;
      const uint32_t col[2] = {(uint32_t)min(c0 + lane, npup_s - 1),
                               (uint32_t)min(c0 + kWave + lane, npup_s - 1)};
      if (ncol == 1)
        gather_rows<1>(gs_s, ents_s, col, lane, at, wc, buf, acc);
      else if (ncol == 2)
        gather_rows<2>(gs_s, ents_s, col, lane, at, wc, buf, acc);
      else if (ncol == 3)
        gather_rows<3>(gs_s, ents_s, col, lane, at, wc, buf, acc);
      else
        gather_rows<4>(gs_s, ents_s, col, lane, at, wc, buf, acc);
    }
  }
  if (xin) {
    float* out = g.grad + (int64_t)b * p.layer_stride + L.offset + x;
    static_for<kG2R>([&](auto yy) __attribute__((always_inline)) {
      if (yy < nrows) out[(int64_t)(y0 + yy) * L.nx] = acc[yy] * L.weight;
    });
  }
}

__global__ __launch_bounds__(kBlock) void zero_kernel(float* x, int64_t n) {
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) x[i] = 0.0f;
}

hipError_t launch_zero(float* x, int64_t n, hipStream_t st) {
  const int zb = (int)std::min<int64_t>((n + kBlock - 1) / kBlock, 8192);
  hipLaunchKernelGGL(zero_kernel, dim3(zb > 0 ? zb : 1), dim3(kBlock), 0, st, x, n);
  return hipGetLastError();
}

template <int NS>
static hipError_t launch_adj(AdjParams a, bool clear_grad, bool clear, hipStream_t st) {
  // atomic mode accumulates into the gradient (gather mode writes every pixel of a valid
  // subaperture of its images; the others stay zero from their allocation)
  hipError_t e = hipSuccess;
  if (clear && !a.gpsi) {
    e = launch_zero(a.grad_layers, a.f.layer_stride * a.f.batch, st);
    if (e != hipSuccess) return e;
  }
  // the gather writes every grid pixel; the rest of the gradient buffer (gaps between the
  // grids inside the stride) is cleared only when there is such a gap
  if (clear && a.gpsi && clear_grad) {
    e = launch_zero(a.grad_layers, a.f.layer_stride * a.f.batch, st);
    if (e != hipSuccess) return e;
  }
  const int64_t tasks = (int64_t)a.f.otf.per_real * a.f.batch;
  if (tasks == 0) return hipSuccess;
  const int64_t waves = tasks;
  const int grid = (int)((waves + kWavesPerBlock - 1) / kWavesPerBlock);
  if (a.f.otf_from_phase)
    hipLaunchKernelGGL((wfs_adjoint_kernel<NS, false>), dim3(grid), dim3(kBlock),
                       a.f.lds_per_wave * kWavesPerBlock, st, a);
  else
    hipLaunchKernelGGL((wfs_adjoint_kernel<NS, true>), dim3(grid), dim3(kBlock),
                       a.f.lds_per_wave * kWavesPerBlock, st, a);
  return hipGetLastError();
}

int adj_lds_bytes(int ns, int n_layers, int n_pix, bool gather) {
  return adj_lds_layout(ns, n_layers, n_pix, gather).total;
}

hipError_t launch_adjoint_gather(const FwdParams& f, const float* gpsi, float* grad,
                                 const int32_t* blk_start, hipStream_t st) {
  GatherParams g;
  g.f = f;
  g.gpsi = gpsi;
  g.grad = grad;
  for (int l = 0; l <= f.n_layers; ++l) g.blk_start[l] = blk_start[l];
  const int64_t blocks = (int64_t)blk_start[f.n_layers] * f.batch;
  if (blocks == 0) return hipSuccess;
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL(wfs_adjoint_gather_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, st, g);
  return hipGetLastError();
}

hipError_t launch_adjoint_gather_tab(const FwdParams& f, const float* gpsi, float* grad,
                                     int2* tab, const AdjSeg* segs, int n_segs, int max_n,
                                     const int64_t* tab_off, const int32_t* blk_start,
                                     hipStream_t st) {
  if (n_segs == 0) return hipSuccess;
  GatherTabParams g;
  g.f = f;
  g.gpsi = gpsi;
  g.grad = grad;
  g.tab = tab;
  g.segs = segs;
  g.tab_off = tab_off;
  for (int l = 0; l <= f.n_layers; ++l) g.blk_start[l] = blk_start[l];
  hipLaunchKernelGGL(wfs_adjoint_taps_kernel, dim3((max_n + kBlock - 1) / kBlock, n_segs),
                     dim3(kBlock), 0, st, g);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int64_t blocks = (int64_t)blk_start[f.n_layers] * f.batch;
  if (blocks == 0) return hipSuccess;
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL(wfs_adjoint_gather_tab_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, st,
                     g);
  return hipGetLastError();
}

int adj_tab_rows() { return kG2TH; }

// FFT-path sensors: one wave per spectrum chunk (fft_adjoint_chunk_m), before the gather
__global__ __launch_bounds__(kBlock) void wfs_adjoint_fft_kernel(AdjParams ap, int lds_per_wave) {
  extern __shared__ __align__(16) char smem[];
  const int w = threadIdx.x >> 6;
  fft_adjoint_wave(ap, blockIdx.x * kWavesPerBlock + w, smem + w * lds_per_wave);
}

int fft_adj_wave_lds_bytes(int n_fft, int n_pix) { return fft_adj_wave_lds_bytes_impl(n_fft, n_pix); }

hipError_t launch_adjoint_fft(const AdjParams& a, int lds_per_wave, hipStream_t st) {
  const int64_t tasks = (int64_t)a.f.fft.per_real * a.f.batch;
  if (tasks == 0) return hipSuccess;
  const int64_t blocks = (tasks + kWavesPerBlock - 1) / kWavesPerBlock;
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL(wfs_adjoint_fft_kernel, dim3((unsigned)blocks), dim3(kBlock),
                     lds_per_wave * kWavesPerBlock, st, a, lds_per_wave);
  return hipGetLastError();
}

hipError_t launch_adjoint(const AdjParams& a, int ns, bool clear_grad, bool clear,
                          hipStream_t st) {
  switch (ns) {
    case 2: return launch_adj<2>(a, clear_grad, clear, st);
    case 3: return launch_adj<3>(a, clear_grad, clear, st);
    case 4: return launch_adj<4>(a, clear_grad, clear, st);
    case 5: return launch_adj<5>(a, clear_grad, clear, st);
    case 6: return launch_adj<6>(a, clear_grad, clear, st);
    case 7: return launch_adj<7>(a, clear_grad, clear, st);
    case 8: return launch_adj<8>(a, clear_grad, clear, st);
    case 9: return launch_adj<9>(a, clear_grad, clear, st);
    case 10: return launch_adj<10>(a, clear_grad, clear, st);
    case 11: return launch_adj<11>(a, clear_grad, clear, st);
    case 12: return launch_adj<12>(a, clear_grad, clear, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace wfs
