// Lag-domain ("OTF") path of the Shack-Hartmann spot model: device functions shared by the
// forward and adjoint kernels.  One 64-lane wavefront handles one subaperture at a time.
//
// The paper's sensor turns the residual phase into X/Y slopes
// (Sec. 2.7); our reading forms the spot as |DFT_N(E)|^2 of the zero-padded subaperture field,
// convolves it with the sodium-profile kernel, shifts, bins and takes the centre of gravity.
// Because the field has n_sub x n_sub support and N >= 2 n_sub, the DFT of the spot is
// exactly c N^2 times the field's autocorrelation A[k] = sum_m E[m] conj(E[m+k]) on the
// (2 n_sub - 1)^2 lags, and binning after the fftshift is, in the Fourier domain, a
// multiplication by s(kx) s(ky) (s(k) = (-1)^k sum_{d<b} e^{2 pi i k d / N}) followed by
// folding the lags modulo n_pix.  So the binned image is
//     B[q] = c Re sum_{K} P[K] e^{2 pi i K.q / n_pix},
//     P[K] = sum_{k = K mod n_pix, half plane} w_k A[k] Kel[k] s(kx) s(ky),
// (w = 1 on the ky = 0 row, 2 above it, using A[-k] = conj A[k]): no N x N array at all.
// The autocorrelation itself runs through a short DFT of each field row (otf_corr).
// The result equals the FFT definition up to rounding; the FP64 oracle checks it.
#pragma once

#include "wfs_common.h"
#include "wfs_project.h"

namespace wfs {

// ------------------------------------------------------------------------------------------
// Lag-domain path
// ------------------------------------------------------------------------------------------

// Sizes of the autocorrelation stage of one subaperture (otf_corr): DFTs of F = 4 Q >=
// 2 n_sub - 1 points, so that no lag wraps around.
__host__ __device__ constexpr int otf_q(int ns) { return (2 * ns + 2) / 4; }
// Lane groups that share the row products of one frequency: groups of 16 or 32 lanes.
__host__ __device__ constexpr int otf_groups(int ns) { return 4 * otf_q(ns) <= 16 ? 4 : 2; }
// Rows of the row transforms: the field's, and zero rows for the groups' row offsets.
__host__ __device__ constexpr int otf_rows(int ns) { return ns + otf_groups(ns) - 1; }
// Row pitch (float2) of the row products: even (16-byte loads), and rows on different banks.
__host__ __device__ constexpr int otf_c_pitch(int ns) { return 4 * otf_q(ns) + 2; }

template <int NS>
struct Otf {
  static constexpr int kLags = 2 * NS - 1;       // dx = -(NS-1) .. NS-1
  static constexpr int kQ = otf_q(NS);
  static constexpr int kF = 4 * kQ;              // DFT points of one field row
  static constexpr int kGroups = otf_groups(NS);
  static constexpr int kRows = otf_rows(NS);
  static constexpr int kCP = otf_c_pitch(NS);
  static constexpr int kAP = kF;                 // row pitch (float2) of the lag array
};

// Twiddles of otf_corr, one row of kOtfTw float2 per residue k0 < Q: exp(-2 pi i m k0 / Q),
// m = 1 .. 5, then exp(-2 pi i s k0 / F), s = 1 .. 3.
constexpr int kOtfTw = 8;
__host__ __device__ constexpr int otf_twiddles(int ns) { return otf_q(ns) * kOtfTw; }

// Per-wave LDS layout (bytes), shared with the host sizing code:
//   E [n_sub][n_sub] float2 |
//   union( taps [n_layers][2 n_sub] Tap (fused gather and adjoint only),
//          row transforms G [4][rows][Q] float2, then row products C [n_sub][pitch] float2
//          over them, lags AW [n_sub][F] float2 behind C, then P (later B) + Z over C ) |
//   tables: twiddles of otf_corr [Q][kOtfTw] float2, s(k) [2 n_sub - 1] float2, image
//           twiddles [n_pix] float2
// With a staged footprint (foot_floats > 0) the field stage also lays out, from offset 0
// (E, the union and the tables are free until the field is formed): stencil entries
// [n_layers][2 n_sub] FootTap (12 bytes) | the footprint [foot_floats] float (first holding
// the window origins, [n_layers][2] int).  The tables are then copied in after the window
// has been read.
struct OtfLds {
  int e_off, tw_off, stab_off, wtab_off, aw_off, taps_off, g_off, c_off, p_off, z_off, b_off;
  int fw_off, fp_off, total;
};

__host__ __device__ inline OtfLds otf_lds_layout(int ns, int n_layers, int n_pix,
                                                 bool with_taps = true, int foot_floats = 0) {
  OtfLds o;
  const int lags = 2 * ns - 1, np2 = n_pix * n_pix;
  o.e_off = 0;
  const int u0 = (ns * ns * 8 + 15) & ~15;
  const int taps = 2 * ns * n_layers * 16;
  const int g = 4 * otf_rows(ns) * otf_q(ns) * 8;
  const int c = ns * otf_c_pitch(ns) * 8;
  o.taps_off = u0;
  o.g_off = u0;
  o.c_off = u0;
  o.p_off = u0;  // the fold reads the lags and writes P: they do not meet
  o.z_off = o.p_off + np2 * 8;
  o.b_off = o.p_off;  // B overwrites P: the image's second pass reads only Z
  o.aw_off = u0 + (c > np2 * 8 ? c : np2 * 8);
  int end = o.z_off + np2 * 8;
  if (o.p_off + 1024 > end) end = o.p_off + 1024;  // matrix-core image: 16 x 16 floats
  if (u0 + g > end) end = u0 + g;
  if (o.aw_off + ns * 4 * otf_q(ns) * 8 > end) end = o.aw_off + ns * 4 * otf_q(ns) * 8;
  if (with_taps && u0 + taps > end) end = u0 + taps;
  o.tw_off = (end + 15) & ~15;
  o.stab_off = o.tw_off + otf_twiddles(ns) * 8;
  o.wtab_off = o.stab_off + lags * 8;
  end = o.wtab_off + n_pix * 8;
  o.fw_off = 0;
  o.fp_off = (2 * ns * n_layers * 12 + 15) & ~15;
  const int fpb = 4 * (foot_floats > 2 * n_layers ? foot_floats : 2 * n_layers);
  if (foot_floats > 0 && o.fp_off + fpb > end) end = o.fp_off + fpb;
  o.total = (end + 15) & ~15;
  return o;
}

// q / D for 0 <= q D < 2^16 (full-rate 24-bit multiply)
template <int D>
__device__ __forceinline__ int small_div(int q) {
  return (int)(((uint32_t)q * (uint32_t)((65536 + D - 1) / D)) >> 16);
}

// Tap of a given layer for the lanes of one half-wave: the layer parameters are wave-uniform
// (scalar loads), two layers per pass (lanes 0-31 and 32-63).
__device__ __forceinline__ Tap tap_of(const DevLayer& L, const DevAffine& A, bool row, int idx,
                                      double stepd) {
  if (!row) {
    const double u = fma(A.ax, (double)idx, A.bx0) + stepd * A.dbx;
    return make_tap(u, L.nx, L.inv_nx, L.boundary, 1);
  }
  const double v = fma(A.ay, (double)idx, A.by0) + stepd * A.dby;
  return make_tap(v, L.ny, L.inv_ny, L.boundary, L.nx);
}

// Sodium-profile entry of the frame at time step `step` (wave-uniform): its first peak and the
// peak count, or no peaks when the plan has no profile table (single Gaussians).
struct NaEntry {
  const float4* pk;
  int n;
};

__device__ __forceinline__ NaEntry na_entry(const FwdParams& p, int64_t step) {
  NaEntry e;
  e.n = 0;
  e.pk = nullptr;
  if (p.na_entries > 0) {
    const int64_t k = step % (int64_t)p.na_entries;
    e.pk = p.na_tab + (k < 0 ? k + p.na_entries : k) * p.na_peaks;
    e.n = p.na_peaks;
  }
  return e;
}

// Sodium transfer function at the lag whose projection on the elongation direction is `proj`
// (lag units), times `scale`: the subaperture's single Gaussian exp(-alpha proj^2), or, with
// a profile entry, sum_j w_j exp(-2 pi^2 sigma_j^2 t^2) e^{-2 pi i dh_j t}, t = gam proj
// (peak j widened by gam sigma_j and shifted by gam dh_j FFT pixels per unit lag, Sec. 2.7).
__device__ __forceinline__ float2 elong_tf(const DevSubap& sb, const NaEntry& el, float proj,
                                           float scale) {
  if (el.n == 0 || sb.gam == 0.0f)
    return make_float2(__expf(-sb.alpha * proj * proj) * scale, 0.0f);
  const float t = sb.gam * proj;
  float kr = 0.0f, ki = 0.0f;
  for (int j = 0; j < el.n; ++j) {
    const float4 q = el.pk[j];  // (2 pi^2 sigma_h^2, dh, w, 0)
    const float m = q.z * __expf(-q.x * t * t);
    float turns = q.y * t;
    turns -= rintf(turns);
    float sn, cs;
    sincos_rev(turns, &sn, &cs);
    kr = fmaf(m, cs, kr);
    ki = fmaf(-m, sn, ki);
  }
  return make_float2(kr * scale, ki * scale);
}

// Phase in turns subtracted at local pixel (row r, column c) of a subaperture: the half-pixel
// centring ramp and the sensor's tip-tilt (both linear in the pixel index).
__device__ __forceinline__ float field_ramp(const DevSensor& S, int r, int c) {
  return fmaf((float)c, S.ramp_x, (float)r * S.ramp_y);
}

// The wave's copies of the small tables (twiddles of otf_corr, lag phases s(k), image
// twiddles: consecutive in the LDS layout) and the pupil amplitude of the lane's pixels.  They
// are loaded at the start, so that their latency passes under the field's own loads, and
// stored once the field stage leaves their LDS free.
template <int NS>
struct OtfTables {
  static constexpr int kPPL = (NS * NS + kWave - 1) / kWave;  // pixels per lane
  static constexpr int kFixed = otf_twiddles(NS) + 2 * NS - 1;
  static constexpr int kPre = kFixed + 8 > kWave ? 2 : 1;     // entries per lane held early
  float2 t[kPre];
  uint8_t amp[kPPL];

  __device__ __forceinline__ float2 entry(const FwdParams& p, const DevSensor& S, int k) const {
    if (k < otf_twiddles(NS)) return p.otf_tw[k];
    if (k < kFixed) return p.stab[S.stab_off + k - otf_twiddles(NS)];
    return k < kFixed + S.n_pix ? p.wtab[S.wtab_off + k - kFixed] : make_float2(0.0f, 0.0f);
  }
  __device__ __forceinline__ void load(const FwdParams& p, const DevSensor& S,
                                       const DevSubap& sb) {
    const int lane = lane_id();
#pragma unroll
    for (int i = 0; i < kPre; ++i) t[i] = entry(p, S, lane + i * kWave);
#pragma unroll
    for (int i = 0; i < kPPL; ++i) {
      const int q = min(lane + i * kWave, NS * NS - 1), r = small_div<NS>(q), c = q - r * NS;
      amp[i] = p.mask[S.mask_off + (sb.a * NS + r) * S.n_pup + sb.b * NS + c];
    }
  }
  __device__ __forceinline__ void store(const FwdParams& p, const DevSensor& S, char* wsm,
                                        const OtfLds& lo) const {
    float2* d = reinterpret_cast<float2*>(wsm + lo.tw_off);
    const int lane = lane_id(), n = kFixed + S.n_pix;
#pragma unroll
    for (int i = 0; i < kPre; ++i)
      if (lane + i * kWave < n) d[lane + i * kWave] = t[i];
    for (int k = lane + kPre * kWave; k < n; k += kWave) d[k] = entry(p, S, k);
  }
};

// Where the lag-domain field stage gets the phase (a compile-time choice, so that each kernel
// only holds the registers of its own path).
constexpr int kFieldGather = 0;  // bilinear stencils straight from the layers, per pixel
constexpr int kFieldPhase = 1;   // the projection kernel's phase buffer p.phase_in
constexpr int kFieldFoot = 2;    // the subaperture's layer footprint, staged in LDS

// One axis of a bilinear stencil for the staged footprint: the weights of make_tap (same
// arithmetic, bit for bit) and the first tap's grid index, wrapped into [0, n) on a periodic
// grid, the floor of the clamped coordinate on a zero-boundary grid.  The window of a
// subaperture starts at the index of its pupil pixel with the smaller coordinate.
__device__ __forceinline__ float2 foot_axis_tap(double c, int32_t n, double inv_n,
                                                int32_t boundary, int* i0_out) {
  if (boundary == 0) {
    const double cw = c - (double)n * floor(c * inv_n);
    const double f0 = floor(cw);
    int32_t i0 = (int32_t)f0;
    const float f = (float)(cw - f0);
    if (i0 >= n) i0 -= n;
    if (i0 < 0) i0 += n;
    *i0_out = i0;
    return make_float2(1.0f - f, f);
  }
  const double cc = fmin(fmax(c, -4.0), (double)n + 4.0);
  const double f0 = floor(cc);
  const int32_t i0 = (int32_t)f0;
  const float f = (float)(cc - f0);
  const bool ok0 = i0 >= 0 && i0 < n;
  const bool ok1 = i0 + 1 >= 0 && i0 + 1 < n;
  *i0_out = i0;
  return make_float2(ok0 ? 1.0f - f : 0.0f, ok1 ? f : 0.0f);
}

// Stencil entry of one pupil column (w0, w1, byte offset of the window-relative column) or
// row (w0 * layer weight, w1 * layer weight, byte offset of the window row) of one layer.
struct FootTap {
  float w0, w1;
  int32_t k;
};

// Phase of the lane's pixels from a footprint staged in LDS (Sec. 2.2, inside the spot wave):
//   1. the origin of each layer window along each axis (the window holds the layer pixels the
//      subaperture's stencils can touch; bounds fixed per sensor and layer), then every
//      stencil entry (lane per layer, axis and pupil index), both from the launch's table of
//      stencil entries (FP64 coordinates, computed once per frame for every pupil index);
//   2. each lane loads up to two window columns (all rows; the column descriptors are read
//      at the start), then the window goes to LDS over the origins table;
//   3. each pixel sums its stencils from LDS, layer by layer.
// Indices, weights and the order of every floating-point operation are those of the
// projection kernel, so the phase (and everything after it) matches the split schedule bit
// for bit.
template <int NS, class PK>
__device__ __forceinline__ void foot_phase(const FwdParams& p, const DevSensor& S,
                                           const DevSubap& sb, int b, int frame, char* wsm,
                                           const OtfLds& lo, const PK& pk, float* ph) {
  constexpr int NPIX = NS * NS;
  constexpr int PPL = (NPIX + kWave - 1) / kWave;
  constexpr int ROWS = NS + 2;                   // window rows loaded per column
  constexpr int SLOT = ROWS | 1;                 // LDS floats per window column (odd)
  constexpr int TPL = 2 * NS;       // stencil entries per layer: columns, then rows
  constexpr int LPP = kWave / TPL;  // layers per pass
  const int lane = lane_id();
  const int nl = p.n_layers;
  FootTap* tab = reinterpret_cast<FootTap*>(wsm + lo.fw_off);  // [nl][2 NS]
  int* forg = reinterpret_cast<int*>(wsm + lo.fp_off);         // [nl][2], until step 2
  float* fp = reinterpret_cast<float*>(wsm + lo.fp_off);
  FootCol fc[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int pc = lane + k * kWave;
    fc[k] = pc < S.foot_ncols ? p.foot_cols[S.foot_cols_off + pc]
                              : FootCol{0, 1, 1, 0, 0, 0, 0, 0};
  }
  // 1. window origins, lane per (layer, axis): the first tap of the pupil index with the
  //    smaller coordinate (the first one: coordinates grow with the index); then the stencil
  //    entries, lane per (layer, axis, pupil index), from the launch's entry table of this
  //    frame.  Everything is loaded before anything is stored: one memory round trip.
  const FootEnt* ent =
      p.foot_ent + (int64_t)frame * p.foot_ent_per_frame + S.foot_ent_off;  // [nl][2][n_pup]
  {
    int org = 0;
    if (lane < 2 * nl) org = ent[lane * S.n_pup + ((lane & 1) ? sb.a * NS : sb.b * NS)].i0;
    const int lp = small_div<TPL>(lane), j = lane - lp * TPL;
    const int axis = j >= NS ? 1 : 0;
    const int idx = axis ? sb.a * NS + (j - NS) : sb.b * NS + j;
    constexpr int kB = 4;  // passes in flight
    for (int l0 = 0; l0 < nl; l0 += kB * LPP) {
      FootEnt E[kB];
#pragma unroll
      for (int k = 0; k < kB; ++k) {
        const int l = min(l0 + k * LPP + lp, nl - 1);
        E[k] = ent[(2 * l + axis) * S.n_pup + idx];
      }
#pragma unroll
      for (int k = 0; k < kB; ++k) {
        const int l = l0 + k * LPP + lp;
        if (lp < LPP && l < nl) {
          FootTap t;
          t.w0 = E[k].w0;  // rows: the projection kernel's ry.w0 * wl
          t.w1 = E[k].w1;
          t.k = E[k].k;  // byte offset in the window
          tab[l * TPL + j] = t;
        }
      }
    }
    if (lane < 2 * nl) forg[lane] = org;
    for (int e = lane + kWave; e < 2 * nl; e += kWave)
      forg[e] = ent[e * S.n_pup + ((e & 1) ? sb.a * NS : sb.b * NS)].i0;
  }
  wave_sync();
  // 2. window columns (32-bit byte offsets: the plan keeps every layer below 2^30 floats),
  // all ROWS rows of a column slot (rows fh.. of a slot are loaded and stored but never
  // read).  Rows leave the grid (wrap, or clamp on a zero-boundary grid) only for windows at
  // a grid edge: when no lane's window does, the rows are plain strides and each column is
  // ROWS unpredicated loads and stores at immediate offsets.
  const char* lay_b = reinterpret_cast<const char*>(p.layers + (int64_t)b * p.layer_stride);
  float val[2][ROWS];
  int cbase[2], oyv[2];
  bool edge = false;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const FootCol& C = fc[k];
    const int l = C.lj >> 8, j = C.lj & 255;
    const int ox = forg[2 * l];
    oyv[k] = forg[2 * l + 1];
    int col = ox + j;
    if (C.boundary == 0) col -= col >= C.nx ? C.nx : 0;
    else col = min(max(col, 0), C.nx - 1);
    cbase[k] = C.offset + col;
    edge = edge || (C.fh > 0 && (oyv[k] < 0 || oyv[k] + ROWS > C.ny));
  }
  if (__builtin_amdgcn_ballot_w64(edge) == 0) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      // a lane without a column reads the realisation's first float ROWS times
      const bool has = fc[k].fh > 0;
      uint32_t off = has ? (uint32_t)(cbase[k] + oyv[k] * fc[k].nx) * 4u : 0u;
      const uint32_t stride = has ? (uint32_t)fc[k].nx * 4u : 0u;
#pragma unroll
      for (int i = 0; i < ROWS; ++i) {
        val[k][i] = *reinterpret_cast<const float*>(lay_b + off);
        off += stride;
      }
    }
  } else {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const FootCol& C = fc[k];
      const bool periodic = C.boundary == 0;
#pragma unroll
      for (int i = 0; i < ROWS; ++i) {
        int rr = oyv[k] + i;
        if (rr >= C.ny) rr = periodic ? rr - C.ny : C.ny - 1;
        rr = max(rr, 0);
        val[k][i] = i < C.fh ? ld_idx(reinterpret_cast<const float*>(lay_b),
                                       (uint32_t)(cbase[k] + rr * C.nx))
                             : 0.0f;
      }
    }
  }
  wave_sync();  // the window overwrites the origins
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    if (fc[k].fh > 0) {
      float* dst = fp + fc[k].dst;
#pragma unroll
      for (int i = 0; i < ROWS; ++i) dst[i] = val[k][i];
      if constexpr (PK::kOn) {  // the lane that holds the poked element's column adds to it
        const int l = fc[k].lj >> 8, row = pk.iy - oyv[k];
        if (l == pk.l && cbase[k] == fc[k].offset + pk.ix && row >= 0 && row < fc[k].fh)
          dst[row] += pk.delta;
      }
    }
  }
  wave_sync();
  // 3. stencils, in the projection kernel's chunks of layers (a last partial chunk is padded
  // with zero-weight repeats of the last layer, as there)
  int pr[PPL], pc[PPL];
  float psi[PPL];
#pragma unroll
  for (int i = 0; i < PPL; ++i) {
    const int q = min(lane + i * kWave, NPIX - 1);
    pr[i] = q / NS;
    pc[i] = q - pr[i] * NS;
    psi[i] = 0.0f;
  }
  auto stencil = [&](int l, bool pad) {
#pragma unroll
    for (int i = 0; i < PPL; ++i) {
      const FootTap cx = tab[l * TPL + pc[i]];
      const FootTap ry = tab[l * TPL + NS + pr[i]];
      // column-major window: the next row is the next float, the next column a slot later
      const float* w0p =
          reinterpret_cast<const float*>(reinterpret_cast<const char*>(fp) + (ry.k + cx.k));
      const float v00 = w0p[0], v10 = w0p[1];
      const float v01 = w0p[SLOT], v11 = w0p[SLOT + 1];
      const float r0v = fmaf(cx.w0, v00, cx.w1 * v01);
      const float r1v = fmaf(cx.w0, v10, cx.w1 * v11);
      const float wy0 = pad ? 0.0f : ry.w0, wy1 = pad ? 0.0f : ry.w1;
      psi[i] = fmaf(wy0, r0v, fmaf(wy1, r1v, psi[i]));
    }
  };
  int l0 = 0;
  for (; l0 + kProjLC <= nl; l0 += kProjLC) {
#pragma unroll
    for (int jj = 0; jj < kProjLC; ++jj) stencil(l0 + jj, false);
  }
  if (l0 < nl) {
#pragma unroll
    for (int jj = 0; jj < kProjLC; ++jj) stencil(min(l0 + jj, nl - 1), l0 + jj >= nl);
  }
#pragma unroll
  for (int i = 0; i < PPL; ++i) ph[i] = psi[i] * S.kappa;
}

// Fills the wave's E region with the subaperture field E[r][c] = A exp(i(psi - pi (r+c)/N)),
// and the wave's copies of the sensor's lag-phase and twiddle tables.  All per-subaperture
// values (S, sb, sid, b) are wave-uniform.  FIELD says where the phase comes from.
template <int NS, int FIELD, class PK = NoPoke>
__device__ __forceinline__ void otf_field(const FwdParams& p, const DevSensor& S,
                                          const DevSubap& sb, int sid, int b, double stepd,
                                          char* wsm, const OtfLds& lo, int frame = 0,
                                          const PK& pk = PK{}) {
  constexpr int NPIX = NS * NS;
  constexpr int PPL = (NPIX + kWave - 1) / kWave;  // pixels per lane
  const int lane = lane_id();
  const int nl = p.n_layers;
  OtfTables<NS> tables;
  tables.load(p, S, sb);
  if constexpr (FIELD != kFieldGather) {
    float ph[PPL];
    if constexpr (FIELD == kFieldFoot) {
      foot_phase<NS>(p, S, sb, b, frame, wsm, lo, pk, ph);
      wave_sync();  // E and the tables overlay the stencil entries and the window just read
    } else {  // the projection kernel already wrote kappa psi
      const float* src = p.phase_in + (int64_t)b * p.phase_per_real + S.phase_off +
                         (int64_t)sb.v * NPIX;
#pragma unroll
      for (int i = 0; i < PPL; ++i) ph[i] = src[min(lane + i * kWave, NPIX - 1)];
    }
    tables.store(p, S, wsm, lo);
    float2* E = reinterpret_cast<float2*>(wsm + lo.e_off);
#pragma unroll
    for (int i = 0; i < PPL; ++i) {
      const int q = lane + i * kWave;
      if (q < NPIX) {
        const int r = small_div<NS>(q), c = q - r * NS;
        float turns = fmaf(ph[i], 0.15915494309189535f, -field_ramp(S, r, c));
        turns -= rintf(turns);
        float sn, cs;
        sincos_rev(turns, &sn, &cs);
        E[q] = tables.amp[i] ? make_float2(cs, sn) : make_float2(0.0f, 0.0f);
      }
    }
    wave_sync();
  } else {
    tables.store(p, S, wsm, lo);
    int pr[PPL], pc[PPL];
#pragma unroll
    for (int i = 0; i < PPL; ++i) {
      const int qq = min(lane + i * kWave, NPIX - 1);
      pr[i] = small_div<NS>(qq);
      pc[i] = qq - pr[i] * NS;
    }
    // taps: [l][0..NS) columns, [l][NS..2NS) rows
    Tap* taps = reinterpret_cast<Tap*>(wsm + lo.taps_off);
    {
      const int g = lane >> 5, j = lane & 31;
      const bool row = j >= NS;
      const int idx = row ? sb.a * NS + (j - NS) : sb.b * NS + j;
      for (int l0 = 0; l0 < nl; l0 += 2) {
        const int l1 = l0 + 1 < nl ? l0 + 1 : l0;
        const DevLayer L0 = cload(p.lay, l0), L1 = cload(p.lay, l1);
        const DevAffine A0 = cload(p.aff, sid * nl + l0), A1 = cload(p.aff, sid * nl + l1);
        const Tap t = tap_of(g ? L1 : L0, g ? A1 : A0, row, idx, stepd);
        if (j < 2 * NS && (g == 0 || l0 + 1 < nl)) taps[(l0 + g) * 2 * NS + j] = t;
      }
    }
    wave_sync();
    // projection: every load of a 4-layer chunk for all of the lane's pixels in flight at once
    const float* lay_b = p.layers + (int64_t)b * p.layer_stride;
    float psi[PPL];
#pragma unroll
    for (int i = 0; i < PPL; ++i) psi[i] = 0.0f;
    // chunks of LC layers with every load in flight; layers past the end repeat the last one
    // with weight 0 (no predicated register arrays)
    constexpr int LC = 5;
    for (int l0 = 0; l0 < nl; l0 += LC) {
      float v[LC][PPL][4];
      Tap cx[LC][PPL], ry[LC][PPL];
      float wl[LC];
#pragma unroll
      for (int jj = 0; jj < LC; ++jj) {
        const int l = min(l0 + jj, nl - 1);
        const DevLayer L = cload(p.lay, l);
        wl[jj] = l0 + jj < nl ? L.weight : 0.0f;
        const float* g = lay_b + L.offset;
#pragma unroll
        for (int i = 0; i < PPL; ++i) {
          cx[jj][i] = taps[l * 2 * NS + pc[i]];
          ry[jj][i] = taps[l * 2 * NS + NS + pr[i]];
          v[jj][i][0] = ld_idx(g, (uint32_t)(ry[jj][i].i0 + cx[jj][i].i0));
          v[jj][i][1] = ld_idx(g, (uint32_t)(ry[jj][i].i0 + cx[jj][i].i1));
          v[jj][i][2] = ld_idx(g, (uint32_t)(ry[jj][i].i1 + cx[jj][i].i0));
          v[jj][i][3] = ld_idx(g, (uint32_t)(ry[jj][i].i1 + cx[jj][i].i1));
        }
      }
#pragma unroll
      for (int jj = 0; jj < LC; ++jj) {
#pragma unroll
        for (int i = 0; i < PPL; ++i) {
          const Tap& a = cx[jj][i];
          const Tap& r = ry[jj][i];
          const float val = r.w0 * fmaf(a.w0, v[jj][i][0], a.w1 * v[jj][i][1]) +
                            r.w1 * fmaf(a.w0, v[jj][i][2], a.w1 * v[jj][i][3]);
          psi[i] = fmaf(wl[jj], val, psi[i]);
        }
      }
    }
    float2* E = reinterpret_cast<float2*>(wsm + lo.e_off);
#pragma unroll
    for (int i = 0; i < PPL; ++i) {
      const int q = lane + i * kWave;
      // phase in turns, reduced to [-1/2, 1/2] before the sincos
      float turns =
          fmaf(psi[i], S.kappa * 0.15915494309189535f, -field_ramp(S, pr[i], pc[i]));
      turns -= rintf(turns);
      float sn, cs;
      sincos_rev(turns, &sn, &cs);
      if (q < NPIX)
        E[q] = tables.amp[i] ? make_float2(cs, sn) : make_float2(0.0f, 0.0f);
    }
    wave_sync();
  }
}

typedef float v4f_t __attribute__((ext_vector_type(4)));

// a + b * w
__device__ __forceinline__ float2 cfma(float2 b, float2 w, float2 a) {
  return make_float2(fmaf(b.x, w.x, fmaf(-b.y, w.y, a.x)), fmaf(b.x, w.y, fmaf(b.y, w.x, a.y)));
}

__device__ __forceinline__ float2 cmul2(float2 b, float2 w) {
  return make_float2(fmaf(b.x, w.x, -(b.y * w.y)), fmaf(b.x, w.y, b.y * w.x));
}

// X[q] = sum_s a[s] (-i)^{q s}, in place
__device__ __forceinline__ void otf_dft4(float2 a[4]) {
  const float2 s02 = make_float2(a[0].x + a[2].x, a[0].y + a[2].y);
  const float2 d02 = make_float2(a[0].x - a[2].x, a[0].y - a[2].y);
  const float2 s13 = make_float2(a[1].x + a[3].x, a[1].y + a[3].y);
  const float2 d13 = make_float2(a[1].x - a[3].x, a[1].y - a[3].y);
  a[0] = make_float2(s02.x + s13.x, s02.y + s13.y);
  a[1] = make_float2(d02.x + d13.y, d02.y - d13.x);
  a[2] = make_float2(s02.x - s13.x, s02.y - s13.y);
  a[3] = make_float2(d02.x - d13.y, d02.y + d13.x);
}

// Sum of a over the two half-waves in lanes 0-31 and of b in lanes 32-63 (ROWS = 32), or of
// a over the two 16-lane rows of each half in its first row and of b in its second (ROWS = 16).
template <int ROWS>
__device__ __forceinline__ float half_sums(float a, float b) {
  const uint32_t ua = __builtin_bit_cast(uint32_t, a), ub = __builtin_bit_cast(uint32_t, b);
  if constexpr (ROWS == 32) {
    const auto r = __builtin_amdgcn_permlane32_swap(ua, ub, false, false);
    return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
  } else {
    const auto r = __builtin_amdgcn_permlane16_swap(ua, ub, false, false);
    return __builtin_bit_cast(float, (uint32_t)r[0]) + __builtin_bit_cast(float, (uint32_t)r[1]);
  }
}

// Weighted lags AW[dy][dx] = w_dy Kel(dx, dy) s(dx) s(dy) A[dy][dx], dy = 0 .. NS-1, dx =
// -(NS-1) .. NS-1 (slot dx + 2 Q of a row), A[dy][dx] = sum E[r][c] conj(E[r+dy][c+dx]),
// through the F-point DFT of the field rows:
//   1. G[r][f] = sum_c E[r][c] e^{-2 pi i f c / F}: lane (r, k0) forms the four frequencies
//      k0 + Q q of its row from the sums over c = s mod 4 and a 4-point DFT;
//   2. C[dy][f] = sum_r G[r][f] conj(G[r+dy][f]): lane (f, group g) takes the first factors
//      r = g mod kGroups, with its rows g + j in registers, so that every lane runs the same
//      products (rows past the field are zero); the groups are added across the wave;
//   3. A[dy][dx] = 1/F sum_f C[dy][f] e^{-2 pi i f dx / F}: lane (dy, k0) forms the lags
//      congruent to k0 modulo Q as in 1, with the same twiddles, and weighs them.
// The kernel is bound by vector issue: for n_sub = 10 a wave of the split field takes 702
// vector instructions, where forming every row pair's lags directly (400 multiply-adds a lane,
// a sum of 55 partial lag rows through LDS, then the weights) made it 986-1,000; busy cycles of a spot
// launch of 128 realisations of six 80 x 80 LGS: -27 %; 100 frames of one, with the projection
// in the waves: 1,176 -> 1,008 us.  The row DFTs on the matrix cores measured slower: FP32 matrix
// instructions hold the vector units for 32 cycles each (16x16x4).
template <int NS>
__device__ __forceinline__ void otf_corr(const DevSubap& sb, const NaEntry& el, char* wsm,
                                         const OtfLds& lo) {
  using O = Otf<NS>;
  constexpr int Q = O::kQ, F = O::kF, GR = O::kGroups, RQ = O::kRows * Q;
  const int lane = lane_id();
  const float2* E = reinterpret_cast<const float2*>(wsm + lo.e_off);
  float2* G = reinterpret_cast<float2*>(wsm + lo.g_off);
  float2* C = reinterpret_cast<float2*>(wsm + lo.c_off);
  float2* aw = reinterpret_cast<float2*>(wsm + lo.aw_off);
  const float2* stab = reinterpret_cast<const float2*>(wsm + lo.stab_off);
  constexpr int kM = (NS + 3) / 4;  // field columns per residue modulo 4
  auto twiddles = [&](int k0, float2 w[kOtfTw]) {
    const float4* t = reinterpret_cast<const float4*>(wsm + lo.tw_off) + k0 * (kOtfTw / 2);
#pragma unroll
    for (int i = 0; i < kOtfTw / 2; ++i) {
      const float4 v = t[i];
      w[2 * i] = make_float2(v.x, v.y);
      w[2 * i + 1] = make_float2(v.z, v.w);
    }
  };
  // 1. row transforms
  constexpr int kU1 = (RQ + kWave - 1) / kWave;
#pragma unroll
  for (int it = 0; it < kU1; ++it) {
    const int u = lane + it * kWave;
    if (RQ % kWave == 0 || it + 1 < kU1 || u < RQ) {
      const int r = small_div<Q>(u), k0 = u - r * Q;
      float2 w[kOtfTw], a[4];
      twiddles(k0, w);
      const float2* e = E + (r < NS ? r : NS - 1) * NS;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        a[s] = s < NS ? e[s < NS ? s : 0] : make_float2(0.0f, 0.0f);
#pragma unroll
        for (int m = 1; m < kM; ++m)
          if (s + 4 * m < NS) a[s] = cfma(e[s + 4 * m], w[m - 1], a[s]);
        if (s > 0 && s < NS) a[s] = cmul2(a[s], w[4 + s]);
      }
      otf_dft4(a);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        G[q * RQ + u] = r < NS ? a[q] : make_float2(0.0f, 0.0f);
    }
  }
  wave_sync();
  {  // 2. row products
    constexpr int GL = kWave / GR;  // lanes of a group
    const int g = lane / GL, fl = lane - g * GL;
    const int f = fl < F ? fl : 0;
    const int q = small_div<Q>(f), k0 = f - q * Q;
    float2 R[NS], acc[NS];
#pragma unroll
    for (int j = 0; j < NS; ++j) R[j] = G[q * RQ + (g + j) * Q + k0];
    wave_sync();  // C overlays G
#pragma unroll
    for (int r = 0; r < NS; r += GR)
#pragma unroll
      for (int dy = 0; r + dy < NS; ++dy) {
        const float2 u = R[r], v = R[r + dy];
        if (r == 0) {
          acc[dy].x = fmaf(u.x, v.x, u.y * v.y);
          acc[dy].y = dy == 0 ? 0.0f : fmaf(u.y, v.x, -(u.x * v.y));
        } else {
          acc[dy].x = fmaf(u.x, v.x, fmaf(u.y, v.y, acc[dy].x));
          if (dy > 0) acc[dy].y = fmaf(u.y, v.x, fmaf(-u.x, v.y, acc[dy].y));
        }
      }
    // lane group g ends with the sums of the lags dy = g kD .. g kD + kD - 1
    constexpr int kD = (NS + GR - 1) / GR;
    float2 t[kD];
#pragma unroll
    for (int i = 0; i < kD; ++i) {
      auto at = [&](int grp) {
        const int dy = grp * kD + i;
        return dy < NS ? acc[dy < NS ? dy : 0] : make_float2(0.0f, 0.0f);
      };
      if constexpr (GR == 2) {
        const float2 a = at(0), b = at(1);
        t[i] = make_float2(half_sums<32>(a.x, b.x), half_sums<32>(a.y, b.y));
      } else {  // groups 0, 1 in lanes 0-31 and 2, 3 in lanes 32-63
        const float2 a = at(0), b = at(1), c = at(2), d = at(3);
        t[i] = make_float2(half_sums<16>(half_sums<32>(a.x, c.x), half_sums<32>(b.x, d.x)),
                           half_sums<16>(half_sums<32>(a.y, c.y), half_sums<32>(b.y, d.y)));
      }
    }
    if (fl < F) {
#pragma unroll
      for (int i = 0; i < kD; ++i)
        if (NS % GR == 0 || g * kD + i < NS) C[(g * kD + i) * O::kCP + fl] = t[i];
    }
  }
  wave_sync();
  // 3. lags and their weights
  constexpr int kU3 = (NS * Q + kWave - 1) / kWave;
#pragma unroll
  for (int it = 0; it < kU3; ++it) {
    const int u = lane + it * kWave;
    if (u < NS * Q) {
      const int dy = small_div<Q>(u);
      int k0 = u - dy * Q;
      asm volatile("" : "+v"(k0));  // read again, not held in registers across the products
      float2 w[kOtfTw], a[4];
      twiddles(k0, w);
      const float4* c = reinterpret_cast<const float4*>(C + dy * O::kCP);
#pragma unroll
      for (int m = 0; m < Q; ++m) {
        const float4 lo4 = c[2 * m], hi4 = c[2 * m + 1];
        const float2 v[4] = {make_float2(lo4.x, lo4.y), make_float2(lo4.z, lo4.w),
                             make_float2(hi4.x, hi4.y), make_float2(hi4.z, hi4.w)};
#pragma unroll
        for (int s = 0; s < 4; ++s) a[s] = m == 0 ? v[s] : cfma(v[s], w[m - 1], a[s]);
        // two steps of loads in flight: all of them would take 8 Q registers
        if (m & 1) __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int s = 1; s < 4; ++s) a[s] = cmul2(a[s], w[4 + s]);
      otf_dft4(a);
      // a[q] is the lag dx = k0 + Q q (less F for q >= 2); slots outside the lags stay unread
      const float2 sy = stab[dy + NS - 1];
      const float scale = dy == 0 ? 1.0f / (float)F : 2.0f / (float)F;
      const float yp = (float)dy * sb.ey;
      if (el.n == 0 || sb.gam == 0.0f) {  // wave-uniform: one real Gaussian
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int dx = k0 + Q * (q < 2 ? q : q - 4);
          const float2 sx = stab[min(max(dx, 1 - NS), NS - 1) + NS - 1];
          const float proj = fmaf((float)dx, sb.ex, yp);
          const float k = __expf(-sb.alpha * proj * proj) * scale;
          const float2 tw = cmul2(sx, sy);
          aw[dy * O::kAP + dx + 2 * Q] = cmul2(a[q], make_float2(tw.x * k, tw.y * k));
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int dx = k0 + Q * (q < 2 ? q : q - 4);
          const float2 sx = stab[min(max(dx, 1 - NS), NS - 1) + NS - 1];
          const float2 k = elong_tf(sb, el, fmaf((float)dx, sb.ex, yp), scale);
          aw[dy * O::kAP + dx + 2 * Q] = cmul2(a[q], cmul2(cmul2(sx, sy), k));
        }
      }
    }
  }
  wave_sync();
}

// Fold modulo n_pix: P[Ky][Kx] = sum over lags (dy, dx) = (Ky, Kx) mod n_pix of AW, lane per K.
template <int NS>
__device__ __forceinline__ void otf_fold(const DevSensor& S, char* wsm, const OtfLds& lo) {
  constexpr int NL = Otf<NS>::kLags;
  const int lane = lane_id();
  const int np = S.n_pix, np2 = np * np;
  const float2* aw = reinterpret_cast<const float2*>(wsm + lo.aw_off);
  float2* P = reinterpret_cast<float2*>(wsm + lo.p_off);
  if (np == 8) {  // the common 8 x 8 image: lane = K, trip counts known (same sums, same order)
    const int Ky = lane >> 3, Kx = lane & 7, dx0 = Kx - 8 * ((Kx + NS - 1) >> 3);
    float2 acc = make_float2(0.0f, 0.0f);
#pragma unroll
    for (int a = 0; a < (NS + 7) / 8; ++a) {
      const int dy = Ky + 8 * a;
#pragma unroll
      for (int c = 0; c < (NL + 7) / 8 + 1; ++c) {
        const int dx = dx0 + 8 * c;
        if (dy < NS && dx < NS) {
          const float2 v = aw[dy * Otf<NS>::kAP + dx + 2 * Otf<NS>::kQ];
          acc.x += v.x;
          acc.y += v.y;
        }
      }
    }
    P[lane] = acc;
    wave_sync();
    return;
  }
  for (int K = lane; K < np2; K += kWave) {
    const int Ky = fdiv(K, np, S.inv_npix), Kx = K - Ky * np;
    const int dx0 = Kx - np * fdiv(Kx + NS - 1, np, S.inv_npix);
    float2 acc = make_float2(0.0f, 0.0f);
    for (int dy = Ky; dy < NS; dy += np) {
      for (int dx = dx0; dx < NS; dx += np) {
        const float2 v = aw[dy * Otf<NS>::kAP + dx + 2 * Otf<NS>::kQ];
        acc.x += v.x;
        acc.y += v.y;
      }
    }
    P[K] = acc;
  }
  wave_sync();
}

// B[q] = c Re sum_K P[K] W^{K.q} on the matrix cores (n_pix <= 8), as two real 16 x 16 x 16
// products of four v_mfma_f32_16x16x4f32 each:  [Zr | Zi] = [Pr | Pi] F1 with
// F1 = [[C, S], [-S, C]], then B = c F2 [Zr ; Zi] with F2 = [C | -S] (C, S: cosine and sine of
// 2 pi (k n mod n_pix) / n_pix, per-sensor tables).  Operand layout: lane l supplies
// A[l%16][l/16] and B[l/16][l%16]; accumulator i of lane l holds D[4 (l/16) + i][l%16].
// The intermediate [Zr | Zi] goes through LDS over the P and Z regions.  The lane's operands
// are loaded before the fold that precedes the image (ImageOps).
struct ImageOps {
  float f1[4], f2[4];
};

__device__ __forceinline__ ImageOps image_ops(const FwdParams& p, const DevSensor& S) {
  ImageOps o;
  const int lane = lane_id();
  const int r16 = lane & 15, kq = lane >> 4;
  const float* F1 = p.mtab + max(S.mtab_off, 0);
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    o.f1[s] = S.mtab_off >= 0 ? F1[(kq + 4 * s) * 16 + r16] : 0.0f;
    o.f2[s] = S.mtab_off >= 0 ? F1[256 + r16 * 16 + kq + 4 * s] : 0.0f;
  }
  return o;
}

__device__ __forceinline__ void otf_image_mfma(const DevSensor& S, const ImageOps& ops,
                                               char* wsm, const OtfLds& lo) {
  const int lane = lane_id();
  const int np = S.n_pix;
  const int r16 = lane & 15, kq = lane >> 4;
  const float2* P = reinterpret_cast<const float2*>(wsm + lo.p_off);
  float* D = reinterpret_cast<float*>(wsm + lo.p_off);  // [16][16]
  float* B = reinterpret_cast<float*>(wsm + lo.b_off);
  float a[4];
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int k = kq + 4 * s, kk = k & 7;
    const float2 v = (r16 < np && kk < np) ? P[r16 * np + kk] : make_float2(0.0f, 0.0f);
    a[s] = k < 8 ? v.x : v.y;
  }
  v4f_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], ops.f1[s], acc, 0, 0, 0);
  wave_sync();
#pragma unroll
  for (int i = 0; i < 4; ++i) D[(4 * kq + i) * 16 + r16] = acc[i];
  wave_sync();
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const int k = kq + 4 * s;
    a[s] = k < 8 ? D[k * 16 + (r16 & 7)] : D[(k - 8) * 16 + 8 + (r16 & 7)];
  }
  acc = (v4f_t){0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int s = 0; s < 4; ++s) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(ops.f2[s], a[s], acc, 0, 0, 0);
  wave_sync();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int qy = 4 * kq + i;
    if (qy < np && r16 < np) B[qy * np + r16] = S.flux_c * acc[i];
  }
  wave_sync();
}

// B[q] = c Re sum_K P[K] W^{K.q}, separable through Z[Ky][qx] (W = e^{2 pi i / n_pix}).
__device__ __forceinline__ void otf_image(const DevSensor& S, const ImageOps& ops, char* wsm,
                                          const OtfLds& lo) {
  if (S.mtab_off >= 0) {
    otf_image_mfma(S, ops, wsm, lo);
    return;
  }
  const int lane = lane_id();
  const int np = S.n_pix, np2 = np * np;
  const float2* P = reinterpret_cast<const float2*>(wsm + lo.p_off);
  float2* Z = reinterpret_cast<float2*>(wsm + lo.z_off);
  float* B = reinterpret_cast<float*>(wsm + lo.b_off);
  const float2* wt = reinterpret_cast<const float2*>(wsm + lo.wtab_off);
  for (int t = lane; t < np2; t += kWave) {
    const int Ky = fdiv(t, np, S.inv_npix), qx = t - Ky * np;
    float2 z = make_float2(0.0f, 0.0f);
    int idx = 0;
#pragma unroll 8
    for (int Kx = 0; Kx < np; ++Kx) {
      const float2 a = P[Ky * np + Kx];
      const float2 w = wt[idx];
      z.x = fmaf(a.x, w.x, fmaf(-a.y, w.y, z.x));
      z.y = fmaf(a.x, w.y, fmaf(a.y, w.x, z.y));
      idx += qx;
      if (idx >= np) idx -= np;
    }
    Z[t] = z;
  }
  wave_sync();
  for (int t = lane; t < np2; t += kWave) {
    const int qy = fdiv(t, np, S.inv_npix), qx = t - qy * np;
    float v = 0.0f;
    int idx = 0;
#pragma unroll 8
    for (int Ky = 0; Ky < np; ++Ky) {
      const float2 z = Z[Ky * np + qx];
      const float2 w = wt[idx];
      v = fmaf(z.x, w.x, fmaf(-z.y, w.y, v));
      idx += qy;
      if (idx >= np) idx -= np;
    }
    B[t] = S.flux_c * v;
  }
  wave_sync();
}

// Noise and centre-of-gravity sums over the binned image (sum B', sum x B', sum y B'), one
// pixel per lane: pixels 2j and 2j + 1 share Philox block j (words x, y and z, w); every lane
// returns the wave totals.
struct Cog {
  float s0, sx, sy;
};

__device__ __forceinline__ Cog cog_sums(const FwdParams& p, const DevSensor& S, int sid, int b,
                                        int v, int64_t step, const float* B) {
  const int lane = lane_id();
  const int np = S.n_pix, np2 = np * np;
  const float half = 0.5f * (float)(np - 1);
  float s0 = 0.0f, sx = 0.0f, sy = 0.0f;
  const bool noisy = S.noisy && p.noise_on;
  for (int q = lane; q < np2; q += kWave) {
    float bq = B[q];
    if (noisy) {
      const uint4 ctr = make_uint4((uint32_t)(q >> 1), (uint32_t)v,
                                   ((uint32_t)b << 8) | (uint32_t)sid, (uint32_t)step);
      const uint4 w = philox4x32_10(ctr, p.seed_lo, p.seed_hi);
      const bool odd = (q & 1) != 0;
      add_noise_one(bq, odd ? w.z : w.x, odd ? w.w : w.y, S.read_noise);
    }
    const int y = fdiv(q, np, S.inv_npix), x = q - y * np;
    s0 += bq;
    sx = fmaf((float)x - half, bq, sx);
    sy = fmaf((float)y - half, bq, sy);
  }
  Cog c;
  c.s0 = wave_sum(s0);
  c.sx = wave_sum(sx);
  c.sy = wave_sum(sy);
  return c;
}

// Slopes (0 when the flux is not positive) and the flux of subaperture v, of frame `frame`
// of a multi-frame launch (outputs [frame][B][...]).
__device__ __forceinline__ void write_slopes(const FwdParams& p, const DevSensor& S, int b,
                                             int v, const Cog& c, int frame = 0) {
  if (lane_id() == 0) {
    const bool ok = c.s0 > 0.0f;
    const int64_t fb = (int64_t)frame * p.batch + b;
    float* out = p.slopes + fb * p.n_slopes + S.slope_off;
    out[v] = ok ? c.sx / c.s0 : 0.0f;
    out[S.n_valid + v] = ok ? c.sy / c.s0 : 0.0f;
    if (p.aux) p.aux[fb * p.n_valid_total + S.aux_off + v] = c.s0;
  }
}

// Binned noise-free (or noisy) image of one subaperture into the wave's B region.
template <int NS, int FIELD, class PK = NoPoke>
__device__ __forceinline__ void otf_spot(const FwdParams& p, const DevSensor& S,
                                         const DevSubap& sb, int sid, int b, int64_t step,
                                         char* wsm, const OtfLds& lo, int frame = 0,
                                         const PK& pk = PK{}) {
  otf_field<NS, FIELD>(p, S, sb, sid, b, (double)step, wsm, lo, frame, pk);
  otf_corr<NS>(sb, na_entry(p, step), wsm, lo);
  const ImageOps ops = image_ops(p, S);
  otf_fold<NS>(S, wsm, lo);
  otf_image(S, ops, wsm, lo);
}

template <int NS, int FIELD>
__device__ void otf_subap(const FwdParams& p, int t, int64_t step, char* wsm, int frame = 0) {
  int b, sid, v;
  t = __builtin_amdgcn_readfirstlane(t);  // wave-uniform: per-subaperture data in SGPRs
  task_of(p.otf, t, b, sid, v);
  const DevSensor S = cload(p.sen, sid);
  const DevSubap sb = cload(p.sub, S.valid_off + v);
  // the layout the host sized the launch with: the per-pixel gather holds its stencil taps
  // in the union (the sensor tables follow whichever of its parts is last)
  const OtfLds lo = otf_lds_layout(NS, p.n_layers, S.n_pix, FIELD == kFieldGather,
                                   FIELD == kFieldFoot ? S.foot_floats : 0);
  otf_spot<NS, FIELD>(p, S, sb, sid, b, step, wsm, lo, frame);
  const Cog c = cog_sums(p, S, sid, b, v, step + p.noise_dstep,
                         reinterpret_cast<const float*>(wsm + lo.b_off));
  write_slopes(p, S, b, v, c, frame);
  wave_sync();
}

}  // namespace wfs
