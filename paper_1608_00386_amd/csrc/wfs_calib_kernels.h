// Sparse calibration (Sec. 2.5): the interaction-matrix entries of the subapertures that an
// actuator poke can reach.  An actuator of a zero-boundary (mirror) grid enters a few pupil
// pixels only -- its bilinear stencils reach one pitch to each side -- and a noise-free
// subaperture that none of them belongs to has the same slopes with and without the poke, so
// its entry is (s - s) / 2a of the unpoked slopes.  The others are formed here from the layers
// themselves, the poked element taken with +a by one wave and -a by the wave beside it, with
// the arithmetic of the dense batch (the staged-footprint field, whose phase equals the
// projection kernel's bit for bit).
#pragma once

#include "wfs_otf.h"

namespace wfs {

// The element `e` of a realisation's layer buffer as a poke (host: at most one layer holds it).
__device__ __forceinline__ Poke poke_at(const FwdParams& p, int64_t e, float delta) {
  Poke k{-1, 0, 0, delta};
  for (int l = 0; l < p.n_layers; ++l) {
    const DevLayer L = cload(p.lay, l);
    const int64_t r = e - L.offset;
    if (r >= 0 && r < (int64_t)L.nx * L.ny) {
      k.l = l;
      k.iy = (int32_t)r / L.nx;
      k.ix = (int32_t)r - k.iy * L.nx;
    }
  }
  return k;
}

// Subapertures [a0, a1] x [b0, b1] of a sensor that hold every pixel whose stencil gives the
// poked element a weight: coordinates in [index - 1, index + 1), with one pupil index of slack
// for the rounding of the reciprocal; a0 > a1 or b0 > b1: none.
struct SubRange {
  int a0, a1, b0, b1;
};

__device__ __forceinline__ void axis_range(double a, double inv_a, double b, int i, int n_pup,
                                           int n_sub, int& s0, int& s1) {
  const double lo = ceil(((double)(i - 1) - b) * inv_a) - 1.0;
  const double hi = floor(((double)(i + 1) - b) * inv_a) + 1.0;
  if (!(hi >= 0.0) || !(lo <= (double)(n_pup - 1))) {
    s0 = 1;
    s1 = 0;
    return;
  }
  s0 = __builtin_amdgcn_readfirstlane(lo < 0.0 ? 0 : (int)lo) / n_sub;
  s1 = __builtin_amdgcn_readfirstlane(hi > (double)(n_pup - 1) ? n_pup - 1 : (int)hi) / n_sub;
}

__device__ __forceinline__ SubRange sub_range(const FwdParams& p, const DevSensor& S, int sid,
                                              const Poke& pk, double stepd) {
  SubRange r{1, 0, 1, 0};
  if (pk.l < 0) return r;
  const DevAffine A = cload(p.aff, (int64_t)sid * p.n_layers + pk.l);
  axis_range(A.ax, A.inv_ax, A.bx0 + stepd * A.dbx, pk.ix, S.n_pup, S.n_sub, r.b0, r.b1);
  axis_range(A.ay, A.inv_ay, A.by0 + stepd * A.dby, pk.iy, S.n_pup, S.n_sub, r.a0, r.a1);
  return r;
}

// FFT-path sensors, realisation b of a chunk: actuator b / 2 at +amp (b even) or -amp.
__device__ __forceinline__ Poke batch_poke(const FwdParams& p, const CalibParams& q, int b) {
  return poke_at(p, q.act_offset + (b >> 1), b & 1 ? -q.amp : q.amp);
}

__device__ __forceinline__ bool poke_touches(const FwdParams& p, const CalibParams& q,
                                             const DevSensor& S, const DevSubap& sb, int sid,
                                             int b, double stepd) {
  const SubRange r = sub_range(p, S, sid, batch_poke(p, q, b), stepd);
  return sb.a >= r.a0 && sb.a <= r.a1 && sb.b >= r.b0 && sb.b <= r.b1;
}

// Block = two (actuator, sensor, cell) tasks, each a pair of waves (+a, -a).
template <int NS>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(6))) void
calib_spot_kernel(FwdParams p, CalibParams q) {
  extern __shared__ __align__(16) char smem[];
  const int64_t step = current_step(p);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pair = wave >> 1, sign = wave & 1;
  char* wsm = smem + wave * p.lds_per_wave;
  const int t = blockIdx.x * 2 + pair;
  const int j = t / q.per_act;
  const int k = (t - j * q.per_act) / q.cells, cell = t - j * q.per_act - k * q.cells;
  bool live = j < q.n_act;
  float cx = 0.0f, cy = 0.0f;
  int64_t at = 0;
  int n_valid = 0;
  if (live) {
    const int sid = p.otf.ids[k];
    const DevSensor S = cload(p.sen, sid);
    const Poke pk = poke_at(p, q.act_offset + j, sign ? -q.amp : q.amp);
    const SubRange r = sub_range(p, S, sid, pk, (double)step);
    const int w = r.b1 - r.b0 + 1, h = r.a1 - r.a0 + 1;
    live = w > 0 && h > 0 && cell < w * h;
    int v = -1;
    if (live) {
      const int cy0 = cell / w;
      v = cload(p.subidx, (int64_t)S.subidx_off + (r.a0 + cy0) * S.n_sa + r.b0 + cell - cy0 * w);
    }
    live = v >= 0;
    if (live) {
      const DevSubap sb = cload(p.sub, S.valid_off + v);
      const OtfLds lo = otf_lds_layout(NS, p.n_layers, S.n_pix, false, S.foot_floats);
      otf_spot<NS, kFieldFoot>(p, S, sb, sid, 0, step, wsm, lo, 0, pk);
      const Cog c = cog_sums(p, S, sid, 0, v, step, reinterpret_cast<const float*>(wsm + lo.b_off));
      const bool ok = c.s0 > 0.0f;
      cx = ok ? c.sx / c.s0 : 0.0f;
      cy = ok ? c.sy / c.s0 : 0.0f;
      at = (int64_t)j * q.ld_im + S.slope_off + v;
      n_valid = S.n_valid;
      wave_sync();
      if (sign && lane_id() == 0) *reinterpret_cast<float2*>(wsm) = make_float2(cx, cy);
    }
  }
  __syncthreads();  // both waves of a pair are live or neither is
  if (live && !sign && lane_id() == 0) {
    const float2 pulled = *reinterpret_cast<const float2*>(wsm + p.lds_per_wave);
    q.im[at] = (cx - pulled.x) / (2.0f * q.amp);
    q.im[at + n_valid] = (cy - pulled.y) / (2.0f * q.amp);
  }
}

template <int NS>
hipError_t launch_calib_ns(const FwdParams& p, const CalibParams& q, hipStream_t st) {
  const int64_t tasks = (int64_t)q.n_act * q.per_act;
  if (tasks == 0) return hipSuccess;
  if (tasks > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipLaunchKernelGGL((calib_spot_kernel<NS>), dim3((unsigned)((tasks + 1) / 2)), dim3(kBlock),
                     p.lds_per_wave * kWavesPerBlock, st, p, q);
  return hipGetLastError();
}

}  // namespace wfs
