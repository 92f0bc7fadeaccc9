// Interaction-matrix calibration (Sec. 2.5 of the paper).
//
// Calibration registers the slopes of one actuator poke at a time through the sensor model.
// Here a batch of 2h realisations carries h pokes at +amplitude followed by the same h pokes
// at -amplitude (push-pull), so one batched forward call measures h columns; a second kernel
// forms each column as the central difference (s+ - s-) / (2 amplitude).  The control matrix
// built from it (Sec. 2.6) is set-up work in a library of its own (tlse.hip).
//
// Where no sensor draws noise and the actuators are elements of mirror grids, only the
// subapertures a poke can reach are formed (wfs_calib_kernels.h); the FFT-path sensors' share
// of that is here: their pixels projected with the poked element, the spectrum chunks of the
// touched subapertures, and the differences.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "wfs_calib_kernels.h"
#include "wfs_project.h"

namespace wfs {

constexpr int kCalBlock = 256;

// Rows of the interaction matrix for slopes no poke reaches: (s - s) / (2 amp) of the unpoked
// slopes s.
__global__ __launch_bounds__(kCalBlock) void calib_fill_kernel(const float* __restrict__ s,
                                                               int32_t n_slopes, float two_amp,
                                                               float* __restrict__ im,
                                                               int64_t ld_im) {
  float* d = im + (int64_t)blockIdx.y * ld_im;
  for (int32_t k = blockIdx.x * kCalBlock + threadIdx.x; k < n_slopes;
       k += gridDim.x * kCalBlock)
    d[k] = (s[k] - s[k]) / two_amp;
}

// Projection of the pixels of the touched FFT-path subapertures (blocks of wfs_project_kernel;
// every realisation reads the same layers).
__global__ __launch_bounds__(kBlock) void calib_project_kernel(FwdParams p, CalibParams q,
                                                               float* phase) {
  extern __shared__ __align__(16) char smem[];
  const int b = blockIdx.x / p.proj_per_real;
  const int2 d = cload(p.proj_desc, blockIdx.x - b * p.proj_per_real);
  const int sid = d.y & 0xFFFFFF, row0 = d.x & 0xFFFF, c0 = (d.x >> 16) * kProjStrip;
  const int rows = kProjRows << (d.y >> 24);
  const double stepd = (double)current_step(p);
  const DevSensor S = cload(p.sen, sid);
  const Poke pk = batch_poke(p, q, b);
  const SubRange r = sub_range(p, S, sid, pk, stepd);
  if (r.a0 > r.a1 || r.b0 > r.b1 || row0 >= (r.a1 + 1) * S.n_sub ||
      row0 + rows <= r.a0 * S.n_sub || c0 >= (r.b1 + 1) * S.n_sub ||
      c0 + kProjStrip <= r.b0 * S.n_sub)
    return;  // block-uniform
  project_block(p, blockIdx.x, phase, stepd, smem, pk);
}

// Their entries: thread per (FFT-path sensor, subaperture), block row per actuator.
__global__ __launch_bounds__(kWave) void calib_fft_diff_kernel(FwdParams p, CalibParams q) {
  const int j = blockIdx.x;
  const double stepd = (double)current_step(p);
  const Poke pk = poke_at(p, q.act_offset + j, 0.0f);
  for (int k = 0; k < p.fft.n; ++k) {
    const int sid = p.fft.ids[k];
    const DevSensor S = cload(p.sen, sid);
    const SubRange r = sub_range(p, S, sid, pk, stepd);
    for (int v = threadIdx.x; v < S.n_valid; v += kWave) {
      const DevSubap sb = p.sub[S.valid_off + v];
      if (sb.a < r.a0 || sb.a > r.a1 || sb.b < r.b0 || sb.b > r.b1) continue;
      const float* sp = p.slopes + (int64_t)(2 * j) * p.n_slopes + S.slope_off + v;
      const float* sm = sp + p.n_slopes;
      float* d = q.im + (int64_t)j * q.ld_im + S.slope_off + v;
      d[0] = (sp[0] - sm[0]) / (2.0f * q.amp);
      d[S.n_valid] = (sp[S.n_valid] - sm[S.n_valid]) / (2.0f * q.amp);
    }
  }
}

// Realisation r < h holds actuator act0 + r at +amp, realisation h + r the same actuator at
// -amp (r < n_chunk; the rest hold no poke), on top of `base` (one realisation) or zero.
__global__ __launch_bounds__(kCalBlock) void calib_poke_kernel(float* __restrict__ layers,
                                                               const float* __restrict__ base,
                                                               int64_t stride, int32_t h,
                                                               int64_t act0, int32_t n_chunk,
                                                               float amp) {
  const int64_t total = 2 * (int64_t)h * stride;
  for (int64_t i = (int64_t)blockIdx.x * kCalBlock + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * kCalBlock) {
    const int64_t r = i / stride, e = i - r * stride;
    const int64_t j = r < h ? r : r - h;
    float v = base ? base[e] : 0.0f;
    if (j < n_chunk && e == act0 + j) v += r < h ? amp : -amp;
    layers[i] = v;
  }
}

// Row j of the interaction matrix (slopes of actuator j): (s[j] - s[h + j]) / (2 amp).
__global__ __launch_bounds__(kCalBlock) void calib_diff_kernel(const float* __restrict__ s,
                                                               int32_t h, int32_t n_slopes,
                                                               float two_amp,
                                                               float* __restrict__ im,
                                                               int64_t ld_im) {
  const int32_t j = blockIdx.y;
  const float* sp = s + (int64_t)j * n_slopes;
  const float* sm = s + (int64_t)(h + j) * n_slopes;
  float* d = im + (int64_t)j * ld_im;
  for (int32_t k = blockIdx.x * kCalBlock + threadIdx.x; k < n_slopes;
       k += gridDim.x * kCalBlock)
    d[k] = (sp[k] - sm[k]) / two_amp;
}

hipError_t calib_fill(const float* slopes, int32_t n_slopes, int32_t n_act, float amp, float* im,
                      int64_t ld_im, hipStream_t st) {
  const int gx = (n_slopes + kCalBlock - 1) / kCalBlock;
  for (int32_t j0 = 0; j0 < n_act; j0 += 65535) {  // grid rows
    const int32_t n = n_act - j0 < 65535 ? n_act - j0 : 65535;
    calib_fill_kernel<<<dim3(gx < 64 ? gx : 64, n), kCalBlock, 0, st>>>(
        slopes, n_slopes, 2.0f * amp, im + (int64_t)j0 * ld_im, ld_im);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_fft_spots(const FwdParams& p, const FftTables& t, const CalibParams* cal,
                            hipStream_t st);

// Entries of the FFT-path sensors for the q.n_act actuators of a chunk: p.batch = 2 q.n_act
// realisations, the sensors' projection blocks, p.phase_in = phase.
hipError_t calib_fft(const FwdParams& p, const FftTables& t, const CalibParams& q, float* phase,
                     int proj_lds, hipStream_t st) {
  const int64_t pb = (int64_t)p.proj_per_real * p.batch;
  if (pb == 0) return hipSuccess;
  if (pb > 0x7FFFFFFF) return hipErrorInvalidValue;
  calib_project_kernel<<<(unsigned)pb, kBlock, proj_lds, st>>>(p, q, phase);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if ((e = launch_fft_spots(p, t, &q, st)) != hipSuccess) return e;
  calib_fft_diff_kernel<<<(unsigned)q.n_act, kWave, 0, st>>>(p, q);
  return hipGetLastError();
}

// instantiated per subaperture size in the wfs_fwd_ns*.hip units
extern template hipError_t launch_calib_ns<2>(const FwdParams&, const CalibParams&, hipStream_t);
extern template hipError_t launch_calib_ns<3>(const FwdParams&, const CalibParams&, hipStream_t);
extern template hipError_t launch_calib_ns<4>(const FwdParams&, const CalibParams&, hipStream_t);
extern template hipError_t launch_calib_ns<5>(const FwdParams&, const CalibParams&, hipStream_t);
extern template hipError_t launch_calib_ns<6>(const FwdParams&, const CalibParams&, hipStream_t);
extern template hipError_t launch_calib_ns<7>(const FwdParams&, const CalibParams&, hipStream_t);
extern template hipError_t launch_calib_ns<8>(const FwdParams&, const CalibParams&, hipStream_t);
extern template hipError_t launch_calib_ns<9>(const FwdParams&, const CalibParams&, hipStream_t);
extern template hipError_t launch_calib_ns<10>(const FwdParams&, const CalibParams&, hipStream_t);
extern template hipError_t launch_calib_ns<11>(const FwdParams&, const CalibParams&, hipStream_t);
extern template hipError_t launch_calib_ns<12>(const FwdParams&, const CalibParams&, hipStream_t);

// Entries of the lag-domain sensors of one subaperture size.
hipError_t calib_spots(const FwdParams& p, int ns, const CalibParams& q, hipStream_t st) {
  switch (ns) {
    case 2: return launch_calib_ns<2>(p, q, st);
    case 3: return launch_calib_ns<3>(p, q, st);
    case 4: return launch_calib_ns<4>(p, q, st);
    case 5: return launch_calib_ns<5>(p, q, st);
    case 6: return launch_calib_ns<6>(p, q, st);
    case 7: return launch_calib_ns<7>(p, q, st);
    case 8: return launch_calib_ns<8>(p, q, st);
    case 9: return launch_calib_ns<9>(p, q, st);
    case 10: return launch_calib_ns<10>(p, q, st);
    case 11: return launch_calib_ns<11>(p, q, st);
    case 12: return launch_calib_ns<12>(p, q, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t calib_poke(float* layers, const float* base, int64_t stride, int32_t h, int64_t act0,
                      int32_t n_chunk, float amp, hipStream_t st) {
  const int64_t total = 2 * (int64_t)h * stride;
  const int64_t blocks = (total + kCalBlock - 1) / kCalBlock;
  const int grid = (int)(blocks < 65536 ? blocks : 65536);
  calib_poke_kernel<<<grid, kCalBlock, 0, st>>>(layers, base, stride, h, act0, n_chunk, amp);
  return hipGetLastError();
}

hipError_t calib_diff(const float* slopes, int32_t h, int32_t n_slopes, int32_t n_chunk,
                      float amp, float* im, int64_t ld_im, hipStream_t st) {
  const int gx = (n_slopes + kCalBlock - 1) / kCalBlock;
  calib_diff_kernel<<<dim3(gx < 64 ? gx : 64, n_chunk), kCalBlock, 0, st>>>(
      slopes, h, n_slopes, 2.0f * amp, im, ld_im);
  return hipGetLastError();
}

}  // namespace wfs
