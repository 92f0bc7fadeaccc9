// The spot launch of the forward model, one kernel per (subaperture size, mode): every
// lag-domain sensor of that size for every realisation at one time step:
// lag-domain path, one subaperture per 64-lane wavefront, with (pipelined frames) the next
// step's projection blocks spread evenly among its blocks.
// The mode is a template parameter so that each kernel only holds the registers of its own
// paths: FIELD says where the lag-domain waves get the phase (kField*), PROJ adds the
// projection blocks.  With the staged footprint (kFieldFoot) one launch can
// cover several frames: the lag-domain blocks repeat once per frame, frame k at step + k.
#pragma once

#include "wfs_otf.h"
#include "wfs_project.h"

namespace wfs {

// Register budget of the lag-domain kernels (waves per SIMD): the split field's LDS (4.7 KB
// per wave at n_sub = 10) lets 8 four-wave blocks share a CU, the staged footprint's 5.
template <int FIELD, bool PROJ>
constexpr int otf_waves_per_simd() {
  return FIELD == kFieldFoot || PROJ ? 6 : 8;
}

template <int NS, int FIELD, bool PROJ>
__global__ __launch_bounds__(kBlock)
__attribute__((amdgpu_waves_per_eu(FIELD == kFieldGather ? 1 : otf_waves_per_simd<FIELD, PROJ>())))
void wfs_forward_kernel(FwdParams p) {
  extern __shared__ __align__(16) char smem[];
  const int64_t step = current_step(p);
  const int n = gridDim.x;
  int L = p.xcd_remap ? xcd_logical_block(blockIdx.x, n) : blockIdx.x;
  if constexpr (PROJ) {
    // pipelined frames: projection blocks of the next step spread evenly among the spot
    // blocks, so memory-latency-bound gathers share the CUs with VALU-bound spot waves.
    // Block L is a projection block when floor((L+1)P/n) > floor(LP/n).
    const int c0 = (int)((int64_t)L * p.proj_blocks / n);
    const int c1 = (int)((int64_t)(L + 1) * p.proj_blocks / n);
    if (c1 > c0) {
      project_block(p, c0, p.phase_out, (double)(step + 1), smem);
      return;
    }
    L -= c1;
  }
  int frame = 0;
  if constexpr (FIELD == kFieldFoot) {  // blocks of frame k follow those of frame k - 1
    frame = L / p.otf_blocks;
    L -= frame * p.otf_blocks;
  }
  const int wave = threadIdx.x >> 6;
  char* wsm = smem + wave * p.lds_per_wave;
  const int total = p.otf.per_real * p.batch;
  // one subaperture per wave and no task loop: a loop would let the compiler hoist per-lane
  // index arithmetic out of it and hold those registers across every stage
  const int t = L * kWavesPerBlock + wave;
  if (t < total) otf_subap<NS, FIELD>(p, t, step + frame, wsm, frame);
}

template <int NS, int FIELD, bool PROJ>
static hipError_t launch_fwd_mode(const FwdParams& p, int grid, int lds, hipStream_t st) {
  hipLaunchKernelGGL((wfs_forward_kernel<NS, FIELD, PROJ>), dim3(grid), dim3(kBlock), lds, st, p);
  return hipGetLastError();
}

// Launch of the spot kernel for subaperture size NS (lag-domain path), mode from the params.
template <int NS>
hipError_t launch_fwd_ns(const FwdParams& p, hipStream_t st) {
  const bool foot = p.otf_from_phase == kFieldFoot;
  const int64_t grid64 = (int64_t)p.proj_blocks + (int64_t)p.otf_blocks * (foot ? p.n_frames : 1);
  if (grid64 == 0) return hipSuccess;
  if (grid64 > 0x7FFFFFFF) return hipErrorInvalidValue;
  const int grid = (int)grid64;
  int lds = p.lds_per_wave * kWavesPerBlock;
  if (p.proj_blocks > 0 && p.proj_lds > lds) lds = p.proj_lds;
  const bool fused = p.otf_from_phase == kFieldGather, proj = p.proj_blocks > 0;
  if (foot) {  // one launch for every frame; no projection blocks
    if (proj || p.n_frames < 1) return hipErrorInvalidValue;
    return launch_fwd_mode<NS, kFieldFoot, false>(p, grid, lds, st);
  }
  if (fused) {  // the pipelined projection only exists in the split schedule
    if (proj) return hipErrorInvalidValue;
    return launch_fwd_mode<NS, kFieldGather, false>(p, grid, lds, st);
  }
  return proj ? launch_fwd_mode<NS, kFieldPhase, true>(p, grid, lds, st)
              : launch_fwd_mode<NS, kFieldPhase, false>(p, grid, lds, st);
}

}  // namespace wfs
