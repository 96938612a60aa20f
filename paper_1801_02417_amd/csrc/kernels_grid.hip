// Kernels of the de-gridding and gridding passes (vis.hpp) and their launches.
#include <mutex>
#include <set>

#include "vis.hpp"

namespace psara {

template <typename R, int MODE, int T>
__global__ void __launch_bounds__(256)
degrid_kernel(const ProbDesc* __restrict__ descs, const int4* __restrict__ items, int src_slot, int out_slot) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  __shared__ double red[8];
  const int4 it = items[blockIdx.x];
  degrid_item<R, MODE, T>(descs[it.x], it, src_slot, out_slot, (Cell<R>*)smem_raw, red);
}

// (FP64: the LDS holds one workgroup per CU, so two waves per SIMD and 256 registers, which
// keeps the FP64 accumulators out of scratch memory)
template <typename R, int MODE, int T>
__global__ void __launch_bounds__(kGridThreads, sizeof(R) == 8 ? 2 : 4)
grid_kernel(const ProbDesc* __restrict__ descs, const int4* __restrict__ items, int src_slot, int use_cfac, int ce) {
  __shared__ unsigned long long acc[8 * (kGridTile + T - 1) * (kGridTile + T - 1)];
  extern __shared__ __align__(16) unsigned char stage_raw[];
  __shared__ double red[kGridRed];
  const int4 it = items[blockIdx.x];
  grid_item<R, MODE, T>(descs[it.x], it, src_slot, use_cfac, ce, acc, stage_raw, red);
}

template <typename R, int MODE, int T>
__global__ void __launch_bounds__(kGridThreads, sizeof(R) == 8 ? 2 : 4)
degrid_grid_kernel(const ProbDesc* __restrict__ descs, const int4* __restrict__ items, int src_slot, int out_slot,
                   int ce) {
  __shared__ unsigned long long acc[8 * (kGridTile + T - 1) * (kGridTile + T - 1)];
  extern __shared__ __align__(16) unsigned char stage_raw[];
  __shared__ double red[kGridRed];
  const int4 it = items[blockIdx.x];
  degrid_grid_item<R, MODE, T>(descs[it.x], it, src_slot, out_slot, ce, acc, stage_raw, red);
}

template <typename R, int T>
void launch_degrid_t(int mode, const LaunchArgs& a, size_t shm, int src_slot, int out_slot) {
  const dim3 grid(a.nitems), block(256);
  if (mode == DG_DUAL) {
    hipLaunchKernelGGL((degrid_kernel<R, DG_DUAL, T>), grid, block, shm, a.stream, a.descs, a.items, src_slot, out_slot);
  } else if (mode == DG_STOKES) {
    hipLaunchKernelGGL((degrid_kernel<R, DG_STOKES, T>), grid, block, shm, a.stream, a.descs, a.items, src_slot, out_slot);
  } else if (mode == DG_FORWARD) {
    hipLaunchKernelGGL((degrid_kernel<R, DG_FORWARD, T>), grid, block, shm, a.stream, a.descs, a.items, src_slot, out_slot);
  } else {
    hipLaunchKernelGGL((degrid_kernel<R, DG_RESIDUAL, T>), grid, block, shm, a.stream, a.descs, a.items, src_slot, out_slot);
  }
}

// taps: the kernel support T of every problem in the launch (4, 6 or 8)
template <typename R>
void launch_degrid(int mode, const LaunchArgs& a, int max_ts, int taps, int src_slot, int out_slot) {
  if (a.nitems <= 0) return;
  const int W = max_ts + taps - 1;
  const size_t shm = (size_t)W * W * sizeof(Cell<R>);
  if (taps == 4) launch_degrid_t<R, 4>(mode, a, shm, src_slot, out_slot);
  else if (taps == 6) launch_degrid_t<R, 6>(mode, a, shm, src_slot, out_slot);
  else launch_degrid_t<R, 8>(mode, a, shm, src_slot, out_slot);
}

template <typename R, int T>
void launch_grid_t(int mode, const LaunchArgs& a, int src_slot, int use_cfac) {
  const dim3 grid(a.nitems), block(kGridThreads);
  const int ce = a.grid_ce;
  const size_t shm = grid_stage_bytes<R>(ce);
  if (mode == GR_DUAL) {
    hipLaunchKernelGGL((grid_kernel<R, GR_DUAL, T>), grid, block, shm, a.stream, a.descs, a.items, src_slot, use_cfac, ce);
  } else if (mode == GR_STOKES) {
    hipLaunchKernelGGL((grid_kernel<R, GR_STOKES, T>), grid, block, shm, a.stream, a.descs, a.items, src_slot, use_cfac, ce);
  } else {
    hipLaunchKernelGGL((grid_kernel<R, GR_PLAIN, T>), grid, block, shm, a.stream, a.descs, a.items, src_slot, use_cfac, ce);
  }
}

// taps: the kernel support T of every problem in the launch (4, 6 or 8)
template <typename R>
void launch_grid(int mode, const LaunchArgs& a, int taps, int src_slot, int use_cfac) {
  if (a.nitems <= 0) return;
  if (taps == 4) launch_grid_t<R, 4>(mode, a, src_slot, use_cfac);
  else if (taps == 6) launch_grid_t<R, 6>(mode, a, src_slot, use_cfac);
  else launch_grid_t<R, 8>(mode, a, src_slot, use_cfac);
}

template <typename R, int T>
void launch_degrid_grid_t(int mode, const LaunchArgs& a, int src_slot, int out_slot) {
  const dim3 grid(a.nitems), block(kGridThreads);
  const int ce = a.grid_ce;
  const size_t shm = grid_stage_bytes<R>(ce);
  if (mode == GR_STOKES) {
    hipLaunchKernelGGL((degrid_grid_kernel<R, GR_STOKES, T>), grid, block, shm, a.stream, a.descs, a.items, src_slot,
                       out_slot, ce);
  } else if (mode == GR_PLAIN) {
    hipLaunchKernelGGL((degrid_grid_kernel<R, GR_PLAIN, T>), grid, block, shm, a.stream, a.descs, a.items, src_slot,
                       out_slot, ce);
  } else {
    hipLaunchKernelGGL((degrid_grid_kernel<R, GR_DUAL, T>), grid, block, shm, a.stream, a.descs, a.items, src_slot,
                       out_slot, ce);
  }
}

template <typename R>
void launch_degrid_grid(int mode, const LaunchArgs& a, int taps, int src_slot, int out_slot) {
  if (a.nitems <= 0) return;
  if (taps == 4) launch_degrid_grid_t<R, 4>(mode, a, src_slot, out_slot);
  else if (taps == 6) launch_degrid_grid_t<R, 6>(mode, a, src_slot, out_slot);
  else launch_degrid_grid_t<R, 8>(mode, a, src_slot, out_slot);
}

// Raise the dynamic-LDS limit of the de-grid / grid kernels once, outside any graph capture.
template <typename R, int T>
void set_degrid_limits_t(int max_ts) {
  const int shm_st = (int)grid_stage_bytes<R>(kChunkEntries);
  hip_check(hipFuncSetAttribute((const void*)grid_kernel<R, GR_DUAL, T>, hipFuncAttributeMaxDynamicSharedMemorySize, shm_st), "attr");
  hip_check(hipFuncSetAttribute((const void*)grid_kernel<R, GR_PLAIN, T>, hipFuncAttributeMaxDynamicSharedMemorySize, shm_st), "attr");
  hip_check(hipFuncSetAttribute((const void*)grid_kernel<R, GR_STOKES, T>, hipFuncAttributeMaxDynamicSharedMemorySize, shm_st), "attr");
  hip_check(hipFuncSetAttribute((const void*)degrid_grid_kernel<R, GR_DUAL, T>, hipFuncAttributeMaxDynamicSharedMemorySize, shm_st), "attr");
  hip_check(hipFuncSetAttribute((const void*)degrid_grid_kernel<R, GR_PLAIN, T>, hipFuncAttributeMaxDynamicSharedMemorySize, shm_st), "attr");
  hip_check(hipFuncSetAttribute((const void*)degrid_grid_kernel<R, GR_STOKES, T>, hipFuncAttributeMaxDynamicSharedMemorySize, shm_st), "attr");
  const int W = max_ts + T - 1;
  const int shm_dg = W * W * (int)sizeof(Cell<R>);
  hip_check(hipFuncSetAttribute((const void*)degrid_kernel<R, DG_DUAL, T>, hipFuncAttributeMaxDynamicSharedMemorySize, shm_dg), "attr");
  hip_check(hipFuncSetAttribute((const void*)degrid_kernel<R, DG_FORWARD, T>, hipFuncAttributeMaxDynamicSharedMemorySize, shm_dg), "attr");
  hip_check(hipFuncSetAttribute((const void*)degrid_kernel<R, DG_RESIDUAL, T>, hipFuncAttributeMaxDynamicSharedMemorySize, shm_dg), "attr");
  hip_check(hipFuncSetAttribute((const void*)degrid_kernel<R, DG_STOKES, T>, hipFuncAttributeMaxDynamicSharedMemorySize, shm_dg), "attr");
}

// Set once per device for every tap count, at the largest de-grid tile (hipFuncSetAttribute is
// a device-wide setting, so later engines and batches need not repeat it).
template <typename R>
void set_grid_kernel_limits(int /*max_ts*/, int /*taps*/) {
  static std::mutex mu;
  static std::set<int> done;
  int dev = 0;
  hip_check(hipGetDevice(&dev), "hipGetDevice");
  std::lock_guard<std::mutex> lk(mu);
  if (done.count(dev)) return;
  set_degrid_limits_t<R, 4>(kMaxDegridTile);
  set_degrid_limits_t<R, 6>(kMaxDegridTile);
  set_degrid_limits_t<R, 8>(kMaxDegridTile);
  done.insert(dev);
}

template void set_grid_kernel_limits<float>(int, int);
template void set_grid_kernel_limits<double>(int, int);
template void launch_degrid<float>(int, const LaunchArgs&, int, int, int, int);
template void launch_degrid<double>(int, const LaunchArgs&, int, int, int, int);
template void launch_grid<float>(int, const LaunchArgs&, int, int, int);
template void launch_grid<double>(int, const LaunchArgs&, int, int, int);
template void launch_degrid_grid<float>(int, const LaunchArgs&, int, int, int);
template void launch_degrid_grid<double>(int, const LaunchArgs&, int, int, int);


}  // namespace psara
