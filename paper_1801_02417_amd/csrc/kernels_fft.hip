// Kernels of the FFT passes (fft_pass.hpp) and their launches.
#include "fft_pass.hpp"

namespace psara {

template <typename R, int CELLS, int PASS, int PM = -1>
__global__ void __launch_bounds__(CELLS / 2)
fft_pass_kernel(const ProbDesc* __restrict__ descs, const int4* __restrict__ items, int src_slot, int dst_slot) {
  __shared__ FftSmem<R, CELLS, PASS> sm;
  const int4 it = items[blockIdx.x];
  fft_pass<R, CELLS, PASS, PM>(descs[it.x], it, src_slot, dst_slot, sm);
}

// the primal-step modes of the row passes (PASS 0 and 4), for one CELLS
template <typename R, int CELLS, int PASS>
void launch_row_primal_t(int mode, const LaunchArgs& a) {
  const dim3 grid(a.nitems);
#define PSARA_RP(PM) \
  hipLaunchKernelGGL((fft_pass_kernel<R, CELLS, PASS, PM>), grid, dim3(CELLS / 2), 0, a.stream, a.descs, a.items, 0, 0)
  switch (mode) {
    case PM_CONSTRAINED: PSARA_RP(PM_CONSTRAINED); break;
    case PM_INIT: PSARA_RP(PM_INIT); break;
    case PM_UNCONSTRAINED: PSARA_RP(PM_UNCONSTRAINED); break;
    case PM_TV_CONSTRAINED: PSARA_RP(PM_TV_CONSTRAINED); break;
    default: PSARA_RP(PM_TV_UNCONSTRAINED); break;
  }
#undef PSARA_RP
}

template <typename R, int PASS>
void launch_row_primal(int mode, const LaunchArgs& a, int cells) {
  if (a.nitems <= 0) return;
  if (cells == 512) launch_row_primal_t<R, 512, PASS>(mode, a);
  else if (cells == 2048) launch_row_primal_t<R, 2048, PASS>(mode, a);
  else launch_row_primal_t<R, 1024, PASS>(mode, a);
}

template <typename R>
void launch_primal_fft(int mode, const LaunchArgs& a, int cells) { launch_row_primal<R, 0>(mode, a, cells); }

template <typename R>
void launch_fused_rows(int mode, const LaunchArgs& a, int cells) { launch_row_primal<R, 4>(mode, a, cells); }

template <typename R>
void launch_fft(int pass, const LaunchArgs& a, int cells, int src_slot, int dst_slot) {
  if (a.nitems <= 0) return;
  const dim3 grid(a.nitems);
#define PSARA_FFT(C, PS) \
  hipLaunchKernelGGL((fft_pass_kernel<R, C, PS>), grid, dim3(C / 2), 0, a.stream, a.descs, a.items, src_slot, dst_slot)
  if (cells == 512) {
    switch (pass) {
      case 0: PSARA_FFT(512, 0); break;
      case 1: PSARA_FFT(512, 1); break;
      case 2: PSARA_FFT(512, 2); break;
      default: PSARA_FFT(512, 3); break;
    }
  } else if (cells == 2048) {
    switch (pass) {
      case 0: PSARA_FFT(2048, 0); break;
      case 1: PSARA_FFT(2048, 1); break;
      case 2: PSARA_FFT(2048, 2); break;
      default: PSARA_FFT(2048, 3); break;
    }
  } else {
    switch (pass) {
      case 0: PSARA_FFT(1024, 0); break;
      case 1: PSARA_FFT(1024, 1); break;
      case 2: PSARA_FFT(1024, 2); break;
      default: PSARA_FFT(1024, 3); break;
    }
  }
#undef PSARA_FFT
}

template void launch_fft<float>(int, const LaunchArgs&, int, int, int);
template void launch_primal_fft<float>(int, const LaunchArgs&, int);
template void launch_primal_fft<double>(int, const LaunchArgs&, int);
template void launch_fused_rows<float>(int, const LaunchArgs&, int);
template void launch_fused_rows<double>(int, const LaunchArgs&, int);
template void launch_fft<double>(int, const LaunchArgs&, int, int, int);

}  // namespace psara
