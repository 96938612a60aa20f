// Kernels of the SARA dictionary (dwt.hpp) and their launches.
#include "dwt.hpp"

namespace psara {

template <typename R, int MODE, int TOM, bool SEP>
__global__ void __launch_bounds__(256)
analysis_kernel(const ProbDesc* __restrict__ descs, const int4* __restrict__ items, int level, int src_slot, int out_coef) {
  __shared__ AnaSmem<R, TOM, SEP> sm;
  const int4 it = items[blockIdx.x];
  analysis_item<R, MODE, TOM, SEP>(descs[it.x], it, level, src_slot, out_coef, sm);
}

// Dirac block for the non-dual modes.  items: {prob, block of 256 pixels, -, partial index}
template <typename R, int MODE>
__global__ void __launch_bounds__(256)
dirac_kernel(const ProbDesc* __restrict__ descs, const int4* __restrict__ items, int src_slot, int out_coef) {
  __shared__ double red[8];
  const int4 it = items[blockIdx.x];
  const ProbDesc& P = descs[it.x];
  if (halted(P)) return;                 // stopped by an adaptive run
  const int N = P.n * P.n;
  const int p = it.y * 256 + threadIdx.x;
  KSum k1, k2;
  if (p < N) apply_coef<R, MODE>(P, out_coef, (size_t)p, ((const V4<R>*)P.img[src_slot])[p], k1, k2);
  if (MODE == AM_OBJECTIVE || MODE == AM_MOMENTS || MODE == AM_MAXABS)
    write_partials<R>(P, it.w, k1, k2, MODE == AM_MAXABS ? -1 : MODE == AM_MOMENTS, red);
}

template <typename R>
__global__ void __launch_bounds__(256)
synthesis_kernel(const ProbDesc* __restrict__ descs, const int4* __restrict__ items, int level, int src_coef) {
  __shared__ SynSmem<R> sm;
  const int4 it = items[blockIdx.x];
  synthesis_item<R>(descs[it.x], it, level, src_coef, sm);
}

// (FP32: at most 96 registers, so five workgroups fit a CU; the kernel needs no more)
template <typename R>
__global__ void __launch_bounds__(256, sizeof(R) == 4 ? 5 : 1)
synthesis_final_kernel(const ProbDesc* __restrict__ descs, const int4* __restrict__ items, int src_coef, int dst_slot,
                       int add_dirac, int dst_slot2) {
  __shared__ SynSmem<R> sm;
  const int4 it = items[blockIdx.x];
  synthesis_final_item<R>(descs[it.x], it, src_coef, dst_slot, add_dirac, dst_slot2, sm);
}

// (at most 128 registers, so two workgroups fit a CU: a batch has hundreds of them.  With 150, FP64
// ran one: 95 against 78 us for the stages of 64 problems of 32^2, 63 against 60 for 16 of 64^2)
template <typename R>
__global__ void __launch_bounds__(kCoarseThreads, 4)
coarse_kernel(const ProbDesc* __restrict__ descs, const int4* __restrict__ items) {
  __shared__ CoarseSmem<R> sm;
  const int4 it = items[blockIdx.x];
  coarse_item<R>(descs[it.x], it, sm);
}

template <typename R>
int coarse_level(int n, int levels, bool pairable) {
  // first level >= 2 whose input low-low band fits; the largest only where it spares the branch
  // its second analysis launch (sides up to twice that), and in FP32 only where the branch may run in
  // the data passes' launches: beside them on another stream the workgroups of 128^2 are the longer
  // ones (256^2 with 1024 FFT cells to a workgroup: 103 us per iteration, 94 with 64^2; FP64's largest,
  // 64^2, takes a quarter of the time, and with half of it 128^2 needs the extra launches)
  const bool whole = n <= 2 * CoarseMax<R>::value && (pairable || sizeof(R) == 8);
  const int most = whole ? CoarseMax<R>::value : CoarseMax<R>::value / 2;
  for (int c = 2; c <= levels; ++c)
    if ((n >> (c - 1)) <= most) return c;
  return levels + 1;
}

template <typename R>
void launch_coarse(const LaunchArgs& a) {
  if (a.nitems <= 0) return;
  hipLaunchKernelGGL((coarse_kernel<R>), dim3(a.nitems), dim3(kCoarseThreads), 0, a.stream, a.descs, a.items);
}

template <typename R, int TOM>
void launch_analysis_t(int mode, int level, const LaunchArgs& a, int src_slot, int out_coef) {
  const dim3 g(a.nitems), b(256);
#define PSARA_ANAL(M) \
  hipLaunchKernelGGL((analysis_kernel<R, M, TOM, false>), g, b, 0, a.stream, a.descs, a.items, level, src_slot, out_coef)
  // (only the iterations' dual lists hold all-bases items, so only AM_DUAL needs the SEP kernel)
  const bool all_bases = (a.ana_wide & kAnaAllBases) != 0;
  switch (mode) {
    case AM_DUAL:
      if (all_bases) {
        hipLaunchKernelGGL((analysis_kernel<R, AM_DUAL, TOM, true>), g, b, 0, a.stream, a.descs, a.items, level, src_slot,
                           out_coef);
      } else {
        PSARA_ANAL(AM_DUAL);
      }
      break;
    case AM_STORE: PSARA_ANAL(AM_STORE); break;
    case AM_REWEIGHT: PSARA_ANAL(AM_REWEIGHT); break;
    case AM_OBJECTIVE: PSARA_ANAL(AM_OBJECTIVE); break;
    case AM_MAXABS: PSARA_ANAL(AM_MAXABS); break;
    default: PSARA_ANAL(AM_MOMENTS); break;
  }
#undef PSARA_ANAL
}

template <typename R>
void launch_analysis(int mode, int level, const LaunchArgs& a, int src_slot, int out_coef) {
  if (a.nitems <= 0) return;
  // the largest tile side among the launch's problems (an unknown largest side takes the widest)
  constexpr int kWide = dwt_ana_tile<R>(1 << 30);
  const int tom = a.max_n > 0 ? dwt_ana_tile<R>(a.max_n >> level, (a.ana_wide & kAnaWide) != 0) : kWide;
  if constexpr (kWide > 8) {
    if (tom > 8) { launch_analysis_t<R, kWide>(mode, level, a, src_slot, out_coef); return; }
  }
  launch_analysis_t<R, 8>(mode, level, a, src_slot, out_coef);
}

template <typename R>
void launch_dirac(int mode, const LaunchArgs& a, int src_slot, int out_coef) {
  if (a.nitems <= 0) return;
  const dim3 g(a.nitems), b(256);
  switch (mode) {
    case AM_STORE: hipLaunchKernelGGL((dirac_kernel<R, AM_STORE>), g, b, 0, a.stream, a.descs, a.items, src_slot, out_coef); break;
    case AM_REWEIGHT: hipLaunchKernelGGL((dirac_kernel<R, AM_REWEIGHT>), g, b, 0, a.stream, a.descs, a.items, src_slot, out_coef); break;
    case AM_OBJECTIVE: hipLaunchKernelGGL((dirac_kernel<R, AM_OBJECTIVE>), g, b, 0, a.stream, a.descs, a.items, src_slot, out_coef); break;
    case AM_MOMENTS: hipLaunchKernelGGL((dirac_kernel<R, AM_MOMENTS>), g, b, 0, a.stream, a.descs, a.items, src_slot, out_coef); break;
    case AM_MAXABS: hipLaunchKernelGGL((dirac_kernel<R, AM_MAXABS>), g, b, 0, a.stream, a.descs, a.items, src_slot, out_coef); break;
    default: hipLaunchKernelGGL((dirac_kernel<R, AM_DUAL>), g, b, 0, a.stream, a.descs, a.items, src_slot, out_coef); break;
  }
}

template <typename R>
void launch_synthesis(int level, int /*coarsest*/, const LaunchArgs& a, int src_coef, int /*dst_slot*/) {
  if (a.nitems <= 0) return;
  hipLaunchKernelGGL((synthesis_kernel<R>), dim3(a.nitems), dim3(256), 0, a.stream, a.descs, a.items, level, src_coef);
}

template <typename R>
void launch_synthesis_final(const LaunchArgs& a, int src_coef, int dst_slot, int add_dirac, int dst_slot2) {
  if (a.nitems <= 0) return;
  hipLaunchKernelGGL((synthesis_final_kernel<R>), dim3(a.nitems), dim3(256), 0, a.stream, a.descs, a.items, src_coef,
                     dst_slot, add_dirac, dst_slot2);
}

template void launch_analysis<float>(int, int, const LaunchArgs&, int, int);
template void launch_analysis<double>(int, int, const LaunchArgs&, int, int);
template void launch_dirac<float>(int, const LaunchArgs&, int, int);
template void launch_dirac<double>(int, const LaunchArgs&, int, int);
template void launch_synthesis<float>(int, int, const LaunchArgs&, int, int);
template void launch_synthesis<double>(int, int, const LaunchArgs&, int, int);
template void launch_synthesis_final<float>(const LaunchArgs&, int, int, int, int);
template void launch_coarse<float>(const LaunchArgs&);
template void launch_coarse<double>(const LaunchArgs&);
template int coarse_level<float>(int, int, bool);
template int coarse_level<double>(int, int, bool);
template void launch_synthesis_final<double>(const LaunchArgs&, int, int, int, int);

}  // namespace psara
