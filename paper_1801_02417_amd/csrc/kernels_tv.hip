// Kernels of the TV priors (tv.hpp), their value, and the launches.
#include "tv.hpp"

namespace psara {

template <typename R>
__global__ void __launch_bounds__(256) tv_dual_kernel(const ProbDesc* __restrict__ descs, const int4* __restrict__ items) {
  const int4 it = items[blockIdx.x];
  tv_dual_item<R>(descs[it.x], it);
}

template <typename R>
__global__ void __launch_bounds__(256) tv_synth_kernel(const ProbDesc* __restrict__ descs, const int4* __restrict__ items) {
  const int4 it = items[blockIdx.x];
  tv_synth_item<R>(descs[it.x], it);
}

// partial sums of sum_i mu_i ||grad S_i(p)|| (+ upsilon_i |S_i(p)|) over the block (region 0)
template <typename R>
__global__ void __launch_bounds__(256) tv_objective_kernel(const ProbDesc* __restrict__ descs, const int4* __restrict__ items) {
  __shared__ double red[8];
  const int4 it = items[blockIdx.x];
  const ProbDesc& P = descs[it.x];
  if (halted(P)) return;                 // stopped by an adaptive run
  const int n = P.n, N = n * n, p = it.y * 256 + threadIdx.x;
  KSum k;
  if (p < N) {
    const int r = p / n, c = p - r * n;
    const V4<R>* __restrict__ S = (const V4<R>*)P.img[IMG_S];
    const V4<R> s = S[p];
    const V4<R> sd = r < n - 1 ? S[p + n] : s;
    const V4<R> sr = c < n - 1 ? S[p + 1] : s;
    const double v[4] = {s.x, s.y, s.z, s.w};
    const double d[4] = {(double)sd.x - s.x, (double)sd.y - s.y, (double)sd.z - s.z, (double)sd.w - s.w};
    const double e[4] = {(double)sr.x - s.x, (double)sr.y - s.y, (double)sr.z - s.z, (double)sr.w - s.w};
    for (int i = 0; i < 4; ++i) {
      k.add(P.tvw[i] * sqrt(d[i] * d[i] + e[i] * e[i]));
      if (P.tv_kind == 2) k.add(P.l1w[i] * fabs(v[i]));
    }
  }
  const KSum t = block_reduce(k, red);
  if (threadIdx.x == 0) {
    double* g = P.partials + 2 * (size_t)P.n_p6;
    g[2 * it.y] = t.s;
    g[2 * it.y + 1] = t.c;
  }
}

template <typename R> void launch_tv_dual(const LaunchArgs& a) {
  if (a.nitems > 0) hipLaunchKernelGGL((tv_dual_kernel<R>), dim3(a.nitems), dim3(256), 0, a.stream, a.descs, a.items);
}
template <typename R> void launch_tv_synth(const LaunchArgs& a) {
  if (a.nitems > 0) hipLaunchKernelGGL((tv_synth_kernel<R>), dim3(a.nitems), dim3(256), 0, a.stream, a.descs, a.items);
}
template <typename R> void launch_tv_objective(const LaunchArgs& a) {
  if (a.nitems > 0) hipLaunchKernelGGL((tv_objective_kernel<R>), dim3(a.nitems), dim3(256), 0, a.stream, a.descs, a.items);
}

template void launch_tv_dual<float>(const LaunchArgs&);
template void launch_tv_dual<double>(const LaunchArgs&);
template void launch_tv_synth<float>(const LaunchArgs&);
template void launch_tv_synth<double>(const LaunchArgs&);
template void launch_tv_objective<float>(const LaunchArgs&);
template void launch_tv_objective<double>(const LaunchArgs&);

}  // namespace psara
