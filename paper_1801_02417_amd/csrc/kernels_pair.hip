// A pass of the data branch and a stage of the SARA (or TV) branch in one launch.
//
// The two branches of an iteration touch different arrays between the row passes, so a stage of
// one may run beside any pass of the other.  As kernels of their own on two streams they cost two
// cross-stream dependencies an iteration, about 8 us each inside a graph, and a kernel boundary
// for every stage; here the workgroups of both are one grid (the list `lead` first, padded to a
// multiple of eight so that every item keeps the XCD its list was ordered for).  The items run the
// device functions of the separate kernels, so the numbers are the same.
#include <algorithm>
#include <mutex>
#include <set>

#include "dwt.hpp"
#include "fft_pass.hpp"
#include "tv.hpp"
#include "vis.hpp"

namespace psara {

struct Pair {
  const ProbDesc* descs;
  const int4* a;      // data branch items
  const int4* b;      // prior branch items
  int na, nb;
  int lead;           // workgroups of the list that comes first, padded
  int b_first;
};

// whether this workgroup has an item, and which
__device__ __forceinline__ bool pair_item(const Pair& q, bool& is_a, int4& it) {
  const int w = blockIdx.x;
  const bool head = w < q.lead;
  is_a = head != (q.b_first != 0);
  const int i = head ? w : w - q.lead;
  if (i >= (is_a ? q.na : q.nb)) return false;
  it = is_a ? q.a[i] : q.b[i];
  return true;
}

template <class A, class B>
constexpr size_t max_size() { return sizeof(A) > sizeof(B) ? sizeof(A) : sizeof(B); }

constexpr int kCells = 512;
static_assert(kCoarseThreads == kGridThreads, "one workgroup size");

// P5 with the first analysis level (SEP: with items that run every basis of a tile)
template <typename R, int TOM, bool SEP>
__global__ void __launch_bounds__(256) p5_analysis_kernel(Pair q) {
  using SA = FftSmem<R, kCells, 1>;
  using SB = AnaSmem<R, TOM, SEP>;
  __shared__ __align__(16) unsigned char raw[max_size<SA, SB>()];
  bool is_a;
  int4 it;
  if (!pair_item(q, is_a, it)) return;
  if (is_a) fft_pass<R, kCells, 1, -1>(q.descs[it.x], it, 0, 0, *(SA*)raw);
  else analysis_item<R, AM_DUAL, TOM, SEP>(q.descs[it.x], it, 1, IMG_X, COEF_A, *(SB*)raw);
}

constexpr size_t acc_bytes(int T) { return sizeof(unsigned long long) * 8 * (kGridTile + T - 1) * (kGridTile + T - 1); }
constexpr size_t kRedBytes = sizeof(double) * kGridRed;

// the fused P6 + P7 with the coarse levels
template <typename R, int T>
__global__ void __launch_bounds__(kGridThreads, sizeof(R) == 8 ? 2 : 4) grid_coarse_kernel(Pair q, int ce) {
  extern __shared__ __align__(16) unsigned char raw[];
  bool is_a;
  int4 it;
  if (!pair_item(q, is_a, it)) return;
  if (is_a) {
    unsigned long long* acc = (unsigned long long*)raw;
    double* red = (double*)(raw + acc_bytes(T));
    unsigned char* stage = raw + acc_bytes(T) + kRedBytes;
    degrid_grid_item<R, GR_DUAL, T>(q.descs[it.x], it, VIS_BV, VIS_BV, ce, acc, stage, red);
  } else {
    coarse_item<R>(q.descs[it.x], it, *(CoarseSmem<R>*)raw);
  }
}

// P8 with the synthesis of the image
template <typename R>
__global__ void __launch_bounds__(256) p8_synthesis_kernel(Pair q) {
  using SA = FftSmem<R, kCells, 2>;
  using SB = SynSmem<R>;
  __shared__ __align__(16) unsigned char raw[max_size<SA, SB>()];
  bool is_a;
  int4 it;
  if (!pair_item(q, is_a, it)) return;
  if (is_a) fft_pass<R, kCells, 2, -1>(q.descs[it.x], it, 1, 0, *(SA*)raw);
  else synthesis_final_item<R>(q.descs[it.x], it, COEF_A, IMG_PSIA, 0, IMG_PSIA2, *(SB*)raw);
}

// the TV branch: P5 with the dual step, P8 with its synthesis
template <typename R>
__global__ void __launch_bounds__(256) p5_tv_dual_kernel(Pair q) {
  __shared__ FftSmem<R, kCells, 1> sm;
  bool is_a;
  int4 it;
  if (!pair_item(q, is_a, it)) return;
  if (is_a) fft_pass<R, kCells, 1, -1>(q.descs[it.x], it, 0, 0, sm);
  else tv_dual_item<R>(q.descs[it.x], it);
}

template <typename R>
__global__ void __launch_bounds__(256) p8_tv_synth_kernel(Pair q) {
  __shared__ FftSmem<R, kCells, 2> sm;
  bool is_a;
  int4 it;
  if (!pair_item(q, is_a, it)) return;
  if (is_a) fft_pass<R, kCells, 2, -1>(q.descs[it.x], it, 2, 0, sm);
  else tv_synth_item<R>(q.descs[it.x], it);
}

static Pair make_pair(const LaunchArgs& a, const LaunchArgs& b, bool b_first, dim3& grid) {
  const int head = b_first ? b.nitems : a.nitems, tail = b_first ? a.nitems : b.nitems;
  const int lead = (head + 7) / 8 * 8;
  grid = dim3(lead + tail);
  return Pair{a.descs, a.items, b.items, a.nitems, b.nitems, lead, b_first ? 1 : 0};
}

template <typename R, int T>
constexpr size_t grid_coarse_lds(int ce) {
  const size_t a = acc_bytes(T) + kRedBytes + grid_stage_bytes<R>(ce), b = sizeof(CoarseSmem<R>);
  return a > b ? a : b;
}

template <typename R, int T>
void launch_grid_coarse_t(const LaunchArgs& a, const LaunchArgs& b) {
  dim3 grid;
  const Pair q = make_pair(a, b, true, grid);
  const size_t lds = grid_coarse_lds<R, T>(a.grid_ce);
  hipLaunchKernelGGL((grid_coarse_kernel<R, T>), grid, dim3(kGridThreads), lds, a.stream, q, a.grid_ce);
}

template <typename R>
void launch_p5_analysis(const LaunchArgs& a, const LaunchArgs& b) {
  dim3 grid;
  const Pair q = make_pair(a, b, false, grid);
  // the largest tile side among the launch's problems, as for the analysis kernel alone
  constexpr int kWide = dwt_ana_tile<R>(1 << 30);
  const int tom = b.max_n > 0 ? dwt_ana_tile<R>(b.max_n >> 1, (b.ana_wide & kAnaWide) != 0) : kWide;
  const bool sep = (b.ana_wide & kAnaAllBases) != 0;
#define PSARA_P5A(TOM, SEP) hipLaunchKernelGGL((p5_analysis_kernel<R, TOM, SEP>), grid, dim3(256), 0, a.stream, q)
  if (tom > 8) {
    if (sep) PSARA_P5A(kWide, true);
    else PSARA_P5A(kWide, false);
  } else {
    if (sep) PSARA_P5A(8, true);
    else PSARA_P5A(8, false);
  }
#undef PSARA_P5A
}

template <typename R>
void launch_grid_coarse(const LaunchArgs& a, const LaunchArgs& b, int taps) {
  if (taps == 4) launch_grid_coarse_t<R, 4>(a, b);
  else if (taps == 6) launch_grid_coarse_t<R, 6>(a, b);
  else launch_grid_coarse_t<R, 8>(a, b);
}

template <typename R>
void launch_p8_synthesis(const LaunchArgs& a, const LaunchArgs& b) {
  dim3 grid;
  const Pair q = make_pair(a, b, false, grid);
  hipLaunchKernelGGL((p8_synthesis_kernel<R>), grid, dim3(256), 0, a.stream, q);
}

template <typename R>
void launch_p5_tv_dual(const LaunchArgs& a, const LaunchArgs& b) {
  dim3 grid;
  const Pair q = make_pair(a, b, false, grid);
  hipLaunchKernelGGL((p5_tv_dual_kernel<R>), grid, dim3(256), 0, a.stream, q);
}

template <typename R>
void launch_p8_tv_synth(const LaunchArgs& a, const LaunchArgs& b) {
  dim3 grid;
  const Pair q = make_pair(a, b, false, grid);
  hipLaunchKernelGGL((p8_tv_synth_kernel<R>), grid, dim3(256), 0, a.stream, q);
}

template <typename R>
void set_pair_kernel_limits() {
  static std::mutex mu;
  static std::set<int> done;
  int dev = 0;
  hip_check(hipGetDevice(&dev), "hipGetDevice");
  std::lock_guard<std::mutex> lk(mu);
  if (done.count(dev)) return;
  auto set = [](const void* f, size_t lds) {
    hip_check(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds), "attr");
  };
  set((const void*)grid_coarse_kernel<R, 4>, grid_coarse_lds<R, 4>(kChunkEntries));
  set((const void*)grid_coarse_kernel<R, 6>, grid_coarse_lds<R, 6>(kChunkEntries));
  set((const void*)grid_coarse_kernel<R, 8>, grid_coarse_lds<R, 8>(kChunkEntries));
  done.insert(dev);
}

#define PSARA_PAIR(R) \
  template void launch_p5_analysis<R>(const LaunchArgs&, const LaunchArgs&); \
  template void launch_grid_coarse<R>(const LaunchArgs&, const LaunchArgs&, int); \
  template void launch_p8_synthesis<R>(const LaunchArgs&, const LaunchArgs&); \
  template void launch_p5_tv_dual<R>(const LaunchArgs&, const LaunchArgs&); \
  template void launch_p8_tv_synth<R>(const LaunchArgs&, const LaunchArgs&); \
  template void set_pair_kernel_limits<R>();
PSARA_PAIR(float)
PSARA_PAIR(double)
#undef PSARA_PAIR

}  // namespace psara
