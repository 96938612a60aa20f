// Oversampled-grid FFT passes of the measurement operator (Sec. 4.1, eq. meas_op:
// F and its adjoint, fused with the zero-padding / scaling Z and the crop / real part).
//
// The 2-D transform of a K x K grid (K = 2n) is split in two line passes through an
// intermediate `half` array of K x n cells stored transposed, [k2][r]:
//   forward  P4: image row r (n pixels, scaled, placed at wrapped positions) -> FFT along
//                columns -> half[k2][r]
//            P5: half[k2][:] (n nonzero rows at wrapped positions) -> FFT along rows ->
//                grid[k2][k1]
//   adjoint  P8: grid[k2][:] -> inverse FFT along rows -> keep the n cropped rows ->
//                half[k2][r]
//            P9: half[:][r] -> inverse FFT along columns -> keep the n cropped columns,
//                real part, scaling -> image row r
// so the zero half of the padded image is never read and the crop never writes unused
// cells.  The grid is stored transposed ([k2][k1]); the de-gridding and gridding kernels
// index it that way.  Every cell carries the four Stokes channels, which share twiddles.
//
// Line FFTs are Stockham autosort passes (radix 8, the last one 8, 4 or 2).  A thread owns one
// Stokes channel of the eight cells tl + q K/8 of a line: these are the inputs of its first
// butterfly, what it reads back after every exchange through LDS, and what the last pass leaves
// it, so the first pass takes its inputs from memory and the last one stores its outputs with no
// LDS in between.  The zero padding and the crop are then the register indices q = 2..5, and four
// adjacent lanes (the channels of a cell) trade their four remaining cells so that each holds
// all channels of one pixel (quad_transpose) for the pointwise steps.  The passes are bound by
// the latency of their memory and LDS round trips, not by bytes; against staging the line in LDS
// first and storing it from there (event times, less the 5 us that the events add): 512^2 image
// P5 24 -> 13 us, P9 + P1 + P4 39 -> 23 us, P8 43 -> 34 us; 128^2 P5 3.9 -> 1.9 us, P9 + P1 + P4
// 8.2 -> 5.0 us.
#pragma once

#include "common.hpp"
#include "launch.hpp"
#include "primal.hpp"

namespace psara {

template <typename R>
__device__ inline void dft2(cplx<R>& a, cplx<R>& b) {
  cplx<R> t = a;
  a = cadd(t, b);
  b = csub(t, b);
}

// multiply by -i (forward) or +i (inverse)
template <typename R>
__device__ inline cplx<R> rot(cplx<R> a, bool inv) { return inv ? cmk(-a.im, a.re) : cmk(a.im, -a.re); }

template <typename R>
__device__ inline void dft4(cplx<R>& a0, cplx<R>& a1, cplx<R>& a2, cplx<R>& a3, bool inv) {
  cplx<R> t0 = cadd(a0, a2), t1 = csub(a0, a2), t2 = cadd(a1, a3), t3 = rot(csub(a1, a3), inv);
  a0 = cadd(t0, t2);
  a2 = csub(t0, t2);
  a1 = cadd(t1, t3);
  a3 = csub(t1, t3);
}

template <typename R>
__device__ inline void dft8(cplx<R>* a, bool inv) {
  cplx<R> e0 = a[0], e1 = a[2], e2 = a[4], e3 = a[6];
  cplx<R> o0 = a[1], o1 = a[3], o2 = a[5], o3 = a[7];
  dft4(e0, e1, e2, e3, inv);
  dft4(o0, o1, o2, o3, inv);
  const R h = R(0.70710678118654752440084436210485);
  // o_k *= w8^k, w8 = exp(-+ 2 pi i / 8)
  o1 = inv ? cmk(h * (o1.re - o1.im), h * (o1.re + o1.im)) : cmk(h * (o1.re + o1.im), h * (o1.im - o1.re));
  o2 = rot(o2, inv);
  o3 = inv ? cmk(-h * (o3.re + o3.im), h * (o3.re - o3.im)) : cmk(h * (o3.im - o3.re), -h * (o3.re + o3.im));
  a[0] = cadd(e0, o0); a[4] = csub(e0, o0);
  a[1] = cadd(e1, o1); a[5] = csub(e1, o1);
  a[2] = cadd(e2, o2); a[6] = csub(e2, o2);
  a[3] = cadd(e3, o3); a[7] = csub(e3, o3);
}

// Where cell c of a line is kept in LDS: one cell in nine is left empty, which puts the radix-8
// pass's writes (eight cells apart) on different banks.
__device__ inline int lds_cell(int c) { return c + (c >> 3); }

// The twiddles of a pass of radix RAD after Ns = K / rem points: butterfly b of the thread is
// j = tl + b K/8.
template <typename R, int RAD>
__device__ __forceinline__ void load_twiddles(cplx<R>* wt, int lk, int ls, int tl, const cplx<R>* __restrict__ tw) {
  constexpr int NB = 8 / RAD, LR = RAD == 8 ? 3 : RAD == 4 ? 2 : 1;
  const int Ns = 1 << ls, step = lk - ls - LR;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const int k = (tl + (b << (lk - 3))) & (Ns - 1);
#pragma unroll
    for (int r = 1; r < RAD; ++r) wt[b * RAD + r] = tw[(r * k) << step];
  }
}

// The butterflies of one pass of radix RAD on v[q] = x[tl + q K/8]: butterfly b takes q = b + r NB.
template <typename R, int RAD, bool INV>
__device__ __forceinline__ void butterflies(cplx<R>* v, const cplx<R>* wt) {
  constexpr int NB = 8 / RAD;
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    cplx<R> a[RAD];
#pragma unroll
    for (int r = 0; r < RAD; ++r) {
      a[r] = v[b + r * NB];
      if (r > 0) {
        cplx<R> w = wt[b * RAD + r];
        if (INV) w.im = -w.im;
        a[r] = cmul(a[r], w);
      }
    }
    if constexpr (RAD == 8) dft8(a, INV);
    else if constexpr (RAD == 4) dft4(a[0], a[1], a[2], a[3], INV);
    else dft2(a[0], a[1]);
#pragma unroll
    for (int r = 0; r < RAD; ++r) v[b + r * NB] = a[r];
  }
}

// FFT of the line (unnormalised) whose cells tl + q K/8 of one channel the thread holds in v: in
// natural order before and after.  x: the line's LDS cells, channel ch at x[4 lds_cell(c) + ch].
// Called by the whole workgroup.
template <typename R, bool INV>
__device__ __forceinline__ void fft_line(cplx<R>* v, cplx<R>* x, int lk, int tl, int ch, const cplx<R>* __restrict__ tw) {
  dft8(v, INV);                                    // the first pass has no twiddles
  for (int ls = 3; ls < lk; ls += 3) {
    // the next pass's twiddles are requested before the exchange, so that they arrive during it
    const int rem = lk - ls;
    cplx<R> wt[8];
    if (rem >= 3) load_twiddles<R, 8>(wt, lk, ls, tl, tw);
    else if (rem == 2) load_twiddles<R, 4>(wt, lk, ls, tl, tw);
    else load_twiddles<R, 2>(wt, lk, ls, tl, tw);
    const int pNs = 1 << (ls - 3);                 // the previous pass: radix 8 after pNs points
    const int base = ((tl >> (ls - 3)) << ls) + (tl & (pNs - 1));
    __syncthreads();                               // the buffer is no longer read
#pragma unroll
    for (int r = 0; r < 8; ++r) x[4 * lds_cell(base + (r << (ls - 3))) + ch] = v[r];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = x[4 * lds_cell(tl + (q << (lk - 3))) + ch];
    if (rem >= 3) butterflies<R, 8, INV>(v, wt);
    else if (rem == 2) butterflies<R, 4, INV>(v, wt);
    else butterflies<R, 2, INV>(v, wt);
  }
}

// The value of lane ^ 1 (X = 1) or lane ^ 2 (X = 2), by a DPP lane move.
template <int X, typename V>
__device__ __forceinline__ V quad_xor(V v) {
  union { V v; int w[sizeof(V) / 4]; } a, b;
  a.v = v;
#pragma unroll
  for (int k = 0; k < (int)(sizeof(V) / 4); ++k) b.w[k] = __builtin_amdgcn_mov_dpp(a.w[k], X == 1 ? 0xB1 : 0x4E, 0xf, 0xf, true);
  return b.v;
}
// Transposes the 4 x 4 values of four adjacent lanes: lane j's a[i] becomes lane i's a[j].
template <typename R>
__device__ __forceinline__ void quad_transpose(R* a) {
  const bool h1 = threadIdx.x & 1, h2 = threadIdx.x & 2;
#pragma unroll
  for (int i = 0; i < 4; i += 2) {
    const R t = quad_xor<1>(h1 ? a[i] : a[i + 1]);
    a[i] = h1 ? t : a[i];
    a[i + 1] = h1 ? a[i + 1] : t;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const R t = quad_xor<2>(h2 ? a[i] : a[i + 2]);
    a[i] = h2 ? t : a[i];
    a[i + 2] = h2 ? a[i + 2] : t;
  }
}

template <typename R>
__device__ inline Cell<R> zero_cell() {
  Cell<R> c;
#pragma unroll
  for (int s = 0; s < 4; ++s) c.s[s] = cmk(R(0), R(0));
  return c;
}

// PASS: 0 = P4 image rows -> half, 1 = P5 half -> grid, 2 = P8 grid -> half, 3 = P9 half -> image,
// 4 = P9, P1 and P4 of the next iteration in one pass: half -> inverse row FFT -> Re phi^dagger B
// of the row's pixels (kept in registers) -> primal step -> X -> forward row FFT -> half.
// PM >= 0 (PASS 0 and 4): the primal step of mode PM runs on each pixel before the row FFT, which
// takes the X it returns (P1 fused into P4).
// items: {prob, first line, -, -}; CELLS/K lines per workgroup.
template <typename R, int CELLS, int PASS>
struct FftSmem {
  static constexpr int kTslMax = CELLS / 256 + 2048 / 8;
  Cell<R> lds[CELLS + CELLS / 8];
  double red[PASS == 2 ? 2 * ((CELLS / 2 + 63) / 64) : 1];
  int2 tsl[PASS == 2 ? kTslMax : 1];
  int tbx[PASS == 2 ? kTslMax : 1];
};
template <typename R, int CELLS, int PASS, int PM = -1>
__device__ __forceinline__ void fft_pass(const ProbDesc& P, const int4 it, int src_slot, int dst_slot,
                                         FftSmem<R, CELLS, PASS>& sm) {
  if (halted(P)) return;                 // stopped by an adaptive run
  Cell<R>* lds = sm.lds;
  const int n = P.n, K = P.K;
  const int lines = CELLS / K;
  const int lgK = lg2(K);                // all powers of two
  const int line0 = it.y;
  const R* __restrict__ s = (const R*)P.deapod;
  cplx<R>* __restrict__ half = (cplx<R>*)P.half;       // cell c, channel ch at 4 c + ch
  cplx<R>* __restrict__ grid = (cplx<R>*)P.grid;
  const cplx<R>* __restrict__ tw = (const cplx<R>*)P.twiddle;
  constexpr int nthr = CELLS / 2;
  // the thread's line, channel and cells tl + q K/8; the pixel its quad lane takes in the pointwise
  // steps is that of the cell q = 0, 1, 6 or 7: column (k + n/2) mod K, since pixel j lies at
  // grid index (j - n/2) mod K
  const int ch = threadIdx.x & 3, grp = threadIdx.x >> 2;
  const int l = grp >> (lgK - 3), tl = grp & ((K >> 3) - 1);
  const int line = line0 + l, e = K >> 3;              // e = n / 4
  cplx<R>* x = (cplx<R>*)lds + 4 * lds_cell(l * K);
  const int col = tl + (ch < 2 ? ch + 2 : ch - 2) * e;
  const bool live = line < (PASS == 1 || PASS == 2 ? K : n);
  cplx<R> v[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) v[q] = cmk(R(0), R(0));

  // the partial-slot table and the slot-box unions of the gridding tiles this workgroup's lines
  // read (their tile rows and the rows before them), staged once so the per-cell gathers index LDS
  int2* tsl = sm.tsl;
  int* tbx = sm.tbx;
  double* red = sm.red;
  int trow0 = 0;
  R gfac = R(1);
  if (PASS == 2) {
    // the factor of the gridded values (src_slot: 0 the one the grid pass stored; 1 the l2-ball
    // factor c = rho2 max(0, 1 - epsilon / ||Bv||) from the per-chunk partials of ||Bv||^2,
    // reduced by every workgroup in the same fixed order and stored, with ||Bv||^2, by the
    // problem's first; 2 one; 3 the first or the second, by the problem's chunk_norm)
    // The sum shares the staging's barrier: its wave totals go to LDS with the tables, and the
    // factor is worked out while the gathers are in flight.
    if (src_slot == 3) src_slot = P.chunk_norm;
    const int ntg = P.ntile_side_g;
    trow0 = line0 / kGridTile - 1;
    const int ntr = min(K - 1, line0 + lines - 1) / kGridTile - trow0 + 1;
    const double* __restrict__ parts = chunk_partials(P);
    const int nparts = src_slot == 1 ? P.n_slots : 0;
    auto tile_at = [&](int i) { return (i & (ntg - 1)) * ntg + ((trow0 + (i >> lg2(ntg)) + ntg) & (ntg - 1)); };
    int2 sl0 = make_int2(0, 0);
    int bx0 = 0;
    if (threadIdx.x < ntr * ntg) {
      sl0 = P.tile_slots[tile_at(threadIdx.x)];
      bx0 = P.tile_box[tile_at(threadIdx.x)];
    }
    if (src_slot == 1) {
      KSum k;
      for (int i = threadIdx.x; i < nparts; i += nthr) {
        KSum o; o.s = parts[2 * i]; o.c = parts[2 * i + 1]; k.merge(o);
      }
      k = wave_reduce(k);
      if ((threadIdx.x & 63) == 0) { red[2 * (threadIdx.x >> 6)] = k.s; red[2 * (threadIdx.x >> 6) + 1] = k.c; }
    }
    for (int i = threadIdx.x; i < ntr * ntg; i += nthr) {
      tsl[i] = i == threadIdx.x ? sl0 : P.tile_slots[tile_at(i)];
      tbx[i] = i == threadIdx.x ? bx0 : P.tile_box[tile_at(i)];
    }
    __syncthreads();
    if (src_slot == 1) {
      KSum t;
      for (int w = 0; w < (nthr + 63) >> 6; ++w) { KSum o; o.s = red[2 * w]; o.c = red[2 * w + 1]; t.merge(o); }
      const double v2 = t.value();
      const double vn = sqrt(v2);
      const double c = (vn > P.eps) ? P.rho2 * (1.0 - P.eps / vn) : 0.0;
      if (line0 == 0 && threadIdx.x == 0) {
        P.scal[SC_CFAC] = c;
        P.scal[SC_VNORM2] = v2;
        P.scal[SC_GFAC] = c;
      }
      gfac = R(c);
    } else if (src_slot == 0) {
      gfac = R(P.scal[SC_GFAC]);
    }
  }
  // P9 + P1 + P4: the primal step's inputs of the thread's pixel are requested now, so their loads
  // overlap the loads and the inverse FFT below (not by FP64's 1024 threads, whose 128 registers
  // would spill them)
  constexpr bool kPrefetch = PASS == 4 && !(sizeof(R) == 8 && CELLS > 1024);
  PrimalIn<R> pin;
  if constexpr (kPrefetch) {
    if (live) pin = primal_load<R, (PM < 0 ? 0 : PM)>(P, line * n + col);
  }
  // ---- load ----
  // (the FP64 kernel with 1024 threads, 128 registers, keeps the gather one pair at a time: the
  // eight pairs' cells in flight would spill)
  constexpr bool kRounds = PASS == 2 && !(sizeof(R) == 8 && CELLS > 1024);
  if constexpr (kRounds) {
    // the gridded values of the thread's cells q and q + nthr: the partial slots of each cell's
    // tile and of the tiles whose halos reach it (the previous tile in k1, in k2, and in both),
    // times the factor the gridding pass left out.  Each (cell, tile) pair's first slot cell and
    // slot count come from the staged tables; the slots are then added round by round (slot
    // index sl of every pair, pairs in a fixed order), and a round loads all eight pairs' cells
    // before adding any (a pair with fewer slots, or none, loads a cell of an existing slot that
    // it does not add), so those loads are in flight together
    const int ntg = P.ntile_side_g, RG = kGridTile + P.T - 1;
    const Cell<R>* __restrict__ gp = (const Cell<R>*)P.gpart;
    const Cell<R>* src[2][4];
    int cnt[2][4];
    int rounds = 0;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const int q = threadIdx.x + u * nthr;
      const int l = q >> lgK, k = q & (K - 1), k2 = line0 + l;
      const int t1 = k / kGridTile, t2 = k2 / kGridTile, a1 = k - t1 * kGridTile, a2 = k2 - t2 * kGridTile;
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const int d1 = d & 1, d2 = d >> 1;
        const int o1 = a1 + d1 * kGridTile, o2 = a2 + d2 * kGridTile;
        src[u][d] = gp;
        cnt[u][d] = 0;
        if (k2 >= K || o1 >= RG || o2 >= RG) continue;
        const int ti = (t2 - d2 - trow0) * ntg + ((t1 - d1 + ntg) & (ntg - 1));
        if (!in_box(tbx[ti], o1, o2)) continue;          // no slot of the tile reaches it
        const int2 ts = tsl[ti];
        src[u][d] = gp + (size_t)ts.x * RG * RG + o2 * RG + o1;
        cnt[u][d] = ts.y;
        rounds = max(rounds, ts.y);
      }
    }
    Cell<R> c[2] = {zero_cell<R>(), zero_cell<R>()};
    for (int sl = 0; sl < rounds; ++sl) {
      Cell<R> o[2][4];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int d = 0; d < 4; ++d) o[u][d] = src[u][d][sl < cnt[u][d] ? (size_t)sl * RG * RG : 0];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int d = 0; d < 4; ++d)
          if (sl < cnt[u][d]) {
#pragma unroll
            for (int ch = 0; ch < 4; ++ch) c[u].s[ch] = cadd(c[u].s[ch], o[u][d].s[ch]);
          }
    }
#pragma unroll
    for (int u = 0; u < 2; ++u) {
#pragma unroll
      for (int ch = 0; ch < 4; ++ch) { c[u].s[ch].re *= gfac; c[u].s[ch].im *= gfac; }
      lds[lds_cell(threadIdx.x + u * nthr)] = c[u];
    }
  }
  if constexpr (PASS == 2 && !kRounds) {
    for (int q = threadIdx.x; q < CELLS; q += nthr) {
      Cell<R> c = zero_cell<R>();
      // the gathers one (cell, tile) pair at a time, in the order of the rounds above
      const int ql = q >> lgK, k = q & (K - 1), k2 = line0 + ql;
      if (k2 < K) {
        const int ntg = P.ntile_side_g, RG = kGridTile + P.T - 1;
        const int t1 = k / kGridTile, t2 = k2 / kGridTile, a1 = k - t1 * kGridTile, a2 = k2 - t2 * kGridTile;
        const Cell<R>* src[4];
        int cnt[4], rounds = 0;
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const int d1 = d & 1, d2 = d >> 1;
          const int o1 = a1 + d1 * kGridTile, o2 = a2 + d2 * kGridTile;
          src[d] = (const Cell<R>*)P.gpart;
          cnt[d] = 0;
          if (o1 >= RG || o2 >= RG) continue;
          const int ti = (t2 - d2 - trow0) * ntg + ((t1 - d1 + ntg) & (ntg - 1));
          if (!in_box(tbx[ti], o1, o2)) continue;
          const int2 ts = tsl[ti];
          src[d] = (const Cell<R>*)P.gpart + (size_t)ts.x * RG * RG + o2 * RG + o1;
          cnt[d] = ts.y;
          rounds = max(rounds, ts.y);
        }
        for (int sl = 0; sl < rounds; ++sl)
#pragma unroll
          for (int d = 0; d < 4; ++d)
            if (sl < cnt[d]) {
              const Cell<R> o = src[d][(size_t)sl * RG * RG];
#pragma unroll
              for (int ch = 0; ch < 4; ++ch) c.s[ch] = cadd(c.s[ch], o.s[ch]);
            }
#pragma unroll
        for (int ch = 0; ch < 4; ++ch) { c.s[ch].re *= gfac; c.s[ch].im *= gfac; }
      }
      lds[lds_cell(q)] = c;
    }
  }
  if constexpr (PASS == 2) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 8; ++q) v[q] = x[4 * lds_cell(tl + q * e) + ch];
  }
  // (cells 0 and 1 hold rows n/2 .., cells 6 and 7 rows 0 .. of the half-transformed columns)
  if constexpr (PASS == 1) {
    if (live) {
      const cplx<R>* h = half + 4 * ((size_t)line * n + tl) + ch;
      v[0] = h[4 * (2 * e)]; v[1] = h[4 * (3 * e)]; v[6] = h[0]; v[7] = h[4 * e];
    }
  }
  if constexpr (PASS >= 3) {
    if (live) {
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = half[4 * ((size_t)(tl + q * e) * n + line) + ch];
    }
  }
  // P4: the thread's pixel of X (with PM the primal step's X), deapodised
  const R sc = (PASS == 0 || PASS >= 3) && live ? s[line] * s[col] : R(0);
  if constexpr (PASS == 0) {
    R a[4] = {R(0), R(0), R(0), R(0)};
    if (live) {
      V4<R> p;
      if constexpr (PM >= 0) p = primal_pixel<R, (PM < 0 ? 0 : PM)>(P, line * n + col);
      else p = ((const V4<R>*)P.img[src_slot])[(size_t)line * n + col];
      a[0] = p.x * sc; a[1] = p.y * sc; a[2] = p.z * sc; a[3] = p.w * sc;
    }
    quad_transpose(a);
    v[0].re = a[0]; v[1].re = a[1]; v[6].re = a[2]; v[7].re = a[3];
  }
  fft_line<R, PASS >= 2>(v, x, lgK, tl, ch, tw);

  if constexpr (PASS >= 3) {
    // crop, Z^dagger and Re give Re phi^dagger B at the thread's pixel (rounded products, not
    // contracted into the primal step's sums: the result is bitwise the one of the separate
    // passes, which store Re phi^dagger B and read it back)
    R a[4] = {v[0].re, v[1].re, v[6].re, v[7].re};
    quad_transpose(a);
    V4<R> g;
    g.x = mul_rn(a[0], sc); g.y = mul_rn(a[1], sc); g.z = mul_rn(a[2], sc); g.w = mul_rn(a[3], sc);
    if constexpr (PASS == 3) {
      if (live) ((V4<R>*)P.img[dst_slot])[(size_t)line * n + col] = g;
      return;
    } else {
      // the primal step takes it, and its X, deapodised and zero-padded, is the row's new input
      a[0] = a[1] = a[2] = a[3] = R(0);
      if (live) {
        if constexpr (!kPrefetch) pin = primal_load<R, (PM < 0 ? 0 : PM)>(P, line * n + col);
        const V4<R> p = primal_pixel_in<R, (PM < 0 ? 0 : PM)>(P, line * n + col, g, pin);
        a[0] = p.x * sc; a[1] = p.y * sc; a[2] = p.z * sc; a[3] = p.w * sc;
      }
      quad_transpose(a);
#pragma unroll
      for (int q = 0; q < 8; ++q) v[q] = cmk(R(0), R(0));
      v[0].re = a[0]; v[1].re = a[1]; v[6].re = a[2]; v[7].re = a[3];
      fft_line<R, false>(v, x, lgK, tl, ch, tw);
    }
  }

  // ---- store ----
  if (!live) return;
  if constexpr (PASS == 0 || PASS == 4) {
#pragma unroll
    for (int q = 0; q < 8; ++q) half[4 * ((size_t)(tl + q * e) * n + line) + ch] = v[q];
  } else if constexpr (PASS == 1) {
#pragma unroll
    for (int q = 0; q < 8; ++q) grid[4 * ((size_t)line * K + tl + q * e) + ch] = v[q];
  } else {
    cplx<R>* h = half + 4 * ((size_t)line * n + tl) + ch;
    h[4 * (2 * e)] = v[0]; h[4 * (3 * e)] = v[1]; h[0] = v[6]; h[4 * e] = v[7];
  }
}

}  // namespace psara
