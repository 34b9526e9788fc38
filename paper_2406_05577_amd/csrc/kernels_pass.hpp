// Axis-pass kernel for gfx950: the lines of one axis, n = R1*R2, sphere or
// scratch on one side and a dense array on the other.
//
// The three passes of a direction (Section 2.2: the padding staged one axis at
// a time) are the same kernel with other addresses:
//   z: the sphere, through the (column, z) table  <->  columns [z][slot][band]
//   y: the columns, through the (slab, y) table   <->  slab planes [y][slab][band]
//   x: the slab planes, through the x table       <->  the grid [y][x][band]
// Inverse passes gather through the table (zeros where it has no entry) and
// write dense; forward passes read dense and scatter what the table keeps.
// The bands of neighbouring lines are contiguous in every array, so a tile
// takes fc consecutive elements of the flattened (line, band) dimension (for
// x: of the bands, and several rows where the bands are few).
//
// Each thread holds R1, then R2, values of one line: DFT_R1 over stride R2,
// twiddles w_n^{i*k} from a table in LDS, an exchange through LDS, DFT_R2
// (Section 2.1). The rows of the exchange are an odd number of pieces apart
// so that the rows a wave reads together start in other banks.
//
// Bound by memory: a pass reads and writes each value once (2.4 flop per byte
// moved at 200 points), with enough workgroups in flight: the exchange sends the
// real and the imaginary parts one after the other, half the LDS for two more
// barriers (144x160x180, 128 complex128 bands, a round trip: 8.80 -> 7.80 ms).
// The y and x passes run over groups of planes whose slab scratch stays in the
// last-level cache between the two, with the grid streamed past it
// (non-temporal): a copy of that shape moved 6.7 TB/s, against 4.5 TB/s over the
// whole scratch at once. At 200x192x216, 20 complex128 bands, the x passes move
// 5.6 TB/s and a round trip takes 2.34 ms (87 ms on the LDS-stage kernels).
#pragma once

#include "bline.hpp"
#include "device_common.hpp"
#include "pass.hpp"

namespace fftb {

template <bool NT, typename T>
__device__ __forceinline__ cpx<T> ld_c(const cpx<T>* p) {
  typedef T v2 __attribute__((ext_vector_type(2)));
  v2 x;
  if constexpr (NT) x = __builtin_nontemporal_load(reinterpret_cast<const v2*>(p));
  else x = *reinterpret_cast<const v2*>(p);
  return {x.x, x.y};
}
template <bool NT, typename T>
__device__ __forceinline__ void st_c(cpx<T>* p, cpx<T> v) {
  typedef T v2 __attribute__((ext_vector_type(2)));
  if constexpr (NT) __builtin_nontemporal_store(v2{v.re, v.im}, reinterpret_cast<v2*>(p));
  else *reinterpret_cast<v2*>(p) = v2{v.re, v.im};
}
// Run f with the uniform flag nt as a constant. The fences keep the compiler
// from merging the two copies, which would drop the non-temporal hint.
template <class F>
__device__ __forceinline__ void with_nt(bool nt, F&& f) {
  if (nt) {
    asm volatile("; streaming" ::: "memory");
    f(std::true_type{});
    asm volatile("; end streaming" ::: "memory");
  } else {
    asm volatile("; cached" ::: "memory");
    f(std::false_type{});
    asm volatile("; end cached" ::: "memory");
  }
}

// floor(n / d) for 0 <= n < 2^22 through a float reciprocal and one correction
__device__ __forceinline__ int pass_div(int n, int d, float inv_d) {
  int q = static_cast<int>(static_cast<float>(n) * inv_d);
  const int rem = n - q * d;
  q += (rem >= d) - (rem < 0);
  return q;
}

template <int S, typename T, int N>
__global__ void __launch_bounds__(pass_max_threads(N, sizeof(T) == 8)) pass_kernel(const PassArgs a) {
  constexpr int R1 = pass_r1(N), R2 = N / R1, RS = R2 | 1;
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* buf = reinterpret_cast<T*>(smem_raw);
  TwEntry<T>* tw = reinterpret_cast<TwEntry<T>*>(smem_raw + a.lds_tw);

  // the tile: sphere, first element f0 of nf, rows, and the two sides' bases
  const int t = static_task_g(a.total, a.group);
  if (t < 0) return;
  int s = 0, f0, nf, nl = 1, trow = N;
  const int32_t* __restrict__ tab = a.tab;
  const cpx<T>* src = reinterpret_cast<const cpx<T>*>(a.src);
  cpx<T>* dst = reinterpret_cast<cpx<T>*>(a.dst);
  int64_t gat, den, pstride, vrow = 0;
  int gstep = 0, dstep = 0;
  if (a.kind == kPassZ) {
    while (s + 1 < a.nsph && t >= a.sph[s + 1].ztile) ++s;
    const PassSph d = a.sph[s];
    f0 = (t - d.ztile) * a.fc;
    nf = d.ncol * d.nb;
    tab += d.gidx_off;
    gat = d.sph_off;
    den = d.col_off;
    pstride = d.colrow;
  } else {
    const int ft = t % a.tiles, rest = t / a.tiles;
    const int pl = a.kind == kPassX ? rest / a.rtiles : rest;  // plane within the group
    const int p = a.p0 + pl;
    s = p / a.nz;
    const int z = p - s * a.nz;
    const PassSph d = a.sph[s];
    f0 = ft * a.fc;
    if (a.kind == kPassY) {
      nf = d.nslab * d.nb;
      tab += d.colidx_off;
      gat = d.col_off + static_cast<int64_t>(z) * d.colrow;
      den = static_cast<int64_t>(pl) * a.splane;
      pstride = d.srow;
    } else {
      const int y0 = (rest - pl * a.rtiles) * a.lines;
      nl = min(a.lines, a.ny - y0);
      nf = d.nb;
      trow = 0;
      tab += d.xinv_off;
      gat = static_cast<int64_t>(pl) * a.splane + static_cast<int64_t>(y0) * d.srow;
      gstep = d.srow;
      vrow = (static_cast<int64_t>(z) * a.ny + y0) * N;
      den = d.grid_off + vrow * d.nb;
      dstep = N * d.nb;
      pstride = d.nb;
    }
    if (f0 >= nf) return;
  }
  const int nb = a.sph[s].nb;
  const int fc = a.fc, nfl = min(fc, nf - f0);
  const float inv_fc = 1.0f / static_cast<float>(fc), inv_nb = 1.0f / static_cast<float>(nb);
  const int c0 = f0 / nb, b0 = f0 - c0 * nb;  // line and band of element f0
  const cpx<T>* gsrc = src + gat;             // inverse: gathered, forward: dense
  const cpx<T>* dsrc = src + den + f0;
  cpx<T>* gdst = dst + gat;
  cpx<T>* ddst = dst + den + f0;
  const bool ntd = a.nt_dense != 0, ntg = a.nt_gather != 0;

  // stage 1: thread (f, i, l) takes positions i + R2*q of line l
  const int items1 = a.lines * R2 * fc;
  cpx<T> v[R1];
  auto load = [&](int it) {
    const int rest = pass_div(it, fc, inv_fc);
    const int f = it - rest * fc, l = rest / R2, i = rest - l * R2;
    const bool ok = f < nfl && l < nl;
    if constexpr (S > 0) {
      const int bb = b0 + (ok ? f : 0);
      const int dc = pass_div(bb, nb, inv_nb);
      const int32_t* __restrict__ row = tab + static_cast<int64_t>(c0 + dc) * trow + i;
      const cpx<T>* base = gsrc + (bb - dc * nb) + l * gstep;
      int g[R1];
#pragma unroll
      for (int q = 0; q < R1; ++q) g[q] = ok ? row[R2 * q] : -1;
      with_nt(ntg, [&](auto nt) {
#pragma unroll
        for (int q = 0; q < R1; ++q)
          v[q] = g[q] >= 0 ? ld_c<decltype(nt)::value>(base + static_cast<int64_t>(g[q]) * nb)
                           : cpx<T>{0, 0};
      });
    } else {
      const cpx<T>* base = dsrc + f + i * pstride + static_cast<int64_t>(l) * dstep;
      with_nt(ntd, [&](auto nt) {
#pragma unroll
        for (int q = 0; q < R1; ++q)
          v[q] = ok ? ld_c<decltype(nt)::value>(base + (R2 * q) * pstride) : cpx<T>{0, 0};
      });
    }
  };
  // stage 2 (or the only stage): thread (f, k1, l) writes positions k1 + R1*k2
  auto emit = [&](int f, int l, int k1, auto& u, auto stride_c, auto count_c) {
    constexpr int ST = decltype(stride_c)::value, CT = decltype(count_c)::value;
    if (f >= nfl || l >= nl) return;
    if constexpr (S > 0) {
      if (a.pot) {
        const T* __restrict__ vr = reinterpret_cast<const T*>(a.pot) + vrow + static_cast<int64_t>(l) * N + k1;
#pragma unroll
        for (int k = 0; k < CT; ++k) u[k] = cscale(u[k], vr[ST * k]);
      }
      cpx<T>* base = ddst + f + k1 * pstride + static_cast<int64_t>(l) * dstep;
      with_nt(ntd, [&](auto nt) {
#pragma unroll
        for (int k = 0; k < CT; ++k) st_c<decltype(nt)::value>(base + (ST * k) * pstride, u[k]);
      });
    } else {
      const int bb = b0 + f;
      const int dc = pass_div(bb, nb, inv_nb);
      const int32_t* __restrict__ row = tab + static_cast<int64_t>(c0 + dc) * trow + k1;
      cpx<T>* base = gdst + (bb - dc * nb) + l * gstep;
      const T sc = static_cast<T>(a.scale);
      int g[CT];
#pragma unroll
      for (int k = 0; k < CT; ++k) g[k] = row[ST * k];
      with_nt(ntg, [&](auto nt) {
#pragma unroll
        for (int k = 0; k < CT; ++k)
          if (g[k] >= 0) st_c<decltype(nt)::value>(base + static_cast<int64_t>(g[k]) * nb, cscale(u[k], sc));
      });
    }
  };

  if constexpr (R2 == 1) {
    for (int it = threadIdx.x; it < items1; it += blockDim.x) {
      load(it);
      dft<R1, S>(v);
      const int l = pass_div(it, fc, inv_fc);
      emit(it - l * fc, l, 0, v, std::integral_constant<int, 1>{}, std::integral_constant<int, R1>{});
    }
    return;
  } else {
    // (the host gives every item of either stage its own thread)
    const int it = threadIdx.x;
    const bool on1 = it < items1;
    if (on1) load(it);
    bl_fill_twiddles<S, T>(tw, reinterpret_cast<const cpx<T>*>(a.root),
                           reinterpret_cast<const cpx<T>*>(a.root_lo), R1, R2);
    __syncthreads();
    const int rest1 = pass_div(it, fc, inv_fc);
    const int f = it - rest1 * fc;
    const int l1 = rest1 / R2, i1 = rest1 - l1 * R2;
    const int l2 = rest1 / R1, k1 = rest1 - l2 * R1;
    const bool on2 = it < a.lines * R1 * fc;
    if (on1) {
      dft<R1, S>(v);
      const TwEntry<T>* tr = tw + i1 * tw_row_stride(R1);
#pragma unroll
      for (int k = 1; k < R1; ++k) {
        const TwEntry<T> w = tr[k];
        if constexpr (std::is_same<T, float>::value)
          v[k] = cmul_hl(v[k], cpx<float>{w.re, w.im}, cpx<float>{w.lre, w.lim});
        else
          v[k] = cmul(v[k], cpx<double>{w.re, w.im});
      }
    }
    T* out = buf + (l1 * R1 * RS + i1) * fc + f;
    const T* in = buf + (l2 * R1 + k1) * RS * fc + f;
    cpx<T> u[R2];
    if (on1) {
#pragma unroll
      for (int k = 0; k < R1; ++k) out[k * RS * fc] = v[k].re;
    }
    __syncthreads();
    if (on2) {
#pragma unroll
      for (int i = 0; i < R2; ++i) u[i].re = in[i * fc];
    }
    __syncthreads();
    if (on1) {
#pragma unroll
      for (int k = 0; k < R1; ++k) out[k * RS * fc] = v[k].im;
    }
    __syncthreads();
    if (on2) {
#pragma unroll
      for (int i = 0; i < R2; ++i) u[i].im = in[i * fc];
      dft<R2, S>(u);
      emit(f, l2, k1, u, std::integral_constant<int, R1>{}, std::integral_constant<int, R2>{});
    }
  }
}

// Lengths compiled, by translation-unit part.
#define FFTB_PASS_LENGTHS_0(X) \
  X(1) X(2) X(3) X(4) X(5) X(6) X(8) X(9) X(10) X(12) X(15) X(16) X(18) X(20) X(24) X(25) X(27) \
  X(30) X(32) X(36) X(40) X(45) X(48) X(50) X(54) X(60)
#define FFTB_PASS_LENGTHS_1(X) \
  X(64) X(72) X(75) X(80) X(81) X(90) X(96) X(100) X(108) X(120) X(125) X(128) X(135) X(144)
#define FFTB_PASS_LENGTHS_2(X) \
  X(150) X(160) X(162) X(180) X(192) X(200) X(216) X(225) X(240) X(243) X(250) X(256)
#define FFTB_PASS_LENGTHS_3(X) \
  X(270) X(288) X(300) X(320) X(324) X(360) X(375) X(384) X(400) X(405) X(432) X(450) X(480) \
  X(486) X(500) X(512)

template <int S, typename T, int N>
hipError_t pass_one(const PassArgs& a, int threads, size_t lds, hipStream_t st, bool attr_only) {
  if (attr_only)
    return hipFuncSetAttribute(reinterpret_cast<const void*>(pass_kernel<S, T, N>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  hipLaunchKernelGGL((pass_kernel<S, T, N>), dim3(pass_grid(a.total, a.group)), dim3(threads), lds, st, a);
  return hipGetLastError();
}

// Launch (or, with attr_only, allow `lds` bytes to) the kernel of length n if
// part P compiles it; *found tells.
template <int S, typename T, int P>
hipError_t pass_part(int n, const PassArgs& a, int threads, size_t lds, hipStream_t st,
                     bool attr_only, bool* found) {
  *found = true;
#define FFTB_X(n_) \
  case n_: return pass_one<S, T, n_>(a, threads, lds, st, attr_only);
  if constexpr (P == 0) {
    switch (n) { FFTB_PASS_LENGTHS_0(FFTB_X) }
  } else if constexpr (P == 1) {
    switch (n) { FFTB_PASS_LENGTHS_1(FFTB_X) }
  } else if constexpr (P == 2) {
    switch (n) { FFTB_PASS_LENGTHS_2(FFTB_X) }
  } else {
    switch (n) { FFTB_PASS_LENGTHS_3(FFTB_X) }
  }
#undef FFTB_X
  *found = false;
  return hipErrorInvalidValue;
}

#define FFTB_PASS_INST(EXT, S, T, P)                                                             \
  EXT template hipError_t pass_part<S, T, P>(int, const PassArgs&, int, size_t, hipStream_t, bool, \
                                             bool*);

}  // namespace fftb
