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
// Each thread holds R1, then R2, values of one line (complex64: of two
// neighbouring bands, 16 bytes per lane): DFT_R1 over stride R2, twiddles
// w_n^{i*k} from a table in LDS, an exchange through LDS, DFT_R2 (Section 2.1).
// The rows of the exchange are an odd number of pieces apart so that the rows a
// wave reads together start in other banks. The tile's table rows are staged in
// LDS as byte offsets where they are few: one coalesced load in the place of R1
// loads per thread, and buffer accesses that need no branch for absent entries.
//
// The potential step's x pass (POT) multiplies the inverse's rows by V on their
// way to the grid and transforms them back in the same workgroup, into the slab
// row that they came from: the grid is written but not read again. 144x160x180,
// 128 complex128 bands: 2.6 ms, where the forward's x pass alone takes 2.2; the
// whole step 5.2 ms, 7.3 as two directions. Arrays of their own after the second
// exchange keep it at 90 registers: with va and vb taken again, live wherever a
// lane has no item, it held 132, a wave less per SIMD, and took 3.8 ms.
//
// Bound by memory: a pass reads and writes each value once (2.4 flop per byte
// moved at 200 points), with enough workgroups in flight: the exchange sends the
// real and the imaginary parts one after the other, half the LDS for two more
// barriers (a round trip 11 % faster at 144x160x180, 128 complex128 bands). The y
// and x passes run over groups of planes whose slab scratch stays in the
// last-level cache between the two, with the grid streamed past it
// (non-temporal): a copy of that shape moved 6.7 TB/s, against 4.5 TB/s over the
// whole scratch at once. At 144^3, 96 complex64 bands, the inverse x, y and z
// passes move 6.1, 5.6 and 5.3 TB/s. Two complex64 bands per lane and staged
// tables are worth 8-14 % (128^3, 108x100x120), staged tables alone 3 % (complex128,
// 144x160x180). At 200x192x216, 20 complex128 bands, a round trip takes 2.26 ms (87
// ms on the LDS-stage kernels).
#pragma once

#include "bline.hpp"
#include "device_common.hpp"
#include "pass.hpp"

namespace fftb {

// One element of a lane: V neighbouring bands (16 bytes: one complex128 or two
// complex64 values, or 8 bytes), at any address that a value may have.
template <typename T, int V>
struct ElemVec {
  typedef T type __attribute__((ext_vector_type(2 * V), aligned(8)));
  // what stores write
  typedef int words __attribute__((ext_vector_type(V * sizeof(T) / 2), aligned(8)));
};
template <typename T, int V>
struct Elem {
  cpx<T> a, b;  // (b: V == 2)
};
template <int V, typename T, typename E>
__device__ __forceinline__ Elem<T, V> unpack(E x) {
  if constexpr (V == 1) return {{x.x, x.y}, {0, 0}};
  else return {{x.x, x.y}, {x.z, x.w}};
}
template <int V, typename T>
__device__ __forceinline__ typename ElemVec<T, V>::words pack(T ar, T ai, T br, T bi) {
  if constexpr (std::is_same<T, double>::value) {
    const long long re = __double_as_longlong(ar), im = __double_as_longlong(ai);
    return {static_cast<int>(re), static_cast<int>(re >> 32), static_cast<int>(im), static_cast<int>(im >> 32)};
  } else if constexpr (V == 1) {
    return {__float_as_int(ar), __float_as_int(ai)};
  } else {
    // (opaque: the compiler would read ar and ai back from their array as one
    // wide load, which keeps the array in scratch memory)
    asm("" : "+v"(ar));
    return {__float_as_int(ar), __float_as_int(ai), __float_as_int(br), __float_as_int(bi)};
  }
}
template <bool NT, int V, typename T>
__device__ __forceinline__ Elem<T, V> ld_el(const cpx<T>* p) {
  using E = typename ElemVec<T, V>::type;
  if constexpr (NT) return unpack<V, T>(__builtin_nontemporal_load(reinterpret_cast<const E*>(p)));
  else return unpack<V, T>(*reinterpret_cast<const E*>(p));
}
template <bool NT, int V, typename T>
__device__ __forceinline__ void st_el(cpx<T>* p, T ar, T ai, T br, T bi) {
  using E = typename ElemVec<T, V>::words;
  if constexpr (NT) __builtin_nontemporal_store(pack<V>(ar, ai, br, bi), reinterpret_cast<E*>(p));
  else *reinterpret_cast<E*>(p) = pack<V>(ar, ai, br, bi);
}
// The same through a buffer of 2 GiB: an offset at or past its end reads zero
// and stores nothing, so absent table entries need no branch.
constexpr unsigned kPassAbsent = 0x80000000u;
__device__ __forceinline__ __amdgpu_buffer_rsrc_t pass_rsrc(const void* base) {
  const uint64_t pa = reinterpret_cast<uint64_t>(base);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(pa));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(pa >> 32));
  void* p = reinterpret_cast<void*>((static_cast<uint64_t>(hi) << 32) | lo);
  return __builtin_amdgcn_make_buffer_rsrc(p, static_cast<short>(0), static_cast<int>(kPassAbsent),
                                           0x00020000);
}
template <bool NT, int V, typename T>
__device__ __forceinline__ Elem<T, V> buf_ld_el(__amdgpu_buffer_rsrc_t r, unsigned off, unsigned soff) {
  typedef T E __attribute__((ext_vector_type(2 * V)));
  if constexpr (sizeof(E) == 16)
    return unpack<V, T>(__builtin_bit_cast(E, __builtin_amdgcn_raw_buffer_load_b128(r, off, soff, NT ? 2 : 0)));
  else
    return unpack<V, T>(__builtin_bit_cast(E, __builtin_amdgcn_raw_buffer_load_b64(r, off, soff, NT ? 2 : 0)));
}
// (No scalar offset here, nor in buf_store: the compiler takes a 16-byte store with
// one to have read its data a cycle earlier and lets the next instruction overwrite
// them, which on gfx950 changed the first word of a few lanes in one of 15 inverse
// transforms of 60x54x50, 16 complex64 bands. Without one it waits.)
template <bool NT, int V, typename T>
__device__ __forceinline__ void buf_st_el(__amdgpu_buffer_rsrc_t r, T ar, T ai, T br, T bi, unsigned off) {
  const typename ElemVec<T, V>::words x = pack<V>(ar, ai, br, bi);
  if constexpr (sizeof(x) == 16) __builtin_amdgcn_raw_buffer_store_b128(x, r, off, 0, NT ? 2 : 0);
  else __builtin_amdgcn_raw_buffer_store_b64(x, r, off, 0, NT ? 2 : 0);
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

// the real or imaginary parts of an element (opaque as in pack)
template <int V, typename T>
__device__ __forceinline__ auto parts(T a, T b) {
  typedef T P __attribute__((ext_vector_type(V)));
  if constexpr (V == 1) {
    return P{a};
  } else {
    asm("" : "+v"(a));
    return P{a, b};
  }
}

// floor(n / d) for 0 <= n < 2^22 through a float reciprocal and one correction
__device__ __forceinline__ int pass_div(int n, int d, float inv_d) {
  int q = static_cast<int>(static_cast<float>(n) * inv_d);
  const int rem = n - q * d;
  q += (rem >= d) - (rem < 0);
  return q;
}

template <int S, typename T, int V, int N, bool POT>
__global__ void __launch_bounds__(pass_max_threads(N, sizeof(T) * V == 4)) pass_kernel(const PassArgs a) {
  constexpr int R1 = pass_r1(N), R2 = N / R1, RS = R2 | 1;
  constexpr unsigned es = sizeof(cpx<T>);
  typedef T Part __attribute__((ext_vector_type(V)));  // the real or imaginary parts of an element
  extern __shared__ __align__(16) unsigned char smem_raw[];
  Part* buf = reinterpret_cast<Part*>(smem_raw);
  TwEntry<T>* tw = reinterpret_cast<TwEntry<T>*>(smem_raw + a.lds_tw);
  unsigned* ltab = reinterpret_cast<unsigned*>(smem_raw + a.lds_tab);

  // the tile: sphere, first element f0 of nf, rows, and the two sides' bases
  const int t = static_task_g(a.total, a.group);
  if (t < 0) return;
  int s = 0, f0, nf, nl = 1, trow = N;
  const int32_t* __restrict__ tab = a.tab;
  const cpx<T>* src = reinterpret_cast<const cpx<T>*>(a.src);
  cpx<T>* dst = reinterpret_cast<cpx<T>*>(a.dst);
  int64_t gat, den, pstride, vrow = 0;
  int gstep = 0, dstep = 0;  // row steps
  if (a.kind == kPassZ) {
    while (s + 1 < a.nsph && t >= a.sph[s + 1].ztile) ++s;
  } else {
    s = (a.p0 + (a.kind == kPassX ? t / (a.tiles * a.rtiles) : t / a.tiles)) / a.nz;
  }
  const PassSph d = a.sph[s];
  if (a.kind == kPassZ) {
    f0 = (t - d.ztile) * a.fc;
    nf = d.ncol * d.nel;
    tab += d.gidx_off;
    gat = d.sph_off;
    den = d.col_off;
    pstride = d.colrow;
  } else {
    const int ft = t % a.tiles, rest = t / a.tiles;
    const int pl = a.kind == kPassX ? rest / a.rtiles : rest;  // plane within the group
    const int z = a.p0 + pl - s * a.nz;
    f0 = ft * a.fc;
    if (a.kind == kPassY) {
      nf = d.nslab * d.nel;
      tab += d.colidx_off;
      gat = d.col_off + static_cast<int64_t>(z) * d.colrow;
      den = static_cast<int64_t>(pl) * a.splane;
      pstride = d.srow;
    } else {
      const int y0 = (rest - pl * a.rtiles) * a.lines;
      nl = min(a.lines, a.ny - y0);
      nf = d.nel;
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
  const int nel = d.nel, nb = d.nb;
  const int fc = a.fc, nfl = min(fc, nf - f0);
  const float inv_fc = 1.0f / static_cast<float>(fc), inv_nel = 1.0f / static_cast<float>(nel);
  const int c0 = f0 / nel, e0 = f0 - c0 * nel;  // line and element of the line at f0
  const bool ntd = a.nt_dense != 0, ntg = a.nt_gather != 0;

  // the tile's table rows in LDS as byte offsets (a.tab_lds: the host has
  // checked that the gathered region and the dense side span less than 2 GiB)
  if constexpr (R2 > 1) {
    if (a.tab_lds) {
      const int nlin = (e0 + nfl - 1) / nel + 1;
      const int32_t* __restrict__ row = tab + static_cast<int64_t>(c0) * trow;
      const unsigned step = static_cast<unsigned>(nb) * es;
      for (int i = threadIdx.x; i < nlin * N; i += blockDim.x) {
        const int g = row[i];
        ltab[i] = g >= 0 ? static_cast<unsigned>(g) * step : kPassAbsent;
      }
    }
  }

  // stage 1: thread (f, i, l) takes positions i + R2*q of line l
  const int items1 = a.lines * R2 * fc;
  cpx<T> va[R1], vb[V == 2 ? R1 : 1];  // the lane's bands
#define FFTB_SET(q, e)                  \
  do {                                  \
    const Elem<T, V> e_ = (e);          \
    va[q].re = e_.a.re;                 \
    va[q].im = e_.a.im;                 \
    if constexpr (V == 2) {             \
      vb[q].re = e_.b.re;               \
      vb[q].im = e_.b.im;               \
    }                                   \
  } while (0)
  auto load = [&](int it) __attribute__((always_inline)) {
    const int rest = pass_div(it, fc, inv_fc);
    const int f = it - rest * fc, l = rest / R2, i = rest - l * R2;
    const bool ok = f < nfl && l < nl;
    const int ee = e0 + (ok ? f : 0);
    const int dc = pass_div(ee, nel, inv_nel);
    const int band = V * (ee - dc * nel);
#pragma unroll
    for (int q = 0; q < R1; ++q) FFTB_SET(q, (Elem<T, V>{{0, 0}, {0, 0}}));
    if (!ok) return;
    if constexpr (S > 0) {
      const cpx<T>* gsrc = src + gat;
      if (R2 > 1 && a.tab_lds) {
        const __amdgpu_buffer_rsrc_t r = pass_rsrc(gsrc);
        const unsigned off = static_cast<unsigned>(band + l * gstep) * es;
        const unsigned* row = ltab + (trow ? dc * N : 0) + i;
        with_nt(ntg, [&](auto nt) __attribute__((always_inline)) {
#pragma unroll
          for (int q = 0; q < R1; ++q)
            FFTB_SET(q, (buf_ld_el<decltype(nt)::value, V, T>(r, row[R2 * q] + off, 0)));
        });
        return;
      }
      const int32_t* __restrict__ row = tab + static_cast<int64_t>(c0 + dc) * trow + i;
      const cpx<T>* base = gsrc + band + l * gstep;
      int g[R1];
#pragma unroll
      for (int q = 0; q < R1; ++q) g[q] = row[R2 * q];
      with_nt(ntg, [&](auto nt) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < R1; ++q)
          if (g[q] >= 0) FFTB_SET(q, (ld_el<decltype(nt)::value, V>(base + static_cast<int64_t>(g[q]) * nb)));
      });
    } else {
      const cpx<T>* dsrc = src + den + static_cast<int64_t>(c0) * nb;
      const int64_t lane = dc * nb + band + i * pstride + static_cast<int64_t>(l) * dstep;
      if (a.tab_lds) {
        const __amdgpu_buffer_rsrc_t r = pass_rsrc(dsrc);
        const unsigned off = static_cast<unsigned>(lane) * es;
        const unsigned step = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(R2 * pstride) * es);
        with_nt(ntd, [&](auto nt) __attribute__((always_inline)) {
#pragma unroll
          for (int q = 0; q < R1; ++q)
            FFTB_SET(q, (buf_ld_el<decltype(nt)::value, V, T>(r, off, q * step)));
        });
      } else {
        with_nt(ntd, [&](auto nt) __attribute__((always_inline)) {
#pragma unroll
          for (int q = 0; q < R1; ++q)
            FFTB_SET(q, (ld_el<decltype(nt)::value, V>(dsrc + lane + (R2 * q) * pstride)));
        });
      }
    }
  };
#define FFTB_GET(k) ua[k].re, ua[k].im, ub[V == 2 ? (k) : 0].re, ub[V == 2 ? (k) : 0].im
  // the last stage of an inverse: thread (f, k1, l) writes positions k1 + ST*k
  auto emit_dense = [&](int f, int l, int k1, auto& ua, auto& ub, auto stride_c, auto count_c)
      __attribute__((always_inline)) {
    constexpr int ST = decltype(stride_c)::value, CT = decltype(count_c)::value;
    const int dc = pass_div(e0 + f, nel, inv_nel);
    const int band = V * (e0 + f - dc * nel);
    cpx<T>* ddst = dst + den + static_cast<int64_t>(c0) * nb;
    const int64_t lane = dc * nb + band + k1 * pstride + static_cast<int64_t>(l) * dstep;
    if (R2 > 1 && a.tab_lds) {
      const __amdgpu_buffer_rsrc_t r = pass_rsrc(ddst);
      const unsigned off = static_cast<unsigned>(lane) * es;
      const unsigned step = __builtin_amdgcn_readfirstlane(static_cast<unsigned>(ST * pstride) * es);
      with_nt(ntd, [&](auto nt) __attribute__((always_inline)) {
        static_for<0, CT>([&](auto kc) __attribute__((always_inline)) {
          constexpr int k = decltype(kc)::value;
          buf_st_el<decltype(nt)::value, V>(r, FFTB_GET(k), off + k * step);
        });
      });
    } else {
      with_nt(ntd, [&](auto nt) __attribute__((always_inline)) {
        static_for<0, CT>([&](auto kc) __attribute__((always_inline)) {
          constexpr int k = decltype(kc)::value;
          st_el<decltype(nt)::value, V>(ddst + lane + (ST * k) * pstride, FFTB_GET(k));
        });
      });
    }
  };
  // the last stage of a forward: the positions that the table keeps, to out
  auto emit_gather = [&](cpx<T>* out, int f, int l, int k1, auto& ua, auto& ub, auto stride_c, auto count_c)
      __attribute__((always_inline)) {
    constexpr int ST = decltype(stride_c)::value, CT = decltype(count_c)::value;
    const int dc = pass_div(e0 + f, nel, inv_nel);
    const int band = V * (e0 + f - dc * nel);
    cpx<T>* gdst = out + gat;
    if (R2 > 1 && a.tab_lds) {
      const __amdgpu_buffer_rsrc_t r = pass_rsrc(gdst);
      const unsigned off = static_cast<unsigned>(band + l * gstep) * es;
      const unsigned* row = ltab + (trow ? dc * N : 0) + k1;
      with_nt(ntg, [&](auto nt) __attribute__((always_inline)) {
        static_for<0, CT>([&](auto kc) __attribute__((always_inline)) {
          constexpr int k = decltype(kc)::value;
          buf_st_el<decltype(nt)::value, V>(r, FFTB_GET(k), row[ST * k] + off);
        });
      });
      return;
    }
    const int32_t* __restrict__ row = tab + static_cast<int64_t>(c0 + dc) * trow + k1;
    cpx<T>* base = gdst + band + l * gstep;
    int g[CT];
    static_for<0, CT>([&](auto kc) __attribute__((always_inline)) {
      g[decltype(kc)::value] = row[ST * decltype(kc)::value];
    });
    with_nt(ntg, [&](auto nt) __attribute__((always_inline)) {
      static_for<0, CT>([&](auto kc) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value;
        if (g[k] >= 0)
          st_el<decltype(nt)::value, V>(base + static_cast<int64_t>(g[k]) * nb, FFTB_GET(k));
      });
    });
  };
  // multiply by w (conjugated in the transform back)
  auto twiddle = [](cpx<T> x, const TwEntry<T>& e, T sg) __attribute__((always_inline)) {
    if constexpr (std::is_same<T, float>::value) return cmul_hl(x, {e.re, sg * e.im}, {e.lre, sg * e.lim});
    else return cmul(x, {e.re, sg * e.im});
  };
  // scale by the potential at positions k1 + ST*k of line l, or by 1/N
  auto weigh = [&](int l, int k1, auto& ua, auto& ub, auto stride_c, auto count_c)
      __attribute__((always_inline)) {
    constexpr int ST = decltype(stride_c)::value, CT = decltype(count_c)::value;
    const T* __restrict__ vr = reinterpret_cast<const T*>(a.pot) + vrow + static_cast<int64_t>(l) * N + k1;
    static_for<0, CT>([&](auto kc) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value;
      const T p = POT ? vr[ST * k] : static_cast<T>(a.scale);
      ua[k].re *= p;
      ua[k].im *= p;
      if constexpr (V == 2) {
        ub[k].re *= p;
        ub[k].im *= p;
      }
    });
  };
  using One = std::integral_constant<int, 1>;
  using C1 = std::integral_constant<int, R1>;
  using C2 = std::integral_constant<int, R2>;
  cpx<T>* back = reinterpret_cast<cpx<T>*>(a.back);

  if constexpr (R2 == 1) {
    for (int it = threadIdx.x; it < items1; it += blockDim.x) {
      load(it);
      const int l = pass_div(it, fc, inv_fc), f = it - l * fc;
      dft<R1, S>(va);
      if constexpr (V == 2) dft<R1, S>(vb);
      if (f >= nfl || l >= nl) continue;
      if constexpr (POT || S < 0) weigh(l, 0, va, vb, One{}, C1{});
      if constexpr (S > 0) emit_dense(f, l, 0, va, vb, One{}, C1{});
      else emit_gather(dst, f, l, 0, va, vb, One{}, C1{});
      if constexpr (POT) {
        if (!back) continue;
        dft<R1, -1>(va);
        if constexpr (V == 2) dft<R1, -1>(vb);
        emit_gather(back, f, l, 0, va, vb, One{}, C1{});
      }
    }
    return;
  } else {
    // (the host gives every item of either stage its own thread)
    const int it = threadIdx.x;
    const bool on1 = it < items1;
    if (S < 0 && on1) load(it);
    bl_fill_twiddles<S, T>(tw, reinterpret_cast<const cpx<T>*>(a.root),
                           reinterpret_cast<const cpx<T>*>(a.root_lo), R1, R2);
    __syncthreads();
    if (S > 0 && on1) load(it);
    const int rest1 = pass_div(it, fc, inv_fc);
    const int f = it - rest1 * fc;
    const int l1 = rest1 / R2, i1 = rest1 - l1 * R2;
    const int l2 = rest1 / R1, k1 = rest1 - l2 * R1;
    const bool on2 = it < a.lines * R1 * fc;
    if (on1) {
      const TwEntry<T>* tr = tw + i1 * tw_row_stride(R1);
      dft<R1, S>(va);
      if constexpr (V == 2) {
        __builtin_amdgcn_sched_barrier(0);  // (one transform's temporaries at a time)
        dft<R1, S>(vb);
        __builtin_amdgcn_sched_barrier(0);
      }
      static_for<1, R1>([&](auto kc) __attribute__((always_inline)) {
        constexpr int k = decltype(kc)::value;
        const TwEntry<T> e = tr[k];
        va[k] = twiddle(va[k], e, 1);
        if constexpr (V == 2) vb[k] = twiddle(vb[k], e, 1);
      });
    }
    cpx<T> ua[R2], ub[V == 2 ? R2 : 1];
    // rows of `from` values at out + k*step become rows of `to` values at in +
    // i*fc, real parts first
    auto exchange = [&](bool w, auto& xa, auto& xb, Part* out, int step, auto from_c, bool r, auto& ya,
                        auto& yb, const Part* in, auto to_c) __attribute__((always_inline)) {
      constexpr int FR = decltype(from_c)::value, TO = decltype(to_c)::value;
      if (w)
        static_for<0, FR>([&](auto kc) __attribute__((always_inline)) {
          constexpr int k = decltype(kc)::value;
          out[k * step] = parts<V>(xa[k].re, xb[V == 2 ? k : 0].re);
        });
      __syncthreads();
      if (r)
        static_for<0, TO>([&](auto ic) __attribute__((always_inline)) {
          constexpr int i = decltype(ic)::value;
          const Part x = in[i * fc];
          ya[i].re = x[0];
          if constexpr (V == 2) yb[i].re = x[1];
        });
      __syncthreads();
      if (w)
        static_for<0, FR>([&](auto kc) __attribute__((always_inline)) {
          constexpr int k = decltype(kc)::value;
          out[k * step] = parts<V>(xa[k].im, xb[V == 2 ? k : 0].im);
        });
      __syncthreads();
      if (r)
        static_for<0, TO>([&](auto ic) __attribute__((always_inline)) {
          constexpr int i = decltype(ic)::value;
          const Part x = in[i * fc];
          ya[i].im = x[0];
          if constexpr (V == 2) yb[i].im = x[1];
        });
    };
    exchange(on1, va, vb, buf + (l1 * R1 * RS + i1) * fc + f, RS * fc, C1{}, on2, ua, ub,
             buf + (l2 * R1 + k1) * RS * fc + f, C2{});
    const bool live2 = on2 && f < nfl && l2 < nl;
    if (on2) {
      dft<R2, S>(ua);
      if constexpr (V == 2) {
        __builtin_amdgcn_sched_barrier(0);
        dft<R2, S>(ub);
      }
    }
    if (live2) {
      if constexpr (POT || S < 0) weigh(l2, k1, ua, ub, C1{}, C2{});
      if constexpr (S > 0) emit_dense(f, l2, k1, ua, ub, C1{}, C2{});
      else emit_gather(dst, f, l2, k1, ua, ub, C1{}, C2{});
    }
    if constexpr (POT) {
      // the forward transform of the weighted row, back into its slab row: the
      // same split with the stages' roles exchanged (R2 values at stride R1 in
      // this thread), whose rows of R1 values take RS1 pieces
      if (!back) return;
      constexpr int RS1 = R1 | 1;
      if (on2) {
        const TwEntry<T>* tc = tw + k1;
        dft<R2, -1>(ua);
        if constexpr (V == 2) {
          __builtin_amdgcn_sched_barrier(0);
          dft<R2, -1>(ub);
          __builtin_amdgcn_sched_barrier(0);
        }
        static_for<1, R2>([&](auto kc) __attribute__((always_inline)) {
          constexpr int k = decltype(kc)::value;
          const TwEntry<T> e = tc[k * tw_row_stride(R1)];
          ua[k] = twiddle(ua[k], e, -1);
          if constexpr (V == 2) ub[k] = twiddle(ub[k], e, -1);
        });
      }
      __syncthreads();
      cpx<T> wa[R1], wb[V == 2 ? R1 : 1];  // (va would stay live where on1 is false)
      exchange(on2, ua, ub, buf + (l2 * R2 * RS1 + k1) * fc + f, RS1 * fc, C2{}, on1, wa, wb,
               buf + (l1 * R2 + i1) * RS1 * fc + f, C1{});
      if (on1 && f < nfl && l1 < nl) {
        dft<R1, -1>(wa);
        if constexpr (V == 2) {
          __builtin_amdgcn_sched_barrier(0);
          dft<R1, -1>(wb);
        }
        emit_gather(back, f, l1, i1, wa, wb, C2{}, C1{});
      }
    }
  }
}
#undef FFTB_SET
#undef FFTB_GET

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

// (S = +2: the x pass of the potential step)
template <int S, typename T, int V, int N>
hipError_t pass_one(const PassArgs& a, int threads, size_t lds, hipStream_t st, bool attr_only) {
  constexpr int SG = S > 0 ? 1 : -1;
  if (attr_only)
    return hipFuncSetAttribute(reinterpret_cast<const void*>(pass_kernel<SG, T, V, N, S == 2>),
                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  hipLaunchKernelGGL((pass_kernel<SG, T, V, N, S == 2>), dim3(pass_grid(a.total, a.group)), dim3(threads),
                     lds, st, a);
  return hipGetLastError();
}

// Launch (or, with attr_only, allow `lds` bytes to) the kernel of length n if
// part P compiles it; *found tells.
template <int S, typename T, int V, int P>
hipError_t pass_part(int n, const PassArgs& a, int threads, size_t lds, hipStream_t st,
                     bool attr_only, bool* found) {
  *found = true;
#define FFTB_X(n_) \
  case n_: return pass_one<S, T, V, n_>(a, threads, lds, st, attr_only);
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

#define FFTB_PASS_INST(EXT, S, T, V, P)                                                          \
  EXT template hipError_t pass_part<S, T, V, P>(int, const PassArgs&, int, size_t, hipStream_t, bool, \
                                             bool*);

}  // namespace fftb
