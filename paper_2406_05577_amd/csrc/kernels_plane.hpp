// Plane kernel for gfx950: the y and x passes of a plane in one launch, for
// planes of few points.
//
// A workgroup holds one plane of `fc` elements in LDS, [y][x][element], and runs
// the two stages of each axis on it (the splits of the axis passes): the first
// gathers the columns through the (slab, y) table, the last writes the grid. The
// stages work in place: position k1 + R1*k2 of a line ends at R2*k1 + k2, and the
// forward runs the stages in the opposite order, from there to the natural
// order, so nothing is permuted. The potential step multiplies the last stage's
// values by V on their way to the grid and goes back from the registers.
//
// Small transforms are bound by their launches, 4 to 5 us each however little
// they do; this saves one per direction and the slab scratch between the passes.
// The radices are arguments (a uniform switch over the codelets), as each pair of
// axes would otherwise be a kernel of its own.
// A round trip at 32^3, 4 complex128 bands: 26.5 -> 22.3 us, the potential step with
// 8: 24.5 -> 19.1; 24^3, 4 x 16 bands 38 -> 28.5; 36x40x45, 20 bands 45 -> 35.
#pragma once

#include "kernels_pass.hpp"

namespace fftb {

// the splits' factors: the first stage's up to 16, the second's up to 8
template <class F>
__device__ __forceinline__ void plane_r1(int r, F&& f) {
  switch (r) {
#define FFTB_R(R) \
  case R: f(std::integral_constant<int, R>{}); break;
    FFTB_R(1) FFTB_R(2) FFTB_R(3) FFTB_R(4) FFTB_R(5) FFTB_R(6) FFTB_R(8) FFTB_R(9) FFTB_R(10)
    FFTB_R(12) FFTB_R(15) FFTB_R(16)
  }
}
template <class F>
__device__ __forceinline__ void plane_r2(int r, F&& f) {
  switch (r) {
    FFTB_R(1) FFTB_R(3) FFTB_R(4) FFTB_R(5) FFTB_R(6) FFTB_R(8)
#undef FFTB_R
  }
}

// R values through load, their transform, store(k, a, b)
template <int R, int S, int V, typename T>
struct PlaneLine {
  cpx<T> a[R], b[V == 2 ? R : 1];
  template <class L>
  __device__ __forceinline__ void load(L&& l) {
    static_for<0, R>([&](auto qc) __attribute__((always_inline)) {
      constexpr int q = decltype(qc)::value;
      const Elem<T, V> e = l(q);
      a[q].re = e.a.re;
      a[q].im = e.a.im;
      if constexpr (V == 2) {
        b[q].re = e.b.re;
        b[q].im = e.b.im;
      }
    });
  }
  template <int SG>
  __device__ __forceinline__ void transform() {
    dft<R, SG>(a);
    if constexpr (V == 2) {
      __builtin_amdgcn_sched_barrier(0);
      dft<R, SG>(b);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  template <class F>
  __device__ __forceinline__ void store(F&& f) {
    static_for<0, R>([&](auto kc) __attribute__((always_inline)) {
      constexpr int k = decltype(kc)::value;
      f(k, a[k], b[V == 2 ? k : 0]);
    });
  }
};

template <int MODE, typename T, int V>
__global__ void __launch_bounds__(512) plane_kernel(const PlaneArgs a) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  using Words = typename ElemVec<T, V>::words;
  using Vec = typename ElemVec<T, V>::type;
  cpx<T>* A = reinterpret_cast<cpx<T>*>(smem_raw);
  TwEntry<T>* twx = reinterpret_cast<TwEntry<T>*>(smem_raw + a.lds_twx);
  TwEntry<T>* twy = reinterpret_cast<TwEntry<T>*>(smem_raw + a.lds_twy);
  int* xi = reinterpret_cast<int*>(smem_raw + a.lds_x);  // x -> slab or -1
  int* sx = xi + a.nx;                                   // slab -> x

  const int t = static_task_g(a.total, a.tiles);
  if (t < 0) return;
  const int pl = t / a.tiles, s = pl / a.nz, z = pl - s * a.nz;
  const PassSph d = a.sph[s];
  const int nx = a.nx, ny = a.ny, nb = d.nb, ns = d.nslab, fc = a.fc;
  const int f0 = (t - pl * a.tiles) * fc;
  if (f0 >= d.nel) return;
  const int nf = min(fc, d.nel - f0);
  const int32_t* __restrict__ ctab = a.colidx + d.colidx_off;
  for (int x = threadIdx.x; x < nx; x += blockDim.x) {
    const int i = a.xinv[d.xinv_off + x];
    xi[x] = i;
    if (i >= 0) sx[i] = x;
  }
  const int r1x = a.r1x, r2x = nx / r1x, r1y = a.r1y, r2y = ny / r1y;
  const int tsx = tw_row_stride(r1x), tsy = tw_row_stride(r1y);
  bl_fill_twiddles<+1, T>(twx, reinterpret_cast<const cpx<T>*>(a.rootx),
                          reinterpret_cast<const cpx<T>*>(a.rootx_lo), r1x, r2x);
  bl_fill_twiddles<+1, T>(twy, reinterpret_cast<const cpx<T>*>(a.rooty),
                          reinterpret_cast<const cpx<T>*>(a.rooty_lo), r1y, r2y);
  const float inv_nf = 1.0f / static_cast<float>(nf), inv_ns = 1.0f / static_cast<float>(ns);
  const float inv_ny = 1.0f / static_cast<float>(ny), inv_r2x = 1.0f / static_cast<float>(r2x);
  const float inv_r1x = 1.0f / static_cast<float>(r1x), inv_r2y = 1.0f / static_cast<float>(r2y);
  const int64_t col0 = d.col_off + static_cast<int64_t>(z) * d.colrow + V * f0;
  const cpx<T>* cin = reinterpret_cast<const cpx<T>*>(a.col_in) + col0;
  cpx<T>* cout = reinterpret_cast<cpx<T>*>(a.col_out) + col0;
  cpx<T>* grid = reinterpret_cast<cpx<T>*>(a.grid) + d.grid_off + static_cast<int64_t>(z) * ny * nx * nb + V * f0;
  const T* __restrict__ pot = reinterpret_cast<const T*>(a.pot) + static_cast<int64_t>(z) * ny * nx;
  __syncthreads();

  // an element of the plane in LDS
  auto get = [&](int row, int x, int f) __attribute__((always_inline)) {
    return unpack<V, T>(*reinterpret_cast<const Vec*>(A + ((row * nx + x) * fc + f) * V));
  };
  auto put = [&](int row, int x, int f, cpx<T> va, cpx<T> vb) __attribute__((always_inline)) {
    *reinterpret_cast<Words*>(A + ((row * nx + x) * fc + f) * V) = pack<V>(va.re, va.im, vb.re, vb.im);
  };
  auto turn = [](cpx<T> x, const TwEntry<T>& e, T sg) __attribute__((always_inline)) {
    if constexpr (std::is_same<T, float>::value) return cmul_hl(x, {e.re, sg * e.im}, {e.lre, sg * e.lim});
    else return cmul(x, {e.re, sg * e.im});
  };
  // items: n2 x n1 lines of nf elements; body(f, index < n1, index < n2)
  auto items = [&](int n1, float inv_n1, int n2, auto&& body) __attribute__((always_inline)) {
    for (int it = threadIdx.x; it < n1 * n2 * nf; it += blockDim.x) {
      const int rest = pass_div(it, nf, inv_nf), j = pass_div(rest, n1, inv_n1);
      body(it - rest * nf, rest - j * n1, j);
    }
  };

  if constexpr (MODE != kPassForward) {
    plane_r1(r1y, [&](auto rc) __attribute__((always_inline)) {
      constexpr int R = decltype(rc)::value;
      items(ns, inv_ns, r2y, [&](int f, int sl, int i) __attribute__((always_inline)) {
        const int32_t* __restrict__ row = ctab + sl * ny + i;
        int g[R];
        static_for<0, R>([&](auto qc) __attribute__((always_inline)) {
          g[decltype(qc)::value] = row[r2y * decltype(qc)::value];
        });
        PlaneLine<R, 1, V, T> v;
        v.load([&](int q) __attribute__((always_inline)) {
          Elem<T, V> e = {{0, 0}, {0, 0}};
          if (g[q] >= 0) e = ld_el<false, V>(cin + static_cast<int64_t>(g[q]) * nb + V * f);
          return e;
        });
        v.template transform<1>();
        const int x = sx[sl];
        v.store([&](int k, cpx<T> p, cpx<T> q) __attribute__((always_inline)) {
          if (k) {
            const TwEntry<T> e = twy[i * tsy + k];
            p = turn(p, e, 1);
            if constexpr (V == 2) q = turn(q, e, 1);
          }
          put(i + r2y * k, x, f, p, q);
        });
      });
    });
    __syncthreads();
    if (r2y > 1) {
      plane_r2(r2y, [&](auto rc) __attribute__((always_inline)) {
        constexpr int R = decltype(rc)::value;
        items(ns, inv_ns, r1y, [&](int f, int sl, int k1) __attribute__((always_inline)) {
          const int x = sx[sl];
          PlaneLine<R, 1, V, T> v;
          v.load([&](int i) __attribute__((always_inline)) { return get(i + R * k1, x, f); });
          v.template transform<1>();
          v.store([&](int k, cpx<T> p, cpx<T> q) __attribute__((always_inline)) { put(k + R * k1, x, f, p, q); });
        });
      });
      __syncthreads();
    }
    plane_r1(r1x, [&](auto rc) __attribute__((always_inline)) {
      constexpr int R = decltype(rc)::value;
      items(r2x, inv_r2x, ny, [&](int f, int i, int y) __attribute__((always_inline)) {
        PlaneLine<R, 1, V, T> v;
        v.load([&](int q) __attribute__((always_inline)) {
          Elem<T, V> e = {{0, 0}, {0, 0}};
          if (xi[i + r2x * q] >= 0) e = get(y, i + r2x * q, f);
          return e;
        });
        v.template transform<1>();
        v.store([&](int k, cpx<T> p, cpx<T> q) __attribute__((always_inline)) {
          if (k) {
            const TwEntry<T> e = twx[i * tsx + k];
            p = turn(p, e, 1);
            if constexpr (V == 2) q = turn(q, e, 1);
          }
          put(y, i + r2x * k, f, p, q);
        });
      });
    });
    __syncthreads();
  }
  // the x stage at the grid
  plane_r2(r2x, [&](auto rc) __attribute__((always_inline)) {
    constexpr int R = decltype(rc)::value;
    items(r1x, inv_r1x, ny, [&](int f, int k1, int row) __attribute__((always_inline)) {
      const int k1y = pass_div(row, r2y, inv_r2y), y = k1y + r1y * (row - k1y * r2y);
      cpx<T>* g = grid + static_cast<int64_t>(y * nx + k1) * nb + V * f;
      const int64_t step = static_cast<int64_t>(r1x) * nb;
      PlaneLine<R, 1, V, T> v;
      if constexpr (MODE == kPassForward) {
        v.load([&](int k) __attribute__((always_inline)) { return ld_el<false, V>(g + k * step); });
      } else {
        v.load([&](int i) __attribute__((always_inline)) { return get(row, i + R * k1, f); });
        v.template transform<1>();
        if constexpr (MODE == kPassPotential)
          static_for<0, R>([&](auto kc) __attribute__((always_inline)) {
            constexpr int k = decltype(kc)::value;
            const T p = pot[y * nx + k1 + r1x * k];
            v.a[k].re *= p;
            v.a[k].im *= p;
            if constexpr (V == 2) {
              v.b[k].re *= p;
              v.b[k].im *= p;
            }
          });
        v.store([&](int k, cpx<T> p, cpx<T> q) __attribute__((always_inline)) {
          st_el<false, V>(g + k * step, p.re, p.im, q.re, q.im);
        });
        if (MODE == kPassInverse || !a.col_out) return;
      }
      v.template transform<-1>();
      v.store([&](int k, cpx<T> p, cpx<T> q) __attribute__((always_inline)) {
        if (k) {
          const TwEntry<T> e = twx[k * tsx + k1];
          p = turn(p, e, -1);
          if constexpr (V == 2) q = turn(q, e, -1);
        }
        put(row, k + R * k1, f, p, q);
      });
    });
  });
  if constexpr (MODE != kPassInverse) {
    if (MODE == kPassPotential && !a.col_out) return;
    __syncthreads();
    plane_r1(r1x, [&](auto rc) __attribute__((always_inline)) {
      constexpr int R = decltype(rc)::value;
      items(r2x, inv_r2x, ny, [&](int f, int i, int row) __attribute__((always_inline)) {
        PlaneLine<R, -1, V, T> v;
        v.load([&](int k1) __attribute__((always_inline)) { return get(row, i + r2x * k1, f); });
        v.template transform<-1>();
        v.store([&](int k, cpx<T> p, cpx<T> q) __attribute__((always_inline)) {
          if (xi[i + r2x * k] >= 0) put(row, i + r2x * k, f, p, q);
        });
      });
    });
    __syncthreads();
    if (r2y > 1) {
      plane_r2(r2y, [&](auto rc) __attribute__((always_inline)) {
        constexpr int R = decltype(rc)::value;
        items(ns, inv_ns, r1y, [&](int f, int sl, int k1) __attribute__((always_inline)) {
          const int x = sx[sl];
          PlaneLine<R, -1, V, T> v;
          v.load([&](int k) __attribute__((always_inline)) { return get(k + R * k1, x, f); });
          v.template transform<-1>();
          v.store([&](int k, cpx<T> p, cpx<T> q) __attribute__((always_inline)) {
            if (k) {
              const TwEntry<T> e = twy[k * tsy + k1];
              p = turn(p, e, -1);
              if constexpr (V == 2) q = turn(q, e, -1);
            }
            put(k + R * k1, x, f, p, q);
          });
        });
      });
      __syncthreads();
    }
    plane_r1(r1y, [&](auto rc) __attribute__((always_inline)) {
      constexpr int R = decltype(rc)::value;
      items(ns, inv_ns, r2y, [&](int f, int sl, int i) __attribute__((always_inline)) {
        const int x = sx[sl];
        const int32_t* __restrict__ row = ctab + sl * ny + i;
        int g[R];
        static_for<0, R>([&](auto qc) __attribute__((always_inline)) {
          g[decltype(qc)::value] = row[r2y * decltype(qc)::value];
        });
        PlaneLine<R, -1, V, T> v;
        v.load([&](int k1) __attribute__((always_inline)) { return get(i + r2y * k1, x, f); });
        v.template transform<-1>();
        v.store([&](int k, cpx<T> p, cpx<T> q) __attribute__((always_inline)) {
          if (g[k] >= 0) st_el<false, V>(cout + static_cast<int64_t>(g[k]) * nb + V * f, p.re, p.im, q.re, q.im);
        });
      });
    });
  }
}

template <typename T, int V>
hipError_t plane_launch(PassMode mode, const PlaneArgs& a, int threads, size_t lds, hipStream_t st, bool attr) {
  const void* f = mode == kPassInverse   ? reinterpret_cast<const void*>(plane_kernel<kPassInverse, T, V>)
                  : mode == kPassForward ? reinterpret_cast<const void*>(plane_kernel<kPassForward, T, V>)
                                         : reinterpret_cast<const void*>(plane_kernel<kPassPotential, T, V>);
  if (attr) return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
  PlaneArgs c = a;
  void* args[] = {&c};
  return hipLaunchKernel(f, dim3(pass_grid(a.total, a.tiles)), dim3(threads), args, lds, st);
}

}  // namespace fftb
