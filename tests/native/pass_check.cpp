// Address check of the axis passes (pass_plan.cpp), built with g++ and the
// sanitizers by tests/test_abi_host.py (no GPU): walks the tiles, threads and
// positions of every pass as the kernel does and checks that each access lies
// in its buffer, that the dense side is covered exactly once and that the
// gathered side reaches every coefficient, column and slab exactly once.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <string>
#include <vector>

#include "../../paper_2406_05577_amd/csrc/pass.hpp"

using namespace fftb;

static int failures = 0;
#define CHECK(c)                                                        \
  do {                                                                  \
    if (!(c) && ++failures < 20) std::fprintf(stderr, "check failed line %d: %s\n", __LINE__, #c); \
  } while (0)

struct Touch {
  std::vector<unsigned char> n;
  explicit Touch(size_t size) : n(size, 0) {}
  void at(int64_t i) {
    CHECK(i >= 0 && i < static_cast<int64_t>(n.size()));
    if (i >= 0 && i < static_cast<int64_t>(n.size()) && n[i] < 3) ++n[i];
  }
  int64_t count(int v) const { return std::count(n.begin(), n.end(), v); }
};

// One launch of a pass: the kernel's tile and item arithmetic.
static void walk(const PassPlan& P, int kind, int nx, int ny, int nz, int p0, int np, Touch& gather,
                 Touch& dense) {
  const PassTile& t = kind == kPassZ ? P.tz : kind == kPassY ? P.ty : P.tx;
  const int n = kind == kPassZ ? nz : kind == kPassY ? ny : nx;
  const int r1 = pass_r1(n), r2 = n / r1;
  const int total = kind == kPassZ ? P.ztotal : kind == kPassY ? np * t.tiles : np * t.tiles * t.rtiles;
  const int v = P.elem == kElemC64x2 ? 2 : 1;
  const std::vector<int32_t>& table = kind == kPassZ ? P.gidx : kind == kPassY ? P.colidx : P.xinv;
  CHECK(t.threads >= 64 && t.threads % 64 == 0);
  CHECK(t.lds_tw + (r2 > 1 ? (r1 | 1) * r2 * 16 : 0) <= static_cast<int>(t.lds));
  for (int b = 0; b < total; ++b) {
    size_t s = 0;
    int f0, nf, nl = 1, trow = n, tab;
    int64_t gat, den, pstride, gstep = 0, dstep = 0;
    if (kind == kPassZ) {
      while (s + 1 < P.sph.size() && b >= P.sph[s + 1].ztile) ++s;
      const PassSph& d = P.sph[s];
      f0 = (b - d.ztile) * t.fc;
      nf = d.ncol * d.nel;
      CHECK(f0 < nf);
      tab = d.gidx_off;
      gat = d.sph_off;
      den = d.col_off;
      pstride = d.colrow;
    } else {
      const int ft = b % t.tiles, rest = b / t.tiles;
      const int pl = kind == kPassX ? rest / t.rtiles : rest;
      const int p = p0 + pl;
      s = static_cast<size_t>(p / nz);
      const int z = p % nz;
      const PassSph& d = P.sph[s];
      f0 = ft * t.fc;
      if (kind == kPassY) {
        nf = d.nslab * d.nel;
        tab = d.colidx_off;
        gat = d.col_off + z * d.colrow;
        den = pl * P.splane;
        pstride = d.srow;
      } else {
        const int y0 = (rest - pl * t.rtiles) * t.lines;
        nl = std::min(t.lines, ny - y0);
        nf = d.nel;
        trow = 0;
        tab = d.xinv_off;
        gat = pl * P.splane + static_cast<int64_t>(y0) * d.srow;
        gstep = d.srow;
        den = d.grid_off + (static_cast<int64_t>(z) * ny + y0) * n * d.nb;
        dstep = static_cast<int64_t>(n) * d.nb;
        pstride = d.nb;
      }
      if (f0 >= nf) continue;
    }
    const int nb = P.sph[s].nb, nel = P.sph[s].nel, nfl = std::min(t.fc, nf - f0), c0 = f0 / nel, e0 = f0 - c0 * nel;
    const int nlin = (e0 + nfl - 1) / nel + 1;
    // the staged table rows: nlin lines (x: one row of the table for all)
    if (t.tab_lds) {
      CHECK(static_cast<size_t>(t.lds_tab) + static_cast<size_t>(nlin) * n * 4 <= t.lds);
      CHECK(tab + static_cast<int64_t>(c0) * trow + static_cast<int64_t>(nlin) * n <= static_cast<int64_t>(table.size()));
      if (kind == kPassX) CHECK(nlin == 1);
    }
    for (int l = 0; l < t.lines; ++l)
      for (int f = 0; f < t.fc; ++f) {
        if (f >= nfl || l >= nl) continue;
        const int ee = e0 + f, dc = ee / nel, j = ee - dc * nel, band = v * j;
        CHECK(dc < nlin);
        for (int pos = 0; pos < n; ++pos) {
          const int64_t ti = tab + static_cast<int64_t>(c0 + dc) * trow + pos;
          CHECK(ti >= 0 && ti < static_cast<int64_t>(table.size()));
          const int g = table[ti];
          for (int w = 0; w < v; ++w) {
            const int64_t go = static_cast<int64_t>(g) * nb + band + w + l * gstep;
            const int64_t d_o = static_cast<int64_t>(c0) * nb + dc * nb + band + w + pos * pstride + l * dstep;
            if (t.tab_lds && g >= 0) CHECK(go * 8 * (P.elem == kElemC128 ? 2 : 1) < (int64_t{1} << 31));
            if (t.tab_lds) CHECK((d_o - c0 * nb) * 8 * (P.elem == kElemC128 ? 2 : 1) < (int64_t{1} << 31));
            if (g >= 0) gather.at(gat + go);
            dense.at(den + d_o);
          }
        }
      }
  }
}

static std::vector<int32_t> some_map(std::mt19937& g, int nx, int ny, int nz, double keep, double ratio) {
  std::vector<int32_t> m;
  std::uniform_real_distribution<double> u(0, 1);
  for (int z = 0; z < nz; ++z)
    for (int y = 0; y < ny; ++y)
      for (int x = 0; x < nx; ++x) {
        auto d = [](int i, int n) { const int j = std::min(i, n - i); return 1.0 * j / n; };
        const double r = std::sqrt(d(x, nx) * d(x, nx) + d(y, ny) * d(y, ny) + d(z, nz) * d(z, nz));
        if (r <= ratio && u(g) <= keep) m.push_back(x + nx * (y + ny * z));
      }
  if (m.empty()) m.push_back(0);
  std::shuffle(m.begin(), m.end(), g);
  return m;
}

static void check(std::mt19937& g, int nx, int ny, int nz, bool fp64, const std::vector<int>& nbs,
                  double keep, double ratio, int64_t budget) {
  std::vector<SphereTables> sph;
  std::vector<int64_t> row_max;
  int64_t sphere = 0, grid = 0;
  for (int nb : nbs) {
    const std::vector<int32_t> m = some_map(g, nx, ny, nz, keep, ratio);
    SphereTables t;
    std::string err;
    CHECK(build_sphere_tables(nx, ny, nz, m.data(), static_cast<int64_t>(m.size()), nb, t, err) == 0);
    sph.push_back(t);
    row_max.push_back(static_cast<int64_t>(t.ncol) * nb + (g() % 2 ? 64 : 0));
    sphere += t.ns * nb;
    grid += static_cast<int64_t>(nx) * ny * nz * nb;
  }
  PassPlan P;
  CHECK(build_pass_plan(nx, ny, nz, fp64, sph, row_max, budget, P));
  if (failures) return;
  CHECK(P.nplanes == nz * static_cast<int>(nbs.size()) && P.group >= 1);
  if (P.plane.on) {
    const PlaneTile& t = P.plane;
    int nel = 0;
    for (const PassSph& d : P.sph) nel = std::max(nel, d.nel);
    const auto tab = [](int n) { return (pass_r1(n) | 1) * (n / pass_r1(n)) * 16; };
    CHECK(nx <= kPlaneMaxN && ny <= kPlaneMaxN && t.fc >= 1 && t.fc * t.tiles >= nel);
    CHECK(t.threads >= 64 && t.threads <= 512 && t.threads % 64 == 0);
    CHECK(t.lds_twx >= nx * ny * t.fc * (P.elem == kElemC64 ? 8 : 16) && t.lds_twx % 16 == 0);
    CHECK(t.lds_twy >= t.lds_twx + tab(nx) && t.lds_x >= t.lds_twy + tab(ny));
    CHECK(static_cast<int>(t.lds) >= t.lds_x + 8 * nx && t.lds <= 160 * 1024 - 1024);
  }
  int64_t cols = 0, slabs = 0, colrows = 0;
  for (size_t i = 0; i < sph.size(); ++i) {
    cols += static_cast<int64_t>(sph[i].ncol) * P.sph[i].nb * nz;
    CHECK(P.sph[i].colrow <= row_max[i]);
    colrows += P.sph[i].colrow * nz;
    slabs += static_cast<int64_t>(sph[i].nslab) * P.sph[i].nb * ny * nz;
  }
  CHECK(colrows == P.col_elems);
  Touch tsph(sphere), tcol(P.col_elems);
  walk(P, kPassZ, nx, ny, nz, 0, 0, tsph, tcol);
  CHECK(tsph.count(1) == sphere);
  CHECK(tcol.count(1) == cols && tcol.count(2) == 0 && tcol.count(3) == 0);
  Touch tcol2(P.col_elems), tgrid(grid);
  int64_t seen = 0;
  for (int p0 = 0; p0 < P.nplanes; p0 += P.group) {
    const int np = std::min(P.group, P.nplanes - p0);
    Touch s1(P.s_elems()), s2(P.s_elems());
    walk(P, kPassY, nx, ny, nz, p0, np, tcol2, s1);
    walk(P, kPassX, nx, ny, nz, p0, np, s2, tgrid);
    CHECK(s1.n == s2.n && s1.count(2) == 0 && s1.count(3) == 0);
    seen += s1.count(1);
  }
  CHECK(seen == slabs);
  CHECK(tcol2.n == tcol.n);
  CHECK(tgrid.count(1) == grid);
}

int main() {
  std::mt19937 g(240605577);
  // every length splits into two codelets
  for (int n = 1; n <= kPassMaxN; ++n) {
    int k = n;
    for (int p : {2, 3, 5})
      while (k % p == 0) k /= p;
    const int r = pass_r1(n);
    CHECK((k == 1) == (r > 0));
    if (r) CHECK(n % r == 0 && pass_codelet(r) && pass_codelet(n / r));
  }
  const int len[] = {1, 2, 3, 5, 6, 10, 12, 15, 16, 18, 20, 24, 25, 27, 30, 36, 45};
  for (int it = 0; it < 60; ++it) {
    const int nx = len[g() % 17], ny = len[g() % 17], nz = len[g() % 17];
    std::vector<int> nbs;
    const int even = it % 3 == 0 ? 2 : 1;  // two bands per lane, complex64
    for (unsigned i = 0; i < 1 + g() % 3; ++i) nbs.push_back(even * (1 + static_cast<int>(g() % (it % 4 ? 9 : 70))));
    check(g, nx, ny, nz, it % 2, nbs, it % 5 ? 1.0 : 0.4, it % 7 ? 0.27 : 9.0, 1 << (10 + g() % 14));
  }
  check(g, 60, 4, 6, true, {37}, 1.0, 0.25, 1 << 20);
  check(g, 4, 125, 3, false, {1, 50}, 1.0, 0.3, 1 << 16);
  check(g, 3, 2, 512, true, {11}, 1.0, 0.3, 1 << 16);
  check(g, 384, 2, 3, false, {300}, 1.0, 0.25, 1 << 20);
  if (failures) return 1;
  std::printf("pass_check OK\n");
  return 0;
}
