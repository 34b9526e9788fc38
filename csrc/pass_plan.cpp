// Host side of the axis passes: tables in slot order, tiles and plane groups.
#include "pass.hpp"

#include <algorithm>
#include <cstdlib>
static int xi(){ const char* v=std::getenv("FFTB_X_ITEMS"); return v?std::atoi(v):256; }
#include <numeric>

namespace fftb {

namespace {

constexpr size_t kPassLdsMax = 160 * 1024 - 1024;

// A tile of a pass over lines of length n: about 256 items per stage in whole
// 128-byte pieces of the fast dimension (nf elements, the sphere's bands or
// its flattened (line, band) index), and for short fast dimensions several
// rows.
bool make_tile(int n, bool fp64, int64_t nf, int nrows, bool even, PassTile& t) {
  const int es = fp64 ? 16 : 8, w = 128 / es;
  const int r1 = pass_r1(n);
  if (!r1) return false;
  const int r2 = n / r1, m = std::max(r1, r2) == n ? 1 : std::max(r1, r2);
  int target = std::max(1, (xi() / m + w / 2) / w) * w;
  const auto lds_of = [&](int fc, int lines) {
    return r2 > 1 ? static_cast<size_t>(lines) * fc * r1 * (r2 | 1) * (es / 2) : size_t{0};
  };
  const size_t tab = r2 > 1 ? static_cast<size_t>(r1 | 1) * r2 * 16 : 0;
  while (target > w && lds_of(target, 1) + tab > kPassLdsMax / 2) target -= w;
  if (2 * nf <= 3 * static_cast<int64_t>(target)) {
    t.fc = static_cast<int>(nf);
  } else if (even) {
    // equal shares of the bands, in whole pieces where the bands are
    const int64_t nch = std::max<int64_t>(1, (nf + target / 2) / target);
    int64_t fc = (nf + nch - 1) / nch;
    if (nf % w == 0) fc = (fc + w - 1) / w * w;
    t.fc = static_cast<int>(fc);
  } else {
    t.fc = target;
  }
  t.lines = std::max(1, std::min(nrows, xi() / (t.fc * m)));
  t.threads = std::min(512, (t.lines * t.fc * m + 63) / 64 * 64);
  const size_t b = (lds_of(t.fc, t.lines) + 15) & ~size_t{15};
  t.lds_tw = static_cast<int>(b);
  t.lds = b + tab;
  t.tiles = static_cast<int>((nf + t.fc - 1) / t.fc);
  t.rtiles = (nrows + t.lines - 1) / t.lines;
  return t.lds <= kPassLdsMax;
}

}  // namespace

bool build_pass_plan(int nx, int ny, int nz, bool fp64, const std::vector<SphereTables>& sph,
                     const std::vector<int64_t>& colrow_max, int64_t s_budget, PassPlan& P) {
  P = PassPlan();
  if (nx > kPassMaxN || ny > kPassMaxN || nz > kPassMaxN) return false;
  if (!pass_r1(nx) || !pass_r1(ny) || !pass_r1(nz)) return false;
  const int es = fp64 ? 16 : 8;
  const int64_t w = 128 / es;
  const int64_t N = static_cast<int64_t>(nx) * ny * nz;
  const auto pad = [w](int64_t v) { return (v + w - 1) / w * w; };
  int64_t soff = 0, goff = 0, coff = 0, max_col = 0, max_slab = 0;
  int32_t max_nb = 0;
  for (size_t i = 0; i < sph.size(); ++i) {
    const SphereTables& s = sph[i];
    if (s.nb >= (1 << 20) || static_cast<int64_t>(s.ncol) * s.nb >= (int64_t{1} << 30) ||
        static_cast<int64_t>(s.nslab) * s.nb >= (int64_t{1} << 30))
      return false;
    // column slots by (y, x): the columns of a y row are neighbours, as the
    // slabs of a slab row are, so that the y pass reads and writes runs
    std::vector<int32_t> order(s.ncol);
    std::iota(order.begin(), order.end(), 0);
    std::sort(order.begin(), order.end(), [&s](int32_t a, int32_t b) {
      return s.col_y[a] != s.col_y[b] ? s.col_y[a] < s.col_y[b] : s.col_xi[a] < s.col_xi[b];
    });
    PassSph d = {};
    d.sph_off = soff;
    d.grid_off = goff;
    d.col_off = coff;
    d.nb = s.nb;
    d.ncol = s.ncol;
    d.nslab = s.nslab;
    const int64_t row = static_cast<int64_t>(s.ncol) * s.nb;
    d.colrow = pad(row) <= colrow_max[i] ? pad(row) : row;
    d.srow = static_cast<int32_t>(pad(static_cast<int64_t>(s.nslab) * s.nb));
    if (P.gidx.size() + static_cast<size_t>(s.ncol) * nz >= (size_t{1} << 31)) return false;
    d.gidx_off = static_cast<int32_t>(P.gidx.size());
    d.colidx_off = static_cast<int32_t>(P.colidx.size());
    d.xinv_off = static_cast<int32_t>(P.xinv.size());
    P.colidx.resize(P.colidx.size() + static_cast<size_t>(s.nslab) * ny, -1);
    P.gidx.reserve(P.gidx.size() + static_cast<size_t>(s.ncol) * nz);
    for (int32_t slot = 0; slot < s.ncol; ++slot) {
      const int32_t c = order[slot];
      P.colidx[d.colidx_off + static_cast<size_t>(s.col_xi[c]) * ny + s.col_y[c]] = slot;
      P.gidx.insert(P.gidx.end(), s.gidx.begin() + static_cast<size_t>(c) * nz,
                    s.gidx.begin() + static_cast<size_t>(c + 1) * nz);
    }
    P.xinv.insert(P.xinv.end(), s.xinv.begin(), s.xinv.end());
    soff += s.ns * s.nb;
    goff += N * s.nb;
    coff += d.colrow * nz;
    max_col = std::max(max_col, row);
    max_slab = std::max(max_slab, static_cast<int64_t>(s.nslab) * s.nb);
    max_nb = std::max(max_nb, s.nb);
    P.splane = std::max(P.splane, static_cast<int64_t>(d.srow) * ny);
    P.sph.push_back(d);
  }
  P.col_elems = coff;
  P.nplanes = static_cast<int>(sph.size()) * nz;
  if (!make_tile(nz, fp64, max_col, 1, false, P.tz) || !make_tile(ny, fp64, max_slab, 1, false, P.ty) ||
      !make_tile(nx, fp64, max_nb, ny, true, P.tx))
    return false;
  for (auto& d : P.sph) {
    d.ztile = P.ztotal;
    P.ztotal += static_cast<int>((static_cast<int64_t>(d.ncol) * d.nb + P.tz.fc - 1) / P.tz.fc);
  }
  // equal groups of planes within the budget
  const int64_t most = std::max<int64_t>(1, s_budget / (P.splane * es));
  const int64_t groups = (P.nplanes + most - 1) / most;
  P.group = static_cast<int>((P.nplanes + groups - 1) / groups);
  return static_cast<int64_t>(P.group) * std::max(P.ty.tiles, P.tx.tiles * P.tx.rtiles) < (int64_t{1} << 31);
}

}  // namespace fftb
