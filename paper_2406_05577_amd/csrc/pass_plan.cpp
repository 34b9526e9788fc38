// Host side of the axis passes: tables in slot order, tiles and plane groups.
#include "pass.hpp"

#include <algorithm>

namespace fftb {

namespace {

constexpr size_t kPassLdsMax = 160 * 1024 - 1024;
// LDS spent on staged table rows: a few lines' worth
constexpr size_t kPassTabMax = 8 * 1024;

// A tile of a pass over lines of length n: whole 128-byte pieces of the fast
// dimension (nf elements of `es` bytes, the sphere's bands or its flattened (line,
// band) index), as many as make 256 items per stage (four waves: a fifth, mostly
// idle one cost the 144-point inverse passes 10-35 %, and 200 points over 320
// threads 10-20 %) or one, all of the dimension where it is at most half longer
// than that (384 items and more: 512 points, 8 complex64 bands), and for short
// fast dimensions several rows. even: the fast dimension is cut into equal
// shares. ragged: the band vectors are no whole 128-byte lines; a tile then takes
// them whole where it can.
bool make_tile(int n, int es, int64_t nf, int nrows, bool even, bool ragged, PassTile& t) {
  const int w = 128 / es;
  const int r1 = pass_r1(n);
  if (!r1) return false;
  const int r2 = n / r1, m = r2 == 1 ? 1 : std::max(r1, r2);
  int target = std::max(1, 256 / (m * w)) * w;
  const auto lds_of = [&](int fc, int lines) {
    // (the larger of the two exchanges of the potential's x pass)
    const int rows = std::max(r1 * (r2 | 1), r2 * (r1 | 1));
    return r2 > 1 ? static_cast<size_t>(lines) * fc * rows * (es / 2) : size_t{0};
  };
  const size_t tab = r2 > 1 ? static_cast<size_t>(r1 | 1) * r2 * 16 : 0;
  while (target > w && lds_of(target, 1) + tab > kPassLdsMax / 2) target -= w;
  const int most = pass_max_threads(n, es == 8);
  if (2 * nf <= 3 * static_cast<int64_t>(target)) {
    t.fc = static_cast<int>(nf);
  } else if (even) {
    // equal shares of the bands: in whole pieces where the bands are, else as
    // few as eight waves and half the LDS allow (a cut leaves two half-written
    // lines: 200x192x216, 20 complex128 bands, inverse x pass 1.60 ms in two
    // tiles, 0.63 ms whole; more waves: 50x48x96, 82 bands, 0.39 against 0.32 ms)
    int64_t share = target;
    if (ragged) {
      share = std::max(1, 512 / m);
      while (share > target && lds_of(static_cast<int>(share), 1) + tab > kPassLdsMax / 2) --share;
    }
    const int64_t nch = ragged ? (nf + share - 1) / share : std::max<int64_t>(1, (nf + share / 2) / share);
    int64_t fc = (nf + nch - 1) / nch;
    if (!ragged) fc = (fc + w - 1) / w * w;
    t.fc = static_cast<int>(fc);
  } else {
    t.fc = target;
  }
  t.lines = std::max(1, std::min(nrows, 256 / (t.fc * m)));
  t.threads = (t.lines * t.fc * m + 63) / 64 * 64;
  if (r2 == 1) t.threads = std::min(t.threads, 256);
  const size_t b = (lds_of(t.fc, t.lines) + 15) & ~size_t{15};
  t.lds_tw = static_cast<int>(b);
  t.lds_tab = static_cast<int>(b + tab);
  t.lds = b + tab;
  t.tiles = static_cast<int>((nf + t.fc - 1) / t.fc);
  t.rtiles = (nrows + t.lines - 1) / t.lines;
  return t.lds <= kPassLdsMax && t.threads <= most;
}

// Stage the table rows of a tile (of at most `lines` lines) in LDS where a line's
// row serves four lanes or more (with one band per line the staging only adds a
// step: 81^3, 8 x 1 complex128 bands, y passes 29 -> 35 us) and both sides span
// less than 2 GiB.
void stage_tables(int n, int64_t lines, int64_t span, PassTile& t) {
  const size_t b = static_cast<size_t>(lines) * n * 4;
  if (n == pass_r1(n) || b > kPassTabMax || 4 * lines > t.fc + 4 || span >= (int64_t{1} << 31)) return;
  t.tab_lds = true;
  t.lds += b;
}

// The plane kernel's tile for planes of nx x ny points, if it serves them: at most
// one 128-byte line of elements, fewer where the planes alone are few workgroups
// for the 256 CUs, and all workgroups resident at once or nearly (a round trip,
// passes -> plane kernel: 32^3, 4 complex128 bands, 128 workgroups of one element
// 26.5 -> 22.3 us, 24.0 in 32 of four; 36x40x45, 20 bands, 225 workgroups 45 -> 35;
// 32^3, 64 bands, 256 of 128 KB 48 -> 46; more than that gains nothing: 32^3, 256
// bands, 1024: 116 -> 117; 48^3, 64 complex64 bands, 384 of 147 KB: 69 -> 77;
// 36x40x45, 200 complex128 bands, 2250: 181 -> 220).
void make_plane(int nx, int ny, int es, int64_t nel, int64_t nplanes, PlaneTile& t) {
  if (nx > kPlaneMaxN || ny > kPlaneMaxN) return;
  const auto tab = [](int n) {
    const int r1 = pass_r1(n);
    return static_cast<size_t>(r1 | 1) * (n / r1) * 16;
  };
  const size_t pts = static_cast<size_t>(nx) * ny * es;
  const size_t tables = tab(nx) + tab(ny) + 8 * static_cast<size_t>(nx) + 16;
  const auto blocks = [&](int fc) { return nplanes * ((nel + fc - 1) / fc); };
  int fc = static_cast<int>(std::min<int64_t>(nel, 128 / es));
  while (fc > 1 && (blocks(fc) < 192 || pts * fc + tables > kPassLdsMax)) fc = (fc + 1) / 2;
  t.fc = fc;
  t.tiles = static_cast<int>((nel + fc - 1) / fc);
  t.lds_twx = static_cast<int>((pts * fc + 15) & ~size_t{15});
  t.lds_twy = t.lds_twx + static_cast<int>(tab(nx));
  t.lds_x = t.lds_twy + static_cast<int>(tab(ny));
  t.lds = t.lds_x + 8 * static_cast<size_t>(nx);
  const int items = fc * std::max(ny * std::max(pass_r1(nx), nx / pass_r1(nx)),
                                  nx * std::max(pass_r1(ny), ny / pass_r1(ny)));
  t.threads = std::min(512, (items + 63) / 64 * 64);
  const int64_t resident = std::min<int64_t>(kPassLdsMax / t.lds, 2048 / t.threads);
  t.on = blocks(fc) <= 320 * resident;
}

}  // namespace

bool build_pass_plan(int nx, int ny, int nz, bool fp64, const std::vector<SphereTables>& sph,
                     const std::vector<int64_t>& colrow_max, int64_t s_budget, PassPlan& P) {
  P = PassPlan();
  if (nx > kPassMaxN || ny > kPassMaxN || nz > kPassMaxN) return false;
  if (!pass_r1(nx) || !pass_r1(ny) || !pass_r1(nz)) return false;
  const int cs = fp64 ? 16 : 8;     // bytes per value
  const int64_t cw = 128 / cs;      // values per 128-byte line
  const int64_t N = static_cast<int64_t>(nx) * ny * nz;
  const auto pad = [cw](int64_t v) { return (v + cw - 1) / cw * cw; };
  // complex64: two bands per lane where every count is even (odd counts would
  // end their band vectors in half elements, whose separate stores took the
  // inverse x pass of 240x200x250, 17 bands, from 0.77 to 2.9 ms)
  int v = fp64 ? 1 : 2;
  for (const auto& s : sph) {
    if (s.nb >= (1 << 20)) return false;
    if (s.nb % 2) v = 1;
  }
  P.elem = fp64 ? kElemC128 : v == 2 ? kElemC64x2 : kElemC64;
  const int es = cs * v;  // bytes per element
  size_t entries = 0;
  for (const auto& s : sph) entries += static_cast<size_t>(s.ncol) * nz;
  if (entries >= (size_t{1} << 31)) return false;
  P.gidx.reserve(entries);
  int64_t soff = 0, goff = 0, coff = 0, max_col = 0, max_slab = 0;
  int64_t span_z = 0, span_y = 0, span_x = 0;  // bytes of the larger side of a tile's accesses
  int32_t max_nel = 0, min_nel = 1 << 30;
  bool ragged = false;
  for (size_t i = 0; i < sph.size(); ++i) {
    const SphereTables& s = sph[i];
    PassSph d = {};
    d.sph_off = soff;
    d.grid_off = goff;
    d.col_off = coff;
    d.nb = s.nb;
    d.nel = s.nb / v;
    d.ncol = s.ncol;
    d.nslab = s.nslab;
    if (static_cast<int64_t>(s.ncol) * s.nb >= (int64_t{1} << 30) ||
        static_cast<int64_t>(s.nslab) * s.nb >= (int64_t{1} << 30))
      return false;
    // column slots by (y, x): the columns of a y row are neighbours, as the
    // slabs of a slab row are, so that the y pass reads and writes runs
    // (the columns come ordered by (x, y): one bucket per y keeps the x order)
    std::vector<int32_t> start(ny + 1, 0), order(s.ncol);
    for (int32_t c = 0; c < s.ncol; ++c) ++start[s.col_y[c] + 1];
    for (int y = 0; y < ny; ++y) start[y + 1] += start[y];
    for (int32_t c = 0; c < s.ncol; ++c) order[start[s.col_y[c]]++] = c;
    const int64_t row = static_cast<int64_t>(s.ncol) * s.nb;
    d.colrow = pad(row) <= colrow_max[i] ? pad(row) : row;
    d.srow = static_cast<int32_t>(pad(static_cast<int64_t>(s.nslab) * s.nb));
    d.gidx_off = static_cast<int32_t>(P.gidx.size());
    d.colidx_off = static_cast<int32_t>(P.colidx.size());
    d.xinv_off = static_cast<int32_t>(P.xinv.size());
    P.colidx.resize(P.colidx.size() + static_cast<size_t>(s.nslab) * ny, -1);
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
    max_col = std::max(max_col, static_cast<int64_t>(s.ncol) * d.nel);
    max_slab = std::max(max_slab, static_cast<int64_t>(s.nslab) * d.nel);
    max_nel = std::max(max_nel, d.nel);
    min_nel = std::min(min_nel, d.nel);
    ragged = ragged || s.nb % cw != 0;
    span_z = std::max(span_z, std::max(s.ns * s.nb, d.colrow * nz) * cs);
    span_y = std::max(span_y, std::max(d.colrow, static_cast<int64_t>(d.srow) * ny) * cs);
    span_x = std::max(span_x, static_cast<int64_t>(ny) * std::max<int64_t>(nx * static_cast<int64_t>(s.nb), d.srow) * cs);
    P.splane = std::max(P.splane, static_cast<int64_t>(d.srow) * ny);
    P.sph.push_back(d);
  }
  P.col_elems = coff;
  P.nplanes = static_cast<int>(sph.size()) * nz;
  if (!make_tile(nz, es, max_col, 1, false, ragged, P.tz) ||
      !make_tile(ny, es, max_slab, 1, false, ragged, P.ty) ||
      !make_tile(nx, es, max_nel, ny, true, ragged, P.tx))
    return false;
  stage_tables(nz, (P.tz.fc - 1 + min_nel - 1) / min_nel + 1, span_z, P.tz);
  stage_tables(ny, (P.ty.fc - 1 + min_nel - 1) / min_nel + 1, span_y, P.ty);
  stage_tables(nx, 1, span_x, P.tx);
  // tiles that cut the band vectors of a ragged band count inside a 128-byte
  // line meet their neighbours in one L2 (whole lines spread over the XCDs:
  // sending 16 runs of whole lines to one XCD took 10.0 ms instead of 7.9 ms at
  // 128^3, 256 complex128 bands)
  if (ragged) {
    P.tz.group = 8;
    P.ty.group = std::min(8, P.ty.tiles);
    P.tx.group = P.tx.tiles;
  }
  for (auto& d : P.sph) {
    d.ztile = P.ztotal;
    P.ztotal += static_cast<int>((static_cast<int64_t>(d.ncol) * d.nel + P.tz.fc - 1) / P.tz.fc);
  }
  make_plane(nx, ny, es, max_nel, P.nplanes, P.plane);
  // equal groups of planes within the budget
  const int64_t most = std::max<int64_t>(1, s_budget / (P.splane * cs));
  const int64_t groups = (P.nplanes + most - 1) / most;
  P.group = static_cast<int>((P.nplanes + groups - 1) / groups);
  return static_cast<int64_t>(P.group) * std::max(P.ty.tiles, P.tx.tiles * P.tx.rtiles) < (int64_t{1} << 31);
}

}  // namespace fftb
