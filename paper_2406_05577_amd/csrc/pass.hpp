// Axis passes: the transform as three kernels, one axis each, for every axis
// length n = R1*R2 with codelets R1 and R2 (all 2,3,5-smooth lengths up to
// 512). Shared by the host planner (pass_plan.cpp) and the kernels
// (kernels_pass.hpp).
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "plan.hpp"

namespace fftb {

// ---- the split n = R1*R2 ---------------------------------------------------
constexpr int kPassMaxN = 512;
// in-register codelets the passes use
constexpr bool pass_codelet(int r) {
  return r == 1 || r == 2 || r == 3 || r == 4 || r == 5 || r == 6 || r == 8 || r == 9 || r == 10 ||
         r == 12 || r == 15 || r == 16 || r == 18 || r == 20 || r == 24 || r == 25 || r == 27 ||
         r == 32;
}
// First stage: one codelet up to 16, else the smallest codelet at or above the
// root of n whose cofactor is a codelet too (the two stages then hold about
// as many values per thread and keep about as many threads busy). 0: none.
constexpr int pass_r1(int n) {
  if (n <= 16 && pass_codelet(n)) return n;
  for (int r = 2; r <= 32; ++r)
    if (r * r >= n && n % r == 0 && pass_codelet(r) && pass_codelet(n / r)) return r;
  return 0;
}

// Threads per workgroup the kernels are compiled for (16-byte elements of longer
// codelets need more than the 128 registers that 1024 threads leave).
constexpr int pass_max_threads(int n, bool small) {
  return small || pass_r1(n) <= 12 ? 1024 : 512;
}
// Longest x and y lines of the plane kernel: second factors of at most 8.
constexpr int kPlaneMaxN = 64;

// Blocks of a launch whose tiles go to the XCDs in runs of `group`.
constexpr int pass_grid(int total, int group) {
  return (total + 8 * group - 1) / (8 * group) * (8 * group);
}

enum { kPassZ = 0, kPassY = 1, kPassX = 2 };
// (kPassPotential: the x pass that multiplies by V, with or without the way back)
enum PassMode { kPassInverse, kPassForward, kPassPotential };
// What a lane holds of a point: one complex64, two neighbouring bands of
// complex64, one complex128 value.
enum PassElem { kElemC64 = 0, kElemC64x2 = 1, kElemC128 = 2 };

// Per-sphere descriptor (device resident); offsets and strides in complex
// values (data) or int32 entries (tables).
struct PassSph {
  int64_t sph_off, grid_off, col_off;
  int64_t colrow;      // stride between z planes of the column scratch
  int32_t nb, ncol, nslab;
  int32_t nel;         // elements per band vector
  int32_t srow;        // stride between y rows of a slab plane
  int32_t gidx_off;    // ncol*nz: (column slot, z) -> coefficient or -1
  int32_t colidx_off;  // nslab*ny: (slab, y) -> column slot or -1
  int32_t xinv_off;    // nx: x -> slab or -1
  int32_t ztile;       // first tile of the sphere in the z pass
};

struct PassArgs {
  int kind;            // kPassZ / kPassY / kPassX
  int nx, ny, nz, nsph;
  int p0;              // y, x: first plane of the group (plane = sphere*nz + z)
  int tiles;           // y, x: band tiles per plane / per row group
  int rtiles;          // x: row groups per plane
  int total;           // tiles of the launch
  int group;           // consecutive tiles that run on one XCD
  int fc, lines;       // a tile: fc elements of the fast dimension x `lines` rows (x)
  int lds_tw;          // byte offset of the twiddle table in LDS
  int lds_tab;         // byte offset of the staged table rows
  int tab_lds;         // stage the tile's table rows in LDS, 32-bit offsets on both sides
  int nt_dense, nt_gather;  // streaming accesses on either side
  int64_t splane;      // stride between planes of the slab scratch
  const PassSph* sph;
  const int32_t* tab;  // gidx / colidx / xinv
  const void *root, *root_lo;  // exp(-2*pi*i*j/n) (FP32: hi and lo)
  const void* src;
  void* dst;
  const void* pot;     // potential x pass: V[z][y][x]
  void* back;          // and the slab scratch its transform back goes to, or null
  double scale;        // z, forward: 1/N (1 elsewhere)
};

struct PlaneArgs {
  int nx, ny, nz;
  int r1x, r1y;        // first factors of the axes' splits
  int tiles, fc;       // a tile: one plane of fc elements
  int total;           // tiles of the launch
  int lds_twx, lds_twy, lds_x;  // byte offsets in LDS: twiddles, slab tables
  const PassSph* sph;
  const int32_t *colidx, *xinv;
  const void *rootx, *rootx_lo, *rooty, *rooty_lo;
  const void* col_in;
  void* col_out;       // (potential: null without the way back)
  void* grid;
  const void* pot;
};

// ---- host side -------------------------------------------------------------
struct PassTile {
  int fc = 0, lines = 1, threads = 64;
  int tiles = 0, rtiles = 0;
  int group = 1;  // consecutive tiles that share an XCD
  size_t lds = 0;
  int lds_tw = 0, lds_tab = 0;
  bool tab_lds = false;
};

// The plane kernel's tile (on: the planes run as one launch of it).
struct PlaneTile {
  bool on = false;
  int fc = 0, threads = 0, tiles = 0;
  size_t lds = 0;
  int lds_twx = 0, lds_twy = 0, lds_x = 0;
};

struct PassPlan {
  PlaneTile plane;
  std::vector<PassSph> sph;
  std::vector<int32_t> gidx, colidx, xinv;
  PassTile tz, ty, tx;
  int ztotal = 0;         // tiles of the z pass
  PassElem elem = kElemC64;
  int nplanes = 0;        // planes of all spheres
  int group = 0;          // planes per y/x launch pair
  int64_t splane = 0;     // slab scratch values per plane
  int64_t col_elems = 0;  // column scratch values
  int64_t s_elems() const { return splane * group; }
  // Four groups or more: the planes on two streams, each with half of the slab
  // scratch, so that the end of a launch overlaps the other stream's launches
  // (256^3, 24 complex128 bands, a round trip 5.41 -> 5.15 ms; 144x160x180, 128
  // bands, the potential step 5.38 -> 5.19 ms; 128^3, 256 complex64 bands, forward
  // 1.82 -> 1.74 ms). Fewer lose by the smaller launches (108x100x120, 50 complex64
  // bands, two groups: 0.497 -> 0.507 ms).
  bool two_streams() const { return !plane.on && group >= 2 && nplanes > 3 * group; }
};

// Build the pass plan; false where a length has no split or a size does not
// fit its index types. colrow_max: per sphere the most values a z plane of
// its columns may take (rows are padded only within it); s_budget: the
// most bytes the slab scratch of one group should take.
bool build_pass_plan(int nx, int ny, int nz, bool fp64, const std::vector<SphereTables>& sph,
                     const std::vector<int64_t>& colrow_max, int64_t s_budget, PassPlan& out);

}  // namespace fftb
