// Where a paint leaves the halo of its windows (gfx950).
//
// A block's window has one layer of cells above the block's own 8^3 along every
// axis.  They belong to the blocks above: the 64 above in z only to the lowest z
// layer of the next block in z, and so on for the seven combinations of axes.
// Each combination is a field of its own, indexed by the block the values belong
// to, so that every entry has exactly one block that paints it: the blocks with a
// single work item store theirs without atomics, and the consumer of the grid
// (the z pass of the FFT, or k_add_halo) adds them while it reads:
//   z   [z / 8][x][y]      y   [y / 8][x][z]      x   [x / 8][z / 8][y][z mod 8]
//   yz  [y / 8][x / 8][z / 8][x mod 8]  xz  [x / 8][z / 8][y]      xy  [x / 8][y / 8][z]
//   xyz [x / 8][y / 8][z / 8]
// (a cell with x, y and z multiples of 8 takes all seven.)  The consumers
// go through planes of x row by row: what a row y = 0 mod 8 takes along y and what the
// rows of a plane x = 0 mod 8 take along x (in the slab layout of the grid itself)
// then lies as the rows do.
// A pass of its own that added the x and y halos from a staging slot per work item
// into the grid took 33 us for one field and 58 for three at 256^3 in FP32 (4 % of an
// evaluation): on a y face it moves whole cache lines for one row of four.
#pragma once

#include "common.h"

namespace ic {

struct HaloMap {
  int lm, lnb;  // log2 of the grid side and of the blocks per side
  using U = unsigned;
  __host__ __device__ explicit constexpr HaloMap(int lm_) : lm(lm_), lnb(lm_ - 3) {}
  __host__ __device__ constexpr U face() const { return 1u << (2 * lm + lnb); }
  __host__ __device__ constexpr U edge() const { return 1u << (lm + 2 * lnb); }
  // entries of one field's halo, a multiple of 128 bytes
  __host__ __device__ constexpr U size() const {
    return (3 * face() + 3 * edge() + (1u << (3 * lnb)) + 31u) & ~31u;
  }
  __host__ __device__ constexpr U z(U bz, U x, U y) const { return (bz << lm | x) << lm | y; }
  __host__ __device__ constexpr U y(U by, U x, U zz) const {
    return face() + ((by << lm | x) << lm | zz);
  }
  __host__ __device__ constexpr U x(U bx, U yy, U zz) const {
    return 2 * face() + (((bx << lnb | zz >> 3) << lm | yy) << 3 | (zz & 7u));
  }
  __host__ __device__ constexpr U yz(U by, U bz, U x) const {
    return 3 * face() + (((by << lnb | x >> 3) << lnb | bz) << 3 | (x & 7u));
  }
  __host__ __device__ constexpr U xz(U bx, U bz, U y) const {
    return 3 * face() + edge() + ((bx << lnb | bz) << lm | y);
  }
  __host__ __device__ constexpr U xy(U bx, U by, U z) const {
    return 3 * face() + 2 * edge() + ((bx << lnb | by) << lm | z);
  }
  __host__ __device__ constexpr U xyz(U bx, U by, U bz) const {
    return 3 * face() + 3 * edge() + ((bx << lnb | by) << lnb | bz);
  }
  // Entry of window cell (kx, ky, kz), at least one of them 8, of the block at
  // (bx, by, bz).
  __device__ __forceinline__ U of_window(U bx, U by, U bz, U kx, U ky, U kz) const {
    const U m = (1u << lnb) - 1;
    const U ux = (bx + 1) & m, uy = (by + 1) & m, uz = (bz + 1) & m;
    const U cx = bx << 3 | kx, cy = by << 3 | ky, cz = bz << 3 | kz;
    if (kx < 8)
      return ky < 8 ? z(uz, cx, cy) : (kz < 8 ? y(uy, cx, cz) : yz(uy, uz, cx));
    if (ky < 8) return kz < 8 ? x(ux, cy, cz) : xz(ux, uz, cy);
    return kz < 8 ? xy(ux, uy, cz) : xyz(ux, uy, uz);
  }
  // What cell (cx, cy, cz), cx a multiple of 8, takes from the x part of the halo h.
  template <typename V>
  __device__ __forceinline__ V sum_x(const V* __restrict__ h, U cx, U cy, U cz) const {
    const bool on_y = (cy & 7u) == 0, on_z = (cz & 7u) == 0;
    const U bx = cx >> 3, by = cy >> 3, bz = cz >> 3;
    // loaded whether the cell takes them or not: no load waits for another
    const V a = h[x(bx, cy, cz)], b = h[xz(bx, bz, cy)], c = h[xy(bx, by, cz)],
            d = h[xyz(bx, by, bz)];
    return a + (on_z ? b : V(0)) + (on_y ? c : V(0)) + (on_y && on_z ? d : V(0));
  }
  // What any cell takes from it.
  template <typename V>
  __device__ __forceinline__ V sum(const V* __restrict__ h, U cx, U cy, U cz) const {
    const bool on_y = (cy & 7u) == 0, on_z = (cz & 7u) == 0;
    const U by = cy >> 3, bz = cz >> 3;
    V v = V(0);
    if (on_z) v += h[z(bz, cx, cy)];
    if (on_y) {
      const V a = h[y(by, cx, cz)], b = h[yz(by, bz, cx)];
      v += a;
      v += on_z ? b : V(0);
    }
    if ((cx & 7u) == 0) v += sum_x(h, cx, cy, cz);
    return v;
  }
};

}  // namespace ic
