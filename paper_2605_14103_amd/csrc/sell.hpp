// Sliced ELLPACK (SELL) storage shared by the solvers: device view, host
// builder and device copies.
#pragma once

#include <hip/hip_runtime.h>

#include <tuple>
#include <utility>
#include <vector>

#include "common.hpp"

namespace pfx {

// Sliced ELLPACK: rows are grouped in slices of 64 (one wavefront), each
// slice padded to its longest row.  Entry p of the row on lane l of slice s
// sits at off[s] + 64 p + l; padding entries have column 0 and value 0.
template <typename V>
struct Sell {
  const int* off;     // [n_slices]
  const int* width;   // [n_slices]
  const int* col;
  const V* val;
};

// Packed sliced layout: the slices of Sell, but each lane's entries are
// grouped in fours.  Group g of the row on lane l of slice s is group index
// off[s] + 64 g + l; it holds four 16-bit columns at col[4 index ..] and four
// values.  The values of the 64 groups of one (slice, g) lie in sizeof(V) / 4
// planes of 16 bytes per lane, so a group is one 8-byte column load and
// sizeof(V) / 4 16-byte value loads, and each load of a wave covers
// consecutive addresses.  (With a lane's values side by side instead, four
// lanes of a complex FP64 load touch two lines, and the address unit takes
// twice as long: the Jacobian-vector product of the 2000-bus grid took 29 k
// cycles against 24 k with four scenarios per CU, by clock reads in a copy of
// the kernel.)  Offsets and widths count
// groups; padding entries have column 0 and value 0.  Entry
// p of that row is entry number 4 (off[s] + 64 (p / 4) + l) + p % 4, with its value
// at psell_at of that number.
template <typename V>
__host__ __device__ inline int64_t psell_at(int64_t entry) {
  constexpr int per = 16 / (int)sizeof(V);   // values in 16 bytes
  const int64_t g = entry / 4, block = g / 64, lane = g % 64, u = entry % 4;
  return block * 256 + u / per * (64 * per) + lane * per + u % per;
}

// the entry number of a value index (the inverse of psell_at)
template <typename V>
__host__ __device__ inline int64_t psell_entry(int64_t at) {
  constexpr int per = 16 / (int)sizeof(V);
  const int64_t block = at / 256, r = at % 256, plane = r / (64 * per), lane = r % (64 * per) / per;
  return 4 * (64 * block + lane) + plane * per + r % per;
}

template <typename V>
struct PSell {
  const int* off;
  const int* width;
  const unsigned short* col;
  const V* val;
};

template <typename T>
struct Vec2;
template <>
struct Vec2<double> {
  using type = double2;
};
template <>
struct Vec2<float> {
  using type = float2;
};

// Host-built sliced ELLPACK with device copies of its values in FP64 and FP32.
struct SellBuffers {
  int n_slices = 0;
  long entries = 0;
  DeviceBuffer off, width, col, val64, val32;
  template <typename V>
  Sell<V> view() const;
};

// Host side: rows (a multiple of 64 of them) as (column, value re, value im)
// lists; builds slices of 64 consecutive rows whose widths are at least 1 and
// multiples of `quantum` (padding entries are zeros).
using SellEntry = std::tuple<int, double, double>;
using SellRow = std::vector<SellEntry>;

struct SellHost {
  std::vector<int> off, width, col;
  std::vector<double> re, im;
  long entries = 0;
};

SellHost build_sell(const std::vector<SellRow>& rows, int quantum = 1);

// Device copies: values in FP64 and FP32, complex values as (re, im) pairs.
void upload_sell(Context* ctx, const SellHost& h, bool cplx, SellBuffers& b);

// Packed layout (columns below 65536) with device copies of its values in
// FP64 and FP32 (complex values as (re, im) pairs); rows as for build_sell (a
// multiple of 64).
struct PSellBuffers {
  int n_slices = 0;
  long entries = 0;
  DeviceBuffer off, width, col, val64, val32;
  template <typename V>
  PSell<V> view() const;
};
// `parts`: what some kernel reads (the rest takes no memory and no copy); without
// `slices` the kernel has the offsets and widths from lists of its own.
// Returns the slices' group offsets and widths (as uploaded).
struct PSellParts {
  bool fp64 = true, fp32 = true, slices = true;
};
std::pair<std::vector<int>, std::vector<int>> upload_psell(Context* ctx, const std::vector<SellRow>& rows,
                                                           PSellBuffers& b, bool cplx = false,
                                                           PSellParts parts = {});

}  // namespace pfx
