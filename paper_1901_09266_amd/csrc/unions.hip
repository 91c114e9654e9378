// Host construction of the pattern's tiles for the kernels of several days
// (days_kernels.hip): 16 lines by the union of their columns.
//
// A tile multiplies every column of the union with all 16 lines, so what its
// lines have in common decides the padding.  Links usually come in driving
// order and share most of their ODs with their neighbours (17 of 12.5 columns
// per link on a corridor with 8% incidence); ODs come in any order, so a second
// order, by first and then last column, is tried and kept when its unions are
// smaller in total.
#include <algorithm>
#include <numeric>
#include <vector>

#include "dode_internal.h"

namespace {

// Sorted union of the columns of lines order[16i .. 16i+15], per tile.
std::vector<std::vector<int32_t>> unions(const std::vector<int32_t>& order, int32_t n_cols,
                                         const std::vector<int32_t>& ptr,
                                         const std::vector<int32_t>& idx) {
  const int32_t nt = ((int32_t)order.size() + 15) / 16;
  std::vector<std::vector<int32_t>> u(nt);
  std::vector<int32_t> seen(n_cols, -1);
  for (int32_t i = 0; i < nt; ++i) {
    for (size_t r = 16 * (size_t)i; r < std::min(order.size(), 16 * (size_t)(i + 1)); ++r)
      for (int32_t j = ptr[order[r]]; j < ptr[order[r] + 1]; ++j)
        if (seen[idx[j]] != i) {
          seen[idx[j]] = i;
          u[i].push_back(idx[j]);
        }
    std::sort(u[i].begin(), u[i].end());
  }
  return u;
}

// Runs of 16 columns of a union.
int32_t n_runs(const std::vector<int32_t>& u) { return ((int32_t)u.size() + 15) / 16; }

int64_t all_runs(const std::vector<std::vector<int32_t>>& u) {
  int64_t n = 0;
  for (const auto& c : u) n += n_runs(c);
  return n;
}

}  // namespace

HostUnion build_union(int32_t n_lines, int32_t n_cols, const std::vector<int32_t>& ptr,
                      const std::vector<int32_t>& idx, const std::vector<int32_t>& slot, bool f64) {
  std::vector<int32_t> order(n_lines);
  std::iota(order.begin(), order.end(), 0);
  auto u = unions(order, n_cols, ptr, idx);
  std::vector<int32_t> sorted = order;
  std::stable_sort(sorted.begin(), sorted.end(), [&](int32_t x, int32_t y) {
    auto key = [&](int32_t l, bool last) {
      return ptr[l + 1] > ptr[l] ? idx[last ? ptr[l + 1] - 1 : ptr[l]] : n_cols;
    };
    return std::make_pair(key(x, false), key(x, true)) < std::make_pair(key(y, false), key(y, true));
  });
  auto us = unions(sorted, n_cols, ptr, idx);
  if (all_runs(us) < all_runs(u)) {
    u.swap(us);
    order.swap(sorted);
  }
  HostUnion out;
  const int32_t nt = out.n_tiles = (int32_t)u.size();
  order.resize((size_t)nt * 16, -1);
  std::vector<int32_t> run(4 * (size_t)nt), off(nt + 1, 0), col, map;
  for (int32_t k = 0; k < 4 * nt; ++k) {
    const int32_t* l = order.data() + 4 * k;
    run[k] = l[0] >= 0 && l[0] % 4 == 0 && l[1] == l[0] + 1 && l[2] == l[0] + 2 && l[3] == l[0] + 3;
  }
  std::vector<int32_t> at(n_cols, -1);   // entry of a line at a column
  for (int32_t i = 0; i < nt; ++i) {
    const int32_t nr = n_runs(u[i]);
    const size_t r0 = off[i], m0 = map.size();
    off[i + 1] = off[i] + nr;
    // column 16 r + 4 j + g of a run: product j, lane group g; padding columns
    // repeat the last (value 0)
    for (int32_t k = 0; k < 16 * nr; ++k)
      col.push_back(u[i][std::min<size_t>(16 * (k / 16) + 4 * (k % 4) + k % 16 / 4, u[i].size() - 1)]);
    map.resize(m0 + 256 * (size_t)nr, -1);
    for (int32_t r = 0; r < 16; ++r) {
      const int32_t l = order[16 * (size_t)i + r];
      if (l < 0) continue;
      for (int32_t j = ptr[l]; j < ptr[l + 1]; ++j) at[idx[j]] = slot[j];
      // lane of tile row r: the FP64 product gives lane group g the rows g,
      // g+4, g+8, g+12 of its operand, the FP32 product rows 4g..4g+3
      const int32_t m = f64 ? 4 * (r % 4) + r / 4 : r;
      for (size_t k = 0; k < u[i].size(); ++k)
        map[256 * (r0 + k / 16) + 4 * (16 * (k % 4) + m) + k % 16 / 4] = at[u[i][k]];
      for (int32_t j = ptr[l]; j < ptr[l + 1]; ++j) at[idx[j]] = -1;
    }
  }
  out.code_of.swap(map);
  for (const auto* v : {&order, &run, &col, &off})   // columns 16-byte aligned
    out.buf.insert(out.buf.end(), v->begin(), v->end());
  return out;
}

DevUnion HostUnion::at(const int32_t* p) const {
  DevUnion d;
  d.n_tiles = n_tiles;
  d.line = p;
  d.run = p + 16 * (size_t)n_tiles;
  d.col = p + 20 * (size_t)n_tiles;
  d.off = p + buf.size() - (n_tiles + 1);
  return d;
}
