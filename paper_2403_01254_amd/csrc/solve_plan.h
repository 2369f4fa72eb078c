// Block-sparse elimination of a problem's system, planned on the host from which frames share an edge.
//
// A map's frames see their neighbours only: 64 frames with 6 edges each fill a twentieth of the dense triangle, and the
// blocks of the factor fit one workgroup's LDS where the dense triangle (0.6 MB) does not.  The plan holds an
// elimination order of small fill, the blocks of L column by column, and for each column the block products that
// update the columns after it.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

namespace rkhsba {

constexpr int kLdsSystem = 128;            // unknowns of the largest system whose dense triangle is eliminated in LDS
constexpr size_t kSparseLds = 148 * 1024;  // blocks, right side, a column's products and the plan
constexpr int kSparseMaxFrames = 512;

// Words of a plan (16 bits each): n frames, off-diagonal blocks, updates, most block rows below a diagonal block; the
// order; for each column its first off-diagonal block and its first update (n + 1 each); the off-diagonal blocks'
// rows, then their columns; 3 words an update: off-diagonal i, k, target id.  Block ids: p for the diagonal block of
// column p, then n + o for the off-diagonal block o in column order; rows and columns are positions in the order.
constexpr int kSparseHeader = 4;
#if defined(__HIP__) || defined(__HIPCC__)
#define RKHSBA_HD __host__ __device__
#else
#define RKHSBA_HD
#endif
RKHSBA_HD inline int sparse_words(int n_frames, int n_off, int n_upd) {
  return kSparseHeader + 3 * n_frames + 2 + 2 * n_off + 3 * n_upd;
}
// LDS bytes: the doubles (blocks; right side; the system's diagonal; products of a column's rows and of the right side;
// a diagonal block's L) and the plan.
RKHSBA_HD inline size_t sparse_doubles(int n_frames, int n_off, int rows_max) {
  return 36 * (size_t)(n_frames + n_off) + 12 * (size_t)n_frames + 6 * (size_t)(6 * rows_max + 1) + 16;
}

// The plan of n frames with the given adjacency (n x n, symmetric), or nothing where it would not fit.
inline std::vector<uint16_t> sparse_plan(int n, std::vector<uint8_t> adj) {
  std::vector<uint16_t> plan;
  if (n < 1 || n > kSparseMaxFrames) return plan;
  const size_t max_blocks = kSparseLds / (36 * sizeof(double));
  // greedy minimum degree (ties: the earlier frame); eliminating a frame joins its remaining neighbours
  std::vector<int> order, position(n, -1), degree(n, 0);
  auto count = [&](int f) {
    degree[f] = 0;
    for (int g = 0; g < n; ++g) degree[f] += position[g] < 0 && g != f && adj[(size_t)f * n + g];
  };
  for (int f = 0; f < n; ++f) count(f);
  std::vector<std::vector<int>> below(n);  // frames of column p's off-diagonal blocks
  size_t blocks = n, updates = 0;
  size_t rows_max = 0;
  for (int p = 0; p < n; ++p) {
    int best = -1;
    for (int f = 0; f < n; ++f)
      if (position[f] < 0 && (best < 0 || degree[f] < degree[best])) best = f;
    position[best] = p;
    order.push_back(best);
    for (int g = 0; g < n; ++g)
      if (position[g] < 0 && adj[(size_t)best * n + g]) below[p].push_back(g);
    blocks += below[p].size();
    updates += below[p].size() * (below[p].size() + 1) / 2;
    rows_max = std::max(rows_max, below[p].size());
    if (blocks > max_blocks || updates > 60000) return plan;
    for (int g : below[p])
      for (int h : below[p])
        if (g != h) adj[(size_t)g * n + h] = 1;
    for (int g : below[p]) count(g);
  }
  const int n_off = (int)blocks - n, n_upd = (int)updates;
  const size_t words = (size_t)sparse_words(n, n_off, n_upd);
  if (sparse_doubles(n, n_off, (int)rows_max) * sizeof(double) + words * sizeof(uint16_t) > kSparseLds ||
      6 * rows_max + 1 > 1024)
    return plan;
  std::vector<std::vector<int>> rows(n);  // positions below the diagonal, ascending
  std::vector<int> first(n + 1, 0);
  for (int p = 0; p < n; ++p) {
    for (int f : below[p]) rows[p].push_back(position[f]);
    std::sort(rows[p].begin(), rows[p].end());
    first[p + 1] = first[p] + (int)rows[p].size();
  }
  auto put = [&](int v) { plan.push_back((uint16_t)v); };
  put(n);
  put(n_off);
  put(n_upd);
  put((int)rows_max);
  for (int f : order) put(f);
  for (int p = 0; p <= n; ++p) put(first[p]);
  int u = 0;
  put(0);
  for (int p = 0; p < n; ++p) {
    u += (int)(rows[p].size() * (rows[p].size() + 1) / 2);
    put(u);
  }
  for (int p = 0; p < n; ++p)
    for (int r : rows[p]) put(r);
  for (int p = 0; p < n; ++p)
    for (size_t k = 0; k < rows[p].size(); ++k) put(p);
  for (int p = 0; p < n; ++p)
    for (size_t i = 0; i < rows[p].size(); ++i)
      for (size_t k = 0; k <= i; ++k) {
        const int ri = rows[p][i], rk = rows[p][k];
        put(first[p] + (int)i);
        put(first[p] + (int)k);
        if (ri == rk) {
          put(ri);
        } else {
          const auto at = std::lower_bound(rows[rk].begin(), rows[rk].end(), ri);
          put(n + first[rk] + (int)(at - rows[rk].begin()));
        }
      }
  return plan;
}

}  // namespace rkhsba
