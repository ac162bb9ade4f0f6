// Windowed layout of an explicit matrix (host side, at lattice creation).
//
// The sparse Chebyshev step gathers phi_n at the column indices of every
// entry.  In the slice layout of the input order a slice of 128 consecutive
// rows touches a long, mostly unused column range, and each gathered value
// is read from the caches once per entry that names it.  Here the rows are
// regrouped into slices of nr (256 or 128) rows that are compact in the matrix graph
// (grown breadth-first from the lowest unassigned row, so a slice is a ball
// of neighbouring orbitals), and each slice records its window: the sorted
// distinct columns its entries name.  The recursion kernel stages a slice's
// window of phi_n in LDS once per step and gathers from there with 16-bit
// window-local indices; rows keep their index in every vector (only slice
// membership changes), so nothing outside the recursion kernel sees the
// regrouping.
#include <algorithm>
#include <cstdint>
#include <cstring>
#include <functional>
#include <thread>
#include <vector>

#include "csp_internal.h"

namespace csp {

bool build_ell_windows(int64_t N, int D, const int32_t* col, const double* val, int nr,
                       const std::function<bool(const std::vector<int32_t>&)>& accept,
                       EllWindows* w) {
  // entries in quads: slice, quad q of a row's entries 4q .. 4q + 3, row,
  // entry inside the quad ([n_sl][D4][nr][4]); entries past D are padding
  const int D4 = (D + 3) / 4;
  w->D4 = D4;
  w->nr = nr;
  w->rows.clear();
  w->rows.reserve((size_t)(N + N / 16 + 2 * nr));

  // ---- slices grown breadth-first over the matrix graph.  A search that
  // dead-ends among assigned rows leaves its rows (a pocket) for later.
  std::vector<uint8_t> taken((size_t)N, 0);
  std::vector<int32_t> queue, rest;
  queue.reserve(nr);
  for (int64_t seed = 0; seed < N; ++seed) {
    if (taken[seed]) continue;
    queue.clear();
    queue.push_back(static_cast<int32_t>(seed));
    taken[seed] = 1;
    for (size_t head = 0; head < queue.size() && (int)queue.size() < nr; ++head) {
      const int32_t* cr = col + (size_t)queue[head] * D;
      for (int k = 0; k < D && (int)queue.size() < nr; ++k) {
        const int32_t j = cr[k];
        if (j >= 0 && !taken[j]) {
          taken[j] = 1;
          queue.push_back(j);
        }
      }
    }
    std::vector<int32_t>& to = (int)queue.size() == nr ? w->rows : rest;
    to.insert(to.end(), queue.begin(), queue.end());
  }
  // ---- the pockets' rows, in the order they were found.  A slice of rows
  // from many pockets names far more columns than the others, gathers from
  // global memory and sets the time of the whole step (45 us a launch of
  // 200^2 rows at D = 121, 5 columns, against 30 us), so a slice is closed,
  // its other lanes idle, before its window passes that of the full slices
  // (the 90th percentile and a tenth).  At most a sixteenth of the rows may
  // be lost to idle lanes, and no further round of the 256 CUs begun; after
  // that, or with no full slice to compare with, slices are filled.
  {
    std::vector<int32_t> mark((size_t)N, -1);
    int32_t stamp = 0;
    auto added = [&](int32_t r) {   // columns that row r would add to the window
      const int32_t* cr = col + (size_t)r * D;
      int n = 0;
      for (int k = 0; k < D; ++k) n += cr[k] >= 0 && mark[cr[k]] != stamp;
      return n;
    };
    auto add = [&](int32_t r) {     // (columns named twice by a row count once)
      const int32_t* cr = col + (size_t)r * D;
      int n = 0;
      for (int k = 0; k < D; ++k)
        if (cr[k] >= 0 && mark[cr[k]] != stamp) {
          mark[cr[k]] = stamp;
          ++n;
        }
      return n;
    };
    int64_t cap = INT64_MAX;
    const int64_t full = (int64_t)w->rows.size() / nr;
    if (full > 0 && !rest.empty()) {
      // windows of up to 256 full slices spread over all of them
      std::vector<int64_t> sz;
      for (int64_t q = 0; q < std::min<int64_t>(full, 256); ++q) {
        const int32_t* rows = w->rows.data() + (size_t)(q * full / std::min<int64_t>(full, 256)) * nr;
        ++stamp;
        int64_t W = 0;
        for (int t = 0; t < nr; ++t) W += add(rows[t]);
        sz.push_back(W);
      }
      std::sort(sz.begin(), sz.end());
      cap = sz[sz.size() * 9 / 10] * 11 / 10;
    }
    // idle lanes allowed: no more slices than the CUs' current round holds
    const int64_t least = (N + nr - 1) / nr;
    int64_t idle = std::min<int64_t>(N / 16, ((least + 255) / 256 * 256 - least) * nr);
    ++stamp;
    int cnt = 0;
    int64_t W = 0;
    for (int32_t r : rest) {
      if (cnt > 0 && cnt < nr && W + added(r) > cap && idle >= nr - cnt) {
        idle -= nr - cnt;
        w->rows.insert(w->rows.end(), nr - cnt, -1);
        cnt = nr;
      }
      if (cnt == nr) {
        ++stamp;
        cnt = 0;
        W = 0;
      }
      W += add(r);
      w->rows.push_back(r);
      ++cnt;
    }
    if (w->rows.size() % nr) w->rows.insert(w->rows.end(), nr - w->rows.size() % nr, -1);
  }
  const int64_t n_sl = (int64_t)w->rows.size() / nr;
  const size_t n = (size_t)n_sl * D4 * nr * 4;
  w->n_slices = n_sl;
  w->sizes.assign((size_t)n_sl, 0);
  // rows ascending inside the slice, idle lanes last: neighbouring lanes then
  // read neighbouring rows of the vectors and, for matrices with a regular
  // pattern, neighbouring positions of the window (fewer LDS bank conflicts)
  for (int64_t sl = 0; sl < n_sl; ++sl) {
    int32_t* rows = w->rows.data() + (size_t)sl * nr;
    std::sort(rows, std::find(rows, rows + nr, -1));
  }

  // ---- windows, slices split over threads (each with its own column marks)
  std::vector<std::vector<int32_t>> wins((size_t)n_sl);
  auto windows = [&](int64_t sl_lo, int64_t sl_hi) {
    std::vector<uint8_t> mark((size_t)N, 0);
    for (int64_t sl = sl_lo; sl < sl_hi; ++sl) {
      const int32_t* rows = w->rows.data() + (size_t)sl * nr;
      std::vector<int32_t>& win = wins[sl];
      for (int t = 0; t < nr; ++t) {
        const int32_t r = rows[t];
        if (r < 0) continue;
        const int32_t* cr = col + (size_t)r * D;
        for (int k = 0; k < D; ++k) {
          const int32_t j = cr[k];
          if (j >= 0 && !mark[j]) {
            mark[j] = 1;
            win.push_back(j);
          }
        }
      }
      std::sort(win.begin(), win.end());
      for (int32_t j : win) mark[j] = 0;
      w->sizes[sl] = static_cast<int32_t>(win.size());
    }
  };
  // ---- the entries in slice order
  auto entries = [&](int64_t sl_lo, int64_t sl_hi) {
    std::vector<int32_t> pos((size_t)N, 0);
    for (int64_t sl = sl_lo; sl < sl_hi; ++sl) {
      const int32_t* rows = w->rows.data() + (size_t)sl * nr;
      const std::vector<int32_t>& win = wins[sl];
      for (size_t q = 0; q < win.size(); ++q) pos[win[q]] = static_cast<int32_t>(q);
      const size_t o = (size_t)sl * D4 * nr * 4;
      for (int t = 0; t < nr; ++t) {
        const int32_t r = rows[t];
        for (int k = 0; k < 4 * D4; ++k) {
          const size_t e = o + ((size_t)(k >> 2) * nr + t) * 4 + (k & 3);
          if (r < 0 || k >= D) {
            // lanes past N and entries past D: a valid index with the value 0
            w->col[e] = r < 0 ? 0 : r;
            w->loc[e] = 0;
            continue;
          }
          const int32_t j = col[(size_t)r * D + k];
          const double v = j >= 0 ? val[(size_t)r * D + k] : 0.0;
          // padding entries: the row itself with the value 0 (the row need
          // not be in its own window, so its local index is 0, also with
          // value 0)
          w->col[e] = j >= 0 ? j : r;
          w->loc[e] = j >= 0 && pos[j] <= 0xffff ? static_cast<uint16_t>(pos[j]) : 0;
          w->v64[e] = v;
          w->v32[e] = static_cast<float>(v);
        }
      }
    }
  };
  int nt = (int)std::min<int64_t>(16, std::max<unsigned>(1u, std::thread::hardware_concurrency()));
  if (N * (int64_t)D < (int64_t)1 << 22) nt = 1;
  nt = (int)std::min<int64_t>(nt, n_sl);
  auto split = [&](const std::function<void(int64_t, int64_t)>& f) {
    std::vector<std::thread> pool;
    for (int q = 1; q < nt; ++q) pool.emplace_back(f, n_sl * q / nt, n_sl * (q + 1) / nt);
    f(0, n_sl / nt);
    for (auto& th : pool) th.join();
  };
  split(windows);
  if (!accept(w->sizes)) return false;
  // The slices with the largest windows take the longest (past the LDS budget
  // they gather from global memory): they go first in each of the eight
  // stretches of slices that the launch gives to an XCD, so that they run
  // beside the others and not after them (900^2 rows at D = 121, 5 columns,
  // 64 steps of the moment form: 28.6 -> 25.8 ms; 512^2: 10.6 -> 10.2 ms).
  {
    std::vector<int32_t> by(w->sizes);
    std::nth_element(by.begin(), by.begin() + n_sl / 2, by.end());
    const int64_t large = (int64_t)by[n_sl / 2] * 11 / 10;
    std::vector<int64_t> head, body, order;
    for (int64_t sl = 0; sl < n_sl; ++sl) (w->sizes[sl] > large ? head : body).push_back(sl);
    for (int64_t b = 0; b < 8; ++b) {
      for (size_t q = b; q < head.size(); q += 8) order.push_back(head[q]);
      const int64_t nb = (int64_t)body.size();
      for (int64_t q = nb * b / 8; q < nb * (b + 1) / 8; ++q) order.push_back(body[q]);
    }
    std::vector<int32_t> rows(w->rows.size());
    std::vector<std::vector<int32_t>> ws((size_t)n_sl);
    for (int64_t sl = 0; sl < n_sl; ++sl) {
      std::copy_n(w->rows.data() + order[sl] * nr, nr, rows.data() + sl * nr);
      ws[sl] = std::move(wins[order[sl]]);
      w->sizes[sl] = static_cast<int32_t>(ws[sl].size());
    }
    w->rows.swap(rows);
    wins.swap(ws);
  }
  w->loc.assign(n, 0);
  w->col.assign(n, 0);
  w->v64.assign(n, 0.0);
  w->v32.assign(n, 0.0f);
  split(entries);
  w->off.assign(n_sl + 1, 0);
  for (int64_t sl = 0; sl < n_sl; ++sl) w->off[sl + 1] = w->off[sl] + w->sizes[sl];
  w->idx.resize((size_t)w->off[n_sl]);
  for (int64_t sl = 0; sl < n_sl; ++sl)
    std::copy(wins[sl].begin(), wins[sl].end(), w->idx.begin() + w->off[sl]);
  return true;
}

}  // namespace csp
