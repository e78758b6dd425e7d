// Host-side checks of curve samples before a geometry is built: finite samples, positive
// orientation, read-off points inside their bodies, and the resolution warning (curves
// resolved by their nodes; no node closer than a few node spacings to another body).
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <string>
#include <unordered_map>
#include <vector>

#include "internal.h"

namespace bie {
namespace {

// Winding number of the closed polygon (x[k], y[k]), k = 0..n-1, around (px, py); 0 outside.
int winding(const double *x, const double *y, int n, double px, double py) {
  int wn = 0;
  for (int k = 0; k < n; ++k) {
    const int k1 = k + 1 == n ? 0 : k + 1;
    const double ax = x[k] - px, ay = y[k] - py, bx = x[k1] - px, by = y[k1] - py;
    const double cr = ax * by - ay * bx;  // > 0: p left of the edge
    if (ay <= 0.0) {
      if (by > 0.0 && cr > 0.0) ++wn;
    } else if (by <= 0.0 && cr < 0.0) {
      --wn;
    }
  }
  return wn;
}

// Bodies by cell of a coarse grid over all nodes: those whose bounding box, enlarged by the body's
// `reach`, meets the cell. About two cells per body, fewer where those would list more than four
// bodies per node (boxes that cover one another).
struct BodyGrid {
  struct Box {
    double x0, x1, y0, y1, reach;
    bool holds(double x, double y, double by) const {
      return x >= x0 - by && x <= x1 + by && y >= y0 - by && y <= y1 + by;
    }
  };
  std::vector<Box> box;
  double wmax = 0.0, x0, y0, cell;
  int nx, ny;
  std::vector<int> start, list;  // bodies of cell c: list[start[c]] .. list[start[c + 1] - 1]
  static constexpr int kFew = 8;  // in cells of more bodies, their boxes are not looked at one by one

  int column(double x) const { return (int)std::max(0.0, std::min(nx - 1.0, (x - x0) / cell)); }
  int row(double y) const { return (int)std::max(0.0, std::min(ny - 1.0, (y - y0) / cell)); }

  // No other body's enlarged box meets that of b's nodes.
  bool alone(int b) const {
    const Box &q = box[b];
    for (int r = row(q.y0); r <= row(q.y1); ++r)
      for (int c = column(q.x0); c <= column(q.x1); ++c) {
        const int e0 = start[(size_t)r * nx + c], e1 = start[(size_t)r * nx + c + 1];
        if (e1 - e0 > kFew) return false;
        for (int e = e0; e < e1; ++e) {
          const Box &o = box[list[e]];
          if (list[e] != b && q.x0 <= o.x1 + o.reach && q.x1 >= o.x0 - o.reach &&
              q.y0 <= o.y1 + o.reach && q.y1 >= o.y0 - o.reach)
            return false;
        }
      }
    return true;
  }

  BodyGrid(const double *x, const double *y, const std::vector<double> &w,
           const std::vector<int> &ptr, double gap_factor) {
    const int N = (int)ptr.size() - 1, M = ptr[N];
    double x1 = x[0], y1 = y[0];
    x0 = x[0];
    y0 = y[0];
    for (int b = 0; b < N; ++b) {
      Box q{x[ptr[b]], x[ptr[b]], y[ptr[b]], y[ptr[b]], 0.0};
      double wb = 0.0;
      for (int k = ptr[b]; k < ptr[b + 1]; ++k) {
        q.x0 = std::min(q.x0, x[k]);
        q.x1 = std::max(q.x1, x[k]);
        q.y0 = std::min(q.y0, y[k]);
        q.y1 = std::max(q.y1, y[k]);
        wb = std::max(wb, w[k]);
      }
      q.reach = gap_factor * wb * (1.0 + 1e-9);
      wmax = std::max(wmax, wb);
      box.push_back(q);
      x0 = std::min(x0, q.x0);
      x1 = std::max(x1, q.x1);
      y0 = std::min(y0, q.y0);
      y1 = std::max(y1, q.y1);
    }
    const double W = x1 - x0, H = y1 - y0;
    cell = std::max(std::sqrt(W / (2.0 * N)) * std::sqrt(H), std::max(W, H) / (4.0 * N));
    for (;; cell *= 2.0) {
      nx = cell > 0.0 ? 1 + (int)std::min(4.0 * N, W / cell) : 1;
      ny = cell > 0.0 ? 1 + (int)std::min(4.0 * N, H / cell) : 1;
      if (!(cell > 0.0)) cell = 1.0;
      start.assign((size_t)nx * ny + 1, 0);
      long long total = 0;
      for (const Box &q : box)
        total += (long long)(column(q.x1 + q.reach) - column(q.x0 - q.reach) + 1) *
                 (row(q.y1 + q.reach) - row(q.y0 - q.reach) + 1);
      if (total <= 4LL * M || nx * ny == 1) break;
    }
    for (int pass = 0; pass < 2; ++pass) {
      for (int b = 0; b < N; ++b) {
        const Box &q = box[b];
        const int c1 = column(q.x1 + q.reach), r1 = row(q.y1 + q.reach);
        for (int r = row(q.y0 - q.reach); r <= r1; ++r)
          for (int c = column(q.x0 - q.reach); c <= c1; ++c) {
            int &at = start[(size_t)r * nx + c + (pass == 0)];
            if (pass) list[at] = b;
            ++at;
          }
      }
      if (pass == 0) {
        for (size_t c = 1; c < start.size(); ++c) start[c] += start[c - 1];
        list.resize(start.back());
      } else {  // each start now stands at its cell's end
        for (size_t c = start.size() - 1; c > 0; --c) start[c] = start[c - 1];
        start[0] = 0;
      }
    }
  }
};

// Smallest |x_i - x_k| / w_k over nodes i, k of different bodies, if below gap_factor (else
// gap_factor, with wi = wk = -1): uniform grid of cells of size gap_factor * max w, only the 3 x 3
// cells around a node can hold such a pair. Only nodes that can be part of one go through it: i has to
// lie within gap_factor max w of k's body's box, and k as close to the box of such i. With all
// nodes in the grid, every node met its own body's: 4 of 5 ms of a geometry's creation for the 40
// dense particles between the two plates of the nanocomposite lattice. Bodies are looked up by
// cell: a body whose box holds the others (a wall, a container) is listed once per cell, where
// comparing boxes in order of x made each body meet all those left of it (20,000 discs in a ring of
// 20,000 nodes: 1,190 ms, here 11; with all nodes in the grid 63).
double min_gap_ratio(const double *x, const double *y, const std::vector<double> &w,
                     const std::vector<int> &ptr, double gap_factor, int &wi, int &wk) {
  const int N = (int)ptr.size() - 1, M = ptr[N];
  wi = wk = -1;
  const BodyGrid bodies(x, y, w, ptr, gap_factor);
  const double x0 = bodies.x0, y0 = bodies.y0;
  const double cell = gap_factor * bodies.wmax;
  if (!(cell > 0.0)) return gap_factor;
  // nodes i near another body, and per body the box of the nodes near it
  std::vector<int> body_of, I;
  std::vector<BodyGrid::Box> hit(N, {1.0, -1.0, 0.0, 0.0, 0.0});
  auto strike = [&](int c, int i) {
    BodyGrid::Box &h = hit[c];
    if (h.x0 > h.x1) h = {x[i], x[i], y[i], y[i], 0.0};
    h.x0 = std::min(h.x0, x[i]);
    h.x1 = std::max(h.x1, x[i]);
    h.y0 = std::min(h.y0, y[i]);
    h.y1 = std::max(h.y1, y[i]);
  };
  std::vector<BodyGrid::Box> crowd(bodies.start.size() - 1, {1.0, -1.0, 0.0, 0.0, 0.0});
  body_of.resize(M);
  for (int b = 0; b < N; ++b) {
    std::fill(body_of.begin() + ptr[b], body_of.begin() + ptr[b + 1], b);
    if (bodies.alone(b)) continue;
    for (int i = ptr[b]; i < ptr[b + 1]; ++i) {
      const int c = bodies.row(y[i]) * bodies.nx + bodies.column(x[i]);
      const int e0 = bodies.start[c], e1 = bodies.start[c + 1];
      if (e1 - e0 > BodyGrid::kFew) {
        BodyGrid::Box &h = crowd[c];
        if (h.x0 > h.x1) h = {x[i], x[i], y[i], y[i], 0.0};
        h.x0 = std::min(h.x0, x[i]);
        h.x1 = std::max(h.x1, x[i]);
        h.y0 = std::min(h.y0, y[i]);
        h.y1 = std::max(h.y1, y[i]);
        I.push_back(i);
        continue;
      }
      bool near = false;
      for (int e = e0; e < e1; ++e) {
        const int q = bodies.list[e];
        if (q == b || !bodies.box[q].holds(x[i], y[i], bodies.box[q].reach)) continue;
        near = true;
        strike(q, i);
      }
      if (near) I.push_back(i);
    }
  }
  for (size_t c = 0; c + 1 < bodies.start.size(); ++c) {
    const BodyGrid::Box &h = crowd[c];
    if (h.x0 > h.x1) continue;
    for (int e = bodies.start[c]; e < bodies.start[c + 1]; ++e) {
      BodyGrid::Box &q = hit[bodies.list[e]];
      if (q.x0 > q.x1) q = h;
      q.x0 = std::min(q.x0, h.x0);
      q.x1 = std::max(q.x1, h.x1);
      q.y0 = std::min(q.y0, h.y0);
      q.y1 = std::max(q.y1, h.y1);
    }
  }
  // cell indices >= 0, neighbours down to -1: hashed as unsigned (no shift of a negative value)
  auto key = [](long long ix, long long iy) {
    return ((unsigned long long)ix << 32) ^ ((unsigned long long)iy & 0xffffffffULL);
  };
  auto at = [&](double v, double v0) { return (long long)std::floor((v - v0) / cell); };
  std::unordered_map<unsigned long long, std::vector<int>> grid;
  for (int c = 0; c < N; ++c) {
    if (hit[c].x0 > hit[c].x1) continue;
    for (int k = ptr[c]; k < ptr[c + 1]; ++k)
      if (hit[c].holds(x[k], y[k], bodies.box[c].reach))
        grid[key(at(x[k], x0), at(y[k], y0))].push_back(k);
  }
  if (grid.empty()) return gap_factor;
  double worst = gap_factor;
  for (int i : I) {
    const long long cx = at(x[i], x0), cy = at(y[i], y0);
    for (long long dx = -1; dx <= 1; ++dx)
      for (long long dy = -1; dy <= 1; ++dy) {
        auto it = grid.find(key(cx + dx, cy + dy));
        if (it == grid.end()) continue;
        for (int k : it->second) {
          if (body_of[k] == body_of[i]) continue;
          const double px = x[i] - x[k], py = y[i] - y[k], b = worst * w[k], bb = b * b;
          // (the exact ratio only where the squares, in range, do not rule the pair out)
          if (bb > 1e-280 && bb < 1e300 && px * px + py * py > bb * (1.0 + 1e-9)) continue;
          const double d = std::hypot(px, py) / w[k];
          if (d < worst) {
            worst = d;
            wi = i;
            wk = k;
          }
        }
      }
  }
  return worst;
}

}  // namespace

int check_curves(int N, const int32_t *npb, const double *curve, const double *interior,
                 std::string &msg) {
  long long M = 0;
  for (int b = 0; b < N; ++b) M += npb[b];
  const double *X = curve, *Y = curve + M, *DX = curve + 2 * M, *DY = curve + 3 * M,
               *DDX = curve + 4 * M, *DDY = curve + 5 * M;
  std::vector<double> w(M);
  std::vector<int> ptr(N + 1, 0);
  for (int b = 0; b < N; ++b) ptr[b + 1] = ptr[b] + npb[b];
  int resolve = BIE_OK;
  std::string resolve_msg;
  for (int b = 0, k0 = 0; b < N; k0 += npb[b], ++b) {
    const int n = npb[b];
    const double h = 2.0 * kPi / n;
    double area = 0.0, len = 0.0, cx = 0.0, cy = 0.0, turn = 0.0;
    for (int k = k0; k < k0 + n; ++k) {
      for (int a = 0; a < 6; ++a)
        if (!std::isfinite(curve[a * M + k])) {
          msg = "non-finite curve samples on body " + std::to_string(b);
          return BIE_EINVAL;
        }
      double sp = std::sqrt(DX[k] * DX[k] + DY[k] * DY[k]);
      if (!(sp > 1e-140 && sp < 1e140)) sp = std::hypot(DX[k], DY[k]);  // squares out of range
      w[k] = h * sp;
      area += 0.5 * h * (X[k] * DY[k] - Y[k] * DX[k]);
      len += w[k];
      cx += w[k] * X[k];
      cy += w[k] * Y[k];
      // curvature times arc length: (x' y'' - y' x'') / |x'|^2 dt
      if (sp > 0.0) turn += h * (DX[k] * DDY[k] - DY[k] * DDX[k]) / (sp * sp);
    }
    if (!(area > 0.0)) {
      msg = "body " + std::to_string(b) + " is not positively oriented (signed area <= 0)";
      return BIE_EINVAL;
    }
    // the read-off point: the caller's, else the arc-length centroid
    const double px = interior ? interior[2 * b] : cx / len;
    const double py = interior ? interior[2 * b + 1] : cy / len;
    if (!std::isfinite(px) || !std::isfinite(py) || winding(X + k0, Y + k0, n, px, py) != 1) {
      msg = "read-off point (" + std::to_string(px) + ", " + std::to_string(py) + ") of body " +
            std::to_string(b) +
            " is not inside its curve (the default is the arc-length centroid; pass interior "
            "points for bodies whose centroid lies outside)";
      return BIE_EINVAL;
    }
    // the trapezoidal sum of the curvature against arc length is the turning number 2 pi of a
    // simple closed curve, up to the aliasing error of the samples
    const double err = std::fabs(turn - 2.0 * kPi) / (2.0 * kPi);
    if (resolve == BIE_OK && !(err <= kResolveTurn)) {
      resolve = BIE_ERESOLVE;
      resolve_msg = "body " + std::to_string(b) +
                    " is under-resolved: its trapezoidal turning number misses 2 pi by " +
                    std::to_string(err) + " (relative); use more nodes";
    }
  }
  if (resolve == BIE_OK && N > 1) {
    int wi, wk;
    const double r = min_gap_ratio(X, Y, w, ptr, kResolveGap, wi, wk);
    if (wi >= 0) {
      auto body_of = [&](int k) {
        return (int)(std::upper_bound(ptr.begin(), ptr.end(), k) - ptr.begin()) - 1;
      };
      resolve = BIE_ERESOLVE;
      resolve_msg = "bodies " + std::to_string(body_of(wi)) + " and " +
                    std::to_string(body_of(wk)) + " are closer than " +
                    std::to_string(kResolveGap) + " node spacings (" + std::to_string(r) +
                    " spacings of body " + std::to_string(body_of(wk)) +
                    "); use more nodes on the closer bodies";
    }
  }
  msg = resolve_msg;
  return resolve;
}

}  // namespace bie
