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

// The closest pair found so far: ratio |x_i - x_k| / w_k, nodes i and k (-1: none below the bound);
// of equal ratios the one with the smallest i.
struct GapPair {
  double worst;
  int wi = -1, wk = -1;
  void offer(double d, int i, int k) {
    if (d < worst || (d == worst && wi >= 0 && i < wi)) {
      worst = d;
      wi = i;
      wk = k;
    }
  }
};

// All pairs (i, k), i from I and k from K, nodes of two bodies. Long lists go through a uniform grid
// of cells of size `reach` (no pair below the bound is further apart), short ones are compared
// directly.
void closest_of(const double *x, const double *y, const std::vector<double> &w,
                const std::vector<int> &I, const std::vector<int> &K, double reach, GapPair &g) {
  auto compare = [&](int i, int k) {
    const double dx = x[i] - x[k], dy = y[i] - y[k], b = g.worst * w[k];
    // (the exact ratio only where the squares do not rule the pair out)
    if (dx * dx + dy * dy <= b * b * (1.0 + 1e-9)) g.offer(std::hypot(dx, dy) / w[k], i, k);
  };
  if ((double)I.size() * (double)K.size() <= 1e5 || !(reach > 0.0)) {
    for (int i : I)
      for (int k : K) compare(i, k);
    return;
  }
  // cell indices >= 0, neighbours down to -1: hashed as unsigned (no shift of a negative value)
  auto key = [](long long ix, long long iy) {
    return ((unsigned long long)ix << 32) ^ ((unsigned long long)iy & 0xffffffffULL);
  };
  double x0 = x[I[0]], y0 = y[I[0]];
  for (const auto *v : {&I, &K})
    for (int k : *v) {
      x0 = std::min(x0, x[k]);
      y0 = std::min(y0, y[k]);
    }
  std::unordered_map<unsigned long long, std::vector<int>> grid;
  for (int k : K)
    grid[key((long long)std::floor((x[k] - x0) / reach), (long long)std::floor((y[k] - y0) / reach))]
        .push_back(k);
  for (int i : I) {
    const long long cx = (long long)std::floor((x[i] - x0) / reach);
    const long long cy = (long long)std::floor((y[i] - y0) / reach);
    for (long long dx = -1; dx <= 1; ++dx)
      for (long long dy = -1; dy <= 1; ++dy) {
        auto it = grid.find(key(cx + dx, cy + dy));
        if (it == grid.end()) continue;
        for (int k : it->second) compare(i, k);
      }
  }
}

// Smallest |x_i - x_k| / w_k over nodes i, k of different bodies, if below gap_factor (else
// gap_factor, with wi = wk = -1). A pair below it lies within gap_factor max w of k's body, so only
// bodies whose bounding boxes come that close are compared, and of those only the nodes inside
// each other's enlarged boxes: a grid over all nodes (cells of the largest spacing) tested every
// node against its own body's, 4 of 5 ms of a geometry's creation for the 40 dense particles
// between the two plates of the nanocomposite lattice.
double min_gap_ratio(const double *x, const double *y, const std::vector<double> &w,
                     const std::vector<int> &ptr, double gap_factor, int &wi, int &wk) {
  const int N = (int)ptr.size() - 1;
  struct Box {
    double x0, x1, y0, y1, reach;
    int body;
  };
  std::vector<Box> box(N);
  double width = 0.0;
  for (int b = 0; b < N; ++b) {
    Box q{x[ptr[b]], x[ptr[b]], y[ptr[b]], y[ptr[b]], 0.0, b};
    double wmax = 0.0;
    for (int k = ptr[b]; k < ptr[b + 1]; ++k) {
      q.x0 = std::min(q.x0, x[k]);
      q.x1 = std::max(q.x1, x[k]);
      q.y0 = std::min(q.y0, y[k]);
      q.y1 = std::max(q.y1, y[k]);
      wmax = std::max(wmax, w[k]);
    }
    q.reach = gap_factor * wmax;
    width = std::max(width, q.x1 - q.x0);
    box[b] = q;
  }
  std::sort(box.begin(), box.end(), [](const Box &a, const Box &b) { return a.x0 < b.x0; });
  GapPair g{gap_factor};
  std::vector<int> I, K;
  for (const Box &c : box) {  // k's body
    const double r = c.reach;
    auto from = std::lower_bound(box.begin(), box.end(), c.x0 - r - width,
                                 [](const Box &a, double v) { return a.x0 < v; });
    for (auto b = from; b != box.end() && b->x0 <= c.x1 + r; ++b) {  // i's body
      if (b->body == c.body || b->x1 < c.x0 - r || b->y0 > c.y1 + r || b->y1 < c.y0 - r) continue;
      auto inside = [&](int body, const Box &q, std::vector<int> &out) {
        out.clear();
        for (int k = ptr[body]; k < ptr[body + 1]; ++k)
          if (x[k] >= q.x0 - r && x[k] <= q.x1 + r && y[k] >= q.y0 - r && y[k] <= q.y1 + r)
            out.push_back(k);
      };
      inside(b->body, c, I);
      inside(c.body, *b, K);
      if (!I.empty() && !K.empty()) closest_of(x, y, w, I, K, r, g);
    }
  }
  wi = g.wi;
  wk = g.wk;
  return g.worst;
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
