// What an epoch prepares from its radius alone: as a launch of its own at its head (smooth.hip), or by workgroups of
// the launch that adds up the nodes' instances (segsum.hip).
#pragma once
#include "som_internal.hpp"

#include <math.h>

namespace som {

// twice the embedded column distance between destination column xi (row parity pi) and source
// column xb (row parity pb)
__device__ __forceinline__ int col_offset2(int xi, int xb, int pi, int pb, int hex, int toroid, int cols) {
  int m = 2 * (xi - xb) + (hex ? pi - pb : 0);
  m = m < 0 ? -m : m;
  if (toroid && 2 * cols - m < m) m = 2 * cols - m;
  return m;
}

__device__ __forceinline__ int row_offset(int yi, int yb, int toroid, int rows) {
  int a = yi > yb ? yi - yb : yb - yi;
  if (toroid && rows - a < a) a = rows - a;
  return a;
}

// The cooled radius, the two Gaussian factor tables, the coefficient matrices of
// the smoothing passes (or the weight table of a neighbourhood with compact support; smooth.hip has their layouts), and
// the counters that the search of this epoch starts from.
struct EpochTables {
  EpochParams *params;
  float *gx, *gy;             // [2 cols + 1], [rows]
  float *GxT, *GyT;           // or null
  int xi_pad, e_pad;
  float *H2;                  // or null
  int rows, cols, hex, toroid, function, compact;
  unsigned *zero;             // words to clear, or null
  int zero_words;
};

constexpr int kSmoothTile = 16;

__device__ __forceinline__ int direct_table_width(int cols, int toroid) {
  return (toroid ? cols : 2 * cols - 1) + kSmoothTile;
}

// Where the epoch is in its schedule.
struct EpochSchedule {
  int epoch, n_epochs;
  double r0, rN, s0, sN;
  int cooling, scale_cooling;
};

// Thread `at` of `stride`.
__device__ __forceinline__ void write_epoch_tables(const EpochTables &t, const EpochSchedule &q, int64_t at, int64_t stride) {
  const double radius = cooled(q.r0, q.rN, q.n_epochs, q.epoch, q.cooling);
  const double inv = 1.0 / (8.0 * radius * radius);
  const double ya = t.hex ? 3.0 : 4.0;
  if (at == 0) {
    t.params->radius = radius;
    t.params->scale = cooled(q.s0, q.sN, q.n_epochs, q.epoch, q.scale_cooling);
    t.params->inv8r2 = inv;
  }
  auto gx = [&](int m) { return (float)exp(-(double)m * (double)m * inv); };
  auto gy = [&](int a) { return (float)exp(-ya * (double)a * (double)a * inv); };
  const int rows = t.rows, cols = t.cols, par = t.hex ? 2 : 1;
  const int64_t n_gx = 2 * (int64_t)cols + 1, n_f = n_gx + rows;
  const int64_t n_GxT = t.GxT ? (int64_t)par * par * cols * t.xi_pad : 0, n_GyT = t.GyT ? (int64_t)par * rows * t.e_pad : 0;
  const int width = direct_table_width(cols, t.toroid);
  const int64_t n_H2 = t.H2 ? (int64_t)(t.hex ? 3 : 1) * rows * width : 0;
  for (int64_t o = at; o < t.zero_words; o += stride) t.zero[o] = 0u;
  for (int64_t o = at; o < n_f; o += stride) {
    if (o < n_gx) t.gx[o] = gx((int)o);
    else t.gy[o - n_gx] = gy((int)(o - n_gx));
  }
  for (int64_t o = at; o < n_GxT + n_GyT; o += stride) {
    if (o < n_GxT) {
      const int xi = (int)(o % t.xi_pad);
      const int xb = (int)((o / t.xi_pad) % cols);
      const int ps = (int)((o / ((int64_t)t.xi_pad * cols)) % par);
      const int img = (int)(o / ((int64_t)t.xi_pad * cols * par));
      t.GxT[o] = xi < cols ? gx(col_offset2(xi, xb, img, ps, t.hex, t.toroid, cols)) : 0.f;
    } else {
      const int64_t p = o - n_GxT;
      const int e = (int)(p % t.e_pad);
      const int yb = (int)((p / t.e_pad) % rows);
      const int cls = (int)(p / ((int64_t)t.e_pad * rows));
      const int yi = par * e + cls;
      t.GyT[p] = yi < rows ? gy(row_offset(yi, yb, t.toroid, rows)) : 0.f;
    }
  }
  const double reach = 4.0 * radius * radius;     // 4 d^2 <= 4 r^2: inside the radius
  for (int64_t o = at; o < n_H2; o += stride) {
    const int c = (int)(o % width);
    const int a_raw = (int)((o / width) % rows);
    const int cls = (int)(o / ((int64_t)width * rows));
    const int dpar = t.hex ? cls - 1 : 0;
    const int dx = t.toroid ? c % cols : c - (cols - 1);
    long long m = 2ll * dx + dpar;
    m = m < 0 ? -m : m;
    long long a = a_raw;
    if (t.toroid) {
      if (2ll * cols - m < m) m = 2ll * cols - m;
      if (rows - a < a) a = rows - a;
    }
    const double d2 = (double)(m * m + (t.hex ? 3 : 4) * a * a);
    const bool inside = d2 <= reach;
    float h;
    if (t.function == SOM_NEIGHBORHOOD_BUBBLE) h = inside ? 1.f : 0.f;
    else h = (t.compact && !inside) ? 0.f : (float)exp(-d2 * inv);
    t.H2[o] = h;
  }
}

// search: a filter pass follows whose counters are cleared on the way.  work: items of the longest loop.
EpochTables epoch_tables(const som_ctx *c, bool search, int64_t *work);
EpochSchedule epoch_schedule(const som_ctx *c, int epoch, int n_epochs, double r0, double rN, double s0, double sN, int cooling);

}  // namespace som
