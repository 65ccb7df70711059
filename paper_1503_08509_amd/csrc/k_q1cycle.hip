// The multigrid cycle below the first order-1 level of at most kQ1Max
// elements per axis, in one block per system (float64).
//
// Those levels hold at most 8000 nodes: their operator, transfer and coarse
// solve launches (17 per cycle from 16^3 down, 4 to 6 us each whatever the
// level holds) took 0.40 of the 1.9 ms of a replayed evaluation of 4096
// charges on 16^3 elements.  Here a level's iterate and its predecessor stay
// in LDS (its right side too, except a first level above 18^3, which reads it
// from global memory), and a step costs one barrier: 31 us per cycle from
// 16^3 against 76 us of launches, 12 against 38 from 8^3, 50 against 84 from
// 20^3.  Bound by each step's chain of LDS reads, update and barrier: each
// thread sums three values per plane (centre, sides, corners of the 3 x 3
// square) and reuses them along its run of nodes in z.  (The iterate and right
// side held in registers over a level's visit, a fifth fewer LDS reads: 31.4
// against 30.6 us from 16^3.)  21^3 would fit too (157 kB with its 7^3 level) but
// has not been timed in this form and keeps its launches; from 22^3 two iterates
// do not fit the LDS.
#include <algorithm>

#include "kernels.hpp"

namespace fep3m {

namespace {

constexpr int kThreads = 1024;

__device__ __forceinline__ int up(int i, int n) { return i + 1 == n ? 0 : i + 1; }
__device__ __forceinline__ int down(int i, int n) { return i == 0 ? n - 1 : i - 1; }

// A thread's share of a level: a run of nodes along z in one (x, y) column,
// with the offsets of the column's neighbours (worked out once per visit).
struct Own {
  int z0, z1;             // its nodes (none where z0 >= z1)
  int ix, iy;
  int at, xl, xr, yl, yr;  // its column's offset in a plane, and its row and column neighbours'
  __device__ __forceinline__ explicit Own(int n) {
    const int n2 = n * n, groups = min(n, kThreads / n2), run = (n + groups - 1) / groups;
    const int g = threadIdx.x / n2, c = threadIdx.x - g * n2;
    ix = c % n;
    iy = c / n;
    z0 = g < groups ? g * run : n;
    z1 = min(z0 + run, n);
    at = c;
    xl = down(ix, n) - ix;
    xr = up(ix, n) - ix;
    yl = (down(iy, n) - iy) * n;
    yr = (up(iy, n) - iy) * n;
  }
};

// fn(node, x, (K x)(node)) on the thread's nodes
template <class F>
__device__ __forceinline__ void q1_apply(const Q1Level &L, const Own &o, const double *x, F &&fn) {
  const int n = L.n, n2 = n * n;
  if (o.z0 < o.z1) {
    double a[3], b[3], c[3];   // sums of the planes below, at and above the node
    auto plane = [&](int z, double(&s)[3]) {
      const double *p = x + z * n2 + o.at;
      s[0] = p[0];
      s[1] = (p[o.xl] + p[o.xr]) + (p[o.yl] + p[o.yr]);
      s[2] = (p[o.yl + o.xl] + p[o.yl + o.xr]) + (p[o.yr + o.xl] + p[o.yr + o.xr]);
    };
    plane(down(o.z0, n), a);
    plane(o.z0, b);
#pragma unroll 4
    for (int z = o.z0; z < o.z1; ++z) {
      plane(up(z, n), c);
      const double y = L.st[0] * b[0] + L.st[1] * (b[1] + a[0] + c[0]) + L.st[2] * (b[2] + a[1] + c[1]) +
                       L.st[3] * (a[2] + c[2]);
      fn(z * n2 + o.at, b[0], y);
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        a[j] = b[j];
        b[j] = c[j];
      }
    }
  }
  __syncthreads();
}

// Residual r on n^3 nodes to the right side fc on (n / R)^3: coarse node c
// gathers the fine nodes within R of R c.
template <int R>
__device__ __forceinline__ void q1_restrict(int n, const double *r, double *fc) {
  const int nc = n / R, nc2 = nc * nc, n2 = n * n;
  for (int i = threadIdx.x; i < nc2 * nc; i += kThreads) {
    const int cz = i / nc2, cy = (i - cz * nc2) / nc, cx = i - cz * nc2 - cy * nc;
    int xo[2 * R - 1];
#pragma unroll
    for (int d = 1 - R; d < R; ++d) xo[d + R - 1] = R * cx + d < 0 ? R * cx + d + n : R * cx + d;
    double sz = 0.0;
#pragma unroll
    for (int dz = 1 - R; dz < R; ++dz) {
      const double *pz = r + (R * cz + dz < 0 ? R * cz + dz + n : R * cz + dz) * n2;
      double sy = 0.0;
#pragma unroll
      for (int dy = 1 - R; dy < R; ++dy) {
        const double *row = pz + (R * cy + dy < 0 ? R * cy + dy + n : R * cy + dy) * n;
        double sx = 0.0;
#pragma unroll
        for (int dx = 1 - R; dx < R; ++dx) sx += (R - abs(dx)) * (1.0 / R) * row[xo[dx + R - 1]];
        sy += (R - abs(dy)) * (1.0 / R) * sx;
      }
      sz += (R - abs(dz)) * (1.0 / R) * sy;
    }
    fc[i] = sz;
  }
}

// Exact solve on the last level by its one-dimensional eigenbasis (in LDS),
// as k_coarse_solve; a: right side and solution, b: scratch.
__device__ __forceinline__ void q1_coarse(int n, const double *V, const double *lam, double *a, double *b) {
  const int n2 = n * n, n3 = n2 * n;
  auto transform = [&](const double *in, double *out, int stride, bool to_modes, bool scale) {
    for (int i = threadIdx.x; i < n3; i += kThreads) {
      const int k = i / stride % n, base = i - k * stride;
      double s = 0.0;
      for (int c = 0; c < n; ++c) s += (to_modes ? V[c * n + k] : V[k * n + c]) * in[base + c * stride];
      if (scale) s = i == 0 ? 0.0 : s / (lam[i % n] + lam[i / n % n] + lam[i / n2]);
      out[i] = s;
    }
    __syncthreads();
  };
  transform(a, b, 1, true, false);
  transform(b, a, n, true, false);
  transform(a, b, n2, true, true);
  transform(b, a, n2, false, false);
  transform(a, b, n, false, false);
  transform(b, a, 1, false, false);
}

__global__ __launch_bounds__(kThreads) void k_q1_cycle(Q1Cycle q, const double *f, double *__restrict__ xout) {
  extern __shared__ double lds[];
  const int N0 = q.lv[0].n * q.lv[0].n * q.lv[0].n, tid = threadIdx.x;
  f += size_t(blockIdx.x) * N0;
  xout += size_t(blockIdx.x) * N0;
  double *X[kQ1Levels], *Xp[kQ1Levels], *Fl[kQ1Levels];
  double *V = lds, *lam = lds + q.nlast * q.nlast;
  for (int i = tid; i < q.nlast * (q.nlast + 1); i += kThreads) lds[i] = i < q.nlast * q.nlast ? q.V[i] : q.lam[i - q.nlast * q.nlast];
  {
    double *p = lds + q.nlast * (q.nlast + 1);
#pragma unroll
    for (int l = 0; l < kQ1Levels; ++l) {
      const int N = l < q.levels ? q.lv[l].n * q.lv[l].n * q.lv[l].n : 0;
      X[l] = p;
      Xp[l] = p + N;
      Fl[l] = p + 2 * N;
      p += l == 0 && !q.f_lds ? 2 * N : 3 * N;
    }
  }
  if (q.f_lds) {
    for (int i = tid; i < N0; i += kThreads) Fl[0][i] = f[i];
    f = Fl[0];
  }
  __syncthreads();
#pragma unroll
  for (int l = 0; l + 1 < kQ1Levels; ++l) {   // down
    if (l + 1 >= q.levels) continue;
    const Q1Level &L = q.lv[l];
    const double *F = l == 0 ? f : Fl[l];
    const int n = L.n, n2 = n * n;
    double *x = X[l], *xp = Xp[l];
    const Own o(n);
    const double first = L.c2[0] * L.invd;
    for (int z = o.z0; z < o.z1; ++z) {
      const int i = z * n2 + o.at;
      x[i] = first * F[i];
      xp[i] = 0.0;
    }
    __syncthreads();
    for (int s = 1; s < q.deg; ++s) {
      const double c1 = L.c1[s], c2 = L.c2[s] * L.invd;
      q1_apply(L, o, x, [&](int i, double xv, double y) { xp[i] = xv + c1 * (xv - xp[i]) + c2 * (F[i] - y); });
      double *t = x;
      x = xp;
      xp = t;
    }
    q1_apply(L, o, x, [&](int i, double, double y) { xp[i] = F[i] - y; });
    const int nc = q.lv[l + 1].n;
    if (2 * nc == n) q1_restrict<2>(n, xp, Fl[l + 1]);
    else q1_restrict<3>(n, xp, Fl[l + 1]);
    X[l] = x;
    Xp[l] = xp;
    __syncthreads();
  }
#pragma unroll
  for (int l = 1; l < kQ1Levels; ++l)
    if (l == q.levels - 1) {
      q1_coarse(q.lv[l].n, V, lam, Fl[l], X[l]);
      X[l] = Fl[l];   // where the last transform leaves the solution
    }
#pragma unroll
  for (int l = kQ1Levels - 2; l >= 0; --l) {   // up
    if (l + 1 >= q.levels) continue;
    const Q1Level &L = q.lv[l];
    const double *F = l == 0 ? f : Fl[l];
    const int n = L.n, n2 = n * n, nc = q.lv[l + 1].n, nc2 = nc * nc, r = n / nc;
    const double w1 = 1.0 / r;
    double *x = X[l], *xp = Xp[l];
    const Own o(n);
    {   // x += P ec, the column's interpolation in x and y once per coarse plane
      const double *ec = X[l + 1];
      const int x0 = o.ix / r, y0 = o.iy / r, x1 = up(x0, nc), y1 = up(y0, nc);
      const double u = (o.ix - x0 * r) * w1, v = (o.iy - y0 * r) * w1;
      const int o00 = y0 * nc + x0, o10 = y0 * nc + x1, o01 = y1 * nc + x0, o11 = y1 * nc + x1;
      auto at = [&](int zc) {
        const double *p = ec + zc * nc2;
        return (1.0 - v) * ((1.0 - u) * p[o00] + u * p[o10]) + v * ((1.0 - u) * p[o01] + u * p[o11]);
      };
      int zc = o.z0 / r, k = o.z0 - zc * r;
      for (int z = o.z0; z < o.z1; ++z) {
        const double w = k * w1;
        x[z * n2 + o.at] += (1.0 - w) * at(zc) + w * at(up(zc, nc));
        if (++k == r) {
          k = 0;
          ++zc;
        }
      }
    }
    __syncthreads();
    for (int s = 0; s < q.deg; ++s) {
      const double c1 = L.c1[s], c2 = L.c2[s] * L.invd;
      if (s == 0) q1_apply(L, o, x, [&](int i, double xv, double y) { xp[i] = xv + c2 * (F[i] - y); });
      else q1_apply(L, o, x, [&](int i, double xv, double y) { xp[i] = xv + c1 * (xv - xp[i]) + c2 * (F[i] - y); });
      double *t = x;
      x = xp;
      xp = t;
    }
    X[l] = x;
  }
  for (int i = tid; i < N0; i += kThreads) xout[i] = X[0][i];
}

}  // namespace

size_t q1_cycle_lds(const Q1Cycle &q) {
  size_t d = size_t(q.nlast) * (q.nlast + 1);
  for (int l = 0; l < q.levels; ++l) d += size_t(l == 0 && !q.f_lds ? 2 : 3) * q.lv[l].n * q.lv[l].n * q.lv[l].n;
  return d * sizeof(double);
}

Q1Level q1_level(const LevelOp &op) {
  Q1Level L{};
  L.n = op.n;
  const double kd = op.ke[0] + op.ke[3], ko = op.ke[1], md = op.me[0] + op.me[3], mo = op.me[1];
  L.st[0] = 3.0 * kd * md * md;                     // the node, its 6 sides, 12 edges, 8 corners
  L.st[1] = ko * md * md + 2.0 * kd * mo * md;
  L.st[2] = 2.0 * ko * mo * md + kd * mo * mo;
  L.st[3] = 3.0 * ko * mo * mo;
  L.invd = 1.0 / L.st[0];
  return L;
}

void launch_q1_cycle(hipStream_t s, int nsys, const Q1Cycle &q, const double *f, double *x) {
  hipLaunchKernelGGL(k_q1_cycle, dim3(nsys), dim3(kThreads), q1_cycle_lds(q), s, q, f, x);
}

}  // namespace fep3m
