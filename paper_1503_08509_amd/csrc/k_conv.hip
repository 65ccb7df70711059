// Near-screen field and its transpose by the convolution theorem on lattices
// of any factorable edge, for every screen family and for the boxes
// (k_fft.hip: the one-element q = 3 screen on power-of-two lattices).
//
//   Psi_E[m] = sum_D sum_a T[a][D][m] C[E - D][a]
//   B_E[a]   = sum_D sum_m T[a][D][m] g[E + D][m]
//
// As in k_fft.hip two real channels share a complex one, the tables'
// spectrum S[k][a][m] = sum_D T[a][D][m] exp(-2 pi i k.D / N) is kept for one
// octant of frequencies (the tables are symmetric under axis reflections) and
// one block handles the up to 8 frequencies of an orbit.  A periodic mesh of
// n elements is its own lattice (N = n); a box is padded with zeros to
// N >= n + n_sr, so that no offset wraps onto a charge, and the passes skip
// the rows that are zero or not wanted.
//
// What bounds it: memory (the spectrum once per evaluation and configuration
// and the node fields twice per pass), and below about 24^3 elements the 13
// launches.  The table sums this replaces for the default near_field option
// take 2 na M 343 operations per element (na moments, M nodes) and gave each
// brick of 4 x 4 x 8 elements to one block, so small meshes left most compute
// units idle: near field and moment adjoint together 2.9 ms at n = 27
// (q = 3), 2.8 ms in a grounded box of 32^3, 4.9 ms for the 27-element q = 2
// screen at n = 24; here 0.29, 0.42 and 0.22 ms.
#include "kernels.hpp"
#include "table_symmetry.hpp"

namespace fep3m {

namespace {

// cos and sin of 2 pi k / R at compile time
constexpr double taylor(double t, bool cosine) {
  double s = cosine ? 1.0 : t, term = s;
  for (int i = cosine ? 1 : 2; i < 24; i += 2) {
    term *= -t * t / (double(i) * double(i + 1));
    s += term;
  }
  return s;
}
constexpr double kPi = 3.14159265358979323846;
constexpr double turn(int k, int R, bool cosine) {
  k %= R;
  double x = 2.0 * double(k) / double(R), sc = 1.0, ss = 1.0;   // angle / pi in [0, 2)
  if (x > 1.0) { x = 2.0 * double(R - k) / double(R); ss = -1.0; }
  if (x > 0.5) { x = double(2 * (x == 2.0 * double(k) / double(R) ? R - 2 * k : 2 * k - R)) / double(2 * R); sc = -1.0; }
  const double c = x <= 0.25 ? taylor(kPi * x, true) : taylor(kPi * (0.5 - x), false);
  const double s = x <= 0.25 ? taylor(kPi * x, false) : taylor(kPi * (0.5 - x), true);
  return cosine ? sc * c : ss * s;
}
template <int R>
struct Turns {
  double c[R], s[R];
  constexpr Turns() : c(), s() {
    for (int k = 0; k < R; ++k) {
      c[k] = turn(k, R, true);
      s[k] = turn(k, R, false);
    }
  }
};

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

constexpr int split_of(int R) { return R == 4 ? 2 : R == 6 ? 2 : R == 8 ? 2 : R == 9 ? 3 : R == 10 ? 2 : 0; }

// In-register DFT, exp(-2 pi i j k / R), natural order in and out.
template <int R>
__device__ __forceinline__ void dft(double2 (&v)[R]) {
  constexpr Turns<R> w{};
  constexpr int A = split_of(R);
  if constexpr (R == 1) {
  } else if constexpr (R == 2) {
    const double2 a = v[0];
    v[0] = cadd(a, v[1]);
    v[1] = csub(a, v[1]);
  } else if constexpr (A != 0) {   // R = A B: A-point DFTs over stride B, twiddles, B-point DFTs
    constexpr int B = R / A;
    double2 u[A][B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
      double2 t[A];
#pragma unroll
      for (int a = 0; a < A; ++a) t[a] = v[a * B + b];
      dft<A>(t);
#pragma unroll
      for (int a = 0; a < A; ++a)
        u[a][b] = a * b == 0 ? t[a] : cmul(t[a], make_double2(w.c[a * b % R], -w.s[a * b % R]));
    }
#pragma unroll
    for (int a = 0; a < A; ++a) {
      dft<B>(u[a]);
#pragma unroll
      for (int b = 0; b < B; ++b) v[a + A * b] = u[a][b];
    }
  } else {   // odd prime: sums and differences of the pairs (j, R - j)
    constexpr int H = (R - 1) / 2;
    double2 s[H], d[H], x0 = v[0], dc = v[0];
#pragma unroll
    for (int j = 0; j < H; ++j) {
      s[j] = cadd(v[j + 1], v[R - 1 - j]);
      d[j] = csub(v[j + 1], v[R - 1 - j]);
      dc = cadd(dc, s[j]);
    }
    v[0] = dc;
#pragma unroll
    for (int k = 1; k <= H; ++k) {
      double2 e = x0, o = make_double2(0.0, 0.0);
#pragma unroll
      for (int j = 0; j < H; ++j) {
        const double c = w.c[(j + 1) * k % R], q = w.s[(j + 1) * k % R];
        e.x += c * s[j].x;
        e.y += c * s[j].y;
        o.x += q * d[j].x;
        o.y += q * d[j].y;
      }
      v[k] = make_double2(e.x + o.y, e.y - o.x);       // e - i o
      v[R - k] = make_double2(e.x - o.y, e.y + o.x);
    }
  }
}

constexpr int kCols = 32;   // columns (one channel of one line) per block

// One axis of a transform over [cfg][z][y][x][channel] complex arrays of edge N.
struct ConvPass {
  int N, r1, r2;        // N = r1 r2
  int CH;               // complex channels
  int axis;             // 0 x, 1 y, 2 z
  int nin, nout;        // entries along the axis that are not zero / that are wanted
  int e1, e2;           // extents of the other two axes (the faster one first)
  int n, nch;           // real arrays: elements per axis, channels
  int nb;
  bool inverse;
  const double2 *tw;    // exp(-2 pi i j / N)
  const double2 *in;
  const double *rin;
  double2 *out;
  double *rout;
  const double *phi;    // W: mesh potential (null: none), order p, nodes per axis, periodic
  int p, P;
  bool wrap;
  double sign;          // real output: its factor
};

enum ConvIn : int { kInComplex = 0, kInReal = 1 };
enum ConvOut : int { kOutComplex = 0, kOutW = 1, kOutReal = 2 };

template <int IN>
__device__ __forceinline__ double2 conv_load(const ConvPass &a, size_t base, size_t step, size_t ebase, int ch, int j) {
  if (j >= a.nin) return make_double2(0.0, 0.0);
  double2 v;
  if constexpr (IN == kInReal) {
    const double *q = a.rin + (ebase + j) * a.nch + 2 * ch;
    v = make_double2(q[0], 2 * ch + 1 < a.nch ? q[1] : 0.0);
  } else {
    v = a.in[base + step * j];
  }
  return a.inverse ? make_double2(v.y, v.x) : v;   // the inverse is the forward DFT between swapped parts
}

template <int R, int IN>
__device__ __forceinline__ void conv_step1(const ConvPass &a, double2 *L, const double2 *tw, size_t base, size_t step,
                                           size_t ebase, int ch, int col, int j2) {
  double2 v[R];
#pragma unroll
  for (int j = 0; j < R; ++j) v[j] = conv_load<IN>(a, base, step, ebase, ch, j * a.r2 + j2);
  dft<R>(v);
#pragma unroll
  for (int k = 0; k < R; ++k) L[(k * a.r2 + j2) * kCols + col] = k == 0 ? v[0] : cmul(v[k], tw[j2 * k]);
}

template <int R, int OUT>
__device__ __forceinline__ void conv_step2(const ConvPass &a, const double2 *L, size_t base, size_t step, size_t ebase,
                                           int cfg, int i1, int i2, int ch, int col, int k1) {
  double2 v[R];
#pragma unroll
  for (int j = 0; j < R; ++j) v[j] = L[(k1 * R + j) * kCols + col];
  dft<R>(v);
#pragma unroll
  for (int k2 = 0; k2 < R; ++k2) {
    const int k = k1 + a.r1 * k2;
    if (k >= a.nout) continue;
    const double2 z = a.inverse ? make_double2(v[k2].y, v[k2].x) : v[k2];
    if constexpr (OUT == kOutComplex) {
      a.out[base + step * k] = z;
    } else {   // x axis: the element's real channels
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int m = 2 * ch + h;
        if (m >= a.nch) continue;
        double r = a.sign * (h ? z.y : z.x);
        if (OUT == kOutW && a.phi) {
          const int q1 = a.p + 1, mx = m % q1, my = (m / q1) % q1, mz = m / (q1 * q1);
          int gx = a.p * k + mx, gy = a.p * i1 + my, gz = a.p * i2 + mz;
          if (a.wrap) {
            gx -= gx >= a.P ? a.P : 0;
            gy -= gy >= a.P ? a.P : 0;
            gz -= gz >= a.P ? a.P : 0;
          }
          r += a.phi[((size_t(cfg) * a.P + gz) * a.P + gy) * a.P + gx];
        }
        a.rout[(ebase + k) * a.nch + m] = r;
      }
    }
  }
}

#define FEP3M_RADIX_SWITCH(r, CALL) \
  switch (r) {                      \
    case 1: CALL(1); break;         \
    case 2: CALL(2); break;         \
    case 3: CALL(3); break;         \
    case 4: CALL(4); break;         \
    case 5: CALL(5); break;         \
    case 6: CALL(6); break;         \
    case 7: CALL(7); break;         \
    case 8: CALL(8); break;         \
    case 9: CALL(9); break;         \
    case 10: CALL(10); break;       \
    case 11: CALL(11); break;       \
    default: CALL(13); break;       \
  }

// Two radix steps per pass (N = r1 r2, each at most 13): the columns of a
// block are consecutive in memory along the channels and, for the y and z
// passes, along x; one LDS round trip between the steps.
template <int IN, int OUT>
__global__ __launch_bounds__(256) void k_conv_pass(ConvPass a) {
  __shared__ double2 L[kConvMaxN * kCols];
  __shared__ double2 tw[kConvMaxN];
  const int tid = threadIdx.x;
  for (int i = tid; i < a.N; i += 256) tw[i] = a.tw[i];
  const size_t N = a.N, total = size_t(a.nb) * a.e1 * a.e2 * a.CH;
  const int col = tid % kCols;
  const size_t c = size_t(blockIdx.x) * kCols + col;
  const bool on = c < total;
  const size_t l = (on ? c : 0) / a.CH;
  const int ch = int((on ? c : 0) - l * a.CH);
  const int i1 = int(l % a.e1), i2 = int(l / a.e1 % a.e2), cfg = int(l / a.e1 / a.e2);
  const size_t s1 = a.axis == 0 ? N : 1, s2 = a.axis == 2 ? N : N * N;
  const size_t step = (a.axis == 0 ? 1 : a.axis == 1 ? N : N * N) * a.CH;
  const size_t base = (size_t(cfg) * N * N * N + i1 * s1 + i2 * s2) * a.CH + ch;
  const size_t ebase = ((size_t(cfg) * a.n + i2) * a.n + i1) * a.n;   // real arrays (x axis: i1 = y, i2 = z)
  __syncthreads();
  if (on)
    for (int j2 = tid / kCols; j2 < a.r2; j2 += 256 / kCols) {
#define CALL(R) conv_step1<R, IN>(a, L, tw, base, step, ebase, ch, col, j2)
      FEP3M_RADIX_SWITCH(a.r1, CALL)
#undef CALL
    }
  __syncthreads();
  if (on)
    for (int k1 = tid / kCols; k1 < a.r1; k1 += 256 / kCols) {
#define CALL(R) conv_step2<R, OUT>(a, L, base, step, ebase, cfg, i1, i2, ch, col, k1)
      FEP3M_RADIX_SWITCH(a.r2, CALL)
#undef CALL
    }
}

// The spectrum is kept for one octant and takes the rest by reflection, so the
// tables behind it must be symmetric to the last bit: what they miss (1e-14 of
// their largest value) would pass between the two channels of a complex one,
// from node to node with changing sign, where the forces' derivative picks it
// up (an error of 1.4e-13 instead of 1.8e-14: one-element q = 2, 9^3).
__global__ __launch_bounds__(256) void k_conv_symmetrise(size_t count, int p, int nl, int nsr, double *T) {
  const size_t i = size_t(blockIdx.x) * 256 + threadIdx.x;
  if (i < count) symmetrise_entry(i, p, nl, nsr, T);
}

// Spectrum at 8 octant frequencies per block and one moment (blockIdx.y).
__global__ __launch_bounds__(256) void k_conv_spec(int N, int NO, int nsr, int na, int M, const double *__restrict__ T,
                                                   const double2 *__restrict__ tw, double2 *__restrict__ S) {
  constexpr int FB = 8;
  __shared__ double2 ph[FB][343];
  const int SD = 2 * nsr + 1, ND = SD * SD * SD, H = N / 2 + 1;
  const int ko0 = blockIdx.x * FB, a = blockIdx.y;
  for (int i = threadIdx.x; i < FB * ND; i += blockDim.x) {
    const int f = i / ND, iD = i % ND, ko = min(ko0 + f, NO - 1);
    const int kx = ko % H, ky = (ko / H) % H, kz = ko / (H * H);
    const int Dx = iD % SD - nsr, Dy = (iD / SD) % SD - nsr, Dz = iD / (SD * SD) - nsr;
    int e = (kx * Dx + ky * Dy + kz * Dz) % N;
    e += e < 0 ? N : 0;
    ph[f][iD] = tw[e];
  }
  __syncthreads();
  for (int m = threadIdx.x; m < M; m += blockDim.x) {
    double2 acc[FB];
#pragma unroll
    for (int f = 0; f < FB; ++f) acc[f] = make_double2(0.0, 0.0);
    const double *Ta = T + size_t(a) * ND * M + m;
    for (int iD = 0; iD < ND; ++iD) {
      const double t = Ta[size_t(iD) * M];
#pragma unroll
      for (int f = 0; f < FB; ++f) {
        acc[f].x += t * ph[f][iD].x;
        acc[f].y += t * ph[f][iD].y;
      }
    }
#pragma unroll
    for (int f = 0; f < FB; ++f)
      if (ko0 + f < NO) S[(size_t(ko0 + f) * na + a) * M + m] = acc[f];
  }
}

// The products at the orbit of one octant frequency k under the axis
// reflections (member r: axes in the bit mask r reflected), one configuration
// per block.  With S_r[a][R_r m] = sigma_r(a) S[a][m] (sigma: -1 for an odd
// power along a reflected axis), member r's fields are taken at reflected
// nodes, so every member uses the same spectrum value:
//   Psi_r[R_r m] = sum_a S[a][m] sigma_r(a) C_r[a],
//   B_r[a] = sigma_r(a) sum_m conj(S[a][m]) g_r[R_r m].
// Psi: one thread per node (MB members each).  B is a real product with 16
// columns (member r, real or imaginary part) on the float64 matrix cores: 16
// rows of (moment, part) per tile, summed over the nodes, the spectrum values
// read from memory as the left operand, the nodes split over the waves that
// the tiles leave.  16 lanes per moment instead, with a chain of loads each:
// 175 us in a box of 32^3, 96 so; both products of the 27-element q = 2 screen
// at 24^3 174 and 83 us.  (Psi by matrix-core steps too: 62 to 88 us in that
// box, whose 8 moments make four steps of a tile.)
struct ConvProd {
  int N, NO, p, nl, na, M, CHc, CHm;
  int MR;   // row stride of the nodes' values in LDS
  double scale;
  const double2 *S, *zc, *zg;
  double2 *zpsi, *za;
};
typedef double f64x4 __attribute__((ext_vector_type(4)));

__host__ __device__ constexpr int conv_tiles(int na) { return (2 * na + 15) / 16; }
__host__ __device__ constexpr int conv_split(int tiles) { return tiles >= 3 ? 1 : 4 / tiles; }   // waves that share a tile

template <int MB>
__device__ __forceinline__ void conv_psi(const ConvProd &a, const double2 *Sk, const double2 *Cs, double2 *Ps, int m, int r0,
                                         int q1) {
  double2 acc[MB];
#pragma unroll
  for (int r = 0; r < MB; ++r) acc[r] = make_double2(0.0, 0.0);
  for (int i = 0; i < a.na; ++i) {
    const double2 s = Sk[size_t(i) * a.M + m];
#pragma unroll
    for (int r = 0; r < MB; ++r) {
      const double2 c = Cs[i * 8 + r0 + r];
      acc[r].x += s.x * c.x - s.y * c.y;
      acc[r].y += s.x * c.y + s.y * c.x;
    }
  }
  const int mx = m % q1, my = (m / q1) % q1, mz = m / (q1 * q1);
#pragma unroll
  for (int r = 0; r < MB; ++r) {
    const int q = r0 + r;
    const int t = (((q & 4) ? q1 - 1 - mz : mz) * q1 + ((q & 2) ? q1 - 1 - my : my)) * q1 + ((q & 1) ? q1 - 1 - mx : mx);
    Ps[q * a.MR + t] = acc[r];
  }
}

template <bool PSI, bool ADJ>
__global__ __launch_bounds__(256) void k_conv_prod(ConvProd a) {
  extern __shared__ double2 lds[];
  double2 *Cs = lds;                                  // [na][8]: sigma_r C_r
  double *Gs = reinterpret_cast<double *>(Cs + (PSI ? 8 * a.na : 0));   // [8][MR][2]: g_r at R_r m; then Psi_r
  double *Ds = Gs + 16 * a.MR;                        // [split][tiles][16][16]: S by g
  const int N = a.N, H = N / 2 + 1, tid = threadIdx.x, M = a.M, MR = a.MR;
  const int nb = gridDim.x / a.NO, cfg = blockIdx.x % nb, ko = blockIdx.x / nb;   // a frequency's configurations in turn
  const int kx = ko % H, ky = (ko / H) % H, kz = ko / (H * H);
  const int q1 = a.p + 1;
  int pm = 0;
  if (kx != 0 && 2 * kx != N) pm |= 1;
  if (ky != 0 && 2 * ky != N) pm |= 2;
  if (kz != 0 && 2 * kz != N) pm |= 4;
  const size_t N3 = size_t(N) * N * N;
  auto fidx = [&](int r) {   // lattice index of member r (a bit outside pm reflects onto itself)
    r &= pm;
    const int x = (r & 1) ? N - kx : kx, y = (r & 2) ? N - ky : ky, z = (r & 4) ? N - kz : kz;
    return size_t(cfg) * N3 + (size_t(z) * N + y) * N + x;
  };
  const double2 *Sk = a.S + size_t(ko) * a.na * M;
  auto sigma = [&](int i, int r) {
    const int ax = i % a.nl, ay = (i / a.nl) % a.nl, az = i / (a.nl * a.nl);
    return (((r & 1) & ax) ^ ((r >> 1) & ay & 1) ^ ((r >> 2) & az & 1)) & 1 ? -1.0 : 1.0;
  };
  auto refl = [&](int m, int r) {
    const int mx = m % q1, my = (m / q1) % q1, mz = m / (q1 * q1);
    return (((r & 4) ? q1 - 1 - mz : mz) * q1 + ((r & 2) ? q1 - 1 - my : my)) * q1 + ((r & 1) ? q1 - 1 - mx : mx);
  };
  if constexpr (PSI) {   // unpack the real channels' transforms: Z(f), Z(-f)
    for (int i = tid; i < 8 * a.na; i += 256) {
      const int r = i & 7, m = i >> 3;
      const double2 z = a.zc[fidx(r) * a.CHc + (m >> 1)], zm = a.zc[fidx(r ^ 7) * a.CHc + (m >> 1)];
      const double g = 0.5 * sigma(m, r);
      Cs[i] = (m & 1) ? make_double2(g * (z.y + zm.y), -g * (z.x - zm.x)) : make_double2(g * (z.x + zm.x), g * (z.y - zm.y));
    }
  }
  if constexpr (ADJ) {
    for (int i = tid; i < 8 * a.CHm; i += 256) {
      const int r = i / a.CHm, c = i % a.CHm;
      const double2 z = a.zg[fidx(r) * a.CHm + c], zm = a.zg[fidx(r ^ 7) * a.CHm + c];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int m = 2 * c + h;
        if (m >= M) continue;
        double *g = Gs + 2 * (r * MR + refl(m, r));
        g[0] = h ? 0.5 * (z.y + zm.y) : 0.5 * (z.x + zm.x);
        g[1] = h ? -0.5 * (z.x - zm.x) : 0.5 * (z.y - zm.y);
      }
    }
    for (int i = tid; i < 16 * (MR - M); i += 256) Gs[2 * ((i >> 1) / (MR - M) * MR + M + (i >> 1) % (MR - M)) + (i & 1)] = 0.0;
  }
  __syncthreads();
  if constexpr (ADJ) {
    const int lane = tid & 63, wave = tid >> 6, i16 = lane & 15, kq = lane >> 4;
    const int tiles = conv_tiles(a.na), split = conv_split(tiles), steps = (M + 3) / 4;
    for (int u = wave; u < tiles * split; u += 4) {
      const int t = u % tiles, part = u / tiles;
      const int row = min(16 * t + i16, 2 * a.na - 1);   // rows past the last are not used
      const double *s = reinterpret_cast<const double *>(Sk + size_t(row >> 1) * M) + (row & 1), *g = Gs + (i16 >> 1) * 2 * MR + (i16 & 1);
      f64x4 acc{0.0, 0.0, 0.0, 0.0};
#pragma unroll 8
      for (int ks = part; ks < steps; ks += split) {
        const int m = 4 * ks + kq;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(s[2 * min(m, M - 1)], g[2 * m], acc, 0, 0, 0);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) Ds[(part * tiles + t) * 256 + (kq + 4 * v) * 16 + i16] = acc[v];
    }
    __syncthreads();
    for (int i = tid; i < 8 * a.CHc; i += 256) {
      const int r = i / a.CHc, c = i % a.CHc;
      if (r & ~pm) continue;
      double2 B[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int j = 2 * c + h;
        double re = 0.0, im = 0.0;
        if (j < a.na)
          for (int part = 0; part < split; ++part) {
            const double *d = Ds + part * tiles * 256 + 2 * j * 16 + 2 * r;
            re += d[0] + d[17];
            im += d[1] - d[16];
          }
        const double g = j < a.na ? sigma(j, r) : 0.0;
        B[h] = make_double2(g * re, g * im);
      }
      a.za[fidx(r) * a.CHc + c] = make_double2((B[0].x - B[1].y) * a.scale, (B[0].y + B[1].x) * a.scale);
    }
  }
  if constexpr (PSI) {   // Gs was last read before the barrier above
    // threads beyond one per node share a node's members
    double2 *Ps = reinterpret_cast<double2 *>(Gs);
    if (M <= 64) conv_psi<2>(a, Sk, Cs, Ps, min(tid & 63, M - 1), 2 * (tid >> 6), q1);
    else if (M <= 128) conv_psi<4>(a, Sk, Cs, Ps, min(tid & 127, M - 1), 4 * (tid >> 7), q1);
    else
      for (int m = tid; m < M; m += 256) conv_psi<8>(a, Sk, Cs, Ps, m, 0, q1);
    __syncthreads();
    for (int i = tid; i < 8 * a.CHm; i += 256) {
      const int r = i / a.CHm, c = i % a.CHm;
      if (r & ~pm) continue;
      const double2 u = Ps[r * MR + 2 * c], v = 2 * c + 1 < M ? Ps[r * MR + 2 * c + 1] : make_double2(0.0, 0.0);
      a.zpsi[fidx(r) * a.CHm + c] = make_double2((u.x - v.y) * a.scale, (u.y + v.x) * a.scale);
    }
  }
}

template <int IN, int OUT>
void pass(hipStream_t s, const ConvPass &a) {
  const size_t total = size_t(a.nb) * a.e1 * a.e2 * a.CH;
  hipLaunchKernelGGL((k_conv_pass<IN, OUT>), dim3(unsigned((total + kCols - 1) / kCols)), dim3(256), 0, s, a);
}

ConvPass pass_of(const ConvPlan &c, int nb, int nch, bool inverse) {
  ConvPass a{};
  a.N = c.N;
  a.r1 = c.r1;
  a.r2 = c.r2;
  a.CH = (nch + 1) / 2;
  a.n = c.n;
  a.nch = nch;
  a.nb = nb;
  a.inverse = inverse;
  a.tw = c.tw;
  a.p = c.p;
  a.P = c.box ? c.p * c.n + 1 : c.p * c.n;
  a.wrap = !c.box;
  a.sign = 1.0;
  return a;
}

// Axis order x, y, z of a forward transform from a real array: only the rows
// inside the n^3 elements hold data.
void forward(hipStream_t s, const ConvPlan &c, int nb, int nch, const double *in, double2 *z) {
  ConvPass a = pass_of(c, nb, nch, false);
  a.rin = in;
  a.in = z;
  a.out = z;
  a.nin = c.n;
  a.nout = c.N;
  a.axis = 0;
  a.e1 = a.e2 = c.n;
  pass<kInReal, kOutComplex>(s, a);
  a.axis = 1;
  a.e1 = c.N;
  pass<kInComplex, kOutComplex>(s, a);
  a.axis = 2;
  a.e2 = c.N;
  pass<kInComplex, kOutComplex>(s, a);
}

// z, y, then x into a real array: only the n^3 elements are wanted.
template <int OUT>
void inverse(hipStream_t s, const ConvPlan &c, int nb, int nch, double2 *z, double *out, double sign, const double *phi) {
  ConvPass a = pass_of(c, nb, nch, true);
  a.in = z;
  a.out = z;
  a.rout = out;
  a.sign = sign;
  a.phi = phi;
  a.nin = c.N;
  a.nout = c.n;
  a.axis = 2;
  a.e1 = a.e2 = c.N;
  pass<kInComplex, kOutComplex>(s, a);
  a.axis = 1;
  a.e2 = c.n;
  pass<kInComplex, kOutComplex>(s, a);
  a.axis = 0;
  a.e1 = c.n;
  pass<kInComplex, OUT>(s, a);
}

}  // namespace

bool conv_plan(int n, int nsr, int p, int nl, bool box, ConvPlan &c) {
  c = ConvPlan{};
  c.n = n;
  c.N = conv_edge(n, nsr, box);
  c.nsr = nsr;
  c.p = p;
  c.nl = nl;
  c.na = nl * nl * nl;
  c.M = (p + 1) * (p + 1) * (p + 1);
  c.box = box;
  return c.N > 0 && radices(c.N, c.r1, c.r2);
}

void launch_conv_spec(hipStream_t s, const ConvPlan &c, double *T) {
  const int S = 2 * c.nsr + 1;
  const size_t count = size_t(c.na) * S * S * S * c.M;
  hipLaunchKernelGGL(k_conv_symmetrise, dim3(unsigned((count + 255) / 256)), dim3(256), 0, s, count, c.p, c.nl, c.nsr, T);
  const int H = c.N / 2 + 1, NO = H * H * H;
  hipLaunchKernelGGL(k_conv_spec, dim3((NO + 7) / 8, c.na), dim3(256), 0, s, c.N, NO, c.nsr, c.na, c.M, T, c.tw, c.S);
}

void launch_conv_products(hipStream_t s, const ConvPlan &c, int nb, const double *C, const double *gE) {
  if (C) forward(s, c, nb, c.na, C, c.zc);
  if (gE) forward(s, c, nb, c.M, gE, c.zg);
  ConvProd a{};
  const int H = c.N / 2 + 1;
  a.N = c.N;
  a.NO = H * H * H;
  a.p = c.p;
  a.nl = c.nl;
  a.na = c.na;
  a.M = c.M;
  a.CHc = (c.na + 1) / 2;
  a.CHm = (c.M + 1) / 2;
  a.scale = 1.0 / (double(c.N) * c.N * c.N);
  a.S = c.S;
  a.zc = c.zc;
  a.zg = c.zg;
  a.zpsi = c.zpsi;
  a.za = c.za;
  const dim3 grid(unsigned(a.NO) * nb);
  a.MR = (c.M + 3) / 4 * 4 | 1;   // odd: the members' rows on different banks
  const int tiles = conv_tiles(c.na);
  const size_t lds = ((C ? size_t(16) * c.na : 0) + size_t(16) * a.MR + (gE ? size_t(256) * tiles * conv_split(tiles) : 0)) *
                     sizeof(double);
  if (C && gE) hipLaunchKernelGGL((k_conv_prod<true, true>), grid, dim3(256), lds, s, a);
  else if (C) hipLaunchKernelGGL((k_conv_prod<true, false>), grid, dim3(256), lds, s, a);
  else hipLaunchKernelGGL((k_conv_prod<false, true>), grid, dim3(256), lds, s, a);
}

void launch_conv_psi(hipStream_t s, const ConvPlan &c, int nb, const double *phi, double *W) {
  inverse<kOutW>(s, c, nb, c.M, c.zpsi, W, -1.0, phi);
}

void launch_conv_adjoint(hipStream_t s, const ConvPlan &c, int nb, double sign, double *A) {
  inverse<kOutReal>(s, c, nb, c.na, c.za, A, sign, nullptr);
}

}  // namespace fep3m
