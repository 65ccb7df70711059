// Near-screen field and its transpose by the convolution theorem.
//
// Both near-field contractions are periodic convolutions over the element
// lattice whose kernel is the table of Section 3 (eq. sc, the Remark's
// order-p tables), with 8 moment channels on one side and the (p+1)^3 node
// channels on the other:
//
//   Psi_E[m] = sum_D sum_a T[a][D][m] C[E - D][a]    (element-to-point field)
//   B_E[a]   = sum_D sum_m T[a][D][m] g[E + D][m]    (its transpose, in the
//                                                     moment adjoint)
//
// With X^(k) = sum_E X[E] exp(-2 pi i k.E / n) and the table spectrum
//   S[k][a][m] = sum_D T[a][D][m] exp(-2 pi i k.D / n)
// they read Psi^_m(k) = sum_a S[k][a][m] C^_a(k) and
// B^_a(k) = sum_m conj(S[k][a][m]) g^_m(k) (T is real).  The same linear maps
// as the direct sums, evaluated with 3-D FFTs of the element lattice: about
// 2 * 8 * 216 * 16 FLOP per element for the products against 1.19 MFLOP per
// element for the direct sums; the work becomes memory-bound.
//
// Layout: every transformed field is [config][z][y][x][channel] complex
// (double2), channel fastest, where two consecutive real channels form one
// complex channel: the moments C[E][8] are 4 complex channels in place, the
// node fields [E][216] are 108.  One complex FFT of the pair (X_2c + i X_2c+1)
// transforms both real channels; X^_2c(k) = (Z(k) + conj Z(-k)) / 2 and
// X^_2c+1(k) = (Z(k) - conj Z(-k)) / 2i separate them in the products, which
// also pack their two real outputs the same way, so the inverse transforms
// return real pairs directly.  The tables are symmetric under the three axis
// reflections, so the spectrum is kept for one octant of frequencies
// (0 <= k_x, k_y, k_z <= n/2: 0.99 GB at n = 64) and each product block
// handles the orbit of one octant frequency (which holds -k as well).  With
// forces both products run in the same blocks: one read of the spectrum.
//
// FFTs: one kernel per axis, decimation in time in LDS (radix-2 stages
// taken two at a time).  A block holds lb lines x cc channels of length n
// (at most 2048 complex values):
// rows of cc consecutive channels (and lb consecutive elements across the
// line for the y and z passes) are contiguous in memory.  Twiddles come from
// a table computed on the host.  n is a power of two, 8 .. 64.
#include "kernels.hpp"

namespace fep3m {

namespace {

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// conj(a) b
__device__ __forceinline__ double2 cmulc(double2 a, double2 b) {
  return make_double2(a.x * b.x + a.y * b.y, a.x * b.y - a.y * b.x);
}

constexpr int kFftCap = 2048;   // complex values per FFT block (32 KB of LDS)

}  // namespace

// Block shape of an FFT pass: cc channels (a divisor of nch) x lb lines of
// length n, at most kFftCap complex values.
constexpr int fft_cc(int n, int nch) {
  int cc = nch;
  while (n * cc > kFftCap || nch % cc != 0) --cc;
  return cc;
}
constexpr int fft_lb(int n, int nch) {
  const int cc = fft_cc(n, nch);
  int lb = 1;
  while (2 * lb <= n && n * 2 * lb * cc <= kFftCap) lb *= 2;
  return lb;
}

// One axis of a batched 3-D FFT over [cfg][z][y][x][NCH] complex values,
// n = 2^LOGN.  EPI 0: store the transformed values to dst (src == dst
// allowed: a block reads all its values before it writes).  EPI 1 (last
// inverse pass of the field): the values are (Psi_2c, Psi_2c+1) of element
// E; store W_E[m] = phi(node of m) - Psi_m to Wout (float64 or float32),
// phi the order-po mesh potential.  MESH (along x, NCH = po^3, W null): the
// forward transform reads its values from the real mesh vectors 2 cfg and
// 2 cfg + 1 of phi as real and imaginary parts (channel: node within the
// element, x fastest), the inverse one writes them to those of Wout; nsys
// vectors in all.  The passes of its own that this replaces took 305 us each
// way at 64^3, p = 5.
template <int LOGN, int NCH, bool INV, int EPI, class WT, bool MESH = false>
__global__ __launch_bounds__(256) void k_fft_axis(int axis, const double2 *src, double2 *dst,
                                                  const double2 *__restrict__ tw, const double *__restrict__ phi,
                                                  WT *__restrict__ Wout, int po, int nsys) {
  constexpr int N = 1 << LOGN, CC = fft_cc(N, NCH), LB = fft_lb(N, NCH);
  constexpr int U = LB * CC, TOT = N * U;
  constexpr int NCHUNK = NCH / CC, NG = N / LB;
  __shared__ double2 buf[TOT];   // [j][u], u = l CC + c
  __shared__ double2 tws[N / 2];
  int b = blockIdx.x;
  const int chunk = b % NCHUNK;
  b /= NCHUNK;
  const int g = b % NG;
  b /= NG;
  const int outer = b % N;
  const int cfg = b / N;
  size_t sj, sl, so;
  if (axis == 0) { sj = NCH; sl = size_t(N) * NCH; so = size_t(N) * N * NCH; }
  else if (axis == 1) { sj = size_t(N) * NCH; sl = NCH; so = size_t(N) * N * NCH; }
  else { sj = size_t(N) * N * NCH; sl = NCH; so = size_t(N) * NCH; }
  const size_t base = size_t(cfg) * N * N * N * NCH + size_t(outer) * so + size_t(g) * LB * sl + size_t(chunk) * CC;
  const int tid = threadIdx.x;
  // position (j, l, c) of value i: the thread order follows memory
  auto coords = [&](int i, int &j, int &l, int &c) {
    c = i % CC;
    const int r = i / CC;
    if (axis == 0) { j = r % N; l = r / N; } else { l = r % LB; j = r / LB; }
  };
  // MESH: values in the order of the mesh's rows; their address in vector 2 cfg
  auto mesh_at = [&](int i, int &j, int &u) -> size_t {
    constexpr int PO = NCH == 27 ? 3 : NCH == 64 ? 4 : NCH == 125 ? 5 : 6, P = PO * N;
    int l, c;
    if constexpr (CC % PO == 0) {
      const int r = i / PO / N;
      j = i / PO % N;
      c = r % (CC / PO) * PO + i % PO;
      l = r / (CC / PO);
    } else {
      coords(i, j, l, c);
    }
    u = l * CC + c;
    const int ch = chunk * CC + c, ky = ch / PO % PO, kz = ch / (PO * PO);
    return ((size_t(2 * cfg) * P + PO * outer + kz) * P + PO * (g * LB + l) + ky) * P + PO * j + ch % PO;
  };
  const size_t next = size_t(po) * N * po * N * po * N;   // from vector 2 cfg to 2 cfg + 1
  const bool two = 2 * cfg + 1 < nsys;
  if (tid < N / 2) tws[tid] = tw[tid];
  if constexpr (MESH && !INV) {
    for (int i = tid; i < TOT; i += 256) {
      int j, u;
      const size_t a = mesh_at(i, j, u);
      buf[int(__brev(unsigned(j)) >> (32 - LOGN)) * U + u] = make_double2(phi[a], two ? phi[a + next] : 0.0);
    }
  } else
  for (int i = tid; i < TOT; i += 256) {   // stored in bit-reversed order of j
    int j, l, c;
    coords(i, j, l, c);
    buf[int(__brev(unsigned(j)) >> (32 - LOGN)) * U + l * CC + c] = src[base + j * sj + l * sl + c];
  }
  __syncthreads();
  // Radix-2 stages (half-size h = 2^s, twiddle W_2h^pos), taken two at a
  // time: one pass over LDS does stages s and s + 1 on the four values
  // j0 + {0, h, 2h, 3h} (the same operations in the same order, so the
  // result equals the stage-by-stage one); an odd count starts with a single
  // stage.
  if (LOGN & 1) {
    for (int t = tid; t < (N / 2) * U; t += 256) {   // s = 0: twiddle 1
      const int u = t % U, j0 = 2 * (t / U);
      const double2 x0 = buf[j0 * U + u], x1 = cmul(buf[(j0 + 1) * U + u], tws[0]);
      buf[j0 * U + u] = cadd(x0, x1);
      buf[(j0 + 1) * U + u] = csub(x0, x1);
    }
    __syncthreads();
  }
#pragma unroll
  for (int s = LOGN & 1; s < LOGN; s += 2) {
    const int h = 1 << s;
    for (int t = tid; t < (N / 4) * U; t += 256) {
      const int u = t % U, bf = t / U;
      const int pos = bf & (h - 1);
      const int j0 = ((bf >> s) << (s + 2)) + pos;
      double2 w1 = tws[pos << (LOGN - 1 - s)], w2 = tws[pos << (LOGN - 2 - s)],
              w3 = tws[(pos + h) << (LOGN - 2 - s)];
      if (INV) { w1.y = -w1.y; w2.y = -w2.y; w3.y = -w3.y; }
      const double2 x0 = buf[j0 * U + u], x1 = buf[(j0 + h) * U + u];
      const double2 x2 = buf[(j0 + 2 * h) * U + u], x3 = buf[(j0 + 3 * h) * U + u];
      const double2 t1 = cmul(x1, w1), t3 = cmul(x3, w1);
      const double2 a0 = cadd(x0, t1), a1 = csub(x0, t1), a2 = cadd(x2, t3), a3 = csub(x2, t3);
      const double2 t2 = cmul(a2, w2), t4 = cmul(a3, w3);
      buf[j0 * U + u] = cadd(a0, t2);
      buf[(j0 + h) * U + u] = cadd(a1, t4);
      buf[(j0 + 2 * h) * U + u] = csub(a0, t2);
      buf[(j0 + 3 * h) * U + u] = csub(a1, t4);
    }
    __syncthreads();
  }
  if constexpr (MESH && INV) {
    for (int i = tid; i < TOT; i += 256) {
      int j, u;
      const size_t a = mesh_at(i, j, u);
      const double2 v = buf[j * U + u];
      Wout[a] = v.x;
      if (two) Wout[a + next] = v.y;
    }
  } else if (EPI == 0) {
    for (int i = tid; i < TOT; i += 256) {
      int j, l, c;
      coords(i, j, l, c);
      dst[base + j * sj + l * sl + c] = buf[j * U + l * CC + c];
    }
  } else {
    const int Q1 = po + 1, NM = Q1 * Q1 * Q1, P = po * N;
    const size_t M = size_t(N) * N * N;
    phi += size_t(cfg) * P * P * P;
    for (int i = tid; i < TOT; i += 256) {
      int j, l, c;
      coords(i, j, l, c);
      int ex, ey, ez;
      const int lc = g * LB + l;
      if (axis == 0) { ex = j; ey = lc; ez = outer; }
      else if (axis == 1) { ey = j; ex = lc; ez = outer; }
      else { ez = j; ex = lc; ey = outer; }
      const double2 v = buf[j * U + l * CC + c];
      const size_t E = size_t(cfg) * M + (size_t(ez) * N + ey) * N + ex;
      const int ch = chunk * CC + c;
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const int m = 2 * ch + q;
        const int mx = m % Q1, my = (m / Q1) % Q1, mz = m / (Q1 * Q1);
        int gx = po * ex + mx, gy = po * ey + my, gz = po * ez + mz;
        gx -= gx >= P ? P : 0;
        gy -= gy >= P ? P : 0;
        gz -= gz >= P ? P : 0;
        const double ph = phi[(size_t(gz) * P + gy) * P + gx];
        Wout[E * NM + m] = WT(ph - (q == 0 ? v.x : v.y));
      }
    }
  }
}

// Spectrum products over the orbit of one octant frequency k (0 <= k_x,
// k_y, k_z <= n/2) under the reflections of the axes whose component is
// neither 0 nor n/2 (pm): the up to 8 frequencies R k, among them -k.  The
// tables are symmetric under each axis reflection R (node m -> R m, offset
// D -> R D, moment a -> (-1)^(a.R) a), so S[a][m](R k) = (-1)^(a.R)
// S[a][R m](k): one stored row of 8 x 216 values serves the whole orbit.
//   PSI: Zpsi(R k)[c] = (Psi^_2c + i Psi^_2c+1)(R k) * scale
//   ADJ: ZA(R k)[j] = (B^_2j + i B^_2j+1)(R k) * scale
// Moments are indexed a = a_x + 2 a_y + 4 a_z (each 0 or 1), nodes
// m = m_x + 6 (m_y + 6 m_z).
//
// Bound by memory (the spectrum, the transformed deposits and the field: 1.9
// GB at 64^3, 0.38 ms at the copy rate) if the LDS reads of the products stay
// below: a thread of the first product takes two frequencies of the orbit that
// differ in k_x, which share their spectrum values (their node pairs swapped);
// the second one is a 16 x 216 x 16 real product (moment and part of S by
// frequency and part of the deposit), 54 float64 matrix-core steps over the
// waves, on deposits stored under their reflected node.  One frequency per
// thread and a thread per output of the second product read 0.66 MB of LDS
// per orbit: 767 us; 482 so (130 and 66 us at 32^3).  Rows of 217 values keep the steps' 16 rows on
// different banks.
constexpr int kOrbitThreads = 512;
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <bool PSI, bool ADJ>
__global__ __launch_bounds__(kOrbitThreads) void k_spec_orbit(int n, int NO, const double2 *__restrict__ S,
                                                    const double2 *__restrict__ ZC, double2 *__restrict__ Zpsi,
                                                    const double2 *__restrict__ Zg, double2 *__restrict__ ZA,
                                                    double scale) {
  constexpr int Q1 = 6, NM = Q1 * Q1 * Q1, NC = NM / 2, NT = kOrbitThreads, NQ = NT / 64;
  constexpr int NR = NM + 1;   // row stride
  static_assert(NM % 4 == 0 && NQ * 256 <= 2 * 8 * NR, "steps of the transposed product");
  __shared__ double2 Ss[8 * NR + 1];   // one spare slot
  __shared__ double2 Cs[8][8];
  __shared__ double2 Gs[ADJ ? 8 * NR : 1];   // reused for the partial sums
  const int H = n / 2 + 1;
  const int ko = blockIdx.x % NO, cfg = blockIdx.x / NO;
  const int kx = ko % H, ky = (ko / H) % H, kz = ko / (H * H);
  int pm = 0;
  if (kx != 0 && 2 * kx != n) pm |= 1;
  if (ky != 0 && 2 * ky != n) pm |= 2;
  if (kz != 0 && 2 * kz != n) pm |= 4;
  auto fidx = [&](int r) {
    const int x = (r & 1) ? n - kx : kx, y = (r & 2) ? n - ky : ky, z = (r & 4) ? n - kz : kz;
    return size_t((z * n + y) * n + x);
  };
  auto refl = [](int m, int r) {
    int mx = m % Q1, my = (m / Q1) % Q1, mz = m / (Q1 * Q1);
    if (r & 1) mx = Q1 - 1 - mx;
    if (r & 2) my = Q1 - 1 - my;
    if (r & 4) mz = Q1 - 1 - mz;
    return (mz * Q1 + my) * Q1 + mx;
  };
  const size_t M = size_t(n) * n * n;
  const int tid = threadIdx.x;
  const double2 *Sk = S + size_t(ko) * 8 * NM;
  {   // all loads of the row in flight before the LDS stores
    constexpr int KS = (8 * NM + NT - 1) / NT;
    double2 v[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) v[k] = Sk[min(tid + NT * k, 8 * NM - 1)];   // clamped: no branch per load
    asm volatile("" ::: "memory");   // compiler fence: all loads issue before the stores
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      const int i = tid + NT * k;
      Ss[i < 8 * NM ? i + i / NM : 8 * NR] = v[k];   // lanes past the end: spare slot
    }
  }
  if constexpr (PSI) if (tid < 64) {   // C^_a at each orbit frequency, from Z(f) and Z(-f)
    const int r = tid >> 3, a = tid & 7;
    if ((r & ~pm) == 0) {
      const double2 z = ZC[(size_t(cfg) * M + fidx(r)) * 4 + (a >> 1)];
      const double2 zm = ZC[(size_t(cfg) * M + fidx(r ^ pm)) * 4 + (a >> 1)];
      Cs[r][a] = (a & 1) ? make_double2(0.5 * (z.y + zm.y), -0.5 * (z.x - zm.x))
                         : make_double2(0.5 * (z.x + zm.x), 0.5 * (z.y - zm.y));
    }
  }
  if constexpr (ADJ) {
    constexpr int KG = (8 * NC + NT - 1) / NT;
    double2 z[KG], zm[KG];
#pragma unroll
    for (int k = 0; k < KG; ++k) {   // unconditional loads (frequencies outside the orbit read k itself)
      const int i = min(tid + NT * k, 8 * NC - 1), r = (i / NC) & pm, c = i % NC;
      z[k] = Zg[(size_t(cfg) * M + fidx(r)) * NC + c];
      zm[k] = Zg[(size_t(cfg) * M + fidx(r ^ pm)) * NC + c];
    }
    asm volatile("" ::: "memory");
#pragma unroll
    for (int k = 0; k < KG; ++k) {   // rows outside the orbit are summed but not used
      const int i = min(tid + NT * k, 8 * NC - 1), r = i / NC, c = i % NC;
      Gs[r * NR + refl(2 * c, r)] = make_double2(0.5 * (z[k].x + zm[k].x), 0.5 * (z[k].y - zm[k].y));
      Gs[r * NR + refl(2 * c + 1, r)] = make_double2(0.5 * (z[k].y + zm[k].y), -0.5 * (z[k].x - zm[k].x));
    }
  }
  __syncthreads();
  if constexpr (PSI) {
    for (int i = tid; i < 4 * NC; i += NT) {   // frequencies r and r + 1, channel c of the first
      const int r = 2 * (i / NC), c = i % NC;
      if (r & ~pm) continue;
      const int m0 = refl(2 * c, r), m1 = m0 + 1;   // S rows' pair; with k_x reversed nodes m1, m0 of channel c2
      const int c2 = c - 2 * (c % (Q1 / 2)) + Q1 / 2 - 1;
      double2 P0 = make_double2(0.0, 0.0), P1 = P0, R0 = P0, R1 = P0;
      auto mac = [](double2 &P, double2 s, double2 ch) {   // P += s ch with its roundings spelled out: the float32
        P.x += fma(s.x, ch.x, -(s.y * ch.y));              // element field of mixed precision follows from the sum,
        P.y += fma(s.x, ch.y, s.y * ch.x);                 // and a last bit can move its rounding
      };
#pragma unroll
      for (int a = 0; a < 8; ++a) {
        const double2 s0 = Ss[a * NR + m0], s1 = Ss[a * NR + m1];
        const double sg = (__popc(a & r) & 1) ? -1.0 : 1.0;
        const double2 ch = make_double2(sg * Cs[r][a].x, sg * Cs[r][a].y);
        mac(P0, s0, ch);
        mac(P1, s1, ch);
        const double sh = (a & 1) ? -sg : sg;
        const double2 dh = make_double2(sh * Cs[r + 1][a].x, sh * Cs[r + 1][a].y);
        mac(R0, s1, dh);
        mac(R1, s0, dh);
      }
      Zpsi[(size_t(cfg) * M + fidx(r)) * NC + c] = make_double2((P0.x - P1.y) * scale, (P0.y + P1.x) * scale);
      if (pm & 1)
        Zpsi[(size_t(cfg) * M + fidx(r + 1)) * NC + c2] = make_double2((R0.x - R1.y) * scale, (R0.y + R1.x) * scale);
    }
  }
  if constexpr (ADJ) {
    // D[2 a + s][2 r + g] = sum_m S_s[a][m] G_g[r][m], s and g the real (0) or
    // imaginary part: every wave takes each NQ-th step of four nodes
    const int lane = tid & 63, wave = tid >> 6, i16 = lane & 15, kq = lane >> 4;
    const double *sp = reinterpret_cast<const double *>(Ss) + (i16 >> 1) * 2 * NR + 2 * kq + (i16 & 1);
    const double *gp = reinterpret_cast<const double *>(Gs) + (i16 >> 1) * 2 * NR + 2 * kq + (i16 & 1);
    f64x4 acc{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < (NM / 4 + NQ - 1) / NQ; ++k) {
      const int ks = wave + NQ * k;
      if (ks < NM / 4) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(sp[8 * ks], gp[8 * ks], acc, 0, 0, 0);
    }
    __syncthreads();
    double *red = reinterpret_cast<double *>(Gs);   // [wave][row][column]
#pragma unroll
    for (int v = 0; v < 4; ++v) red[wave * 256 + (kq + 4 * v) * 16 + i16] = acc[v];
    __syncthreads();
    double t = 0.0;
    if (tid < 256) {
#pragma unroll
      for (int w = 0; w < NQ; ++w) t += red[w * 256 + tid];
    }
    double *D = reinterpret_cast<double *>(Ss);   // its rows are read
    if (tid < 256) D[tid] = t;
    __syncthreads();
    if (tid < 32) {   // A0 + i A1 of moments 2 j and 2 j + 1, A = sum conj(S) G with the reflection's sign
      const int r = tid >> 2, j = tid & 3;
      if ((r & ~pm) == 0) {
        double2 A[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int a = 2 * j + q;
          const double sg = (__popc(a & r) & 1) ? -1.0 : 1.0;
          const double *d = D + 2 * a * 16 + 2 * r;
          A[q] = make_double2(sg * (d[0] + d[17]), sg * (d[1] - d[16]));
        }
        ZA[(size_t(cfg) * M + fidx(r)) * 4 + j] = make_double2((A[0].x - A[1].y) * scale, (A[0].y + A[1].x) * scale);
      }
    }
  }
}

// Table spectrum S[ko][a][m] at the octant frequencies ko = k_x + H (k_y +
// H k_z), H = n/2 + 1: 8 frequencies per block, one thread per node m, the
// phases exp(-2 pi i k.D / n) = tw[(k.D) mod n] of the block's frequencies
// in LDS.
template <int NSR>
__global__ __launch_bounds__(256) void k_spec_build(int n, int NO, int nm, const double *__restrict__ T,
                                                    const double2 *__restrict__ twf, double2 *__restrict__ S) {
  constexpr int SD = 2 * NSR + 1, ND = SD * SD * SD, FB = 8;
  __shared__ double2 ph[FB][ND];
  const int H = n / 2 + 1;
  const int ko0 = blockIdx.x * FB;
  for (int i = threadIdx.x; i < FB * ND; i += blockDim.x) {
    const int f = i / ND, iD = i % ND;
    const int ko = min(ko0 + f, NO - 1);
    const int kx = ko % H, ky = (ko / H) % H, kz = ko / (H * H);
    const int Dx = iD % SD - NSR, Dy = (iD / SD) % SD - NSR, Dz = iD / (SD * SD) - NSR;
    int e = (kx * Dx + ky * Dy + kz * Dz) % n;
    e += e < 0 ? n : 0;
    ph[f][iD] = twf[e];
  }
  __syncthreads();
  const int m = threadIdx.x;
  if (m >= nm) return;
  for (int a = 0; a < 8; ++a) {
    double2 acc[FB];
#pragma unroll
    for (int f = 0; f < FB; ++f) acc[f] = make_double2(0.0, 0.0);
    const double *Ta = T + size_t(a) * ND * nm + m;
    for (int iD = 0; iD < ND; ++iD) {
      const double t = Ta[size_t(iD) * nm];
#pragma unroll
      for (int f = 0; f < FB; ++f) {
        acc[f].x += t * ph[f][iD].x;
        acc[f].y += t * ph[f][iD].y;
      }
    }
#pragma unroll
    for (int f = 0; f < FB; ++f)
      if (ko0 + f < NO) S[(size_t(ko0 + f) * 8 + a) * nm + m] = acc[f];
  }
}

// A[E][a] = 4 pi <lambda_E, G_a> - B_E[a], B from the inverse transform.
// Eight lanes per element: lane k < Q1 contracts node plane k with the x and
// y moments, then lane a sums moment a over the planes (through LDS), so A
// and B move in whole lines.  Bound by the reads of lambda, whose rows of Q1
// nodes overlap between elements: 118 us at 64^3 and 25 us on any small mesh
// with one thread per element (a chain of 216 loads), 86 and 6 us so.
template <int PO>
__global__ __launch_bounds__(256) void k_adj_finish(int n, int nb, const double *__restrict__ lam,
                                                    const double *__restrict__ gw, const double *__restrict__ Bn,
                                                    double *__restrict__ Aout) {
  constexpr int Q1 = PO + 1;
  static_assert(Q1 <= 8, "one lane per node plane");
  __shared__ double pl[32][8][5];   // [element][plane][moment in x, y]
  __shared__ double g[2 * Q1];
  const size_t M = size_t(n) * n * n;
  const int el8 = threadIdx.x >> 3, k = threadIdx.x & 7;
  const size_t E = size_t(blockIdx.x) * 32 + el8;
  const bool ok = E < size_t(nb) * M;
  if (threadIdx.x < 2 * Q1) g[threadIdx.x] = gw[threadIdx.x];
  __syncthreads();
  if (ok && k < Q1) {
    const int cfg = int(E / M);
    const int el = int(E % M);
    const int ex = el % n, ey = (el / n) % n, ez = el / (n * n);
    const int P = PO * n;
    int gz = PO * ez + k;
    gz -= gz >= P ? P : 0;
    const double *plane = lam + (size_t(cfg) * P + gz) * P * P;
    const int xl = PO * ex + PO >= P ? 0 : PO * ex + PO;   // the last node of the row, on the next element's face
    double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int my = 0; my < Q1; ++my) {
      int gy = PO * ey + my;
      gy -= gy >= P ? P : 0;
      const double *row = plane + size_t(gy) * P;
      double r0 = 0.0, r1 = 0.0;
#pragma unroll
      for (int mx = 0; mx < Q1; ++mx) {
        const double v = row[mx == PO ? xl : PO * ex + mx];
        r0 += v * g[mx];
        r1 += v * g[Q1 + mx];
      }
      s[0] += r0 * g[my];
      s[1] += r1 * g[my];
      s[2] += r0 * g[Q1 + my];
      s[3] += r1 * g[Q1 + my];
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) pl[el8][k][a] = s[a];
  }
  __syncthreads();
  if (!ok) return;
  double a1 = 0.0;
#pragma unroll
  for (int mz = 0; mz < Q1; ++mz) a1 += pl[el8][mz][k & 3] * g[(k >> 2) * Q1 + mz];
  Aout[E * 8 + k] = 4.0 * M_PI * a1 - Bn[E * 8 + k];
}

// ------------------------------------------------------------- launchers

bool fft_size_ok(int n) { return n >= 8 && n <= 64 && (n & (n - 1)) == 0; }

size_t spec_freqs(int n) { return size_t(n / 2 + 1) * (n / 2 + 1) * (n / 2 + 1); }

namespace {

template <int LOGN, int NCH, bool INV, int EPI, class WT, bool MESH>
void fft_launch(hipStream_t s, int nb, int axis, const double2 *src, double2 *dst, const double2 *tw,
                const double *phi, WT *W, int po, int nsys) {
  constexpr int N = 1 << LOGN, CC = fft_cc(N, NCH), LB = fft_lb(N, NCH);
  const dim3 grid(unsigned(size_t(nb) * N * (N / LB) * (NCH / CC)));
  hipLaunchKernelGGL((k_fft_axis<LOGN, NCH, INV, EPI, WT, MESH>), grid, dim3(256), 0, s, axis, src, dst, tw, phi, W, po,
                     nsys);
}

template <int NCH, bool INV, int EPI, class WT, bool MESH = false>
void fft_pass_n(hipStream_t s, int nb, int n, int axis, const double2 *src, double2 *dst, const double2 *tw,
                const double *phi, WT *W, int po, int nsys = 0) {
  switch (n) {
    case 8: fft_launch<3, NCH, INV, EPI, WT, MESH>(s, nb, axis, src, dst, tw, phi, W, po, nsys); break;
    case 16: fft_launch<4, NCH, INV, EPI, WT, MESH>(s, nb, axis, src, dst, tw, phi, W, po, nsys); break;
    case 32: fft_launch<5, NCH, INV, EPI, WT, MESH>(s, nb, axis, src, dst, tw, phi, W, po, nsys); break;
    default: fft_launch<6, NCH, INV, EPI, WT, MESH>(s, nb, axis, src, dst, tw, phi, W, po, nsys); break;
  }
}

// nch: 4 (moments) or 108 (node fields); EPI 1 only for node fields
template <bool INV, int EPI, class WT>
void fft_pass(hipStream_t s, int nb, int n, int nch, int axis, const double2 *src, double2 *dst,
              const double2 *tw, const double *phi, WT *W, int po) {
  if (EPI == 0 && nch == 4)
    fft_pass_n<4, INV, 0, WT>(s, nb, n, axis, src, dst, tw, phi, W, po);
  else
    fft_pass_n<108, INV, EPI, WT>(s, nb, n, axis, src, dst, tw, phi, W, po);
}

template <bool INV>
int fft_pass_nodes(hipStream_t s, int nb, int n, int nch, int axis, double2 *z, const double2 *tw) {
  switch (nch) {
    case 27: fft_pass_n<27, INV, 0, double>(s, nb, n, axis, z, z, tw, nullptr, nullptr, 0); return 0;
    case 64: fft_pass_n<64, INV, 0, double>(s, nb, n, axis, z, z, tw, nullptr, nullptr, 0); return 0;
    case 125: fft_pass_n<125, INV, 0, double>(s, nb, n, axis, z, z, tw, nullptr, nullptr, 0); return 0;
    case 216: fft_pass_n<216, INV, 0, double>(s, nb, n, axis, z, z, tw, nullptr, nullptr, 0); return 0;
    default: return -1;
  }
}

// forward 3-D transform: src (real pairs) -> dst, x then y then z
void fft3_forward(hipStream_t s, int nb, int n, int nch, const double2 *src, double2 *dst, const double2 *tw) {
  fft_pass<false, 0, double>(s, nb, n, nch, 0, src, dst, tw, nullptr, nullptr, 0);
  fft_pass<false, 0, double>(s, nb, n, nch, 1, dst, dst, tw, nullptr, nullptr, 0);
  fft_pass<false, 0, double>(s, nb, n, nch, 2, dst, dst, tw, nullptr, nullptr, 0);
}

}  // namespace

int launch_fft_nodes(hipStream_t s, int nb, int n, int nch, int axis, double2 *z, const double2 *tw, bool inverse) {
  if (!fft_size_ok(n)) return -1;
  return inverse ? fft_pass_nodes<true>(s, nb, n, nch, axis, z, tw) : fft_pass_nodes<false>(s, nb, n, nch, axis, z, tw);
}

int launch_fft_nodes_from_mesh(hipStream_t s, int nsys, int n, int p, const double *v, double2 *z, const double2 *tw) {
  if (!fft_size_ok(n)) return -1;
  const int nb = (nsys + 1) / 2;
  double *none = nullptr;
  switch (p) {
    case 3: fft_pass_n<27, false, 0, double, true>(s, nb, n, 0, z, z, tw, v, none, p, nsys); return 0;
    case 4: fft_pass_n<64, false, 0, double, true>(s, nb, n, 0, z, z, tw, v, none, p, nsys); return 0;
    case 5: fft_pass_n<125, false, 0, double, true>(s, nb, n, 0, z, z, tw, v, none, p, nsys); return 0;
    case 6: fft_pass_n<216, false, 0, double, true>(s, nb, n, 0, z, z, tw, v, none, p, nsys); return 0;
    default: return -1;
  }
}

int launch_fft_nodes_to_mesh(hipStream_t s, int nsys, int n, int p, double2 *z, double *v, const double2 *tw) {
  if (!fft_size_ok(n)) return -1;
  const int nb = (nsys + 1) / 2;
  const double *none = nullptr;
  switch (p) {
    case 3: fft_pass_n<27, true, 0, double, true>(s, nb, n, 0, z, z, tw, none, v, p, nsys); return 0;
    case 4: fft_pass_n<64, true, 0, double, true>(s, nb, n, 0, z, z, tw, none, v, p, nsys); return 0;
    case 5: fft_pass_n<125, true, 0, double, true>(s, nb, n, 0, z, z, tw, none, v, p, nsys); return 0;
    case 6: fft_pass_n<216, true, 0, double, true>(s, nb, n, 0, z, z, tw, none, v, p, nsys); return 0;
    default: return -1;
  }
}

void launch_spec_build(hipStream_t s, int n, int nsr, int p, const double *T, const double2 *twf, double2 *S) {
  const int nm = (p + 1) * (p + 1) * (p + 1);
  const int NO = int(spec_freqs(n));
  const dim3 grid(unsigned((NO + 7) / 8));
  switch (nsr) {
    case 1: hipLaunchKernelGGL(k_spec_build<1>, grid, dim3(256), 0, s, n, NO, nm, T, twf, S); break;
    case 2: hipLaunchKernelGGL(k_spec_build<2>, grid, dim3(256), 0, s, n, NO, nm, T, twf, S); break;
    default: hipLaunchKernelGGL(k_spec_build<3>, grid, dim3(256), 0, s, n, NO, nm, T, twf, S); break;
  }
}

int launch_near_fft(hipStream_t s, int nb, int n, int p, const double *C, const double *gE, const double2 *S,
                    const double2 *tw, double2 *zc, double2 *zpsi, double2 *zg, double2 *za) {
  if (p != 5 || !fft_size_ok(n) || (!C && !gE)) return -1;
  const int nc = (p + 1) * (p + 1) * (p + 1) / 2;
  const int NO = int(spec_freqs(n));
  const double scale = 1.0 / (double(n) * n * n);
  if (C) fft3_forward(s, nb, n, 4, reinterpret_cast<const double2 *>(C), zc, tw);
  if (gE) fft3_forward(s, nb, n, nc, reinterpret_cast<const double2 *>(gE), zg, tw);
  const dim3 grid(unsigned(size_t(nb) * NO));
  if (C && gE)
    hipLaunchKernelGGL((k_spec_orbit<true, true>), grid, dim3(kOrbitThreads), 0, s, n, NO, S, zc, zpsi, zg, za, scale);
  else if (C)
    hipLaunchKernelGGL((k_spec_orbit<true, false>), grid, dim3(kOrbitThreads), 0, s, n, NO, S, zc, zpsi, zg, za, scale);
  else
    hipLaunchKernelGGL((k_spec_orbit<false, true>), grid, dim3(kOrbitThreads), 0, s, n, NO, S, zc, zpsi, zg, za, scale);
  if (gE)
    for (int axis = 0; axis < 3; ++axis) fft_pass<true, 0, double>(s, nb, n, 4, axis, za, za, tw, nullptr, nullptr, 0);
  return 0;
}

template <class WT>
int launch_psi_fft_finish(hipStream_t s, int nb, int n, int p, const double2 *tw, const double *phi, double2 *zpsi,
                          WT *Wel) {
  if (p != 5 || !fft_size_ok(n)) return -1;
  const int nc = (p + 1) * (p + 1) * (p + 1) / 2;
  // z, y, then x with the W epilogue: along x the mesh potential is read in
  // contiguous rows (nodes p e_x + m_x) and W in runs of one element's nodes
  fft_pass<true, 0, double>(s, nb, n, nc, 2, zpsi, zpsi, tw, nullptr, nullptr, p);
  fft_pass<true, 0, double>(s, nb, n, nc, 1, zpsi, zpsi, tw, nullptr, nullptr, p);
  fft_pass<true, 1, WT>(s, nb, n, nc, 0, zpsi, zpsi, tw, phi, Wel, p);
  return 0;
}
template int launch_psi_fft_finish<double>(hipStream_t, int, int, int, const double2 *, const double *, double2 *,
                                           double *);
template int launch_psi_fft_finish<float>(hipStream_t, int, int, int, const double2 *, const double *, double2 *,
                                          float *);

int launch_adj_fft_finish(hipStream_t s, int nb, int n, int p, const double *lam, const double *gw, const double2 *za,
                          double *A) {
  if (!fft_size_ok(n)) return -1;
  return launch_adj_lambda(s, nb, n, p, lam, gw, reinterpret_cast<const double *>(za), A);
}

int launch_adj_lambda(hipStream_t s, int nb, int n, int p, const double *lam, const double *gw, const double *Bn,
                      double *A) {
  if (p != 5) return -1;
  const size_t ne = size_t(nb) * n * n * n;
  hipLaunchKernelGGL(k_adj_finish<5>, dim3(unsigned((ne + 31) / 32)), dim3(256), 0, s, n, nb, lam, gw, Bn, A);
  return 0;
}

}  // namespace fep3m
