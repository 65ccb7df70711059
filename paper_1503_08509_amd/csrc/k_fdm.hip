// Exact periodic mesh solve by Fourier analysis over the element lattice
// (the solver option of fep3m.h for meshes whose edge is a power of two).
//
// On the uniform periodic mesh the 1-D operators K1, M1 are block circulant:
// node p e + k (owned local index k < p of element e) couples only to the
// nodes of elements e - 1, e, e + 1.  A DFT over the element index turns them
// into p x p Hermitian blocks per frequency f,
//   K^(f) = B0 + B+ w^f + B- w^-f,   w = exp(2 pi i / n),
// and the 3-D operator K = K1 (x) M1 (x) M1 + ... into independent p^3 x p^3
// blocks per frequency triple.  With the generalized eigenvectors of each
// 1-D block, K^(f) W_f = M^(f) W_f diag(lam_f), W_f^H M^(f) W_f = I, the block
// solve is  x^ = (W (x) W (x) W) diag(1 / (lam_x + lam_y + lam_z)) (W (x) W (x) W)^H b^
// (the constant mode, all three null modes at f = 0, dropped: int phi = 0).
//
// Data path per solve (two real systems as the real and imaginary parts of
// one complex system: the operator is real): an FFT along x that reads the
// mesh vectors and writes element-major complex channels [E][kz][ky][kx], an
// FFT along y, one kernel for the FFT along z, the blocks' solve and the way
// back along z, then y and x, the last into the mesh vectors (real part:
// first system, imaginary part: second).
#include <algorithm>
#include <type_traits>

#include "kernels.hpp"

namespace fep3m {
namespace {

__device__ __forceinline__ double2 zadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 zsub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 zmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// v <- its DFT over R = 1, 2, 4 or 8 values, in natural order; INV: the
// conjugate factors.
template <int R, bool INV>
__device__ __forceinline__ void dft(double2 (&v)[R]) {
  if constexpr (R == 2) {
    const double2 a = v[0];
    v[0] = zadd(a, v[1]);
    v[1] = zsub(a, v[1]);
  } else if constexpr (R > 2) {
    constexpr int H = R / 2;
    constexpr double S = 0.70710678118654752440;
    double2 e[H], o[H];
#pragma unroll
    for (int k = 0; k < H; ++k) {
      e[k] = v[2 * k];
      o[k] = v[2 * k + 1];
    }
    dft<H, INV>(e);
    dft<H, INV>(o);
#pragma unroll
    for (int k = 0; k < H; ++k) {   // o[k] times exp(-+ 2 pi i k / R)
      double2 t = o[k];
      if (4 * k == R) t = INV ? make_double2(-t.y, t.x) : make_double2(t.y, -t.x);
      else if (8 * k == R) t = INV ? make_double2(S * (t.x - t.y), S * (t.x + t.y)) : make_double2(S * (t.x + t.y), S * (t.y - t.x));
      else if (8 * k == 3 * R) t = INV ? make_double2(-S * (t.x + t.y), S * (t.x - t.y)) : make_double2(S * (t.y - t.x), -S * (t.x + t.y));
      v[k] = zadd(e[k], t);
      v[k + H] = zsub(e[k], t);
    }
  }
}

// The z direction of the solve: for each (fx, fy) the n p^3 values along z
// stand in LDS while they are transformed (n = A B: z = g + A m to f = k1 +
// B k2, slot k1 A + k2), multiplied by W^H along x, y and z, divided by the
// eigenvalue sums (times scale, the inverse transforms' 1 / n^3), multiplied
// back and transformed back, so that they cross memory once each way.
// W[f][k][i]: component k of mode i of frequency f; lam[f][i].
//
// Bound by float64 arithmetic (the six 1-D products, 9600 complex dots of p
// per 64 x 125 values), LDS and, at one block of 16 waves per compute unit for
// p = 5, n = 64 (128 KB), the latency of each column's loads, which nothing
// overlaps: the next column's values held in registers meanwhile spilled (644 to
// 810 us against 516 at 64^3, p = 5).  A wave takes whole slots, p^2 lines at a time, so the products'
// steps need no block barrier, and W is uniform (x, y) or read by broadcast
// (z).  Separate z passes and a solve of one block per frequency triple took
// 235 + 551 + 223 us at 64^3, p = 5 (three trips through memory); this 516.
template <int PO, int LOGN>
struct ZSolve {
  static constexpr int N = 1 << LOGN, NCH = PO * PO * PO, P2 = PO * PO;
  static constexpr int A = LOGN >= 6 ? 8 : LOGN >= 4 ? 4 : 1, B = N / A;
  static constexpr int NT = A * NCH <= 256 ? 256 : (A * NCH + 63) / 64 * 64;
  static constexpr size_t LDS = (size_t(N) * NCH + N) * sizeof(double2);
  static constexpr bool OK = NT <= 1024 && LDS + 64 <= 160 * 1024;
};

// orders the LDS accesses of one wave's lanes
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef const f64x2 __attribute__((address_space(4))) *CPtr;
typedef const f64x2 __attribute__((address_space(1))) *GPtr;

// v <- conj(W)^T v (TRANS, into modes) or W v for one line of PO values.  The
// pointer is made opaque at each row, so that one row of W is held at a time
// (in scalar registers where it is uniform): all 25 at once spilled.
template <int PO, bool TRANS, class Ptr>
__device__ __forceinline__ void mode_line(Ptr w, double2 (&v)[PO]) {
  double2 r[PO];
#pragma unroll
  for (int i = 0; i < PO; ++i) r[i] = make_double2(0.0, 0.0);
#pragma unroll
  for (int k = 0; k < PO; ++k) {
    double &last = TRANS ? r[PO - 1].y : r[k > 0 ? k - 1 : 0].y;   // of the row before
    if constexpr (std::is_same_v<Ptr, CPtr>) asm volatile("" : "+s"(w), "+v"(last));
    else asm volatile("" : "+v"(w), "+v"(last));
#pragma unroll
    for (int i = 0; i < PO; ++i) {
      const f64x2 a = w[k * PO + i];
      if (TRANS) {   // out i += conj(W[k][i]) in k
        r[i].x = fma(a.y, v[k].y, fma(a.x, v[k].x, r[i].x));
        r[i].y = fma(-a.y, v[k].x, fma(a.x, v[k].y, r[i].y));
      } else {       // out k += W[k][i] in i
        r[k].x = fma(-a.y, v[i].y, fma(a.x, v[i].x, r[k].x));
        r[k].y = fma(a.y, v[i].x, fma(a.x, v[i].y, r[k].y));
      }
    }
  }
#pragma unroll
  for (int i = 0; i < PO; ++i) v[i] = r[i];
}

template <int PO, int LOGN>
__global__ __launch_bounds__((ZSolve<PO, LOGN>::NT), 4) void k_fs_zsolve(int items, const double2 *__restrict__ W,
                                                                      const double *__restrict__ lam,
                                                                      const double2 *__restrict__ tw, double2 *Z,
                                                                      double scale) {
  using C = ZSolve<PO, LOGN>;
  constexpr int N = C::N, NCH = C::NCH, P2 = C::P2, A = C::A, B = C::B, NT = C::NT;
  constexpr int SPW = 64 / P2;   // slots a wave takes at a time
  extern __shared__ double2 zlds[];
  double2 *buf = zlds, *tws = zlds + N * NCH;
  constexpr size_t SZ = size_t(N) * N * NCH;
  // opaque, so that what follows from it is formed where it is needed and not
  // kept in registers over the whole loop (28 spilled)
  auto fresh = [](int v) {
    asm volatile("" : "+v"(v));
    return v;
  };
  auto base = [](int it) { return size_t(it / (N * N)) * N * SZ + size_t(it % (N * N)) * NCH; };
  if (threadIdx.x < N) tws[threadIdx.x] = tw[threadIdx.x];
#pragma unroll 1
  for (int it = blockIdx.x; it < items; it += gridDim.x) {
    __syncthreads();   // the slots of the item before are read
    int tid = fresh(threadIdx.x);
    if (tid < A * NCH) {   // thread (g, c)
      const int g1 = tid / NCH, c1 = tid - g1 * NCH;
      const double2 *src = Z + base(it) + (unsigned(g1) * unsigned(SZ) + c1);
      double2 v[B];
#pragma unroll
      for (int k = 0; k < B; ++k) v[k] = src[size_t(A * k) * SZ];
      dft<B, false>(v);
#pragma unroll
      for (int k = 0; k < B; ++k) buf[(k * A + g1) * NCH + c1] = A == 1 ? v[k] : zmul(v[k], tws[g1 * k]);
    }
    __syncthreads();
    if constexpr (A > 1) {
#pragma unroll 1
      for (int t = fresh(threadIdx.x); t < B * NCH; t += NT) {
        const int k1 = t / NCH;
        double2 *s = buf + k1 * A * NCH + (t - k1 * NCH);
        double2 v[A];
#pragma unroll
        for (int g = 0; g < A; ++g) v[g] = s[g * NCH];
        dft<A, false>(v);
#pragma unroll
        for (int g = 0; g < A; ++g) s[g * NCH] = v[g];
      }
      __syncthreads();
    }
    {
      const int fx = it % N, fy = it / N % N;
      const CPtr wx = (CPtr)(W + fx * P2), wy = (CPtr)(W + fy * P2);
      tid = fresh(threadIdx.x);
      const int lane = tid & 63, wave = tid >> 6;
      const int sl = lane / P2, ln = lane - sl * P2, la = ln % PO, lb = ln / PO;
#pragma unroll 1
      for (int s0 = wave * SPW; s0 < N; s0 += NT / 64 * SPW) {   // the same trip count for a wave's lanes
        const int slot = s0 + sl;
        const bool on = sl < SPW && slot < N;
        double2 *q = buf + (on ? slot : 0) * NCH;
        const int fz = A == 1 ? slot : slot / A + B * (slot % A);
        double2 v[PO];
        // lines along x: (ky, kz) = (la, lb); y: (kx, kz); z: (kx, ky)
        auto load = [&](int o, int stride) {
#pragma unroll
          for (int k = 0; k < PO; ++k) v[k] = q[o + k * stride];
        };
        auto store = [&](int o, int stride) {
          if (on) {
#pragma unroll
            for (int k = 0; k < PO; ++k) q[o + k * stride] = v[k];
          }
          wave_sync();
        };
        load(on ? ln * PO : 0, 1);
        mode_line<PO, true>(wx, v);
        store(ln * PO, 1);
        load(on ? lb * P2 + la : 0, PO);
        mode_line<PO, true>(wy, v);
        store(lb * P2 + la, PO);
        load(on ? ln : 0, P2);
        {
          const GPtr wz = (GPtr)(W + (on ? fz : 0) * P2);
          mode_line<PO, true>(wz, v);
          const double lxy = lam[fx * PO + la % PO] + lam[fy * PO + (lb < PO ? lb : 0)];
#pragma unroll
          for (int k = 0; k < PO; ++k) {
            const double den = lxy + lam[(on ? fz : 0) * PO + k];
            const double r = den == 0.0 ? 0.0 : scale / den;
            v[k].x *= r;
            v[k].y *= r;
            if (k + 1 < PO) asm volatile("" : "+v"(v[k].x), "+v"(v[k + 1].x));   // one division at a time
          }
          mode_line<PO, false>(wz, v);
        }
        store(ln, P2);
        load(on ? lb * P2 + la : 0, PO);
        mode_line<PO, false>(wy, v);
        store(lb * P2 + la, PO);
        load(on ? ln * PO : 0, 1);
        mode_line<PO, false>(wx, v);
        store(ln * PO, 1);
      }
    }
    __syncthreads();
    if constexpr (A > 1) {
#pragma unroll 1
      for (int t = fresh(threadIdx.x); t < B * NCH; t += NT) {
        const int k1 = t / NCH;
        double2 *s = buf + k1 * A * NCH + (t - k1 * NCH);
        double2 v[A];
#pragma unroll
        for (int g = 0; g < A; ++g) v[g] = s[g * NCH];
        dft<A, true>(v);
#pragma unroll
        for (int g = 0; g < A; ++g) {
          const double2 w = tws[g * k1];
          s[g * NCH] = zmul(v[g], make_double2(w.x, -w.y));
        }
      }
      __syncthreads();
    }
    tid = fresh(threadIdx.x);
    if (tid < A * NCH) {
      const int g1 = tid / NCH, c1 = tid - g1 * NCH;
      double2 v[B];
#pragma unroll
      for (int k = 0; k < B; ++k) v[k] = buf[(k * A + g1) * NCH + c1];
      dft<B, true>(v);
      double2 *dst = Z + base(it) + (unsigned(g1) * unsigned(SZ) + c1);
#pragma unroll
      for (int k = 0; k < B; ++k) dst[size_t(A * k) * SZ] = v[k];
    }
  }
}

template <int PO, int LOGN>
void zsolve(hipStream_t s, int ncs, const double2 *W, const double *lam, const double2 *tw, double2 *Z, double scale) {
  using C = ZSolve<PO, LOGN>;
  const int items = ncs << (2 * LOGN);
  // as many blocks as stay resident (LDS; waves of at most 128 registers)
  const int per_cu = int(std::min<size_t>(160 * 1024 / (C::LDS + 64), size_t(std::max(1, 1024 / C::NT))));
  hipLaunchKernelGGL((k_fs_zsolve<PO, LOGN>), dim3(std::min(items, 256 * per_cu)), dim3(C::NT), C::LDS, s, items, W, lam,
                     tw, Z, scale);
}

// The same products alone, where the z direction does not fit LDS (p = 6, n =
// 64).  One frequency triple per block: the p^3 values of complex system cs at
// (fx, fy, fz), transformed by W^H along x, y, z, divided by the eigenvalue
// sums (times `scale`, the inverse transform's 1 / n^3), transformed back.
// W[f][k][i]: component k of mode i of frequency f; lam[f][i].
template <int PO>
__global__ __launch_bounds__(256) void k_fs_solve(int n, const double2 *__restrict__ W, const double *__restrict__ lam,
                                                  double2 *__restrict__ Z, double scale) {
  constexpr int NCH = PO * PO * PO, P2 = PO * PO;
  __shared__ double2 buf[2][NCH];
  __shared__ double2 w[3][P2];
  __shared__ double l[3][PO];
  const size_t M = size_t(n) * n * n;
  const size_t f = blockIdx.x % M, cs = blockIdx.x / M;
  const int fx = int(f % n), fy = int((f / n) % n), fz = int(f / (size_t(n) * n));
  const int tid = threadIdx.x;
  const int fa[3] = {fx, fy, fz};
  for (int i = tid; i < 3 * P2; i += blockDim.x) w[i / P2][i % P2] = W[size_t(fa[i / P2]) * P2 + i % P2];
  for (int i = tid; i < 3 * PO; i += blockDim.x) l[i / PO][i % PO] = lam[size_t(fa[i / PO]) * PO + i % PO];
  double2 *zf = Z + (cs * M + f) * NCH;
  const bool act = tid < NCH;
  const int kx = tid % PO, ky = (tid / PO) % PO, kz = tid / P2;
  if (act) buf[0][tid] = zf[tid];
  __syncthreads();
  // y = (W^H)_z (W^H)_y (W^H)_x b: out index i along the axis takes
  // sum_k conj(W[k][i]) in[k]
  int cur = 0;
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
    if (act) {
      const int i = ax == 0 ? kx : (ax == 1 ? ky : kz);
      const int stride = ax == 0 ? 1 : (ax == 1 ? PO : P2);
      const int base = tid - i * stride;
      double2 s = make_double2(0.0, 0.0);
#pragma unroll
      for (int k = 0; k < PO; ++k) {
        const double2 a = w[ax][k * PO + i], b = buf[cur][base + k * stride];
        s.x += a.x * b.x + a.y * b.y;
        s.y += a.x * b.y - a.y * b.x;
      }
      buf[cur ^ 1][tid] = s;
    }
    cur ^= 1;
    __syncthreads();
  }
  if (act) {
    const double den = l[0][kx] + l[1][ky] + l[2][kz];
    const double r = den == 0.0 ? 0.0 : scale / den;
    buf[cur][tid].x *= r;
    buf[cur][tid].y *= r;
  }
  __syncthreads();
  // x = W_x W_y W_z y: out index k along the axis takes sum_i W[k][i] in[i]
#pragma unroll
  for (int ax = 0; ax < 3; ++ax) {
    if (act) {
      const int k = ax == 0 ? kx : (ax == 1 ? ky : kz);
      const int stride = ax == 0 ? 1 : (ax == 1 ? PO : P2);
      const int base = tid - k * stride;
      double2 s = make_double2(0.0, 0.0);
#pragma unroll
      for (int i = 0; i < PO; ++i) {
        const double2 a = w[ax][k * PO + i], b = buf[cur][base + i * stride];
        s.x += a.x * b.x - a.y * b.y;
        s.y += a.x * b.y + a.y * b.x;
      }
      buf[cur ^ 1][tid] = s;
    }
    cur ^= 1;
    __syncthreads();
  }
  if (act) zf[tid] = buf[cur][tid];
}

// Dense transform along one axis of nsys P^3 arrays [z][y][x]:
// out[line][o] = sum_k A(o, k) in[line][k], A(o, k) = V[k + o P] (TRANS:
// V^T, the forward transform into modes) or V[o + k P] (back), V the
// column-major eigenvector matrix.  A block covers 64 outputs x 64 lines,
// k in chunks of KC staged in LDS, the next chunk's operands fetched into
// registers while the current one is multiplied; each of the four waves
// owns 32 x 32 of the block as 2 x 2 float64 matrix-core tiles (16 x 16 x 4
// steps: lane l supplies row l % 16, k l / 16 of the left operand and
// k l / 16, column l % 16 of the right one; accumulator value v of lane l is
// row l / 16 + 4 v, column l % 16).  LR: the tile rows are lines and the
// columns outputs (along x, where outputs are contiguous, so a store covers
// 16 consecutive outputs); otherwise rows are outputs and columns lines
// (along y and z, where consecutive lines are consecutive x).  Line
// addresses are formed once per block (no division in the k loop).  The
// steps accumulate in k order like fused multiply-adds, so every output
// equals a sequential loop over k.
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <bool TRANS, bool LR>
__global__ __launch_bounds__(256) void k_axis_transform(int P, int axis, int nsys, const double *__restrict__ V,
                                                        const double *__restrict__ in, double *__restrict__ out) {
  constexpr int KC = 16, NR = KC * 64 / 256;   // operands per thread and chunk, for each matrix
  __shared__ double As[KC][65];   // [k][o]
  __shared__ double Xs[KC][65];   // [k][line]
  const size_t P2 = size_t(P) * P, per = P2 * P;
  const int otiles = (P + 63) / 64;
  const size_t lines = P2 * nsys;
  const size_t ltile = blockIdx.x / otiles;
  const int o0 = (blockIdx.x % otiles) * 64;
  const size_t l0 = ltile * 64;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int r16 = lane & 15, kq = lane >> 4;
  const int wo = (w & 1) * 32, wl = (w >> 1) * 32;
  const size_t kstride = axis == 0 ? 1 : (axis == 1 ? size_t(P) : P2);
  // address of element 0 of line l = (system, a, b), a, b the other two axes
  auto line_base = [&](size_t l) -> size_t {
    const size_t sys = l / P2, r = l % P2;
    if (axis == 0) return sys * per + r * P;
    if (axis == 1) return sys * per + (r / P) * P2 + (r % P);
    return sys * per + r;
  };
  // this thread's staging slots: (k in chunk, line or output) and the line
  // or matrix addresses at k = 0
  int xk[NR], ak[NR], ao[NR];
  size_t xb[NR];
  bool xok[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const int i = tid + 256 * r;
    int kk, ll;
    if (axis == 0) { kk = i % KC; ll = i / KC; } else { ll = i % 64; kk = i / 64; }
    xk[r] = kk;
    xok[r] = l0 + ll < lines;
    xb[r] = xok[r] ? line_base(l0 + ll) : 0;
    int k2, oo;
    if (TRANS) { k2 = i % KC; oo = i / KC; } else { oo = i % 64; k2 = i / 64; }
    ak[r] = k2;
    ao[r] = o0 + oo;
  }
  double xv[NR], av[NR];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int k = k0 + xk[r];
      xv[r] = (k < P && xok[r]) ? in[xb[r] + size_t(k) * kstride] : 0.0;
      const int ka = k0 + ak[r], o = ao[r];
      av[r] = (ka < P && o < P) ? (TRANS ? V[ka + size_t(o) * P] : V[o + size_t(ka) * P]) : 0.0;
    }
  };
  f64x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f64x4{0.0, 0.0, 0.0, 0.0};
  fetch(0);
  for (int k0 = 0; k0 < P; k0 += KC) {
    __syncthreads();   // the previous chunk is consumed
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const int i = tid + 256 * r;
      if (axis == 0) Xs[i % KC][i / KC] = xv[r]; else Xs[i / 64][i % 64] = xv[r];
      if (TRANS) As[i % KC][i / KC] = av[r]; else As[i / 64][i % 64] = av[r];
    }
    __syncthreads();
    if (k0 + KC < P) fetch(k0 + KC);
#pragma unroll
    for (int ks = 0; ks < KC; ks += 4) {
      double xa[2], ob[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) xa[i] = Xs[ks + kq][wl + 16 * i + r16];
#pragma unroll
      for (int j = 0; j < 2; ++j) ob[j] = As[ks + kq][wo + 16 * j + r16];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = LR ? __builtin_amdgcn_mfma_f64_16x16x4f64(xa[i], ob[j], acc[i][j], 0, 0, 0)
                         : __builtin_amdgcn_mfma_f64_16x16x4f64(ob[j], xa[i], acc[i][j], 0, 0, 0);
    }
  }
  if (LR) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const size_t l = l0 + wl + 16 * i + kq + 4 * v;
        if (l >= lines) continue;
        const size_t b = line_base(l);
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int o = o0 + wo + 16 * j + r16;
          if (o < P) out[b + size_t(o) * kstride] = acc[i][j][v];
        }
      }
  } else {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const size_t l = l0 + wl + 16 * i + r16;
      if (l >= lines) continue;
      const size_t b = line_base(l);
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int o = o0 + wo + 16 * j + kq + 4 * v;
          if (o < P) out[b + size_t(o) * kstride] = acc[i][j][v];
        }
    }
  }
}

// The transforms of a box's axes, whose modes are even or odd under reversal.
// With s_i = x_i + x_(P-1-i) and d_i = x_i - x_(P-1-i) (i < H = (P + 1) / 2;
// the middle node's s is x itself, its d zero) the even modes need s alone and
// the odd ones d, and backwards x_i and x_(P-1-i) are the sum and difference
// of an even and an odd part: two products of half the size.
//
// A block of NW waves takes 16 lines: their halves stand in LDS, each wave
// multiplies 16 x 16 tiles of both parts by float64 matrix-core steps (layout
// as in k_axis_transform above), the matrices packed in the order the lanes read them,
// [part][tile][step][lane].  Bound by memory and latency (16 us of copying and
// 8 of products at P = 159, one array): 49 us per transform with the full
// matrix in 64 x 64 tiles, 33 so (the division by eigenvalues included).  Along x the tile's rows are lines, so that
// 16 consecutive outputs are stored together; else its columns.
struct ParityShape {
  int H, T, KS;   // half size, tiles of 16 outputs, steps of 4
  __host__ __device__ explicit ParityShape(int P) : H((P + 1) / 2), T((H + 15) / 16), KS((H + 3) / 4) {}
  __host__ __device__ size_t part() const { return size_t(T) * KS * 64; }
};
constexpr int kLineStride = 17;   // of the 16 lines' values in LDS: stores along x then hit all banks

template <bool TO_MODES, bool AXIS0>
__global__ __launch_bounds__(512) void k_parity_transform(int P, int axis, int nsys, const double *__restrict__ G,
                                                          const double *__restrict__ lam, int i0,
                                                          const double *__restrict__ in, double *__restrict__ out) {
  extern __shared__ double plds[];
  const ParityShape sh(P);
  const int H = sh.H, H4 = 4 * sh.KS;
  double *Xe = plds, *Xo = plds + H4 * kLineStride;
  const size_t P2 = size_t(P) * P, per = P2 * P, lines = P2 * nsys, l0 = size_t(blockIdx.x) * 16;
  const int tid = threadIdx.x, nt = blockDim.x, lane = tid & 63, r16 = lane & 15, kq = lane >> 4;
  const size_t kst = AXIS0 ? 1 : (axis == 1 ? size_t(P) : P2);
  auto line_base = [&](size_t l) -> size_t {   // address of element 0 of line l
    const size_t sys = l / P2;
    const int r = int(l - sys * P2);
    if (AXIS0) return sys * per + size_t(r) * P;
    if (axis == 1) return sys * per + size_t(r / P) * P2 + r % P;
    return sys * per + r;
  };
  for (int i = tid; i < 16 * H4; i += nt) {
    const int k = AXIS0 ? i % H4 : i / 16, l = AXIS0 ? i / H4 : i % 16;
    double a = 0.0, b = 0.0;
    if (k < H && l0 + l < lines) {
      const double *x = in + line_base(l0 + l);
      if (TO_MODES) {
        const double u = x[size_t(k) * kst], v = x[size_t(P - 1 - k) * kst];
        const bool mid = 2 * k + 1 == P;
        a = mid ? u : u + v;
        b = mid ? 0.0 : u - v;
      } else {
        a = x[size_t(k) * kst];
        b = H + k < P ? x[size_t(H + k) * kst] : 0.0;
      }
    }
    Xe[k * kLineStride + l] = a;
    Xo[k * kLineStride + l] = b;
  }
  __syncthreads();
  const double *Ge = G + (TO_MODES ? size_t(0) : 2 * sh.part()), *Go = Ge + sh.part();
  for (int t = tid >> 6; t < sh.T; t += nt >> 6) {
    f64x4 ae{0.0, 0.0, 0.0, 0.0}, ao{0.0, 0.0, 0.0, 0.0};
    const double *ge = Ge + size_t(t) * sh.KS * 64 + lane, *go = Go + size_t(t) * sh.KS * 64 + lane;
    const double *xe = Xe + kq * kLineStride + r16, *xo = Xo + kq * kLineStride + r16;
#pragma unroll 5
    for (int ks = 0; ks < sh.KS; ++ks) {
      const double me = ge[ks * 64], mo = go[ks * 64];
      const double ve = xe[4 * ks * kLineStride], vo = xo[4 * ks * kLineStride];
      ae = AXIS0 ? __builtin_amdgcn_mfma_f64_16x16x4f64(ve, me, ae, 0, 0, 0)
                 : __builtin_amdgcn_mfma_f64_16x16x4f64(me, ve, ae, 0, 0, 0);
      ao = AXIS0 ? __builtin_amdgcn_mfma_f64_16x16x4f64(vo, mo, ao, 0, 0, 0)
                 : __builtin_amdgcn_mfma_f64_16x16x4f64(mo, vo, ao, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = kq + 4 * v;   // of the tile
      const int o = 16 * t + (AXIS0 ? r16 : row);
      const size_t l = l0 + (AXIS0 ? row : r16);
      if (o >= H || l >= lines) continue;
      double *y = out + line_base(l);
      double a = ae[v], b = ao[v];
      if (TO_MODES) {
        const bool has = H + o < P;
        if (lam) {
          const int r = int(l % P2), x = r % P, yy = r / P;
          const double lxy = lam[x] + lam[yy];
          a = x == i0 && yy == i0 && o == i0 ? 0.0 : a / (lxy + lam[o]);
          if (has) b = x == i0 && yy == i0 && H + o == i0 ? 0.0 : b / (lxy + lam[H + o]);
        }
        y[size_t(o) * kst] = a;
        if (has) y[size_t(H + o) * kst] = b;
      } else {
        const bool mid = 2 * o + 1 == P;
        y[size_t(o) * kst] = mid ? a : a + b;
        if (!mid) y[size_t(P - 1 - o) * kst] = a - b;
      }
    }
  }
}

template <int PO>
int fs_solve_impl(hipStream_t s, int nsys, int n, const double *rhs, double *out, double2 *Z, const double2 *tw,
                  const double2 *W, const double *lam) {
  const int ncs = (nsys + 1) / 2;
  const size_t M = size_t(n) * n * n;
  const double scale = 1.0 / double(M);
  constexpr int NCH = PO * PO * PO;
  if (launch_fft_nodes_from_mesh(s, nsys, n, PO, rhs, Z, tw) != 0) return -1;
  if (launch_fft_nodes(s, ncs, n, NCH, 1, Z, tw, false) != 0) return -1;
  bool done = true;
  switch (n) {
    case 8: zsolve<PO, 3>(s, ncs, W, lam, tw, Z, scale); break;
    case 16: zsolve<PO, 4>(s, ncs, W, lam, tw, Z, scale); break;
    case 32: zsolve<PO, 5>(s, ncs, W, lam, tw, Z, scale); break;
    default:
      if constexpr (ZSolve<PO, 6>::OK) zsolve<PO, 6>(s, ncs, W, lam, tw, Z, scale);
      else done = false;
  }
  if (!done) {
    launch_fft_nodes(s, ncs, n, NCH, 2, Z, tw, false);
    hipLaunchKernelGGL(k_fs_solve<PO>, dim3(unsigned(M * ncs)), dim3(256), 0, s, n, W, lam, Z, scale);
    launch_fft_nodes(s, ncs, n, NCH, 2, Z, tw, true);
  }
  launch_fft_nodes(s, ncs, n, NCH, 1, Z, tw, true);
  return launch_fft_nodes_to_mesh(s, nsys, n, PO, Z, out, tw);
}

}  // namespace

void launch_axis_transform(hipStream_t s, int P, int axis, int nsys, const double *V, bool to_modes, const double *in,
                           double *out) {
  const size_t lines = size_t(P) * P * nsys;
  const unsigned grid = unsigned(((lines + 63) / 64) * ((P + 63) / 64));
  if (to_modes && axis == 0)
    hipLaunchKernelGGL((k_axis_transform<true, true>), dim3(grid), dim3(256), 0, s, P, axis, nsys, V, in, out);
  else if (to_modes)
    hipLaunchKernelGGL((k_axis_transform<true, false>), dim3(grid), dim3(256), 0, s, P, axis, nsys, V, in, out);
  else if (axis == 0)
    hipLaunchKernelGGL((k_axis_transform<false, true>), dim3(grid), dim3(256), 0, s, P, axis, nsys, V, in, out);
  else
    hipLaunchKernelGGL((k_axis_transform<false, false>), dim3(grid), dim3(256), 0, s, P, axis, nsys, V, in, out);
}

// LDS holds both halves of 16 lines: P up to 1200
bool parity_fits(int P) { return P >= 1 && size_t(4 * ParityShape(P).KS) * 2 * kLineStride * sizeof(double) <= 160 * 1024; }
size_t parity_size(int P) { return 4 * ParityShape(P).part(); }

void parity_pack(int P, const double *V, double *G) {
  const ParityShape sh(P);
  const int H = sh.H;
  for (int dir = 0; dir < 2; ++dir)
    for (int odd = 0; odd < 2; ++odd)
      for (int t = 0; t < sh.T; ++t)
        for (int ks = 0; ks < sh.KS; ++ks)
          for (int l = 0; l < 64; ++l) {
            const int k = 4 * ks + l / 16, o = 16 * t + l % 16;
            const int node = dir ? o : k, mode = (dir ? k : o) + (odd ? H : 0);
            const bool ok = node < H && (dir ? k : o) < (odd ? P - H : H) && !(odd && 2 * node + 1 == P);
            *G++ = ok ? V[node + size_t(mode) * P] : 0.0;
          }
}

void launch_parity_transform(hipStream_t s, int P, int axis, int nsys, const double *G, bool to_modes, const double *lam,
                             int i0, const double *in, double *out) {
  const ParityShape sh(P);
  const unsigned grid = unsigned((size_t(P) * P * nsys + 15) / 16);
  const int rounds = (sh.T + 7) / 8, nw = (sh.T + rounds - 1) / rounds;   // waves, at most eight
  const size_t lds = size_t(4 * sh.KS) * 2 * kLineStride * sizeof(double);
  if (to_modes && axis == 0)
    hipLaunchKernelGGL((k_parity_transform<true, true>), dim3(grid), dim3(64 * nw), lds, s, P, axis, nsys, G, lam, i0, in, out);
  else if (to_modes)
    hipLaunchKernelGGL((k_parity_transform<true, false>), dim3(grid), dim3(64 * nw), lds, s, P, axis, nsys, G, lam, i0, in, out);
  else if (axis == 0)
    hipLaunchKernelGGL((k_parity_transform<false, true>), dim3(grid), dim3(64 * nw), lds, s, P, axis, nsys, G, lam, i0, in, out);
  else
    hipLaunchKernelGGL((k_parity_transform<false, false>), dim3(grid), dim3(64 * nw), lds, s, P, axis, nsys, G, lam, i0, in, out);
}

int launch_fs_solve(hipStream_t s, int nsys, int n, int p, const double *rhs, double *out, double2 *Z,
                    const double2 *tw, const double2 *W, const double *lam) {
  switch (p) {
    case 3: return fs_solve_impl<3>(s, nsys, n, rhs, out, Z, tw, W, lam);
    case 4: return fs_solve_impl<4>(s, nsys, n, rhs, out, Z, tw, W, lam);
    case 5: return fs_solve_impl<5>(s, nsys, n, rhs, out, Z, tw, W, lam);
    case 6: return fs_solve_impl<6>(s, nsys, n, rhs, out, Z, tw, W, lam);
    default: return -1;
  }
}

}  // namespace fep3m
