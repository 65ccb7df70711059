// The matrix-free mesh operator for orders 3 to 6, with the smoothing step,
// the dot product or the restriction that follows it fused in.
//
//   K = K1 (x) M1 (x) M1 + M1 (x) K1 (x) M1 + M1 (x) M1 (x) K1
//
// A block owns TX x TY columns of elements and marches ZE elements along z.
// Per element it forms A = Mz x, B = Kz x on its (x, y) input columns (each
// column needs the element's PO + 1 planes only: the row of the upper vertex
// is carried to the next element in a register), then C1 = My A,
// C2 = Ky A + My B and K x = Kx C1 + Mx C2 in place in LDS.  In the y and x
// passes one lane takes one element of one column or row; the upper vertex
// row goes to the lane of the next element.
//
// What bounds it and what was measured (p = 5, 64^3 elements, two systems,
// 65.5M nodes; a Chebyshev step moves 2.1 GB of vectors, D^-1 K x 1.05 GB):
// the tile form it replaces (2^3 elements, 16^3 inputs per 10^3 nodes, 36
// multiplications per element matrix) issued 205 vector instructions per node
// and took 0.85 and 0.74 ms: bound by issue and LDS, not by memory.  Marching
// re-reads 1.7 instead of 4.1 inputs per node; even-odd element matrices need
// 18 multiplications and 12 coefficients, so the coefficients stay in scalar
// registers (with 36 the compiler moved them through vector lanes and the
// marching form took 0.92 and 0.81 ms); the row strides keep 16 consecutive
// lanes on distinct bank pairs (conflict cycles 6.6e7 to 2.1e7 per launch).
// Now 0.62 and 0.47 ms, 104 vector instructions per node (average over the modes); on 32^3 elements
// 0.085 to 0.058 ms, on 16^3 16.4 to 11.7 us, on 8^3 7.8 to 5.1 us.
// Two blocks of 12 waves per compute unit overlap one block's memory phase
// with the other's passes, which is why the registers are held to 80:
// x on the owned nodes waits in LDS, x_prev is fetched after the x pass.
// Memory alone (the same loads and stores, no passes) takes 0.52 and 0.31 ms.
// Measured and not kept: one block with two LDS buffers and half the
// barriers (0.70 ms), 2 x 2 columns (0.69 ms), 4 x 2 columns (0.66 ms).
#include "kernels.hpp"
#include "march_plan.hpp"
#include "mesh_device.hpp"

namespace fep3m {

// Element matrices of the centrosymmetric, symmetric kind (m[a][b] = m[b][a] =
// m[p - a][p - b], true of the GLL mass and stiffness) in even-odd form: with
// s_j = v_j + v_{p-j}, d_j = v_j - v_{p-j} (j below the middle) the products
// split into E s and O d with symmetric halves, and row k is (E s)_k + (O d)_k,
// row p - k is (E s)_k - (O d)_k.  18 instead of 36 multiplications at p = 5,
// and 12 distinct coefficients per matrix, few enough to stay in scalar registers.
template <class T, int PO>
struct EvenOdd {
  static constexpr int H = (PO + 1) / 2, C = (PO + 1) % 2, NE = H + C;   // pairs, middle node, even unknowns
  T e[NE * (NE + 1) / 2], o[H * (H + 1) / 2];
};
// float32 keeps the whole matrices and one sum per node, own element first,
// then the element below (band_apply): the mixed-precision V-cycle's rounding
// reaches the results (1e-9), so its order of additions is fixed.  Their
// coefficients fit the scalar registers.
template <class T, int PO>
struct MarchOp {
  int n, P;
  EvenOdd<T, PO> m, k;
  T dk[kMaxP], dm[kMaxP];
};
template <int PO>
struct MarchOp<float, PO> {
  int n, P;
  float m[(PO + 1) * (PO + 1)], k[(PO + 1) * (PO + 1)];
  float dk[kMaxP], dm[kMaxP];
};

__host__ __device__ constexpr int sym_at(int i, int j) { return i <= j ? j * (j + 1) / 2 + i : i * (i + 1) / 2 + j; }

template <class T, int PO>
__device__ __forceinline__ void eo_split(const T *v, T (&s)[EvenOdd<T, PO>::NE], T (&d)[EvenOdd<T, PO>::H]) {
  using M = EvenOdd<T, PO>;
#pragma unroll
  for (int j = 0; j < M::H; ++j) {
    s[j] = v[j] + v[PO - j];
    d[j] = v[j] - v[PO - j];
  }
  if (M::C) s[M::NE - 1] = v[M::H];
}
template <class T, int PO, bool ACC>
__device__ __forceinline__ void eo_mul(const EvenOdd<T, PO> &m, const T (&s)[EvenOdd<T, PO>::NE],
                                       const T (&d)[EvenOdd<T, PO>::H], T (&E)[EvenOdd<T, PO>::NE],
                                       T (&O)[EvenOdd<T, PO>::H]) {
  using M = EvenOdd<T, PO>;
#pragma unroll
  for (int k = 0; k < M::NE; ++k) {
    T a = ACC ? E[k] : T(0);
#pragma unroll
    for (int j = 0; j < M::NE; ++j) a = (!ACC && j == 0) ? m.e[sym_at(k, j)] * s[j] : a + m.e[sym_at(k, j)] * s[j];
    E[k] = a;
  }
#pragma unroll
  for (int k = 0; k < M::H; ++k) {
    T a = ACC ? O[k] : T(0);
#pragma unroll
    for (int j = 0; j < M::H; ++j) a = (!ACC && j == 0) ? m.o[sym_at(k, j)] * d[j] : a + m.o[sym_at(k, j)] * d[j];
    O[k] = a;
  }
}
// rows 0 .. PO (or the first NR of them) from the even and odd parts
template <class T, int PO, int NR>
__device__ __forceinline__ void eo_rows(const T (&E)[EvenOdd<T, PO>::NE], const T (&O)[EvenOdd<T, PO>::H], T (&r)[NR]) {
  using M = EvenOdd<T, PO>;
#pragma unroll
  for (int k = 0; k < NR; ++k)
    r[k] = k < M::H ? E[k] + O[k < M::H ? k : 0] : (M::C && k == M::H) ? E[M::NE - 1] : E[PO - k] - O[PO - k < M::H ? PO - k : 0];
}

// Element at a 32-bit byte offset from a block-uniform base: the base stays in
// scalar registers and the offset is the load's only vector operand.
template <class T>
__device__ __forceinline__ T &at(T *base, unsigned bytes) {
  return *reinterpret_cast<T *>(reinterpret_cast<char *>(base) + bytes);
}
template <class T>
__device__ __forceinline__ const T &at(const T *base, unsigned bytes) {
  return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + bytes);
}

// LDS layout of a tile: row stride R and the padding of a plane, and the lane
// order of the y and x tasks.  Chosen by counting bank conflicts over a step
// (16 lanes of 8 bytes per cycle over 16 bank pairs, a model that gives the
// measured conflict cycles to 1 to 5%).
//   YS: the tasks of one y element sit together (else those of one column);
//   XS: the tasks of one x element sit together; XZ: consecutive rows walk z.
template <int PO, int TX, int TY>
struct MarchLayout;
template <> struct MarchLayout<5, 4, 4> { static constexpr int R = 28, PAD = 2; static constexpr bool YS = true, XS = false, XZ = false; };
template <> struct MarchLayout<5, 2, 2> { static constexpr int R = 17, PAD = 0; static constexpr bool YS = true, XS = false, XZ = false; };
template <> struct MarchLayout<4, 4, 4> { static constexpr int R = 23, PAD = 2; static constexpr bool YS = true, XS = true, XZ = false; };
template <> struct MarchLayout<3, 8, 4> { static constexpr int R = 31, PAD = 5; static constexpr bool YS = false, XS = true, XZ = true; };
template <> struct MarchLayout<3, 4, 4> { static constexpr int R = 20, PAD = 0; static constexpr bool YS = true, XS = false, XZ = false; };
template <> struct MarchLayout<6, 2, 2> { static constexpr int R = 19, PAD = 11; static constexpr bool YS = true, XS = true, XZ = false; };

template <int PO, int TX, int TY, int NT>
struct MarchShape : MarchLayout<PO, TX, TY> {
  using L = MarchLayout<PO, TX, TY>;
  static constexpr int OX = TX * PO, OY = TY * PO;            // owned nodes per plane
  static constexpr int IX = OX + PO + 1, IY = OY + PO + 1;    // input columns
  static constexpr int SA = IY * L::R + L::PAD;               // plane stride
  static constexpr int ZW = L::R * IY <= NT ? L::R : IX;      // threads per row of input columns
  static constexpr int OWN = PO * OX * OY;                    // owned nodes per step
  static constexpr int NIT = (OWN + NT - 1) / NT;
  static constexpr int CW = 64 / (TY + 1);                    // y pass: columns per wave
  static constexpr int RW = 64 / (TX + 1);                    // x pass: rows per wave
  static constexpr int NW = NT / 64;
  static constexpr int CX = 3 * TX + 1, CY = 3 * TY + 1;      // coarse (order 3) nodes the tile restricts to
  static_assert(ZW * IY <= NT, "one input column per thread");
  static_assert(CW * NW >= PO * IX && RW * NW >= PO * OY, "one pass of the block's waves");
  static_assert(PO == 3 || (64 % TX == 0 && 64 / TX * NW >= PO * OY && 64 % TY == 0 && 64 / TY * NW >= PO * CX && CX * CY <= NT),
                "one pass of the block's waves in the restriction");
  static_assert(PO == 3 || (PO * OY * CX <= 2 * PO * SA && PO * CX * CY <= OWN),
                "the restriction reuses the tile's arrays");
};

// the value of the lane below (lane 0: its own)
__device__ __forceinline__ double lane_below(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, 0x138, 0xf, 0xf, false),
                          __builtin_amdgcn_update_dpp(lo, lo, 0x138, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_below(float v) {
  const int i = __float_as_int(v);
  return __int_as_float(__builtin_amdgcn_update_dpp(i, i, 0x138, 0xf, 0xf, false));
}

constexpr int kChebFirst = 9;   // kCheb without x_prev

// Restriction to order 3 on the same elements: weight w[s * 4 + j] of fine
// node s of an element on its coarse node j (j = 3: the upper vertex).
template <class T, int PO>
struct MarchRestrict {
  T w[PO * 4];
};
template <class T, int PO>
__device__ __forceinline__ void restrict_element(const MarchRestrict<T, PO> &rw, const T (&v)[PO], T (&o)[4]) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    o[j] = rw.w[j] * v[0];
#pragma unroll
    for (int q = 1; q < PO; ++q) o[j] += rw.w[q * 4 + j] * v[q];
  }
}

// Modes as in ApplyMode.  kResidualRestrict writes, instead of nodes, the
// block's (3 ZE' + 1) CY CX partial coarse values (ZE' <= ZE its elements)
// to out + block * (3 ze + 1) CY CX.
template <class T, int PO, int TX, int TY, int NT, int WPS, int MODE>
__global__ __launch_bounds__(NT, WPS) void k_apply_march(MarchOp<T, PO> op, MarchRestrict<T, PO> rw, int ze,
                                                         const T *__restrict__ x, const T *__restrict__ f,
                                                         const T *xprev, T *out, T c1, T c2, T s0,
                                                         double *__restrict__ partial) {
  using S = MarchShape<PO, TX, TY, NT>;
  using EO = EvenOdd<T, PO>;
  constexpr int IX = S::IX, IY = S::IY, OX = S::OX, OY = S::OY, NIT = S::NIT, Q1 = PO + 1, R = S::R;
  constexpr bool zstart = MODE == kChebZ2, need_d = MODE == kCheb || MODE == kChebDot;
  constexpr bool cheb = need_d || MODE == kChebFirst;
  constexpr bool rr = MODE == kResidualRestrict;
  constexpr bool norm = MODE == kResidualNorm;
  constexpr bool need_f = MODE == kResidual || norm || rr || cheb || zstart || MODE == kChebZ3;
  constexpr bool need_x = cheb || MODE == kChebZ3 || MODE == kApplyDot;
  constexpr bool need_id = MODE != kApplyDot && MODE != kResidual && !norm && !rr;
  __shared__ T AB[2 * PO * S::SA];
  __shared__ T Xo[need_x || rr ? S::OWN : 1];   // x (rr: the residual) on the owned nodes
  __shared__ T invd[PO * PO * PO];
  // dot modes: each thread's sum, kept in LDS between steps
  constexpr bool dot = MODE == kApplyDot || MODE == kChebDot || norm;
  __shared__ double sum[dot ? NT : 1];
  __shared__ double sum2[norm ? NT : 1];
  const int P = op.P, n = op.n;
  const size_t P2 = size_t(P) * P;
  const int ntx = (n + TX - 1) / TX, nty = (n + TY - 1) / TY, nz = (n + ze - 1) / ze;
  const int blk = xcd_linear(blockIdx.x, gridDim.x);
  int b = blk;
  const int bx = b % ntx;
  b /= ntx;
  const int by = b % nty;
  b /= nty;
  const int bz = b % nz;
  const size_t off = size_t(b / nz) * P * P2;
  constexpr bool band = sizeof(T) == 4;
  const T *src = (zstart ? f : x) + off;
  const int tid = threadIdx.x;
  const int ox0 = bx * OX, oy0 = by * OY;
  const int e0 = bz * ze, e1 = min(e0 + ze, n);
  if (need_id) {
    for (int i = tid; i < PO * PO * PO; i += NT) {
      const int kx = i % PO, ky = (i / PO) % PO, kz = i / (PO * PO);
      const T dkx = pick<PO>(op.dk, kx), dky = pick<PO>(op.dk, ky), dkz = pick<PO>(op.dk, kz);
      const T dmx = pick<PO>(op.dm, kx), dmy = pick<PO>(op.dm, ky), dmz = pick<PO>(op.dm, kz);
      invd[i] = T(1) / (dkx * dmy * dmz + dmx * dky * dmz + dmx * dmy * dkz);
    }
    __syncthreads();
  }
  // owned nodes of this thread in every step: offset from the step's first node, LDS index, inverse diagonal
  unsigned eoff[NIT], eidx[NIT];   // eidx: LDS index, and the local node index above it
#pragma unroll
  for (int r = 0; r < NIT; ++r) {
    const int li = tid + NT * r;
    const int lc = li < S::OWN ? li : 0;
    const int ox = lc % OX, oy = (lc / OX) % OY, oz = lc / (OX * OY);
    const bool ok = li < S::OWN && ox0 + ox < P && oy0 + oy < P;
    eoff[r] = ok ? unsigned((oz * P + oy) * P + ox) * unsigned(sizeof(T)) : 0u;
    eidx[r] = unsigned(oz * S::SA + oy * R + ox) | unsigned((ox % PO) + PO * ((oy % PO) + PO * oz)) << 16 |
              (ok ? 0x80000000u : 0u);
  }
  // this thread's input column
  const int lx = tid % S::ZW, ly = tid / S::ZW;
  const bool col = lx < IX && ly < IY;
  const unsigned coff = col ? unsigned(wrapi(oy0 - PO + ly, P) * P + wrapi(ox0 - PO + lx, P)) * unsigned(sizeof(T)) : 0u;
  T *const za = AB + (col ? ly * R + lx : 0);
  const bool own = lx >= PO && lx < PO + OX && ly >= PO && ly < PO + OY;
  T *const xw = Xo + (need_x && own ? (ly - PO) * OX + lx - PO : 0);
  const T *idc = invd + (lx % PO) + PO * (ly % PO);
  // y pass: task (column, y element from one below the tile), x pass: (row, x element likewise)
  const int lane = tid & 63, wave = tid >> 6;
  const int ye = S::YS ? lane / S::CW : lane % (TY + 1), yc = S::YS ? lane % S::CW : lane / (TY + 1);
  const int ycol = wave * S::CW + yc;
  const bool yon = lane < S::CW * (TY + 1) && ycol < PO * IX;
  T *const ya = AB + (yon ? (ycol / IX) * S::SA + ye * PO * R + ycol % IX : 0);
  const int xe = S::XS ? lane / S::RW : lane % (TX + 1), xc = S::XS ? lane % S::RW : lane / (TX + 1);
  const int xrow = wave * S::RW + xc;
  const bool xon = lane < S::RW * (TX + 1) && xrow < PO * OY;
  T *const xa = AB + (xon ? (S::XZ ? (xrow % PO) * S::SA + (xrow / PO) * R : (xrow / OY) * S::SA + (xrow % OY) * R) + xe * PO : 0);
  // planes of the current element (zp: and of the one below), the next one's
  T zin[Q1], nx[PO], zp[band ? PO : 1];
  T cA, cB, cR = T(0);   // carried rows of A, B; restriction: carried upper vertex
  T s[EO::NE], d[EO::H], E[EO::NE], O[EO::H];
  {
    const int zb = PO * (e0 == 0 ? n - 1 : e0 - 1);
#pragma unroll
    for (int j = 0; j < PO; ++j) zin[j] = at(src + size_t(zb + j) * P2, coff);
    zin[PO] = at(src + size_t(PO * e0) * P2, coff);
#pragma unroll
    for (int j = 0; j < PO; ++j) nx[j] = at(src + size_t(wrapi(PO * e0 + 1 + j, P)) * P2, coff);
    if (zstart) {
#pragma unroll
      for (int j = 0; j <= PO; ++j) zin[j] *= s0 * idc[PO * PO * (j % PO)];
    }
    if constexpr (!band) {
      eo_split<T, PO>(zin, s, d);
      eo_mul<T, PO, false>(op.m, s, d, E, O);
      cA = E[0] - O[0];
      eo_mul<T, PO, false>(op.k, s, d, E, O);
      cB = E[0] - O[0];
    }
  }
  if (dot) sum[tid] = 0.0;
  if (norm) sum2[tid] = 0.0;
  // pass z of element e: its rows from the PO + 1 input planes; the upper
  // vertex row is carried to the next element
  auto pass_z = [&]() {
    if constexpr (band) {
#pragma unroll
      for (int j = 0; j < PO; ++j) zp[j] = zin[j];
    }
    zin[0] = zin[PO];
#pragma unroll
    for (int j = 0; j < PO; ++j) zin[j + 1] = zstart ? nx[j] * (s0 * idc[PO * PO * ((j + 1) % PO)]) : nx[j];
    if (need_x && own) {
#pragma unroll
      for (int k = 0; k < PO; ++k) xw[k * OX * OY] = zin[k];
    }
    if constexpr (band) {
      T v[2 * PO + 1], r[PO];
#pragma unroll
      for (int j = 0; j < PO; ++j) v[j] = zp[j];
#pragma unroll
      for (int j = 0; j <= PO; ++j) v[PO + j] = zin[j];
      band_apply<PO, PO>(op.m, v, r);
      if (col) {
#pragma unroll
        for (int k = 0; k < PO; ++k) za[k * S::SA] = r[k];
      }
      band_apply<PO, PO>(op.k, v, r);
      if (col) {
#pragma unroll
        for (int k = 0; k < PO; ++k) za[(PO + k) * S::SA] = r[k];
      }
    } else {
      T r[Q1];
      eo_split<T, PO>(zin, s, d);
      eo_mul<T, PO, false>(op.m, s, d, E, O);
      eo_rows<T, PO, Q1>(E, O, r);
      r[0] += cA;
      cA = r[PO];
      if (col) {
#pragma unroll
        for (int k = 0; k < PO; ++k) za[k * S::SA] = r[k];
      }
      eo_mul<T, PO, false>(op.k, s, d, E, O);
      eo_rows<T, PO, Q1>(E, O, r);
      r[0] += cB;
      cB = r[PO];
      if (col) {
#pragma unroll
        for (int k = 0; k < PO; ++k) za[(PO + k) * S::SA] = r[k];
      }
    }
  };
  auto load_z = [&](int e) {
#pragma unroll
    for (int j = 0; j < PO; ++j) nx[j] = at(src + size_t(wrapi(PO * e + 1 + j, P)) * P2, coff);
  };
  for (int e = e0; e < e1; ++e) {
    pass_z();
    __syncthreads();
    // pass y, in place: an element's upper vertex row goes to the lane of the
    // next element of its column
    if constexpr (band) {
      T v[2 * PO + 1], r1[PO], r2[PO];
      const T *q = ye > 0 ? ya - PO * R : ya;   // from the element below
#pragma unroll
      for (int j = 0; j <= 2 * PO; ++j) v[j] = q[j * R];
      band_apply<PO, PO>(op.m, v, r1);
      band_apply<PO, PO>(op.k, v, r2);
#pragma unroll
      for (int j = 0; j <= 2 * PO; ++j) v[j] = q[PO * S::SA + j * R];
      band_apply_acc<PO, PO>(op.m, v, r2);
      asm volatile("" ::: "memory");   // the wave's reads precede its writes
      __builtin_amdgcn_wave_barrier();
      if (yon && ye > 0) {
#pragma unroll
        for (int k = 0; k < PO; ++k) {
          ya[(k - PO) * R] = r1[k];
          ya[PO * S::SA + (k - PO) * R] = r2[k];
        }
      }
    } else {
      T v[Q1], r1[Q1], r2[Q1];
#pragma unroll
      for (int j = 0; j <= PO; ++j) v[j] = ya[j * R];
      eo_split<T, PO>(v, s, d);
      eo_mul<T, PO, false>(op.m, s, d, E, O);
      eo_rows<T, PO, Q1>(E, O, r1);
      eo_mul<T, PO, false>(op.k, s, d, E, O);
#pragma unroll
      for (int j = 0; j <= PO; ++j) v[j] = ya[PO * S::SA + j * R];
      eo_split<T, PO>(v, s, d);
      eo_mul<T, PO, true>(op.m, s, d, E, O);
      eo_rows<T, PO, Q1>(E, O, r2);
      r1[0] += S::YS ? __shfl_up(r1[PO], S::CW) : lane_below(r1[PO]);
      r2[0] += S::YS ? __shfl_up(r2[PO], S::CW) : lane_below(r2[PO]);
      asm volatile("" ::: "memory");   // the wave's reads precede its writes
      __builtin_amdgcn_wave_barrier();
      if (yon && ye > 0) {
#pragma unroll
        for (int k = 0; k < PO; ++k) {
          ya[(k - PO) * R] = r1[k];
          ya[PO * S::SA + (k - PO) * R] = r2[k];
        }
      }
    }
    // epilogue operands, in flight behind the x pass
    const size_t tb = off + (size_t(PO * e) * P + oy0) * P + ox0;
    T pf_f[NIT], pf_d[NIT];
#pragma unroll
    for (int r = 0; r < NIT; ++r) {
      pf_f[r] = need_f ? at(f + tb, eoff[r]) : T(0);
    }
    __syncthreads();
    // pass x, in place likewise
    if constexpr (band) {
      T v[2 * PO + 1], r[PO];
      const T *q = xe > 0 ? xa - PO : xa;
#pragma unroll
      for (int j = 0; j <= 2 * PO; ++j) v[j] = q[j];
      band_apply<PO, PO>(op.k, v, r);
#pragma unroll
      for (int j = 0; j <= 2 * PO; ++j) v[j] = q[PO * S::SA + j];
      band_apply_acc<PO, PO>(op.m, v, r);
      asm volatile("" ::: "memory");
      __builtin_amdgcn_wave_barrier();
      if (xon && xe > 0) {
#pragma unroll
        for (int k = 0; k < PO; ++k) xa[k - PO] = r[k];
      }
    } else {
      T v[Q1], r[Q1];
#pragma unroll
      for (int j = 0; j <= PO; ++j) v[j] = xa[j];
      eo_split<T, PO>(v, s, d);
      eo_mul<T, PO, false>(op.k, s, d, E, O);
#pragma unroll
      for (int j = 0; j <= PO; ++j) v[j] = xa[PO * S::SA + j];
      eo_split<T, PO>(v, s, d);
      eo_mul<T, PO, true>(op.m, s, d, E, O);
      eo_rows<T, PO, Q1>(E, O, r);
      r[0] += S::XS ? __shfl_up(r[PO], S::RW) : lane_below(r[PO]);
      asm volatile("" ::: "memory");
      __builtin_amdgcn_wave_barrier();
      if (xon && xe > 0) {
#pragma unroll
        for (int k = 0; k < PO; ++k) xa[k - PO] = r[k];
      }
    }
#pragma unroll
    for (int r = 0; r < NIT; ++r) pf_d[r] = need_d ? at(xprev + tb, eoff[r]) : T(0);
    __syncthreads();
    if (e + 1 < e1) load_z(e + 1);
    if constexpr (rr) {
#pragma unroll
      for (int r = 0; r < NIT; ++r) {
        const int li = tid + NT * r;
        if (li < S::OWN) Xo[li] = int(eidx[r]) < 0 ? pf_f[r] - AB[eidx[r] & 0xffff] : T(0);
      }
      __syncthreads();
      constexpr int CX = S::CX, CY = S::CY;
      T v[PO], o[4];
      {   // x: (row, element) to R1 [z][y][CX] in AB
        const int row = wave * (64 / TX) + lane / TX, ex = lane % TX;
        const bool on = row < PO * OY;
        const T *q = Xo + (on ? row * OX + ex * PO : 0);
#pragma unroll
        for (int j = 0; j < PO; ++j) v[j] = q[j];
        restrict_element<T, PO>(rw, v, o);
        const T c = lane_below(o[3]);
        if (ex > 0) o[0] += c;
        T *w = AB + row * CX + 3 * ex;
        if (on) {
#pragma unroll
          for (int j = 0; j < 3; ++j) w[j] = o[j];
          if (ex == TX - 1) w[3] = o[3];
        }
      }
      __syncthreads();
      {   // y: (z, CX, element) to R2 [z][CY][CX] in Xo
        const int c0 = wave * (64 / TY) + lane / TY, ey = lane % TY;
        const bool on = c0 < PO * CX;
        const int z = on ? c0 / CX : 0, cx = on ? c0 % CX : 0;
        const T *q = AB + (z * OY + ey * PO) * CX + cx;
#pragma unroll
        for (int j = 0; j < PO; ++j) v[j] = q[j * CX];
        restrict_element<T, PO>(rw, v, o);
        const T c = lane_below(o[3]);
        if (ey > 0) o[0] += c;
        T *w = Xo + (z * CY + 3 * ey) * CX + cx;
        if (on) {
#pragma unroll
          for (int j = 0; j < 3; ++j) w[j * CX] = o[j];
          if (ey == TY - 1) w[3 * CX] = o[3];
        }
      }
      __syncthreads();
      if (tid < CX * CY) {   // z: this element's three planes, its upper vertex carried on
#pragma unroll
        for (int j = 0; j < PO; ++j) v[j] = Xo[j * CX * CY + tid];
        restrict_element<T, PO>(rw, v, o);
        T *w = out + (size_t(blk) * (3 * ze + 1) + 3 * (e - e0)) * (CX * CY) + tid;
        w[0] = o[0] + cR;
        w[CX * CY] = o[1];
        w[2 * CX * CY] = o[2];
        cR = o[3];
        if (e + 1 == e1) w[3 * CX * CY] = cR;
      }
      // no barrier: the next z pass writes AB, last read before the barrier above, and
      // the residual's next write to Xo is three barriers away
      continue;
    }
    T res[NIT];
    double acc = dot ? sum[tid] : 0.0, acc2 = norm ? sum2[tid] : 0.0;
#pragma unroll
    for (int r = 0; r < NIT; ++r) {
      const T y = AB[eidx[r] & 0xffff], id = need_id ? invd[(eidx[r] >> 16) & 0x7fff] : T(0);
      T xv = zstart ? pf_f[r] * (s0 * id) : need_x ? Xo[min(tid + NT * r, S::OWN - 1)] : T(0);
      if (band && zstart) asm volatile("" : "+v"(xv));   // rounded here, as the z pass's input was
      const T rr = (pf_f[r] - y) * id;
      T v;
      if (MODE == kApplyDot) v = y;
      else if (MODE == kResidual || norm) v = pf_f[r] - y;
      else if (need_d) v = xv + c1 * (xv - pf_d[r]) + c2 * rr;
      else if (cheb || zstart) v = xv + c1 * xv + c2 * rr;
      else if (MODE == kChebZ3) v = xv + c1 * (xv - s0 * id * pf_f[r]) + c2 * rr;
      else v = -rr;
      if (MODE == kApplyDot && int(eidx[r]) < 0) acc += double(xv) * double(y);
      if (MODE == kChebDot && int(eidx[r]) < 0) acc += double(v) * double(pf_f[r]);
      if (norm && int(eidx[r]) < 0) {
        acc += double(v) * double(v);
        acc2 += double(pf_f[r]) * double(pf_f[r]);
      }
      res[r] = v;
    }
    if (dot) sum[tid] = acc;
    if (norm) sum2[tid] = acc2;
    if (!norm) {
      T *const dst = out + tb;
#pragma unroll
      for (int r = 0; r < NIT; ++r)
        if (int(eidx[r]) < 0) at(dst, eoff[r]) = res[r];
    }
    __syncthreads();   // the next z pass overwrites what the epilogue read
  }
  if (dot) {
    double t = sum[tid];
    __syncthreads();
    t = block_sum_waves(t, sum);
    if (tid == 0) partial[blk] = t;   // blk is system-major
    if (norm) {
      __syncthreads();
      double t2 = sum2[tid];
      __syncthreads();
      t2 = block_sum_waves(t2, sum2);
      if (tid == 0) out[blk] = T(t2);
    }
  }
}

template <class T, int PO>
static MarchOp<T, PO> march_op(const LevelOpT<T> &op) {
  MarchOp<T, PO> o{};
  o.n = op.n;
  o.P = op.P;
  constexpr int Q1 = PO + 1;
  if constexpr (sizeof(T) == 4) {
    for (int i = 0; i < Q1 * Q1; ++i) {
      o.m[i] = op.me[i];
      o.k[i] = op.ke[i];
    }
  } else {
    using M = EvenOdd<T, PO>;
    auto fill = [](const T *a, M &m) {
      for (int k = 0; k < M::NE; ++k)
        for (int j = k; j < M::NE; ++j)
          m.e[sym_at(k, j)] = (j < M::H) ? T(0.5) * (a[k * Q1 + j] + a[k * Q1 + PO - j]) : a[k * Q1 + j];
      for (int k = 0; k < M::H; ++k)
        for (int j = k; j < M::H; ++j) m.o[sym_at(k, j)] = T(0.5) * (a[k * Q1 + j] - a[k * Q1 + PO - j]);
    };
    fill(op.me, o.m);
    fill(op.ke, o.k);
  }
  for (int k = 0; k < kMaxP; ++k) {
    o.dk[k] = op.dk[k];
    o.dm[k] = op.dm[k];
  }
  return o;
}

namespace {

template <class T, int PO, int TX, int TY, int NT, int WPS>
int march_impl(hipStream_t s, int nsys, const MarchPlan &pl, const LevelOpT<T> &op, const TransferT<T> *tr, const T *x,
               const T *f, T *out, const T *d, T *xo, T c1, T c2, int mode, double *partial, T s0) {
  const int K = pl.blocks();
  const MarchOp<T, PO> mo = march_op<T, PO>(op);
  MarchRestrict<T, PO> rw{};
  if (tr)
    for (int i = 0; i < 4 * PO; ++i) rw.w[i] = tr->w[i];
  const bool cheb = mode == kCheb || mode == kChebDot || mode == kChebZ2 || mode == kChebZ3;
  T *const dst = cheb ? xo : out;
  // without x_prev (null, or c1 = 0) the step has its own form; with the dot
  // it reads x in x_prev's place, which c1 = 0 takes out
  if (mode == kCheb && (c1 == T(0) || !d)) {
    mode = kChebFirst;
    c1 = T(0);
  }
  if (mode == kChebDot && (c1 == T(0) || !d)) {
    d = x;
    c1 = T(0);
  }
#define FEP3M_MARCH(M)                                                                                              \
  case M:                                                                                                          \
    hipLaunchKernelGGL((k_apply_march<T, PO, TX, TY, NT, WPS, M>), dim3(nsys * K), dim3(NT), 0, s, mo, rw, pl.ze, x, \
                       f, d, dst, c1, c2, s0, partial);                                                            \
    break
  switch (mode) {
    FEP3M_MARCH(kResidual);
    FEP3M_MARCH(kCheb);
    FEP3M_MARCH(kChebFirst);
    FEP3M_MARCH(kChebZ2);
    FEP3M_MARCH(kChebZ3);
    case kApplyDot:
    case kDinvApply:
    case kChebDot:
    case kResidualNorm:   // the float32 cycle has none of these
      if constexpr (sizeof(T) == 8) {
        switch (mode) {
          FEP3M_MARCH(kApplyDot);
          FEP3M_MARCH(kDinvApply);
          FEP3M_MARCH(kChebDot);
          FEP3M_MARCH(kResidualNorm);
        }
        break;
      } else {
        return -1;
      }
    case kResidualRestrict:
      if constexpr (PO > 3 && sizeof(T) == 8) {
        switch (mode) { FEP3M_MARCH(kResidualRestrict); }
        break;
      } else {
        return -1;
      }
    default: return -1;
  }
#undef FEP3M_MARCH
  return K;
}

template <class T>
int march(hipStream_t s, int nb, int nsys, const LevelOpT<T> &op, const TransferT<T> *tr, const T *x, const T *f, T *out,
          const T *d, T *xo, T c1, T c2, int mode, double *partial, T s0) {
  const bool shared = mode == kApplyDot || mode == kChebDot || mode == kResidualNorm || mode == kResidualRestrict;
  const MarchPlan pl = march_plan(op.p, op.n, nb, nsys, shared);
#define FEP3M_TILE(PO, TX, TY, NT, W) \
  return march_impl<T, PO, TX, TY, NT, W>(s, nsys, pl, op, tr, x, f, out, d, xo, c1, c2, mode, partial, s0)
  switch (op.p * 10 + pl.tx) {
    case 38: FEP3M_TILE(3, 8, 4, 512, 8);
    case 34: FEP3M_TILE(3, 4, 4, 256, 6);
    case 54: FEP3M_TILE(5, 4, 4, 768, 6);
    case 52: FEP3M_TILE(5, 2, 2, 256, 5);
  }
  if constexpr (sizeof(T) == 8) {   // the other orders' screens run in float64
    switch (op.p * 10 + pl.tx) {
      case 44: FEP3M_TILE(4, 4, 4, 512, 6);
      case 62: FEP3M_TILE(6, 2, 2, 384, 4);
    }
  }
  return -1;
#undef FEP3M_TILE
}

// Partial coarse values summed per coarse node (order 3): those of its own
// block and, for a node on the block's lower faces, the upper vertex values
// of the blocks below, in a fixed order.
// One row of coarse nodes per block, so that only x is worked out per node
// (123 us at 64^3, two systems, with all three indices per node; 85 us).
__global__ __launch_bounds__(256) void k_march_restrict_sum(MarchPlan pl, int n, const double *__restrict__ partall,
                                                            double *__restrict__ fcall) {
  const int Pc = 3 * n, gy = blockIdx.x % Pc, gz = blockIdx.x / Pc % Pc, cfg = blockIdx.x / Pc / Pc;
  const int cx = 3 * pl.tx + 1, cy = 3 * pl.ty + 1, cz = 3 * pl.ze + 1;
  const double *part = partall + size_t(cfg) * pl.blocks() * cx * cy * cz;
  double *fc = fcall + ((size_t(cfg) * Pc + gz) * Pc + gy) * Pc;
  // blocks (one or two) that hold coarse node g of an axis and its index in them
  auto owners = [n](int g, int te, int nt, int(&t)[2], int(&k)[2]) {
    const int w = 3 * te;
    t[0] = g / w;
    k[0] = g - t[0] * w;
    if (k[0] != 0) return 1;
    t[1] = t[0] == 0 ? nt - 1 : t[0] - 1;
    k[1] = t[0] == 0 ? 3 * (n - te * (nt - 1)) : w;   // the last block of an axis may hold fewer elements
    return 2;
  };
  int ty[2], ky[2], tz[2], kz[2];
  const int ny = owners(gy, pl.ty, pl.ny, ty, ky), nz = owners(gz, pl.ze, pl.nz, tz, kz);
  for (int gx = threadIdx.x; gx < Pc; gx += blockDim.x) {
    int tx[2], kx[2];
    const int nx = owners(gx, pl.tx, pl.nx, tx, kx);
    double s = 0.0;
    for (int iz = 0; iz < nz; ++iz)
      for (int iy = 0; iy < ny; ++iy) {
        const size_t row = size_t(tz[iz] * pl.ny + ty[iy]) * pl.nx;
        const int at = (kz[iz] * cy + ky[iy]) * cx;
        s += part[(row + tx[0]) * (cx * cy * cz) + at + kx[0]];
        if (nx == 2) s += part[(row + tx[1]) * (cx * cy * cz) + at + kx[1]];
      }
    fc[gx] = s;
  }
}

}  // namespace

int march_blocks(int p, int n, int nb) { return shared_plan(p, n, nb).blocks(); }

size_t march_restrict_size(int p, int n, int nb) {
  const MarchPlan q = shared_plan(p, n, nb);
  return size_t(q.blocks()) * (3 * q.tx + 1) * (3 * q.ty + 1) * (3 * q.ze + 1);
}

template <class T>
int launch_march(hipStream_t s, int nb, int nsys, const LevelOpT<T> &op, const T *x, const T *f, T *out, const T *d,
                 T *xo, T c1, T c2, int mode, double *partial, T s0) {
  return march<T>(s, nb, nsys, op, nullptr, x, f, out, d, xo, c1, c2, mode, partial, s0);
}

int launch_march_restrict(hipStream_t s, int nb, int nsys, const LevelOp &op, const Transfer &tr, const double *x,
                          const double *f, double *part, double *fc) {
  if (tr.pf != op.p || tr.pc != 3 || tr.r != 1 || op.p < 4) return -1;
  const int K = march<double>(s, nb, nsys, op, &tr, x, f, part, nullptr, nullptr, 0.0, 0.0, kResidualRestrict, nullptr,
                              0.0);
  if (K < 0) return K;
  const int Pc = 3 * op.n;
  hipLaunchKernelGGL(k_march_restrict_sum, dim3(unsigned(nsys) * Pc * Pc), dim3(Pc >= 256 ? 256 : 64 * ((Pc + 63) / 64)), 0,
                     s, shared_plan(op.p, op.n, nb), op.n, part, fc);
  return K;
}

#define FEP3M_MARCH_INSTANTIATE(T)                                                                                  \
  template int launch_march<T>(hipStream_t, int, int, const LevelOpT<T> &, const T *, const T *, T *, const T *, T *, T, \
                               T, int, double *, T);
FEP3M_MARCH_INSTANTIATE(double)
FEP3M_MARCH_INSTANTIATE(float)
#undef FEP3M_MARCH_INSTANTIATE

}  // namespace fep3m
