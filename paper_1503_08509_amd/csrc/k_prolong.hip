// Prolongation between the orders of one mesh (5, 4 or 6 from 3, and 3 from
// 1): xf += P ec in three separable passes, the block marching along z over
// columns of TX x TY elements.
//
// Bound by memory: xf once in and once out and the coarse values (16 B per
// fine node and 8 B per coarse one in float64).  The tiles of 3^3 elements it
// replaces passed every stage through LDS (60 KB, two blocks per compute
// unit) with the loads of xf ahead of all passes: 347 us at 64^3, p = 5 from
// 3, two systems (1.16 GB, 3.3 TB/s), 271 us in float32.  Here the x pass is
// formed per fine node from four LDS values as the node is updated, and the
// next element's nodes and coarse planes are in flight meanwhile: 247 and
// 158 us (3 from 1: 72 to 47 us).  Each value is summed over the coarse nodes in the same order as
// before, z then y then x.
#include "kernels.hpp"
#include "mesh_device.hpp"

namespace fep3m {

namespace {

template <class T, int PF, int PC>
struct ProlongW {
  T w[PF * (PC + 1)];   // w[s * (PC + 1) + j]: coarse basis j at fine node s of an element
};

template <class T, int PF, int PC, int TX, int TY, int NT>
__global__ __launch_bounds__(NT) void k_prolong(ProlongW<T, PF, PC> pw, int n, int ze, const T *__restrict__ ecall,
                                                T *__restrict__ xfall) {
  constexpr int Q = PC + 1, FX = PF * TX, FY = PF * TY, CX = PC * TX + 1, CY = PC * TY + 1;
  constexpr int OWN = PF * FX * FY, NIT = (OWN + NT - 1) / NT;
  static_assert(CX * CY <= NT, "one coarse column per thread");
  __shared__ T H1[PF * CY * CX];   // [fz][cy][cx]
  __shared__ T H2[PF * FY * CX];   // [fz][fy][cx]
  __shared__ T W[PF * Q];
  const int Pf = PF * n, Pc = PC * n;
  const int ntx = (n + TX - 1) / TX, nty = (n + TY - 1) / TY, nz = (n + ze - 1) / ze;
  int b = xcd_linear(blockIdx.x, gridDim.x);
  const int bx = b % ntx;
  b /= ntx;
  const int by = b % nty;
  b /= nty;
  const int bz = b % nz, cfg = b / nz;
  const T *ec = ecall + size_t(cfg) * Pc * Pc * Pc;
  T *xf = xfall + size_t(cfg) * Pf * Pf * Pf;
  const int tid = threadIdx.x, e0 = bz * ze, e1 = min(e0 + ze, n);
  if (tid < PF * Q) W[tid] = pw.w[tid];
  // this thread's coarse column and fine nodes
  const bool col = tid < CX * CY;
  const int cx = tid % CX, cy = tid / CX;
  const unsigned coff = col ? unsigned((PC * TY * by + cy) % Pc * Pc + (PC * TX * bx + cx) % Pc) : 0u;
  const size_t Pc2 = size_t(Pc) * Pc, Pf2 = size_t(Pf) * Pf;
  unsigned foff[NIT];
  int hoff[NIT];   // H2 row of the node's element in x; its basis row above; -1: not owned
#pragma unroll
  for (int r = 0; r < NIT; ++r) {
    const int li = tid + NT * r, fx = li % FX, fy = li / FX % FY, fz = li / (FX * FY);
    const bool ok = li < OWN && FX * bx + fx < Pf && FY * by + fy < Pf;
    foff[r] = ok ? unsigned((fz * Pf + FY * by + fy) * Pf + FX * bx + fx) : 0u;
    hoff[r] = ok ? (fz * FY + fy) * CX + fx / PF * PC + (fx % PF << 16) : -1;
  }
  T v[Q], nv[PC], nf[NIT];
  v[0] = ec[size_t(PC * e0) * Pc2 + coff];
#pragma unroll
  for (int j = 0; j < PC; ++j) nv[j] = ec[size_t(wrapi(PC * e0 + 1 + j, Pc)) * Pc2 + coff];
#pragma unroll
  for (int r = 0; r < NIT; ++r) nf[r] = xf[size_t(PF * e0) * Pf2 + foff[r]];
  __syncthreads();
  for (int e = e0; e < e1; ++e) {
    T cur[NIT];
#pragma unroll
    for (int j = 0; j < PC; ++j) v[j + 1] = nv[j];
#pragma unroll
    for (int r = 0; r < NIT; ++r) cur[r] = nf[r];
    if (e + 1 < e1) {
#pragma unroll
      for (int j = 0; j < PC; ++j) nv[j] = ec[size_t(wrapi(PC * (e + 1) + 1 + j, Pc)) * Pc2 + coff];
#pragma unroll
      for (int r = 0; r < NIT; ++r) nf[r] = xf[size_t(PF * (e + 1)) * Pf2 + foff[r]];
    }
    if (col) {
#pragma unroll
      for (int f = 0; f < PF; ++f) {
        T a = T(0);
#pragma unroll
        for (int j = 0; j < Q; ++j) a += pw.w[f * Q + j] * v[j];
        H1[(f * CY + cy) * CX + cx] = a;
      }
    }
    v[0] = v[PC];
    __syncthreads();
    for (int t = tid; t < PF * TY * CX; t += NT) {   // y: (fz, element, cx)
      const int x = t % CX, ey = t / CX % TY, fz = t / (CX * TY);
      const T *h = H1 + (fz * CY + ey * PC) * CX + x;
      T u[Q];
#pragma unroll
      for (int j = 0; j < Q; ++j) u[j] = h[j * CX];
      T *o = H2 + (fz * FY + ey * PF) * CX + x;
#pragma unroll
      for (int f = 0; f < PF; ++f) {
        T a = T(0);
#pragma unroll
        for (int j = 0; j < Q; ++j) a += pw.w[f * Q + j] * u[j];
        o[f * CX] = a;
      }
    }
    __syncthreads();
    T *const dst = xf + size_t(PF * e) * Pf2;
#pragma unroll
    for (int r = 0; r < NIT; ++r) {
      const T *h = H2 + (hoff[r] & 0xffff), *w = W + (hoff[r] < 0 ? 0 : hoff[r] >> 16) * Q;
      if (hoff[r] < 0) continue;
      T a = T(0);
#pragma unroll
      for (int j = 0; j < Q; ++j) a += w[j] * h[j];
      dst[foff[r]] = cur[r] + a;
    }
    // the next z pass writes H1, last read before the barrier above; H2's next writes follow the next barrier
  }
}

template <class T, int PF, int PC, int TX, int TY, int NT>
int prolong(hipStream_t s, int nsys, const TransferT<T> &tr, const T *in, T *out) {
  const int n = tr.nf, cols = nsys * ((n + TX - 1) / TX) * ((n + TY - 1) / TY);
  // marches as long as four blocks per compute unit stay
  int ze = 1;
  while (2 * ze <= 16 && 2 * ze <= n && cols * ((n + 2 * ze - 1) / (2 * ze)) >= 1024) ze *= 2;
  ProlongW<T, PF, PC> pw;
  for (int i = 0; i < PF * (PC + 1); ++i) pw.w[i] = tr.w[i];
  hipLaunchKernelGGL((k_prolong<T, PF, PC, TX, TY, NT>), dim3(cols * ((n + ze - 1) / ze)), dim3(NT), 0, s, pw, n, ze, in,
                     out);
  return 0;
}

}  // namespace

template <class T>
int launch_prolong(hipStream_t s, int nsys, const TransferT<T> &tr, const T *in, T *out) {
  if (tr.r != 1) return -1;
  switch (tr.pf * 10 + tr.pc) {
    case 53: return prolong<T, 5, 3, 4, 4, 512>(s, nsys, tr, in, out);
    case 43: return prolong<T, 4, 3, 4, 4, 512>(s, nsys, tr, in, out);
    case 63: return prolong<T, 6, 3, 4, 4, 512>(s, nsys, tr, in, out);
    case 31: return prolong<T, 3, 1, 8, 4, 256>(s, nsys, tr, in, out);
    default: return -1;
  }
}
template int launch_prolong<double>(hipStream_t, int, const Transfer &, const double *, double *);
template int launch_prolong<float>(hipStream_t, int, const TransferF &, const float *, float *);

}  // namespace fep3m
