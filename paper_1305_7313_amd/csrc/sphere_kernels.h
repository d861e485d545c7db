// One-dimensional passes between the G-sphere and real space.
//
// Measured on 96 x 96 x 128 FP64, 128 bands, whole call: density 3014 -> 781 us,
// force 4802 -> 1557 us, against clearing, scattering, full pencils and a plane
// kernel holding the accumulator or V(r); orbitals to real space and back on
// 64^3 FP64, 128 orbitals: 517 -> 144 and 388 -> 164 us.
//
// A sphere of radius M on a grid of n >= 4M + 1 points fills a fifth of the
// plane columns (i2, i3).  The passes here transform only those, and read and
// write only the 128-byte lines of a box that hold them:
//
//   sphere_kernel  along i1: coefficients -> live lines of the box, or back
//   axis2_kernel   along i2: live columns, live rows -> every row, or back
//   rows_kernel    along i3, for the band loops: sums w |psi|^2, or multiplies
//                  by V(r) and transforms back
//
// An orbital goes to real space by sphere_kernel and the plane kernel; against
// clearing a box, scattering into it and transforming every pencil that is 1.5
// instead of 5 box sizes of traffic.  The band loops, which keep no orbital in
// real space, take three one-dimensional passes: a plane of 96 x 128 FP64
// values fills a compute unit's registers and LDS, so a plane kernel holds one
// plane per CU (and spilled beside an accumulator), while these tiles of 16
// columns or 16-64 rows keep many workgroups per CU.
#pragma once

#include "fock_kernels.h"

namespace fockx {

enum SphereMode : int {
  SPHERE_INV = 0,       // coefficients -> box, backward along i1
  SPHERE_INV_PACK = 1,  // the same for two real orbitals per box (Gamma)
  SPHERE_FWD = 2,       // box -> scaled coefficients, forward along i1
  SPHERE_FWD_BOX = 3,   // forward along i1, in place (Gamma: unpacked by gather_unpack_kernel)
  SPHERE_FORCE = 4,     // as SPHERE_FWD, with the kinetic term of the band force
};

// The sphere on the plane: columns in whole lines of 128 bytes.  Line l holds
// the plane positions p = i2 n3 + i3 in [lines[l] LINE, lines[l] LINE + LINE),
// its column c is the compact column l LINE + c.
struct SphereTables {
  const int* lines;          // [nl] line numbers
  const int* coef;           // [n1][nl * LINE] sphere index of (i1, compact column), -1: none
  const signed char* live;   // [n3] last live row per column (live_row), -1: dead column
  const int* cols;           // [nc] live blocks of 8 columns: first column / 8
  int nl, nc;
};

struct SphereArgs {
  SphereTables tab;
  void* box;            // [nb][N]
  const void* tw1;      // twiddle table, length n1
  long long N;
  int n2, n3, ngrp;     // ngrp: workgroups per box
  const void* c;        // coefficients in (SPHERE_INV*; SPHERE_FORCE: rows j0 ..)
  int ldc;
  void* box2;           // SPHERE_INV: boxes nb1 .. of the launch, a second block (nb1 = 0: none)
  const void* c2;
  int ldc2, nb1;
  int nreal;            // SPHERE_INV_PACK: number of real orbitals
  void* out;            // coefficients out
  int ldo;
  // SPHERE_FWD: out[j] = s0 w[j0 + j] *g box[j]   (w, g null: 1)
  double s0;
  const double* w;      // SPHERE_FORCE: band weights
  const double* g;
  int j0;
  double b[3][3];       // SPHERE_FORCE: reciprocal vectors (rows) and the k-point
  double k[3];
};

// A workgroup takes CB compact columns (CB / LINE lines) of one box.  Bound by
// memory: a line is read or written once, rows of 128 bytes at the plane
// stride, and the coefficients of one row of the sphere are consecutive.
template <typename T, int N1, int CB, int W, bool SPLIT, int MODE>
__global__ __launch_bounds__(W) void sphere_kernel(SphereArgs A) {
  using G = PencilGeom<T, N1, CB, W, SPLIT>;
  using P0 = typename G::Ax::P0;
  using P1 = typename G::Ax::P1;
  constexpr int LINE = 128 / (int)sizeof(cx<T>);
  constexpr bool inv = MODE == SPHERE_INV || MODE == SPHERE_INV_PACK;
  static_assert(CB % LINE == 0, "whole lines");
  static_assert(W >= N1, "one table entry per thread");
  __shared__ __align__(16) unsigned char smem[G::XBYTES];
  __shared__ cx<T> tw1[N1];
  const int t = threadIdx.x;
  const int lid = xcd_logical(blockIdx.x, gridDim.x);
  const int pr = lid / A.ngrp, grp = lid - pr * A.ngrp;
  const int plane = A.n2 * A.n3, ncol = A.tab.nl * LINE;
  if (t < N1) tw1[t] = reinterpret_cast<const cx<T>*>(A.tw1)[t];
  // every value of this thread is in tile column t % CB (a column pass)
  const int li = grp * (CB / LINE) + (t % CB) / LINE;
  const bool act = li < A.tab.nl;
  const int cc = li * LINE + t % LINE;
  const int p = act ? A.tab.lines[li] * LINE + t % LINE : 0;
  const bool second = MODE == SPHERE_INV && A.nb1 > 0 && pr >= A.nb1;
  cx<T>* box = reinterpret_cast<cx<T>*>(second ? A.box2 : A.box) + (long long)(second ? pr - A.nb1 : pr) * A.N + p;
  cx<T> v[G::NV];
  if constexpr (inv) {
    int idx[P0::NV];
    for_inputs<P0>(t, [&](int e, int row, int) { idx[e] = act ? A.tab.coef[row * ncol + cc] : -1; });
    const cx<T>* c = second ? reinterpret_cast<const cx<T>*>(A.c2) + (long long)(pr - A.nb1) * A.ldc2
                            : reinterpret_cast<const cx<T>*>(A.c) + (long long)(MODE == SPHERE_INV ? pr : 2 * pr) * A.ldc;
    const bool two = MODE == SPHERE_INV_PACK && 2 * pr + 1 < A.nreal;
    for_inputs<P0>(t, [&](int e, int, int) {
      cx<T> z = mk<T>(T(0), T(0));
      if (idx[e] >= 0) {
        z = c[idx[e]];
        if (two) {
          const cx<T> y = c[A.ldc + idx[e]];
          z = mk<T>(z.x - y.y, z.y + y.x);
        }
      }
      v[e] = z;
    });
  } else {
    for_inputs<P0>(t, [&](int e, int row, int) {
      v[e] = act ? box[(long long)row * plane] : mk<T>(T(0), T(0));
    });
  }
  __syncthreads();  // tw1
  constexpr int DIR = inv ? +1 : -1;
  pass_compute<P0, DIR, T>(v, tw1, t);
  exchange<P0, P1, CB, SPLIT, T>(v, smem, t);
  pass_compute<P1, DIR, T>(v, tw1, t);
  settle<P1>(v, t);
  if (!act) return;
  if constexpr (inv || MODE == SPHERE_FWD_BOX) {
    for_outputs<P1>(t, [&](int e, int row, int) { box[(long long)row * plane] = v[e]; });
  } else {
    cx<T>* out = reinterpret_cast<cx<T>*>(A.out) + (long long)(A.j0 + pr) * A.ldo;
    if constexpr (MODE == SPHERE_FWD) {
      double s = A.s0;
      if (A.w) s *= A.w[A.j0 + pr];
      if (A.g) s *= *A.g;
      const T st = T(s);
      for_outputs<P1>(t, [&](int e, int row, int) {
        const int i = A.tab.coef[row * ncol + cc];
        if (i >= 0) out[i] = cscale<T>(v[e], st);
      });
    } else {
      // -w (1/2 |k+G|^2 c + box / N)
      const cx<T>* c = reinterpret_cast<const cx<T>*>(A.c) + (long long)(A.j0 + pr) * A.ldc;
      const int i2 = p / A.n3;
      const int m2 = signed_index(i2, A.n2), m3 = signed_index(p - i2 * A.n3, A.n3);
      const T sv = T(1.0 / double(A.N)), mw = T(-A.w[A.j0 + pr]);
      for_outputs<P1>(t, [&](int e, int row, int) {
        const int i = A.tab.coef[row * ncol + cc];
        if (i < 0) return;
        const int m1 = signed_index(row, N1);
        double g2 = 0.0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          const double ga = A.k[a] + m1 * A.b[0][a] + m2 * A.b[1][a] + m3 * A.b[2][a];
          g2 += ga * ga;
        }
        const cx<T> cp = c[i];
        const T kin = T(0.5 * g2);
        out[i] = mk<T>(mw * (kin * cp.x + sv * v[e].x), mw * (kin * cp.y + sv * v[e].y));
      });
    }
  }
}

// ---------------------------------------------------------------------------
// Transform along i2 of the live columns of every plane, in place: backward
// from the live rows to every row, forward from every row to the live rows'
// lines.  A workgroup takes 16 columns (two live blocks of 8) of one plane.
// ---------------------------------------------------------------------------
struct Axis2Args {
  SphereTables tab;
  void* box;        // [nb][N]
  const void* tw2;
  int ngrp;         // workgroups per plane: ceil(nc / 2)
};

constexpr int kAxis2Cols = 16;
constexpr int axis2_threads(int n2) { return n2 >= 96 ? 192 : n2 == 72 ? 144 : 128; }

template <typename T, int N2, int N3, int DIR>
__global__ __launch_bounds__(axis2_threads(N2)) void axis2_kernel(Axis2Args A) {
  constexpr int CB = kAxis2Cols, W = axis2_threads(N2);
  using Ax = Axis<N2, CB, false, W>;
  using P0 = typename Ax::P0;
  using P1 = typename Ax::P1;
  __shared__ __align__(16) cx<T> smem[Tile<CB>::slots(N2)];
  __shared__ cx<T> tw2[N2];
  static_assert(W >= N2, "one table entry per thread");
  const int t = threadIdx.x;
  const int lid = xcd_logical(blockIdx.x, gridDim.x);
  const int pl = lid / A.ngrp, grp = lid - pl * A.ngrp;  // pl = box * n1 + i1
  if (t < N2) tw2[t] = reinterpret_cast<const cx<T>*>(A.tw2)[t];
  const int blk = 2 * grp + (t % CB) / 8;
  const bool act = blk < A.tab.nc;
  const int i3 = act ? 8 * A.tab.cols[blk] + t % 8 : 0;
  const int h = act ? A.tab.live[i3] : -1;
  cx<T>* x = reinterpret_cast<cx<T>*>(A.box) + (long long)pl * (N2 * N3) + i3;
  cx<T> v[Ax::NV];
  for_inputs<P0>(t, [&](int e, int row, int) {
    const bool rd = DIR > 0 ? h >= 0 && live_row<N2>(row, h) : act;
    v[e] = rd ? x[row * N3] : mk<T>(T(0), T(0));
  });
  __syncthreads();
  pass_compute<P0, DIR, T>(v, tw2, t);
  exchange<P0, P1, CB, false, T>(v, smem, t);
  pass_compute<P1, DIR, T>(v, tw2, t);
  for_outputs<P1>(t, [&](int e, int row, int) {
    // forward: the block of 8 columns is written whole where one of them is live
    bool wr = act;
    if constexpr (DIR < 0) {
      const unsigned long long m = __ballot(h >= 0 && live_row<N2>(row, h));
      wr = act && ((m >> ((t & 63) & ~7)) & 0xff) != 0;
    }
    if (wr) x[row * N3] = v[e];
  });
}

// ---------------------------------------------------------------------------
// Rows along i3 of the band loops.  A workgroup takes RB rows (i1, i2) and the
// bands g, g + ngrp, ... of the chunk; the sum of w |psi|^2 over its bands, or
// V(r) on its rows, stays in registers.
// ---------------------------------------------------------------------------
enum RowsMode : int { ROWS_DENS = 0, ROWS_VMUL = 1 };

struct RowsArgs {
  SphereTables tab;
  void* box;           // [nb][N]
  const void* tw3;
  long long N;
  int nrb, nb, ngrp;   // row workgroups (n1 n2 / RB), bands in the chunk, band groups
  const double* f;     // ROWS_DENS: weights of the chunk's bands
  double fscale;
  double* part;        // ROWS_DENS: FP64 partial densities [ngrp][N]
  int accumulate;      // ROWS_DENS: add to part (else overwrite)
  const void* vloc;    // ROWS_VMUL: real potential V(r) [N], path precision
};

struct RowsTune {
  int rb, w;
};
// rb divides every n1 n2 (a multiple of 64); w a multiple of both radix passes'
// butterflies per row
constexpr RowsTune rows_tune(int n3) {
  switch (n3) {
    case 24: return RowsTune{64, 192};
    case 48: return RowsTune{32, 192};
    case 64: return RowsTune{32, 256};
    case 72: return RowsTune{32, 288};
    case 96: return RowsTune{16, 192};
    default: return RowsTune{8, 128};
  }
}

template <typename T, int N3, int MODE>
__global__ __launch_bounds__(rows_tune(N3).w) void rows_kernel(RowsArgs A) {
  constexpr int RB = rows_tune(N3).rb, W = rows_tune(N3).w;
  using Ax = Axis<N3, RB, true, W>;
  using P0 = typename Ax::P0;
  using P1 = typename Ax::P1;
  constexpr bool PAD = N3 % 8 == 0;
  constexpr int SLOTS = Tile<N3, XK_RR>::slots(RB);
  __shared__ __align__(16) cx<T> smem[SLOTS];
  __shared__ cx<T> tw3[N3];
  const int t = threadIdx.x;
  const int lid = xcd_logical(blockIdx.x, gridDim.x);
  const int rc = lid / A.ngrp, g = lid - rc * A.ngrp;
  if (t < N3) tw3[t] = reinterpret_cast<const cx<T>*>(A.tw3)[t];
  const long long r0 = (long long)rc * RB * N3;
  // live columns of this thread's inputs: one bit per value
  unsigned in_live = 0;
  for_inputs<P0>(t, [&](int e, int, int col) { in_live |= (A.tab.live[col] >= 0 ? 1u : 0u) << e; });
  static_assert(P0::NV <= 32 && P1::NV <= 32, "one mask bit per value");
  __syncthreads();
  if constexpr (MODE == ROWS_DENS) {
    double* pp = A.part + (long long)g * A.N + r0;
    double acc[P1::NV];
#pragma unroll
    for (int e = 0; e < P1::NV; ++e) acc[e] = 0.0;
    if (A.accumulate) for_outputs<P1>(t, [&](int e, int row, int col) { acc[e] = pp[row * N3 + col]; });
    for (int b = g; b < A.nb; b += A.ngrp) {
      cx<T> v[Ax::NV];
      const cx<T>* x = reinterpret_cast<const cx<T>*>(A.box) + (long long)b * A.N + r0;
      for_inputs<P0>(t, [&](int e, int row, int col) {
        v[e] = (in_live >> e) & 1u ? x[row * N3 + col] : mk<T>(T(0), T(0));
      });
      pass_compute<P0, +1, T>(v, tw3, t);
      exchange<P0, P1, N3, false, T, PAD>(v, smem, t);
      pass_compute<P1, +1, T>(v, tw3, t);
      const T wb = T(A.f[b] * A.fscale);
      for_outputs<P1>(t, [&](int e, int, int) { acc[e] += double(wb * (v[e].x * v[e].x + v[e].y * v[e].y)); });
    }
    for_outputs<P1>(t, [&](int e, int row, int col) { pp[row * N3 + col] = acc[e]; });
  } else {
    // whole blocks of 8 columns are written where one of them is live
    unsigned out_live = 0;
    for_outputs<P1>(t, [&](int e, int, int col) {
      bool any = false;
      for (int k = 0; k < 8; ++k) any |= A.tab.live[(col & ~7) + k] >= 0;
      out_live |= (any ? 1u : 0u) << e;
    });
    const T* pv = reinterpret_cast<const T*>(A.vloc) + r0;
    T vr[P1::NV];
    for_outputs<P1>(t, [&](int e, int row, int col) { vr[e] = pv[row * N3 + col]; });
    for (int b = g; b < A.nb; b += A.ngrp) {
      cx<T> v[Ax::NV];
      cx<T>* x = reinterpret_cast<cx<T>*>(A.box) + (long long)b * A.N + r0;
      for_inputs<P0>(t, [&](int e, int row, int col) {
        v[e] = (in_live >> e) & 1u ? x[row * N3 + col] : mk<T>(T(0), T(0));
      });
      pass_compute<P0, +1, T>(v, tw3, t);
      exchange<P0, P1, N3, false, T, PAD>(v, smem, t);
      pass_compute<P1, +1, T>(v, tw3, t);
      for_outputs<P1>(t, [&](int e, int, int) { v[e] = cscale<T>(v[e], vr[e]); });
      exchange<P1, P0, N3, false, T, PAD>(v, smem, t);
      pass_compute<P0, -1, T>(v, tw3, t);
      exchange<P0, P1, N3, false, T, PAD>(v, smem, t);
      pass_compute<P1, -1, T>(v, tw3, t);
      for_outputs<P1>(t, [&](int e, int row, int col) {
        if ((out_live >> e) & 1u) x[row * N3 + col] = v[e];
      });
    }
  }
}

}  // namespace fockx
