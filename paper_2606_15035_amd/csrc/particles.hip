// Particle-side kernels for gfx950: orbit current scatter, orbit gather with
// the orbit-discrete gradient and canonical-momentum push, the consistency
// sweep, and the end-of-step update.
//
// One lane per particle, or four in the gather of small counts and of FP64 particles
// beyond their block's node box; particle arrays are structure-of-arrays doubles
// (component a of particle i at a*np + i).  The mesh fields a particle reads
// during the gather are interleaved per node (kGbufStride doubles per node:
// grad_h phi^{n+1/2}, A^n, A^{n+1}) so that one stencil node costs one short
// run of contiguous loads.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "internal.hpp"
#include "orbit.hpp"
#include "reduce.hpp"

namespace ecpic {

namespace {

template <int R>
struct Quad;
template <>
struct Quad<1> {
  static constexpr int NQ = 2;  // 2 n_q - 1 >= 3 r  ->  n_q = 2 for r = 1
};
template <>
struct Quad<2> {
  static constexpr int NQ = 4;  // n_q = 4 for r = 2
};
template <>
struct Quad<3> {
  static constexpr int NQ = 5;  // n_q = 5 for r = 3
};

// ---- field accessors ------------------------------------------------------
struct AosFields {
  const double* __restrict__ g;
  __device__ __forceinline__ void load9(int64_t node, double* f) const {
    const double* p = g + node * kGbufStride;
#pragma unroll
    for (int k = 0; k < 9; ++k) f[k] = p[k];
  }
  __device__ __forceinline__ double A0(int64_t node, int l) const { return g[node * kGbufStride + 3 + l]; }
  __device__ __forceinline__ double A1(int64_t node, int l) const { return g[node * kGbufStride + 6 + l]; }
};

// Accessors of the push path.  A stencil node is addressed by its unwrapped
// integer coordinates in the particle's frame; row() folds (ix, iy), node()
// adds iz and returns the node's kGbufStride doubles
// [grad_h phi (3) | A^n (3) | A^{n+1} (3) | pad].
struct GlobalGather {  // the interleaved gather buffer in global memory
  const double* __restrict__ g;
  int mask0, mask1, mask2, shx, shy;
  __device__ __forceinline__ int row(int ix, int iy) const {
    return ((ix & mask0) << shx) | ((iy & mask1) << shy);
  }
  __device__ __forceinline__ const double* node(int row, int iz) const {
    return g + (int64_t)(row | (iz & mask2)) * kGbufStride;
  }
};

typedef __attribute__((address_space(3))) const double lds_cdouble;

struct TileGather {  // a block's LDS copy of the nodes its orbits touch
  lds_cdouble* t;
  int ox, oy, oz;    // particle frame -> tile coordinates
  int dy, dz;        // tile extents along y and z
  __device__ __forceinline__ int row(int ix, int iy) const { return ((ix + ox) * dy + (iy + oy)) * dz + oz; }
  __device__ __forceinline__ lds_cdouble* node(int row, int iz) const {
    return t + (row + iz) * kGbufStride;
  }
};

struct SoaFields {
  const double* __restrict__ gphi;
  const double* __restrict__ a0;
  const double* __restrict__ a1;
  int64_t nc;
  __device__ __forceinline__ void load9(int64_t node, double* f) const {
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      f[l] = gphi[l * nc + node];
      f[3 + l] = a0[l * nc + node];
      f[6 + l] = a1[l * nc + node];
    }
  }
  __device__ __forceinline__ double A0(int64_t node, int l) const { return a0[l * nc + node]; }
  __device__ __forceinline__ double A1(int64_t node, int l) const { return a1[l * nc + node]; }
};

__device__ __forceinline__ int64_t node_of(const Grid& G, int ix, int iy, int iz) {
  return node_index(G, ix, iy, iz);
}

// ---- one orbit piece: current scatter -------------------------------------
// Iw[a][b][c] = int_{s0}^{s1} S_g(x(s)) ds for the stencil node first + (a, b, c)
// (eq. split-Sbar); first is the unwrapped index of the piece's first stencil node.
// NP quadrature points sq[] with weights wq[] against the stencil of base
template <int R, int NP>
__device__ __forceinline__ void sbar_points(const Grid& G, const double* x0, const double* d,
                                            const double* base, const double* sq,
                                            const double* wq,
                                            double (&Iw)[R + 1][R + 1][R + 1], int* first) {
  constexpr int W = R + 1;
#pragma unroll
  for (int a = 0; a < W; ++a)
#pragma unroll
    for (int b = 0; b < W; ++b)
#pragma unroll
      for (int c = 0; c < W; ++c) Iw[a][b][c] = 0.0;
#pragma unroll
  for (int q = 0; q < NP; ++q) {
    const double s = sq[q];
    const double wt = wq[q];
    double wx[W], wy[W], wz[W];
    Spline<R>::w((x0[0] + s * d[0]) * G.invH[0] - base[0], wx);
    Spline<R>::w((x0[1] + s * d[1]) * G.invH[1] - base[1], wy);
    Spline<R>::w((x0[2] + s * d[2]) * G.invH[2] - base[2], wz);
#pragma unroll
    for (int a = 0; a < W; ++a) {
      const double xa = wt * wx[a];
#pragma unroll
      for (int b = 0; b < W; ++b) {
        const double xy = xa * wy[b];
#pragma unroll
        for (int c = 0; c < W; ++c) Iw[a][b][c] += xy * wz[c];
      }
    }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) first[a] = to_int_clamped(base[a]) + Spline<R>::first_off;
}

// the n_q-point rule of a piece [s0, s1] (its stencil comes with the piece)
template <int R>
__device__ __forceinline__ void piece_rule(double s0, double s1, double* sq, double* wq) {
  constexpr int NQ = Quad<R>::NQ;
  const double h = s1 - s0;
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    sq[q] = s0 + 0.5 * h * (1.0 + Gauss<NQ>::x(q));
    wq[q] = 0.5 * h * Gauss<NQ>::w(q);
  }
}

// point q of the rule over the whole orbit (no splitting): the stencil is
// the one of x(s_q) itself (comparison runs)
template <int R>
__device__ __forceinline__ void unsplit_point(const Grid& G, const QuadRule& rule, int q,
                                              const double* x0, const double* d, double* base,
                                              double& s, double& w) {
  s = rule.s[q];
  w = rule.w[q];
  point_base<R>(x0, d, s, G, base);
}

template <int R>
__device__ __forceinline__ void piece_sbar(const Grid& G, const double* x0, const double* d,
                                           double s0, double s1, const double* base,
                                           double (&Iw)[R + 1][R + 1][R + 1], int* first) {
  constexpr int NQ = Quad<R>::NQ;
  double sq[NQ], wq[NQ];
  piece_rule<R>(s0, s1, sq, wq);
  sbar_points<R, NQ>(G, x0, d, base, sq, wq, Iw, first);
}

// J_g += (q vbar / dV) int_{s0}^{s1} S_g(x(s)) ds straight into global memory
// (eq. orbit-current, split form)
template <int R>
__device__ __forceinline__ void scatter_piece(const Grid& G, const double* x0, const double* d,
                                              double s0, double s1, const double* base,
                                              const double* c3, double* __restrict__ J) {
  constexpr int W = R + 1;
  double Iw[W][W][W];
  int f[3];
  piece_sbar<R>(G, x0, d, s0, s1, base, Iw, f);
  const int64_t nc = G.ncell;
#pragma unroll
  for (int a = 0; a < W; ++a) {
    const int ix = wrapi(f[0] + a, G.n[0]);
#pragma unroll
    for (int b = 0; b < W; ++b) {
      const int iy = wrapi(f[1] + b, G.n[1]);
#pragma unroll
      for (int c = 0; c < W; ++c) {
        const int64_t g = node_of(G, ix, iy, wrapi(f[2] + c, G.n[2]));
        const double w = Iw[a][b][c];
        unsafeAtomicAdd(J + g, w * c3[0]);
        unsafeAtomicAdd(J + nc + g, w * c3[1]);
        unsafeAtomicAdd(J + 2 * nc + g, w * c3[2]);
      }
    }
  }
}

// ---- one orbit piece: gather --------------------------------------------
// gp_l  += sum_g (grad_h phi)_lg int S_g ds                 (eq. gphibar-definition)
// D_lj  += sum_g int A_lg(s) d_j S_g(x(s)) ds, A_g(s) = (1-s) A^n + s A^{n+1}  (eq. split-DA)
// with WITH_U also Ub_l += sum_g U_lg int S_g ds and pou += int sum_g S_g ds.
// The n_q-point rule is evaluated once per piece; each stencil node then
// accumulates its weight integrals over the quadrature points and is
// contracted with the node's field values.
template <int R, int NQ, bool WITH_U, class Acc>
__device__ __forceinline__ void gather_points(const Grid& G, const double* x0, const double* d,
                                              const double* base, const double* sqs,
                                              const double* wqs, const Acc& acc,
                                              const double* __restrict__ Uh, double* gp,
                                              double (*D)[3], double* Ub, double& pou) {
  constexpr int W = R + 1;
  double X[NQ][W], dX[NQ][W], Y[NQ][W], dY[NQ][W];
  double Zw[NQ][W], Z0[NQ][W], Z1[NQ][W], dZ0[NQ][W], dZ1[NQ][W];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const double s = sqs[q];
    const double wt = wqs[q];
    const double w0 = wt * (1.0 - s), w1 = wt * s;
    double wz[W], dz[W];
    Spline<R>::wd((x0[0] + s * d[0]) * G.invH[0] - base[0], X[q], dX[q]);
    Spline<R>::wd((x0[1] + s * d[1]) * G.invH[1] - base[1], Y[q], dY[q]);
    Spline<R>::wd((x0[2] + s * d[2]) * G.invH[2] - base[2], wz, dz);
#pragma unroll
    for (int k = 0; k < W; ++k) {
      dX[q][k] *= G.invH[0];
      dY[q][k] *= G.invH[1];
      const double dzk = dz[k] * G.invH[2];
      Zw[q][k] = wt * wz[k];
      Z0[q][k] = w0 * wz[k];
      Z1[q][k] = w1 * wz[k];
      dZ0[q][k] = w0 * dzk;
      dZ1[q][k] = w1 * dzk;
    }
  }
  const int fx = to_int_clamped(base[0]) + Spline<R>::first_off;
  const int fy = to_int_clamped(base[1]) + Spline<R>::first_off;
  const int fz = to_int_clamped(base[2]) + Spline<R>::first_off;
#pragma unroll
  for (int a = 0; a < W; ++a) {
    const int ix = wrapi(fx + a, G.n[0]);
#pragma unroll
    for (int b = 0; b < W; ++b) {
      const int iy = wrapi(fy + b, G.n[1]);
      double xy[NQ], dxy[NQ], xdy[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        xy[q] = X[q][a] * Y[q][b];
        dxy[q] = dX[q][a] * Y[q][b];
        xdy[q] = X[q][a] * dY[q][b];
      }
#pragma unroll
      for (int c = 0; c < W; ++c) {
        const int64_t g = node_of(G, ix, iy, wrapi(fz + c, G.n[2]));
        double f[9];
        acc.load9(g, f);
        double I = 0.0, K0x = 0.0, K1x = 0.0, K0y = 0.0, K1y = 0.0, K0z = 0.0, K1z = 0.0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          I += xy[q] * Zw[q][c];
          K0x += dxy[q] * Z0[q][c];
          K1x += dxy[q] * Z1[q][c];
          K0y += xdy[q] * Z0[q][c];
          K1y += xdy[q] * Z1[q][c];
          K0z += xy[q] * dZ0[q][c];
          K1z += xy[q] * dZ1[q][c];
        }
#pragma unroll
        for (int l = 0; l < 3; ++l) {
          gp[l] += f[l] * I;
          D[l][0] += f[3 + l] * K0x + f[6 + l] * K1x;
          D[l][1] += f[3 + l] * K0y + f[6 + l] * K1y;
          D[l][2] += f[3 + l] * K0z + f[6 + l] * K1z;
        }
        if constexpr (WITH_U) {
#pragma unroll
          for (int l = 0; l < 3; ++l) Ub[l] += Uh[l * G.ncell + g] * I;
          pou += I;
        }
      }
    }
  }
}

template <int R, bool WITH_U, class Acc>
__device__ __forceinline__ void gather_piece(const Grid& G, const double* x0, const double* d,
                                             double s0, double s1, const double* base,
                                             const Acc& acc, const double* __restrict__ Uh,
                                             double* gp, double (*D)[3], double* Ub, double& pou) {
  constexpr int NQ = Quad<R>::NQ;
  double sq[NQ], wq[NQ];
  piece_rule<R>(s0, s1, sq, wq);
  gather_points<R, NQ, WITH_U>(G, x0, d, base, sq, wq, acc, Uh, gp, D, Ub, pou);
}

// weight and derivative (per unit of cell coordinate) of stencil node k at t, for
// a k that differs from lane to lane
template <int R>
__device__ __forceinline__ void lane_weight(int k, double t, double& w, double& dw) {
  double ws[R + 1], ds[R + 1];
  Spline<R>::wd(t, ws, ds);
  w = ws[0];
  dw = ds[0];
#pragma unroll
  for (int j = 1; j <= R; ++j) {
    w = k == j ? ws[j] : w;
    dw = k == j ? ds[j] : dw;
  }
}

// ---- one orbit piece: gather for the push ----------------------------------
// The push needs grad phi-bar and (D A)^T vbar only.  With b_g(s) = vbar . A_g(s),
//   ((D A)^T vbar)_j = sum_g int b_g(s) d_j S_g(x(s)) ds,
// so each node first contracts its A^n, A^{n+1} with vbar and the quadrature
// then carries one scalar per node instead of the 3x3 matrix D.  The tensor
// product S_g = X_a Y_b Z_c is used once more: along each z column of the
// stencil the quadrature-point sums B_q = sum_c b_c(s_q) Z_c(q) and
// B'_q = sum_c b_c(s_q) Z'_c(q) are formed first, and the x and y factors
// multiply those column sums, not every node.  Derivatives are taken per unit
// of cell coordinate: dtv accumulates H_j ((D A)^T vbar)_j, and the caller
// multiplies by 1/H_j once per particle.
// LANES = 1: the whole stencil.  4: lane `part` of a quad takes the rows of its
// plane a = part (degree 1: the one row a = part / 2, b = part % 2), and the sums
// of the quad are the particle's.
template <int R, int LANES, int NQ, class Acc>
__device__ __forceinline__ void push_points(const Grid& G, const double* x0, const double* d,
                                            const double* base, const double* sq,
                                            const double* wq, const double* vb, const Acc& acc,
                                            int part, double* gp, double* dtv) {
  constexpr int W = R + 1;
  double tx[NQ], ty[NQ], Z[NQ][W], dZ[NQ][W];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const double s = sq[q];
    tx[q] = (x0[0] + s * d[0]) * G.invH[0] - base[0];
    ty[q] = (x0[1] + s * d[1]) * G.invH[1] - base[1];
    Spline<R>::wd((x0[2] + s * d[2]) * G.invH[2] - base[2], Z[q], dZ[q]);
  }
  const int fx = to_int_clamped(base[0]) + Spline<R>::first_off;
  const int fy = to_int_clamped(base[1]) + Spline<R>::first_off;
  const int fz = to_int_clamped(base[2]) + Spline<R>::first_off;
  // one row (a, b): Xw, dXw = quadrature weight x X_a, x dX_a/dx; ybd gives Y_b, dY_b
  auto stencil_row = [&](int a, int b, const double (&Xw)[NQ], const double (&dXw)[NQ],
                         auto&& ybd) {
    double xyw[NQ], dxyw[NQ], xdyw[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      double Yq, dYq;
      ybd(ty[q], Yq, dYq);
      xyw[q] = Xw[q] * Yq;
      dxyw[q] = dXw[q] * Yq;
      xdyw[q] = Xw[q] * dYq;
    }
    const int row = acc.row(fx + a, fy + b);
    double B[NQ], dB[NQ];
#pragma unroll
    for (int c = 0; c < W; ++c) {
      const auto p = acc.node(row, fz + c);
      double f[9];
#pragma unroll
      for (int k = 0; k < 9; ++k) f[k] = p[k];
      const double a0 = vb[0] * f[3] + vb[1] * f[4] + vb[2] * f[5];  // vbar . A^n_g
      const double da = vb[0] * f[6] + vb[1] * f[7] + vb[2] * f[8] - a0;
      double I = 0.0;
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        I += xyw[q] * Z[q][c];
        const double bq = a0 + sq[q] * da;  // vbar . A_g(s_q)
        B[q] = c == 0 ? bq * Z[q][c] : B[q] + bq * Z[q][c];
        dB[q] = c == 0 ? bq * dZ[q][c] : dB[q] + bq * dZ[q][c];
      }
      gp[0] += f[0] * I;
      gp[1] += f[1] * I;
      gp[2] += f[2] * I;
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      dtv[0] += dxyw[q] * B[q];
      dtv[1] += xdyw[q] * B[q];
      dtv[2] += xyw[q] * dB[q];
    }
  };
  if constexpr (LANES == 1) {
#pragma unroll
    for (int a = 0; a < W; ++a) {
      double Xw[NQ], dXw[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        double Xq, dXq;
        Spline<R>::wk(a, tx[q], Xq, dXq);
        Xw[q] = wq[q] * Xq;
        dXw[q] = wq[q] * dXq;
      }
#pragma unroll
      for (int b = 0; b < W; ++b)
        stencil_row(a, b, Xw, dXw,
                    [&](double t, double& y, double& dy) { Spline<R>::wk(b, t, y, dy); });
    }
  } else {
    const int a = R == 1 ? part / 2 : part;
    if (a < W) {
      double Xw[NQ], dXw[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        double Xq, dXq;
        lane_weight<R>(a, tx[q], Xq, dXq);
        Xw[q] = wq[q] * Xq;
        dXw[q] = wq[q] * dXq;
      }
      if constexpr (R == 1) {
        const int b = part % 2;
        stencil_row(a, b, Xw, dXw,
                    [&](double t, double& y, double& dy) { lane_weight<R>(b, t, y, dy); });
      } else {
#pragma unroll
        for (int b = 0; b < W; ++b)
          stencil_row(a, b, Xw, dXw,
                      [&](double t, double& y, double& dy) { Spline<R>::wk(b, t, y, dy); });
      }
    }
  }
}

template <int R, int LANES, class Acc>
__device__ __forceinline__ void push_piece(const Grid& G, const double* x0, const double* d,
                                           double s0, double s1, const double* base,
                                           const double* vb, const Acc& acc, int part, double* gp,
                                           double* dtv) {
  constexpr int NQ = Quad<R>::NQ;
  double sq[NQ], wq[NQ];
  piece_rule<R>(s0, s1, sq, wq);
  push_points<R, LANES, NQ>(G, x0, d, base, sq, wq, vb, acc, part, gp, dtv);
}

// point interpolant of A^n (which = 0) or A^{n+1} (which = 1) at x, whose
// stencil nodes are moved into the particle frame by +shift[a] (a multiple
// of n[a]; zero unless x is a wrapped end point)
// LANES, part: as in push_points
template <int R, int LANES, class Acc>
__device__ __forceinline__ void point_A_acc(const Grid& G, const double* x, const int* shift,
                                            const Acc& acc, int which, int part, double* out) {
  constexpr int W = R + 1;
  double w[3][W];
  int f[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double u = x[a] * G.invH[a];
    const double base = floor(u + Spline<R>::base_off);
    Spline<R>::w(u - base, w[a]);
    f[a] = to_int_clamped(base) + Spline<R>::first_off + shift[a];
  }
  out[0] = out[1] = out[2] = 0.0;
  const int off = which ? 6 : 3;
  auto stencil_row = [&](int a, int b, double wxy) {
    const int row = acc.row(f[0] + a, f[1] + b);
#pragma unroll
    for (int c = 0; c < W; ++c) {
      const auto p = acc.node(row, f[2] + c);
      const double wt = wxy * w[2][c];
#pragma unroll
      for (int l = 0; l < 3; ++l) out[l] += p[off + l] * wt;
    }
  };
  if constexpr (LANES == 1) {
#pragma unroll
    for (int a = 0; a < W; ++a)
#pragma unroll
      for (int b = 0; b < W; ++b) stencil_row(a, b, w[0][a] * w[1][b]);
  } else {
    const int a = R == 1 ? part / 2 : part;
    double wa = w[0][0];
#pragma unroll
    for (int k = 1; k < W; ++k) wa = a == k ? w[0][k] : wa;
    if (a < W) {
      if constexpr (R == 1) {
        stencil_row(a, part % 2, wa * (part % 2 ? w[1][1] : w[1][0]));
      } else {
#pragma unroll
        for (int b = 0; b < W; ++b) stencil_row(a, b, wa * w[1][b]);
      }
    }
  }
}

// point interpolant F_h(x) = sum_g F_g S_g(x) of A^n (which = 0) or A^{n+1} (which = 1)
template <int R, class Acc>
__device__ __forceinline__ void point_A(const Grid& G, const double* x, const Acc& acc, int which,
                                        double* out) {
  constexpr int W = R + 1;
  double w[3][W];
  int f[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double u = x[a] * G.invH[a];
    const double base = floor(u + Spline<R>::base_off);
    Spline<R>::w(u - base, w[a]);
    f[a] = to_int_clamped(base) + Spline<R>::first_off;
  }
  out[0] = out[1] = out[2] = 0.0;
#pragma unroll
  for (int a = 0; a < W; ++a) {
    const int ix = wrapi(f[0] + a, G.n[0]);
#pragma unroll
    for (int b = 0; b < W; ++b) {
      const int iy = wrapi(f[1] + b, G.n[1]);
      const double wxy = w[0][a] * w[1][b];
#pragma unroll
      for (int c = 0; c < W; ++c) {
        const int64_t g = node_of(G, ix, iy, wrapi(f[2] + c, G.n[2]));
        const double wt = wxy * w[2][c];
#pragma unroll
        for (int l = 0; l < 3; ++l) out[l] += (which ? acc.A1(g, l) : acc.A0(g, l)) * wt;
      }
    }
  }
}

__device__ __forceinline__ void load3(const double* __restrict__ p, int64_t np, int64_t i,
                                      double* o) {
  o[0] = p[i];
  o[1] = p[np + i];
  o[2] = p[2 * np + i];
}

// ---- kernels ---------------------------------------------------------------

template <class T>
__global__ __launch_bounds__(kBlock) void k_extrapolate(int64_t n3, const T* __restrict__ v,
                                                       const T* __restrict__ vprev,
                                                       double* __restrict__ vit,
                                                       double* __restrict__ vbar) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n3) return;
  const double w = 2.0 * (double)v[i] - (double)vprev[i];  // v^{n+1,0} = 2 v^n - v^{n-1}
  vit[i] = w;
  if (vbar) vbar[i] = 0.5 * (w + (double)v[i]);
}

// Orbit current of P.chunk particles per block.  The lanes are spread over a
// span of P.span >= P.chunk consecutive sorted particles (chunk_particle), so
// that the 64 lanes of a wavefront sit in different cells and their LDS
// additions rarely hit the same address; P.span / P.chunk blocks interleave over
// one span.  How long both are: auto_span and auto_chunk in api.hip.
// Pass 1 finds the box of nodes the block's orbits touch (unwrapped indices
// relative to its first particle); where that box exceeds the tile (thermal plasmas: the fastest particle of a block
// sets it), the box of the block's start stencils, widened by as many nodes as
// fit, takes its place.  Pass 2 accumulates the current in an LDS tile over
// that box; the tile is then flushed with one global atomic per non-zero node
// value.  Pieces outside the box go straight to global memory, as does every
// piece of a block whose start stencils alone exceed the tile (unsorted
// particles).
// The LDS serves the 64-bit additions of 16 neighbouring lanes at a time, one
// per bank pair.  64 lanes one cell apart sit in a 4x4x4 block of cells (the
// sort's order); lane l takes segment 4 (l % 16) + l / 16 of the chunk, so that
// 16 neighbouring lanes are four cells apart in the order, and the tile's rows
// are padded (TileStrides) so that such lanes rarely share a bank pair.
constexpr int kScatterNodes = 3072;  // 72 KB: two blocks share a CU

struct TileStrides {
  int sy, sx;  // slots between neighbours along y and x; along z 1
  // sy = 0 mod 16 and sx = 4 mod 16, at least dz and dy sy
  __device__ __forceinline__ TileStrides(int dy, int dz)
      : sy((dz + 15) & ~15), sx(dy * sy + 4) {}
};

// Extra nodes per side, at most 4, by which a box of extents dim can grow and
// still fit `nodes` slots; -1 if it does not fit as it is.
__device__ __forceinline__ int plain_slack(const int* dim, int nodes) {
  // each extent is bounded first so that the products cannot overflow
  if (!(dim[0] > 0 && dim[0] <= nodes && dim[1] <= nodes && dim[2] <= nodes)) return -1;
  int e = -1;
  while (e < 4 && (int64_t)(dim[0] + 2 * e + 2) * (dim[1] + 2 * e + 2) * (dim[2] + 2 * e + 2) <=
                      nodes)
    ++e;
  return e;
}

// The same for the scatter tile with its padded rows.
__device__ __forceinline__ int box_slack(const int* dim) {
  if (!(dim[0] > 0 && dim[0] <= kScatterNodes && dim[1] <= kScatterNodes &&
        dim[2] <= kScatterNodes))
    return -1;
  int e = -1;
  while (e < 4) {
    const int g = 2 * (e + 1);
    const TileStrides s(dim[1] + g, dim[2] + g);
    if ((int64_t)(dim[0] + g) * s.sx > kScatterNodes) break;
    ++e;
  }
  return e;
}

// x^n, vbar^p = (v^{n+1,p} + v^n) / 2 and the unwrapped displacement
// d = dt vbar^p of particle i; vbar^p read from vbar when the previous pass
// (or the step's set-up) wrote it, else formed from v^n and the iterate
template <class PS>
__device__ __forceinline__ void orbit_of(const StepParams& P, const PS& st,
                                         const double* __restrict__ vit,
                                         const double* __restrict__ vbar, int64_t i, double* x0,
                                         double* d, double* vb) {
  st.x_of(P.G, P.np, i, x0);
  if (vbar) {
    load3(vbar, P.np, i, vb);
  } else {
    double va[3], vi[3];
    st.v_of(P.np, i, va);
    load3(vit, P.np, i, vi);
#pragma unroll
    for (int a = 0; a < 3; ++a) vb[a] = 0.5 * (vi[a] + va[a]);
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) d[a] = P.dt * vb[a];
}

// Fixed-point quantum count of a current contribution w: the product
// w x scale rounded once to the nearest integer (ties to even), as the
// two's-complement bit pattern that 64-bit integer atomics add.  Adding
// 1.5 x 2^52 in the same fused operation leaves that integer in the low
// mantissa bits of the sum while the sum stays in (2^52, 2^53), which holds
// for |w scale| < 2^50: one FMA and one 64-bit subtraction in place of a
// rounding and a software FP64 -> int64 conversion.  The caller guarantees
// the range (the scatter checks it once per particle and flags a particle
// outside it).
__device__ __forceinline__ unsigned long long quantize_in_range(double w, double scale) {
  constexpr double kMagic = 0x1.8p52;
  const double t = fma(w, scale, kMagic);
  return (unsigned long long)(__double_as_longlong(t) - __double_as_longlong(kMagic));
}

// Bound on |w scale| for quantize_in_range.  The orbit weights of a piece
// are at most 1, so a particle whose |c_l| scale stays below it has every
// contribution in range.
constexpr double kFixedRange = 0x1p50;

// The same rounding for any w (a conversion outside the range).
__device__ __forceinline__ unsigned long long quantize(double w, double scale) {
  if (fabs(w) * scale < kFixedRange) return quantize_in_range(w, scale);
  return (unsigned long long)(long long)rint(w * scale);
}

// The node box of a scatter block's chunk (first particle `base`): reference
// cell sref (that of the first particle), origin tlo relative to it and extents
// dim, per axis, block-uniform; taken from bx when an earlier pass of the step
// stored it.  index(k), k < per_thread, are the thread's particles; slack(dim)
// is the number of nodes by which a box can grow on every side and still fit
// the kernel's tile, negative if it does not fit.
// crossed(k, n): called there for each of them with the knots that its orbit crosses.
template <int R, class PS, class Index, class Slack, class Crossed>
__device__ __forceinline__ void scatter_box(const StepParams& P, const PS& st,
                                            const double* __restrict__ vit,
                                            const double* __restrict__ vbar, const ChunkBoxes& bx,
                                            int64_t base, int per_thread,
                                            Index&& index, Slack&& slack, Crossed&& crossed,
                                            int (&sref)[3], int (&tlo)[3], int (&dim)[3]) {
  constexpr int W = R + 1;
  __shared__ int s_ref[3];
  if (bx.reuse) {  // found by this chunk in the step's first pass
    const int* b = bx.box + (int64_t)blockIdx.x * kBoxInts;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      sref[a] = b[a];
      tlo[a] = b[3 + a];
      dim[a] = b[6 + a];
    }
  } else {
    if (threadIdx.x == 0) {
      double x0[3];
      st.x_of(P.G, P.np, min(base, P.np - 1), x0);  // a span's last blocks may be empty
#pragma unroll
      for (int a = 0; a < 3; ++a)
        s_ref[a] = to_int_clamped(floor(x0[a] * P.G.invH[a] + Spline<R>::base_off));
    }
    __syncthreads();
#pragma unroll
    for (int a = 0; a < 3; ++a) sref[a] = s_ref[a];
    // pass 1: the boxes of the nodes the chunk's orbits touch and (cmin, cmax)
    // of those its start stencils touch
    int rmin[3] = {0x3fffffff, 0x3fffffff, 0x3fffffff};
    int rmax[3] = {-0x3fffffff, -0x3fffffff, -0x3fffffff};
    int cmin[3] = {0x3fffffff, 0x3fffffff, 0x3fffffff};
    int cmax[3] = {-0x3fffffff, -0x3fffffff, -0x3fffffff};
    for (int k = 0; k < per_thread; ++k) {
      const int64_t i = index(k);
      if (i >= P.np) {
        crossed(k, 0);
        continue;
      }
      double x0[3], d[3], vb[3];
      orbit_of(P, st, vit, vbar, i, x0, d, vb);
      int knots = 0;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        int lo, n, b0;
        orbit_nodes<R>(x0[a], d[a], P.G.invH[a], lo, n, b0);
        const int rel = min_image(lo - sref[a], P.G.n[a]);
        rmin[a] = min(rmin[a], rel);
        rmax[a] = max(rmax[a], rel + n);
        cmin[a] = min(cmin[a], rel + (b0 - lo));
        cmax[a] = max(cmax[a], rel + (b0 - lo) + W);
        knots += min(knots_crossed(x0[a], d[a], P.G.invH[a], Spline<R>::base_off), kMaxPieces);
      }
      crossed(k, knots);
    }
    int mv[12] = {rmin[0], rmin[1], rmin[2], -rmax[0], -rmax[1], -rmax[2],
                  cmin[0], cmin[1], cmin[2], -cmax[0], -cmax[1], -cmax[2]};
    block_min_ints<12>(mv);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      tlo[a] = mv[a];
      dim[a] = -mv[3 + a] - tlo[a] + 1;
    }
    if (slack(dim) < 0) {
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        tlo[a] = mv[6 + a];
        dim[a] = -mv[9 + a] - tlo[a] + 1;
      }
      const int e = max(slack(dim), 0);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        tlo[a] -= e;
        dim[a] += 2 * e;
      }
    }
    if (bx.box && threadIdx.x == 0) {
      int* b = bx.box + (int64_t)blockIdx.x * kBoxInts;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        b[a] = sref[a];
        b[3 + a] = tlo[a];
        b[6 + a] = dim[a];
      }
    }
  }
#pragma unroll
  for (int a = 0; a < 3; ++a) {  // block-uniform
    sref[a] = __builtin_amdgcn_readfirstlane(sref[a]);
    tlo[a] = __builtin_amdgcn_readfirstlane(tlo[a]);
    dim[a] = __builtin_amdgcn_readfirstlane(dim[a]);
  }
}

// MULTI: the particles carry species (one byte each); otherwise every
// particle has the coefficients of species 0, kept in scalar registers
template <int R, class PS, bool SPLIT, bool MULTI>
__global__ __launch_bounds__(kBlock) __attribute__((
    amdgpu_waves_per_eu(2))) void k_scatter(StepParams P, PS st,
                                                   const double* __restrict__ vit,
                                                   const double* __restrict__ vbar,
                                                   CurrentOut out, Scratch sc,
                                                   ChunkBoxes bx) {
  constexpr int W = R + 1;
  constexpr bool FIX = PS::kMixed;  // int64 fixed-point deposit
  __shared__ double tile[3 * kScatterNodes];  // FIX: int64 quanta in the same bytes
  unsigned long long* tile_q = reinterpret_cast<unsigned long long*>(tile);
  const int per_thread = P.chunk / kBlock;  // at most 16
  const int block = P.by_xcd ? xcd_block(blockIdx.x, gridDim.x) : blockIdx.x;
  const int64_t base = chunk_base(P.chunk, P.span, block);
  // The order of the particles of a lane (see ChunkBoxes): candidates r = 0 ..
  // per_lane - 1 of its segment, the one of place p to slot p / kWaves of wavefront
  // p % kWaves.  The counts lie in the tile, not in use yet, in rows padded against
  // bank conflicts.
  constexpr int kWaves = kBlock / kWave;
  const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
  const int per_lane = P.chunk / kWave, lane_row = lane * (per_lane + 4);
  uint8_t* lane_knots = reinterpret_cast<uint8_t*>(tile);
  uint8_t* lane_order = bx.lane_order + (int64_t)blockIdx.x * P.chunk;
  double js[1] = {0.0};
  double bad = 0.0;
  late_reduce_init<2>();
  int sref[3], tlo[3], dim[3];
  scatter_box<R>(P, st, vit, vbar, bx, base, per_thread,
                 [&](int k) { return chunk_particle(base, P.span, k); },
                 [](const int* d) { return box_slack(d); },
                 [&](int k, int n) {
                   if (SPLIT && bx.lane_order) lane_knots[lane_row + wid + kWaves * k] = (uint8_t)n;
                 },
                 sref, tlo, dim);
  if (SPLIT && bx.lane_order && !bx.reuse) {
    for (int k = 0; k < per_thread; ++k) {
      const int own = wid + kWaves * k, n = lane_knots[lane_row + own];
      int place = 0;
      for (int r = 0; r < per_lane; ++r) {
        const int m = lane_knots[lane_row + r];
        place += m > n || (m == n && r < own) ? 1 : 0;
      }
      lane_order[((place % kWaves) * kWave + lane) * per_thread + place / kWaves] = (uint8_t)own;
    }
    __syncthreads();
  }
  auto particle = [&](int k) {
    if (!(SPLIT && bx.lane_order)) return chunk_particle(base, P.span, k);
    return chunk_particle(base, P.span, 0) - wid + lane_order[(int)threadIdx.x * per_thread + k];
  };
  const bool use_tile = box_slack(dim) >= 0;  // block-uniform
  const TileStrides ts(dim[1], dim[2]);
  const int nt = use_tile ? dim[0] * ts.sx : 0;
  for (int t = threadIdx.x; t < 3 * nt; t += kBlock) tile[t] = 0.0;  // also integer zero
  __syncthreads();
  // pass 2: accumulate.  Pieces whose stencil lies outside the tile are
  // skipped and their particles marked; a third pass adds those pieces to
  // global memory.  Keeping the global path out of the main loop keeps the
  // loop's register count (and so the kernel's occupancy) that of the tile path.
  const int64_t nc = P.G.ncell;
  unsigned outside_mask = 0u;
  auto process = [&](int k, auto global_phase) -> bool {
    constexpr bool GLOBAL = decltype(global_phase)::value;
    bool outside = false;
    const int64_t i = particle(k);
    if (i >= P.np) return false;
    double x0[3], d[3], vb[3], c3[3];
    orbit_of(P, st, vit, vbar, i, x0, d, vb);
    if (!GLOBAL) {  // J_s: q_i max_a |vbar_a|, once per particle
      const double vmax = fmax(fabs(vb[0]), fmax(fabs(vb[1]), fabs(vb[2])));
      js[0] += (MULTI ? species_value(P.aq, st.species(i)) : P.aq[0]) * vmax;
    }
    // FP64: q_i vbar / dV; fixed point: (q_i / q_0) vbar in units of the quantum
    const double cq = MULTI ? species_value(P.cq, st.species(i)) : P.cq[0];
    int shift[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      c3[a] = cq * vb[a];
      int lo, n, b0;
      orbit_nodes<R>(x0[a], d[a], P.G.invH[a], lo, n, b0);
      const int raw = lo - sref[a];
      shift[a] = min_image(raw, P.G.n[a]) - raw;  // particle frame -> chunk frame
    }
    auto deposit = [&](const double (&Iw)[W][W][W], const int* f) {
      const int ox = f[0] - sref[0] + shift[0] - tlo[0];
      const int oy = f[1] - sref[1] + shift[1] - tlo[1];
      const int oz = f[2] - sref[2] + shift[2] - tlo[2];
      const bool inside = use_tile && ox >= 0 && oy >= 0 && oz >= 0 && ox + W <= dim[0] &&
                          oy + W <= dim[1] && oz + W <= dim[2];
      outside = outside || !inside;
      if (!GLOBAL && inside) {
#pragma unroll
        for (int a = 0; a < W; ++a)
#pragma unroll
          for (int b = 0; b < W; ++b)
#pragma unroll
            for (int c = 0; c < W; ++c) {
              const int t = (ox + a) * ts.sx + (oy + b) * ts.sy + (oz + c);
              const double w = Iw[a][b][c];
#pragma unroll
              for (int l = 0; l < 3; ++l) {
                if constexpr (FIX)
                  atomicAdd(&tile_q[3 * t + l], quantize_in_range(w * c3[l], out.fix_scale));
                else
                  atomicAdd(&tile[3 * t + l], w * c3[l]);
              }
            }
      } else if (GLOBAL && !inside) {
#pragma unroll
        for (int a = 0; a < W; ++a)
#pragma unroll
          for (int b = 0; b < W; ++b)
#pragma unroll
            for (int c = 0; c < W; ++c) {
              const int64_t g = node_index(P.G, f[0] + a, f[1] + b, f[2] + c);
              const double w = Iw[a][b][c];
#pragma unroll
              for (int l = 0; l < 3; ++l) {
                if constexpr (FIX)
                  atomicAdd(out.Jfix + l * nc + g, quantize_in_range(w * c3[l], out.fix_scale));
                else
                  unsafeAtomicAdd(out.J + l * nc + g, w * c3[l]);
              }
            }
      }
    };
    // Cubic stencils (64 nodes): the weights are never held all at once.
    // Per quadrature point the three 1-D factors are kept (wq folded into the
    // x factor); each node's weight is summed over the points when it is
    // deposited.  Same integrals, a quarter of the registers.
    auto deposit_factored = [&](const double (&X)[Quad<R>::NQ][W],
                                const double (&Y)[Quad<R>::NQ][W],
                                const double (&Z)[Quad<R>::NQ][W], const int* f) {
      constexpr int NQ = Quad<R>::NQ;
      const int ox = f[0] - sref[0] + shift[0] - tlo[0];
      const int oy = f[1] - sref[1] + shift[1] - tlo[1];
      const int oz = f[2] - sref[2] + shift[2] - tlo[2];
      const bool inside = use_tile && ox >= 0 && oy >= 0 && oz >= 0 && ox + W <= dim[0] &&
                          oy + W <= dim[1] && oz + W <= dim[2];
      outside = outside || !inside;
      if (GLOBAL == inside) return;
#pragma unroll
      for (int a = 0; a < W; ++a)
#pragma unroll
        for (int b = 0; b < W; ++b) {
          double xy[NQ];
#pragma unroll
          for (int q = 0; q < NQ; ++q) xy[q] = X[q][a] * Y[q][b];
#pragma unroll
          for (int c = 0; c < W; ++c) {
            double w = 0.0;
#pragma unroll
            for (int q = 0; q < NQ; ++q) w += xy[q] * Z[q][c];
            if (!GLOBAL) {
              const int t = (ox + a) * ts.sx + (oy + b) * ts.sy + (oz + c);
#pragma unroll
              for (int l = 0; l < 3; ++l) {
                if constexpr (FIX)
                  atomicAdd(&tile_q[3 * t + l], quantize_in_range(w * c3[l], out.fix_scale));
                else
                  atomicAdd(&tile[3 * t + l], w * c3[l]);
              }
            } else {
              const int64_t g = node_index(P.G, f[0] + a, f[1] + b, f[2] + c);
#pragma unroll
              for (int l = 0; l < 3; ++l) {
                if constexpr (FIX)
                  atomicAdd(out.Jfix + l * nc + g, quantize_in_range(w * c3[l], out.fix_scale));
                else
                  unsafeAtomicAdd(out.J + l * nc + g, w * c3[l]);
              }
            }
          }
        }
    };
    bool ok = true;
    if constexpr (SPLIT && R >= 3) {
      ok = for_each_piece<R>(x0, d, P.G, [&](double s0, double s1, const double* base) {
        constexpr int NQ = Quad<R>::NQ;
        double sq[NQ], wq[NQ], X[NQ][W], Y[NQ][W], Z[NQ][W];
        int f[3];
        piece_rule<R>(s0, s1, sq, wq);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          const double sv = sq[q];
          Spline<R>::w((x0[0] + sv * d[0]) * P.G.invH[0] - base[0], X[q]);
          Spline<R>::w((x0[1] + sv * d[1]) * P.G.invH[1] - base[1], Y[q]);
          Spline<R>::w((x0[2] + sv * d[2]) * P.G.invH[2] - base[2], Z[q]);
#pragma unroll
          for (int a = 0; a < W; ++a) X[q][a] *= wq[q];
        }
#pragma unroll
        for (int a = 0; a < 3; ++a) f[a] = to_int_clamped(base[a]) + Spline<R>::first_off;
        deposit_factored(X, Y, Z, f);
      });
    } else if constexpr (SPLIT) {
      // One x slice of the stencil at a time: the point sums of its 3 x 3 nodes
      // are deposited before the next slice's are formed, so only 9 weights
      // are live (the same sums, in the same order, as the whole stencil's).
      ok = for_each_piece<R>(x0, d, P.G, [&](double s0, double s1, const double* base) {
        constexpr int NQ = Quad<R>::NQ;
        double sq[NQ], wq[NQ], tx[NQ], Y[NQ][W], Z[NQ][W];
        piece_rule<R>(s0, s1, sq, wq);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          tx[q] = (x0[0] + sq[q] * d[0]) * P.G.invH[0] - base[0];
          Spline<R>::w((x0[1] + sq[q] * d[1]) * P.G.invH[1] - base[1], Y[q]);
          Spline<R>::w((x0[2] + sq[q] * d[2]) * P.G.invH[2] - base[2], Z[q]);
        }
        int f[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) f[a] = to_int_clamped(base[a]) + Spline<R>::first_off;
        const int ox = f[0] - sref[0] + shift[0] - tlo[0];
        const int oy = f[1] - sref[1] + shift[1] - tlo[1];
        const int oz = f[2] - sref[2] + shift[2] - tlo[2];
        const bool inside = use_tile && ox >= 0 && oy >= 0 && oz >= 0 && ox + W <= dim[0] &&
                            oy + W <= dim[1] && oz + W <= dim[2];
        outside = outside || !inside;
        if (GLOBAL == inside) return;
#pragma unroll
        for (int a = 0; a < W; ++a) {
          double Ia[W][W];
#pragma unroll
          for (int b = 0; b < W; ++b)
#pragma unroll
            for (int c = 0; c < W; ++c) Ia[b][c] = 0.0;
#pragma unroll
          for (int q = 0; q < NQ; ++q) {
            double Xq, dXq;
            Spline<R>::wk(a, tx[q], Xq, dXq);
            const double xa = wq[q] * Xq;
#pragma unroll
            for (int b = 0; b < W; ++b) {
              const double xy = xa * Y[q][b];
#pragma unroll
              for (int c = 0; c < W; ++c) Ia[b][c] += xy * Z[q][c];
            }
          }
#pragma unroll
          for (int b = 0; b < W; ++b)
#pragma unroll
            for (int c = 0; c < W; ++c) {
              const double w = Ia[b][c];
              if (!GLOBAL) {
                const int t = (ox + a) * ts.sx + (oy + b) * ts.sy + (oz + c);
#pragma unroll
                for (int l = 0; l < 3; ++l) {
                  if constexpr (FIX)
                    atomicAdd(&tile_q[3 * t + l], quantize_in_range(w * c3[l], out.fix_scale));
                  else
                    atomicAdd(&tile[3 * t + l], w * c3[l]);
                }
              } else {
                const int64_t g = node_index(P.G, f[0] + a, f[1] + b, f[2] + c);
#pragma unroll
                for (int l = 0; l < 3; ++l) {
                  if constexpr (FIX)
                    atomicAdd(out.Jfix + l * nc + g, quantize_in_range(w * c3[l], out.fix_scale));
                  else
                    unsafeAtomicAdd(out.J + l * nc + g, w * c3[l]);
                }
              }
            }
        }
      });
    } else {
      for (int q = 0; q < P.rule.n; ++q) {
        double base[3], sq, wq, Iw[W][W][W];
        int f[3];
        unsplit_point<R>(P.G, P.rule, q, x0, d, base, sq, wq);
        sbar_points<R, 1>(P.G, x0, d, base, &sq, &wq, Iw, f);
        deposit(Iw, f);
      }
    }
    if (!ok && !GLOBAL) bad = 1.0;
    if constexpr (FIX) {  // contributions beyond the fixed-point range
      const double cmax = fmax(fabs(c3[0]), fmax(fabs(c3[1]), fabs(c3[2])));
      if (!GLOBAL && !(cmax * out.fix_scale < kFixedRange)) bad = fmax(bad, 1.5);
    }
    return outside;
  };
  for (int k = 0; k < per_thread; ++k)
    if (process(k, std::false_type{})) outside_mask |= 1u << k;
  for (int k = 0; k < per_thread; ++k)
    if ((outside_mask >> k) & 1u) process(k, std::true_type{});
  __syncthreads();
  // padding slots stay zero
  const float inv_sx = 1.0f / (float)ts.sx, inv_sy = 1.0f / (float)ts.sy;
  for (int t = threadIdx.x; t < nt; t += kBlock) {
    const int cx = div_small(t, inv_sx), yz = t - cx * ts.sx;
    const int cy = div_small(yz, inv_sy), cz = yz - cy * ts.sy;
    const int64_t g = node_index(P.G, sref[0] + tlo[0] + cx, sref[1] + tlo[1] + cy,
                                 sref[2] + tlo[2] + cz);
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      if constexpr (FIX) {
        const unsigned long long val = tile_q[3 * t + l];
        if (val != 0ull) atomicAdd(out.Jfix + l * nc + g, val);
      } else {
        const double val = tile[3 * t + l];
        if (val != 0.0) unsafeAtomicAdd(out.J + l * nc + g, val);
      }
    }
  }
  const double part[2] = {js[0], bad};
  const bool ismax[2] = {false, true};
  double blk[2];
  if (late_reduce<2>(part, ismax, blk)) {
    sc.region(P_JS)[blockIdx.x] = blk[0];  // J_s partials, summed in order by k_finish
    atomic_max_nonneg(sc.spread_copy(S_BAD), blk[1]);
  }
}

// The FP64 current of dense plasmas by matrix instructions (degree 2; when it is
// taken: use_scatter_mm in api.hip).  In the kernel
// above every orbit piece takes 3 (r+1)^3 LDS additions per lane, and those
// bound it.  Consecutive sorted particles share their stencils (the sort's
// key is the base node of the first piece), and for particles of one stencil
// the current is a product,
//   J[node][l] += sum_i Sbar[node][i] c[i][l],   c = q vbar / dV,
// summed over the particles.  A wavefront therefore takes 64 consecutive
// particles at a time, forms the weights of one piece of each, groups the
// lanes by stencil, and hands the weights through LDS to
// v_mfma_f64_4x4x4: its four blocks are 16 stencil nodes, its K four particles
// of one group, its columns the three current components (the fourth is not
// used).  The products of a group stay in one register pair per lane and go to
// the block's LDS tile with one addition per node and component.  One x slice
// of the stencil ((r+1)^2 <= 16 nodes) is handled at a time.
// Pieces outside the tile go to global memory particle by particle, after the
// main loop.
constexpr int kMmNodes = 1024;              // 24 KB tile
constexpr int kMmStride = kWave + 1;        // slots of a row of the weight buffer: odd, so
                                            // 16 rows read at one slot use 16 bank pairs
// slots of a wavefront's weight buffer: (r+1)^2 rows of weights, 3 of current
// components; the last reads of a group may reach 15 slots past the last row
template <int R>
constexpr int kMmBuf = ((R + 1) * (R + 1) + 3) * kMmStride + 16;

template <int R, bool MULTI>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3))) void k_scatter_mm(
    StepParams P, Fp64Store st, const double* __restrict__ vit, const double* __restrict__ vbar,
    double* __restrict__ J, Scratch sc, ChunkBoxes bx) {
  constexpr int W = R + 1, NQ = Quad<R>::NQ, kRows = W * W;
  __shared__ double tile[3 * kMmNodes];
  __shared__ double wbuf[kBlock / kWave][kMmBuf<R>];
  const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
  const int run = P.chunk / (kBlock / kWave);  // consecutive particles per wavefront
  const int64_t base = (int64_t)blockIdx.x * P.chunk;
  double js[1] = {0.0};
  double bad = 0.0;
  int turns = 0;  // of this wavefront: groups, and pieces outside the tile
  late_reduce_init<2>();
  int sref[3], tlo[3], dim[3];
  scatter_box<R>(P, st, vit, vbar, bx, base, P.chunk / kBlock,
                 [&](int k) { return base + wid * run + k * kWave + lane; },
                 [](const int* d) { return plain_slack(d, kMmNodes); }, [](int, int) {}, sref,
                 tlo, dim);
  const bool use_tile = plain_slack(dim, kMmNodes) >= 0;  // block-uniform
  const int sy = dim[2], sx = dim[1] * dim[2], nt = use_tile ? dim[0] * sx : 0;
  for (int t = threadIdx.x; t < 3 * nt; t += kBlock) tile[t] = 0.0;
  double* wb = wbuf[wid];
  for (int t = lane; t < kMmBuf<R>; t += kWave) wb[t] = 0.0;
  __syncthreads();
  // operand positions of this lane: A row = lane % 16, B column = lane % 4,
  // K index = lane / 16; result row 4 ((lane / 4) % 4) + lane / 16, column lane % 4
  const int kk = lane >> 4, col = lane & 3;
  const double* wa = wb + min(lane & 15, kRows - 1) * kMmStride + kk;
  const double* wc = wb + (kRows + min(col, 2)) * kMmStride + kk;
  const int row = 4 * ((lane >> 2) & 3) + kk;
  const bool out_lane = row < kRows && col < 3;
  double* tout = tile + 3 * ((row / W) * sy + row % W) + col;
  unsigned outside_mask = 0u;
  for (int it = 0; it * kWave < run; ++it) {
    const int64_t i = base + wid * run + it * kWave + lane;
    bool live = i < P.np;
    if (__ballot(live) == 0ull) break;
    double x0[3] = {0.0, 0.0, 0.0}, d[3] = {0.0, 0.0, 0.0}, c3[3] = {0.0, 0.0, 0.0};
    int off[3];  // particle frame -> tile
    if (live) {
      double vb[3];
      orbit_of(P, st, vit, vbar, i, x0, d, vb);
      const double vmax = fmax(fabs(vb[0]), fmax(fabs(vb[1]), fabs(vb[2])));
      const int sp = MULTI ? st.species(i) : 0;
      js[0] += (MULTI ? species_value(P.aq, sp) : P.aq[0]) * vmax;
      const double cq = MULTI ? species_value(P.cq, sp) : P.cq[0];
#pragma unroll
      for (int a = 0; a < 3; ++a) c3[a] = cq * vb[a];
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      int lo, n, b0;
      orbit_nodes<R>(x0[a], d[a], P.G.invH[a], lo, n, b0);
      const int raw = lo - sref[a];
      off[a] = min_image(raw, P.G.n[a]) - raw - sref[a] - tlo[a] + Spline<R>::first_off;
    }
    Crossings<R> cr;
    cr.init(x0, d, P.G);
    double s0 = 0.0;
    bool outside = false;
    for (int piece = 0; piece < kMaxPieces; ++piece) {
      if (__ballot(live) == 0ull) break;
      const double s1 = cr.next();
      const int ox = cr.base[0] + off[0], oy = cr.base[1] + off[1], oz = cr.base[2] + off[2];
      const bool inside = use_tile && ox >= 0 && oy >= 0 && oz >= 0 && ox + W <= dim[0] &&
                          oy + W <= dim[1] && oz + W <= dim[2];
      const bool has = live && s1 > s0;
      outside = outside || (has && !inside);
      const bool dep = has && inside;
      const int t0 = ox * sx + oy * sy + oz;
      // groups of lanes with one stencil, in consecutive slots; lane g keeps
      // group g's stencil, first slot and size
      unsigned long long todo = __ballot(dep);
      int ngroups = 0, filled = 0, slot = 0, gt = 0, gp = 0, gn = 0;
      while (todo) {
        const int leader = __ffsll((long long)todo) - 1;
        const int tl = __builtin_amdgcn_readlane(t0, leader);
        const unsigned long long grp = __ballot(t0 == tl) & todo;
        const int n = __popcll(grp);
        if ((grp >> lane) & 1ull)
          slot = filled + __builtin_amdgcn_mbcnt_hi((unsigned)(grp >> 32),
                                                    __builtin_amdgcn_mbcnt_lo((unsigned)grp, 0u));
        if (lane == ngroups) {
          gt = tl;
          gp = filled;
          gn = n;
        }
        ++ngroups;
        filled += n;
        todo &= ~grp;
      }
      turns += ngroups + __popcll(__ballot(has && !inside));
      if (ngroups > 0) {
        double sq[NQ], wq[NQ], tx[NQ], Y[NQ][W], Z[NQ][W];
        piece_rule<R>(s0, s1, sq, wq);
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
          tx[q] = (x0[0] + sq[q] * d[0]) * P.G.invH[0] - (double)cr.base[0];
          Spline<R>::w((x0[1] + sq[q] * d[1]) * P.G.invH[1] - (double)cr.base[1], Y[q]);
          Spline<R>::w((x0[2] + sq[q] * d[2]) * P.G.invH[2] - (double)cr.base[2], Z[q]);
        }
        if (dep)
#pragma unroll
          for (int l = 0; l < 3; ++l) wb[(kRows + l) * kMmStride + slot] = c3[l];
#pragma unroll
        for (int a = 0; a < W; ++a) {
          double Ia[W][W];
#pragma unroll
          for (int b = 0; b < W; ++b)
#pragma unroll
            for (int c = 0; c < W; ++c) Ia[b][c] = 0.0;
#pragma unroll
          for (int q = 0; q < NQ; ++q) {
            double Xq, dXq;
            Spline<R>::wk(a, tx[q], Xq, dXq);
            const double xa = wq[q] * Xq;
#pragma unroll
            for (int b = 0; b < W; ++b) {
              const double xy = xa * Y[q][b];
#pragma unroll
              for (int c = 0; c < W; ++c) Ia[b][c] += xy * Z[q][c];
            }
          }
          // a wavefront's LDS operations complete in order: the fences only
          // keep the compiler from moving them across each other
          __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
          if (dep)
#pragma unroll
            for (int b = 0; b < W; ++b)
#pragma unroll
              for (int c = 0; c < W; ++c) wb[(b * W + c) * kMmStride + slot] = Ia[b][c];
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
          for (int g = 0; g < ngroups; ++g) {
            const int tg = __builtin_amdgcn_readlane(gt, g);
            const int p = __builtin_amdgcn_readlane(gp, g), n = __builtin_amdgcn_readlane(gn, g);
            double acc = 0.0;
            for (int j = 0; j < n; j += 8) {  // two products, their operands read together
              double A[2], B[2];
#pragma unroll
              for (int u = 0; u < 2; ++u) {
                A[u] = wa[p + j + 4 * u];
                const double cv = wc[p + j + 4 * u];
                B[u] = j + 4 * u + kk < n ? cv : 0.0;
              }
#pragma unroll
              for (int u = 0; u < 2; ++u)
                acc = __builtin_amdgcn_mfma_f64_4x4x4f64(A[u], B[u], acc, 0, 0, 0);
            }
            if (out_lane) atomicAdd(tout + 3 * (tg + a * sx), acc);
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
        }
      }
      if (s1 >= 1.0) live = false;
      cr.consume(s1);
      s0 = s1;
    }
    if (live) bad = 1.0;  // more than kMaxPieces pieces
    if (outside) outside_mask |= 1u << it;
  }
  for (int it = 0; it * kWave < run; ++it) {
    if (!((outside_mask >> it) & 1u)) continue;
    const int64_t i = base + wid * run + it * kWave + lane;
    double x0[3], d[3], vb[3], c3[3];
    orbit_of(P, st, vit, vbar, i, x0, d, vb);
    const double cq = MULTI ? species_value(P.cq, st.species(i)) : P.cq[0];
    int off[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      c3[a] = cq * vb[a];
      int lo, n, b0;
      orbit_nodes<R>(x0[a], d[a], P.G.invH[a], lo, n, b0);
      const int raw = lo - sref[a];
      off[a] = min_image(raw, P.G.n[a]) - raw - sref[a] - tlo[a] + Spline<R>::first_off;
    }
    for_each_piece<R>(x0, d, P.G, [&](double s0, double s1, const double* bs) {
      const int ox = (int)bs[0] + off[0], oy = (int)bs[1] + off[1], oz = (int)bs[2] + off[2];
      const bool inside = use_tile && ox >= 0 && oy >= 0 && oz >= 0 && ox + W <= dim[0] &&
                          oy + W <= dim[1] && oz + W <= dim[2];
      if (!inside) scatter_piece<R>(P.G, x0, d, s0, s1, bs, c3, J);
    });
  }
  __syncthreads();
  const int64_t nc = P.G.ncell;
  const float inv_sx = 1.0f / (float)max(sx, 1), inv_sy = 1.0f / (float)max(sy, 1);
  for (int t = threadIdx.x; t < nt; t += kBlock) {
    const int cx = div_small(t, inv_sx), yz = t - cx * sx;
    const int cy = div_small(yz, inv_sy), cz = yz - cy * sy;
    const int64_t g = node_index(P.G, sref[0] + tlo[0] + cx, sref[1] + tlo[1] + cy,
                                 sref[2] + tlo[2] + cz);
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      const double val = tile[3 * t + l];
      if (val != 0.0) unsafeAtomicAdd(J + l * nc + g, val);
    }
  }
  if (lane == 0) unsafeAtomicAdd(sc.spread_copy(S_GROUPS), (double)turns);
  const double part[2] = {js[0], bad};
  const bool ismax[2] = {false, true};
  double blk[2];
  if (late_reduce<2>(part, ismax, blk)) {
    sc.region(P_JS)[blockIdx.x] = blk[0];  // J_s partials, summed in order by k_finish
    atomic_max_nonneg(sc.spread_copy(S_BAD), blk[1]);
  }
}

// Gather + push of one particle (index i of store st) through accessor acc:
// grad phi-bar and (D A)^T vbar over the orbit pieces, then P^{n+1,p} and
// v^{n+1,p+1}.  The orbit loop sets the kernel's register count, so nothing that
// can be had again is kept through it: v^n and the species are read after it,
// and x0, d and i are hidden from the compiler there, which would otherwise
// carry cell coordinates and addresses formed before the loop to their uses
// behind it (28 spilled registers, 0.35 against 0.28 ms per pass at 32^3).
// With LANES = 4 the quad's lanes all end with the particle's v^{n+1,p+1}.
template <int R, bool SPLIT, int LANES, class Acc, class PS>
__device__ __forceinline__ void gather_push_one(const StepParams& P, const Acc& acc, const PS& st,
                                                int part, int& i, double (&x0)[3],
                                                double (&d)[3], const double (&vb)[3],
                                                const double* __restrict__ vit, double* vn,
                                                double (&va)[3], double (&vi)[3],
                                                double& npieces, double& bad) {
  double gp[3] = {0.0, 0.0, 0.0};
  double dtv[3] = {0.0, 0.0, 0.0};  // H_j ((D A)^T vbar)_j until the pieces are summed
  if constexpr (SPLIT) {
    const bool ok = for_each_piece<R>(x0, d, P.G, [&](double s0, double s1, const double* base) {
      push_piece<R, LANES>(P.G, x0, d, s0, s1, base, vb, acc, part, gp, dtv);
      npieces += 1.0;
    });
    if (!ok) bad = 1.0;
  } else {
    for (int q = 0; q < P.rule.n; ++q) {
      double base[3], sq, wq;
      unsplit_point<R>(P.G, P.rule, q, x0, d, base, sq, wq);
      push_points<R, LANES, 1>(P.G, x0, d, base, &sq, &wq, vb, acc, part, gp, dtv);
    }
    npieces += 1.0;
  }
  asm volatile(""
               : "+v"(i), "+v"(x0[0]), "+v"(x0[1]), "+v"(x0[2]), "+v"(d[0]), "+v"(d[1]), "+v"(d[2])
               :
               : "memory");
  // A_h^n(x^n) rebuilds P^n = m v^n + q A_h^n(x^n) (eq. discrete-canonical-relation);
  // A_h^{n+1}(x^{n+1}) at the wrapped end point closes the velocity (eq. orbit-v-update).
  const int spc = st.species(i);
  const double qi = species_value(P.qs, spc), mi = species_value(P.ms, spc);
  st.v_of(P.np, i, va);
  // for the caller too, on its way while the interpolants are formed (read again
  // behind them: 0.5% more time per step at 2,097,152 and 33,554,432 particles)
  load3(vit, P.np, i, vi);
  double x1[3], A0s[3], A1e[3];
  int zero[3] = {0, 0, 0}, sh1[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    x1[a] = wrap_pos(x0[a] + d[a], P.G.L[a], P.G.invL[a]);
    sh1[a] = (int)rint((x0[a] + d[a] - x1[a]) * P.G.invL[a]) * P.G.n[a];
  }
  point_A_acc<R, LANES>(P.G, x0, zero, acc, 0, part, A0s);
  point_A_acc<R, LANES>(P.G, x1, sh1, acc, 1, part, A1e);
#pragma unroll
  for (int j = 0; j < 3; ++j) {
    if constexpr (LANES == 4) {
      gp[j] = quad_sum(gp[j]);
      dtv[j] = quad_sum(dtv[j]);
      A0s[j] = quad_sum(A0s[j]);
      A1e[j] = quad_sum(A1e[j]);
    }
    const double Pn = mi * va[j] + qi * A0s[j];
    const double DAv = dtv[j] * P.G.invH[j];                  // ((D A)^T vbar)_j
    const double P1 = Pn + P.dt * (-qi * gp[j] + qi * DAv);   // eq. orbit-P-update
    vn[j] = (P1 - qi * A1e[j]) / mi;                          // eq. orbit-v-update
  }
}

// Where a gather block reads the fields from.
//   GATHER_TILE  the block's LDS copy of the nodes its orbits touch
//   GATHER_MESH  an LDS copy of the whole mesh (meshes of at most
//                kGatherTileNodes nodes): no box to find, none to miss
//   GATHER_LIST  global memory, for the particles that GATHER_TILE listed
enum GatherFrom { GATHER_TILE, GATHER_MESH, GATHER_LIST };

// 78 KB of LDS: two blocks share a CU, as their registers would have it anyway
constexpr int kGatherTileNodes = 1000;

struct MeshGather {  // the whole mesh in LDS, nodes in flat order
  lds_cdouble* t;
  int mask0, mask1, mask2, shx, shy;
  __device__ __forceinline__ int row(int ix, int iy) const {
    return ((ix & mask0) << shx) | ((iy & mask1) << shy);
  }
  __device__ __forceinline__ lds_cdouble* node(int row, int iz) const {
    return t + (row | (iz & mask2)) * kGbufStride;
  }
};

// Maxima, counts and sums of a block's particles, taken wavefront by wavefront
// as they finish (no block barrier after the orbit loops: a wavefront with fewer
// pieces does not wait for the block's slowest one), so that they hold no
// registers through the orbit loops.
constexpr int kMaxGatherBatches = 4;
struct GatherTotals {
  unsigned long long dvm, vm, bad;  // bit patterns of non-negative doubles
  int pieces;
  double aa[kMaxGatherBatches * kBlock / kWave][2];  // one row per 64 particles (or wavefront)
  unsigned int done;
};

// The gather and push of one batch of 256 / LANES particles; i = particle (of the
// lane's quad, with four lanes each), or active false.  With inside(x0, d) false the lane's particle is left to the list.
template <int R, bool SPLIT, int LANES, class PS, class Acc, class Inside>
__device__ __forceinline__ void gather_batch(const StepParams& P, const PS& st, int i,
                                             bool active, const double* __restrict__ vit,
                                             double* __restrict__ vnew,
                                             double* __restrict__ vbar_out, Acc&& make_acc,
                                             Inside&& inside, const AndersonPrev& prev,
                                             GatherTotals& tot, int aa_sum) {
  double dvm = 0.0, vm = 0.0, bad = 0.0, npieces = 0.0;
  double aa[2] = {0.0, 0.0};
  const int part = LANES == 1 ? 0 : (int)threadIdx.x % LANES;
  if (active) {
    double x0[3], vb[3], d[3];
    {
      double va[3], vi[3];
      st.x_of(P.G, P.np, i, x0);
      st.v_of(P.np, i, va);
      load3(vit, P.np, i, vi);
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        vb[a] = 0.5 * (vi[a] + va[a]);
        d[a] = P.dt * vb[a];
      }
    }
    int shift[3];
    if (inside(i, x0, d, shift)) {
      double vn[3], va[3], vi[3];
      gather_push_one<R, SPLIT, LANES>(P, make_acc(shift), st, part, i, x0, d, vb, vit, vn, va, vi,
                                       npieces, bad);
      // vn is complete here: otherwise its y and z sums sink behind the branches
      // below and every field value they use stays in registers until then
      // (more than 200 spilled)
      asm volatile("" : "+v"(vn[0]), "+v"(vn[1]), "+v"(vn[2]), "+v"(i) : : "memory");
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        if (LANES == 1 || part == j) {
          vnew[j * P.np + i] = vn[j];
          if (vbar_out) vbar_out[j * P.np + i] = 0.5 * (vn[j] + va[j]);  // the next pass's vbar
        }
        dvm = fmax(dvm, fabs(vn[j] - vi[j]));
        vm = fmax(vm, fabs(vn[j]));
        if (!isfinite(vn[j])) bad = 2.0;  // max-reductions drop NaN: flag it explicitly
      }
      if (part != 0) npieces = 0.0;
      if (prev.w && part == 0) {  // Anderson mixing over one difference: dF . dF and dF . f_p
#pragma unroll
        for (int j = 0; j < 3; ++j) {
          const int64_t e = j * P.np + i;
          const double f0 = vn[j] - vi[j], df = f0 - (prev.g[e] - prev.w[e]);
          aa[0] += df * df;
          aa[1] += df * f0;
        }
      }
    }
  }
  dvm = wave_max(dvm);
  vm = wave_max(vm);
  bad = wave_max(bad);
  npieces = wave_sum(npieces);
  if (threadIdx.x % kWave == 0) {
    atomicMax(&tot.dvm, (unsigned long long)__double_as_longlong(dvm));
    atomicMax(&tot.vm, (unsigned long long)__double_as_longlong(vm));
    if (bad > 0.0) atomicMax(&tot.bad, (unsigned long long)__double_as_longlong(bad));
    atomicAdd(&tot.pieces, (int)npieces);
  }
  if (prev.w) {
    aa[0] = wave_sum(aa[0]);
    aa[1] = wave_sum(aa[1]);
    if (threadIdx.x % kWave == 0)
      for (int k = 0; k < 2; ++k) tot.aa[aa_sum][k] += aa[k];
  }
}

__device__ __forceinline__ void totals_init(GatherTotals& tot) {
  if (threadIdx.x == 0) {
    tot.dvm = tot.vm = tot.bad = 0ull;
    tot.pieces = 0;
    tot.done = 0u;
    for (auto& a : tot.aa) a[0] = a[1] = 0.0;
  }
}

// by every wavefront when it has finished; the last one of the block folds the
// block's totals into the global slots.  aa_row of aa_rows: the block's row of
// the Anderson sums.
__device__ __forceinline__ void totals_finish(GatherTotals& tot, const Scratch& sc, bool anderson,
                                              int aa_row, int aa_rows) {
  if (threadIdx.x % kWave != 0) return;
  __threadfence_block();  // the wavefront's totals before its arrival
  if (atomicAdd(&tot.done, 1u) != kBlock / kWave - 1) return;
  __threadfence_block();
  atomic_max_nonneg(sc.spread_copy(S_DVMAX), __longlong_as_double((long long)tot.dvm));
  atomic_max_nonneg(sc.spread_copy(S_VMAX), __longlong_as_double((long long)tot.vm));
  atomic_max_nonneg(sc.spread_copy(S_BAD), __longlong_as_double((long long)tot.bad));
  // integer counts: the atomic sum is exact and order-free
  if (tot.pieces > 0) unsafeAtomicAdd(sc.spread_copy(S_PIECES), (double)tot.pieces);
  if (anderson)
    for (int k = 0; k < 2; ++k) {
      double a = tot.aa[0][k];
      for (int w = 1; w < kMaxGatherBatches * kBlock / kWave; ++w) a += tot.aa[w][k];
      sc.region(P_AA)[k * aa_rows + aa_row] = a;
    }
}

// The order in which a gather block takes its particles: by the knots that
// their orbits cross, the most first, as stored where these are equal.  A
// wavefront runs its 64 orbits in lockstep, as long as its longest one: with
// the particles as stored it ran 1.9 pieces for 1.3 per orbit on average (cold
// beams, 64 per cell).  Per pass, as stored / ordered: quadratic, 2,097,152
// 280 / 249 us; mixed, 33,554,432 with orbits of several cells 6565 / 5571 us;
// cubic, 524,288 in two batches of 256 257 / 209 us.  Blocks of one batch keep the
// stored order: one wavefront would get all the long orbits and the others
// would be done early (300,007 at 9 per cell: 112 / 126 us).  cls:
// the thread's counts (batch k in bits 4k .. 4k+3); hist: 256 ints of LDS;
// order: one entry per particle slot of the block.  Called by the whole block.
__device__ __forceinline__ void block_order(unsigned cls, int batches, int* hist,
                                            uint16_t* __restrict__ order) {
  constexpr int kSets = kMaxGatherBatches * kBlock / kWave;  // 64 particles each
  static_assert(kBlock == 16 * kSets, "one thread per count and set");
  const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
  hist[threadIdx.x] = 0;
  __syncthreads();
  // hist[(15 - count) * kSets + set]; rank: the lane's place among those of its count
  int rank[kMaxGatherBatches];
#pragma unroll
  for (int k = 0; k < kMaxGatherBatches; ++k) {
    rank[k] = 0;
    if (k >= batches) continue;
    const int c = 15 - (int)((cls >> (4 * k)) & 15u);
    unsigned long long todo = __ballot(true);
    while (todo) {
      const int leader = __ffsll((long long)todo) - 1;
      const int lc = __builtin_amdgcn_readlane(c, leader);
      const unsigned long long group = __ballot(c == lc);
      if (c == lc) rank[k] = __popcll(group & ((1ull << lane) - 1ull));
      if (lane == leader) hist[lc * kSets + k * (kBlock / kWave) + wid] = __popcll(group);
      todo &= ~group;
    }
  }
  __syncthreads();
  const int n = hist[threadIdx.x];
  int incl = n;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int t = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += t;
  }
  __syncthreads();
  hist[threadIdx.x] = incl;
  __syncthreads();
  int before = 0;
  for (int w = 0; w < wid; ++w) before += hist[w * kWave + kWave - 1];
  __syncthreads();
  hist[threadIdx.x] = before + incl - n;  // slots before this count and set
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kMaxGatherBatches; ++k) {
    if (k >= batches) continue;
    const int c = 15 - (int)((cls >> (4 * k)) & 15u);
    order[hist[c * kSets + k * (kBlock / kWave) + wid] + rank[k]] =
        (uint16_t)(k * kBlock + threadIdx.x);
  }
  __syncthreads();
}

// Two waves per SIMD for the quadratic gather: its orbit loop fits 256
// registers, and asking for the occupancy makes the compiler keep it (it would
// otherwise go to one wave and twice the registers for a few more values).  Not from
// global memory, where the compiler's own choice (the same two waves, the loads in another
// order) was the faster one: 524,288 unsorted, per pass mixed 890 -> 708 us, FP64 810 -> 752.
template <int R, int FROM>
constexpr int kGatherWavesPerSimd = R == 2 && FROM != GATHER_LIST ? 2 : 1;

constexpr int kShortList = 32768;  // half of the chip's lanes at one wave per SIMD

// One block = P.gper batches of 256 consecutive cell-sorted particles.
// GATHER_TILE: the block finds the box of nodes its orbits touch; where that box exceeds the tile it takes the box of its start stencils,
// widened by as many nodes as fit.  It copies the gather fields of the box into
// LDS, and every stencil read of the orbit loop then comes from LDS; particles
// whose orbit leaves the box go to the list, all of them if not even the start
// stencils fit.  The list is a second kernel (GATHER_LIST), so each keeps its own register budget.
// After the first Picard pass of a step the block takes the box it stored in
// that pass.
template <int R, int FROM, class PS, bool SPLIT, int LANES>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(
    kGatherWavesPerSimd<R, FROM>))) void k_gather_push(StepParams P, PS st,
                                                 const double* __restrict__ vit,
                                                 double* __restrict__ vnew,
                                                 double* __restrict__ vbar_out, AosFields F,
                                                 GatherList list, Scratch sc,
                                                 AndersonPrev prev, ChunkBoxes bx, int aa_row0,
                                                 int aa_rows) {
  constexpr int W = R + 1;
  __shared__ GatherTotals tot;
  totals_init(tot);
  const int bid = blockIdx.x;
  if constexpr (FROM == GATHER_LIST) {
    __syncthreads();
    const int count = *list.count;  // written by the tiled kernel (previous launch)
    // Every lane reads nodes of its own, 5 cache lines each, so that a particle's chain of
    // rows and one CU's line rate bound the kernel.  With four lanes per particle (when:
    // launch_gather_push), per pass: 300,007 particles at 9 per cell 56 -> 25
    // us, 100,002 at 12 16 -> 9 us.
    // A short list's entry j goes to block j % grid: all CUs share it.  Of a long one
    // neighbouring entries go to a wavefront, since particles listed together lie together
    // (both gather kernels, short / long rule: 524,288 unsorted 598 / 455 us, 2,097,152
    // with orbits of 5 cells 9395 / 8477; 41,000 with orbits of one cell 130 / 134).
    constexpr int kEntries = kBlock / LANES;
    const bool spread = count < kShortList;
    const int64_t grid = gridDim.x;
    for (int64_t t = spread ? bid : bid * kEntries; t < count; t += kEntries * grid) {
      const int64_t j = t + threadIdx.x / LANES * (spread ? grid : 1);
      const bool active = j < count;
      gather_batch<R, SPLIT, LANES>(
          P, st, active ? list.particle[j] : 0, active, vit, vnew, vbar_out,
          [&](const int*) {
            return GlobalGather{F.g, P.G.mask[0], P.G.mask[1], P.G.mask[2], P.G.shx, P.G.shy};
          },
          [](int, const double*, const double*, int*) { return true; }, prev, tot,
          threadIdx.x / kWave);
    }
    totals_finish(tot, sc, prev.w != nullptr, aa_row0 + bid, aa_rows);
  } else {
    __shared__ double2 tile2[kGatherTileNodes * kGbufStride / 2];
    lds_cdouble* tile = (lds_cdouble*)(reinterpret_cast<double*>(tile2));
    const double2* g2 = reinterpret_cast<const double2*>(F.g);
    constexpr int kBatch = kBlock / LANES;  // particles
    const int64_t first = (int64_t)bid * P.gper * kBatch;
    if constexpr (FROM == GATHER_MESH) {
      const int n2 = (int)P.G.ncell * (kGbufStride / 2);
      for (int t = threadIdx.x; t < n2; t += kBlock) tile2[t] = g2[t];
      __syncthreads();
      for (int k = 0; k < P.gper; ++k) {
        const int64_t i = first + k * kBatch + threadIdx.x / LANES;
        gather_batch<R, SPLIT, LANES>(
            P, st, (int)i, i < P.np, vit, vnew, vbar_out,
            [&](const int*) {
              return MeshGather{tile, P.G.mask[0], P.G.mask[1], P.G.mask[2], P.G.shx, P.G.shy};
            },
            [](int, const double*, const double*, int*) { return true; }, prev, tot,
            threadIdx.x / kWave);
      }
    } else {
      // the block's node box: reference node sref, origin tlo relative to it and
      // extents dim, per axis (dim[0] < 0: not even the start stencils fit)
      int sref[3], tlo[3], dim[3];
      if (bx.reuse) {  // the box this block found in the step's first pass
        const int* b = bx.box + (int64_t)bid * kBoxInts;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          sref[a] = b[a];
          tlo[a] = b[3 + a];
          dim[a] = b[6 + a];
        }
      } else {
        __shared__ int s_ref[3];
        if (threadIdx.x == 0) {
          double x0[3];
          st.x_of(P.G, P.np, first, x0);
#pragma unroll
          for (int a = 0; a < 3; ++a)
            s_ref[a] = to_int_clamped(floor(x0[a] * P.G.invH[a] + Spline<R>::base_off));
        }
        __syncthreads();
        int mv[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) mv[k] = 0x3fffffff;
#pragma unroll
        for (int a = 0; a < 3; ++a) sref[a] = s_ref[a];
        unsigned cls = 0u;  // per batch: knots that the thread's orbit crosses, in 4 bits
        for (int k = 0; k < P.gper; ++k) {
          const int64_t i = first + k * kBatch + threadIdx.x / LANES;
          if (i >= P.np) break;
          int crossed = 0;
          double x0[3], va[3], vi[3];
          st.x_of(P.G, P.np, i, x0);
          st.v_of(P.np, i, va);
          load3(vit, P.np, i, vi);
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            const double d = P.dt * (0.5 * (vi[a] + va[a]));
            int lo, n, b0;
            orbit_nodes<R>(x0[a], d, P.G.invH[a], lo, n, b0);
            const int rel = min_image(lo - sref[a], P.G.n[a]);
            mv[a] = min(mv[a], rel);
            mv[3 + a] = min(mv[3 + a], -(rel + n));
            mv[6 + a] = min(mv[6 + a], rel + (b0 - lo));
            mv[9 + a] = min(mv[9 + a], -(rel + (b0 - lo) + W));
            crossed += min(knots_crossed(x0[a], d, P.G.invH[a], Spline<R>::base_off), 15);
          }
          cls |= (unsigned)min(crossed, 15) << (4 * k);
        }
        if (SPLIT && LANES == 1 && bx.order)
          block_order(cls, P.gper, reinterpret_cast<int*>(tile2),
                      bx.order + first);
        block_min_ints<12>(mv);
#pragma unroll
        for (int a = 0; a < 3; ++a) {
          tlo[a] = mv[a];
          dim[a] = -mv[3 + a] - tlo[a] + 1;
        }
        if (plain_slack(dim, kGatherTileNodes) < 0) {
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            tlo[a] = mv[6 + a];
            dim[a] = -mv[9 + a] - tlo[a] + 1;
          }
          const int e = plain_slack(dim, kGatherTileNodes);
          if (e < 0) dim[0] = -1;
#pragma unroll
          for (int a = 0; a < 3; ++a)
            if (e > 0) {
              tlo[a] -= e;
              dim[a] += 2 * e;
            }
        }
        if (bx.box && threadIdx.x == 0) {
          int* b = bx.box + (int64_t)bid * kBoxInts;
#pragma unroll
          for (int a = 0; a < 3; ++a) {
            b[a] = sref[a];
            b[3 + a] = tlo[a];
            b[6 + a] = dim[a];
          }
        }
      }
#pragma unroll
      for (int a = 0; a < 3; ++a) {  // block-uniform
        sref[a] = __builtin_amdgcn_readfirstlane(sref[a]);
        tlo[a] = __builtin_amdgcn_readfirstlane(tlo[a]);
        dim[a] = __builtin_amdgcn_readfirstlane(dim[a]);
      }
      // Not even the start stencils fit: the block's particles to the list at once (one by
      // one their counter's atomics took 75 of 100 us, 524,288 unsorted)
      if (dim[0] <= 0) {
        __shared__ int s_place;
        const int n = (int)min((int64_t)P.gper * kBatch, P.np - first);
        __syncthreads();  // totals_init
        if (threadIdx.x == 0) s_place = atomicAdd(list.count, n);
        __syncthreads();
        for (int t = threadIdx.x; t < n; t += kBlock) list.particle[s_place + t] = (int)first + t;
        totals_finish(tot, sc, prev.w != nullptr, aa_row0 + bid, aa_rows);
        return;
      }
      const int nt2 = dim[0] * dim[1] * dim[2] * (kGbufStride / 2);
      const float inv_d1 = 1.0f / (float)dim[1], inv_d2 = 1.0f / (float)dim[2];
      for (int t = threadIdx.x; t < nt2; t += kBlock) {
        const int nd = t / (kGbufStride / 2), part = t % (kGbufStride / 2);
        const int q = div_small(nd, inv_d2), cx = div_small(q, inv_d1);
        const int cz = nd - q * dim[2], cy = q - cx * dim[1];
        const int64_t g = node_index(P.G, sref[0] + tlo[0] + cx, sref[1] + tlo[1] + cy,
                                     sref[2] + tlo[2] + cz);
        tile2[t] = g2[g * (kGbufStride / 2) + part];
      }
      __syncthreads();
      // Sets of 64 particles, the longest orbits first, go to the wavefronts there and
      // back (0 1 2 3, 3 2 1 0, ..); which wavefront is the first changes from block to
      // block, since wavefront w of every block sits on the same SIMD.
      constexpr int kWaves = kBlock / kWave;
      const int wid = __builtin_amdgcn_readfirstlane(((int)threadIdx.x / kWave + bid / 8) % kWaves);
      for (int k = 0; k < P.gper; ++k) {
        const int set = k * kWaves + (k & 1 ? kWaves - 1 - wid : wid);
        const int64_t slot = first + set * (kWave / LANES) + threadIdx.x % kWave / LANES;
        const int64_t i = SPLIT && LANES == 1 && bx.order ? first + bx.order[slot] : slot;
        gather_batch<R, SPLIT, LANES>(
            P, st, (int)i, i < P.np, vit, vnew, vbar_out,
            [&](const int* shift) {
              return TileGather{tile, shift[0] - sref[0] - tlo[0], shift[1] - sref[1] - tlo[1],
                                shift[2] - sref[2] - tlo[2], dim[1], dim[2]};
            },
            [&](int ip, const double* x0, const double* d, int* shift) {
              bool in = true;
#pragma unroll
              for (int a = 0; a < 3; ++a) {
                int lo, n, b0;
                orbit_nodes<R>(x0[a], d[a], P.G.invH[a], lo, n, b0);
                const int rel = min_image(lo - sref[a], P.G.n[a]);
                shift[a] = rel - (lo - sref[a]);
                in = in && d[a] == d[a] && rel >= tlo[a] && rel + n < tlo[a] + dim[a];
              }
              if (!in && threadIdx.x % LANES == 0) list.particle[atomicAdd(list.count, 1)] = ip;
              return in;
            },
            prev, tot, set);
      }
    }
    totals_finish(tot, sc, prev.w != nullptr, aa_row0 + bid, aa_rows);
  }
}

// Consistency sweep of the accepted iterate: Ubar, Ebar = -gphibar - Ubar,
// sum_i q vbar . Ebar, R_A = A_h^{n+1}(x^{n+1}) - A_h^n(x^n) - dt (Ubar + D vbar)
// (eq. RA-test) and the partition of unity sum_g Sbar_g.
template <int R, class PS, bool SPLIT>
__global__ __launch_bounds__(kBlock) void k_sweep(StepParams P, PS st,
                                                 const double* __restrict__ vit, AosFields F,
                                                 const double* __restrict__ Uh, Scratch sc) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  double sums[2] = {0.0, 0.0};  // work, |R_A|^2
  double ramax = 0.0, poudev = 0.0;
  if (i < P.np) {
    const double qi = species_value(P.qs, st.species(i));
    double x0[3], va[3], vi[3], vb[3], d[3];
    st.x_of(P.G, P.np, i, x0);
    st.v_of(P.np, i, va);
    load3(vit, P.np, i, vi);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      vb[a] = 0.5 * (vi[a] + va[a]);
      d[a] = P.dt * vb[a];
    }
    double gp[3] = {0.0, 0.0, 0.0}, Ub[3] = {0.0, 0.0, 0.0};
    double D[3][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
    double pou = 0.0;
    if constexpr (SPLIT) {
      for_each_piece<R>(x0, d, P.G, [&](double s0, double s1, const double* base) {
        gather_piece<R, true>(P.G, x0, d, s0, s1, base, F, Uh, gp, D, Ub, pou);
      });
    } else {
      for (int q = 0; q < P.rule.n; ++q) {
        double base[3], sq, wq;
        unsplit_point<R>(P.G, P.rule, q, x0, d, base, sq, wq);
        gather_points<R, 1, true>(P.G, x0, d, base, &sq, &wq, F, Uh, gp, D, Ub, pou);
      }
    }
    double x1[3], A0s[3], A1e[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) x1[a] = wrap_pos(x0[a] + d[a], P.G.L[a], P.G.invL[a]);
    point_A<R>(P.G, x0, F, 0, A0s);
    point_A<R>(P.G, x1, F, 1, A1e);
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      const double Dv = D[l][0] * vb[0] + D[l][1] * vb[1] + D[l][2] * vb[2];
      const double ra = A1e[l] - A0s[l] - P.dt * (Ub[l] + Dv);
      sums[1] += ra * ra;
      ramax = fmax(ramax, fabs(ra));
      sums[0] += qi * vb[l] * (-gp[l] - Ub[l]);
    }
    poudev = fabs(pou - 1.0);
  }
  const double rm = block_max(ramax), pm = block_max(poudev);
  if (threadIdx.x == 0) {
    atomic_max_nonneg(sc.spread_copy(S_RAMAX), rm);
    atomic_max_nonneg(sc.spread_copy(S_POU), pm);
  }
  double s2[2] = {sums[0], sums[1]};
  block_partials<2>(s2, sc.region(P_SWEEP));  // -> S_WORK, S_RA2
}

// Accept the step: x^{n+1} = x^n + dt vbar^p (wrapped), v^{n-1} <- v^n,
// v^n <- v^{n+1,p+1} (with the store's rounding, keyed by the particle's
// stored state and the step).  The kinetic energies are those of the stored
// values.
template <class PS>
__global__ __launch_bounds__(kBlock) void k_finalize(StepParams P, PS st,
                                                    const double* __restrict__ vit,
                                                    const double* __restrict__ vnew, uint64_t step,
                                                    Scratch sc) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  double s[2] = {0.0, 0.0};  // K^{n+1}, K^{n+1} - K^n
  if (i < P.np) {
    double x0[3], vo[3], vi[3], vn[3], x1[3], w[3];
    const double mi = species_value(P.ms, st.species(i));
    st.x_of(P.G, P.np, i, x0);
    st.v_of(P.np, i, vo);
    load3(vit, P.np, i, vi);
    load3(vnew, P.np, i, vn);
#pragma unroll
    for (int a = 0; a < 3; ++a)
      x1[a] = wrap_pos(x0[a] + P.dt * 0.5 * (vi[a] + vo[a]), P.G.L[a], P.G.invL[a]);
    const uint64_t key = splitmix64(st.state_key(P.np, i) ^ (step * 0xd1b54a32d192ed03ull));
    st.set_x(P.G, P.np, i, x1);
    st.set_vp(P.np, i, vo);
    st.accept_v(P.np, i, vn, key, w);
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      s[0] += 0.5 * mi * w[a] * w[a];
      s[1] += 0.5 * mi * (w[a] - vo[a]) * (w[a] + vo[a]);
    }
  }
  block_partials<2>(s, sc.region(P_K));  // -> S_K, S_DK
}

template <class PS>
__global__ __launch_bounds__(kBlock) void k_kinetic(StepParams P, PS st, Scratch sc) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  double s[2] = {0.0, 0.0};
  if (i < P.np) {
    double va[3];
    st.v_of(P.np, i, va);
    const double mi = species_value(P.ms, st.species(i));
#pragma unroll
    for (int a = 0; a < 3; ++a) s[0] += 0.5 * mi * va[a] * va[a];
  }
  block_partials<2>(s, sc.region(P_K));
}

// which = 0: x (wrapped into [0, L)), 1: v^n, 2: v^{n-1}; src and dst in the
// caller's order, particle i at id[i]
template <class PS>
__global__ __launch_bounds__(kBlock) void k_import(StepParams P, PS st, int which,
                                                  const int* __restrict__ id,
                                                  const double* __restrict__ src) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= P.np) return;
  double w[3];
  load3(src, P.np, id[i], w);
  if (which == 0) {
#pragma unroll
    for (int a = 0; a < 3; ++a) w[a] = wrap_pos(w[a], P.G.L[a], P.G.invL[a]);
    st.set_x(P.G, P.np, i, w);
  } else if (which == 1) {
    st.set_v(P.np, i, w);
  } else {
    st.set_vp(P.np, i, w);
  }
}

template <class PS>
__global__ __launch_bounds__(kBlock) void k_export(StepParams P, PS st, int which,
                                                  const int* __restrict__ id,
                                                  double* __restrict__ dst) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= P.np) return;
  double w[3];
  if (which == 0)
    st.x_of(P.G, P.np, i, w);
  else if (which == 1)
    st.v_of(P.np, i, w);
  else
    st.vp_of(P.np, i, w);
  const int64_t k = id[i];
#pragma unroll
  for (int a = 0; a < 3; ++a) dst[a * P.np + k] = w[a];
}

__global__ __launch_bounds__(kBlock) void k_fixed_current(int64_t n,
                                                         unsigned long long* __restrict__ Jfix,
                                                         double* __restrict__ J, double unit) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  J[i] = unit * (double)(long long)Jfix[i];
  Jfix[i] = 0ull;
}

// rho_g += q S_g(x_i) / dV (eq. source-moments), point shape.  Mixed state:
// S_g as fixed-point quanta into out.Jfix (rho = q / dV / scale x quanta).
template <int R, class PS>
__global__ __launch_bounds__(kBlock) void k_deposit_rho(StepParams P, PS st, CurrentOut out) {
  constexpr int W = R + 1;
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= P.np) return;
  double w[3][W], x0[3];
  int f[3];
  st.x_of(P.G, P.np, i, x0);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const double u = x0[a] * P.G.invH[a];
    const double base = floor(u + Spline<R>::base_off);
    Spline<R>::w(u - base, w[a]);
    f[a] = to_int_clamped(base) + Spline<R>::first_off;
  }
  const double cq = species_value(P.cq, st.species(i));  // q_i / dV; fixed point: q_i / q_0
#pragma unroll
  for (int a = 0; a < W; ++a)
#pragma unroll
    for (int b = 0; b < W; ++b)
#pragma unroll
      for (int cc = 0; cc < W; ++cc) {
        const int64_t g = node_of(P.G, wrapi(f[0] + a, P.G.n[0]), wrapi(f[1] + b, P.G.n[1]),
                                  wrapi(f[2] + cc, P.G.n[2]));
        const double s = w[0][a] * w[1][b] * w[2][cc];
        if constexpr (PS::kMixed)
          atomicAdd(out.Jfix + g, quantize(cq * s, out.fix_scale));
        else
          unsafeAtomicAdd(out.J + g, cq * s);
      }
}

// Orbit integrals of independent particles against SoA fields (kernel-level check).
template <int R, bool SPLIT>
__global__ __launch_bounds__(kBlock) void k_orbit_gather_soa(QuadRule rule, Grid G, int64_t n,
                                                            const double* __restrict__ x0s,
                                                            const double* __restrict__ ds,
                                                            SoaFields F,
                                                            const double* __restrict__ Uh,
                                                            double* __restrict__ out) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  double x0[3], d[3];
  load3(x0s, n, i, x0);
  load3(ds, n, i, d);
  double gp[3] = {0.0, 0.0, 0.0}, Ub[3] = {0.0, 0.0, 0.0};
  double D[3][3] = {{0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}, {0.0, 0.0, 0.0}};
  double pou = 0.0;
  int pieces = 0;
  bool ok = true;
  if constexpr (SPLIT) {
    ok = for_each_piece<R>(x0, d, G, [&](double s0, double s1, const double* base) {
      gather_piece<R, true>(G, x0, d, s0, s1, base, F, Uh, gp, D, Ub, pou);
      ++pieces;
    });
  } else {
    for (int q = 0; q < rule.n; ++q) {
      double base[3], sq, wq;
      unsplit_point<R>(G, rule, q, x0, d, base, sq, wq);
      gather_points<R, 1, true>(G, x0, d, base, &sq, &wq, F, Uh, gp, D, Ub, pou);
    }
    pieces = rule.n;
  }
  double x1[3], A0s[3], A1e[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) x1[a] = wrap_pos(x0[a] + d[a], G.L[a], G.invL[a]);
  point_A<R>(G, x0, F, 0, A0s);
  point_A<R>(G, x1, F, 1, A1e);
  double* o = out + 24 * i;
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    o[l] = gp[l];
    o[3 + l] = Ub[l];
#pragma unroll
    for (int j = 0; j < 3; ++j) o[6 + 3 * l + j] = D[l][j];
    o[15 + l] = A1e[l];
    o[18 + l] = A0s[l];
  }
  o[21] = pou;
  o[22] = ok ? (double)pieces : -1.0;
  o[23] = 0.0;
}

template <int R, bool SPLIT>
__global__ __launch_bounds__(kBlock) void k_orbit_deposit_soa(QuadRule rule, Grid G, int64_t n,
                                                             const double* __restrict__ x0s,
                                                             const double* __restrict__ ds,
                                                             const double* __restrict__ qv,
                                                             double* __restrict__ J) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  double x0[3], d[3], c3[3];
  load3(x0s, n, i, x0);
  load3(ds, n, i, d);
  load3(qv, n, i, c3);
#pragma unroll
  for (int a = 0; a < 3; ++a) c3[a] /= G.dV;
  if constexpr (SPLIT) {
    for_each_piece<R>(x0, d, G, [&](double s0, double s1, const double* base) {
      scatter_piece<R>(G, x0, d, s0, s1, base, c3, J);
    });
  } else {
    constexpr int W = R + 1;
    for (int q = 0; q < rule.n; ++q) {
      double base[3], sq, wq, Iw[W][W][W];
      int f[3];
      unsplit_point<R>(G, rule, q, x0, d, base, sq, wq);
      sbar_points<R, 1>(G, x0, d, base, &sq, &wq, Iw, f);
      for (int a = 0; a < W; ++a)
        for (int b = 0; b < W; ++b)
          for (int c = 0; c < W; ++c) {
            const int64_t g = node_index(G, f[0] + a, f[1] + b, f[2] + c);
#pragma unroll
            for (int l = 0; l < 3; ++l) unsafeAtomicAdd(J + l * G.ncell + g, Iw[a][b][c] * c3[l]);
          }
    }
  }
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

}  // namespace

int64_t scatter_blocks(int64_t np, int chunk, int span) {
  return (np + span - 1) / span * (span / chunk);
}
int64_t particle_blocks(int64_t np) { return (np + kBlock - 1) / kBlock; }

// ---- launchers ---------------------------------------------------------------

// f(std::integral_constant<int, r>{}) for the spline degree r = 1, 2, 3
template <class F>
void by_degree(int r, F&& f) {
  if (r == 1)
    f(std::integral_constant<int, 1>{});
  else if (r == 2)
    f(std::integral_constant<int, 2>{});
  else
    f(std::integral_constant<int, 3>{});
}

template <class PS>
void launch_extrapolate(hipStream_t s, int64_t np, const PS& st, double* vit, double* vbar) {
  if (np <= 0) return;
  k_extrapolate<<<blocks_for(3 * np), kBlock, 0, s>>>(3 * np, st.v, st.vp, vit, vbar);
}

// Blocks of at least two batches of 256 order their lanes' particles.  Per pass, as
// stored / ordered: mixed, 33,554,432 at 128 per cell with orbits of several cells,
// 2048 per block 3383 / 2877 us; mixed, 2,097,152 cold beams, 2048 per block 144 /
// 137 us; cubic, 524,288, 512 per block 76.6 / 73.6 us.
constexpr int kLaneOrderChunk = 512;

template <class PS>
void launch_scatter(hipStream_t s, int r, const StepParams& P, const PS& st, const double* vit,
                    const double* vbar, CurrentOut out, Scratch sc, ChunkBoxes bx) {
  if (P.np <= 0) return;
  const bool multi = P.nsp > 1;
  if (P.chunk < kLaneOrderChunk) bx.lane_order = nullptr;
  // degree x (split) x species
  const unsigned nblk = (unsigned)scatter_blocks(P.np, P.chunk, P.span);
  auto go = [&](auto R, auto SPLIT) {
    if (multi)
      k_scatter<R.value, PS, SPLIT.value, true>
          <<<nblk, kBlock, 0, s>>>(P, st, vit, vbar, out, sc, bx);
    else
      k_scatter<R.value, PS, SPLIT.value, false>
          <<<nblk, kBlock, 0, s>>>(P, st, vit, vbar, out, sc, bx);
  };
  if constexpr (!PS::kMixed) {
    if (!P.split) {
      by_degree(r, [&](auto R) { go(R, std::false_type{}); });
      return;
    }
  }
  if constexpr (!PS::kMixed) {
    if (P.scatter_mm) {  // degree 2
      if (multi)
        k_scatter_mm<2, true><<<nblk, kBlock, 0, s>>>(P, st, vit, vbar, out.J, sc, bx);
      else
        k_scatter_mm<2, false><<<nblk, kBlock, 0, s>>>(P, st, vit, vbar, out.J, sc, bx);
      return;
    }
  }
  by_degree(r, [&](auto R) { go(R, std::true_type{}); });
}

// Batches of 256 particles per gather block: as many as leave four blocks per
// compute unit, at most 4, and no more than the particles of 32 cells, whose box
// fits the tile (4x4x2 cells with cubic stencils and orbits of a cell: 9x9x7 nodes).
int gather_batches(int64_t np, int64_t ncell) {
  int g = kMaxGatherBatches;
  while (g > 1 && (np < (int64_t)g * kBlock * 1024 || g * kBlock * ncell > 32 * np)) g /= 2;
  return g;
}

// Up to this count a gather's particles take four lanes each: such a launch takes
// what one particle's chain of pieces and rows takes.  Beyond it the blocks, of 64
// particles with a node box each, are too many.  Per pass with one / four lanes:
// linear, 4,096 particles in a mesh of 256 nodes 9.9 / 8.6 us; quadratic, 32,769
// 26.1 / 21.6 us, 100,002 36 / 56 us; linear, 131,072 15 / 36 us.
constexpr int64_t kQuadGather = 40960;

GatherGrid gather_grid(int64_t np, int64_t ncell) {
  GatherGrid g;
  g.lanes = np <= kQuadGather ? 4 : 1;
  g.batches = gather_batches(np, ncell);
  const int64_t per = (int64_t)g.batches * (kBlock / g.lanes);
  g.blocks = (int)((np + per - 1) / per);
  g.whole_mesh = ncell <= kGatherTileNodes;
  g.list_blocks = g.whole_mesh ? 0 : std::min((int)blocks_for(np), 512);
  return g;
}

int64_t gather_slots(int64_t np, int64_t ncell) {
  const GatherGrid g = gather_grid(np, ncell);
  return g.batches > 1 ? (int64_t)g.blocks * g.batches * kBlock : 0;
}

template <class PS>
void launch_gather_push(hipStream_t s, int r, StepParams P, const PS& st, const double* vit,
                        double* vnew, double* vbar_out, const double* gbuf, GatherList list,
                        Scratch sc, AndersonPrev prev, ChunkBoxes bx) {
  if (P.np <= 0) return;
  AosFields F{gbuf};
  const GatherGrid g = gather_grid(P.np, P.G.ncell);
  P.gper = g.batches;
  const int rows = g.blocks + g.list_blocks;
  auto go = [&](auto R, auto SPLIT) {
    auto run = [&](auto LANES) {
      if (g.whole_mesh)
        k_gather_push<R.value, GATHER_MESH, PS, SPLIT.value, LANES.value>
            <<<g.blocks, kBlock, 0, s>>>(P, st, vit, vnew, vbar_out, F, list, sc, prev, bx, 0, rows);
      else
        k_gather_push<R.value, GATHER_TILE, PS, SPLIT.value, LANES.value>
            <<<g.blocks, kBlock, 0, s>>>(P, st, vit, vnew, vbar_out, F, list, sc, prev, bx, 0, rows);
    };
    auto far = [&](auto LANES) {
      if (!g.whole_mesh)
        k_gather_push<R.value, GATHER_LIST, PS, SPLIT.value, LANES.value>
            <<<g.list_blocks, kBlock, 0, s>>>(P, st, vit, vnew, vbar_out, F, list, sc, prev,
                                              ChunkBoxes{}, g.blocks, rows);
    };
    if (g.lanes == 4) {
      run(std::integral_constant<int, 4>{});
      far(std::integral_constant<int, 4>{});
    } else {
      run(std::integral_constant<int, 1>{});
      // Four lanes per listed particle add a particle's terms in another order than one.
      // Which particles are listed goes by the particles of a block, hence by the
      // order of the particles, and the mixed form's results do not: there all
      // of a launch's particles are summed alike.
      // In the FP64 form one lane is the faster one, but for cubic stencils, where most
      // particles are listed (one / four lanes per pass: 524,288 at 128 per cell, orbits of 3
      // cells 975 / 1549 us, never sorted 355 / 403; cubic 262,144 941 / 879; a tenth
      // of 262,144 listed 213 / 171).
      if (PS::kMixed || (list.most && R.value < 3))
        far(std::integral_constant<int, 1>{});
      else
        far(std::integral_constant<int, 4>{});
    }
  };
  if constexpr (!PS::kMixed) {
    if (!P.split) {
      by_degree(r, [&](auto R) { go(R, std::false_type{}); });
      return;
    }
  }
  by_degree(r, [&](auto R) { go(R, std::true_type{}); });
}

template <class PS>
void launch_sweep(hipStream_t s, int r, const StepParams& P, const PS& st, const double* vit,
                  const double* gbuf, const double* Uhalf, Scratch sc) {
  if (P.np <= 0) return;
  AosFields F{gbuf};
  if constexpr (!PS::kMixed) {
    if (!P.split) {
      by_degree(r, [&](auto R) {
        k_sweep<R.value, PS, false><<<blocks_for(P.np), kBlock, 0, s>>>(P, st, vit, F, Uhalf, sc);
      });
      return;
    }
  }
  by_degree(r, [&](auto R) {
    k_sweep<R.value, PS, true><<<blocks_for(P.np), kBlock, 0, s>>>(P, st, vit, F, Uhalf, sc);
  });
}

template <class PS>
void launch_finalize(hipStream_t s, const StepParams& P, const PS& st, const double* vit,
                     const double* vnew, uint64_t step, Scratch sc) {
  if (P.np <= 0) return;
  k_finalize<PS><<<blocks_for(P.np), kBlock, 0, s>>>(P, st, vit, vnew, step, sc);
}

template <class PS>
void launch_kinetic(hipStream_t s, const StepParams& P, const PS& st, Scratch sc) {
  if (P.np <= 0) return;
  k_kinetic<PS><<<blocks_for(P.np), kBlock, 0, s>>>(P, st, sc);
}

template <class PS>
void launch_deposit_rho(hipStream_t s, int r, const StepParams& P, const PS& st, CurrentOut out) {
  if (P.np <= 0) return;
  by_degree(r, [&](auto R) {
    k_deposit_rho<R.value, PS><<<blocks_for(P.np), kBlock, 0, s>>>(P, st, out);
  });
}

template <class PS>
void launch_import(hipStream_t s, const StepParams& P, const PS& st, int which, const int* id,
                   const double* src) {
  if (P.np <= 0) return;
  k_import<PS><<<blocks_for(P.np), kBlock, 0, s>>>(P, st, which, id, src);
}

template <class PS>
void launch_export(hipStream_t s, const StepParams& P, const PS& st, int which, const int* id,
                   double* dst) {
  if (P.np <= 0) return;
  k_export<PS><<<blocks_for(P.np), kBlock, 0, s>>>(P, st, which, id, dst);
}

void launch_fixed_current(hipStream_t s, int64_t n, unsigned long long* Jfix, double* J,
                          double unit) {
  if (n <= 0) return;
  k_fixed_current<<<blocks_for(n), kBlock, 0, s>>>(n, Jfix, J, unit);
}

#define ECPIC_INSTANTIATE_STORE(PS)                                                              \
  template void launch_extrapolate<PS>(hipStream_t, int64_t, const PS&, double*, double*);                \
  template void launch_scatter<PS>(hipStream_t, int, const StepParams&, const PS&, const double*, \
                                   const double*, CurrentOut, Scratch, ChunkBoxes);              \
  template void launch_gather_push<PS>(hipStream_t, int, StepParams, const PS&, const double*,  \
                                       double*, double*, const double*, GatherList,             \
                                       Scratch, AndersonPrev, ChunkBoxes);                       \
  template void launch_sweep<PS>(hipStream_t, int, const StepParams&, const PS&, const double*,  \
                                 const double*, const double*, Scratch);                         \
  template void launch_finalize<PS>(hipStream_t, const StepParams&, const PS&, const double*,     \
                                    const double*, uint64_t, Scratch);                           \
  template void launch_kinetic<PS>(hipStream_t, const StepParams&, const PS&, Scratch);          \
  template void launch_deposit_rho<PS>(hipStream_t, int, const StepParams&, const PS&,          \
                                       CurrentOut);                                              \
  template void launch_import<PS>(hipStream_t, const StepParams&, const PS&, int, const int*,    \
                                  const double*);                                                \
  template void launch_export<PS>(hipStream_t, const StepParams&, const PS&, int, const int*,    \
                                  double*);

ECPIC_INSTANTIATE_STORE(Fp64Store)
ECPIC_INSTANTIATE_STORE(MixedStore)
#undef ECPIC_INSTANTIATE_STORE

void launch_orbit_gather_soa(hipStream_t s, int r, const QuadRule* rule, const Grid& G,
                             int64_t n, const double* x0, const double* d, const double* gphi,
                             const double* U, const double* A0, const double* A1, double* out) {
  if (n <= 0) return;
  SoaFields F{gphi, A0, A1, G.ncell};
  const QuadRule ru = rule ? *rule : QuadRule{};
  const unsigned nb = blocks_for(n);
  by_degree(r, [&](auto R) {
    if (rule)
      k_orbit_gather_soa<R.value, false><<<nb, kBlock, 0, s>>>(ru, G, n, x0, d, F, U, out);
    else
      k_orbit_gather_soa<R.value, true><<<nb, kBlock, 0, s>>>(ru, G, n, x0, d, F, U, out);
  });
}

void launch_orbit_deposit_soa(hipStream_t s, int r, const QuadRule* rule, const Grid& G,
                              int64_t n, const double* x0, const double* d, const double* qv,
                              double* J) {
  if (n <= 0) return;
  const QuadRule ru = rule ? *rule : QuadRule{};
  const unsigned nb = blocks_for(n);
  by_degree(r, [&](auto R) {
    if (rule)
      k_orbit_deposit_soa<R.value, false><<<nb, kBlock, 0, s>>>(ru, G, n, x0, d, qv, J);
    else
      k_orbit_deposit_soa<R.value, true><<<nb, kBlock, 0, s>>>(ru, G, n, x0, d, qv, J);
  });
}

}  // namespace ecpic
