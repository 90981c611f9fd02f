// Particle side of the adjoint of a converged step (degree 2, split orbits).
//
// The converged step solves w = G(w; x, v, F) with vbar = (w + v)/2,
// d = dt vbar and (P^n rebuilt from eq. discrete-canonical-relation)
//   G = v + (q/m) [A0_h(x) - A1_h(x + d)] + (q dt/m) [-gphibar + (D A)^T vbar],
//   gphibar = sum_g gphi_g Sbar_g,
//   ((D A)^T vbar)_j = sum_g int b_g(s) d_j S_g(x(s)) ds,  b_g(s) = vbar.((1-s) A0_g + s A1_g),
// (eqs. orbit-push, split-Sbar, split-DA), and the current
//   J_g = (q/dV) sum_i vbar_i Sbar_ig   (eq. orbit-current).
// For a particle with push adjoint eta = (q/m) xi and current adjoint
// mu = (q/dV) lambda_J, the kernels below add the derivatives with respect
// to x, d and vbar, and scatter the push's mesh adjoints of gphi, A0 and A1.
// Inside each split piece the integrands are polynomials of degree <= 6 in s
// (4-point Gauss-Legendre is exact); the piece ends move with x and d, but
// the integrands b_g d_j S_g and S_g are continuous across knots for degree
// 2, so no end-point terms arise.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "internal.hpp"
#include "orbit.hpp"
#include "reduce.hpp"

namespace ecpic {

namespace {

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

// weights and first derivatives (physical units) of the three degree-2
// stencil nodes along one axis
struct Axis2 {
  double w[3], dw[3];
  __device__ __forceinline__ void at(double t, double invH) {
    Spline<2>::wd(t, w, dw);
#pragma unroll
    for (int o = 0; o < 3; ++o) dw[o] *= invH;
  }
};

// The nine values of a node that the push reads (components l of grad phi, A^n
// and A^{n+1} as 0 + l, 3 + l and 6 + l) and the nine adjoints that it adds to,
// in the block's LDS tile over its particles' node box, or in global memory.
// Nodes are given in the particle's unwrapped frame.  The tile pointers carry the
// LDS address space, so the additions are LDS atomics (through a plain pointer
// they compiled to flat atomics, the slower path that serves either memory).
constexpr int kAdjTileNodes = 1000;
typedef __attribute__((address_space(3))) double lds_double;
struct TileNodes {
  lds_double* field;
  lds_double* sum;
  int o[3];    // particle's frame -> tile
  int sy, sx;  // nodes between neighbours along y and x; along z 1
  __device__ __forceinline__ int at(int ix, int iy, int iz) const {
    return (ix + o[0]) * sx + (iy + o[1]) * sy + (iz + o[2]);
  }
  __device__ __forceinline__ double get(int n, int k) const { return field[n + k * kAdjTileNodes]; }
  __device__ __forceinline__ void add(int n, int k, double v) const {
    __hip_atomic_fetch_add(&sum[n + k * kAdjTileNodes], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
};
__device__ __forceinline__ const double* mesh_field(const AdjParticleArgs& P, int k) {
  return (k < 3 ? P.gphi : (k < 6 ? P.A0 : P.A1)) + (int64_t)(k % 3) * P.G.ncell;
}
__device__ __forceinline__ double* mesh_sum(const AdjParticleArgs& P, int k) {
  return (k < 3 ? P.lgphi : (k < 6 ? P.lA0 : P.lA1)) + (int64_t)(k % 3) * P.G.ncell;
}
struct MeshNodes {
  const AdjParticleArgs& P;
  __device__ __forceinline__ int64_t at(int ix, int iy, int iz) const {
    return node_index(P.G, ix, iy, iz);
  }
  __device__ __forceinline__ double get(int64_t n, int k) const { return mesh_field(P, k)[n]; }
  __device__ __forceinline__ void add(int64_t n, int k, double v) const {
    unsafeAtomicAdd(mesh_sum(P, k) + n, v);
  }
};

// Node values of the polynomial functional with moments m[k] = M(t^k): the
// degree-2 node weights along an axis are 1/8 - t/2 + t^2/2, 3/4 - t^2 and
// 1/8 + t/2 + t^2/2.
__device__ __forceinline__ void nodes_of_moments(double (&m)[3]) {
  const double lo = 0.125 * m[0] + 0.5 * (m[2] - m[1]);
  const double mid = 0.75 * m[0] - m[2];
  m[2] = lo + m[1];
  m[1] = mid;
  m[0] = lo;
}
// and the coefficients in t of the sum of node values f[k] against these weights
__device__ __forceinline__ void coefficients_of_nodes(double (&f)[3]) {
  const double c2 = 0.5 * (f[0] + f[2]) - f[1];
  const double c1 = 0.5 * (f[2] - f[0]);
  f[0] = f[1] + 0.25 * c2;
  f[1] = c1;
  f[2] = c2;
}

// Values that the compiler may not carry over in derived form: it kept the points'
// weights and their products from one row, and from one half of a row, to the next
// (96 registers spilled at two wavefronts per SIMD).
template <int N>
__device__ __forceinline__ void recompute_from(double (&v)[N]) {
#pragma unroll
  for (int k = 0; k < N; ++k) asm volatile("" : "+v"(v[k]));
}

// weight and derivative (per unit of cell coordinate) of stencil node k at t, for
// a k that differs from lane to lane
__device__ __forceinline__ void weight_at(int k, double t, double& w, double& dw) {
  const double c0 = k == 1 ? 0.75 : 0.125, c2 = k == 1 ? -1.0 : 0.5;
  const double m = 0.5 * (k - 1) + c2 * t;
  w = c0 + t * m;
  dw = m + c2 * t;
}

// The push terms of one particle (eta = (q/m) xi) in tensor-product form.  With
// eta'_j = eta_j / H_j and derivatives per unit of cell coordinate (S_g = X_a Y_b
// Z_c; the degree-2 second derivatives are 1, -2, 1), w_q the weights of the
// four-point rule of a piece:
//  - per node, three point sums feed the mesh adjoints and the vbar adjoint:
//      Sbar = sum_q w S,  T0 = sum_q w (1 - s) eta'.grad S,  T1 = sum_q w s eta'.grad S
//    (dL/dgphi_l = -dt eta_l Sbar, dL/dA0_l = dt vbar_l T0, dL/dA1_l = dt vbar_l T1;
//    lvbar += dt (A0_g T0 + A1_g T1)); a stencil row (a, b) takes them from three
//    moments each in the z coordinate of the points;
//  - the x and d adjoints, dt / H_k sum_g sum_q w_q (1, s) [b_g(s_q) (eta'.grad)(d_k S_g)
//    - (eta.gphi_g) d_k S_g] with b_g(s) = (1 - s) vbar.A0_g + s vbar.A1_g, need of a
//    row the polynomials in z that its values b0 = vbar.A0, b1 = vbar.A1 and eg =
//    eta.gphi make; their values and derivatives at the points meet the row's x
//    and y factors, which give the Hessian terms.
// With the polynomials in place of the points' z weights a particle fits one lane
// at 256 registers.
// LANES = 1: one lane per particle.  4: lane `part` of a quad takes the stencil
// planes a = part (part = 3: none) of the pieces and of the end points.
template <int LANES, class Nodes>
__device__ __forceinline__ void push_adjoint(const AdjParticleArgs& P, int64_t i, int part,
                                             const Nodes& nodes) {
  const Grid& G = P.G;
  const int64_t np = P.np;
  double x0[3], vb[3], d[3], eta[3], ep[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    x0[a] = P.x[a * np + i];
    vb[a] = P.vb[a * np + i];
    d[a] = P.dt * vb[a];
    eta[a] = P.qm * P.xi[a * np + i];
    ep[a] = eta[a] * G.invH[a];
  }
  // piece terms of lx and ld per unit of cell coordinate (times 1 / H_k below)
  double lx[3] = {0.0, 0.0, 0.0}, ld[3] = {0.0, 0.0, 0.0}, lvb[3] = {0.0, 0.0, 0.0};
  const bool ok = for_each_piece<2>(x0, d, G, [&](double s0, double s1, const double* base) {
    const double len = s1 - s0;
    double sq[4], tx[4], ty[4], tz[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      sq[q] = s0 + 0.5 * len * (1.0 + Gauss<4>::x(q));
      tx[q] = (x0[0] + sq[q] * d[0]) * G.invH[0] - base[0];
      ty[q] = (x0[1] + sq[q] * d[1]) * G.invH[1] - base[1];
      tz[q] = (x0[2] + sq[q] * d[2]) * G.invH[2] - base[2];
    }
    double hw[1] = {0.5 * P.dt * len};  // dt in the weights
    const int fx = to_int_clamped(base[0]) + Spline<2>::first_off;
    const int fy = to_int_clamped(base[1]) + Spline<2>::first_off;
    const int fz = to_int_clamped(base[2]) + Spline<2>::first_off;
#pragma unroll 1
    for (int a = LANES == 1 ? 0 : part; a < 3; a += LANES) {
      const double ex = a == 1 ? -2.0 * ep[0] : ep[0];  // eta'_x X''
#pragma unroll 1
      for (int b = 0; b < 3; ++b) {
        const double ey = b == 1 ? -2.0 * ep[1] : ep[1];  // eta'_y Y''
        recompute_from(hw);
        recompute_from(sq);
        recompute_from(tx);
        recompute_from(ty);
        recompute_from(tz);
        double S[3] = {0.0, 0.0, 0.0}, T0[3] = {0.0, 0.0, 0.0}, T1[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          double X, dX, Y, dY;
          if constexpr (LANES == 1)
            Spline<2>::wk(a, tx[q], X, dX);
          else
            weight_at(a, tx[q], X, dX);
          Spline<2>::wk(b, ty[q], Y, dY);
          const double w = hw[0] * Gauss<4>::w(q), q1 = w * sq[q], q0 = w - q1;
          const double xy = X * Y, pe = ep[0] * (dX * Y) + ep[1] * (X * dY), r = ep[2] * xy;
          const double u0 = w * xy, u1 = u0 * tz[q];
          const double e1 = pe * tz[q] + r, e2 = (e1 + r) * tz[q];
          S[0] += u0;
          S[1] += u1;
          S[2] += u1 * tz[q];
          T0[0] += q0 * pe;
          T0[1] += q0 * e1;
          T0[2] += q0 * e2;
          T1[0] += q1 * pe;
          T1[1] += q1 * e1;
          T1[2] += q1 * e2;
        }
        nodes_of_moments(S);
        nodes_of_moments(T0);
        nodes_of_moments(T1);
        double b0[3], b1[3], eg[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const auto n = nodes.at(fx + a, fy + b, fz + c);
          double f[9];  // grad phi, A^n, A^{n+1}
#pragma unroll
          for (int k = 0; k < 9; ++k) f[k] = nodes.get(n, k);
          b0[c] = b1[c] = eg[c] = 0.0;
#pragma unroll
          for (int l = 0; l < 3; ++l) {
            eg[c] += eta[l] * f[l];
            b0[c] += vb[l] * f[3 + l];
            b1[c] += vb[l] * f[6 + l];
            lvb[l] += f[3 + l] * T0[c] + f[6 + l] * T1[c];
          }
#pragma unroll
          for (int l = 0; l < 3; ++l) {
            nodes.add(n, l, -eta[l] * S[c]);
            nodes.add(n, 3 + l, vb[l] * T0[c]);
            nodes.add(n, 6 + l, vb[l] * T1[c]);
          }
        }
        recompute_from(hw);
        recompute_from(sq);
        recompute_from(tx);
        recompute_from(ty);
        recompute_from(tz);
        coefficients_of_nodes(b0);
        coefficients_of_nodes(b1);
        coefficients_of_nodes(eg);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          double X, dX, Y, dY;
          if constexpr (LANES == 1)
            Spline<2>::wk(a, tx[q], X, dX);
          else
            weight_at(a, tx[q], X, dX);
          Spline<2>::wk(b, ty[q], Y, dY);
          const double t = tz[q], w = hw[0] * Gauss<4>::w(q), q1 = w * sq[q], q0 = w - q1;
          // the row's b(s) and eta.grad phi at the point, with the weight, and their z derivatives
          const double B2 = q0 * b0[2] + q1 * b1[2], B1 = q0 * b0[1] + q1 * b1[1];
          const double m = B1 + t * B2, C = q0 * b0[0] + q1 * b1[0] + t * m, dC = m + t * B2;
          const double k = eg[1] + t * eg[2];
          const double E = w * (eg[0] + t * k), dE = w * (k + t * eg[2]);
          const double g = ep[2] * dC - E, h = 2.0 * ep[2] * B2 - dE;
          const double YC = Y * C, dYC = dY * C;
          const double rx = ex * YC + dX * (ep[1] * dYC + Y * g);
          const double ry = dX * (ep[0] * dYC) + X * (ey * C + dY * g);
          const double rz = ep[0] * (dX * (Y * dC)) + X * (ep[1] * (dY * dC) + Y * h);
          lx[0] += rx;
          lx[1] += ry;
          lx[2] += rz;
          ld[0] += sq[q] * rx;
          ld[1] += sq[q] * ry;
          ld[2] += sq[q] * rz;
        }
      }
    }
  });
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    lx[k] *= G.invH[k];
    ld[k] *= G.invH[k];
  }
  // + A0_h(x0) and - A1_h(x0 + d), end point wrapped
#pragma unroll 1
  for (int end = 0; end < 2; ++end) {
    const double sgn = end ? -1.0 : 1.0;
    const int comp = end ? 6 : 3;
    recompute_from(x0);
    recompute_from(d);
    int first[3];
    Axis2 ax[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double x1 = wrap_pos(x0[a] + d[a], G.L[a], G.invL[a]);
      const double u = (end ? x1 : x0[a]) * G.invH[a];
      const double base = floor(u + Spline<2>::base_off);
      ax[a].at(u - base, G.invH[a]);
      // back to the frame of the unwrapped orbit
      first[a] = to_int_clamped(base) + Spline<2>::first_off +
                 (end ? (int)rint((x0[a] + d[a] - x1) * G.invL[a]) * G.n[a] : 0);
    }
    double e[3] = {0.0, 0.0, 0.0};
#pragma unroll 1
    for (int a = LANES == 1 ? 0 : part; a < 3; a += LANES) {
      const double wx = a == 0 ? ax[0].w[0] : (a == 1 ? ax[0].w[1] : ax[0].w[2]);
      const double dwx = a == 0 ? ax[0].dw[0] : (a == 1 ? ax[0].dw[1] : ax[0].dw[2]);
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        const double wxy = wx * ax[1].w[b];
        double f0 = 0.0, f1 = 0.0;  // the row's eta.A against Z and Z'
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const auto n = nodes.at(first[0] + a, first[1] + b, first[2] + c);
          const double Sg = sgn * (wxy * ax[2].w[c]);
          double eF = 0.0;
#pragma unroll
          for (int l = 0; l < 3; ++l) {
            eF += eta[l] * nodes.get(n, comp + l);
            nodes.add(n, comp + l, eta[l] * Sg);
          }
          f0 += eF * ax[2].w[c];
          f1 += eF * ax[2].dw[c];
        }
        e[0] += dwx * ax[1].w[b] * f0;
        e[1] += wx * ax[1].dw[b] * f0;
        e[2] += wxy * f1;
      }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      lx[k] += sgn * e[k];
      ld[k] += end ? sgn * e[k] : 0.0;
    }
  }
  if (!ok) atomic_max_nonneg(P.sc.spread_copy(S_BAD), 1.0);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if constexpr (LANES == 4) {
      lx[a] = quad_sum(lx[a]);
      ld[a] = quad_sum(ld[a]);
      lvb[a] = quad_sum(lvb[a]);
    }
    if (LANES == 1 || part == a) {
      P.lx[a * np + i] = lx[a];
      P.ld[a * np + i] = ld[a];
      P.lvb[a * np + i] = lvb[a];
    }
  }
}

// The current terms alone (eta = 0: the current's adjoint mu seen by one
// particle), in the tensor-product form of the forward gather: per stencil
// row (a, b) the x and y factors of every quadrature point are formed once,
// and per node only the seven point sums
//   I = sum_q w_q X Y Z,  I_k = sum_q w_q d_k(X Y Z),  I_k^s = sum_q w_q s_q d_k(X Y Z)
// (derivatives per unit of cell coordinate, scaled by 1/H once per particle)
// meet the node's mu:  lvbar += mu_g I,  lx += (vbar . mu_g) I_k,
// ld += (vbar . mu_g) I_k^s.  The same sums as a node-by-node evaluation,
// with about a third of its arithmetic.
// UPDATE false: lx, ld and lvbar are the current's terms.  True: the push's terms
// (written before) are added, lx is stored, and the next iterate xn = b + (lvbar +
// dt ld) / 2 is formed here, with max|xn - xi| and max|xn| into the spread slots
// S_DVMAX and S_VMAX (as separate kernels: 170 us more per iteration at 2,097,152
// particles, zeroing the three arrays included).
template <bool UPDATE>
__device__ __forceinline__ void current_adjoint_one(const AdjParticleArgs& P, int64_t i,
                                                    const double* __restrict__ bvec,
                                                    double* __restrict__ xn, double& dm,
                                                    double& xm) {
  const Grid& G = P.G;
  const int64_t np = P.np, nc = G.ncell;
  double x0[3], vb[3], d[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    x0[a] = P.x[a * np + i];
    vb[a] = P.vb[a * np + i];
    d[a] = P.dt * vb[a];
  }
  double lx[3] = {0.0, 0.0, 0.0}, ld[3] = {0.0, 0.0, 0.0}, lvb[3] = {0.0, 0.0, 0.0};
  const bool ok = for_each_piece<2>(x0, d, G, [&](double s0, double s1, const double* base) {
    const double h = s1 - s0;
    double sq[4], wq[4], tx[4], ty[4], Z[4][3], dZ[4][3];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      sq[q] = s0 + 0.5 * h * (1.0 + Gauss<4>::x(q));
      wq[q] = 0.5 * h * Gauss<4>::w(q);
      tx[q] = (x0[0] + sq[q] * d[0]) * G.invH[0] - base[0];
      ty[q] = (x0[1] + sq[q] * d[1]) * G.invH[1] - base[1];
      Spline<2>::wd((x0[2] + sq[q] * d[2]) * G.invH[2] - base[2], Z[q], dZ[q]);
    }
    const int fx = to_int_clamped(base[0]) + Spline<2>::first_off;
    const int fy = to_int_clamped(base[1]) + Spline<2>::first_off;
    const int fz = to_int_clamped(base[2]) + Spline<2>::first_off;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      double Xw[4], dXw[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        double Xq, dXq;
        Spline<2>::wk(a, tx[q], Xq, dXq);
        Xw[q] = wq[q] * Xq;
        dXw[q] = wq[q] * dXq;
      }
#pragma unroll
      for (int b = 0; b < 3; ++b) {
        double xyw[4], dxyw[4], xdyw[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          double Yq, dYq;
          Spline<2>::wk(b, ty[q], Yq, dYq);
          xyw[q] = Xw[q] * Yq;
          dxyw[q] = dXw[q] * Yq;
          xdyw[q] = Xw[q] * dYq;
        }
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const int64_t g = node_index(G, fx + a, fy + b, fz + c);
          const double m0 = P.mu[g], m1 = P.mu[nc + g], m2 = P.mu[2 * nc + g];
          const double vm = vb[0] * m0 + vb[1] * m1 + vb[2] * m2;
          double I = 0.0, Ix = 0.0, Iy = 0.0, Iz = 0.0, Ixs = 0.0, Iys = 0.0, Izs = 0.0;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const double zx = dxyw[q] * Z[q][c], zy = xdyw[q] * Z[q][c], zz = xyw[q] * dZ[q][c];
            I += xyw[q] * Z[q][c];
            Ix += zx;
            Iy += zy;
            Iz += zz;
            Ixs += sq[q] * zx;
            Iys += sq[q] * zy;
            Izs += sq[q] * zz;
          }
          lvb[0] += m0 * I;
          lvb[1] += m1 * I;
          lvb[2] += m2 * I;
          lx[0] += vm * Ix;
          lx[1] += vm * Iy;
          lx[2] += vm * Iz;
          ld[0] += vm * Ixs;
          ld[1] += vm * Iys;
          ld[2] += vm * Izs;
        }
      }
    }
  });
  if (!ok) atomic_max_nonneg(P.sc.spread_copy(S_BAD), 1.0);
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int64_t e = a * np + i;
    lx[a] *= G.invH[a];
    ld[a] *= G.invH[a];
    if constexpr (UPDATE) {
      P.lx[e] += lx[a];
      const double x = bvec[e] + 0.5 * ((P.lvb[e] + lvb[a]) + P.dt * (P.ld[e] + ld[a]));
      xn[e] = x;
      dm = fmax(dm, fabs(x - P.xi[e]));
      xm = fmax(xm, fabs(x));
      if (!isfinite(x)) dm = INFINITY;
    } else {
      P.lx[e] = lx[a];
      P.ld[e] = ld[a];
      P.lvb[e] = lvb[a];
    }
  }
}

// A wavefront takes eight particles each of eight neighbouring segments, at the same
// place in each: by the segments' order its orbits cross about the same number of
// knots.
template <bool UPDATE>
__global__ __launch_bounds__(kBlock) void k_current_adjoint(AdjParticleArgs P, int segment,
                                                            const double* __restrict__ b,
                                                            double* __restrict__ xn) {
  // segments are powers of two, at least 8
  const int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  const int64_t first = j & ~(int64_t)(8 * segment - 1);  // of the eight segments
  const int lane = (int)j % kWave, row = (int)(j - first) / kWave;
  const int64_t i = first + (lane / 8) * segment + row * 8 + lane % 8;
  double dm = 0.0, xm = 0.0;
  if (i < P.np) current_adjoint_one<UPDATE>(P, i, b, xn, dm, xm);
  if (UPDATE) {
    dm = block_max(dm);
    xm = block_max(xm);
    if (threadIdx.x == 0) {
      atomic_max_nonneg(P.sc.spread_copy(S_DVMAX), dm);
      atomic_max_nonneg(P.sc.spread_copy(S_VMAX), xm);
    }
  }
}
// The push terms over cell-sorted particles, in blocks of P.chunk particles
// whose lanes are spread over P.span, as in the current scatter: the block finds
// the node box of its particles' orbits and end points (clipped to the start
// stencils plus what fits, where the box exceeds the tile), copies the box's
// fields into LDS, sums the nine mesh adjoints of its particles in a second LDS
// array over it, and adds that to global memory once.  Particles that reach beyond
// the box go to P.list, and k_push_adjoint_list takes them from global memory (a
// second path in this kernel cost it registers and scalar spills).
// Rows are padded where that fits (as TileStrides in particles.hip: the 64-bit
// additions of 16 neighbouring lanes then rarely share a bank pair).
// Bound by instruction issue and the LDS about equally (2,097,152 particles of a
// 32^3 mesh: 13,500 vector instructions and 1,490 LDS instructions per wavefront),
// two wavefronts per SIMD.  Measured per launch, one step of the transposed
// iteration: 2220 us with the points' weights held in 512 registers (one wavefront
// per SIMD), 2080 with two lanes per particle, 1720 in this form with a node's nine
// values side by side, 1675 with one plane per value, 1427 with planes 4 mod 16
// apart where rows of 16 do not fit, 1267 with the particles of a lane by the knots that
// they cross (k_segment_order); 32,769 particles of 16^3: 125, 91, and 51 with
// four lanes per particle, 48 in that order.
struct AdjStrides {
  int sy, sx;
  bool fits;
  __device__ __forceinline__ AdjStrides(const int* dim) : sy(1), sx(1), fits(false) {
    // each extent is bounded first so that the products cannot overflow
    if (!(dim[0] > 0 && dim[0] <= kAdjTileNodes && dim[1] <= kAdjTileNodes &&
          dim[2] <= kAdjTileNodes && (int64_t)dim[0] * dim[1] * dim[2] <= kAdjTileNodes))
      return;
    // rows of 16, then rows as they are with planes 4 mod 16 apart, then no padding
    sy = (dim[2] + 15) & ~15;
    sx = dim[1] * sy + 4;
    if (dim[0] * sx > kAdjTileNodes) {
      sy = dim[2];
      sx = ((dim[1] * sy + 11) & ~15) + 4;
    }
    if (dim[0] * sx > kAdjTileNodes) sx = dim[1] * sy;
    fits = true;
  }
};

constexpr int kAdjBlock = 512;

// particle k of this thread in block blk, and the block's first: as chunk_base and
// chunk_particle (reduce.hpp) for groups of LANES lanes
template <int LANES>
__device__ __forceinline__ int64_t group_base(int chunk, int span, int blk) {
  const int per_span = span / chunk;
  return (int64_t)(blk / per_span) * span + (blk % per_span) * (chunk / (kWave / LANES));
}
template <int LANES>
__device__ __forceinline__ int64_t group_particle(int64_t base, int span, int k) {
  constexpr int kGroups = kWave / LANES;
  const int g = (threadIdx.x % kWave) / LANES, seg = 4 * (g % (kGroups / 4)) + g / (kGroups / 4);
  return base + seg * (span / kGroups) + (int)(threadIdx.x / kWave) + (kAdjBlock / kWave) * k;
}

template <int LANES>
__global__ __launch_bounds__(kAdjBlock) __attribute__((
    amdgpu_waves_per_eu(2))) void k_push_adjoint_tiled(AdjParticleArgs P) {
  __shared__ double field[9 * kAdjTileNodes];
  __shared__ double sum[9 * kAdjTileNodes];
  __shared__ int s_ref[3];
  const Grid& G = P.G;
  const int per_thread = P.chunk * LANES / kAdjBlock;
  const int64_t base = group_base<LANES>(P.chunk, P.span, blockIdx.x);
  if (threadIdx.x == 0)
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      // its z, and the middle of the sort's 4 x 4 column in x and y: a block in two
      // columns then stays within half a period of it, also where that is 8 cells.
      // (A span's last blocks may be empty.)
      const double u = P.x[a * P.np + min(base, P.np - 1)] * G.invH[a];
      s_ref[a] = to_int_clamped(floor(u + Spline<2>::base_off));
      if (a < 2) s_ref[a] = (s_ref[a] & ~3) + 1;
    }
  __syncthreads();
  // node boxes: the orbits from x0 to x0 + d (unwrapped), which also hold both end
  // points' stencils, and the start stencils alone
  int mv[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) mv[k] = 0x3fffffff;
  for (int k = 0; k < per_thread; ++k) {
    const int64_t i = group_particle<LANES>(base, P.span, k);
    if (i >= P.np) continue;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      int lo, n, b0;
      orbit_nodes<2>(P.x[a * P.np + i], P.dt * P.vb[a * P.np + i], G.invH[a], lo, n, b0);
      const int rel = min_image(lo - s_ref[a], G.n[a]);
      mv[a] = min(mv[a], rel);
      mv[3 + a] = min(mv[3 + a], -(rel + n));
      mv[6 + a] = min(mv[6 + a], rel + (b0 - lo));
      mv[9 + a] = min(mv[9 + a], -(rel + (b0 - lo) + 3));
    }
  }
  block_min_ints<12, kAdjBlock>(mv);
  int tlo[3], dim[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    tlo[a] = mv[a];
    dim[a] = -mv[3 + a] - tlo[a] + 1;
  }
  if (!AdjStrides(dim).fits) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      tlo[a] = mv[6 + a];
      dim[a] = -mv[9 + a] - tlo[a] + 1;
    }
    for (int e = 0; e < 4; ++e) {  // widened while it fits
      const int wider[3] = {dim[0] + 2, dim[1] + 2, dim[2] + 2};
      if (!AdjStrides(wider).fits) break;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        tlo[a] -= 1;
        dim[a] = wider[a];
      }
    }
  }
  const AdjStrides str(dim);
  if (!str.fits) dim[0] = dim[1] = dim[2] = 0;  // every particle to the list
  const int nt = dim[0] * dim[1] * dim[2];
  const float inv_d1 = 1.0f / (float)max(dim[1], 1), inv_d2 = 1.0f / (float)max(dim[2], 1);
  // node t of the box: its slot in the tile and its place in the mesh
  auto box_node = [&](int t, int& slot, int64_t& g) {
    const int q = div_small(t, inv_d2), cx = div_small(q, inv_d1);
    const int cz = t - q * dim[2], cy = q - cx * dim[1];
    slot = cx * str.sx + cy * str.sy + cz;
    g = node_index(G, s_ref[0] + tlo[0] + cx, s_ref[1] + tlo[1] + cy, s_ref[2] + tlo[2] + cz);
  };
  for (int t = threadIdx.x; t < nt; t += kAdjBlock) {
    int slot;
    int64_t g;
    box_node(t, slot, g);
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      field[slot + k * kAdjTileNodes] = mesh_field(P, k)[g];
      sum[slot + k * kAdjTileNodes] = 0.0;
    }
  }
  __syncthreads();
  for (int k = 0; k < per_thread; ++k) {
    const int64_t i = group_particle<LANES>(base, P.span, k);
    if (i >= P.np) continue;
    TileNodes nodes{(lds_double*)field, (lds_double*)sum, {0, 0, 0}, str.sy, str.sx};
    bool inside = true;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double d = P.dt * P.vb[a * P.np + i];
      int lo, n, b0;
      orbit_nodes<2>(P.x[a * P.np + i], d, G.invH[a], lo, n, b0);
      const int raw = lo - s_ref[a];
      // particle frame -> chunk frame -> tile
      nodes.o[a] = min_image(raw, G.n[a]) - raw - s_ref[a] - tlo[a];
      inside = inside && lo + nodes.o[a] >= 0 && lo + n + nodes.o[a] < dim[a] && d == d;
    }
    if (inside)
      push_adjoint<LANES>(P, i, (int)threadIdx.x % LANES, nodes);
    else if (threadIdx.x % LANES == 0)
      P.list[atomicAdd(P.nlist, 1)] = (int)i;
  }
  __syncthreads();
  for (int t = threadIdx.x; t < nt; t += kAdjBlock) {
    int slot;
    int64_t g;
    box_node(t, slot, g);
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const double val = sum[slot + k * kAdjTileNodes];
      if (val != 0.0) unsafeAtomicAdd(mesh_sum(P, k) + g, val);
    }
  }
}

// The particles of P.list.  Fewer entries than lanes: entry j by block j % grid (few lanes
// per wavefront: every lane reads nodes of its own).  More: neighbouring entries, which lie
// together, to a wavefront.  Per step of five iterations, the first / the second: 524,288 in
// 32^3 with orbits of 0.3 cells 4.93 / 6.02 ms, 20,000 in 64^3 6.80 / 7.94; with orbits of 5
// cells 403 / 335, 131,072 in 16^3 with orbits of 2.5 cells 51.7 / 45.5.
__global__ __launch_bounds__(kBlock) void k_push_adjoint_list(AdjParticleArgs P) {
  const int count = *P.nlist;
  const int64_t lanes = (int64_t)kBlock * gridDim.x;
  const int64_t first = count < lanes ? (int64_t)threadIdx.x * gridDim.x + blockIdx.x
                                      : (int64_t)blockIdx.x * kBlock + threadIdx.x;
  for (int64_t j = first; j < count; j += lanes) push_adjoint<1>(P, P.list[j], 0, MeshNodes{P});
}

// Particles of every segment of `segment` consecutive ones by the knots that their
// orbits cross, the most first, as they come where these are equal.  The lanes of the
// push terms sit in different segments at the same place of each
// (group_particle), and a wavefront runs its orbits in lockstep, as long as its
// longest one: 1.9 pieces for 1.3 per orbit on average (cold beams, 64 per cell).
// 2,097,152 particles, as sorted / in this order: push terms 1454 / 1267 us per launch,
// current terms 450 / 380 us; the order itself takes 80 us once per transposed step.
// One wavefront per segment; it counts first, then moves x, v, w and the ids.
constexpr int kSegCounts = 16;  // 15: fifteen or more
__device__ __forceinline__ int knots_of(const Grid& G, double dt, const Fp64Store& p, int64_t np,
                                        int64_t i) {
  int c = 0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const int64_t e = a * np + i;
    c += min(knots_crossed(p.x[e], dt * (0.5 * (p.vp[e] + p.v[e])), G.invH[a],
                           Spline<2>::base_off),
             kSegCounts);
  }
  return min(c, kSegCounts - 1);
}
__global__ __launch_bounds__(kWave) void k_segment_order(Grid G, double dt, int64_t np, int segment,
                                                        Fp64Store src, Fp64Store dst,
                                                        const int* __restrict__ id,
                                                        int* __restrict__ id2) {
  const int64_t first = (int64_t)blockIdx.x * segment;
  const int n = (int)min((int64_t)segment, np - first);
  const int lane = threadIdx.x;
  int at = 0;  // lane c: particles that cross c knots, then the next place for one
  for (int t = 0; t < n; t += kWave) {
    const bool active = t + lane < n;
    const int c = active ? knots_of(G, dt, src, np, first + t + lane) : -1;
#pragma unroll
    for (int k = 0; k < kSegCounts; ++k) {
      const int m = __popcll(__ballot(c == k));
      at += lane == k ? m : 0;
    }
  }
  int before = 0;
#pragma unroll
  for (int k = 1; k < kSegCounts; ++k) {
    const int m = __builtin_amdgcn_readlane(at, k);
    before += lane < k ? m : 0;
  }
  at = before;
  for (int t = 0; t < n; t += kWave) {
    const bool active = t + lane < n;
    const int c = active ? knots_of(G, dt, src, np, first + t + lane) : -1;
    int place = 0;
#pragma unroll
    for (int k = 0; k < kSegCounts; ++k) {
      const unsigned long long group = __ballot(c == k);
      const int start = __builtin_amdgcn_readlane(at, k);
      place = c == k ? start + __popcll(group & ((1ull << lane) - 1ull)) : place;
      at += lane == k ? __popcll(group) : 0;
    }
    if (active) {
      src.move_to(dst, np, first + t + lane, first + place);
      id2[first + place] = id[first + t + lane];
    }
  }
}

// vbar = (w + v)/2
__global__ __launch_bounds__(kBlock) void k_vbar(int64_t n3, const double* __restrict__ w,
                                                const double* __restrict__ v,
                                                double* __restrict__ vb) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n3) vb[i] = 0.5 * (w[i] + v[i]);
}

// b = lv1 + (lvb + dt (ld + lx1)) / 2, lxacc = lx1 + lx
__global__ __launch_bounds__(kBlock) void k_adjoint_rhs(int64_t n3, double dt,
                                                       const double* __restrict__ lx1,
                                                       const double* __restrict__ lv1,
                                                       const double* __restrict__ lx,
                                                       const double* __restrict__ ld,
                                                       const double* __restrict__ lvb,
                                                       double* __restrict__ b,
                                                       double* __restrict__ lxacc) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n3) return;
  const double x1 = lx1 ? lx1[i] : 0.0;
  b[i] = (lv1 ? lv1[i] : 0.0) + 0.5 * (lvb[i] + dt * (ld[i] + x1));
  lxacc[i] = x1 + lx[i];
}

// lx0 = lxacc + lx, lv0 = 2 xi - lv1
__global__ __launch_bounds__(kBlock) void k_adjoint_out(int64_t n3, const double* __restrict__ lxacc,
                                                       const double* __restrict__ lx,
                                                       const double* __restrict__ xi,
                                                       const double* __restrict__ lv1,
                                                       double* __restrict__ lx0,
                                                       double* __restrict__ lv0) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n3) return;
  lx0[i] = lxacc[i] + lx[i];
  lv0[i] = 2.0 * xi[i] - (lv1 ? lv1[i] : 0.0);
}

}  // namespace

void launch_push_adjoint(hipStream_t s, const AdjParticleArgs& P) {
  if (P.np <= 0) return;
  const unsigned blocks = (unsigned)scatter_blocks(P.np, P.chunk, P.span);
  if (P.chunk >= kAdjBlock)
    k_push_adjoint_tiled<1><<<blocks, kAdjBlock, 0, s>>>(P);
  else
    k_push_adjoint_tiled<4><<<blocks, kAdjBlock, 0, s>>>(P);
  k_push_adjoint_list<<<std::min(blocks_for(P.np), 256u), kBlock, 0, s>>>(P);
}

int adjoint_segment(int chunk, int span) { return span / (chunk >= kAdjBlock ? kWave : kWave / 4); }

void launch_segment_order(hipStream_t s, const Grid& G, double dt, int64_t np, int segment,
                          const Fp64Store& src, const Fp64Store& dst, const int* id, int* id2) {
  if (np > 0)
    k_segment_order<<<(unsigned)((np + segment - 1) / segment), kWave, 0, s>>>(G, dt, np, segment,
                                                                              src, dst, id, id2);
}

void launch_current_adjoint(hipStream_t s, const AdjParticleArgs& P, const double* b, double* xn) {
  if (P.np <= 0) return;
  const int segment = adjoint_segment(P.chunk, P.span);
  const int64_t per = std::max(8 * segment, kBlock);  // whole groups of eight segments
  const unsigned blocks = (unsigned)((P.np + per - 1) / per * (per / kBlock));
  if (b)
    k_current_adjoint<true><<<blocks, kBlock, 0, s>>>(P, segment, b, xn);
  else
    k_current_adjoint<false><<<blocks, kBlock, 0, s>>>(P, segment, nullptr, nullptr);
}

void launch_vbar(hipStream_t s, int64_t n3, const double* w, const double* v, double* vb) {
  if (n3 > 0) k_vbar<<<blocks_for(n3), kBlock, 0, s>>>(n3, w, v, vb);
}

void launch_adjoint_rhs(hipStream_t s, int64_t n3, double dt, const double* lx1, const double* lv1,
                        const double* lx, const double* ld, const double* lvb, double* b,
                        double* lxacc) {
  if (n3 > 0) k_adjoint_rhs<<<blocks_for(n3), kBlock, 0, s>>>(n3, dt, lx1, lv1, lx, ld, lvb, b, lxacc);
}

void launch_adjoint_out(hipStream_t s, int64_t n3, const double* lxacc, const double* lx,
                        const double* xi, const double* lv1, double* lx0, double* lv0) {
  if (n3 > 0) k_adjoint_out<<<blocks_for(n3), kBlock, 0, s>>>(n3, lxacc, lx, xi, lv1, lx0, lv0);
}

}  // namespace ecpic
