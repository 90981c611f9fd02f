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
// in the block's LDS tile over its particles' node box, or in global memory for
// a node outside the box.  at() takes the node in the particle's unwrapped frame
// (ix, iy, iz).  The tile pointers carry the LDS address space, so the additions
// are LDS atomics (through a plain pointer they compiled to flat atomics, the
// slower path that serves either memory).
typedef __attribute__((address_space(3))) double lds_double;
struct AdjNode {
  int t;      // first of the node's nine values in the tile, negative outside it
  int64_t g;  // flat index in the mesh
};
struct AdjTile {
  const AdjParticleArgs* P;
  lds_double* field;
  lds_double* sum;
  int o[3], dim[3];  // particle's frame -> tile, extents (0: no tile)
  int sy, sx;        // nodes between neighbours along y and x; along z 1
  __device__ __forceinline__ AdjNode at(int ix, int iy, int iz) const {
    const int tx = ix + o[0], ty = iy + o[1], tz = iz + o[2];
    const bool in = tx >= 0 && ty >= 0 && tz >= 0 && tx < dim[0] && ty < dim[1] && tz < dim[2];
    return {in ? 9 * (tx * sx + ty * sy + tz) : -1, node_index(P->G, ix, iy, iz)};
  }
  __device__ __forceinline__ const double* global_field(int k) const {
    return (k < 3 ? P->gphi : (k < 6 ? P->A0 : P->A1)) + (int64_t)(k % 3) * P->G.ncell;
  }
  __device__ __forceinline__ double* global_sum(int k) const {
    return (k < 3 ? P->lgphi : (k < 6 ? P->lA0 : P->lA1)) + (int64_t)(k % 3) * P->G.ncell;
  }
  template <int K0, int N>
  __device__ __forceinline__ void load(const AdjNode& n, double (&f)[N]) const {
    if (n.t >= 0) {
#pragma unroll
      for (int k = 0; k < N; ++k) f[k] = field[n.t + K0 + k];
    } else {
#pragma unroll
      for (int k = 0; k < N; ++k) f[k] = global_field(K0 + k)[n.g];
    }
  }
  template <int K0, int N>
  __device__ __forceinline__ void add(const AdjNode& n, const double (&v)[N]) const {
    if (n.t >= 0) {
#pragma unroll
      for (int k = 0; k < N; ++k)
        __hip_atomic_fetch_add(&sum[n.t + K0 + k], v[k], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
    } else {
#pragma unroll
      for (int k = 0; k < N; ++k) unsafeAtomicAdd(global_sum(K0 + k) + n.g, v[k]);
    }
  }
};

// The push terms of particle i (eta = (q/m) xi) in tensor-product form.
// With eta'_j = eta_j / H_j and derivatives per unit of cell coordinate
// (S_g = X_a Y_b Z_c; the degree-2 second derivatives are 1, -2, 1):
//  - per node, three point sums feed the mesh adjoints and the vbar adjoint:
//      Sbar = sum_q w S,  T0 = sum_q w (1 - s) eta'.grad S,  T1 = sum_q w s eta'.grad S
//    (dL/dgphi_l = -dt eta_l Sbar, dL/dA0_l = dt vbar_l T0, dL/dA1_l = dt vbar_l T1;
//    lvbar += dt (A0_g T0 + A1_g T1));
//  - the x and d adjoints, dt / H_k sum_g sum_q w_q (1, s) [b_g(s_q) (eta'.grad)(d_k S_g)
//    - (eta.gphi_g) d_k S_g] with b_g(s) = (1 - s) vbar.A0_g + s vbar.A1_g, need
//    per stencil row only the z-column sums of b0 = vbar.A0, b1 = vbar.A1 and
//    eg = eta.gphi against Z and Z' at each point (and against Z'', the same at
//    every point); the row's x and y factors then give the Hessian terms.
// The same sums as a node-by-node evaluation, with about a quarter of its
// arithmetic.
__device__ __forceinline__ void push_adjoint(const AdjParticleArgs& P, int64_t i,
                                             const AdjTile& tile) {
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
  // piece terms of lx and ld per unit of cell coordinate (times dt / H_k below)
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
#pragma unroll 1
    for (int a = 0; a < 3; ++a) {
      const double ddX = a == 1 ? -2.0 : 1.0;
      double Xq[4], dXq[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) Spline<2>::wk(a, tx[q], Xq[q], dXq[q]);
#pragma unroll 1
      for (int b = 0; b < 3; ++b) {
        const double ddY = b == 1 ? -2.0 : 1.0;
        double Yq[4], dYq[4], xy[4], dxy[4], xdy[4], pe[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          Spline<2>::wk(b, ty[q], Yq[q], dYq[q]);
          xy[q] = Xq[q] * Yq[q];
          dxy[q] = dXq[q] * Yq[q];
          xdy[q] = Xq[q] * dYq[q];
          pe[q] = ep[0] * dxy[q] + ep[1] * xdy[q];  // (eta'_x d_x + eta'_y d_y)(X Y)
        }
        double C0[4], C0d[4], C1[4], C1d[4], Eg[4], Egd[4], C0dd = 0.0, C1dd = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const double ddZ = c == 1 ? -2.0 : 1.0;
          const AdjNode node = tile.at(fx + a, fy + b, fz + c);
          double f[9];  // grad phi, A^n, A^{n+1}
          tile.load<0>(node, f);
          double b0 = 0.0, b1 = 0.0, eg = 0.0;
#pragma unroll
          for (int l = 0; l < 3; ++l) {
            b0 += vb[l] * f[3 + l];
            b1 += vb[l] * f[6 + l];
            eg += eta[l] * f[l];
          }
          double Sbar = 0.0, T0 = 0.0, T1 = 0.0;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const double z = Z[q][c], dz = dZ[q][c];
            C0[q] = c == 0 ? b0 * z : C0[q] + b0 * z;
            C0d[q] = c == 0 ? b0 * dz : C0d[q] + b0 * dz;
            C1[q] = c == 0 ? b1 * z : C1[q] + b1 * z;
            C1d[q] = c == 0 ? b1 * dz : C1d[q] + b1 * dz;
            Eg[q] = c == 0 ? eg * z : Eg[q] + eg * z;
            Egd[q] = c == 0 ? eg * dz : Egd[q] + eg * dz;
            const double edS = pe[q] * z + ep[2] * xy[q] * dz;  // eta'.grad S
            Sbar += wq[q] * xy[q] * z;
            T0 += wq[q] * (1.0 - sq[q]) * edS;
            T1 += wq[q] * sq[q] * edS;
          }
          C0dd += b0 * ddZ;
          C1dd += b1 * ddZ;
          double v[9];
#pragma unroll
          for (int l = 0; l < 3; ++l) {
            lvb[l] += P.dt * (f[3 + l] * T0 + f[6 + l] * T1);
            v[l] = -P.dt * eta[l] * Sbar;
            v[3 + l] = P.dt * vb[l] * T0;
            v[6 + l] = P.dt * vb[l] * T1;
          }
          tile.add<0>(node, v);
        }
        // the row's share of sum_g b (eta'.grad)(d_k S_g) (with b0 and b1) and
        // of sum_g eg d_k S_g, per point
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const double dxdy = dXq[q] * dYq[q];
          // (eta'.grad)(d_k S) summed over the row against b0 and b1
          const double hx = ep[0] * ddX * Yq[q] + ep[1] * dxdy;     // with Z
          const double hy = ep[0] * dxdy + ep[1] * Xq[q] * ddY;     // with Z
          const double u0x = hx * C0[q] + ep[2] * dxy[q] * C0d[q];
          const double u0y = hy * C0[q] + ep[2] * xdy[q] * C0d[q];
          const double u0z = pe[q] * C0d[q] + ep[2] * xy[q] * C0dd;
          const double u1x = hx * C1[q] + ep[2] * dxy[q] * C1d[q];
          const double u1y = hy * C1[q] + ep[2] * xdy[q] * C1d[q];
          const double u1z = pe[q] * C1d[q] + ep[2] * xy[q] * C1dd;
          // d_k S summed over the row against eg
          const double vx = dxy[q] * Eg[q], vy = xdy[q] * Eg[q], vz = xy[q] * Egd[q];
          const double q0 = wq[q] * (1.0 - sq[q]), q1 = wq[q] * sq[q];
          lx[0] += q0 * u0x + q1 * u1x - wq[q] * vx;
          lx[1] += q0 * u0y + q1 * u1y - wq[q] * vy;
          lx[2] += q0 * u0z + q1 * u1z - wq[q] * vz;
          ld[0] += sq[q] * (q0 * u0x + q1 * u1x - wq[q] * vx);
          ld[1] += sq[q] * (q0 * u0y + q1 * u1y - wq[q] * vy);
          ld[2] += sq[q] * (q0 * u0z + q1 * u1z - wq[q] * vz);
        }
      }
    }
  });
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    lx[k] *= P.dt * G.invH[k];
    ld[k] *= P.dt * G.invH[k];
  }
  // + A0_h(x0) - A1_h(x0 + d), end point wrapped
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const double sgn = e == 0 ? 1.0 : -1.0;
    double base[3];
    int first[3], sh[3];
    Axis2 ax[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      const double xp = e == 0 ? x0[a] : wrap_pos(x0[a] + d[a], G.L[a], G.invL[a]);
      const double u = xp * G.invH[a];
      base[a] = floor(u + Spline<2>::base_off);
      first[a] = to_int_clamped(base[a]) + Spline<2>::first_off;
      ax[a].at(u - base[a], G.invH[a]);
      // periods between the wrapped end point and the unwrapped orbit end
      sh[a] = e == 0 ? 0 : (int)rint((x0[a] + d[a] - xp) * G.invL[a]) * G.n[a];
    }
    for (int a = 0; a < 3; ++a)
      for (int b = 0; b < 3; ++b)
        for (int c = 0; c < 3; ++c) {
          const AdjNode node =
              tile.at(first[0] + a + sh[0], first[1] + b + sh[1], first[2] + c + sh[2]);
          const double S = ax[0].w[a] * ax[1].w[b] * ax[2].w[c];
          const double dS[3] = {ax[0].dw[a] * ax[1].w[b] * ax[2].w[c],
                                ax[0].w[a] * ax[1].dw[b] * ax[2].w[c],
                                ax[0].w[a] * ax[1].w[b] * ax[2].dw[c]};
          double f[3], v[3];
          if (e == 0)
            tile.load<3>(node, f);
          else
            tile.load<6>(node, f);
          double eF = 0.0;
#pragma unroll
          for (int l = 0; l < 3; ++l) {
            eF += eta[l] * f[l];
            v[l] = sgn * eta[l] * S;
          }
          if (e == 0)
            tile.add<3>(node, v);
          else
            tile.add<6>(node, v);
#pragma unroll
          for (int kk = 0; kk < 3; ++kk) {
            lx[kk] += sgn * eF * dS[kk];
            if (e == 1) ld[kk] += sgn * eF * dS[kk];
          }
        }
  }
  if (!ok) P.bad[0] = 1.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    P.lx[a * np + i] += lx[a];
    P.ld[a * np + i] += ld[a];
    P.lvb[a * np + i] += lvb[a];
  }
}

// The current terms alone (eta = 0: the current's adjoint mu seen by one
// particle), in the tensor-product form of the forward gather: per stencil
// row (a, b) the x and y factors of every quadrature point are formed once,
// and per node only the seven point sums
//   I = sum_q w_q X Y Z,  I_k = sum_q w_q d_k(X Y Z),  I_k^s = sum_q w_q s_q d_k(X Y Z)
// (derivatives per unit of cell coordinate, scaled by 1/H once per particle)
// meet the node's mu:  lvbar += mu_g I,  lx += (vbar . mu_g) I_k,
// ld += (vbar . mu_g) I_k^s.  The same sums as the node-by-node form above,
// with about a third of its arithmetic.
__global__ __launch_bounds__(kBlock) void k_current_adjoint(AdjParticleArgs P) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i >= P.np) return;
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
  if (!ok) P.bad[0] = 1.0;
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    P.lx[a * np + i] += lx[a] * G.invH[a];
    P.ld[a * np + i] += ld[a] * G.invH[a];
    P.lvb[a * np + i] += lvb[a];
  }
}

// The push terms over cell-sorted particles, in blocks of P.chunk particles
// whose lanes are spread over P.span, as in the current scatter: the block finds
// the node box of its particles' orbits and end points (clipped to the start
// stencils plus what fits, where the box exceeds the tile), copies the box's
// fields into LDS, sums the nine mesh adjoints of its particles in a second LDS
// array over it, and adds that to global memory once.  The kernel runs at one
// wavefront per SIMD (its registers), so one block per CU loses nothing to the
// 144 KB.
// Rows are padded where that fits (as TileStrides in particles.hip: the 64-bit
// additions of 16 neighbouring lanes then rarely share a bank pair).
constexpr int kAdjTileNodes = 1000;

struct AdjStrides {
  int sy, sx;
  bool fits;
  __device__ __forceinline__ AdjStrides(const int* dim) : sy(1), sx(1), fits(false) {
    // each extent is bounded first so that the products cannot overflow
    if (!(dim[0] > 0 && dim[0] <= kAdjTileNodes && dim[1] <= kAdjTileNodes &&
          dim[2] <= kAdjTileNodes))
      return;
    sy = (dim[2] + 15) & ~15;
    sx = dim[1] * sy + 4;
    if ((int64_t)dim[0] * sx > kAdjTileNodes) {
      sy = dim[2];
      sx = dim[1] * sy;
    }
    fits = (int64_t)dim[0] * sx <= kAdjTileNodes;
  }
};

__global__ __launch_bounds__(kBlock) void k_push_adjoint_tiled(AdjParticleArgs P) {
  __shared__ double field[9 * kAdjTileNodes];
  __shared__ double sum[9 * kAdjTileNodes];
  __shared__ int s_ref[3];
  const Grid& G = P.G;
  const int per_thread = P.chunk / kBlock;
  const int64_t base = chunk_base(P.chunk, P.span, blockIdx.x);
  if (threadIdx.x == 0)
#pragma unroll
    for (int a = 0; a < 3; ++a)  // a span's last blocks may be empty
      s_ref[a] = to_int_clamped(
          floor(P.x[a * P.np + min(base, P.np - 1)] * G.invH[a] + Spline<2>::base_off));
  __syncthreads();
  // node boxes: the orbits from x0 to x0 + d (unwrapped), which also hold both end
  // points' stencils, and the start stencils alone
  int mv[12];
#pragma unroll
  for (int k = 0; k < 12; ++k) mv[k] = 0x3fffffff;
  for (int k = 0; k < per_thread; ++k) {
    const int64_t i = chunk_particle(base, P.span, k);
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
  block_min_ints<12>(mv);
  AdjTile tile{&P, (lds_double*)field, (lds_double*)sum, {0, 0, 0}, {0, 0, 0}, 1, 1};
  int tlo[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    tlo[a] = mv[a];
    tile.dim[a] = -mv[3 + a] - tlo[a] + 1;
  }
  if (!AdjStrides(tile.dim).fits) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      tlo[a] = mv[6 + a];
      tile.dim[a] = -mv[9 + a] - tlo[a] + 1;
    }
    for (int e = 0; e < 4; ++e) {  // widened while it fits
      const int wider[3] = {tile.dim[0] + 2, tile.dim[1] + 2, tile.dim[2] + 2};
      if (!AdjStrides(wider).fits) break;
#pragma unroll
      for (int a = 0; a < 3; ++a) {
        tlo[a] -= 1;
        tile.dim[a] = wider[a];
      }
    }
  }
  const AdjStrides str(tile.dim);
  tile.sy = str.sy;
  tile.sx = str.sx;
  if (!str.fits) tile.dim[0] = tile.dim[1] = tile.dim[2] = 0;  // every node in global memory
  const int nt = tile.dim[0] * tile.dim[1] * tile.dim[2];
  const float inv_d1 = 1.0f / (float)max(tile.dim[1], 1), inv_d2 = 1.0f / (float)max(tile.dim[2], 1);
  // node t of the box: its slot in the tile and its place in the mesh
  auto box_node = [&](int t, int& slot, int64_t& g) {
    const int q = div_small(t, inv_d2), cx = div_small(q, inv_d1);
    const int cz = t - q * tile.dim[2], cy = q - cx * tile.dim[1];
    slot = 9 * (cx * tile.sx + cy * tile.sy + cz);
    g = node_index(G, s_ref[0] + tlo[0] + cx, s_ref[1] + tlo[1] + cy, s_ref[2] + tlo[2] + cz);
  };
  for (int t = threadIdx.x; t < nt; t += kBlock) {
    int slot;
    int64_t g;
    box_node(t, slot, g);
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      field[slot + k] = tile.global_field(k)[g];
      sum[slot + k] = 0.0;
    }
  }
  __syncthreads();
  for (int k = 0; k < per_thread; ++k) {
    const int64_t i = chunk_particle(base, P.span, k);
    if (i >= P.np) continue;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      int lo, n, b0;
      orbit_nodes<2>(P.x[a * P.np + i], P.dt * P.vb[a * P.np + i], G.invH[a], lo, n, b0);
      const int raw = lo - s_ref[a];
      // particle frame -> chunk frame -> tile
      tile.o[a] = min_image(raw, G.n[a]) - raw - s_ref[a] - tlo[a];
    }
    push_adjoint(P, i, tile);
  }
  __syncthreads();
  for (int t = threadIdx.x; t < nt; t += kBlock) {
    int slot;
    int64_t g;
    box_node(t, slot, g);
#pragma unroll
    for (int k = 0; k < 9; ++k) {
      const double val = sum[slot + k];
      if (val != 0.0) unsafeAtomicAdd(tile.global_sum(k) + g, val);
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

// xn = b + (lvb + dt ld)/2; max|xn - xi| and max|xn| into red[0], red[1]
__global__ __launch_bounds__(kBlock) void k_adjoint_update(int64_t n3, double dt,
                                                          const double* __restrict__ b,
                                                          const double* __restrict__ lvb,
                                                          const double* __restrict__ ld,
                                                          const double* __restrict__ xi,
                                                          double* __restrict__ xn,
                                                          double* __restrict__ red) {
  double dm = 0.0, xm = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n3;
       i += (int64_t)gridDim.x * kBlock) {
    const double x = b[i] + 0.5 * (lvb[i] + dt * ld[i]);
    xn[i] = x;
    dm = fmax(dm, fabs(x - xi[i]));
    xm = fmax(xm, fabs(x));
    if (!isfinite(x)) dm = INFINITY;
  }
  block_max_to(dm, red);
  block_max_to(xm, red + 1);
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

void launch_particle_adjoint(hipStream_t s, const AdjParticleArgs& P, bool eta, bool mu) {
  if (P.np <= 0) return;
  if (eta)
    k_push_adjoint_tiled<<<(unsigned)scatter_blocks(P.np, P.chunk, P.span), kBlock, 0, s>>>(P);
  if (mu) k_current_adjoint<<<blocks_for(P.np), kBlock, 0, s>>>(P);
}

void launch_vbar(hipStream_t s, int64_t n3, const double* w, const double* v, double* vb) {
  if (n3 > 0) k_vbar<<<blocks_for(n3), kBlock, 0, s>>>(n3, w, v, vb);
}

void launch_adjoint_rhs(hipStream_t s, int64_t n3, double dt, const double* lx1, const double* lv1,
                        const double* lx, const double* ld, const double* lvb, double* b,
                        double* lxacc) {
  if (n3 > 0) k_adjoint_rhs<<<blocks_for(n3), kBlock, 0, s>>>(n3, dt, lx1, lv1, lx, ld, lvb, b, lxacc);
}

void launch_adjoint_update(hipStream_t s, int64_t n3, double dt, const double* b,
                           const double* lvb, const double* ld, const double* xi, double* xn,
                           double* red) {
  // a grid of at most 1024 blocks: every block adds its two maxima to the
  // same two words, so fewer blocks mean fewer contended atomics
  if (n3 > 0)
    k_adjoint_update<<<std::min(blocks_for(n3), 1024u), kBlock, 0, s>>>(n3, dt, b, lvb, ld, xi, xn,
                                                                        red);
}

void launch_adjoint_out(hipStream_t s, int64_t n3, const double* lxacc, const double* lx,
                        const double* xi, const double* lv1, double* lx0, double* lv0) {
  if (n3 > 0) k_adjoint_out<<<blocks_for(n3), kBlock, 0, s>>>(n3, lxacc, lx, xi, lv1, lx0, lv0);
}

}  // namespace ecpic
