// Mesh-side kernels for gfx950: batched radix-2 FFT passes in LDS, the
// per-mode continuity + Crank-Nicolson update, the initial Poisson solve and
// the Parseval / constraint reductions.
//
// Spectral fields are full complex spectra data[b*ncell + g] with the node /
// mode index g = (ix*Ny + iy)*Nz + iz.  The Fourier symbol of d/dx_a at mode
// index m is i k~ with k~ = 2 pi m_s / L_a, m_s the signed index, and
// k~ = 0 on the Nyquist index; Delta_h -> -|k~|^2 (Sec. 3.3).  Forward
// transforms are unnormalised; the 1/ncell of the inverse is folded into the
// kernel that prepares its input.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "internal.hpp"
#include "reduce.hpp"

namespace ecpic {

namespace {

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cscale(double2 a, double s) { return make_double2(a.x * s, a.y * s); }
// i * k * a
__device__ __forceinline__ double2 ik(double k, double2 a) { return make_double2(-k * a.y, k * a.x); }

__device__ __forceinline__ int brev(int e, int logn) {
  return (int)(__brev((unsigned)e) >> (32 - logn));
}

// w v, or conj(w) v, with the products rounded in a fixed order: the same bits
// whichever kernel a transform runs in (in the mixed form the rounding of the
// accepted velocities is keyed by the stored bits, down to transverse velocities
// that are themselves rounding).
template <bool CONJ>
__device__ __forceinline__ double2 twiddle(double2 w, double2 v) {
#pragma clang fp contract(off)
  if (CONJ)
    return make_double2(__builtin_fma(w.x, v.x, w.y * v.y), __builtin_fma(w.x, v.y, -(w.y * v.x)));
  return make_double2(__builtin_fma(w.x, v.x, -(w.y * v.y)), __builtin_fma(w.y, v.x, w.x * v.y));
}

// LDS slot of point e of a run: one slot of padding every 8 points, so that
// threads that hold 8 neighbouring points each, and bit-reversed writes, do not
// share a bank
__device__ __forceinline__ int pad8(int e) { return e + (e >> 3); }

// Transforms of pencils of N = 2^logN points held in LDS: radix-2 decimation in
// time on bit-reversed input, up to three stages at a time in registers (8
// points per thread and LDS round trip, one barrier for the three).  Pencil p's
// point e is at(p, e); count pencils (a power of two if ACROSS), all threads of
// the block; tw: the table exp(-2 pi i t / N), t < N/2 (in LDS or global memory),
// conjugated for INV.  Neighbouring threads take neighbouring groups of one
// pencil, or with ACROSS the same group of neighbouring pencils.  Ends with a
// barrier.
template <bool INV, bool ACROSS, int S, class At>
__device__ __forceinline__ void fft_stages(int N, int logN, int count, int loghs,
                                           const double2* tw, At&& at) {
  constexpr int R = 1 << S;
  const int logper = logN - S, per = 1 << logper;  // groups of R points per pencil
  const int hs = 1 << loghs, logcount = 31 - __clz(count);
  for (int u = threadIdx.x; u < count * per; u += blockDim.x) {
    const int p = ACROSS ? u & (count - 1) : u >> logper;
    const int j = ACROSS ? u >> logcount : u & (per - 1);
    const int pos = j & (hs - 1), i0 = ((j >> loghs) << (loghs + S)) + pos;
    double2 v[R];
#pragma unroll
    for (int m = 0; m < R; ++m) v[m] = at(p, i0 + m * hs);
#pragma unroll
    for (int st = 0; st < S; ++st) {
      const int h = 1 << st;
#pragma unroll
      for (int k = 0; k < h; ++k) {  // the twiddle of stage loghs + st at pos + k hs
        const double2 w = tw[(pos + k * hs) << (logN - 1 - loghs - st)];
#pragma unroll
        for (int m = k; m < R; m += 2 * h) {
          const double2 x = v[m], y = twiddle<INV>(w, v[m + h]);
          v[m] = cadd(x, y);
          v[m + h] = csub(x, y);
        }
      }
    }
#pragma unroll
    for (int m = 0; m < R; ++m) at(p, i0 + m * hs) = v[m];
  }
  __syncthreads();
}

template <bool INV, bool ACROSS, class At>
__device__ __forceinline__ void fft_pencils(int N, int logN, int count, const double2* tw,
                                            At&& at) {
  int done = 0;
  while (logN - done >= 5 || logN - done == 3) {
    fft_stages<INV, ACROSS, 3>(N, logN, count, done, tw, at);
    done += 3;
  }
  while (logN > done) {  // 2 or 4 stages left, N being 4 to 256
    fft_stages<INV, ACROSS, 2>(N, logN, count, done, tw, at);
    done += 2;
  }
}

struct FftPass {
  const double2* src;  // complex input of MODE 0 and 2 (may be data), times scale
  double scale;
  double2* data;
  const double2* tw;  // exp(-2 pi i t / N), t < N/2
  int64_t ncell;
  int64_t stride;     // distance between consecutive elements of a pencil
  int64_t npb;        // pencils per batch field = ncell / N
  int64_t npencils;   // nb * npb
  int N, logN, logS;  // logS = log2(stride)
  int logpts;         // log2 of the points per block
  RealIO io;          // real input (forward first pass) or output (inverse last pass)
  const double* prev; // optional: max |in - prev| -> S_DJMAX (a spread slot)
  double* clear;      // optional: real buffer (same layout as prev) zeroed by the pass
  Scratch sc;
};

// MODE 0: complex to complex; 1: real input -> complex; 2: complex -> real output.
// A block holds 2^logpts points, P = 2^logpts / N neighbouring pencils: 2048, so
// that a strided pass moves runs of at least 8 points (128 bytes; with 512 points
// per block the y and x passes at 128^3 moved 64-byte runs at 2.5 TB/s), or 512
// where 2048 would leave compute units without a block (launch_pass).
constexpr int kFftPoints = 2048;

template <int MODE, bool INV>
__global__ __launch_bounds__(kBlock) void k_fft(FftPass A) {
  // P runs of N + N / 8 + 1 slots, P <= kFftPoints / 4
  __shared__ double2 buf[kFftPoints + kFftPoints / 8 + kFftPoints / 4];
  __shared__ double2 tw[128];
  const int N = A.N, logP = A.logpts - A.logN, P = 1 << logP, ld = pad8(N) + 1;
  const int points = 1 << A.logpts;
  for (int t = threadIdx.x; t < N / 2; t += kBlock) tw[t] = A.tw[t];
  const int64_t first = (int64_t)blockIdx.x << logP;
  const int count = (int)min((int64_t)P, A.npencils - first);
  const int lognpb = 63 - __clzll((unsigned long long)A.npb);
  // element u of the block: pencil and position, neighbouring threads at
  // neighbouring addresses
  auto place = [&](int u, int& pl, int& e, int64_t& b, int64_t& g) {
    if (A.stride == 1) {
      pl = u >> A.logN;
      e = u & (N - 1);
    } else {
      pl = u & (P - 1);
      e = u >> logP;
    }
    const int64_t pencil = first + pl;
    b = pencil >> lognpb;
    const int64_t pin = pencil & (A.npb - 1);
    const int64_t outer = pin >> A.logS, inner = pin & (A.stride - 1);
    g = (((outer << A.logN) + e) << A.logS) + inner;
  };
  double dmax = 0.0;
  for (int u = threadIdx.x; u < points; u += kBlock) {
    int pl, e;
    int64_t b, g;
    place(u, pl, e, b, g);
    if (pl >= count) continue;
    double2 val;
    if constexpr (MODE == 1) {
      const double re = A.io.p[b][g * A.io.stride[b]];
      if (A.prev) dmax = fmax(dmax, fabs(re - A.prev[b * A.ncell + g]));
      if (A.clear) A.clear[b * A.ncell + g] = 0.0;  // after prev was read (same element)
      val = make_double2(re, 0.0);
    } else {
      val = cscale(A.src[b * A.ncell + g], A.scale);
    }
    buf[pl * ld + pad8(brev(e, A.logN))] = val;
  }
  __syncthreads();
  fft_pencils<INV, false>(N, A.logN, count, tw,
                          [&](int p, int e) -> double2& { return buf[p * ld + pad8(e)]; });
  for (int u = threadIdx.x; u < points; u += kBlock) {
    int pl, e;
    int64_t b, g;
    place(u, pl, e, b, g);
    if (pl >= count) continue;
    if constexpr (MODE == 2)
      A.io.p[b][g * A.io.stride[b]] = buf[pl * ld + pad8(e)].x;
    else
      A.data[b * A.ncell + g] = buf[pl * ld + pad8(e)];
  }
  if constexpr (MODE == 1) {
    if (A.prev) {
      const double r = block_max(dmax);
      if (threadIdx.x == 0) atomic_max_nonneg(A.sc.spread_copy(S_DJMAX), r);
    }
  }
}

__device__ __forceinline__ double ktil(int m, int N, double L) {
  if (2 * m == N) return 0.0;
  const int ms = (2 * m < N) ? m : m - N;
  return 6.283185307179586476925286766559 * (double)ms / L;
}

__device__ __forceinline__ void mode_k(const Grid& G, int64_t g, double* k) {
  const int iz = (int)g & G.mask[2];
  const int iy = ((int)g >> G.shy) & G.mask[1];
  const int ix = (int)g >> G.shx;
  k[0] = ktil(ix, G.n[0], G.L[0]);
  k[1] = ktil(iy, G.n[1], G.L[1]);
  k[2] = ktil(iz, G.n[2], G.L[2]);
}

// field order in a spectral level: phi, psi, Ax, Ay, Az, Ux, Uy, Uz, rho
enum { F_PHI = 0, F_PSI = 1, F_A = 2, F_U = 5, F_RHO = 8 };

// |E|^2 / (2 sigma1) + |B|^2 / (2 sigma2) of one mode (E = -i k phi - U, B = i k x A)
__device__ __forceinline__ double mode_energy(const double* k, double2 phi, const double2* A,
                                              const double2* U, double h1, double h2) {
  double e = 0.0;
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    const double2 E = csub(make_double2(k[l] * phi.y, -k[l] * phi.x), U[l]);
    e += h1 * (E.x * E.x + E.y * E.y);
  }
  const double2 B0 = csub(ik(k[1], A[2]), ik(k[2], A[1]));
  const double2 B1 = csub(ik(k[2], A[0]), ik(k[0], A[2]));
  const double2 B2 = csub(ik(k[0], A[1]), ik(k[1], A[0]));
  e += h2 * (B0.x * B0.x + B0.y * B0.y + B1.x * B1.x + B1.y * B1.y + B2.x * B2.x + B2.y * B2.y);
  return e;
}

// Continuity (eq. cn-continuity) and CN (eq. cn-field-update) for every mode:
//   rho1 = rho0 - dt i k.J,  rho_h = (rho0 + rho1)/2,
//   psi1 = [(1 - a^2 w^2) psi0 - 2 a w^2 phi0 + dt kappa^2 sigma1 rho_h] / (1 + a^2 w^2),
//   phi1 = phi0 + a (psi0 + psi1),  a = dt/2, w^2 = kappa^2 |k|^2,
// and (A_l, U_l) likewise with sigma2 J_l.  The closed form is the exact
// inverse of the 2x2 CN system of each (value, rate) pair.
// One mode: c = the 9 level-n spectra (field order of a level), J = the 3
// current spectra; out = the 9 level-(n+1) spectra, inv = the inverse-transform
// inputs [i k phi^{n+1/2} (3), A^{n+1} (3)] / ncell, sums = JE, W^{n+1} and
// W^{n+1} - W^n of this mode (times dV / ncell, Parseval).
__device__ __forceinline__ void cn_mode(const FieldParams& F, const double* k, const double2* J,
                                        const double2* c, double2* out, double2* inv,
                                        double* sums) {
  const Grid& G = F.G;
  const double dt = F.dt, a = 0.5 * dt, kap2 = F.kappa * F.kappa;
  const double w2 = kap2 * (k[0] * k[0] + k[1] * k[1] + k[2] * k[2]);
  const double inv_den = 1.0 / (1.0 + a * a * w2);
  const double c_old = 1.0 - a * a * w2, c_x = 2.0 * a * w2;
  double2 A0[3], U0[3], A1[3], U1[3];
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    A0[l] = c[F_A + l];
    U0[l] = c[F_U + l];
  }
  const double2 phi0 = c[F_PHI], psi0 = c[F_PSI], rho0 = c[F_RHO];
  const double2 divJ = cadd(cadd(ik(k[0], J[0]), ik(k[1], J[1])), ik(k[2], J[2]));
  const double2 rho1 = csub(rho0, cscale(divJ, dt));
  const double2 rhoh = cscale(cadd(rho0, rho1), 0.5);
  const double src1 = dt * kap2 * F.sigma1, src2 = dt * kap2 * F.sigma2;
  double2 psi1, phi1;
  psi1.x = (c_old * psi0.x - c_x * phi0.x + src1 * rhoh.x) * inv_den;
  psi1.y = (c_old * psi0.y - c_x * phi0.y + src1 * rhoh.y) * inv_den;
  phi1 = cadd(phi0, cscale(cadd(psi0, psi1), a));
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    U1[l].x = (c_old * U0[l].x - c_x * A0[l].x + src2 * J[l].x) * inv_den;
    U1[l].y = (c_old * U0[l].y - c_x * A0[l].y + src2 * J[l].y) * inv_den;
    A1[l] = cadd(A0[l], cscale(cadd(U0[l], U1[l]), a));
  }
  out[F_PHI] = phi1;
  out[F_PSI] = psi1;
  out[F_RHO] = rho1;
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    out[F_A + l] = A1[l];
    out[F_U + l] = U1[l];
  }
  // inverse-transform inputs: grad_h phi^{n+1/2} and A^{n+1}, scaled by 1/ncell
  const double sc = 1.0 / (double)G.ncell;
  const double2 phih = cscale(cadd(phi0, phi1), 0.5);
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    inv[l] = cscale(ik(k[l], phih), sc);
    inv[3 + l] = cscale(A1[l], sc);
  }
  // Parseval: sum_g f_g h_g = (1/ncell) sum_k Re(conj(f^_k) h^_k)
  const double h1 = 0.5 / F.sigma1, h2 = 0.5 / F.sigma2;
  double je = 0.0;
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    const double2 Uh = cscale(cadd(U0[l], U1[l]), 0.5);
    const double2 Eh = csub(make_double2(k[l] * phih.y, -k[l] * phih.x), Uh);  // -i k phi - U
    je += J[l].x * Eh.x + J[l].y * Eh.y;
  }
  const double e1 = mode_energy(k, phi1, A1, U1, h1, h2);
  // W^{n+1} - W^n per mode as (f1 - f0).(f1 + f0) to keep the difference accurate
  double de = 0.0;
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    const double2 E1 = csub(make_double2(k[l] * phi1.y, -k[l] * phi1.x), U1[l]);
    const double2 E0 = csub(make_double2(k[l] * phi0.y, -k[l] * phi0.x), U0[l]);
    const double2 dE = csub(E1, E0), sE = cadd(E1, E0);
    de += h1 * (dE.x * sE.x + dE.y * sE.y);
  }
  double2 dA[3], sA[3];
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    dA[l] = csub(A1[l], A0[l]);
    sA[l] = cadd(A1[l], A0[l]);
  }
  const double2 dB[3] = {csub(ik(k[1], dA[2]), ik(k[2], dA[1])),
                         csub(ik(k[2], dA[0]), ik(k[0], dA[2])),
                         csub(ik(k[0], dA[1]), ik(k[1], dA[0]))};
  const double2 sB[3] = {csub(ik(k[1], sA[2]), ik(k[2], sA[1])),
                         csub(ik(k[2], sA[0]), ik(k[0], sA[2])),
                         csub(ik(k[0], sA[1]), ik(k[1], sA[0]))};
#pragma unroll
  for (int l = 0; l < 3; ++l) de += h2 * (dB[l].x * sB[l].x + dB[l].y * sB[l].y);
  const double f = G.dV / (double)G.ncell;
  sums[0] = je * f;
  sums[1] = e1 * f;
  sums[2] = de * f;
}

__global__ __launch_bounds__(kBlock) void k_half_U(Grid G, const double2* cur, const double2* next,
                                                  double2* inv) {
  const int64_t nc = G.ncell;
  const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (g >= nc) return;
  const double sc = 0.5 / (double)nc;
#pragma unroll
  for (int l = 0; l < 3; ++l)
    inv[l * nc + g] = cscale(cadd(cur[(F_U + l) * nc + g], next[(F_U + l) * nc + g]), sc);
}

// phi^0 from -Delta_h phi = sigma1 rho on modes with k~ != 0; rho and phi zero
// on every mode where k~ = 0 (this removes the mean and the uniform
// background); psi = A = U = 0.
__global__ __launch_bounds__(kBlock) void k_poisson_init(FieldParams F, double2* cur) {
  const Grid& G = F.G;
  const int64_t nc = G.ncell;
  const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (g >= nc) return;
  double k[3];
  mode_k(G, g, k);
  const double k2 = k[0] * k[0] + k[1] * k[1] + k[2] * k[2];
  double2 rho = cur[F_RHO * nc + g];
  double2 phi = make_double2(0.0, 0.0);
  if (k2 == 0.0)
    rho = make_double2(0.0, 0.0);
  else
    phi = cscale(rho, F.sigma1 / k2);
  cur[F_RHO * nc + g] = rho;
  cur[F_PHI * nc + g] = phi;
  cur[F_PSI * nc + g] = make_double2(0.0, 0.0);
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    cur[(F_A + l) * nc + g] = make_double2(0.0, 0.0);
    cur[(F_U + l) * nc + g] = make_double2(0.0, 0.0);
  }
}

// G_h = psi/kappa^2 + i k.A and R_h = i k.E - sigma1 rho (E = -i k phi - U),
// scaled by 1/ncell, and W of the level.
__global__ __launch_bounds__(kBlock) void k_constraints(FieldParams F, const double2* cur,
                                                       double2* inv, Scratch sc) {
  const Grid& G = F.G;
  const int64_t nc = G.ncell;
  const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  double w[1] = {0.0};
  if (g < nc) {
    double k[3];
    mode_k(G, g, k);
    const double2 phi = cur[F_PHI * nc + g], psi = cur[F_PSI * nc + g], rho = cur[F_RHO * nc + g];
    double2 A[3], U[3];
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      A[l] = cur[(F_A + l) * nc + g];
      U[l] = cur[(F_U + l) * nc + g];
    }
    const double kap2 = F.kappa * F.kappa;
    double2 gh = cscale(psi, 1.0 / kap2);
    double2 divE = make_double2(0.0, 0.0);
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      gh = cadd(gh, ik(k[l], A[l]));
      const double2 E = csub(make_double2(k[l] * phi.y, -k[l] * phi.x), U[l]);
      divE = cadd(divE, ik(k[l], E));
    }
    const double2 rh = csub(divE, cscale(rho, F.sigma1));
    const double s = 1.0 / (double)nc;
    inv[g] = cscale(gh, s);
    inv[nc + g] = cscale(rh, s);
    w[0] = mode_energy(k, phi, A, U, 0.5 / F.sigma1, 0.5 / F.sigma2) * G.dV / (double)nc;
  }
  block_partials<1>(w, sc.region(P_W));  // -> S_WCUR
}

__global__ __launch_bounds__(kBlock) void k_field_energy(FieldParams F, const double2* cur,
                                                        Scratch sc) {
  const Grid& G = F.G;
  const int64_t nc = G.ncell;
  const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  double w[1] = {0.0};
  if (g < nc) {
    double k[3];
    mode_k(G, g, k);
    double2 A[3], U[3];
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      A[l] = cur[(F_A + l) * nc + g];
      U[l] = cur[(F_U + l) * nc + g];
    }
    w[0] = mode_energy(k, cur[F_PHI * nc + g], A, U, 0.5 / F.sigma1, 0.5 / F.sigma2) * G.dV /
           (double)nc;
  }
  block_partials<1>(w, sc.region(P_W));  // -> S_WCUR
}

__global__ __launch_bounds__(kBlock) void k_norms(int64_t nc, const double* gf, const double* rf,
                                                 Scratch sc) {
  const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  double gv = 0.0, rv = 0.0;
  if (g < nc) {
    gv = gf[g];
    rv = rf[g];
  }
  const double gm = block_max(fabs(gv)), rm = block_max(fabs(rv));
  if (threadIdx.x == 0) {
    atomic_max_nonneg(sc.spread_copy(S_GMAX), gm);
    atomic_max_nonneg(sc.spread_copy(S_RMAX), rm);
  }
  double s[2] = {gv * gv, rv * rv};
  block_partials<2>(s, sc.region(P_NORM));  // -> S_GL2, S_RL2
}

struct FinishArgs {
  Scratch sc;
  FinishJob job[kMaxFinishJobs];
  int njobs;
  int* clear_int;  // optional: its value to S_FAR, then zero (a work-list count)
  HostRead read;
};

constexpr int kFinishThreads = 1024;  // one wavefront per row, 16 rows at a time
static_assert(kSpread == kWave, "the finishing kernel folds one copy per lane");

// One block; every requested row is reduced by one wavefront in a fixed
// order (lanes stride the row, then a fixed butterfly): a row of block
// partials is summed into its slot, a spread slot's copies are folded by max
// (slot = max) or sum (slot += sum) and then cleared for the next pass.
__global__ __launch_bounds__(kFinishThreads) void k_finish(FinishArgs F) {
  constexpr int NW = kFinishThreads / kWave;
  const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
  if (F.clear_int && threadIdx.x == kFinishThreads - 1) {  // of a wavefront without a row, mostly
    F.sc.red[S_FAR] = (double)*F.clear_int;
    *F.clear_int = 0;
  }
  int row = 0;
  for (int j = 0; j < F.njobs; ++j) {
    const FinishJob jb = F.job[j];
    for (int m = 0; m < jb.M; ++m, ++row) {
      if (row % NW != wid) continue;
      double* slot = F.sc.red + jb.slot + m;
      if (jb.op == F_SUM) {
        const double* r = F.sc.region(jb.site) + (size_t)(jb.row0 + m) * jb.nb;
        double acc = 0.0;
#pragma unroll 8
        for (int b = lane; b < jb.nb; b += kWave) acc += r[b];
        acc = wave_sum(acc);
        if (lane == 0) *slot = acc;
      } else {
        double* cp = F.sc.spread + ((size_t)(jb.slot + m) * kSpread + lane) * kSpreadStride;
        const double c = *cp;  // kSpread == kWave: one copy per lane
        *cp = 0.0;
        if (jb.op == F_SPREAD_MAX) {
          const double r = wave_max(c);
          if (lane == 0) *slot = r;
        } else {
          const double r = wave_sum(c);
          if (lane == 0) *slot += r;
        }
      }
    }
  }
  // Straight into the host's memory: a copy queued behind this kernel is a launch of
  // its own (4,096 particles: 3.4 us of the GPU's time in every pass).
  if (F.read.count > 0) {  // uniform
    __syncthreads();
    if ((int)threadIdx.x < F.read.count) F.read.dst[threadIdx.x] = F.sc.red[F.read.first + threadIdx.x];
  }
}

__global__ __launch_bounds__(kBlock) void k_reset_slots(Scratch sc, int first, int count) {
  const int i = blockIdx.x * kBlock + threadIdx.x;
  if (i >= count * (kSpread + 1)) return;
  const int j = i / (kSpread + 1), c = i % (kSpread + 1);
  if (c == kSpread)
    sc.red[first + j] = 0.0;
  else
    sc.spread[((size_t)(first + j) * kSpread + c) * kSpreadStride] = 0.0;
}

__global__ __launch_bounds__(kBlock) void k_spec_copy(int64_t n, const double2* src, double2* dst,
                                                     double scale) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) dst[i] = cscale(src[i], scale);
}

__global__ __launch_bounds__(kBlock) void k_accept_A(int64_t nc, double* gbuf) {
  const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (g >= nc) return;
#pragma unroll
  for (int l = 0; l < 3; ++l) gbuf[g * kGbufStride + 3 + l] = gbuf[g * kGbufStride + 6 + l];
}

__global__ __launch_bounds__(kBlock) void k_set_A0(int64_t nc, const double* A, double* gbuf) {
  const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (g >= nc) return;
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    gbuf[g * kGbufStride + 3 + l] = A[l * nc + g];
    gbuf[g * kGbufStride + 6 + l] = A[l * nc + g];
  }
}

__global__ __launch_bounds__(kBlock) void k_fill(int64_t n, double* p, double v) {
  const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (i < n) p[i] = v;
}

inline unsigned blocks_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

int ilog2(int n) {
  int l = 0;
  while ((1 << l) < n) ++l;
  return l;
}

// One pass along `axis` over nb batch fields.
template <int MODE, bool INV>
void fft_pass(hipStream_t s, const Grid& G, int nb, const double2* src, double2* data, int axis,
              const double2* tw, const RealIO* io, const double* prev, double* clear,
              const Scratch& sc, double scale = 1.0) {
  FftPass A{};
  A.src = src;
  A.scale = scale;
  A.data = data;
  A.tw = tw;
  A.ncell = G.ncell;
  A.N = G.n[axis];
  A.logN = ilog2(A.N);
  int64_t stride = 1;
  for (int a = axis + 1; a < 3; ++a) stride *= G.n[a];
  A.stride = stride;
  A.logS = ilog2((int)stride);
  A.npb = G.ncell / A.N;
  A.npencils = (int64_t)nb * A.npb;
  if (io) A.io = *io;
  A.prev = prev;
  A.clear = clear;
  A.sc = sc;
  // (16^3, 9 fields: 72 blocks of 512 points 5.6 us, 18 of 2048 7.4 us)
  A.logpts = nb * G.ncell >= (int64_t)512 * kFftPoints ? 11 : 9;
  const int P = (1 << A.logpts) / A.N;
  const unsigned nblk = (unsigned)((A.npencils + P - 1) / P);
  k_fft<MODE, INV><<<nblk, kBlock, 0, s>>>(A);
}

// ---- field solve ------------------------------------------------------------
// Forward transform of the current along z and y, then per block of x-pencils the
// forward transform along x, the continuity + CN update of every mode of those
// pencils and the inverse transform along x of the six gather fields, then the
// inverse along y and z into the gather buffer.  Where an x-plane fits LDS
// (ny nz <= 4096) the two directions of a plane run back to back in one kernel
// per field and plane (both indices bit-reversed at load): three kernels in all.
// Four x-pencils per block: at 32^3 that is 256 blocks (16 pencils per block: 64
// blocks, 23 us for the pencil kernel alone).  Three radix-2 stages per LDS round
// trip against one: the pencil kernel 8.9 -> 7.1 us at 16x4x4, 18.2 -> 11.3 us at
// 64x32x16, 13.4 -> 10.4 us at 32^3, 53.5 -> 42.4 us at 64^3.  At 128^3 the
// separate x passes and CN kernel read and wrote 1.5 GB, the pencil kernel 0.9.
constexpr int kPlaneMax = 4096;  // ny nz limit of the plane kernels (64 KB of LDS)

bool plane_fits(const Grid& G) { return G.n[1] * G.n[2] <= kPlaneMax; }

struct PlaneArgs {
  Grid G;
  const double2* tw_y;  // exp(-2 pi i t / ny), t < ny/2
  const double2* tw_z;
  int logy, logz;
  // forward: real input (io), optional prev / clear (laid out like the fields one
  // after the other), complex output
  const double* prev;
  double* clear;
  double2* cout;
  // inverse: complex input, real output through io
  const double2* cin;
  RealIO io;
  Scratch sc;
};

// INVERSE = false: block = (field, x-plane) of the forward transform;
// true: of the inverse transform (conjugate twiddles, real output).
template <bool INVERSE>
__global__ __launch_bounds__(kBlock) void k_fft_plane(PlaneArgs A) {
  __shared__ double2 buf[kPlaneMax + kPlaneMax / 8];
  __shared__ double2 tw_y[128], tw_z[128];
  const Grid& G = A.G;
  for (int t = threadIdx.x; t < G.n[1] / 2; t += kBlock) tw_y[t] = A.tw_y[t];
  for (int t = threadIdx.x; t < G.n[2] / 2; t += kBlock) tw_z[t] = A.tw_z[t];
  const int ny = G.n[1], nz = G.n[2], plane = ny * nz, nx = G.n[0];
  const int b = blockIdx.x / nx, ix = blockIdx.x % nx;
  const int64_t base = (int64_t)ix * plane, fo = (int64_t)b * G.ncell;
  double dmax = 0.0;
  for (int e = threadIdx.x; e < plane; e += kBlock) {
    const int iy = e >> A.logz, iz = e & (nz - 1);
    const int64_t g = base + e;
    double2 v;
    if constexpr (INVERSE) {
      v = A.cin[fo + g];
    } else {
      const double re = A.io.p[b][g * A.io.stride[b]];
      if (A.prev) dmax = fmax(dmax, fabs(re - A.prev[fo + g]));
      if (A.clear) A.clear[fo + g] = 0.0;  // after prev was read (same element)
      v = make_double2(re, 0.0);
    }
    buf[pad8((brev(iy, A.logy) << A.logz) | brev(iz, A.logz))] = v;
  }
  __syncthreads();
  // along z: rows of nz; along y: columns of ny, nz apart
  fft_pencils<INVERSE, false>(nz, A.logz, ny, tw_z, [&](int p, int e) -> double2& {
    return buf[pad8((p << A.logz) + e)];
  });
  fft_pencils<INVERSE, true>(ny, A.logy, nz, tw_y, [&](int p, int e) -> double2& {
    return buf[pad8((e << A.logz) + p)];
  });
  for (int e = threadIdx.x; e < plane; e += kBlock) {
    const int64_t g = base + e;
    if constexpr (INVERSE)
      A.io.p[b][g * A.io.stride[b]] = buf[pad8(e)].x;
    else
      A.cout[fo + g] = buf[pad8(e)];
  }
  if constexpr (!INVERSE) {
    if (A.prev) {
      const double r = block_max(dmax);
      if (threadIdx.x == 0) atomic_max_nonneg(A.sc.spread_copy(S_DJMAX), r);
    }
  }
}

struct PencilArgs {
  FieldParams F;
  const double2* tw_x;
  int logx, npl;       // pencils per block
  const double2* Jh;   // 3 fields after the z and y transforms
  const double2* cur;  // level n (9 fields)
  double2* next;       // level n+1 (9 fields)
  double2* inv;        // 6 gather fields after the inverse x transform
  Scratch sc;
};

// slots of a field: npl runs of nx + nx / 8 + 1 points, npl nx <= 2 kBlock, npl <= 4
constexpr int kPencilLds = 2 * kBlock + kBlock / 4 + 4;

__global__ __launch_bounds__(kBlock) void k_cn_pencils(PencilArgs A) {
  __shared__ double2 buf[6 * kPencilLds];  // three currents, then six gather fields
  __shared__ double2 tw[128];
  const Grid& G = A.F.G;
  for (int t = threadIdx.x; t < G.n[0] / 2; t += kBlock) tw[t] = A.tw_x[t];
  const int nx = G.n[0], npl = A.npl, lognpl = 31 - __clz(npl), ld = pad8(nx) + 1;
  const int64_t S = (int64_t)G.n[1] * G.n[2], nc = G.ncell;
  // Blocks go round robin to the 8 XCDs, each with its own L2.  A block reads and
  // writes 64 of the 128 bytes of a line, so neighbouring blocks take places 8
  // apart: both halves of a line then meet in one L2 (315 -> 270 us at 128^3, 41 -> 34
  // us at 64^3).
  const int per_xcd = gridDim.x / kXcds;
  const int block = gridDim.x % kXcds == 0
                        ? (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds
                        : blockIdx.x;
  const int64_t q0 = (int64_t)block * npl;  // first pencil (iy nz + iz) of the block
  const int span = npl * nx;
  auto slot = [&](int f, int pl, int e) -> double2& {
    return buf[f * kPencilLds + pl * ld + pad8(e)];
  };
  // pencil q of a transform: field q / npl, pencil q % npl of the block
  auto at = [&](int q, int e) -> double2& { return slot(q >> lognpl, q & (npl - 1), e); };
  // the three current spectra, pencil by pencil, bit-reversed along x
  for (int f = 0; f < 3; ++f)
    for (int u = threadIdx.x; u < span; u += kBlock) {
      const int kx = u >> lognpl, pl = u & (npl - 1);
      slot(f, pl, brev(kx, A.logx)) = A.Jh[f * nc + kx * S + q0 + pl];
    }
  __syncthreads();
  fft_pencils<false, false>(nx, A.logx, 3 * npl, tw, at);
  // continuity + CN of every mode of the block's pencils, at most two per thread;
  // every current is read before the first gather field takes its place
  double sums[3] = {0.0, 0.0, 0.0};
  double2 J[2][3];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int u = threadIdx.x + h * kBlock;
    if (u < span)
#pragma unroll
      for (int l = 0; l < 3; ++l) J[h][l] = slot(l, u & (npl - 1), u >> lognpl);
  }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int u = threadIdx.x + h * kBlock;
    if (u >= span) continue;
    const int kx = u >> lognpl, pl = u & (npl - 1);
    const int64_t g = kx * S + q0 + pl;
    double k[3];
    mode_k(G, g, k);
    double2 c[9], out[9], iv[6];
    double s3[3];
#pragma unroll
    for (int f = 0; f < 9; ++f) c[f] = A.cur[f * nc + g];
    cn_mode(A.F, k, J[h], c, out, iv, s3);
#pragma unroll
    for (int f = 0; f < 9; ++f) A.next[f * nc + g] = out[f];
#pragma unroll
    for (int f = 0; f < 6; ++f) slot(f, pl, brev(kx, A.logx)) = iv[f];
    sums[0] += s3[0];
    sums[1] += s3[1];
    sums[2] += s3[2];
  }
  __syncthreads();
  fft_pencils<true, false>(nx, A.logx, 6 * npl, tw, at);
  for (int f = 0; f < 6; ++f)
    for (int u = threadIdx.x; u < span; u += kBlock) {
      const int kx = u >> lognpl, pl = u & (npl - 1);
      A.inv[f * nc + kx * S + q0 + pl] = slot(f, pl, kx);
    }
  block_partials<3>(sums, A.sc.region(P_CN));  // -> S_JE, S_WNEXT, S_DW
}

// Inverse transform along z of the six gather fields of kGatherFftNodes
// neighbouring nodes, written into the gather buffer's records: whole runs of
// records leave together (one field at a time, 8 of every 80 bytes per pass, took
// 178 us at 128^3).  both_levels: A^{n+1} into the A^n slots too.
constexpr int kGatherFftNodes = 512;

struct GatherPass {
  const double2* data;
  const double2* tw;
  int64_t ncell;
  int N, logN;
  double* gbuf;
  int both_levels;
};

__global__ __launch_bounds__(kBlock) void k_fft_gather(GatherPass A) {
  constexpr int kRun = kGatherFftNodes + kGatherFftNodes / 8;
  __shared__ double2 buf[6 * kRun];
  __shared__ double2 tw[128];
  for (int t = threadIdx.x; t < A.N / 2; t += kBlock) tw[t] = A.tw[t];
  const int64_t g0 = (int64_t)blockIdx.x * kGatherFftNodes;
  for (int u = threadIdx.x; u < 6 * kGatherFftNodes; u += kBlock) {
    const int f = u / kGatherFftNodes, e = u % kGatherFftNodes;
    const int row = e & ~(A.N - 1);
    buf[f * kRun + pad8(row | brev(e & (A.N - 1), A.logN))] = A.data[f * A.ncell + g0 + e];
  }
  __syncthreads();
  const int logrows = 9 - A.logN;  // rows of N points per field: 512 / N
  fft_pencils<true, false>(A.N, A.logN, 6 << logrows, tw, [&](int p, int e) -> double2& {
    return buf[(p >> logrows) * kRun + pad8(((p & ((1 << logrows) - 1)) << A.logN) + e)];
  });
  const int per = A.both_levels ? 9 : 6;
  for (int u = threadIdx.x; u < per * kGatherFftNodes; u += kBlock) {
    const int e = u / per, k = u - e * per;
    const int slot = per == 9 || k < 3 ? k : k + 3;  // place in the record
    const int f = slot < 6 ? slot : slot - 3;        // grad phi 0-2, A 3-5
    A.gbuf[(g0 + e) * kGbufStride + slot] = buf[f * kRun + pad8(e)].x;
  }
}

// ---- adjoint of the field update ----------------------------------------
// Complex spectra carry adjoints in the convention dL = Re sum conj(lambda) dz;
// every coefficient of cn_mode is real except -dt i k of the continuity update,
// whose adjoint is +dt i k.  Given the adjoints l1 of the next level (9
// fields, may be null) and the gather-side adjoints lg = [grad phi^{n+1/2}
// (3), A^{n+1} (3), A^n (3)] as spectra (may be null; A^n only when lcur is
// set), writes the adjoint of J^ to lJh and adds the current level's share to
// lcur (may be null).  Transposes cn_mode's arithmetic step by step.
__global__ __launch_bounds__(kBlock) void k_cn_adjoint(FieldParams F, const double2* l1,
                                                      const double2* lg, double2* lcur,
                                                      double2* lJh) {
  const Grid& G = F.G;
  const int64_t nc = G.ncell;
  const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (g >= nc) return;
  double k[3];
  mode_k(G, g, k);
  const double dt = F.dt, a = 0.5 * dt, kap2 = F.kappa * F.kappa;
  const double w2 = kap2 * (k[0] * k[0] + k[1] * k[1] + k[2] * k[2]);
  const double inv_den = 1.0 / (1.0 + a * a * w2);
  const double c_old = 1.0 - a * a * w2, c_x = 2.0 * a * w2;
  const double src1 = dt * kap2 * F.sigma1, src2 = dt * kap2 * F.sigma2;
  const double2 z = make_double2(0.0, 0.0);
  auto at = [&](const double2* p, int f) { return p ? p[f * nc + g] : z; };
  // gather side: grad phi^{n+1/2} = i k (phi0 + phi1)/2 -> (-i k / 2) per component
  double2 lphi_g = z;
  if (lg)
#pragma unroll
    for (int l = 0; l < 3; ++l) lphi_g = cadd(lphi_g, ik(-0.5 * k[l], lg[l * nc + g]));
  const double2 lphi1 = cadd(at(l1, F_PHI), lphi_g);
  // phi1 = phi0 + a psi0 + a psi1; psi1 = (c_old psi0 - c_x phi0 + src1 rho_h) inv_den
  const double2 lpsi1 = cadd(at(l1, F_PSI), cscale(lphi1, a));
  const double2 lphi0 = csub(cadd(lphi1, lphi_g), cscale(lpsi1, c_x * inv_den));
  const double2 lpsi0 = cadd(cscale(lphi1, a), cscale(lpsi1, c_old * inv_den));
  const double2 lrhoh = cscale(lpsi1, src1 * inv_den);
  // rho_h = (rho0 + rho1)/2, rho1 = rho0 - dt i k.J
  const double2 lrho1 = cadd(at(l1, F_RHO), cscale(lrhoh, 0.5));
  const double2 lrho0 = cadd(lrho1, cscale(lrhoh, 0.5));
  double2 lJ[3], lA0[3], lU0[3];
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    const double2 lA1 = cadd(at(l1, F_A + l), lg ? lg[(3 + l) * nc + g] : z);
    const double2 lU1 = cadd(at(l1, F_U + l), cscale(lA1, a));
    lA0[l] = csub(lA1, cscale(lU1, c_x * inv_den));
    if (lg && lcur) lA0[l] = cadd(lA0[l], lg[(6 + l) * nc + g]);
    lU0[l] = cadd(cscale(lA1, a), cscale(lU1, c_old * inv_den));
    lJ[l] = cadd(cscale(lU1, src2 * inv_den), ik(dt * k[l], lrho1));
    lJh[l * nc + g] = lJ[l];
  }
  if (lcur) {
    lcur[F_PHI * nc + g] = cadd(lcur[F_PHI * nc + g], lphi0);
    lcur[F_PSI * nc + g] = cadd(lcur[F_PSI * nc + g], lpsi0);
    lcur[F_RHO * nc + g] = cadd(lcur[F_RHO * nc + g], lrho0);
#pragma unroll
    for (int l = 0; l < 3; ++l) {
      lcur[(F_A + l) * nc + g] = cadd(lcur[(F_A + l) * nc + g], lA0[l]);
      lcur[(F_U + l) * nc + g] = cadd(lcur[(F_U + l) * nc + g], lU0[l]);
    }
  }
}

// Adjoint of W (eq. field-energy) with respect to the spectra of the
// present level, before the inverse transforms: with E = -i k phi - U and
// B = i k x A evaluated as real fields and scaled by dV/sigma, lE and lB are
// their forward transforms / ncell; writes the 9-field adjoint spectrum (lF
// may be the same buffer as lEB).
__global__ __launch_bounds__(kBlock) void k_energy_adjoint(Grid G, const double2* lEB,
                                                          double2* lF) {
  const int64_t nc = G.ncell;
  const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (g >= nc) return;
  double k[3];
  mode_k(G, g, k);
  const double2 z = make_double2(0.0, 0.0);
  double2 lE[3], lB[3];  // all inputs first: lF may alias lEB (same mode, other rows)
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    lE[l] = lEB[l * nc + g];
    lB[l] = lEB[(3 + l) * nc + g];
  }
  double2 lphi = z, lA[3] = {z, z, z};
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    lphi = cadd(lphi, ik(k[l], lE[l]));          // E_l = -i k_l phi - U_l
    const int p = (l + 1) % 3, q = (l + 2) % 3;  // B_l = i (k_p A_q - k_q A_p)
    lA[q] = cadd(lA[q], ik(-k[p], lB[l]));
    lA[p] = cadd(lA[p], ik(k[q], lB[l]));
  }
#pragma unroll
  for (int l = 0; l < 3; ++l) lF[(F_U + l) * nc + g] = cscale(lE[l], -1.0);
  lF[F_PHI * nc + g] = lphi;
  lF[F_PSI * nc + g] = z;
  lF[F_RHO * nc + g] = z;
#pragma unroll
  for (int l = 0; l < 3; ++l) lF[(F_A + l) * nc + g] = lA[l];
}

// E = -i k phi - U and B = i k x A of the present level, / ncell (inverse
// transform inputs of the energy adjoint)
__global__ __launch_bounds__(kBlock) void k_fields_EB(Grid G, const double2* cur, double2* EB) {
  const int64_t nc = G.ncell;
  const int64_t g = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  if (g >= nc) return;
  double k[3];
  mode_k(G, g, k);
  const double sc = 1.0 / (double)nc;
  const double2 phi = cur[F_PHI * nc + g];
  double2 A[3];
#pragma unroll
  for (int l = 0; l < 3; ++l) {
    A[l] = cur[(F_A + l) * nc + g];
    EB[l * nc + g] = cscale(csub(ik(-k[l], phi), cur[(F_U + l) * nc + g]), sc);
  }
  EB[3 * nc + g] = cscale(csub(ik(k[1], A[2]), ik(k[2], A[1])), sc);
  EB[4 * nc + g] = cscale(csub(ik(k[2], A[0]), ik(k[0], A[2])), sc);
  EB[5 * nc + g] = cscale(csub(ik(k[0], A[1]), ik(k[1], A[0])), sc);
}

}  // namespace

namespace {

// the z and y passes of a forward transform, real input; max|in - prev| and clear
// as in fft3_forward
void forward_zy(hipStream_t s, const Grid& G, int nb, double2* data, const RealIO& in,
                const double* prev, const double2* const* tw, const Scratch& sc, double* clear) {
  if (plane_fits(G)) {
    PlaneArgs A{};
    A.G = G;
    A.tw_y = tw[1];
    A.tw_z = tw[2];
    A.logy = ilog2(G.n[1]);
    A.logz = ilog2(G.n[2]);
    A.io = in;
    A.prev = prev;
    A.clear = clear;
    A.cout = data;
    A.sc = sc;
    k_fft_plane<false><<<nb * G.n[0], kBlock, 0, s>>>(A);
    return;
  }
  fft_pass<1, false>(s, G, nb, nullptr, data, 2, tw[2], &in, prev, clear, sc);
  fft_pass<0, false>(s, G, nb, data, data, 1, tw[1], nullptr, nullptr, nullptr, sc);
}

// the y and z passes of an inverse transform, real output
void inverse_yz(hipStream_t s, const Grid& G, int nb, double2* data, const RealIO& out,
                const double2* const* tw) {
  if (plane_fits(G)) {
    PlaneArgs B{};
    B.G = G;
    B.tw_y = tw[1];
    B.tw_z = tw[2];
    B.logy = ilog2(G.n[1]);
    B.logz = ilog2(G.n[2]);
    B.cin = data;
    B.io = out;
    k_fft_plane<true><<<nb * G.n[0], kBlock, 0, s>>>(B);
    return;
  }
  fft_pass<0, true>(s, G, nb, data, data, 1, tw[1], nullptr, nullptr, nullptr, Scratch{});
  fft_pass<2, true>(s, G, nb, data, data, 2, tw[2], &out, nullptr, nullptr, Scratch{});
}

}  // namespace

void fft3_forward(hipStream_t s, const Grid& G, int nb, double2* data, const RealIO& in,
                  const double2* const* tw, Scratch sc, double scale) {
  forward_zy(s, G, nb, data, in, nullptr, tw, sc, nullptr);
  fft_pass<0, false>(s, G, nb, data, data, 0, tw[0], nullptr, nullptr, nullptr, sc, scale);
}

void fft3_inverse(hipStream_t s, const Grid& G, int nb, const double2* src, double2* data,
                  const RealIO& out, const double2* const* tw, double scale) {
  fft_pass<0, true>(s, G, nb, src, data, 0, tw[0], nullptr, nullptr, nullptr, Scratch{}, scale);
  inverse_yz(s, G, nb, data, out, tw);
}

namespace {
int pencils_per_block(const Grid& G) { return std::min(4, kBlock / (G.n[0] / 2)); }
}  // namespace

int cn_pencil_blocks(const Grid& G) {
  return (int)((int64_t)G.n[1] * G.n[2] / pencils_per_block(G));
}

void field_solve(hipStream_t s, const FieldParams& F, const RealIO& J, const double* prev,
                 double* clear, const double2* cur, double2* next, double2* Jh, double2* batch,
                 const GatherOut& out, const double2* const* tw, Scratch sc) {
  const Grid& G = F.G;
  forward_zy(s, G, 3, Jh, J, prev, tw, sc, clear);
  PencilArgs C{};
  C.F = F;
  C.tw_x = tw[0];
  C.logx = ilog2(G.n[0]);
  C.npl = pencils_per_block(G);
  C.Jh = Jh;
  C.cur = cur;
  C.next = next;
  C.inv = batch;
  C.sc = sc;
  k_cn_pencils<<<cn_pencil_blocks(G), kBlock, 0, s>>>(C);
  if (!out.gbuf) {
    inverse_yz(s, G, 6, batch, out.io, tw);
    return;
  }
  if (plane_fits(G)) {
    RealIO io{};
    for (int l = 0; l < 3; ++l) {
      io.p[l] = out.gbuf + l;          // grad_h phi^{n+1/2}
      io.p[3 + l] = out.gbuf + 6 + l;  // A^{n+1}
      io.stride[l] = io.stride[3 + l] = kGbufStride;
    }
    inverse_yz(s, G, 6, batch, io, tw);
    if (out.both_levels) launch_accept_A(s, G.ncell, out.gbuf);
    return;
  }
  fft_pass<0, true>(s, G, 6, batch, batch, 1, tw[1], nullptr, nullptr, nullptr, Scratch{});
  GatherPass P{};
  P.data = batch;
  P.tw = tw[2];
  P.ncell = G.ncell;
  P.N = G.n[2];
  P.logN = ilog2(P.N);
  P.gbuf = out.gbuf;
  P.both_levels = out.both_levels ? 1 : 0;
  k_fft_gather<<<(unsigned)(G.ncell / kGatherFftNodes), kBlock, 0, s>>>(P);
}

void launch_half_U(hipStream_t s, const Grid& G, const double2* cur, const double2* next,
                   double2* inv) {
  k_half_U<<<blocks_for(G.ncell), kBlock, 0, s>>>(G, cur, next, inv);
}

void launch_poisson_init(hipStream_t s, const FieldParams& F, double2* cur) {
  k_poisson_init<<<blocks_for(F.G.ncell), kBlock, 0, s>>>(F, cur);
}

void launch_constraint_spectra(hipStream_t s, const FieldParams& F, const double2* cur,
                               double2* inv, Scratch sc) {
  k_constraints<<<blocks_for(F.G.ncell), kBlock, 0, s>>>(F, cur, inv, sc);
}

void launch_field_energy(hipStream_t s, const FieldParams& F, const double2* cur, Scratch sc) {
  k_field_energy<<<blocks_for(F.G.ncell), kBlock, 0, s>>>(F, cur, sc);
}

void launch_constraint_norms(hipStream_t s, int64_t ncell, const double* g, const double* r,
                             Scratch sc) {
  k_norms<<<blocks_for(ncell), kBlock, 0, s>>>(ncell, g, r, sc);
}

void launch_spec_copy(hipStream_t s, int64_t count, const double2* src, double2* dst,
                      double scale) {
  if (count <= 0) return;
  k_spec_copy<<<blocks_for(count), kBlock, 0, s>>>(count, src, dst, scale);
}

void launch_accept_A(hipStream_t s, int64_t ncell, double* gbuf) {
  k_accept_A<<<blocks_for(ncell), kBlock, 0, s>>>(ncell, gbuf);
}

void launch_set_A0(hipStream_t s, int64_t ncell, const double* A, double* gbuf) {
  k_set_A0<<<blocks_for(ncell), kBlock, 0, s>>>(ncell, A, gbuf);
}

void launch_finish(hipStream_t s, Scratch sc, const FinishJob* jobs, int njobs, int* clear_int,
                   HostRead read) {
  FinishArgs F;
  F.sc = sc;
  F.njobs = njobs < kMaxFinishJobs ? njobs : kMaxFinishJobs;
  for (int j = 0; j < F.njobs; ++j) F.job[j] = jobs[j];
  F.clear_int = clear_int;
  F.read = read;
  if (F.njobs > 0 || clear_int || read.count > 0) k_finish<<<1, kFinishThreads, 0, s>>>(F);
}

int64_t mesh_blocks(int64_t ncell) { return (ncell + kBlock - 1) / kBlock; }

void launch_fill(hipStream_t s, int64_t count, double* p, double value) {
  if (count <= 0) return;
  k_fill<<<blocks_for(count), kBlock, 0, s>>>(count, p, value);
}

void launch_reset_slots(hipStream_t s, const Scratch& sc, int first, int count) {
  if (count <= 0) return;
  k_reset_slots<<<blocks_for((int64_t)count * (kSpread + 1)), kBlock, 0, s>>>(sc, first, count);
}

}  // namespace ecpic

namespace ecpic {

void launch_cn_adjoint(hipStream_t s, const FieldParams& F, const double2* l1, const double2* lg,
                       double2* lcur, double2* lJh) {
  k_cn_adjoint<<<blocks_for(F.G.ncell), kBlock, 0, s>>>(F, l1, lg, lcur, lJh);
}

void launch_energy_adjoint(hipStream_t s, const Grid& G, const double2* lEB, double2* lF) {
  k_energy_adjoint<<<blocks_for(G.ncell), kBlock, 0, s>>>(G, lEB, lF);
}

void launch_fields_EB(hipStream_t s, const Grid& G, const double2* cur, double2* EB) {
  k_fields_EB<<<blocks_for(G.ncell), kBlock, 0, s>>>(G, cur, EB);
}

}  // namespace ecpic
