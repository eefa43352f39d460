// pencil.h -- the stage of 3D Cartesian elements (N = 3 to 7) on meshes that fill the chip, with
// one line of nodes per thread: EC flux differencing in float64, LLF or HLL interface fluxes.
// The same semidiscretisation as k_stage, split differently.
//
// A block (or wave) takes whole elements and works through the directions z, y, x; a thread
// holds the n nodes of one line in registers.  Against k_stage's one node per thread
//   - every pair flux of a line is formed and both its contributions added in registers: no
//     LDS atomics, operator coefficients and series constants as scalar operands;
//   - a line has one minus and one plus face, so the interface fluxes run with all lanes
//     (k_stage: 2/n of them in each direction);
//   - elements of several waves meet at five block barriers instead of one per pair round.
// At N = 3 and 32^3 elements the right-hand side issues 1 834 vector instructions per four
// elements against 3 028 in k_stage.  What bounds it then is memory: at 64^3 elements a
// Runge-Kutta stage moves 2.9 GB (counted between the L2s and the rest, 2.4 GB algorithmic) in
// 584 us, 4.9 TB/s of the 6.0 TB/s that a copy reaches (k_stage: 702 us).
//
// The lines change threads through LDS (five planes of the block's nodes): first the states
// of the home lines (x), read in z and y layout; when the y lines are in registers the buffer
// takes the z sums, then the z and y sums, on their way to the home lines.  The conserved home
// line stays in registers for the x primitives and the update where they allow it; reading it
// again cost more (N = 3, 64^3: 480 against 413 us per right-hand side).  Two waves per SIMD: at
// three (168 VGPRs, N = 3) the compiler spills, and even 20 spilled registers cost more than the
// third wave gives; at one (N = 7, the conserved line held in AGPRs) near-equal states took 1 660 us
// per step at 24^3, as with two, but every wait is exposed where pairs leave the near-equal series
// (all of them: 3 590 against 2 130).
#pragma once
#include <hip/hip_runtime.h>

#include "kernels.h"

namespace dgx {

// Keeps the phases of a stage apart: nothing moves across, neither memory accesses nor the
// scheduler's register-hungry interleaving.
__device__ __forceinline__ void phase_fence() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// The split by degree: EB elements per block (per wave, where the lines of whole elements fill
// one), one line of a direction per thread.  Lanes without a line: none for N = 3 and 7, 2 %
// (N = 4), 16 % (N = 5; in blocks of four waves 2 %, but 24^3 then takes 749 us per step
// against 702: fewer, larger blocks leave more of the last round idle), 23 % (N = 6; four waves
// 4 %, 1 406 against 1 262 us at 24^3).
template <int N>
struct PencilMap {
  static constexpr int n = N + 1, NL = n * n, NN = n * n * n;
  static constexpr int THREADS = N == 4 || N == 5 ? 128 : 64;
  static constexpr bool WAVE = THREADS == 64;        // the waves of a block are independent
  static constexpr int EB = THREADS / NL;
  static constexpr bool FULL = EB * NL == THREADS;   // every thread has a line of its own
};

template <int N>
struct Pencil : PencilMap<N> {
  static_assert(N >= 3 && N <= 7, "degrees with enough pairs per line");
  static constexpr int WAVES = 2;   // per SIMD: 256 registers
  static constexpr bool HOLD = N <= 5;   // the conserved home line stays in registers, or is read
                                         // twice again
  static constexpr bool PRE = N <= 4;    // faces loaded a direction ahead
  // Pairs of a row whose means are formed together: as many as the registers hold.  More share the
  // code of the middle and far branches, which at N = 7 is larger than the instruction cache
  // (right-hand side at 24^3 with every pair in the middle branch: 370 us, 390 with three, 422 with
  // two; N = 6 12^3 near-equal pairs 29.5, 31.0 with four).
  static constexpr int ROW = N <= 4 ? N + 1 : N == 6 ? 3 : 4;
};

// LDS buffer: [variable][node of the block's (wave's) elements].
template <int N>
struct PencilLds {
  double q[5][PencilMap<N>::EB * PencilMap<N>::NN];   // the conserved state; then sums
};

// Position in a plane of the buffer of node (i, j, k) of element slot le.  n = 4: i ^ 4j ^ 37k ^
// 16 le_0 ^ 128 le_1; n = 8: i ^ 9j ^ 72k (permutations): the 32 lanes that an 8-byte LDS access
// serves at a time hold, for a fixed node of their lines, 32 different positions modulo 32 in
// all three directions, no bank conflicts.  Other n: the natural order (strides of 5, 6, 7
// conflict little).  A line's node m is at base ^ (m step) or base + m step.
template <int N>
struct PencilPos {
  static constexpr int n = N + 1;
  static constexpr bool XOR = n == 4 || n == 8;
  template <int D>
  static __device__ __forceinline__ int at(int base, int m) {
    if constexpr (n == 4) return base ^ (m * (D == 0 ? 1 : D == 1 ? 4 : 37));
    else if constexpr (n == 8) return base ^ (m * (D == 0 ? 1 : D == 1 ? 9 : 72));
    else return base + m * (D == 0 ? 1 : D == 1 ? n : n * n);
  }
  static __device__ __forceinline__ int elem(int le) {
    return n == 4 ? ((le & 1) * 16) ^ ((le >> 1) * 128) : le * n * n * n;
  }
};

// A thread's place in its tile.  Threads beyond the tile's lines repeat its last line, lanes
// beyond the mesh its last element (on: neither).
template <int N>
struct PencilPlace {
  int t, le, line, la, lb;   // la, lb: the line's place in the other two directions
  int e, ec[3];
  bool on;
  unsigned ho;               // byte offset of the home line (x line (j, k) = (la, lb)) in a plane
  int bx, by, bz;            // LDS positions of the thread's x, y and z lines

  __device__ __forceinline__ PencilPlace(const Geom& g, int tile) {
    using P = PencilMap<N>;
    using X = PencilPos<N>;
    t = P::WAVE ? (int)(threadIdx.x & 63u) : (int)threadIdx.x;
    const bool own = P::FULL || t < P::EB * P::NL;
    const int tl = own ? t : P::EB * P::NL - 1;
    le = tl / P::NL;
    line = tl - le * P::NL;
    lb = line / P::n;
    la = line - lb * P::n;
    const int er = tile * P::EB + le;
    on = own && er < g.E;
    e = er < g.E ? er : (int)g.E - 1;
    elem_xyz(g, e, ec);
    ho = ((unsigned)e * P::NN + line * P::n) * 8u;
    const int eb = X::elem(le);
    bx = X::template at<2>(X::template at<1>(eb, la), lb);
    by = X::template at<2>(X::template at<0>(eb, la), lb);
    bz = X::template at<1>(X::template at<0>(eb, la), lb);
  }
};

template <int N>
__device__ __forceinline__ void pencil_sync() {
  if constexpr (PencilMap<N>::WAVE) wave_sync();
  else __syncthreads();
}

// The operator table read through the scalar cache: nothing writes it while a stage runs.
typedef const double __attribute__((address_space(4)))* ConstTab;
__device__ __forceinline__ ConstTab const_tab(const double* p) {
  return (ConstTab)(unsigned long long)p;
}

// The value at a 32-bit byte offset into a plane (one variable of every node): a uniform base
// and a per-lane offset, so a lane holds one register per address.
__device__ __forceinline__ double ld(const double* base, unsigned off, int i = 0) {
  return reinterpret_cast<const double*>(reinterpret_cast<const char*>(base) + off)[i];
}
__device__ __forceinline__ void st(double* base, unsigned off, int i, double v) {
  reinterpret_cast<double*>(reinterpret_cast<char*>(base) + off)[i] = v;
}

template <typename NT>
__device__ __forceinline__ void st_out(double* base, unsigned off, int i, double v, NT nt) {
  store_one(reinterpret_cast<double*>(reinterpret_cast<char*>(base) + off) + i, v, nt);
}

// A line's nodes: density, momentum and velocity (component 0 along the line, then the other two in
// cyclic order), twice the pressure and the energy.  Interface and subcell fluxes take the momentum
// as it is stored, as every kernel does: formed again as rho v it would be off by v's rounding
// (2.3e-15, to one side), and the two elements of a face would see different jumps.
template <int n>
struct PLine {
  double rho[n], m[3][n], v[3][n], p2[n], E[n];
};

// Twice the pressure from rho, v (components x, y, z: the same value whatever the line's
// direction) and E.
__device__ __forceinline__ double pencil_p2(double gm1, double rho, double vx, double vy,
                                            double vz, double E) {
  return 2.0 * (gm1 * (E - 0.5 * rho * (vx * vx + vy * vy + vz * vz)));
}

// The EC flux of a pair (a, b) along the line from rl = {{rho}}_ln and
// ib = 2/((gamma - 1) {{beta}}_ln), scaled by powers of two that save multiplications: twice
// the mass flux, four times the others (exact; taken back when the sums are used).
__device__ __forceinline__ void pencil_pair(double rl, double ib, double a0, double a1, double a2,
                                            double ap, double b0, double b1, double b2, double bp,
                                            double (&f)[5]) {
  const double s0 = a0 + b0, s1 = a1 + b1, s2 = a2 + b2;
  f[0] = rl * s0;
  f[1] = fma(f[0], s0, ap + bp);
  f[2] = f[0] * s1;
  f[3] = f[0] * s2;
  const double h = fma(a0, b0, fma(a1, b1, fma(a2, b2, ib)));
  f[4] = fma(f[0], h, fma(ap, b0, bp * a0));
}

// A float64 constant held in scalar registers (an FMA takes it from there).
__device__ __forceinline__ double sconst(double c) {
  asm("" : "+s"(c));
  return c;
}

// A step of a Horner scheme with the coefficient in scalar registers, set just before it (left to
// the compiler it is moved to vector registers first; through sconst all of a polynomial's
// coefficients are live at once and spill).
struct HornerScalar {
  __device__ __forceinline__ double operator()(double p, double x, double c) const {
    double r;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(r) : "v"(p), "v"(x), "s"(c));
    return r;
  }
};

// a/b (b normal): the refined reciprocal and one residual correction.
__device__ __forceinline__ double div_nr(double a, double b) {
  const double r = rcp_nr(b), q = a * r;
  return fma(fma(-b, q, a), r, q);
}

// (b - a)/ln(b/a) of a pair with z^2 >= 0.1, and its inverse: ln(hi/lo) = k ln 2 + 2 artanh s with
// hi/lo = 2^k m, m in [1/sqrt 2, sqrt 2), s = (m - 1)/(m + 1) from the mantissas, whose difference is
// exact.  NaN where a or b is not positive.
__device__ __forceinline__ double pencil_ln_ratio(double hi, double lo) {
  double mh = __builtin_amdgcn_frexp_mant(hi);
  const double ml = __builtin_amdgcn_frexp_mant(lo);
  int ex = __builtin_amdgcn_frexp_exp(hi) - __builtin_amdgcn_frexp_exp(lo);
  const double sc = mh > 1.4142135623730951 * ml ? 0.5 : mh < 0.7071067811865476 * ml ? 2.0 : 1.0;
  ex += sc == 0.5 ? 1 : sc == 2.0 ? -1 : 0;
  mh *= sc;
  const double s = (mh - ml) * rcp_nr(mh + ml);
  const double l = fma(0.6931471805599453, (double)ex, s * inv_ln_mean_mid(s * s, HornerScalar()));
  return lo > 0.0 ? l : __builtin_nan("");
}

// The two logarithmic means of a pair for the lanes beyond the polynomials.
__device__ __forceinline__ void pencil_far(double a, double b, double c, double d, double& rl,
                                           double& ib) {
  const double zr = (b - a) * rcp_nr1(a + b), zb = (d - c) * rcp_nr1(c + d);
  const double hr = fmax(a, b), lr = fmin(a, b), hb = fmax(c, d), lb = fmin(c, d);
  if (!(zr * zr < 0.1)) rl = div_nr(hr - lr, pencil_ln_ratio(hr, lr));
  if (!(zb * zb < 0.1)) ib = div_nr(pencil_ln_ratio(hb, lb), hb - lb);
}

// The logarithmic means rl = {{rho}}_ln and ib = 2/((gamma - 1) {{beta}}_ln) of the pairs (i, m), m
// in [m0, m1), of a line; be: (gamma - 1) beta / 2 of the nodes.  The near-equal series serves all
// lanes; a wave with a lane beyond it forms the polynomials of the middle branch as well, all pairs
// of the row in flight together, and only one with a lane beyond z^2 = 0.1 takes the logarithm: a
// loop over the pairs, one at a time at the head of the chunk, whose registers rotate, keeps the
// code and the registers of that path small (park and unpark free registers meanwhile).
template <int n, int ROW, typename Park, typename Unpark>
__device__ __forceinline__ void pencil_means(double (&rho)[n], double (&be)[n], int i, int m0, int m1,
                                             Park park, Unpark unpark, double (&rl)[ROW],
                                             double (&ib)[ROW]) {
  const double c1 = sconst(-1.0 / 6.0), c2 = sconst(-2.0 / 45.0), c3 = -22.0 / 945.0;
  const double e1 = sconst(2.0 / 3.0), e2 = sconst(2.0 / 5.0), e3 = 2.0 / 7.0;
  double xr[ROW], xb[ROW];
  bool mid = false;
#pragma unroll
  for (int m = m0; m < m1; ++m) {
    const int j = m - m0;
    const double sr = rho[i] + rho[m], dr = rho[m] - rho[i];
    const double zr = dr * rcp_nr1(sr);
    const double sb = be[i] + be[m], db = be[m] - be[i];
    const double rb = rcp_nr1(sb);
    const double zb = db * rb;
    xr[j] = zr * zr;
    xb[j] = zb * zb;
    rl[j] = sr * fma(xr[j], fma(xr[j], fma(xr[j], c3, c2), c1), 0.5);
    ib[j] = rb * fma(xb[j], fma(xb[j], fma(xb[j], e3, e2), e1), 2.0);
    mid |= !(xr[j] < 1.0e-4) | !(xb[j] < 1.0e-4);
  }
  if (__builtin_expect(__any(mid) != 0, 0)) {
    bool far = false;
#pragma unroll
    for (int m = m0; m < m1; ++m) {
      const int j = m - m0;
      const double pr = (rho[i] + rho[m]) * ln_mean_mid(xr[j], HornerScalar());
      const double pb = rcp_nr1(be[i] + be[m]) * inv_ln_mean_mid(xb[j], HornerScalar());
      if (!(xr[j] < 1.0e-4)) rl[j] = pr;
      if (!(xb[j] < 1.0e-4)) ib[j] = pb;
      far |= !(xr[j] < 0.1) | !(xb[j] < 0.1);
    }
    if (__any(far)) {
      park();
#pragma unroll 1
      for (int c = m0; c < m1; ++c) {
        pencil_far(rho[i], rho[m0], be[i], be[m0], rl[0], ib[0]);
        const double t0 = rho[m0], t1 = be[m0], t2 = rl[0], t3 = ib[0];
#pragma unroll
        for (int m = m0; m < m1 - 1; ++m) {
          rho[m] = rho[m + 1];
          be[m] = be[m + 1];
          rl[m - m0] = rl[m - m0 + 1];
          ib[m - m0] = ib[m - m0 + 1];
        }
        rho[m1 - 1] = t0;
        be[m1 - 1] = t1;
        rl[m1 - 1 - m0] = t2;
        ib[m1 - 1 - m0] = t3;
      }
      unpark();
    }
  }
}

// Two-point fluxes of every pair of the line, contracted into acc (scaled as pencil_pair's).
// be: (gamma - 1) beta / 2 of the nodes; SC: every contribution times dg (the share of the flux
// differencing where it is blended).  Row I (pairs (I, m), m > I) in chunks of ROW pairs from M0 on,
// then the rows after it: a recursion, not loops, which at n = 8 pass the compiler's limit on
// unrolling and would leave the line in memory.
template <int n, int ROW, bool SC, int I = 0, int M0 = 1, typename Park, typename Unpark>
__device__ __forceinline__ void pencil_volume(PLine<n>& q, double (&be)[n], ConstTab S, double dg,
                                              Park park, Unpark unpark, double (&acc)[n][5]) {
  constexpr int M1 = M0 + ROW < n ? M0 + ROW : n;
  double rl[ROW], ib[ROW];
  pencil_means<n, ROW>(q.rho, be, I, M0, M1, park, unpark, rl, ib);
#pragma unroll
  for (int m = M0; m < M1; ++m) {
    double f[5];
    pencil_pair(rl[m - M0], ib[m - M0], q.v[0][I], q.v[1][I], q.v[2][I], q.p2[I], q.v[0][m],
                q.v[1][m], q.v[2][m], q.p2[m], f);
    double cim = S[I * TMAX + m], cmi = S[m * TMAX + I];
    if constexpr (SC) {
      cim *= dg;
      cmi *= dg;
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      acc[I][v] = fma(cim, f[v], acc[I][v]);
      acc[m][v] = fma(cmi, f[v], acc[m][v]);
    }
  }
  // the sums are formed here: sunk past the next rows they would keep every flux alive
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    asm("" : "+v"(acc[I][v]));
#pragma unroll
    for (int m = M0; m < M1; ++m) asm("" : "+v"(acc[m][v]));
  }
  if constexpr (M1 < n) pencil_volume<n, ROW, SC, I, M1>(q, be, S, dg, park, unpark, acc);
  else if constexpr (I + 2 < n) pencil_volume<n, ROW, SC, I + 1, I + 2>(q, be, S, dg, park, unpark, acc);
}

// Primitives of a face state: component k of the vectors along direction D + k.  Both sides of an
// interface form them with the same operations (the kinetic energy in the order x, y, z), so its
// two elements evaluate the same flux.
__device__ __forceinline__ void pencil_face_prim(double gamma, double rho, double v0, double v1,
                                                 double v2, double p2, Prim<double>& q) {
  q.rho = rho;
  q.v[0] = v0;
  q.v[1] = v1;
  q.v[2] = v2;
  q.p = 0.5 * p2;
  q.c = sqrt_pos1(gamma * q.p * rcp_nr1(rho));
}

// Lifted interface flux at one end of a line (scaled as pencil_pair's), node m; un: the state
// across the face.
template <int D, int n>
__device__ __forceinline__ void pencil_face(const Geom& g, int surf, bool plus, const PLine<n>& q,
                                            int m, const double (&un)[5], double lift,
                                            double (&out)[5]) {
  const double um[5] = {q.rho[m], q.m[0][m], q.m[1][m], q.m[2][m], q.E[m]};
  Prim<double> qm, qn;
  pencil_face_prim(g.gamma, um[0], q.v[0][m], q.v[1][m], q.v[2][m], q.p2[m], qm);
  const double inv = rcp_nr1(un[0]);
  double vn[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) vn[k] = un[1 + k] * inv;
  const double p2 = pencil_p2(g.gamma - 1.0, un[0], vn[(3 - D) % 3], vn[(4 - D) % 3], vn[(5 - D) % 3], un[4]);
  pencil_face_prim(g.gamma, un[0], vn[0], vn[1], vn[2], p2, qn);
  if (!((un[0] > 0.0) && (p2 > 0.0) && (p2 < 2.0e300) && (un[0] < 1.0e300))) *g.flag = 1;
  double F[5], half;
  if (surf == SURF_LLF)
    half = plus ? llf_flux<3, 0>(um, qm, un, qn, g.gamma, F) : llf_flux<3, 0>(un, qn, um, qm, g.gamma, F);
  else
    half = plus ? hll_flux<3, 0>(um, qm, un, qn, g.gamma, F) : hll_flux<3, 0>(un, qn, um, qm, g.gamma, F);
  const double c = half * lift;
  out[0] = 2.0 * c * F[0];
#pragma unroll
  for (int v = 1; v < 5; ++v) out[v] = 4.0 * c * F[v];
}

// The neighbours' face nodes of a line in direction D: at [0] across its minus end, at [1]
// across its plus end; momentum components in the order D, D + 1, D + 2.
template <int N, int D>
__device__ __forceinline__ void pencil_face_load(const double* __restrict__ u, const Geom& g, int e,
                                                 const int (&ec)[3], int la, int lb, size_t ENN,
                                                 double (&un)[2][5]) {
  constexpr int n = N + 1, NN = n * n * n, nd = Stride<D, n>::value;
  constexpr int na = D == 0 ? n : 1, nb = D == 2 ? n : n * n;
  const int nod = la * na + lb * nb;
  const unsigned o[2] = {((unsigned)elem_nb(g, e, ec, D, -1) * NN + nod + N * nd) * 8u,
                         ((unsigned)elem_nb(g, e, ec, D, 1) * NN + nod) * 8u};
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    un[s][0] = ld(u, o[s]);
#pragma unroll
    for (int k = 0; k < 3; ++k) un[s][1 + k] = ld(u + (1 + (D + k) % 3) * ENN, o[s]);
    un[s][4] = ld(u + 4 * ENN, o[s]);
  }
}

// A line's states and primitives from the LDS.
template <int N, int D>
__device__ __forceinline__ void pencil_read(const PencilLds<N>& s, int bl, double gm1,
                                            PLine<N + 1>& q, double (&be)[N + 1]) {
#pragma unroll
  for (int m = 0; m < N + 1; ++m) {
    const int x = PencilPos<N>::template at<D>(bl, m);
    q.rho[m] = s.q[0][x];
    const double inv = rcp_nr1(q.rho[m]);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      q.m[k][m] = s.q[1 + (D + k) % 3][x];
      q.v[k][m] = q.m[k][m] * inv;
    }
    q.E[m] = s.q[4][x];
    q.p2[m] = pencil_p2(gm1, q.rho[m], q.v[(3 - D) % 3][m], q.v[(4 - D) % 3][m],
                        q.v[(5 - D) % 3][m], q.E[m]);
  }
#pragma unroll
  for (int m = 0; m < N + 1; ++m) be[m] = (gm1 * q.rho[m]) * rcp_nr1(q.p2[m]);
}

// The running sums of a line from and to the LDS (component order of the line in registers).
template <int N, int D>
__device__ __forceinline__ void pencil_sums_get(const PencilLds<N>& s, int bl,
                                                double (&acc)[N + 1][5]) {
#pragma unroll
  for (int m = 0; m < N + 1; ++m) {
    const int x = PencilPos<N>::template at<D>(bl, m);
    acc[m][0] = s.q[0][x];
#pragma unroll
    for (int k = 0; k < 3; ++k) acc[m][1 + k] = s.q[1 + (D + k) % 3][x];
    acc[m][4] = s.q[4][x];
  }
}

template <int N, int D>
__device__ __forceinline__ void pencil_sums_put(PencilLds<N>& s, int bl,
                                                const double (&acc)[N + 1][5]) {
#pragma unroll
  for (int m = 0; m < N + 1; ++m) {
    const int x = PencilPos<N>::template at<D>(bl, m);
    s.q[0][x] = acc[m][0];
#pragma unroll
    for (int k = 0; k < 3; ++k) s.q[1 + (D + k) % 3][x] = acc[m][1 + k];
    s.q[4][x] = acc[m][4];
  }
}

template <int N, int D>
__device__ __forceinline__ void pencil_faces(const Geom& g, int surf, ConstTab tab,
                                             const PLine<N + 1>& q, const double (&un)[2][5],
                                             double (&f)[2][5]) {
  pencil_face<D, N + 1>(g, surf, false, q, 0, un[0], tab[TAB_LIFT + 2 * D], f[0]);
  pencil_face<D, N + 1>(g, surf, true, q, N, un[1], tab[TAB_LIFT + 2 * D + 1], f[1]);
}

// The line as conserved states with their primitives, node m.
template <int n>
__device__ __forceinline__ void pencil_node(const PLine<n>& q, int m, double gamma, double (&u)[5],
                                            Prim<double>& p) {
  p.rho = q.rho[m];
  p.p = 0.5 * q.p2[m];
  p.c = sqrt_pos1(gamma * p.p * rcp_nr1(p.rho));
  u[0] = p.rho;
  u[4] = q.E[m];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    p.v[k] = q.v[k][m];
    u[1 + k] = q.m[k][m];
  }
}

// Subcell finite-volume part of a line (fv_dir), weighted by al and scaled as pencil_pair's:
// w: -(2/h)/w_i of the direction.
template <int n>
__device__ __forceinline__ void pencil_fv(const PLine<n>& q, int fvf, double gamma, ConstTab w,
                                          double al, double (&acc)[n][5]) {
  double uL[5], uR[5];
  Prim<double> L, R;
  pencil_node<n>(q, 0, gamma, uL, L);
#pragma unroll
  for (int m = 0; m < n - 1; ++m) {
    pencil_node<n>(q, m + 1, gamma, uR, R);
    double F[5];
    const double h = fvf == SURF_LLF ? llf_flux<3, 0>(uL, L, uR, R, gamma, F)
                                     : hll_flux<3, 0>(uL, L, uR, R, gamma, F);
    const double ah = 4.0 * al * h, a = ah * w[m], b = ah * w[m + 1];
    acc[m][0] = fma(0.5 * a, F[0], acc[m][0]);
    acc[m + 1][0] = fma(-0.5 * b, F[0], acc[m + 1][0]);
#pragma unroll
    for (int v = 1; v < 5; ++v) {
      acc[m][v] = fma(a, F[v], acc[m][v]);
      acc[m + 1][v] = fma(-b, F[v], acc[m + 1][v]);
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      asm("" : "+v"(acc[m][v]), "+v"(acc[m + 1][v]));
      uL[v] = uR[v];
    }
    L = R;
  }
}

// Sum over each row of 16 lanes, in every lane of the row.
__device__ __forceinline__ double row_sum16(double x) {
  x += dpp_f64<0xB1, 0xF>(0.0, x);
  x += dpp_f64<0x4E, 0xF>(0.0, x);
  x += dpp_f64<0x141, 0xF>(0.0, x);
  return x + dpp_f64<0x140, 0xF>(0.0, x);
}

// The raw indicator of the home lines' new state (k_indicator's computation): the transform of
// rho p line by line in x, y and z through a plane of the buffer, the energies summed over the
// element's sixteen lanes.
template <int N>
__device__ __forceinline__ void pencil_indicator(double* buf, const StageArgs& a, const Geom& g,
                                                 const PencilPlace<N>& w, ConstTab V,
                                                 const double (&um)[5][N + 1]) {
  using X = PencilPos<N>;
  constexpr int n = N + 1;
  static_assert(PencilMap<N>::NL == 16, "an element is a row of lanes");
  double in[n], out[n];
  bool ok = true;
#pragma unroll
  for (int i = 0; i < n; ++i) {
    const double u5[5] = {um[0][i], um[1][i], um[2][i], um[3][i], um[4][i]};
    ok &= rho_p<3>(u5, g.gamma, in[i]);
  }
  if (w.on && !ok) *g.flag = 1;
  auto transform = [&]() {
#pragma unroll
    for (int i = 0; i < n; ++i) {
      out[i] = 0.0;
#pragma unroll
      for (int m = 0; m < n; ++m) out[i] = fma(V[i * TMAX + m], in[m], out[i]);
    }
  };
  transform();
  pencil_sync<N>();
#pragma unroll
  for (int i = 0; i < n; ++i) buf[X::template at<0>(w.bx, i)] = out[i];
  pencil_sync<N>();
#pragma unroll
  for (int i = 0; i < n; ++i) in[i] = buf[X::template at<1>(w.by, i)];
  transform();
#pragma unroll
  for (int i = 0; i < n; ++i) buf[X::template at<1>(w.by, i)] = out[i];
  pencil_sync<N>();
#pragma unroll
  for (int i = 0; i < n; ++i) in[i] = buf[X::template at<2>(w.bz, i)];
  transform();
  double t0 = 0.0, t1 = 0.0, t2 = 0.0;
#pragma unroll
  for (int i = 0; i < n; ++i) {
    const double c = out[i] * out[i];
    const int mx = max(i, max(w.la, w.lb));
    t0 += c;
    t1 += mx <= N - 1 ? c : 0.0;
    t2 += mx <= N - 2 ? c : 0.0;
  }
  t0 = row_sum16(t0);
  t1 = row_sum16(t1);
  t2 = row_sum16(t2);
  if (w.on && w.line == 0) {
    double en;
    a.alpha_next[w.e] = indicator_alpha(t0, t1, t2, a.ind_thr, a.ind_sharp, a.ind_amin,
                                        a.ind_amax, a.ind_xcut, en);
  }
}

// Max over each row of 16 lanes, in every lane of the row (see wave_max_lane63).
__device__ __forceinline__ double row_max16(double x) {
  x = fmax(x, dpp_f64<0xB1, 0xF>(x, x));
  x = fmax(x, dpp_f64<0x4E, 0xF>(x, x));
  x = fmax(x, dpp_f64<0x141, 0xF>(x, x));
  return fmax(x, dpp_f64<0x140, 0xF>(x, x));
}

// sum_d (2/h_d) max over the element's lines of l_d, in the thread that writes it: line 0, or 63
// of 64.  buf: LDS that is free by now (unused for N = 3 and 7).
template <int N>
__device__ __forceinline__ double pencil_elem_speed(double* buf, ConstTab tab,
                                                    const PencilPlace<N>& w,
                                                    const double (&l)[3]) {
  constexpr int NL = PencilMap<N>::NL;
  double lam = 0.0;
  if constexpr (NL == 16) {
#pragma unroll
    for (int d = 0; d < 3; ++d) lam += tab[TAB_JAC + d] * row_max16(l[d]);
  } else if constexpr (NL == 64) {
#pragma unroll
    for (int d = 0; d < 3; ++d) lam += tab[TAB_JAC + d] * wave_max_lane63(l[d]);
  } else {   // maxima of non-negative doubles as integers
    unsigned long long* const mx = reinterpret_cast<unsigned long long*>(buf) + w.le * 3;
    pencil_sync<N>();
    if (w.line < 3) mx[w.line] = 0;
    pencil_sync<N>();
#pragma unroll
    for (int d = 0; d < 3; ++d)
      if (w.on && l[d] > 0.0)
        __hip_atomic_fetch_max(&mx[d], (unsigned long long)__double_as_longlong(l[d]),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    pencil_sync<N>();
#pragma unroll
    for (int d = 0; d < 3; ++d)
      lam += tab[TAB_JAC + d] * __longlong_as_double((long long)mx[d]);
  }
  return lam;
}

// SC: the volume blended with the subcell finite volumes by the element's factor, and the
// indicator of the output state (N = 3).
template <int N, int EPI, bool SC>
__device__ __forceinline__ void pencil_tile(PencilLds<N>& s, const StageArgs& a, const Geom& g,
                                            int tile) {
  using P = Pencil<N>;
  using X = PencilPos<N>;
  constexpr int n = P::n, NL = P::NL, NN = P::NN;
  const PencilPlace<N> w(g, tile);
  const int la = w.la, lb = w.lb, line = w.line, le = w.le, e = w.e;
  const bool on = w.on;
  const size_t ENN = (size_t)g.E * NN;
  const ConstTab tab = const_tab(g.tab);
  const double gm1 = g.gamma - 1.0;
  const int (&ec)[3] = w.ec;
  unsigned ho = w.ho;
  const int bx = w.bx, by = w.by, bz = w.bz;

  double um[5][n], un[2][5], unb[2][5], f[2][5], acc[n][5], be[n];
  PLine<n> q;
  double al = 0.0, dg = 1.0;
  if constexpr (SC) {
    al = blending_factor<3>(a, g, e);
    dg = 1.0 - al;
  }
  // the subcell part of the line's direction d, where the element blends
  auto subcell = [&](int d) {
    if constexpr (SC) {
      if (al != 0.0) pencil_fv<n>(q, a.fvf, g.gamma, tab + TAB_FV + d * TMAX, al, acc);
      phase_fence();
    }
  };
  auto load_u = [&]() {
#pragma unroll
    for (int v = 0; v < 5; ++v)
#pragma unroll
      for (int i = 0; i < n; ++i) um[v][i] = ld(a.uin + v * ENN, ho, i);
  };
  // conserved -> primitive of the home line
  auto prims = [&]() {
    bool ok = true;
#pragma unroll
    for (int i = 0; i < n; ++i) {
      const double inv = rcp_nr1(um[0][i]);
      q.rho[i] = um[0][i];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        q.m[k][i] = um[1 + k][i];
        q.v[k][i] = um[1 + k][i] * inv;
      }
      q.E[i] = um[4][i];
      q.p2[i] = pencil_p2(gm1, q.rho[i], q.v[0][i], q.v[1][i], q.v[2][i], q.E[i]);
      ok &= (q.rho[i] > 0.0) && (q.p2[i] > 0.0) && (q.p2[i] < 2.0e300) && (q.rho[i] < 1.0e300);
    }
    return ok;
  };
  load_u();
  pencil_face_load<N, 2>(a.uin, g, e, ec, la, lb, ENN, un);
  if constexpr (P::PRE) pencil_face_load<N, 1>(a.uin, g, e, ec, la, lb, ENN, unb);
  if (!prims()) *g.flag = 1;
#pragma unroll
  for (int i = 0; i < n; ++i) {
    const int x = X::template at<0>(bx, i);
    s.q[0][x] = q.rho[i];
#pragma unroll
    for (int k = 0; k < 3; ++k) s.q[1 + k][x] = q.m[k][i];
    s.q[4][x] = q.E[i];
  }
  pencil_sync<N>();

  // ---- z
  pencil_read<N, 2>(s, bz, gm1, q, be);
  pencil_faces<N, 2>(g, a.surf, tab, q, un, f);
#pragma unroll
  for (int m = 0; m < n; ++m)
#pragma unroll
    for (int v = 0; v < 5; ++v) acc[m][v] = m == 0 ? f[0][v] : m == N ? f[1][v] : 0.0;
  phase_fence();
  if constexpr (P::PRE) pencil_face_load<N, 0>(a.uin, g, e, ec, la, lb, ENN, un);
  phase_fence();
  subcell(2);
  pencil_volume<n, P::ROW, SC>(q, be, tab + TAB_S + 2 * TMAX * TMAX, dg, []() {}, []() {}, acc);
  phase_fence();

  // ---- y: once its lines are in registers the buffer takes the sums
  if constexpr (!P::PRE) pencil_face_load<N, 1>(a.uin, g, e, ec, la, lb, ENN, unb);
  pencil_read<N, 1>(s, by, gm1, q, be);
  pencil_sync<N>();
  pencil_sums_put<N, 2>(s, bz, acc);
  pencil_sync<N>();
  pencil_faces<N, 1>(g, a.surf, tab, q, unb, f);
  phase_fence();
  pencil_sums_get<N, 1>(s, by, acc);
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    acc[0][v] += f[0][v];
    acc[N][v] += f[1][v];
  }
  // (a far row's sums wait at their places in the buffer)
  subcell(1);
  pencil_volume<n, P::ROW, SC>(q, be, tab + TAB_S + 1 * TMAX * TMAX, dg,
                               [&]() { pencil_sums_put<N, 1>(s, by, acc); },
                               [&]() { pencil_sums_get<N, 1>(s, by, acc); }, acc);
  phase_fence();
  if constexpr (!P::HOLD) load_u();
  if constexpr (!P::PRE) pencil_face_load<N, 0>(a.uin, g, e, ec, la, lb, ENN, un);
  pencil_sync<N>();
  pencil_sums_put<N, 1>(s, by, acc);
  pencil_sync<N>();

  // ---- x
  if constexpr (P::HOLD) {
#pragma unroll
    for (int v = 0; v < 5; ++v)   // the primitives are formed again: held from the start they
#pragma unroll                    // would cost 32 registers through the other directions
      for (int i = 0; i < n; ++i) asm("" : "+v"(um[v][i]));
  }
  (void)prims();
  pencil_faces<N, 0>(g, a.surf, tab, q, un, f);
  phase_fence();
#pragma unroll
  for (int m = 0; m < n; ++m) be[m] = (gm1 * q.rho[m]) * rcp_nr1(q.p2[m]);
  pencil_sums_get<N, 0>(s, bx, acc);
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    acc[0][v] += f[0][v];
    acc[N][v] += f[1][v];
  }
  subcell(0);
  pencil_volume<n, P::ROW, SC>(q, be, tab + TAB_S, dg,
                               [&]() { pencil_sums_put<N, 0>(s, bx, acc); },
                               [&]() { pencil_sums_get<N, 0>(s, bx, acc); }, acc);
  phase_fence();

  // epilogue: acc[i][v] holds twice (v = 0) and four times the home line's right-hand side
  if constexpr (EPI == EPI_RHS) {
    if (on) {
#pragma unroll
      for (int v = 0; v < 5; ++v)
#pragma unroll
        for (int i = 0; i < n; ++i) st(a.du + v * ENN, ho, i, (v == 0 ? 0.5 : 0.25) * acc[i][v]);
    }
  } else {
    const double dt = NL != 16 && a.dt_from ? stage_dt_from_partials(a) : *a.dt;
    const double dh = 0.5 * dt, dq = 0.25 * dt;
    // Variables whose loads are in flight at once.  N = 6 and 7: one; what the sums still hold leaves
    // no registers for more (N = 6 12^3 188 us per step, 193 with two, 204 with five; 24^3 1 250,
    // 1 260, 1 267).  N = 5: three (19 x 23 x 13 287, 292 with five).
    constexpr int DEPTH = N <= 4 ? 5 : N == 5 ? 3 : 1;
    double kv[DEPTH][n];
    auto load = [&](int v) {
      if constexpr (!P::HOLD) {
        asm("" : "+v"(ho));
#pragma unroll
        for (int i = 0; i < n; ++i) um[v][i] = ld(a.uin + v * ENN, ho, i);
      }
#pragma unroll
      for (int i = 0; i < n; ++i) kv[v % DEPTH][i] = a.A != 0.0 ? ld(a.k + v * ENN, ho, i) : 0.0;
    };
#pragma unroll
    for (int v = 0; v < DEPTH; ++v) load(v);
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      if constexpr (DEPTH < 5) phase_fence();
      if (on) {
        double (&k)[n] = kv[v % DEPTH];
#pragma unroll
        for (int i = 0; i < n; ++i) k[i] = fma(a.A, k[i], (v == 0 ? dh : dq) * acc[i][v]);
        if (a.kw) {
#pragma unroll
          for (int i = 0; i < n; ++i) st(a.k + v * ENN, ho, i, k[i]);
        }
#pragma unroll
        for (int i = 0; i < n; ++i) {
          um[v][i] = fma(a.B, k[i], um[v][i]);
          if constexpr (N > 5) st(a.uout + v * ENN, ho, i, um[v][i]);
        }
      }
      if (v + DEPTH < 5) load(v + DEPTH);
    }
    // (N = 6 and 7 gain nothing from streaming: 24^3 1 271 / 1 270 and 1 665 / 1 722)
    if constexpr (N <= 5) {
      if (on)
        store_out<5>(a.nt_out, [&](int v, auto nt) {
#pragma unroll
          for (int i = 0; i < n; ++i) st_out(a.uout + v * ENN, ho, i, um[v][i], nt);
        });
    }
    phase_fence();
    if (a.speed != nullptr || (NL != 16 && a.speed_slots != nullptr)) {
      double l[3] = {0.0, 0.0, 0.0};
      bool ok = true;
#pragma unroll
      for (int i = 0; i < n; ++i) {
        const double u5[5] = {um[0][i], um[1][i], um[2][i], um[3][i], um[4][i]};
        Prim<double> pn;
        ok &= cons_to_prim<3, false>(u5, g.gamma, pn);
#pragma unroll
        for (int d = 0; d < 3; ++d) l[d] = fmax(l[d], fabs(pn.v[d]) + pn.c);
      }
      if (on && !ok) *g.flag = 1;
      const double lam = pencil_elem_speed<N>(&s.q[0][0], tab, w, l);
      if (on && line == (NL == 64 ? 63 : 0)) {   // (N = 3 meshes are all beyond the slots)
        if (NL != 16 && a.speed_slots) slot_max(a.speed_slots, e, lam);
        else a.speed[e] = lam;
      }
    }
    if constexpr (SC) {
      if (a.alpha_next) pencil_indicator<N>(&s.q[0][0], a, g, w, tab + TAB_VINV, um);
    }
    if constexpr (NL != 16) {
      if (a.t_step && blockIdx.x == 0 && threadIdx.x == 0) stage_time_publish(a, dt);
      if (a.slots_clear && blockIdx.x == 0 && threadIdx.x < (unsigned)DT_SLOTS)
        a.slots_clear[threadIdx.x * DT_SLOT_STRIDE] = 0.0;
    }
  }
}

// Meshes of k_pencil, by degree: about where a line per thread is the faster on near-equal states
// and on those whose pairs leave the near-equal series, where it gains less (its code grows past the
// instruction cache).  Microseconds per adaptive step, k_stage / k_pencil, on TGV Mach 0.1 | TGV
// Mach 1 | random nodes within 10 %:
//   N = 3: 28 x 28 x 27 242 / 233 | 251 / 254 | 272 / 266,  29^3 274 / 258 | 285 / 275 | 310 / 288,
//          32^3 375 / 333 | 382 / 354 | 420 / 374,  64^3 3 526 / 3 008
//   N = 4: 23 x 23 x 24 322 / 317 | 338 / 354 | 368 / 375,  24^3 376 / 348 | 388 / 391 | 418 / 415,
//          26^3 452 / 412 | 457 / 448 | 509 / 482,  28^3 625 / 570 | 642 / 599 | 685 / 621
//          (in ensembles 24^3 gains more: two such runs 1.10, eight runs with two of them 1.09)
//   N = 5: 17 x 17 x 18 295 / 273 | 314 / 322 | 349 / 349,  18^3 320 / 290 | 342 / 338 | 380 / 367,
//          19 x 23 x 13 343 / 292,  20^3 428 / 368 | 458 / 447 | 510 / 484
//   N = 6: 10^3 173 / 148 | 186 / 203 | 204 / 231,  11^3 214 / 181 | 227 / 223 | 249 / 255,
//          12^3 260 / 197 | 280 / 238 | 308 / 270
//   N = 7: 21 x 20 x 20 1 102 / 1 036 | 1 165 / 1 168 | 1 323 / 1 447,  21^3 1 235 / 1 149 |
//          1 312 / 1 285 | 1 478 / 1 560,  23^3 1 594 / 1 467 | 1 684 / 1 636 | 1 924 / 1 918
// The upper limit keeps the meshes beyond 2^28 nodes in k_stage, so that a state of 2^31 values can
// be compared bit for bit with a small mesh's (one kernel for both; offsets here would reach 2^29).
constexpr int64_t PENCIL_MIN_E[5] = {20480, 13500, 5400, 1331, 9261};   // N = 3..7
inline bool use_pencil(int N, int64_t E, int surf) {
  if (N < 3 || N > 7 || (surf != SURF_LLF && surf != SURF_HLL)) return false;
  const int64_t nn = (int64_t)(N + 1) * (N + 1) * (N + 1);
  return E >= PENCIL_MIN_E[N - 3] && E * nn <= ((int64_t)1 << 28);
}
// The same with shock capturing (N = 3; single-wave blocks: two and four waves took 1 and 3 % more
// at 64^3).  Sedov blast, microseconds per adaptive step, k_stage / k_pencil: 26 x 26 x 25 272 / 264,
// 27^3 303 / 264, 32^3 454 / 377, 48^3 1 702 / 1 350, 64^3 3 986 / 3 190; right-hand side 27^3 58.7 /
// 56.1, 64^3 661 / 544.  A stage at 32^3 moves 349 MB in 74 us (4.7 TB/s), N = 3 without blending
// the same in 65: what bounds it beyond memory are the waves of blending elements, whose lines form
// three subcell fluxes more in each direction, and the indicator's three passes through the LDS
// (3 250 vector instructions per wave against 1 920).
constexpr int64_t PENCIL_SHOCK_MIN_E = 16384;
inline bool use_pencil_shock(int64_t E, int surf) {
  return E >= PENCIL_SHOCK_MIN_E && E <= ((int64_t)1 << 22) && (surf == SURF_LLF || surf == SURF_HLL);
}
// Four waves per block (x neighbours share an L1: N = 3, 64^3 3 040 us per step, against 3 240
// with one) from here on; below, single-wave blocks even out the last round (32^3: 342 / 358).
constexpr int64_t PENCIL_WIDE_E = 40960;

// WPB: independent waves per block where a wave holds its elements whole, else 1.
template <int N, int EPI, int WPB, bool SC = false>
__global__ __launch_bounds__((Pencil<N>::THREADS * WPB))
__attribute__((amdgpu_waves_per_eu((Pencil<N>::WAVES), (Pencil<N>::WAVES))))
void k_pencil(StageArgs a, Geom g) {
  using P = Pencil<N>;
  __shared__ PencilLds<N> s[WPB];
  const int w = P::WAVE ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0;
  const int tile = (int)xcd_tile(blockIdx.x, gridDim.x) * WPB + w;
  if ((int64_t)tile * P::EB >= g.E) return;   // (whole waves; the last block starts inside)
  pencil_tile<N, EPI, SC>(s[w], a, g, tile);
}

}  // namespace dgx
