// pencil.h -- the stage of 3D Cartesian elements of 4^3 nodes (N = 3) on meshes that fill the
// chip, with one line of nodes per thread: EC flux differencing in float64, LLF or HLL
// interface fluxes.  The same semidiscretisation as k_stage, split differently.
//
// A wave takes four elements (256 nodes, 64 lines per direction) and works through the
// directions z, y, x; a thread holds one line's four nodes in registers.  Against k_stage's
// one node per thread
//   - every pair flux of a line is formed and both its contributions added in registers: no
//     LDS atomics, operator coefficients and series constants as scalar operands;
//   - a line has one minus and one plus face, so the interface fluxes run with all 64 lanes
//     (k_stage: 32 of 64 in each direction).
// At 32^3 elements the right-hand side issues 1 738 vector instructions per four elements
// against 3 028 in k_stage.  What bounds it then is memory: at 64^3 elements a Runge-Kutta
// stage moves 3.1 GB (counted between the L2s and the rest, 2.4 GB algorithmic) in 600 us,
// 5.2 TB/s of the 6.0 TB/s that a copy reaches.
//
// The lines change lanes through LDS, 10 KB per wave: first the primitives of the home lines
// (x), read in z and y layout; when the y lines are in registers the buffer takes the z sums,
// then the z and y sums, on their way to the home lines.  The conserved home line stays in
// registers (40 of 233 VGPRs) for the x primitives and the update; reading it again instead
// cost more (64^3: 480 against 413 us per right-hand side).  Two waves per SIMD: at three
// (168 VGPRs) the compiler spills, and even 20 spilled registers cost more than the third
// wave gives.  Face states are loaded a direction ahead of their use.
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

constexpr int PENCIL_EW = 4;   // elements of 4^3 nodes per wave

// LDS buffer of a wave: [variable][node of the wave's elements].
struct PencilLds {
  double q[5][64 * PENCIL_EW];   // (rho, v, E); then sums
};

// Position in a plane of the buffer of node (i, j, k) of element le: i ^ 4j ^ 37k ^ 16 le_0 ^
// 128 le_1 (a permutation of 0..255).  The 32 lanes that an 8-byte LDS access serves at a
// time hold, for a fixed node of their lines, 32 different positions modulo 32 in all three
// directions: no bank conflicts.  A line's node m is at base ^ (m step).
template <int D>
__device__ __forceinline__ int pencil_at(int base, int m) {
  return base ^ (m * (D == 0 ? 1 : D == 1 ? 4 : 37));
}
__device__ __forceinline__ int pencil_elem(int le) { return ((le & 1) * 16) ^ ((le >> 1) * 128); }

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

// A line's nodes: density, velocity (v[0] along the line, then the other two in cyclic order),
// twice the pressure and the energy.
struct PLine {
  double rho[4], v[3][4], p2[4], E[4];
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

// artanh(z)/z on [0, 0.1] in x = z^2 (inv_ln_mean_mid's polynomial), coefficients in scalar
// registers.
__device__ __forceinline__ double artanh_q(double x) {
  constexpr double kQ[11] = {1.0, 0.3333333333333325, 0.20000000000033863, 0.14285714280450776,
                             0.11111111529834054, 0.09090889710268459, 0.07692864848122398,
                             0.06656438300891282, 0.060018248406360414, 0.04412879698538037,
                             0.0802184520988054};
  double p = kQ[10];
#pragma unroll
  for (int k = 9; k > 0; --k) p = fma(p, x, sconst(kQ[k]));
  return fma(p, x, 1.0);
}

// artanh(z)/z of the logarithmic means beyond the series: the polynomial below z^2 = 0.1, else
// ln(r)/(2 z) with r = hi/lo = 2^k m, m in [1/sqrt 2, sqrt 2), ln r = k ln 2 + 2 s Q(s^2),
// s = (m - 1)/(m + 1) (s^2 < 0.03).  NaN where r is not positive.
__device__ __forceinline__ double artanh_far(double a, double b, double x) {
  double y = x, k = 0.0, f = 1.0;
  if (!(x < 0.1)) {
    const double hi = fmax(a, b), lo = fmin(a, b);
    const double r = hi * rcp_nr(lo);
    double m = __builtin_amdgcn_frexp_mant(r);
    int ex = __builtin_amdgcn_frexp_exp(r);
    if (m < 0.7071067811865476) {
      m *= 2.0;
      ex -= 1;
    }
    const double sg = (m - 1.0) * rcp_nr(m + 1.0);
    const double iz = (hi + lo) * rcp_nr(hi - lo);   // 1/z
    f = sg * iz;
    k = r > 0.0 ? (0.5 * 0.6931471805599453) * (double)ex * iz : __builtin_nan("");
    y = sg * sg;
  }
  return fma(f, artanh_q(y), k);
}

// The two logarithmic means of a pair for the lanes beyond the near-equal series.
__device__ __forceinline__ void pencil_far(double a, double b, double c, double d, double& rl,
                                           double& ib) {
  const double sr = a + b, zr = (b - a) * rcp_nr1(sr), xr = zr * zr;
  const double qr = artanh_far(a, b, xr);
  if (!(xr < 1.0e-4)) rl = 0.5 * sr * rcp_nr(qr);
  const double sb = c + d, zb = (d - c) * rcp_nr1(sb), xb = zb * zb;
  const double qb = artanh_far(c, d, xb);
  if (!(xb < 1.0e-4)) ib = 2.0 * rcp_nr(sb) * qb;
}

// Two-point fluxes of every pair of the line, contracted into acc (scaled as pencil_pair's).
// be: (gamma - 1) beta / 2 of the nodes.  The near-equal series serves all lanes; where a lane
// of the wave is beyond it, the row's means are formed again one pair at a time, in a loop
// that keeps the code and the registers of that rare path small.
template <typename Park, typename Unpark>
__device__ __forceinline__ void pencil_volume(PLine& q, double (&be)[4], ConstTab S, Park park,
                                              Unpark unpark, double (&acc)[4][5]) {
  constexpr int n = 4;
  const double c1 = sconst(-1.0 / 6.0), c2 = sconst(-2.0 / 45.0), c3 = -22.0 / 945.0;
  const double e1 = sconst(2.0 / 3.0), e2 = sconst(2.0 / 5.0), e3 = 2.0 / 7.0;
#pragma unroll
  for (int i = 0; i < n - 1; ++i) {
    double rl[n], ib[n];   // [m]: the row's means
    bool far = false;
#pragma unroll
    for (int m = i + 1; m < n; ++m) {
      const double sr = q.rho[i] + q.rho[m], dr = q.rho[m] - q.rho[i];
      const double zr = dr * rcp_nr1(sr), xr = zr * zr;
      const double sb = be[i] + be[m], db = be[m] - be[i];
      const double rb = rcp_nr1(sb);
      const double zb = db * rb, xb = zb * zb;
      rl[m] = sr * fma(xr, fma(xr, fma(xr, c3, c2), c1), 0.5);
      ib[m] = rb * fma(xb, fma(xb, fma(xb, e3, e2), e1), 2.0);
      far |= !(xr < 1.0e-4) | !(xb < 1.0e-4);
    }
    if (__builtin_expect(__any(far) != 0, 0)) {
      // one pair at a time at the head of the row, whose registers rotate; park and unpark
      // free registers meanwhile
      park();
#pragma unroll 1
      for (int c = i + 1; c < n; ++c) {
        pencil_far(q.rho[i], q.rho[i + 1], be[i], be[i + 1], rl[i + 1], ib[i + 1]);
        const double t0 = q.rho[i + 1], t1 = be[i + 1], t2 = rl[i + 1], t3 = ib[i + 1];
#pragma unroll
        for (int m = i + 1; m < n - 1; ++m) {
          q.rho[m] = q.rho[m + 1];
          be[m] = be[m + 1];
          rl[m] = rl[m + 1];
          ib[m] = ib[m + 1];
        }
        q.rho[n - 1] = t0;
        be[n - 1] = t1;
        rl[n - 1] = t2;
        ib[n - 1] = t3;
      }
      unpark();
    }
#pragma unroll
    for (int m = i + 1; m < n; ++m) {
      double f[5];
      pencil_pair(rl[m], ib[m], q.v[0][i], q.v[1][i], q.v[2][i], q.p2[i], q.v[0][m], q.v[1][m],
                  q.v[2][m], q.p2[m], f);
      const double cim = S[i * TMAX + m], cmi = S[m * TMAX + i];
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        acc[i][v] = fma(cim, f[v], acc[i][v]);
        acc[m][v] = fma(cmi, f[v], acc[m][v]);
      }
    }
  }
}

// Lifted interface flux at one end of a line (scaled as pencil_pair's); un: the state across
// the face.
__device__ __forceinline__ void pencil_face(const Geom& g, int surf, bool plus, double rho,
                                            double v0, double v1, double v2, double p2, double E,
                                            const double (&un)[5], double lift, double (&out)[5]) {
  Prim<double> qn, qm;
  if (!cons_to_prim<3, false>(un, g.gamma, qn)) *g.flag = 1;
  qm.rho = rho;
  qm.v[0] = v0;
  qm.v[1] = v1;
  qm.v[2] = v2;
  qm.p = 0.5 * p2;
  double F[5], half;
  qm.c = sqrt_pos1(g.gamma * qm.p * rcp_nr1(rho));
  double um[5];
  um[0] = rho;
  um[1] = rho * v0;
  um[2] = rho * v1;
  um[3] = rho * v2;
  um[4] = E;   // as loaded: formed from p it would carry a rounding of E into the jump
  if (surf == SURF_LLF) {
    double fo[5], fn[5];
    phys_flux<3, 0>(um, qm, fo);
    phys_flux<3, 0>(un, qn, fn);
    const double lam = fmax(fabs(qm.v[0]) + qm.c, fabs(qn.v[0]) + qn.c);
    const double sl = plus ? lam : -lam;
#pragma unroll
    for (int v = 0; v < 5; ++v) F[v] = (fo[v] + fn[v]) - sl * (un[v] - um[v]);
    half = 0.5;
  } else if (plus) {
    half = hll_flux<3, 0>(um, qm, un, qn, g.gamma, F);
  } else {
    half = hll_flux<3, 0>(un, qn, um, qm, g.gamma, F);
  }
  const double c = half * lift;
  out[0] = 2.0 * c * F[0];
#pragma unroll
  for (int v = 1; v < 5; ++v) out[v] = 4.0 * c * F[v];
}

// The neighbours' face nodes of a line in direction D: at [0] across its minus end, at [1]
// across its plus end; momentum components in the order D, D + 1, D + 2.
template <int D>
__device__ __forceinline__ void pencil_face_load(const double* __restrict__ u, const Geom& g, int e,
                                                 const int (&ec)[3], int la, int lb, size_t ENN,
                                                 double (&un)[2][5]) {
  constexpr int n = 4, NN = 64, nd = Stride<D, n>::value;
  constexpr int na = D == 0 ? n : 1, nb = D == 2 ? n : n * n;
  const int nod = la * na + lb * nb;
  const unsigned o[2] = {((unsigned)elem_nb(g, e, ec, D, -1) * NN + nod + 3 * nd) * 8u,
                         ((unsigned)elem_nb(g, e, ec, D, 1) * NN + nod) * 8u};
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    un[s][0] = ld(u, o[s]);
#pragma unroll
    for (int k = 0; k < 3; ++k) un[s][1 + k] = ld(u + (1 + (D + k) % 3) * ENN, o[s]);
    un[s][4] = ld(u + 4 * ENN, o[s]);
  }
}

// A line's primitives from the LDS.
template <int D>
__device__ __forceinline__ void pencil_read(const PencilLds& s, int bl, double gm1, PLine& q,
                                            double (&be)[4]) {
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const int x = pencil_at<D>(bl, m);
    q.rho[m] = s.q[0][x];
#pragma unroll
    for (int k = 0; k < 3; ++k) q.v[k][m] = s.q[1 + (D + k) % 3][x];
    q.E[m] = s.q[4][x];
    q.p2[m] = pencil_p2(gm1, q.rho[m], q.v[(3 - D) % 3][m], q.v[(4 - D) % 3][m],
                        q.v[(5 - D) % 3][m], q.E[m]);
  }
#pragma unroll
  for (int m = 0; m < 4; ++m) be[m] = (gm1 * q.rho[m]) * rcp_nr1(q.p2[m]);
}

// The running sums of a line from and to the LDS (component order of the line in registers).
template <int D>
__device__ __forceinline__ void pencil_sums_get(const PencilLds& s, int bl, double (&acc)[4][5]) {
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const int x = pencil_at<D>(bl, m);
    acc[m][0] = s.q[0][x];
#pragma unroll
    for (int k = 0; k < 3; ++k) acc[m][1 + k] = s.q[1 + (D + k) % 3][x];
    acc[m][4] = s.q[4][x];
  }
}

template <int D>
__device__ __forceinline__ void pencil_sums_put(PencilLds& s, int bl, const double (&acc)[4][5]) {
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    const int x = pencil_at<D>(bl, m);
    s.q[0][x] = acc[m][0];
#pragma unroll
    for (int k = 0; k < 3; ++k) s.q[1 + (D + k) % 3][x] = acc[m][1 + k];
    s.q[4][x] = acc[m][4];
  }
}

template <int D>
__device__ __forceinline__ void pencil_faces(const Geom& g, int surf, ConstTab tab,
                                             const PLine& q, const double (&un)[2][5],
                                             double (&f)[2][5]) {
  pencil_face(g, surf, false, q.rho[0], q.v[0][0], q.v[1][0], q.v[2][0], q.p2[0], q.E[0], un[0],
              tab[TAB_LIFT + 2 * D], f[0]);
  pencil_face(g, surf, true, q.rho[3], q.v[0][3], q.v[1][3], q.v[2][3], q.p2[3], q.E[3], un[1],
              tab[TAB_LIFT + 2 * D + 1], f[1]);
}

// Max over each row of 16 lanes, in every lane of the row (see wave_max_lane63).
__device__ __forceinline__ double row_max16(double x) {
  x = fmax(x, dpp_f64<0xB1, 0xF>(x, x));
  x = fmax(x, dpp_f64<0x4E, 0xF>(x, x));
  x = fmax(x, dpp_f64<0x141, 0xF>(x, x));
  return fmax(x, dpp_f64<0x140, 0xF>(x, x));
}

template <int EPI>
__device__ __forceinline__ void pencil_tile(PencilLds& s, const StageArgs& a, const Geom& g,
                                            int tile) {
  constexpr int n = 4, NN = 64;
  const int lane = (int)(threadIdx.x & 63u);
  const int le = lane >> 4, line = lane & 15;
  const int la = line & 3, lb = line >> 2;   // the line's place in the other two directions
  const int er = tile * PENCIL_EW + le;
  const bool on = er < g.E;
  const int e = on ? er : (int)g.E - 1;      // lanes beyond the mesh repeat its last element
  const size_t ENN = (size_t)g.E * NN;
  const ConstTab tab = const_tab(g.tab);
  const double gm1 = g.gamma - 1.0;
  int ec[3];
  elem_xyz(g, e, ec);
  const unsigned ho = ((unsigned)e * NN + line * n) * 8u;   // home: the x line (j, k) = (la, lb)
  const int eb = pencil_elem(le);
  const int bx = pencil_at<2>(pencil_at<1>(eb, la), lb);
  const int by = pencil_at<2>(pencil_at<0>(eb, la), lb);
  const int bz = pencil_at<1>(pencil_at<0>(eb, la), lb);

  double um[5][n], un[2][5], acc[n][5];
  // conserved -> primitive of the home line
  auto prims = [&](PLine& q) {
    bool ok = true;
#pragma unroll
    for (int i = 0; i < n; ++i) {
      const double inv = rcp_nr1(um[0][i]);
      q.rho[i] = um[0][i];
#pragma unroll
      for (int k = 0; k < 3; ++k) q.v[k][i] = um[1 + k][i] * inv;
      q.E[i] = um[4][i];
      q.p2[i] = pencil_p2(gm1, q.rho[i], q.v[0][i], q.v[1][i], q.v[2][i], q.E[i]);
      ok &= (q.rho[i] > 0.0) && (q.p2[i] > 0.0) && (q.p2[i] < 2.0e300) && (q.rho[i] < 1.0e300);
    }
    return ok;
  };
#pragma unroll
  for (int v = 0; v < 5; ++v)
#pragma unroll
    for (int i = 0; i < n; ++i) um[v][i] = ld(a.uin + v * ENN, ho, i);
  // the line's sums into the lane's part of the LDS buffer and back, where the buffer is free
  double* const pk = &s.q[0][0] + (threadIdx.x & 63u);
  auto park = [&]() {
#pragma unroll
    for (int m = 0; m < n; ++m)
#pragma unroll
      for (int v = 0; v < 5; ++v) pk[(m * 5 + v) * 64] = acc[m][v];
  };
  auto unpark = [&]() {
#pragma unroll
    for (int m = 0; m < n; ++m)
#pragma unroll
      for (int v = 0; v < 5; ++v) acc[m][v] = pk[(m * 5 + v) * 64];
  };
  double f[2][5], unb[2][5];
  PLine q;
  double be[n];
  pencil_face_load<2>(a.uin, g, e, ec, la, lb, ENN, un);
  pencil_face_load<1>(a.uin, g, e, ec, la, lb, ENN, unb);
  if (!prims(q)) *g.flag = 1;
#pragma unroll
  for (int i = 0; i < n; ++i) {
    const int x = pencil_at<0>(bx, i);
    s.q[0][x] = q.rho[i];
#pragma unroll
    for (int k = 0; k < 3; ++k) s.q[1 + k][x] = q.v[k][i];
    s.q[4][x] = q.E[i];
  }
  wave_sync();
  pencil_read<2>(s, bz, gm1, q, be);
  pencil_faces<2>(g, a.surf, tab, q, un, f);
#pragma unroll
  for (int m = 0; m < n; ++m)
#pragma unroll
    for (int v = 0; v < 5; ++v) acc[m][v] = m == 0 ? f[0][v] : m == 3 ? f[1][v] : 0.0;
  phase_fence();
  pencil_face_load<0>(a.uin, g, e, ec, la, lb, ENN, un);
  phase_fence();
  // the buffer still holds the primitives here: v and p are read again instead
  auto reread = [&]() {
#pragma unroll
    for (int m = 0; m < n; ++m) {
      const int x = pencil_at<2>(bz, m);
#pragma unroll
      for (int k = 0; k < 3; ++k) q.v[k][m] = s.q[1 + (2 + k) % 3][x];
      q.p2[m] = pencil_p2(gm1, s.q[0][x], s.q[1][x], s.q[2][x], s.q[3][x], s.q[4][x]);
    }
  };
  pencil_volume(q, be, tab + TAB_S + 2 * TMAX * TMAX, []() {}, reread, acc);
  phase_fence();
  pencil_read<1>(s, by, gm1, q, be);
  wave_sync();
  pencil_sums_put<2>(s, bz, acc);
  wave_sync();
  pencil_faces<1>(g, a.surf, tab, q, unb, f);
  phase_fence();
  pencil_sums_get<1>(s, by, acc);
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    acc[0][v] += f[0][v];
    acc[3][v] += f[1][v];
  }
  pencil_volume(q, be, tab + TAB_S + 1 * TMAX * TMAX, park, unpark, acc);
  phase_fence();
  wave_sync();
  pencil_sums_put<1>(s, by, acc);
  wave_sync();
#pragma unroll
  for (int v = 0; v < 5; ++v)   // the primitives are formed again: held from the start they
#pragma unroll                  // would cost 32 registers through the other directions
    for (int i = 0; i < n; ++i) asm("" : "+v"(um[v][i]));
  (void)prims(q);
  pencil_faces<0>(g, a.surf, tab, q, un, f);
  phase_fence();
#pragma unroll
  for (int m = 0; m < n; ++m) be[m] = (gm1 * q.rho[m]) * rcp_nr1(q.p2[m]);
  pencil_sums_get<0>(s, bx, acc);
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    acc[0][v] += f[0][v];
    acc[3][v] += f[1][v];
  }
  pencil_volume(q, be, tab + TAB_S, park, unpark, acc);
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
    double kv[5][n];
#pragma unroll
    for (int v = 0; v < 5; ++v)
#pragma unroll
      for (int i = 0; i < n; ++i) kv[v][i] = a.A != 0.0 ? ld(a.k + v * ENN, ho, i) : 0.0;
    const double dt = a.dt_from ? stage_dt_from_partials(a) : *a.dt;
    const double dh = 0.5 * dt, dq = 0.25 * dt;
    if (on) {
#pragma unroll
      for (int v = 0; v < 5; ++v) {
#pragma unroll
        for (int i = 0; i < n; ++i) kv[v][i] = fma(a.A, kv[v][i], (v == 0 ? dh : dq) * acc[i][v]);
        if (a.kw) {
#pragma unroll
          for (int i = 0; i < n; ++i) st(a.k + v * ENN, ho, i, kv[v][i]);
        }
#pragma unroll
        for (int i = 0; i < n; ++i) {
          um[v][i] = fma(a.B, kv[v][i], um[v][i]);
          st(a.uout + v * ENN, ho, i, um[v][i]);
        }
      }
    }
    phase_fence();
    if (a.speed != nullptr || a.speed_slots != nullptr) {
      double l[3] = {0.0, 0.0, 0.0};
      bool ok = true;
#pragma unroll
      for (int i = 0; i < n; ++i) {
        const double u5[5] = {um[0][i], um[1][i], um[2][i], um[3][i], um[4][i]};
        Prim<double> q;
        ok &= cons_to_prim<3, false>(u5, g.gamma, q);
#pragma unroll
        for (int d = 0; d < 3; ++d) l[d] = fmax(l[d], fabs(q.v[d]) + q.c);
      }
      if (on && !ok) *g.flag = 1;
      double lam = 0.0;   // every lane of an element's row: the element's wave speed
#pragma unroll
      for (int d = 0; d < 3; ++d) lam += tab[TAB_JAC + d] * row_max16(l[d]);
      if (a.speed_slots) {   // one atomic per wave
        const double w = wave_max_lane63(on ? lam : 0.0);
        if (lane == 63) slot_max(a.speed_slots, tile, w);
      } else if (on && line == 0) {
        a.speed[e] = lam;
      }
    }
    if (a.t_step && blockIdx.x == 0 && threadIdx.x == 0) stage_time_publish(a, dt);
    if (a.slots_clear && blockIdx.x == 0 && threadIdx.x < (unsigned)DT_SLOTS)
      a.slots_clear[threadIdx.x * DT_SLOT_STRIDE] = 0.0;
  }
}

// Meshes of k_pencil.  A wave carries four elements, so a mesh needs many more elements than
// the 8 192 that its 2 048 resident waves (two per SIMD) hold at a time for the last round of
// waves not to matter.  TGV, microseconds per step, k_stage against k_pencil: 20^3 115 / 110
// (one full round), 24^3 176 / 181 (1.7 rounds), 28^3 264 / 261, 32^3 379 / 342, 64^3 3 590 /
// 3 040; right-hand sides 28^3 43 / 36, 32^3 61 / 50, 64^3 525 / 402.  Upper limit: byte
// offsets into a plane stay below 2^31 (k_stage's are 64 bits).
constexpr int64_t PENCIL_MIN_E = 20480, PENCIL_MAX_E = (int64_t)1 << 22;
// Four waves per block (x neighbours share an L1: 64^3 3 040 us per step, against 3 240 with
// one) from here on; below, single-wave blocks even out the last round (32^3: 342 against 358).
constexpr int64_t PENCIL_WIDE_E = 40960;

inline bool use_pencil(int64_t E, int surf) {
  return E >= PENCIL_MIN_E && E < PENCIL_MAX_E && (surf == SURF_LLF || surf == SURF_HLL);
}

// The waves of a block are independent (no block barrier).
template <int EPI, int WPB>
__global__ __launch_bounds__(64 * WPB) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_pencil(
    StageArgs a, Geom g) {
  __shared__ PencilLds s[WPB];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = (int)xcd_tile(blockIdx.x, gridDim.x) * WPB + w;
  if ((int64_t)tile * PENCIL_EW >= g.E) return;
  pencil_tile<EPI>(s[w], a, g, tile);
}

}  // namespace dgx
