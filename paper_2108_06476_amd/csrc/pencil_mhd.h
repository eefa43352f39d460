// pencil_mhd.h -- the MHD stages with one line of nodes per thread (see pencil.h for the split):
// the weak form (HLL or LLF) and the entropy-conservative flux differencing with Powell's term
// (EC, LLF or HLL), the semidiscretisations of k_stage_mhd and k_stage_mhd_ec.
#pragma once
#include <hip/hip_runtime.h>

#include "mhd.h"
#include "pencil.h"

namespace dgx {

// LDS buffer: the states (rho, m, E, B) of the tile's nodes; then sums.
template <int N>
struct MhdPencilLds {
  double q[8][PencilMap<N>::EB * PencilMap<N>::NN];
};

// A line's nodes; vectors in the order D, D + 1, D + 2 of the line's direction D.  The momentum is
// kept as it is stored (see PLine).
template <int n>
struct MLine {
  double rho[n], m[3][n], v[3][n], E[n], B[3][n];
};

// Plane of the buffer (and of a state) that holds component c of (rho, v or m, E, B) for a line
// of direction D.
template <int D>
__device__ __forceinline__ constexpr int mhd_plane(int c) {
  return c == 0 || c == 4 ? c : c < 4 ? 1 + (D + c - 1) % 3 : 5 + (D + c - 5) % 3;
}

template <int N, int D>
__device__ __forceinline__ void mhd_line_read(const MhdPencilLds<N>& s, int bl, MLine<N + 1>& q) {
#pragma unroll
  for (int m = 0; m < N + 1; ++m) {
    const int x = PencilPos<N>::template at<D>(bl, m);
    q.rho[m] = s.q[0][x];
    q.E[m] = s.q[4][x];
    const double inv = rcp_nr(q.rho[m]);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      q.m[k][m] = s.q[mhd_plane<D>(1 + k)][x];
      q.v[k][m] = q.m[k][m] * inv;
      q.B[k][m] = s.q[mhd_plane<D>(5 + k)][x];
    }
  }
}

template <int N, int D>
__device__ __forceinline__ void mhd_sums_get(const MhdPencilLds<N>& s, int bl, double (&acc)[N + 1][8]) {
#pragma unroll
  for (int m = 0; m < N + 1; ++m) {
    const int x = PencilPos<N>::template at<D>(bl, m);
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[m][c] = s.q[mhd_plane<D>(c)][x];
  }
}

template <int N, int D>
__device__ __forceinline__ void mhd_sums_put(MhdPencilLds<N>& s, int bl, const double (&acc)[N + 1][8]) {
#pragma unroll
  for (int m = 0; m < N + 1; ++m) {
    const int x = PencilPos<N>::template at<D>(bl, m);
#pragma unroll
    for (int c = 0; c < 8; ++c) s.q[mhd_plane<D>(c)][x] = acc[m][c];
  }
}

// The states across a line's two ends (component order of the line).
template <int N, int D>
__device__ __forceinline__ void mhd_face_load(const double* __restrict__ u, const Geom& g,
                                              const PencilPlace<N>& w, size_t ENN,
                                              double (&un)[2][8]) {
  constexpr int n = N + 1, NN = n * n * n, nd = Stride<D, n>::value;
  constexpr int na = D == 0 ? n : 1, nb = D == 2 ? n : n * n;
  const int nod = w.la * na + w.lb * nb;
  const unsigned o[2] = {((unsigned)elem_nb(g, w.e, w.ec, D, -1) * NN + nod + N * nd) * 8u,
                         ((unsigned)elem_nb(g, w.e, w.ec, D, 1) * NN + nod) * 8u};
#pragma unroll
  for (int s = 0; s < 2; ++s)
#pragma unroll
    for (int c = 0; c < 8; ++c) un[s][c] = ld(u + mhd_plane<D>(c) * ENN, o[s]);
}

// Pointwise values of one node of a line.
struct MPoint {
  double rho, inv, m[3], v[3], E, B[3], p, v2, B2, vB;
};

__device__ __forceinline__ MPoint mhd_point(double gm1, double rho, const double (&m)[3],
                                            const double (&v)[3], double E, const double (&B)[3]) {
  MPoint a;
  a.rho = rho;
  a.inv = 0.0;
  a.E = E;
  a.v2 = a.B2 = a.vB = 0.0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    a.m[k] = m[k];
    a.v[k] = v[k];
    a.B[k] = B[k];
    a.v2 += v[k] * v[k];
    a.B2 += B[k] * B[k];
    a.vB += v[k] * B[k];
  }
  a.p = gm1 * (E - 0.5 * rho * a.v2 - 0.5 * a.B2);
  return a;
}

__device__ __forceinline__ bool mhd_physical(const MPoint& a) {
  return (a.rho > 0.0) && (a.p > 0.0) && (a.p < 1.0e300) && (a.rho < 1.0e300);
}

// Physical flux along the line; the normal field's flux is zero.
__device__ __forceinline__ void mpoint_flux(const MPoint& a, double (&f)[8]) {
  const double m = a.m[0], pt = a.p + 0.5 * a.B2;
  f[0] = m;
  f[1] = m * a.v[0] + (pt - a.B[0] * a.B[0]);
  f[2] = m * a.v[1] - a.B[0] * a.B[1];
  f[3] = m * a.v[2] - a.B[0] * a.B[2];
  f[4] = a.v[0] * (a.E + pt) - a.B[0] * a.vB;
  f[5] = 0.0;
  f[6] = a.v[0] * a.B[1] - a.B[0] * a.v[1];
  f[7] = a.v[0] * a.B[2] - a.B[0] * a.v[2];
}

// Fast magnetosonic speed along component d (a.inv = 1/rho set).
__device__ __forceinline__ double mpoint_cf(const MPoint& a, double gamma, int d) {
  const double c2 = gamma * a.p * a.inv, s = c2 + a.B2 * a.inv;
  const double bd2 = a.B[d] * a.B[d] * a.inv;
  const double disc = fmax(s * s - 4.0 * c2 * bd2, 0.0);
  const double r = disc > 0.0 ? sqrt_pos(disc) : 0.0;
  return sqrt_pos(0.5 * (s + r));
}

// HLL or LLF flux through a face from the minus side L to the plus side R, up to the returned
// factor (see llf_flux).
__device__ __forceinline__ double mpoint_surface_flux(int surf, double gamma, const MPoint& L,
                                                      const MPoint& R, double (&f)[8]) {
  double fL[8], fR[8], du[8];
  mpoint_flux(L, fL);
  mpoint_flux(R, fR);
  du[0] = R.rho - L.rho;
  du[4] = R.E - L.E;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    du[1 + k] = R.m[k] - L.m[k];
    du[5 + k] = R.B[k] - L.B[k];
  }
  const double cL = mpoint_cf(L, gamma, 0), cR = mpoint_cf(R, gamma, 0);
  if (surf == SURF_LLF) {
    const double lam = fmax(fabs(L.v[0]) + cL, fabs(R.v[0]) + cR);
#pragma unroll
    for (int v = 0; v < 8; ++v) f[v] = (fL[v] + fR[v]) - lam * du[v];
    return 0.5;
  }
  const double sL = fmin(L.v[0] - cL, R.v[0] - cR), sR = fmax(L.v[0] + cL, R.v[0] + cR);
  if (sL >= 0.0) {
#pragma unroll
    for (int v = 0; v < 8; ++v) f[v] = fL[v];
    return 1.0;
  }
  if (sR <= 0.0) {
#pragma unroll
    for (int v = 0; v < 8; ++v) f[v] = fR[v];
    return 1.0;
  }
#pragma unroll
  for (int v = 0; v < 8; ++v) f[v] = sR * fL[v] - sL * fR[v] + sL * sR * du[v];
  return rcp_nr(sR - sL);
}

// The EC pair flux (mhd_ec_flux) from the logarithmic means rl = {{rho}}_ln and
// ib = 2/((gamma - 1) {{beta}}_ln), scaled by powers of two: twice the mass flux, eight times the
// energy flux, four times the others.  be: (gamma - 1) beta / 2; rb = 1/(be_L + be_R).
__device__ __forceinline__ void mpair_flux(const MPoint& L, double beL, const MPoint& R, double beR,
                                           double rl, double ib, double rb, double gm1,
                                           double (&f)[8]) {
  double sv[3], sB[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    sv[k] = L.v[k] + R.v[k];
    sB[k] = L.B[k] + R.B[k];
  }
  const double sB2 = L.B2 + R.B2;
  const double c2 = 2.0 * rb * fma(beL, L.v[0], beR * R.v[0]);   // 2 {{beta v}}/{{beta}}
  const double pt = fma(gm1 * (L.rho + R.rho), rb, sB2);
  f[0] = rl * sv[0];
  f[1] = fma(f[0], sv[0], fma(-sB[0], sB[0], pt));
  f[2] = fma(f[0], sv[1], -(sB[0] * sB[1]));
  f[3] = fma(f[0], sv[2], -(sB[0] * sB[2]));
#pragma unroll
  for (int k = 0; k < 3; ++k) f[5 + k] = fma(c2, sB[k], -(sB[0] * sv[k]));
  double e = f[0] * (ib - (L.v2 + R.v2));
#pragma unroll
  for (int k = 0; k < 3; ++k) e = fma(sv[k], f[1 + k], fma(sB[k], f[5 + k], e));
  f[4] = fma(2.0 * sB[0], L.vB + R.vB, fma(-sB2, sv[0], e));
}

// beta_ln-related means of one pair, for a face.
__device__ __forceinline__ void mpair_means(double gm1, const MPoint& L, const MPoint& R,
                                            double& beL, double& beR, double& rl, double& ib,
                                            double& rb) {
  beL = 0.25 * gm1 * L.rho * rcp_nr(L.p);
  beR = 0.25 * gm1 * R.rho * rcp_nr(R.p);
  rl = ln_mean<false>(L.rho, R.rho);
  ib = inv_ln_mean<false>(beL, beR);
  rb = rcp_nr(beL + beR);
}

template <int n>
__device__ __forceinline__ MPoint mhd_line_point(double gm1, const MLine<n>& q, int m) {
  return mhd_point(gm1, q.rho[m], {q.m[0][m], q.m[1][m], q.m[2][m]},
                   {q.v[0][m], q.v[1][m], q.v[2][m]}, q.E[m], {q.B[0][m], q.B[1][m], q.B[2][m]});
}

// Lifted face terms at the two ends of a line: f[0] minus, f[1] plus (scaled as the volume's sums
// for EC).  EC adds Powell's term phi {{B_n}} of the end node.
template <int n, int VOL>
__device__ __forceinline__ void mhd_faces(const Geom& g, int surf, ConstTab lift, double gm1,
                                          const MLine<n>& q, const double (&un)[2][8],
                                          double (&out)[2][8]) {
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    MPoint me = mhd_line_point<n>(gm1, q, s == 0 ? 0 : n - 1);
    const double inv = rcp_nr(un[s][0]);
    MPoint nb = mhd_point(gm1, un[s][0], {un[s][1], un[s][2], un[s][3]},
                          {un[s][1] * inv, un[s][2] * inv, un[s][3] * inv}, un[s][4],
                          {un[s][5], un[s][6], un[s][7]});
    if (!mhd_physical(nb)) *g.flag = 1;
    double F[8], cf = 1.0;
    bool scaled = false;   // F holds the pair flux's powers of two
    if (VOL == VOL_EC && surf == SURF_EC) {
      double beL, beR, rl, ib, rb;
      if (s == 0) {
        mpair_means(gm1, nb, me, beL, beR, rl, ib, rb);
        mpair_flux(nb, beL, me, beR, rl, ib, rb, gm1, F);
      } else {
        mpair_means(gm1, me, nb, beL, beR, rl, ib, rb);
        mpair_flux(me, beL, nb, beR, rl, ib, rb, gm1, F);
      }
      scaled = true;
    } else {
      nb.inv = inv;
      me.inv = rcp_nr(me.rho);
      cf = s == 0 ? mpoint_surface_flux(surf, g.gamma, nb, me, F)
                  : mpoint_surface_flux(surf, g.gamma, me, nb, F);
    }
    const double c0 = lift[s], c = c0 * cf;
    if constexpr (VOL == VOL_EC) {
      const double a = scaled ? 1.0 : 2.0, b = scaled ? 1.0 : 4.0, d = scaled ? 1.0 : 8.0;
      const double cB = c0 * 2.0 * (me.B[0] + nb.B[0]);   // 4 c0 {{B_n}}
      out[s][0] = a * c * F[0];
      out[s][4] = fma(2.0 * cB, me.vB, d * c * F[4]);
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        out[s][1 + k] = fma(cB, me.B[k], b * c * F[1 + k]);
        out[s][5 + k] = fma(cB, me.v[k], b * c * F[5 + k]);
      }
    } else {
#pragma unroll
      for (int v = 0; v < 8; ++v) out[s][v] = c * F[v];
    }
  }
}

// Volume term of a line, weak form: acc_i += sum_m Dhat_im f(u_m).
template <int n>
__device__ __forceinline__ void mhd_weak_line(double gm1, const MLine<n>& q, ConstTab S,
                                              double (&acc)[n][8]) {
#pragma unroll
  for (int m = 0; m < n; ++m) {
    double f[8];
    mpoint_flux(mhd_line_point<n>(gm1, q, m), f);
#pragma unroll
    for (int i = 0; i < n; ++i) {
      const double c = S[i * TMAX + m];
#pragma unroll
      for (int v = 0; v < 8; ++v)
        if (v != 5) acc[i][v] = fma(c, f[v], acc[i][v]);
    }
#pragma unroll
    for (int i = 0; i < n; ++i)
#pragma unroll
      for (int v = 0; v < 8; ++v) asm("" : "+v"(acc[i][v]));
  }
}

// Volume term of a line, EC: every pair's flux and both contributions, Powell's term as each
// node's phi times sum_m S_im {{B_n}}.
template <int n, typename Park, typename Unpark>
__device__ __forceinline__ void mhd_ec_line(double gm1, MLine<n>& q, ConstTab S, Park park,
                                            Unpark unpark, double (&acc)[n][8]) {
  double be[n], v2[n], B2[n], vB[n], pw[n];
#pragma unroll
  for (int m = 0; m < n; ++m) {
    const MPoint a = mhd_line_point<n>(gm1, q, m);
    be[m] = (0.25 * gm1 * a.rho) * rcp_nr(a.p);
    v2[m] = a.v2;
    B2[m] = a.B2;
    vB[m] = a.vB;
    pw[m] = 0.0;
  }
  auto point = [&](int m) {
    MPoint a;
    a.rho = q.rho[m];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      a.v[k] = q.v[k][m];
      a.B[k] = q.B[k][m];
    }
    a.v2 = v2[m];
    a.B2 = B2[m];
    a.vB = vB[m];
    return a;
  };
#pragma unroll
  for (int i = 0; i < n - 1; ++i) {
    double rl[n], ib[n];   // of the pair (i, m) at m - i - 1
    pencil_means<n, n>(q.rho, be, i, i + 1, n, park, unpark, rl, ib);
#pragma unroll
    for (int m = i + 1; m < n; ++m) {
      double f[8];
      const MPoint L = point(i), R = point(m);
      mpair_flux(L, be[i], R, be[m], rl[m - i - 1], ib[m - i - 1], rcp_nr(be[i] + be[m]), gm1, f);
      const double cim = S[i * TMAX + m], cmi = S[m * TMAX + i];
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        acc[i][v] = fma(cim, f[v], acc[i][v]);
        acc[m][v] = fma(cmi, f[v], acc[m][v]);
      }
      const double sB = L.B[0] + R.B[0];   // twice the mean
      pw[i] = fma(cim, sB, pw[i]);
      pw[m] = fma(cmi, sB, pw[m]);
    }
    // (sums formed here, see pencil_volume)
#pragma unroll
    for (int m = i; m < n; ++m) {
      asm("" : "+v"(pw[m]));
#pragma unroll
      for (int v = 0; v < 8; ++v) asm("" : "+v"(acc[m][v]));
    }
  }
#pragma unroll
  for (int m = 0; m < n; ++m) {
    const double c = 2.0 * pw[m];   // four times phi's factor (the energy's: eight)
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      acc[m][1 + k] = fma(q.B[k][m], c, acc[m][1 + k]);
      acc[m][5 + k] = fma(q.v[k][m], c, acc[m][5 + k]);
    }
    acc[m][4] = fma(2.0 * vB[m], c, acc[m][4]);
  }
}

template <int N, int VOL, int EPI>
__device__ __forceinline__ void mhd_pencil_tile(MhdPencilLds<N>& s, const StageArgs& a,
                                                const Geom& g, int tile) {
  using X = PencilPos<N>;
  constexpr int n = N + 1, NN = n * n * n, NL = n * n;
  // The conserved home line stays in registers where they suffice (weak N = 3: 32^3 714 us a
  // step, 810 where the update reads it again, both with plain stores).
  constexpr bool HOLD = VOL == VOL_WEAK && N == 3;
  const PencilPlace<N> w(g, tile);
  const size_t ENN = (size_t)g.E * NN;
  const ConstTab tab = const_tab(g.tab);
  const double gm1 = g.gamma - 1.0;
  unsigned ho = w.ho;
  double um[8][n], un[2][8], f[2][8], acc[n][8];
  MLine<n> q;
  auto load_u = [&]() {
#pragma unroll
    for (int v = 0; v < 8; ++v)
#pragma unroll
      for (int i = 0; i < n; ++i) um[v][i] = ld(a.uin + v * ENN, ho, i);
  };
  auto prims = [&]() {
    bool ok = true;
#pragma unroll
    for (int i = 0; i < n; ++i) {
      const double inv = rcp_nr(um[0][i]);
      q.rho[i] = um[0][i];
      q.E[i] = um[4][i];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        q.m[k][i] = um[1 + k][i];
        q.v[k][i] = um[1 + k][i] * inv;
        q.B[k][i] = um[5 + k][i];
      }
      ok &= mhd_physical(mhd_line_point<n>(gm1, q, i));
    }
    return ok;
  };
  auto volume = [&](int d, auto park, auto unpark) {
    const ConstTab S = tab + TAB_S + d * TMAX * TMAX;
    if constexpr (VOL == VOL_WEAK) mhd_weak_line<n>(gm1, q, S, acc);
    else mhd_ec_line<n>(gm1, q, S, park, unpark, acc);
  };
  auto add_faces = [&]() {
#pragma unroll
    for (int v = 0; v < 8; ++v) {
      acc[0][v] += f[0][v];
      acc[N][v] += f[1][v];
    }
  };
  load_u();
  mhd_face_load<N, 2>(a.uin, g, w, ENN, un);
  if (!prims()) *g.flag = 1;
#pragma unroll
  for (int i = 0; i < n; ++i) {
    const int x = X::template at<0>(w.bx, i);
    s.q[0][x] = q.rho[i];
    s.q[4][x] = q.E[i];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      s.q[1 + k][x] = q.m[k][i];
      s.q[5 + k][x] = q.B[k][i];
    }
  }
  pencil_sync<N>();

  // ---- z
  mhd_line_read<N, 2>(s, w.bz, q);
  mhd_faces<n, VOL>(g, a.surf, tab + TAB_LIFT + 4, gm1, q, un, f);
#pragma unroll
  for (int m = 0; m < n; ++m)
#pragma unroll
    for (int v = 0; v < 8; ++v) acc[m][v] = m == 0 ? f[0][v] : m == N ? f[1][v] : 0.0;
  phase_fence();
  volume(2, []() {}, []() {});
  phase_fence();

  // ---- y: once its lines are in registers the buffer takes the sums
  mhd_face_load<N, 1>(a.uin, g, w, ENN, un);
  mhd_line_read<N, 1>(s, w.by, q);
  pencil_sync<N>();
  mhd_sums_put<N, 2>(s, w.bz, acc);
  pencil_sync<N>();
  mhd_faces<n, VOL>(g, a.surf, tab + TAB_LIFT + 2, gm1, q, un, f);
  phase_fence();
  mhd_sums_get<N, 1>(s, w.by, acc);
  add_faces();
  volume(1, [&]() { mhd_sums_put<N, 1>(s, w.by, acc); }, [&]() { mhd_sums_get<N, 1>(s, w.by, acc); });
  phase_fence();
  if constexpr (!HOLD) load_u();
  mhd_face_load<N, 0>(a.uin, g, w, ENN, un);
  pencil_sync<N>();
  mhd_sums_put<N, 1>(s, w.by, acc);
  pencil_sync<N>();

  // ---- x
  if constexpr (HOLD) {
#pragma unroll
    for (int v = 0; v < 8; ++v)   // formed again, not held (see pencil_tile)
#pragma unroll
      for (int i = 0; i < n; ++i) asm("" : "+v"(um[v][i]));
  }
  (void)prims();
  mhd_faces<n, VOL>(g, a.surf, tab + TAB_LIFT, gm1, q, un, f);
  phase_fence();
  mhd_sums_get<N, 0>(s, w.bx, acc);
  add_faces();
  volume(0, [&]() { mhd_sums_put<N, 0>(s, w.bx, acc); }, [&]() { mhd_sums_get<N, 0>(s, w.bx, acc); });
  phase_fence();

  // epilogue: acc[i] holds the home line's right-hand side (EC: scaled by powers of two)
  const double sc[3] = {VOL == VOL_EC ? 0.5 : 1.0, VOL == VOL_EC ? 0.25 : 1.0,
                        VOL == VOL_EC ? 0.125 : 1.0};
  if constexpr (EPI == EPI_RHS) {
    if (w.on) {
#pragma unroll
      for (int v = 0; v < 8; ++v)
#pragma unroll
        for (int i = 0; i < n; ++i)
          st(a.du + v * ENN, ho, i, (v == 0 ? sc[0] : v == 4 ? sc[2] : sc[1]) * acc[i][v]);
    }
  } else {
    const double dt = *a.dt;   // (these meshes are beyond those whose stages derive it)
    // two variables at a time: all loads in flight at once would take 128 registers
#pragma unroll
    for (int v0 = 0; v0 < 8; v0 += 2) {
      double kv[2][n];
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int i = 0; i < n; ++i) {
          if constexpr (!HOLD) um[v0 + c][i] = ld(a.uin + (v0 + c) * ENN, ho, i);
          kv[c][i] = a.A != 0.0 ? ld(a.k + (v0 + c) * ENN, ho, i) : 0.0;
        }
      if (w.on) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
          const int v = v0 + c;
          const double h = dt * (v == 0 ? sc[0] : v == 4 ? sc[2] : sc[1]);
#pragma unroll
          for (int i = 0; i < n; ++i) kv[c][i] = fma(a.A, kv[c][i], h * acc[i][v]);
          if (a.kw) {
#pragma unroll
            for (int i = 0; i < n; ++i) st(a.k + v * ENN, ho, i, kv[c][i]);
          }
#pragma unroll
          for (int i = 0; i < n; ++i) um[v][i] = fma(a.B, kv[c][i], um[v][i]);
        }
      }
      if constexpr (!HOLD) phase_fence();
    }
    if (w.on)
      store_out<8>(a.nt_out, [&](int v, auto nt) {
#pragma unroll
        for (int i = 0; i < n; ++i) st_out(a.uout + v * ENN, ho, i, um[v][i], nt);
      });
    phase_fence();
    if (a.speed != nullptr) {
      double l[3] = {0.0, 0.0, 0.0};
      bool ok = true;
#pragma unroll
      for (int i = 0; i < n; ++i) {
        const double inv = rcp_nr(um[0][i]);
        MPoint pt = mhd_point(gm1, um[0][i], {um[1][i], um[2][i], um[3][i]},
                              {um[1][i] * inv, um[2][i] * inv, um[3][i] * inv}, um[4][i],
                              {um[5][i], um[6][i], um[7][i]});
        pt.inv = inv;
        ok &= mhd_physical(pt);
#pragma unroll
        for (int d = 0; d < 3; ++d) l[d] = fmax(l[d], fabs(pt.v[d]) + mpoint_cf(pt, g.gamma, d));
      }
      if (w.on && !ok) *g.flag = 1;
      const double lam = pencil_elem_speed<N>(&s.q[0][0], tab, w, l);
      if (w.on && w.line == (NL == 64 ? 63 : 0)) a.speed[w.e] = lam;
    }
  }
}

// Meshes large enough for a line per thread.  Microseconds, a node / a line per thread:
//   N = 3 weak  step  14^3 79 / 86, 16^3 105 / 105, 18^3 135 / 123, 20^3 169 / 149, 24^3 267 / 248,
//                     28^3 436 / 409, 32^3 695 / 635, 40^3 1 375 / 1 216
//               rhs   14^3 11.8 / 11.9, 16^3 15.7 / 13.7, 20^3 27.4 / 21.3, 32^3 96 / 80
//   N = 3 EC    step  14^3 96 / 104, 16^3 126 / 127, 18^3 160 / 150, 24^3 321 / 317, 32^3 835 / 708,
//                     40^3 1 533 / 1 435
//               rhs   14^3 15.3 / 14.5, 16^3 20.3 / 17.2, 20^3 36.2 / 26.0, 32^3 129 / 93
//   N = 4 weak  step  14^3 152 / 159, 20^3 338 / 378, 24^3 645 / 656, 32^3 1 535 / 1 626 (the
//                     state is read again for the update, and 14 of 64 lanes idle)
//               rhs   14^3 24.1 / 21.5, 20^3 56.7 / 52.8, 24^3 92 / 81, 32^3 247 / 193
//   N = 5 weak  step  12^3 169 / 168, 14^3 240 / 246, 16^3 335 / 333, 20^3 705 / 636, 24^3 1 235 / 1 131
//               rhs   10^3 18.5 / 19.3, 12^3 28.1 / 22.9, 16^3 57.7 / 47.8, 24^3 200 / 137
// (N = 4 and 5 EC do not fit 256 registers.)
template <int N, int VOL, int EPI>
constexpr int64_t mhd_pencil_min() {
  if (N == 3) return EPI == EPI_RK ? 5120 : 4096;
  if (N == 4) return VOL == VOL_WEAK && EPI == EPI_RHS ? 2744 : -1;
  if (N == 5) return VOL == VOL_WEAK ? (EPI == EPI_RK ? 5120 : 1728) : -1;
  return -1;   // no such kernel
}

// What bounds it: memory.  A stage of the weak form at 32^3 moves 676 MB (counted between the L2s
// and the rest, 544 MB algorithmic) in 125 us, 5.4 TB/s (143 us with a node per thread); the volume
// and face work of the waves that wait hides behind it: two per SIMD at N = 3 (up to 252 registers)
// and N = 4; at N = 5 (256 registers, up to four spilled) the LDS holds three blocks of two waves,
// one and a half per SIMD.  One wave (N = 3) or element per block: blocks
// of four waves, as k_pencil takes them on large meshes, measured 644 against 635 us at 32^3 and
// 130 against 123 at 18^3.
template <int N, int VOL, int EPI>
__global__ __launch_bounds__(PencilMap<N>::THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_pencil_mhd(StageArgs a, Geom g) {
  __shared__ MhdPencilLds<N> s;
  mhd_pencil_tile<N, VOL, EPI>(s, a, g, (int)xcd_tile(blockIdx.x, gridDim.x));
}

}  // namespace dgx
