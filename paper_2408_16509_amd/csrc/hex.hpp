// Hexahedral FR kernels (order P, Gauss--Legendre points).
//
// Native layout: state u[(pt*5 + v)*E + e] (element fastest, E = padded count),
// traces uf[(fp*5 + v)*E + e], viscous fluxes vf[(pt*9 + q)*E + e] (tau, energy flux) and
// fvn[(fp*4 + v)*E + e] (f_v.n).  Solution point pt = i + N1*(j + N1*k); flux point
// fp = face*N1^2 + q, face = 2*d + (xi_d > 0), q = t0 + N1*t1 over the two tangential
// axes of the face in increasing order.
//
// The element kernels work line by line: a line in direction d through the
// solution points (t0, t1) holds the N1 points that the 1-D operators act on, and
// both of its ends are flux points.  Along such a line the corrected divergence
// of eq:FRfinal with the DG correction reduces to
//     div_d = Dh f~_d + cp F^C(+) + cm F^C(-)
// (Dh = D - gR' l(+1)^T - gL' l(-1)^T, cp = gR', cm = -gL'), so the discontinuous
// normal flux at the ends never needs forming.  In the trace, Euler and gradient
// kernels each thread owns one line of one element per direction pass and the three
// directions' contributions meet in LDS; the NS divergence gives each thread one
// column of points and pulls the three line contractions through its points from LDS.
// The geometric map is trilinear and evaluated on the fly from its 24 monomial
// coefficients (metric terms of linear elements computed from the corners),
// staged per block in LDS.  Curved elements (CUR = true) instead read metric terms
// stored per point (Sec. "Curved elements"), layout cm (element fastest):
//   cm[(pt*9 + d*3 + j)*E + e]      row d of S = J G^{-1} at solution point pt
//   cm[(9*NSP + pt)*E + e]          1/J at solution point pt
//   cm[(10*NSP + fp*3 + j)*E + e]   row d of S at flux point fp of face 2d+s
//
// Arithmetic type T: double (the plain form) or float.  In the float form the
// state is the deviation du = u - u_ref from a constant state at rest and every
// flux is evaluated as f(u) - f(u_ref) in cancellation-free form (Flux<T, DEV>);
// this changes nothing in exact arithmetic because the transformed flux of a
// constant state has zero discrete divergence and zero interface jump.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "physics.hpp"

namespace frmi {

// Workgroups of a launch are dispatched round-robin over the 8 XCDs, each with its
// own L2.  Renumber them so that every XCD works through one contiguous range of
// logical blocks: blocks that read the same cache lines (neighbouring element tiles,
// the lines of one tile) then meet in the same L2 instead of fetching from HBM once
// per XCD.  A bijection on [0, gridDim.x).
__device__ __forceinline__ int64_t xcd_block() {
  const uint32_t b = blockIdx.x, nb = gridDim.x;
  const uint32_t x = b & 7u, i = b >> 3, q = nb >> 3, r = nb & 7u;
  return (int64_t)x * q + (x < r ? x : r) + i;
}

template <typename T>
struct HexK {
  T x[5], lm[5], lp[5], Dh[5][5], cp[5], cm[5];
};

// Reference state of the deviation form (at rest): rho0, E0, p0 = (gamma-1)E0, H0 = E0 + p0.
template <typename T>
struct RefState {
  T rho0, E0, p0, H0;
};

struct Conn {
  const int32_t* nbr_elem;   // [nfaces][E]
  const int32_t* nbr_info;   // [nfaces][E] nbr_face | orient << 3 | is_left << 12
  const int32_t* perm;       // [n_orient][stride]
  int32_t perm_stride;
};

// Inviscid flux along s and the quantities the Riemann solvers need.  DEV: the
// state holds du and the flux returned is f(u).s - f(u_ref).s.
template <typename T, bool DEV>
struct Flux {
  __device__ __forceinline__ static void eval(const T w[5], T sx, T sy, T sz, T gm1, const RefState<T>& R,
                                              T f[5], T& vs, T& p_full) {
    if constexpr (!DEV) {
      flux_dir(w, sx, sy, sz, gm1, f, vs, p_full);
    } else {
      const T rho = R.rho0 + w[0];
      const T ir = rcp(rho);
      const T vx = w[1] * ir, vy = w[2] * ir, vz = w[3] * ir;
      const T dp = gm1 * (w[4] - T(0.5) * (w[1] * vx + w[2] * vy + w[3] * vz));
      vs = vx * sx + vy * sy + vz * sz;
      f[0] = w[1] * sx + w[2] * sy + w[3] * sz;
      f[1] = w[1] * vs + dp * sx;
      f[2] = w[2] * vs + dp * sy;
      f[3] = w[3] * vs + dp * sz;
      f[4] = (R.H0 + w[4] + dp) * vs;
      p_full = R.p0 + dp;
    }
  }
  __device__ __forceinline__ static T rho(const T w[5], const RefState<T>& R) {
    if constexpr (DEV) return R.rho0 + w[0];
    else return w[0];
  }
};

// Rusanov / HLLC on (possibly deviation) states.  In the deviation form the
// constant f(u_ref).n is subtracted, which leaves every solver's formula intact
// because solvers are consistent (𝔉(u, u, n) = f(u).n).
template <typename T, bool DEV>
__device__ __forceinline__ void common_inviscid(int kind, const T uL[5], const T uR[5], const T n[3], T gamma,
                                                const RefState<T>& R, T F[5]) {
  const T gm1 = gamma - T(1);
  T fL[5], fR[5], vnL, vnR, pL, pR;
  Flux<T, DEV>::eval(uL, n[0], n[1], n[2], gm1, R, fL, vnL, pL);
  Flux<T, DEV>::eval(uR, n[0], n[1], n[2], gm1, R, fR, vnR, pR);
  const T rL = Flux<T, DEV>::rho(uL, R), rR = Flux<T, DEV>::rho(uR, R);
  const T cL = fsqrt(fdiv(gamma * pL, rL)), cR = fsqrt(fdiv(gamma * pR, rR));
  if (kind != 1) {
    const T lam = fmax(fabs(vnL) + cL, fabs(vnR) + cR);
#pragma unroll
    for (int v = 0; v < 5; ++v) F[v] = T(0.5) * (fL[v] + fR[v]) - T(0.5) * lam * (uR[v] - uL[v]);
    return;
  }
  const T SL = fmin(vnL - cL, vnR - cR);
  const T SR = fmax(vnL + cL, vnR + cR);
  // pR - pL from the deviation pressures in the float form (same value in exact arithmetic)
  const T dpLR = pR - pL;
  const T Ss = fdiv(dpLR + rL * vnL * (SL - vnL) - rR * vnR * (SR - vnR), rL * (SL - vnL) - rR * (SR - vnR));
  if (T(0) <= SL) {
#pragma unroll
    for (int v = 0; v < 5; ++v) F[v] = fL[v];
    return;
  }
  const bool left = T(0) <= Ss;
  if (!left && !(T(0) < SR)) {
#pragma unroll
    for (int v = 0; v < 5; ++v) F[v] = fR[v];
    return;
  }
  const T* wK = left ? uL : uR;
  const T* fK = left ? fL : fR;
  const T S = left ? SL : SR, vn = left ? vnL : vnR, p = left ? pL : pR, r = left ? rL : rR;
  // U*_K - U_K written without forming U*_K (no cancellation of the total energy):
  //   mass: r (Ss - vn)/(S - Ss); momentum: that times v + fac (Ss - vn) n;
  //   energy: (Ss - vn)/(S - Ss) [r (S - vn) Ss + p + E]
  const T fac = fdiv(r * (S - vn), S - Ss);
  const T q = fdiv(Ss - vn, S - Ss);
  const T E = DEV ? R.E0 + wK[4] : wK[4];
  T dU[5];
  dU[0] = r * q;
  dU[1] = wK[1] * q + fac * (Ss - vn) * n[0];
  dU[2] = wK[2] * q + fac * (Ss - vn) * n[1];
  dU[3] = wK[3] * q + fac * (Ss - vn) * n[2];
  dU[4] = q * (r * (S - vn) * Ss + p + E);
#pragma unroll
  for (int v = 0; v < 5; ++v) F[v] = fK[v] + S * dU[v];
}

// Viscous flux along s from (possibly deviation) state and its gradient.
template <typename T, bool DEV>
__device__ __forceinline__ void viscous(const T w[5], const T g[15], T sx, T sy, T sz, T gamma, T mu, T pr,
                                        const RefState<T>& R, T fv[5]) {
  T u[5] = {w[0], w[1], w[2], w[3], w[4]};
  if constexpr (DEV) { u[0] += R.rho0; u[4] += R.E0; }
  viscous_dir(u, g, sx, sy, sz, gamma, mu, pr, fv);
}

// Navier--Stokes flux of one solution point along several directions s:
// (f_inv - f_v).s.  The velocity, (deviation) pressure and enthalpy, the viscous stress
// tau and the energy flux vector tau v + kappa grad e are formed once per point (the same
// formulas as Flux::eval and viscous_dir); each direction then costs a few products.
template <typename T, bool DEV>
struct PointFluxNS {
  T m[3], vx, vy, vz, dp, h;       // momentum, velocity, (deviation) pressure, (deviation) H v factor
  T tau[6], qe[3];                 // tau_xx, tau_yy, tau_zz, tau_xy, tau_xz, tau_yz; energy flux vector
  __device__ __forceinline__ PointFluxNS(const T w[5], const T g[15], T gamma, T mu, T pr, const RefState<T>& R) {
    const T gm1 = gamma - T(1);
    const T rho = DEV ? R.rho0 + w[0] : w[0];
    const T Et = DEV ? R.E0 + w[4] : w[4];
    const T ir = rcp(rho);
    m[0] = w[1]; m[1] = w[2]; m[2] = w[3];
    vx = w[1] * ir; vy = w[2] * ir; vz = w[3] * ir;
    dp = gm1 * (w[4] - T(0.5) * (w[1] * vx + w[2] * vy + w[3] * vz));
    // DEV: (H0 + dE + dp) multiplies v.s (f(u).s - f(u_ref).s); else (E + p)
    h = DEV ? R.H0 + w[4] + dp : w[4] + dp;
    const T v[3] = {vx, vy, vz};
    T gv[3][3];                                   // gv[i][j] = d v_i / d x_j
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int j = 0; j < 3; ++j) gv[i][j] = (g[(1 + i) * 3 + j] - v[i] * g[j]) * ir;
    const T Er = Et * ir;
    T ge[3];
#pragma unroll
    for (int j = 0; j < 3; ++j)
      ge[j] = (g[12 + j] - Er * g[j] - (w[1] * gv[0][j] + w[2] * gv[1][j] + w[3] * gv[2][j])) * ir;
    const T div = gv[0][0] + gv[1][1] + gv[2][2];
    const T d23 = T(2.0 / 3.0) * div;
    tau[0] = mu * (T(2) * gv[0][0] - d23);
    tau[1] = mu * (T(2) * gv[1][1] - d23);
    tau[2] = mu * (T(2) * gv[2][2] - d23);
    tau[3] = mu * (gv[0][1] + gv[1][0]);
    tau[4] = mu * (gv[0][2] + gv[2][0]);
    tau[5] = mu * (gv[1][2] + gv[2][1]);
    const T kappa = fdiv(mu * gamma, pr);
    qe[0] = tau[0] * vx + tau[3] * vy + tau[4] * vz + kappa * ge[0];
    qe[1] = tau[3] * vx + tau[1] * vy + tau[5] * vz + kappa * ge[1];
    qe[2] = tau[4] * vx + tau[5] * vy + tau[2] * vz + kappa * ge[2];
  }
  __device__ __forceinline__ void dir(T sx, T sy, T sz, T f[5]) const {
    const T vs = vx * sx + vy * sy + vz * sz;
    f[0] = DEV ? m[0] * sx + m[1] * sy + m[2] * sz : (m[0] * sx + m[1] * sy + m[2] * sz);
    f[1] = m[0] * vs + dp * sx - (tau[0] * sx + tau[3] * sy + tau[4] * sz);
    f[2] = m[1] * vs + dp * sy - (tau[3] * sx + tau[1] * sy + tau[5] * sz);
    f[3] = m[2] * vs + dp * sz - (tau[4] * sx + tau[5] * sy + tau[2] * sz);
    f[4] = h * vs - (qe[0] * sx + qe[1] * sy + qe[2] * sz);
  }
  // the viscous part alone, f_v.s, without its zero mass component (4 values)
  __device__ __forceinline__ void visc(T sx, T sy, T sz, T fv[4]) const {
    fv[0] = tau[0] * sx + tau[3] * sy + tau[4] * sz;
    fv[1] = tau[3] * sx + tau[1] * sy + tau[5] * sz;
    fv[2] = tau[4] * sx + tau[5] * sy + tau[2] * sz;
    fv[3] = qe[0] * sx + qe[1] * sy + qe[2] * sz;
  }
};

// Stored viscous flux of a point (PointFluxNS's tau and qe, 9 values) along s, taken off f.
template <typename T>
__device__ __forceinline__ void minus_visc(const T q[9], T sx, T sy, T sz, T f[5]) {
  f[1] -= q[0] * sx + q[3] * sy + q[4] * sz;
  f[2] -= q[3] * sx + q[1] * sy + q[5] * sz;
  f[3] -= q[4] * sx + q[5] * sy + q[2] * sz;
  f[4] -= q[6] * sx + q[7] * sy + q[8] * sz;
}

// The inviscid part of PointFluxNS: f_inv.s along several directions of one point.
template <typename T, bool DEV>
struct PointInv {
  T m[3], vx, vy, vz, dp, h;
  __device__ __forceinline__ PointInv(const T w[5], T gamma, const RefState<T>& R) {
    const T gm1 = gamma - T(1);
    const T rho = DEV ? R.rho0 + w[0] : w[0];
    const T ir = rcp(rho);
    m[0] = w[1]; m[1] = w[2]; m[2] = w[3];
    vx = w[1] * ir; vy = w[2] * ir; vz = w[3] * ir;
    dp = gm1 * (w[4] - T(0.5) * (w[1] * vx + w[2] * vy + w[3] * vz));
    h = DEV ? R.H0 + w[4] + dp : w[4] + dp;
  }
  __device__ __forceinline__ void dir(T sx, T sy, T sz, T f[5]) const {
    const T vs = vx * sx + vy * sy + vz * sz;
    f[0] = m[0] * sx + m[1] * sy + m[2] * sz;
    f[1] = m[0] * vs + dp * sx;
    f[2] = m[1] * vs + dp * sy;
    f[3] = m[2] * vs + dp * sz;
    f[4] = h * vs;
  }
};

// Columns of G = dx/dxi at reference point (a, b, d) of a trilinear map with
// monomial coefficients c[comp*8 + S], S in {1, a, b, d, ab, ad, bd, abd}; c is
// read through the stride `cs` (LDS staging).
template <typename T>
__device__ __forceinline__ void hex_cols(const T* c, int cs, T a, T b, T d, T g[3][3]) {
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const T* q = c + k * 8 * cs;
    const T q1 = q[1 * cs], q2 = q[2 * cs], q3 = q[3 * cs], q4 = q[4 * cs];
    const T q5 = q[5 * cs], q6 = q[6 * cs], q7 = q[7 * cs];
    g[0][k] = q1 + q4 * b + q5 * d + q7 * b * d;
    g[1][k] = q2 + q4 * a + q6 * d + q7 * a * d;
    g[2][k] = q3 + q5 * a + q6 * b + q7 * a * b;
  }
}

template <typename T>
__device__ __forceinline__ void cross3(const T* u, const T* v, T* w) {
  w[0] = u[1] * v[2] - u[2] * v[1];
  w[1] = u[2] * v[0] - u[0] * v[2];
  w[2] = u[0] * v[1] - u[1] * v[0];
}

template <int N1>
__device__ __forceinline__ int line_pt(int d, int a, int t0, int t1) {
  return d == 0 ? a + N1 * (t0 + N1 * t1) : (d == 1 ? t0 + N1 * (a + N1 * t1) : t0 + N1 * (t1 + N1 * a));
}

template <typename T>
__device__ __forceinline__ void line_xi(const HexK<T>& K, int d, int a, int t0, int t1, T xi[3]) {
  const T ta = K.x[t0], tb = K.x[t1], xa = K.x[a];
  xi[0] = d == 0 ? xa : ta;
  xi[1] = d == 0 ? ta : (d == 1 ? xa : tb);
  xi[2] = d == 2 ? xa : tb;
}

template <typename T>
__device__ __forceinline__ void end_xi(const HexK<T>& K, int d, int s, int t0, int t1, T xi[3]) {
  const T ta = K.x[t0], tb = K.x[t1], xe = s ? T(1) : T(-1);
  xi[0] = d == 0 ? xe : ta;
  xi[1] = d == 0 ? ta : (d == 1 ? xe : tb);
  xi[2] = d == 2 ? xe : tb;
}

// S row d = g_{d+1} x g_{d+2}: row d of J G^{-1}.
template <typename T>
__device__ __forceinline__ void srow(const T g[3][3], int d, T s[3]) {
  if (d == 0) cross3(g[1], g[2], s);
  else if (d == 1) cross3(g[2], g[0], s);
  else cross3(g[0], g[1], s);
}

template <typename T>
__device__ __forceinline__ T det_cols(const T g[3][3]) {
  T cr[3];
  cross3(g[1], g[2], cr);
  return g[0][0] * cr[0] + g[0][1] * cr[1] + g[0][2] * cr[2];
}

// Neighbour flux-point slot of end `face` / face-local point q of element e.
struct NbrSlot {
  int64_t elem;
  int fp;
  bool left;
};

template <int NFPF>
__device__ __forceinline__ NbrSlot nbr_slot(const Conn& C, int64_t E, int64_t e, int face, int q) {
  const int info = C.nbr_info[(int64_t)face * E + e];
  NbrSlot s;
  s.elem = C.nbr_elem[(int64_t)face * E + e];
  const int nf = info & 7, orient = (info >> 3) & 511;
  s.left = (info >> 12) & 1;
  s.fp = nf * NFPF + C.perm[orient * C.perm_stride + q];
  return s;
}

template <typename T, int NSP>
__device__ __forceinline__ void cm_srow(const T* __restrict__ cm, int64_t E, int64_t e, int pt, int d, T s[3]) {
#pragma unroll
  for (int j = 0; j < 3; ++j) s[j] = cm[((int64_t)pt * 9 + d * 3 + j) * E + e];
}

template <typename T, int NSP>
__device__ __forceinline__ T cm_rjac(const T* __restrict__ cm, int64_t E, int64_t e, int pt) {
  return cm[((int64_t)9 * NSP + pt) * E + e];
}

template <typename T, int NSP>
__device__ __forceinline__ void cm_fnrm(const T* __restrict__ cm, int64_t E, int64_t e, int fp, T s[3]) {
#pragma unroll
  for (int j = 0; j < 3; ++j) s[j] = cm[((int64_t)10 * NSP + fp * 3 + j) * E + e];
}

// Stage the block's geometry coefficients into LDS: G[g*NE + el].
template <typename T, int NE, int NT>
__device__ __forceinline__ void stage_geo(const T* __restrict__ geo, int64_t E, int64_t e0, T* G) {
  for (int i = threadIdx.x; i < 24 * NE; i += NT) {
    const int g = i / NE, el = i % NE;
    G[i] = geo[(int64_t)g * E + e0 + el];
  }
}

// ---------------------------------------------------------------------------
// Step 1 (eq:disu) at the flux points: traces of u at both ends of every line.
template <typename T, int P>
__global__ void __launch_bounds__(256) hex_trace(const T* __restrict__ u, T* __restrict__ uf, int64_t E, HexK<T> K) {
  constexpr int N1 = P + 1, NL = 3 * N1 * N1;
  const int64_t gtid = xcd_block() * 256 + threadIdx.x;
  const int64_t wave = gtid >> 6;
  const int lane = (int)(gtid & 63);
  const int64_t tile = wave / NL;
  const int l = (int)(wave % NL);
  const int64_t e = tile * 64 + lane;
  if (e >= E) return;
  const int d = l / (N1 * N1), q = l % (N1 * N1), t0 = q % N1, t1 = q / N1;
  T m[5] = {0, 0, 0, 0, 0}, p[5] = {0, 0, 0, 0, 0};
#pragma unroll
  for (int a = 0; a < N1; ++a) {
    const int pt = line_pt<N1>(d, a, t0, t1);
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const T val = u[((int64_t)pt * 5 + v) * E + e];
      m[v] += K.lm[a] * val;
      p[v] += K.lp[a] * val;
    }
  }
  const int fm = (2 * d) * N1 * N1 + q, fp = (2 * d + 1) * N1 * N1 + q;
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    uf[((int64_t)fm * 5 + v) * E + e] = m[v];
    uf[((int64_t)fp * 5 + v) * E + e] = p[v];
  }
}

// Accumulate one direction's divergence contribution into LDS and, in the last
// pass, write R = -div / J.
template <typename T, int N1, int NE, bool CUR>
__device__ __forceinline__ void accumulate_div(int d, const T (&ft)[5][N1], const T (&Fc)[2][5], const HexK<T>& K,
                                               T* DIV, const T* G, const T* __restrict__ cm, int el, int t0, int t1,
                                               int64_t e, int64_t n, int64_t E, T* __restrict__ r) {
  constexpr int NSP = N1 * N1 * N1;
#pragma unroll
  for (int a = 0; a < N1; ++a) {
    const int pt = line_pt<N1>(d, a, t0, t1);
    T div[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      T acc = K.cp[a] * Fc[1][v] + K.cm[a] * Fc[0][v];
#pragma unroll
      for (int b = 0; b < N1; ++b) acc += K.Dh[a][b] * ft[v][b];
      div[v] = acc;
    }
    T* D = DIV + (pt * NE + el);
    if (d == 0) {
#pragma unroll
      for (int v = 0; v < 5; ++v) D[v * NSP * NE] = div[v];
    } else if (d == 1) {
#pragma unroll
      for (int v = 0; v < 5; ++v) D[v * NSP * NE] += div[v];
    } else {
      T iJ;
      if constexpr (CUR) {
        iJ = -cm_rjac<T, NSP>(cm, E, e, pt);
      } else {
        T xi[3], g[3][3];
        line_xi(K, d, a, t0, t1, xi);
        hex_cols(G + el, NE, xi[0], xi[1], xi[2], g);
        iJ = -rcp(det_cols(g));
      }
      if (e < n) {
#pragma unroll
        for (int v = 0; v < 5; ++v) r[((int64_t)pt * 5 + v) * E + e] = (D[v * NSP * NE] + div[v]) * iJ;
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Steps 2-4 for Euler, fused: per line, own traces, neighbour traces, common flux
// (eq:comm_flux) at both ends, transformed flux at the line points and the
// corrected divergence (eq:FRfinal); R = -div / J.
template <typename T, bool DEV, int P, int NE, bool CUR = false>
__global__ void __launch_bounds__(NE*(P + 1)*(P + 1)) hex_div_euler(
    const T* __restrict__ u, const T* __restrict__ uf, const T* __restrict__ geo, const T* __restrict__ cm,
    Conn C, T* __restrict__ r, int64_t E, int64_t n, HexK<T> K, T gamma, int riemann, RefState<T> R) {
  constexpr int N1 = P + 1, NSP = N1 * N1 * N1, NF = N1 * N1, NT = NE * N1 * N1;
  __shared__ T DIV[5 * NSP * NE];
  __shared__ T G[CUR ? 1 : 24 * NE];
  const int el = threadIdx.x % NE, l = threadIdx.x / NE;
  const int64_t e0 = xcd_block() * NE, e = e0 + el;
  const int t0 = l % N1, t1 = l / N1;
  if constexpr (!CUR) stage_geo<T, NE, NT>(geo, E, e0, G);
  __syncthreads();
  const T gm1 = gamma - T(1);
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    T ft[5][N1], tm[5] = {0, 0, 0, 0, 0}, tp[5] = {0, 0, 0, 0, 0};
#pragma unroll
    for (int a = 0; a < N1; ++a) {
      const int pt = line_pt<N1>(d, a, t0, t1);
      T uu[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        uu[v] = u[((int64_t)pt * 5 + v) * E + e];
        tm[v] += K.lm[a] * uu[v];
        tp[v] += K.lp[a] * uu[v];
      }
      T s[3], f[5], vs, pr;
      if constexpr (CUR) {
        cm_srow<T, NSP>(cm, E, e, pt, d, s);
      } else {
        T xi[3], g[3][3];
        line_xi(K, d, a, t0, t1, xi);
        hex_cols(G + el, NE, xi[0], xi[1], xi[2], g);
        srow(g, d, s);
      }
      Flux<T, DEV>::eval(uu, s[0], s[1], s[2], gm1, R, f, vs, pr);
#pragma unroll
      for (int v = 0; v < 5; ++v) ft[v][a] = f[v];
    }
    T Fc[2][5];
#pragma unroll
    for (int sd = 0; sd < 2; ++sd) {
      T nv[3];
      if constexpr (CUR) {
        cm_fnrm<T, NSP>(cm, E, e, (2 * d + sd) * NF + l, nv);
      } else {
        T xi[3], g[3][3];
        end_xi(K, d, sd, t0, t1, xi);
        hex_cols(G + el, NE, xi[0], xi[1], xi[2], g);
        srow(g, d, nv);
      }
      const T sg = sd ? T(1) : T(-1);
      const T mag = fsqrt(nv[0] * nv[0] + nv[1] * nv[1] + nv[2] * nv[2]);
      const NbrSlot ns = nbr_slot<NF>(C, E, e, 2 * d + sd, l);
      T un[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) un[v] = uf[((int64_t)ns.fp * 5 + v) * E + ns.elem];
      const T* own = sd ? tp : tm;
      T uL[5], uR[5], nL[3], F[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) { uL[v] = ns.left ? own[v] : un[v]; uR[v] = ns.left ? un[v] : own[v]; }
      const T sl = fdiv(ns.left ? sg : -sg, mag);
#pragma unroll
      for (int k = 0; k < 3; ++k) nL[k] = nv[k] * sl;
      common_inviscid<T, DEV>(riemann, uL, uR, nL, gamma, R, F);
      const T fs = ns.left ? mag : -mag;
#pragma unroll
      for (int v = 0; v < 5; ++v) Fc[sd][v] = fs * F[v];
    }
    accumulate_div<T, N1, NE, CUR>(d, ft, Fc, K, DIV, G, cm, el, t0, t1, e, n, E, r);
    if (d < 2) __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// The same steps with a thread per line of each direction, for meshes of few blocks, where
// the time is one block's latency: the three directions of an element run side by side, their
// loads are all issued first and they meet in LDS once.  The LDS of three directions allows
// half the elements per block.  Sums in hex_div_euler's order.
// wide_own_traces: the partners' traces are formed here from their lines and hex_trace is not
// launched, where both lines of a thread fit beside the rest of its registers and cost little
// more than the traces when the partners lie scattered.  A whole right-hand side of 2,030
// renumbered elements, us, by hex_trace and hex_div_euler / by hex_trace and this / with the
// lines: p = 3 FP64 straight 23.0 / 20.1 / 23.6, curved 21.1 / 16.6 / 15.4; FP32 straight
// 16.8 / 14.7 / 13.5, curved 14.6 / 12.2 / 10.9; p = 4 FP32 straight 20.8 / 20.7 / 24.2, curved
// 18.7 / 17.6 / 20.0 (p = 4 FP64, 10^3 in order: 24 with the traces, 32 with the lines).
template <typename T, int P, bool CUR>
constexpr bool wide_own_traces() { return P < 3 || (P == 3 && (CUR || sizeof(T) == 4)); }
template <typename T, bool DEV, int P, int NE, bool CUR = false>
__global__ void __launch_bounds__(3 * NE * (P + 1) * (P + 1)) hex_div_euler_wide(
    const T* __restrict__ u, const T* __restrict__ uf, const T* __restrict__ geo, const T* __restrict__ cm,
    Conn C, T* __restrict__ r, int64_t E, int64_t n, HexK<T> K, T gamma, int riemann, RefState<T> R) {
  constexpr int N1 = P + 1, NSP = N1 * N1 * N1, NF = N1 * N1, NT = 3 * NE * NF;
  constexpr bool LN = wide_own_traces<T, P, CUR>();
  __shared__ T DIV[3 * 5 * NSP * NE];              // [d][v][pt][el]
  __shared__ T G[CUR ? 1 : 24 * NE];
  const int el = threadIdx.x % NE, dl = threadIdx.x / NE, d = dl / NF, l = dl % NF;
  const int64_t e0 = xcd_block() * NE, e = e0 + el;
  const int t0 = l % N1, t1 = l / N1;
  const NbrSlot ns0 = nbr_slot<NF>(C, E, e, 2 * d, l), ns1 = nbr_slot<NF>(C, E, e, 2 * d + 1, l);
  T uu[N1][5], ub[LN ? 2 : 1][LN ? N1 : 1][5], un[2][5];
#pragma unroll
  for (int a = 0; a < N1; ++a)
#pragma unroll
    for (int v = 0; v < 5; ++v) uu[a][v] = u[((int64_t)line_pt<N1>(d, a, t0, t1) * 5 + v) * E + e];
  // the partners' lines: point b0 + a st of the face's line
  auto load_nbr = [&](const NbrSlot& ns, int sd) {
    const int dn = ns.fp / (2 * NF), q = ns.fp % NF;
    const int b0 = dn == 0 ? q * N1 : (dn == 1 ? q % N1 + NF * (q / N1) : q), st = dn == 0 ? 1 : (dn == 1 ? N1 : NF);
    const T* const p = u + (int64_t)b0 * 5 * E + ns.elem;
#pragma unroll
    for (int a = 0; a < N1; ++a)
#pragma unroll
      for (int v = 0; v < 5; ++v) ub[sd][a][v] = p[((int64_t)a * st * 5 + v) * E];
  };
  if constexpr (LN) {
    load_nbr(ns0, 0);
    load_nbr(ns1, 1);
  } else {
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      un[0][v] = uf[((int64_t)ns0.fp * 5 + v) * E + ns0.elem];
      un[1][v] = uf[((int64_t)ns1.fp * 5 + v) * E + ns1.elem];
    }
  }
  if constexpr (!CUR) stage_geo<T, NE, NT>(geo, E, e0, G);
  __syncthreads();
  const T gm1 = gamma - T(1);
  if constexpr (LN) {
#pragma unroll
    for (int sd = 0; sd < 2; ++sd) {
      const bool top = ((sd ? ns1.fp : ns0.fp) / NF) & 1;
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        T x = 0;
#pragma unroll
        for (int a = 0; a < N1; ++a) x += (top ? K.lp[a] : K.lm[a]) * ub[sd][a][v];
        un[sd][v] = x;
      }
    }
  }
  // row d of S at reference point xi (straight elements)
  auto metric = [&](const T xi[3], T s[3]) {
    T g[3][3], p[3], q[3];
    hex_cols(G + el, NE, xi[0], xi[1], xi[2], g);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      p[k] = d == 0 ? g[1][k] : (d == 1 ? g[2][k] : g[0][k]);
      q[k] = d == 0 ? g[2][k] : (d == 1 ? g[0][k] : g[1][k]);
    }
    cross3(p, q, s);
  };
  T ft[5][N1], tm[5] = {0, 0, 0, 0, 0}, tp[5] = {0, 0, 0, 0, 0};
#pragma unroll
  for (int a = 0; a < N1; ++a) {
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      tm[v] += K.lm[a] * uu[a][v];
      tp[v] += K.lp[a] * uu[a][v];
    }
    T s[3], f[5], vs, pr;
    if constexpr (CUR) {
      cm_srow<T, NSP>(cm, E, e, line_pt<N1>(d, a, t0, t1), d, s);
    } else {
      T xi[3];
      line_xi(K, d, a, t0, t1, xi);
      metric(xi, s);
    }
    Flux<T, DEV>::eval(uu[a], s[0], s[1], s[2], gm1, R, f, vs, pr);
#pragma unroll
    for (int v = 0; v < 5; ++v) ft[v][a] = f[v];
  }
  T Fc[2][5];
#pragma unroll
  for (int sd = 0; sd < 2; ++sd) {
    T nv[3];
    if constexpr (CUR) {
      cm_fnrm<T, NSP>(cm, E, e, (2 * d + sd) * NF + l, nv);
    } else {
      T xi[3];
      end_xi(K, d, sd, t0, t1, xi);
      metric(xi, nv);
    }
    const T sg = sd ? T(1) : T(-1);
    const T mag = fsqrt(nv[0] * nv[0] + nv[1] * nv[1] + nv[2] * nv[2]);
    const bool left = sd ? ns1.left : ns0.left;
    const T* own = sd ? tp : tm;
    T uL[5], uR[5], nL[3], F[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) { uL[v] = left ? own[v] : un[sd][v]; uR[v] = left ? un[sd][v] : own[v]; }
    const T sl = fdiv(left ? sg : -sg, mag);
#pragma unroll
    for (int k = 0; k < 3; ++k) nL[k] = nv[k] * sl;
    common_inviscid<T, DEV>(riemann, uL, uR, nL, gamma, R, F);
    const T fs = left ? mag : -mag;
#pragma unroll
    for (int v = 0; v < 5; ++v) Fc[sd][v] = fs * F[v];
  }
#pragma unroll
  for (int a = 0; a < N1; ++a) {
    T* D = DIV + (d * 5 * NSP + line_pt<N1>(d, a, t0, t1)) * NE + el;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      T acc = K.cp[a] * Fc[1][v] + K.cm[a] * Fc[0][v];
#pragma unroll
      for (int b = 0; b < N1; ++b) acc += K.Dh[a][b] * ft[v][b];
      D[v * NSP * NE] = acc;
    }
  }
  __syncthreads();
  if (e >= n) return;
  // a point per thread: the three directions' sum
  for (int pt = dl; pt < NSP; pt += 3 * NF) {
    T iJ;
    if constexpr (CUR) {
      iJ = -cm_rjac<T, NSP>(cm, E, e, pt);
    } else {
      T g[3][3];
      hex_cols(G + el, NE, K.x[pt % N1], K.x[pt / N1 % N1], K.x[pt / (N1 * N1)], g);
      iJ = -rcp(det_cols(g));
    }
    const T* D = DIV + pt * NE + el;
#pragma unroll
    for (int v = 0; v < 5; ++v)
      r[((int64_t)pt * 5 + v) * E + e] =
          (D[v * NSP * NE] + D[(5 + v) * NSP * NE] + D[(10 + v) * NSP * NE]) * iJ;
  }
}

// LDS slot of point pt in the gradient kernel's [component][point][element] buffers.
// With 4 points per line and rows of 64 bytes a point row is 16 banks, and the rows a wave
// touches on lines along xi_1 are 4 apart (same 16 banks of 64): the XOR of the point's low
// two bits with the next two spreads them over different bank groups.  A bijection on [0, 64).
template <typename T, int N1, int NE>
__device__ __forceinline__ int gr_slot(int pt) {
  if constexpr (N1 == 4 && NE * sizeof(T) == 64) return pt ^ ((pt >> 2) & 3);
  else return pt;
}

// ---------------------------------------------------------------------------
// Navier--Stokes phase 1: corrected gradient (LDG common solution u^ at the flux points),
// and from it the viscous fluxes: the physical f_v of every solution point (tau and the
// energy flux vector, 9 values where the gradient has 15) and f_v.n of the own trace and the
// traced gradient at the flux points that the viscous common flux reads (4 values for 15; n
// the left side's unit normal).  side_mode: +1 when beta = +1/2 (u^ = u_L, the viscous common
// flux takes the right side only: the left side's jump vanishes and only right sides store
// f_v.n), -1 for beta = -1/2 (the mirror case), 0 in general.
//
// Bound by its bytes (state, partner traces, 9 + up to 9 values per point out).  All the
// global reads are issued first; the state goes to LDS, the line ends form u^ (own traces
// stay in registers), each thread forms all 15 components of its points' gradients in
// registers, and these replace the state in LDS for the traces: four barriers in all.
// Bytes aside it pays for vector instructions (710 per FP32 point at p = 3, half of the issue slots;
// addresses step from one base per array) and for its phases (waves wait half of their cycles).  With the pass that follows it, against storing the
// 15 gradient components and their traces and forming both fluxes later, us (gradient / common
// flux / divergence): 32^3 p = 3 FP32 76 / 49 / 83 -> 73 / 34 / 51, FP64 158 / 120 / 146 ->
// 147 / 74 / 125; 28^3 p = 4 FP64 232 / 123 / 278 -> 223 / 80 / 242; 10^3 p = 3 FP64 gradient
// 21.6 -> 13.6.
template <typename T, bool DEV, int P, int NE, int KT, bool CUR>
__global__ void __launch_bounds__(NE*(P + 1)*(P + 1)*KT) hex_grad(
    const T* __restrict__ u, const T* __restrict__ uf, const T* __restrict__ geo, const T* __restrict__ cm,
    Conn C, T* __restrict__ vf, T* __restrict__ fvn, int64_t E, HexK<T> K, T gamma, T mu, T pr, T beta, int side_mode,
    RefState<T> R) {
  constexpr int N1 = P + 1, NSP = N1 * N1 * N1, NF = N1 * N1, W = NF * KT, NT = NE * W;
  constexpr int PPT = (N1 + KT - 1) / KT, EPT = (6 * NF + W - 1) / W;
  constexpr int ROWS = 15 * NSP > 5 * NSP + 30 * NF ? 15 * NSP : 5 * NSP + 30 * NF;
  __shared__ T S[ROWS * NE];
  __shared__ T G[CUR ? 1 : 24 * NE];
  T* const U = S;                        // the block's state, [v][pt][el]; then the gradients, [c][pt][el]
  T* const UH = S + 5 * NSP * NE;        // u^ at the line ends, [f][v][el]
  const int el = threadIdx.x % NE, w = threadIdx.x / NE;
  const int64_t e0 = xcd_block() * NE, e = e0 + el;
  auto at = [&](int c, int pt) -> int { return (c * NSP + gr_slot<T, N1, NE>(pt)) * NE + el; };
  // ends f = w, w + W, ...: end f's line starts at point b0 with stride st
  auto line_of = [&](int f, int& d, int& b0, int& st) {
    const int q = f % NF;
    d = f / (2 * NF);
    b0 = d == 0 ? q * N1 : (d == 1 ? q % N1 + NF * (q / N1) : q);
    st = d == 0 ? 1 : (d == 1 ? N1 : NF);
  };
  NbrSlot ns[EPT];
  bool need[EPT];
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int f = w + i * W < 6 * NF ? w + i * W : 0;
    ns[i] = nbr_slot<NF>(C, E, e, f / NF, f % NF);
    need[i] = side_mode == 0 || (side_mode > 0 ? !ns[i].left : ns[i].left);
  }
  if constexpr (!CUR) stage_geo<T, NE, NT>(geo, E, e0, G);
  // (one 64-bit address per thread and array, uniform steps from there: the 64-bit products of
  // an address per load were a quarter of the kernel's issue slots)
  const T* const uw = u + (int64_t)w * E + e;
#pragma unroll
  for (int i = 0; i < (5 * NSP + W - 1) / W; ++i) {
    const int row = w + i * W;
    if (row < 5 * NSP) U[at(row % 5, row / 5)] = uw[(int64_t)i * W * E];
  }
  T un[EPT][5], own[EPT][5];
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const T* const un_i = uf + (int64_t)ns[i].fp * 5 * E + ns[i].elem;
#pragma unroll
    for (int v = 0; v < 5; ++v) un[i][v] = need[i] ? un_i[(int64_t)v * E] : T(0);
  }
  __syncthreads();
  // common solution values u^ (LDG) at the line ends
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int f = w + i * W;
    if (f >= 6 * NF) break;
    int d, b0, st;
    line_of(f, d, b0, st);
    const bool sd = (f / NF) & 1;
    const T bs = ns[i].left ? beta : -beta;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      T x = 0;
#pragma unroll
      for (int a = 0; a < N1; ++a) x += (sd ? K.lp[a] : K.lm[a]) * U[at(v, b0 + a * st)];
      own[i][v] = x;
      UH[(f * 5 + v) * NE + el] = need[i] ? T(0.5) * (x + un[i][v]) + bs * (x - un[i][v]) : x;
    }
  }
  __syncthreads();
  // all 15 components at the points (ci, cj, k0 + m KT), and their viscous flux
  const int c2 = w % NF, ci = c2 % N1, cj = c2 / N1, k0 = w / NF;
  T g[PPT][15];
#pragma unroll
  for (int m = 0; m < PPT; ++m) {
    const int k = k0 + m * KT;
    if (k >= N1) break;
    const int pt = c2 + NF * k;
    T sJ[3][3];
    if constexpr (CUR) {
      const T iJ = cm_rjac<T, NSP>(cm, E, e, pt);
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        cm_srow<T, NSP>(cm, E, e, pt, d, sJ[d]);
#pragma unroll
        for (int j = 0; j < 3; ++j) sJ[d][j] *= iJ;
      }
    } else {
      T gc[3][3];
      hex_cols(G + el, NE, K.x[ci], K.x[cj], K.x[k], gc);
      const T iJ = rcp(det_cols(gc));
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        srow(gc, d, sJ[d]);
#pragma unroll
        for (int j = 0; j < 3; ++j) sJ[d][j] *= iJ;
      }
    }
    const int q0 = cj + N1 * k, q1 = NF * 2 + ci + N1 * k, q2 = NF * 4 + c2;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      T gt[3];
      gt[0] = K.cp[ci] * UH[((q0 + NF) * 5 + v) * NE + el] - K.cm[ci] * UH[(q0 * 5 + v) * NE + el];
      gt[1] = K.cp[cj] * UH[((q1 + NF) * 5 + v) * NE + el] - K.cm[cj] * UH[(q1 * 5 + v) * NE + el];
      gt[2] = K.cp[k] * UH[((q2 + NF) * 5 + v) * NE + el] - K.cm[k] * UH[(q2 * 5 + v) * NE + el];
#pragma unroll
      for (int b = 0; b < N1; ++b) {
        gt[0] += K.Dh[ci][b] * U[at(v, b + N1 * (cj + N1 * k))];
        gt[1] += K.Dh[cj][b] * U[at(v, ci + N1 * (b + N1 * k))];
        gt[2] += K.Dh[k][b] * U[at(v, c2 + NF * b)];
      }
#pragma unroll
      for (int j = 0; j < 3; ++j) g[m][v * 3 + j] = sJ[0][j] * gt[0] + sJ[1][j] * gt[1] + sJ[2][j] * gt[2];
    }
    T wv[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) wv[v] = U[at(v, pt)];
    const PointFluxNS<T, DEV> pf(wv, g[m], gamma, mu, pr, R);
    T* const vp = vf + (int64_t)w * 9 * E + e;       // (pt = w + m * W)
#pragma unroll
    for (int q = 0; q < 9; ++q) vp[(int64_t)(m * W * 9 + q) * E] = q < 6 ? pf.tau[q < 6 ? q : 0] : pf.qe[q < 6 ? 0 : q - 6];
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < PPT; ++m) {
    const int k = k0 + m * KT;
    if (k >= N1) break;
#pragma unroll
    for (int c = 0; c < 15; ++c) S[at(c, c2 + NF * k)] = g[m][c];
  }
  __syncthreads();
  T* const fw = fvn + (int64_t)w * 4 * E + e;
#pragma unroll
  for (int i = 0; i < EPT; ++i) {
    const int f = w + i * W;
    // stored only where the common flux will read it
    if (f >= 6 * NF) break;
    if (!need[i]) continue;
    int d, b0, st;
    line_of(f, d, b0, st);
    const bool sd = (f / NF) & 1;
    T gf[15], nv[3], fv[5];
#pragma unroll
    for (int c = 0; c < 15; ++c) {
      T x = 0;
#pragma unroll
      for (int a = 0; a < N1; ++a) x += (sd ? K.lp[a] : K.lm[a]) * S[at(c, b0 + a * st)];
      gf[c] = x;
    }
    if constexpr (CUR) {
      cm_fnrm<T, NSP>(cm, E, e, f, nv);
    } else {
      T xi[3], gc[3][3];
      end_xi(K, d, sd, f % N1, f % NF / N1, xi);
      hex_cols(G + el, NE, xi[0], xi[1], xi[2], gc);
      if (d == 0) srow(gc, 0, nv);
      else if (d == 1) srow(gc, 1, nv);
      else srow(gc, 2, nv);
    }
    const T mag = fsqrt(nv[0] * nv[0] + nv[1] * nv[1] + nv[2] * nv[2]);
    const T sl = fdiv(sd == ns[i].left ? T(1) : T(-1), mag);
    viscous<T, DEV>(own[i], gf, nv[0] * sl, nv[1] * sl, nv[2] * sl, gamma, mu, pr, R, fv);
#pragma unroll
    for (int v = 0; v < 4; ++v) fw[(int64_t)(i * W * 4 + v) * E] = fv[v + 1];
  }
}

// ---------------------------------------------------------------------------
// Navier--Stokes phase 2a: the LDG common flux at every flux-point pair (eq:comm_flux
// with the viscous terms): inviscid Riemann flux along the left side's normal, minus
// the switched viscous flux, plus the penalty.  Threads over (element, flux point),
// lanes over elements; the left side of each pair computes it once and writes
// +|S^T n~| times it into its own slot and the negative into the right side's slot
// (conservative by construction).  With a one-sided switch only the contributing
// side's f_v.n is read (stored by hex_grad in that side's slot).
template <typename T, bool DEV, int P, bool CUR = false>
__global__ void __launch_bounds__(256) hex_face_ns(const T* __restrict__ uf, const T* __restrict__ fvn,
                                                   const T* __restrict__ geo, const T* __restrict__ cm, Conn C,
                                                   T* __restrict__ fc, int64_t E,
                                                   int64_t n, HexK<T> K, T gamma, T beta, T tau,
                                                   int riemann, int side_mode, RefState<T> R) {
  constexpr int N1 = P + 1, NF = N1 * N1, NFP = 6 * NF, NSP = N1 * N1 * N1;
  const int64_t gtid = xcd_block() * 256 + threadIdx.x;
  const int64_t wave = gtid >> 6;
  const int lane = (int)(gtid & 63);
  const int64_t tile = wave / NFP;
  const int fp = (int)(wave % NFP);
  const int64_t e = tile * 64 + lane;
  if (e >= n) return;
  const int face = fp / NF, q = fp % NF, d = face / 2, sd = face % 2, t0 = q % N1, t1 = q / N1;
  const NbrSlot ns = nbr_slot<NF>(C, E, e, face, q);
  // each flux-point pair once: the left side computes it and writes both slots (decided
  // before the geometry is read: which side is left is a property of the face, so the
  // waves of the right sides' faces leave at once)
  if (!ns.left) return;
  T nv[3];
  if constexpr (CUR) {
    cm_fnrm<T, NSP>(cm, E, e, fp, nv);
  } else {
    T c[24];
#pragma unroll
    for (int g = 0; g < 24; ++g) c[g] = geo[(int64_t)g * E + e];
    T xi[3], g[3][3];
    end_xi(K, d, sd, t0, t1, xi);
    hex_cols(c, 1, xi[0], xi[1], xi[2], g);
    srow(g, d, nv);
  }
  const T mag = fsqrt(nv[0] * nv[0] + nv[1] * nv[1] + nv[2] * nv[2]);
  T own[5], un[5], uL[5], uR[5], nL[3], F[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    own[v] = uf[((int64_t)fp * 5 + v) * E + e];
    un[v] = uf[((int64_t)ns.fp * 5 + v) * E + ns.elem];
  }
  const T sg = sd ? T(1) : T(-1);
  const T sl = fdiv(ns.left ? sg : -sg, mag);
#pragma unroll
  for (int k = 0; k < 3; ++k) nL[k] = nv[k] * sl;
#pragma unroll
  for (int v = 0; v < 5; ++v) { uL[v] = ns.left ? own[v] : un[v]; uR[v] = ns.left ? un[v] : own[v]; }
  common_inviscid<T, DEV>(riemann, uL, uR, nL, gamma, R, F);
  const T wL = T(0.5) - beta, wR = T(0.5) + beta;
  const T w_own = ns.left ? wL : wR, w_nbr = ns.left ? wR : wL;
  T fvc[5] = {0, 0, 0, 0, 0};
#pragma unroll
  for (int side = 0; side < 2; ++side) {
    const T wgt = side == 0 ? w_own : w_nbr;
    if (side_mode != 0 && wgt == T(0)) continue;
    const int64_t gs = side == 0 ? (int64_t)fp : (int64_t)ns.fp;
    const int64_t ge = side == 0 ? e : ns.elem;
#pragma unroll
    for (int v = 0; v < 4; ++v) fvc[v + 1] += wgt * fvn[(gs * 4 + v) * E + ge];
  }
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    const T fn = mag * (F[v] - fvc[v] + tau * (uL[v] - uR[v]));
    fc[((int64_t)fp * 5 + v) * E + e] = fn;
    fc[((int64_t)ns.fp * 5 + v) * E + ns.elem] = -fn;
  }
}

// ---------------------------------------------------------------------------
// Navier--Stokes phase 2b: f = f_inv - f_v at the solution points and the
// corrected divergence with the common fluxes of hex_face_ns at the line ends.
// Each thread owns one column (i, j) of one element: it evaluates the transformed
// flux of all three directions at its column's points once (every state and viscous
// flux value is read once) into LDS, then gathers, for each of its points, the three
// line contractions through that point from LDS.
template <typename T, bool DEV, int P, int NE, bool CUR = false>
__global__ void __launch_bounds__(NE*(P + 1)*(P + 1)) hex_div_ns(
    const T* __restrict__ u, const T* __restrict__ vf, const T* __restrict__ fc, const T* __restrict__ geo,
    const T* __restrict__ cm, T* __restrict__ r, int64_t E, int64_t n, HexK<T> K, T gamma, RefState<T> R) {
  constexpr int N1 = P + 1, NSP = N1 * N1 * N1, NF = N1 * N1, NT = NE * N1 * N1;
  // f~ along xi_1 and xi_2 go through LDS ([d][v][pt][el]); along xi_3 the line is the
  // thread's own column, so f~_3 and its common fluxes stay in registers
  __shared__ T FT[2 * 5 * NSP * NE];
  __shared__ T G[CUR ? 1 : 24 * NE];
  const int el = threadIdx.x % NE, l = threadIdx.x / NE;
  const int64_t e0 = xcd_block() * NE, e = e0 + el;
  const int ci = l % N1, cj = l / N1;
  if constexpr (!CUR) stage_geo<T, NE, NT>(geo, E, e0, G);
  __syncthreads();
  const T gm1 = gamma - T(1);
  T* const rl = r + (int64_t)l * 5 * E + e;
  T iJ[N1], f3[N1][5];
  // the state and viscous flux of the column's next point are loaded while the current
  // point's fluxes are formed (two buffers), so a wave keeps loads in flight
  T ub[2][5], gb[2][9];
  const T *const ul = u + (int64_t)l * 5 * E + e, *const vl = vf + (int64_t)l * 9 * E + e;
  auto load_pt = [&](int k, T* uu, T* gg) {
#pragma unroll
    for (int v = 0; v < 5; ++v) uu[v] = ul[(int64_t)(k * NF * 5 + v) * E];
#pragma unroll
    for (int q = 0; q < 9; ++q) gg[q] = vl[(int64_t)(k * NF * 9 + q) * E];
  };
  load_pt(0, ub[0], gb[0]);
#pragma unroll
  for (int k = 0; k < N1; ++k) {
    const int pt = ci + N1 * (cj + N1 * k);
    if (k + 1 < N1) load_pt(k + 1, ub[(k + 1) & 1], gb[(k + 1) & 1]);
    const T* uu = ub[k & 1];
    const T* gg = gb[k & 1];
    T g[3][3];
    if constexpr (CUR) {
      iJ[k] = -cm_rjac<T, NSP>(cm, E, e, pt);
    } else {
      hex_cols(G + el, NE, K.x[ci], K.x[cj], K.x[k], g);
      iJ[k] = -rcp(det_cols(g));
    }
    const PointInv<T, DEV> pf(uu, gamma, R);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      T s[3], f[5];
      if constexpr (CUR) cm_srow<T, NSP>(cm, E, e, pt, d, s);
      else srow(g, d, s);
      pf.dir(s[0], s[1], s[2], f);
      minus_visc(gg, s[0], s[1], s[2], f);
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        if (d < 2) FT[((d * 5 + v) * NSP + pt) * NE + el] = f[v];
        else f3[k][v] = f[v];
      }
    }
  }
  // own column: common fluxes at its two xi_3 ends
  const int q2 = ci + N1 * cj;
  T F4[5], F5[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    F4[v] = fc[(((int64_t)4 * NF + q2) * 5 + v) * E + e];
    F5[v] = fc[(((int64_t)5 * NF + q2) * 5 + v) * E + e];
  }
  // common fluxes at the xi_1 and xi_2 ends of the lines through point k, all five
  // variables at once; the next point's are loaded while the current one is summed
  T fb[2][4][5];
  const T *const f0 = fc + (int64_t)cj * 5 * E + e, *const f1 = fc + (int64_t)ci * 5 * E + e;
  auto load_ends = [&](int k, T (&F)[4][5]) {
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const int64_t o = (int64_t)(N1 * k * 5 + v) * E;
      F[0][v] = f0[o];
      F[1][v] = f0[(int64_t)NF * 5 * E + o];
      F[2][v] = f1[(int64_t)NF * 10 * E + o];
      F[3][v] = f1[(int64_t)NF * 15 * E + o];
    }
  };
  load_ends(0, fb[0]);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N1; ++k) {
    const int pt = ci + N1 * (cj + N1 * k);
    if (k + 1 < N1) load_ends(k + 1, fb[(k + 1) & 1]);
    const T (&F)[4][5] = fb[k & 1];
    // line coordinates of this point in each direction: position a
    const int a0 = ci, a1 = cj;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      T acc = K.cp[k] * F5[v] + K.cm[k] * F4[v];
#pragma unroll
      for (int b = 0; b < N1; ++b) {
        acc += K.Dh[a0][b] * FT[((0 * 5 + v) * NSP + (b + N1 * (cj + N1 * k))) * NE + el];
        acc += K.Dh[a1][b] * FT[((1 * 5 + v) * NSP + (ci + N1 * (b + N1 * k))) * NE + el];
        acc += K.Dh[k][b] * f3[b][v];
      }
      acc += K.cp[a0] * F[1][v] + K.cm[a0] * F[0][v];
      acc += K.cp[a1] * F[3][v] + K.cm[a1] * F[2][v];
      if (e < n) rl[(int64_t)(k * NF * 5 + v) * E] = acc * iJ[k];
    }
  }
}

// Variant with all three directions' f~ in LDS, for FP64 at p = 4, where f~_3 of a
// whole column in registers does not fit beside the rest.  (In FP32 it does, at 166
// VGPRs: 3 waves per SIMD and 40 KB of LDS per 8 elements, three blocks per CU, where
// this variant's 60 KB allow two; bounding the register kernel to 128 VGPRs for a
// fourth block spills and is slower.)
template <typename T, bool DEV, int P, int NE, bool CUR = false>
__global__ void __launch_bounds__(NE*(P + 1)*(P + 1)) hex_div_ns_lds(
    const T* __restrict__ u, const T* __restrict__ vf, const T* __restrict__ fc, const T* __restrict__ geo,
    const T* __restrict__ cm, T* __restrict__ r, int64_t E, int64_t n, HexK<T> K, T gamma, RefState<T> R) {
  constexpr int N1 = P + 1, NSP = N1 * N1 * N1, NF = N1 * N1, NT = NE * N1 * N1;
  __shared__ T FT[3 * 5 * NSP * NE];       // [d][v][pt][el]
  __shared__ T G[CUR ? 1 : 24 * NE];
  const int el = threadIdx.x % NE, l = threadIdx.x / NE;
  const int64_t e0 = xcd_block() * NE, e = e0 + el;
  const int ci = l % N1, cj = l / N1;
  if constexpr (!CUR) stage_geo<T, NE, NT>(geo, E, e0, G);
  __syncthreads();
  const T gm1 = gamma - T(1);
  T* const rl = r + (int64_t)l * 5 * E + e;
  T iJ[N1];
  // as in hex_div_ns: the next point's state and viscous flux load while the current
  // point's fluxes are formed (this variant is held to 1-2 waves per SIMD by its LDS,
  // so registers are not what limits it)
  T ub[2][5], gb[2][9];
  const T *const ul = u + (int64_t)l * 5 * E + e, *const vl = vf + (int64_t)l * 9 * E + e;
  auto load_pt = [&](int k, T* uu, T* gg) {
#pragma unroll
    for (int v = 0; v < 5; ++v) uu[v] = ul[(int64_t)(k * NF * 5 + v) * E];
#pragma unroll
    for (int q = 0; q < 9; ++q) gg[q] = vl[(int64_t)(k * NF * 9 + q) * E];
  };
  load_pt(0, ub[0], gb[0]);
#pragma unroll
  for (int k = 0; k < N1; ++k) {
    const int pt = ci + N1 * (cj + N1 * k);
    if (k + 1 < N1) load_pt(k + 1, ub[(k + 1) & 1], gb[(k + 1) & 1]);
    const T* uu = ub[k & 1];
    const T* gg = gb[k & 1];
    T g[3][3];
    if constexpr (CUR) {
      iJ[k] = -cm_rjac<T, NSP>(cm, E, e, pt);
    } else {
      hex_cols(G + el, NE, K.x[ci], K.x[cj], K.x[k], g);
      iJ[k] = -rcp(det_cols(g));
    }
    const PointInv<T, DEV> pf(uu, gamma, R);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      T s[3], f[5];
      if constexpr (CUR) cm_srow<T, NSP>(cm, E, e, pt, d, s);
      else srow(g, d, s);
      pf.dir(s[0], s[1], s[2], f);
      minus_visc(gg, s[0], s[1], s[2], f);
#pragma unroll
      for (int v = 0; v < 5; ++v) FT[((d * 5 + v) * NSP + pt) * NE + el] = f[v];
    }
  }
  // common fluxes at the six line ends through point k (the xi_3 ends are the same
  // for every k), all variables at once, the next point's loaded during the sums
  const int q2 = ci + N1 * cj;
  T F4[5], F5[5], fb[2][4][5];
#pragma unroll
  for (int v = 0; v < 5; ++v) {
    F4[v] = fc[(((int64_t)4 * NF + q2) * 5 + v) * E + e];
    F5[v] = fc[(((int64_t)5 * NF + q2) * 5 + v) * E + e];
  }
  const T *const f0 = fc + (int64_t)cj * 5 * E + e, *const f1 = fc + (int64_t)ci * 5 * E + e;
  auto load_ends = [&](int k, T (&F)[4][5]) {
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const int64_t o = (int64_t)(N1 * k * 5 + v) * E;
      F[0][v] = f0[o];
      F[1][v] = f0[(int64_t)NF * 5 * E + o];
      F[2][v] = f1[(int64_t)NF * 10 * E + o];
      F[3][v] = f1[(int64_t)NF * 15 * E + o];
    }
  };
  load_ends(0, fb[0]);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N1; ++k) {
    const int pt = ci + N1 * (cj + N1 * k);
    if (k + 1 < N1) load_ends(k + 1, fb[(k + 1) & 1]);
    const T (&F)[4][5] = fb[k & 1];
    // line coordinates of this point in each direction: position a
    const int a0 = ci, a1 = cj, a2 = k;
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      T acc = T(0);
#pragma unroll
      for (int b = 0; b < N1; ++b) {
        acc += K.Dh[a0][b] * FT[((0 * 5 + v) * NSP + (b + N1 * (cj + N1 * k))) * NE + el];
        acc += K.Dh[a1][b] * FT[((1 * 5 + v) * NSP + (ci + N1 * (b + N1 * k))) * NE + el];
        acc += K.Dh[a2][b] * FT[((2 * 5 + v) * NSP + (ci + N1 * (cj + N1 * b))) * NE + el];
      }
      acc += K.cp[a0] * F[1][v] + K.cm[a0] * F[0][v];
      acc += K.cp[a1] * F[3][v] + K.cm[a1] * F[2][v];
      acc += K.cp[a2] * F5[v] + K.cm[a2] * F4[v];
      if (e < n) rl[(int64_t)(k * NF * 5 + v) * E] = acc * iJ[k];
    }
  }
}

}  // namespace frmi
