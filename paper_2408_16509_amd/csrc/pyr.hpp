// Order-4 pyramids with an affine base (Sec. "Mixed elements and domain decomposition":
// the transition element, supported with an affine base), meshes of pyramids only.
//
// The rational pyramid space has no tensor structure and its 55 x 55 operators are dense.
// The steps are those of the other element types: traces at the flux points (eq:disu), the
// common flux along the left side's normal (eq:comm_flux), the transformed flux S f and its
// normal trace, and the corrected divergence D_i f~_i + lift (F^C - f~perp) (eq:FRfinal),
// R = -div / J; Navier--Stokes adds the LDG gradient (corrected by the lifted jump of
// the common solution) and the viscous parts of both fluxes.
//
// Two forms.  The matrix-core form (py*_mma, below) takes 16 elements per block as the N
// dimension of the products; it covers Euler and Navier--Stokes with a one-sided LDG
// switch.  A two-sided switch takes pyr_grad and pyr_div: matrix-vector products with a
// thread per (element, solution point or flux point), elements fastest so that global
// loads and stores are coalesced, the elements' states, transformed fluxes, interface
// jumps and gradients staged in LDS, the operators shared through the caches.
//
// Layouts (element fastest): u, r [(pt*5 + v) E + e]; uf [(fp*5 + v) E + e];
// grad [(pt*15 + 3v + j) E + e]; gradf [(fp*15 + 3v + j) E + e]; geo rows 3i + j
// = S_ij (S = J G^{-1}), row 9 = J.  Operators of the two-sided form: It[j][fp] = l_j(x_fp),
// Dt[i][j][pt] = d l_j / d xi_i (x_pt), Lt[fp][pt] = lift[pt][fp].
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hex.hpp"
#include "tet.hpp"

namespace frmi {

constexpr int PY_NSP = 55, PY_NFP = 85;

template <typename T>
struct PyrK {
  int face_off[6];
  T nref[5][3];
};

template <typename T>
struct PyrOpsDev {
  const T* It;   // [55][85]
  const T* Dt;   // [3][55][55]
  const T* Lt;   // [85][55]
};

__device__ __forceinline__ int pyr_face_of(const int* off, int fp) {
  int f = 0;
#pragma unroll
  for (int k = 1; k < 5; ++k) f += fp >= off[k];
  return f;
}

// Partner of flux point fp of element e: neighbour element, its flux point, and whether
// e is the left side.
template <typename T>
__device__ __forceinline__ void pyr_partner(const Conn& C, const PyrK<T>& K, int64_t E, int64_t e, int fp, int& f,
                                            int64_t& en, int& fpn, bool& left) {
  f = pyr_face_of(K.face_off, fp);
  const int q = fp - K.face_off[f];
  const int info = C.nbr_info[(int64_t)f * E + e];
  en = C.nbr_elem[(int64_t)f * E + e];
  const int fb = info & 7, orient = (info >> 3) & 511;
  left = (info >> 12) & 1;
  fpn = K.face_off[fb] + C.perm[orient * C.perm_stride + q];
}

template <typename T>
__device__ __forceinline__ void pyr_metric(const T* __restrict__ geo, int64_t E, int64_t e, T S[9], T& J) {
#pragma unroll
  for (int k = 0; k < 9; ++k) S[k] = geo[(int64_t)k * E + e];
  J = geo[(int64_t)9 * E + e];
}

// Threads of a block work on NE elements at once, element fastest: thread t takes
// element t % NE and point (t / NE) + k (PY_NT / NE), so that each load or store of a
// point's values covers NE consecutive elements of a row (32 bytes: 8 FP32 or 4 FP64
// elements, which keeps the LDS tiles of the gradient kernel under 50 KB), and the
// tiles staged in LDS serve the dense products with the same mapping.
constexpr int PY_NT = 256;
template <typename T>
constexpr int py_ne() { return sizeof(T) == 8 ? 4 : 8; }
// threads per block of the divergence kernel: FP64 takes 128 (two solution
// points and three flux points per thread, as FP32 at 256: measured faster for FP64,
// slower for FP32); the gradient kernel takes PY_NT for both
template <typename T>
constexpr int py_nt() { return sizeof(T) == 8 ? 128 : PY_NT; }

// Navier--Stokes gradient (LDG): grad~u = D_i u + lift (n~_i (u^ - u_f)), u^ = (uL + uR)/2
// + beta (uL - uR); physical grad_j = sum_i S_ij / J grad~_i u.  Writes grad at the
// solution points and its traces at all flux points (a two-sided viscous common flux;
// one-sided switches take pyr_grad_mma).
template <typename T>
__global__ void __launch_bounds__(PY_NT) pyr_grad(const T* __restrict__ u, const T* __restrict__ uf,
                                                  const T* __restrict__ geo, Conn C, PyrOpsDev<T> O, PyrK<T> K,
                                                  T* __restrict__ grad, T* __restrict__ gradf, int64_t E, T beta) {
  constexpr int NE = py_ne<T>(), ROWS = PY_NT / NE;
  // one LDS tile per element: u (5 x 55) and the LDG jumps (5 x 85), and the physical
  // gradient (15 x 55).  FP32 overlays the gradient on the first two once every thread has
  // read them (26 KB per block instead of 49: four waves per SIMD instead of three); FP64,
  // held to three waves per SIMD by its registers, keeps them apart and saves the barrier.
  constexpr bool OVERLAY = sizeof(T) == 4;
  constexpr int GOFF = OVERLAY ? 0 : 5 * PY_NSP + 5 * PY_NFP;
  __shared__ T W_s[NE][GOFF + 15 * PY_NSP];
  static_assert(5 * PY_NSP + 5 * PY_NFP <= 15 * PY_NSP, "state and jumps fit in the gradient's tile");
  T* Wl = W_s[threadIdx.x % NE];
  auto U_at = [&](int v, int pt) -> T& { return Wl[v * PY_NSP + pt]; };
  auto JM_at = [&](int v, int fp) -> T& { return Wl[5 * PY_NSP + v * PY_NFP + fp]; };
  auto G_at = [&](int q, int pt) -> T& { return Wl[GOFF + q * PY_NSP + pt]; };
  const int el = threadIdx.x % NE, r0 = threadIdx.x / NE;
  const int64_t e = xcd_block() * NE + el;
  for (int pt = r0; pt < PY_NSP; pt += ROWS)
#pragma unroll
    for (int v = 0; v < 5; ++v) U_at(v, pt) = u[((int64_t)pt * 5 + v) * E + e];
  for (int fp = r0; fp < PY_NFP; fp += ROWS) {
    int f, fpn;
    int64_t en;
    bool left;
    pyr_partner(C, K, E, e, fp, f, en, fpn, left);
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      const T uo = uf[((int64_t)fp * 5 + v) * E + e];
      const T un = uf[((int64_t)fpn * 5 + v) * E + en];
      const T uL = left ? uo : un, uR = left ? un : uo;
      JM_at(v, fp) = T(0.5) * (uL + uR) + beta * (uL - uR) - uo;
    }
  }
  T S[9], J;
  pyr_metric(geo, E, e, S, J);
  const T iJ = rcp(J);
  __syncthreads();
  // each thread's solution points at once (every LDS value serves all of them)
  constexpr int NP = (PY_NSP + ROWS - 1) / ROWS, NF = (PY_NFP + ROWS - 1) / ROWS;
  int pts[NP];
#pragma unroll
  for (int k = 0; k < NP; ++k) pts[k] = min(r0 + k * ROWS, PY_NSP - 1);
  T gt[NP][3][5];
#pragma unroll
  for (int k = 0; k < NP; ++k)
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int v = 0; v < 5; ++v) gt[k][i][v] = 0;
  // unrolled by 5: the operator loads of five steps in flight together (measured: FP32
  // 0.84 -> 0.70 ms per launch; the same in the divergence was slower)
#pragma unroll 5
  for (int j = 0; j < PY_NSP; ++j) {
    T x[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) x[v] = U_at(v, j);
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const T d0 = O.Dt[(0 * PY_NSP + j) * PY_NSP + pts[k]];
      const T d1 = O.Dt[(1 * PY_NSP + j) * PY_NSP + pts[k]];
      const T d2 = O.Dt[(2 * PY_NSP + j) * PY_NSP + pts[k]];
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        gt[k][0][v] += d0 * x[v];
        gt[k][1][v] += d1 * x[v];
        gt[k][2][v] += d2 * x[v];
      }
    }
  }
  // the reference normal is constant over a face: lift the face's jumps, then scale
#pragma unroll 1
  for (int f = 0; f < 5; ++f) {
    T sf[NP][5];
#pragma unroll
    for (int k = 0; k < NP; ++k)
#pragma unroll
      for (int v = 0; v < 5; ++v) sf[k][v] = 0;
    for (int fp = K.face_off[f]; fp < K.face_off[f + 1]; ++fp) {
      T y[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) y[v] = JM_at(v, fp);
#pragma unroll
      for (int k = 0; k < NP; ++k) {
        const T l = O.Lt[fp * PY_NSP + pts[k]];
#pragma unroll
        for (int v = 0; v < 5; ++v) sf[k][v] += l * y[v];
      }
    }
    const T n0 = K.nref[f][0], n1 = K.nref[f][1], n2 = K.nref[f][2];
#pragma unroll
    for (int k = 0; k < NP; ++k)
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        gt[k][0][v] += n0 * sf[k][v];
        gt[k][1][v] += n1 * sf[k][v];
        gt[k][2][v] += n2 * sf[k][v];
      }
  }
  if constexpr (OVERLAY) __syncthreads();            // u and the jumps are read: the tile takes grad
#pragma unroll
  for (int k = 0; k < NP; ++k) {
    if (r0 + k * ROWS >= PY_NSP) continue;
    const int pt = pts[k];
#pragma unroll
    for (int v = 0; v < 5; ++v)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        const T g = (S[0 * 3 + j] * gt[k][0][v] + S[1 * 3 + j] * gt[k][1][v] + S[2 * 3 + j] * gt[k][2][v]) * iJ;
        G_at(v * 3 + j, pt) = g;
        grad[((int64_t)pt * 15 + v * 3 + j) * E + e] = g;
      }
  }
  __syncthreads();
  int fps[NF];
#pragma unroll
  for (int k = 0; k < NF; ++k) fps[k] = min(r0 + k * ROWS, PY_NFP - 1);
  T acc[NF][15];
#pragma unroll
  for (int k = 0; k < NF; ++k)
#pragma unroll
    for (int q = 0; q < 15; ++q) acc[k][q] = 0;
  for (int j = 0; j < PY_NSP; ++j) {
    T x[15];
#pragma unroll
    for (int q = 0; q < 15; ++q) x[q] = G_at(q, j);
#pragma unroll
    for (int k = 0; k < NF; ++k) {
      const T l = O.It[j * PY_NFP + fps[k]];
#pragma unroll
      for (int q = 0; q < 15; ++q) acc[k][q] += l * x[q];
    }
  }
#pragma unroll
  for (int k = 0; k < NF; ++k) {
    if (r0 + k * ROWS >= PY_NFP) continue;
#pragma unroll
    for (int q = 0; q < 15; ++q) gradf[((int64_t)fps[k] * 15 + q) * E + e] = acc[k][q];
  }
}

// Corrected divergence of the Navier--Stokes fluxes, R = -div / J.
template <typename T, bool DEV>
__global__ void __launch_bounds__(py_nt<T>()) pyr_div(const T* __restrict__ u, const T* __restrict__ uf,
                                                 const T* __restrict__ grad, const T* __restrict__ gradf,
                                                 const T* __restrict__ geo, Conn C, PyrOpsDev<T> O, PyrK<T> K,
                                                 T* __restrict__ r, int64_t E, T gamma, T mu, T pr, T beta, T tau,
                                                 int riemann, RefState<T> R) {
  constexpr int NE = py_ne<T>(), ROWS = py_nt<T>() / NE;
  __shared__ T F_s[NE][3][5][PY_NSP];
  __shared__ T JM_s[NE][5][PY_NFP];
  const int el = threadIdx.x % NE, r0 = threadIdx.x / NE;
  const int64_t e = xcd_block() * NE + el;
  const T gm1 = gamma - T(1);
  T S[9], J;
  pyr_metric(geo, E, e, S, J);
  // transformed flux f~_i = (S f)_i at the solution points
  for (int pt = r0; pt < PY_NSP; pt += ROWS) {
    T wv[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) wv[v] = u[((int64_t)pt * 5 + v) * E + e];
    T g[15];
#pragma unroll
    for (int k = 0; k < 15; ++k) g[k] = grad[((int64_t)pt * 15 + k) * E + e];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      T f[5], fv[5], vs, ps;
      Flux<T, DEV>::eval(wv, S[i * 3], S[i * 3 + 1], S[i * 3 + 2], gm1, R, f, vs, ps);
      viscous<T, DEV>(wv, g, S[i * 3], S[i * 3 + 1], S[i * 3 + 2], gamma, mu, pr, R, fv);
#pragma unroll
      for (int v = 0; v < 5; ++v) f[v] -= fv[v];
#pragma unroll
      for (int v = 0; v < 5; ++v) F_s[el][i][v][pt] = f[v];
    }
  }
  __syncthreads();
  // normal trace of f~ at each of the thread's flux points (every LDS value serves all)
  constexpr int NP = (PY_NSP + ROWS - 1) / ROWS, NF = (PY_NFP + ROWS - 1) / ROWS;
  int fps[NF];
  T nrk[NF][3];
#pragma unroll
  for (int k = 0; k < NF; ++k) {
    fps[k] = min(r0 + k * ROWS, PY_NFP - 1);
    const int f = pyr_face_of(K.face_off, fps[k]);
#pragma unroll
    for (int q = 0; q < 3; ++q) nrk[k][q] = K.nref[0][q];
#pragma unroll
    for (int ff = 1; ff < 5; ++ff)
      if (f == ff)
#pragma unroll
        for (int q = 0; q < 3; ++q) nrk[k][q] = K.nref[ff][q];
  }
  T fperp[NF][5];
#pragma unroll
  for (int k = 0; k < NF; ++k)
#pragma unroll
    for (int v = 0; v < 5; ++v) fperp[k][v] = 0;
  for (int j = 0; j < PY_NSP; ++j) {
    T x[3][5];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int v = 0; v < 5; ++v) x[i][v] = F_s[el][i][v][j];
#pragma unroll
    for (int k = 0; k < NF; ++k) {
      const T l = O.It[j * PY_NFP + fps[k]];
#pragma unroll
      for (int v = 0; v < 5; ++v) fperp[k][v] += l * (nrk[k][0] * x[0][v] + nrk[k][1] * x[1][v] + nrk[k][2] * x[2][v]);
    }
  }
  // common flux along the left side's normal, minus the normal trace
#pragma unroll
  for (int k = 0; k < NF; ++k) {
    if (r0 + k * ROWS >= PY_NFP) continue;
    const int fp = fps[k];
    int f, fpn;
    int64_t en;
    bool left;
    pyr_partner(C, K, E, e, fp, f, en, fpn, left);
    const T* nr = nrk[k];
    T sn[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) sn[j] = S[0 * 3 + j] * nr[0] + S[1 * 3 + j] * nr[1] + S[2 * 3 + j] * nr[2];
    const T mag = fsqrt(sn[0] * sn[0] + sn[1] * sn[1] + sn[2] * sn[2]);
    const T im = rcp(mag);
    const T sg = left ? T(1) : T(-1);
    const T nL[3] = {sg * sn[0] * im, sg * sn[1] * im, sg * sn[2] * im};
    T uo[5], un[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) {
      uo[v] = uf[((int64_t)fp * 5 + v) * E + e];
      un[v] = uf[((int64_t)fpn * 5 + v) * E + en];
    }
    T uL[5], uR[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) { uL[v] = left ? uo[v] : un[v]; uR[v] = left ? un[v] : uo[v]; }
    T Fc[5];
    common_inviscid<T, DEV>(riemann, uL, uR, nL, gamma, R, Fc);
    // viscous common flux (1/2 - beta) f_v(L) + (1/2 + beta) f_v(R)
    const T wL = T(0.5) - beta, wR = T(0.5) + beta;
    T fvc[5] = {0, 0, 0, 0, 0};
#pragma unroll
    for (int side = 0; side < 2; ++side) {
      const bool is_left = side == 0;
      const T wgt = is_left ? wL : wR;
      const bool own = is_left == left;
      const int64_t gs = own ? (int64_t)fp : (int64_t)fpn, ge = own ? e : en;
      T g[15], fv[5];
#pragma unroll
      for (int q = 0; q < 15; ++q) g[q] = gradf[(gs * 15 + q) * E + ge];
      viscous<T, DEV>(is_left ? uL : uR, g, nL[0], nL[1], nL[2], gamma, mu, pr, R, fv);
#pragma unroll
      for (int v = 0; v < 5; ++v) fvc[v] += wgt * fv[v];
    }
#pragma unroll
    for (int v = 0; v < 5; ++v) Fc[v] += tau * (uL[v] - uR[v]) - fvc[v];
#pragma unroll
    for (int v = 0; v < 5; ++v) JM_s[el][v][fp] = mag * sg * Fc[v] - fperp[k][v];
  }
  __syncthreads();
  // corrected divergence at each of the thread's solution points
  int pts[NP];
#pragma unroll
  for (int k = 0; k < NP; ++k) pts[k] = min(r0 + k * ROWS, PY_NSP - 1);
  T div[NP][5];
#pragma unroll
  for (int k = 0; k < NP; ++k)
#pragma unroll
    for (int v = 0; v < 5; ++v) div[k][v] = 0;
  for (int j = 0; j < PY_NSP; ++j) {
    T x[3][5];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int v = 0; v < 5; ++v) x[i][v] = F_s[el][i][v][j];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const T d0 = O.Dt[(0 * PY_NSP + j) * PY_NSP + pts[k]];
      const T d1 = O.Dt[(1 * PY_NSP + j) * PY_NSP + pts[k]];
      const T d2 = O.Dt[(2 * PY_NSP + j) * PY_NSP + pts[k]];
#pragma unroll
      for (int v = 0; v < 5; ++v) div[k][v] += d0 * x[0][v] + d1 * x[1][v] + d2 * x[2][v];
    }
  }
  for (int fp = 0; fp < PY_NFP; ++fp) {
    T y[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) y[v] = JM_s[el][v][fp];
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const T l = O.Lt[fp * PY_NSP + pts[k]];
#pragma unroll
      for (int v = 0; v < 5; ++v) div[k][v] += l * y[v];
    }
  }
  const T iJ = -rcp(J);
#pragma unroll
  for (int k = 0; k < NP; ++k)
    if (r0 + k * ROWS < PY_NSP)
#pragma unroll
      for (int v = 0; v < 5; ++v) r[((int64_t)pts[k] * 5 + v) * E + e] = div[k][v] * iJ;
}

// ---------------------------------------------------------------------------
// The same steps on the matrix cores: a block takes 16 elements, the N dimension of the
// 16x16x4 products (Mma16), so each operator value a wave loads serves the products of
// all variables.  Rows: solution points padded to 4 tiles of 16; flux points in 6 tiles of
// one face each (the base's 25 points in tiles 0 and 1, triangle f in tile f + 1), so a
// tile's reference normal, sides and partner element are one value per element.  K rows
// of the lift: the base's 25 points padded to 28, then 16 per triangle.  The row past the
// 55 points reads row 54 against a zero operator column.
// With a one-sided LDG switch (beta = +-1/2) the gradient kernel forms the common flux of
// every flux-point pair once, on the side whose gradient it takes, where the gradient's
// traces are in registers (5 values stored instead of 15), and stores S_i . f_v at the
// solution points (12 instead of 15); the divergence reads both.  A two-sided switch takes
// pyr_grad and pyr_div.
constexpr int PYM_NE = 16, PYM_NT = 256, PYM_KP = 56, PYM_M = 64, PYM_FT = 6, PYM_FM = 16 * PYM_FT, PYM_KL = 28 + 4 * 16;

// Flux point of row `row` of flux tile ft (-1: padding), its face, its K row in the lift.
__host__ __device__ constexpr int pym_fp(int ft, int row) {
  return ft == 0 ? row : (ft == 1 ? (row < 9 ? 16 + row : -1) : (row < 15 ? 25 + 15 * (ft - 2) + row : -1));
}
__host__ __device__ constexpr int pym_face(int ft) { return ft < 2 ? 0 : ft - 1; }
__host__ __device__ constexpr int pym_off(int f) { return f == 0 ? 0 : 25 + 15 * (f - 1); }
__host__ __device__ constexpr int pym_krow0(int f) { return f == 0 ? 0 : 28 + 16 * (f - 1); }

// Operators, transposed and zero-padded: It[56][96] (columns: flux tiles), Dt[3][56][64],
// Lt[92][64].
template <typename T>
struct PymOps {
  const T *It, *Dt, *Lt;
};

// Tile-by-tile layouts of what the gradient kernel leaves for the divergence: rows of one
// 16-element tile contiguous (the tetrahedra's tet_fv_index / tet_fc_index).
__device__ __forceinline__ int64_t pym_fv_index(int64_t e0, int row, int el) {
  return e0 * (12 * PY_NSP) + (int64_t)row * PYM_NE + el;
}
__device__ __forceinline__ int64_t pym_fc_index(int64_t e, int row) {
  return (e / PYM_NE) * (PYM_NE * 5 * PY_NFP) + (int64_t)row * PYM_NE + e % PYM_NE;
}

template <typename T>
__global__ void __launch_bounds__(64 * PYM_FT) pyr_trace_mma(const T* __restrict__ u, T* __restrict__ uf, int64_t E,
                                                             PymOps<T> O) {
  using M = Mma16<T>;
  constexpr int NE = PYM_NE, NT = 64 * PYM_FT;
  __shared__ T U[5 * PY_NSP * NE];
  const int t = threadIdx.x, w = t / 64, lane = t % 64, kr = lane / 16, col = lane % 16;
  const int64_t e0 = xcd_block() * NE;
#pragma unroll
  for (int j = 0; j < (5 * PY_NSP * NE + NT - 1) / NT; ++j) {
    const int i = t + j * NT;
    if (i < 5 * PY_NSP * NE) U[i] = u[(int64_t)(i / NE) * E + e0 + i % NE];
  }
  __syncthreads();
  typename M::V acc[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) acc[v] = typename M::V{0, 0, 0, 0};
#pragma unroll 7
  for (int k0 = 0; k0 < PYM_KP; k0 += 4) {
    const int k = min(k0 + kr, PY_NSP - 1);
    const T a = O.It[(k0 + kr) * PYM_FM + 16 * w + col];
#pragma unroll
    for (int v = 0; v < 5; ++v) acc[v] = M::run(a, U[(k * 5 + v) * NE + col], acc[v]);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int fp = pym_fp(w, M::row(lane, q));
    if (fp < 0) continue;
#pragma unroll
    for (int v = 0; v < 5; ++v) uf[((int64_t)fp * 5 + v) * E + e0 + col] = acc[v][q];
  }
}

// Navier--Stokes gradient with a one-sided switch (side_mode = sign of beta), the
// transformed viscous flux at the points and the common flux of the pairs this side forms.
template <typename T, bool DEV>
__global__ void __launch_bounds__(PYM_NT) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 3 : 1)))
pyr_grad_mma(const T* __restrict__ u, const T* __restrict__ uf,
                                                       const T* __restrict__ geo, Conn C, PymOps<T> O, PyrK<T> K,
                                                       T* __restrict__ fv, T* __restrict__ fc, int64_t E,
                                                       int side_mode, T gamma, T mu, T pr, T tau, int riemann,
                                                       RefState<T> R) {
  using M = Mma16<T>;
  constexpr int NE = PYM_NE, NT = PYM_NT;
  // u [pt*5 + v][el] and the jumps [K row*5 + v][el]; then the physical gradient
  // [pt*15 + c][el] over both
  constexpr int JO = 5 * PY_NSP * NE;
  constexpr int LEN = JO + 5 * PYM_KL * NE > 15 * PY_NSP * NE ? JO + 5 * PYM_KL * NE : 15 * PY_NSP * NE;
  __shared__ T W[LEN];
  __shared__ T SJ[10 * NE];
  const int t = threadIdx.x, w = t / 64, lane = t % 64, kr = lane / 16, col = lane % 16;
  const int64_t e0 = xcd_block() * NE, e = e0 + col;
  // the gather in three rounds of loads (connectivity and states, point permutation, traces),
  // each issued for all of the thread's items before any is used: with one item after the
  // other a block spent 9.7 of its 36 us here
  constexpr int NU = (5 * PY_NSP * NE + NT - 1) / NT, NJ = (PY_NFP * NE + NT - 1) / NT;
  const int tel = t % NE, tr = t / NE;
  static_assert(NT % NE == 0, "rows per pass");
  int inf[NJ], nel[NJ], fac[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int fp = min(tr + j * (NT / NE), PY_NFP - 1);
    fac[j] = fp < 25 ? 0 : 1 + (fp - 25) / 15;
    inf[j] = C.nbr_info[(int64_t)fac[j] * E + e0 + tel];
    nel[j] = C.nbr_elem[(int64_t)fac[j] * E + e0 + tel];
  }
  T ur[NU];
#pragma unroll
  for (int j = 0; j < NU; ++j)
    ur[j] = u[(int64_t)min(tr + j * (NT / NE), 5 * PY_NSP - 1) * E + e0 + tel];
  for (int i = t; i < 10 * NE; i += NT) SJ[i] = geo[(int64_t)(i / NE) * E + e0 + i % NE];
  int fpn[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int fp = min(tr + j * (NT / NE), PY_NFP - 1);
    fpn[j] = pym_off(inf[j] & 7) + C.perm[((inf[j] >> 3) & 511) * C.perm_stride + fp - pym_off(fac[j])];
  }
  // jump of the common solution: the partner's trace minus the own one where the switch
  // names the partner's side, else zero
  T jm[NJ][5];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int fp = min(tr + j * (NT / NE), PY_NFP - 1);
    const bool formed = (((inf[j] >> 12) & 1) != 0) != (side_mode > 0);
    // not formed: both addresses the own trace, a zero jump from one line
    const int64_t o = (int64_t)fp * 5 * E + e0 + tel, p = formed ? (int64_t)fpn[j] * 5 * E + nel[j] : o;
#pragma unroll
    for (int v = 0; v < 5; ++v) jm[j][v] = uf[p + v * E] - uf[o + v * E];
    if (!formed) {
#pragma unroll
      for (int v = 0; v < 5; ++v) jm[j][v] = T(0);     // also where a trace is not finite
    }
  }
#pragma unroll
  for (int j = 0; j < NU; ++j) {
    const int i = t + j * NT;
    if (i < 5 * PY_NSP * NE) W[i] = ur[j];
  }
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int fp = tr + j * (NT / NE);
    if (fp >= PY_NFP) continue;
#pragma unroll
    for (int v = 0; v < 5; ++v)
      W[JO + ((pym_krow0(fac[j]) + fp - pym_off(fac[j])) * 5 + v) * NE + tel] = jm[j][v];
  }
  for (int i = t; i < 7 * 5 * NE; i += NT) {           // padding rows 25, 26, 27 and one per triangle
    const int r = i / (5 * NE);
    W[JO + (r < 3 ? 25 + r : 28 + 16 * (r - 3) + 15) * 5 * NE + i % (5 * NE)] = T(0);
  }
  __syncthreads();
  // reference gradient of point tile w, all variables (FP64: the lift's operator values load
  // during the derivatives; FP32 has no registers for them at three waves per SIMD)
  constexpr bool kAhead = sizeof(T) == 8;
  T la[kAhead ? PYM_KL / 4 : 1];
  if constexpr (kAhead) {
#pragma unroll
    for (int s = 0; s < PYM_KL / 4; ++s) la[s] = O.Lt[(4 * s + kr) * PYM_M + 16 * w + col];
  }
  typename M::V gt[3][5];
#pragma unroll
  for (int i = 0; i < 3; ++i)
#pragma unroll
    for (int v = 0; v < 5; ++v) gt[i][v] = typename M::V{0, 0, 0, 0};
#pragma unroll 7
  for (int k0 = 0; k0 < PYM_KP; k0 += 4) {
    const int k = min(k0 + kr, PY_NSP - 1);
    T b[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) b[v] = W[(k * 5 + v) * NE + col];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      const T a = O.Dt[(i * PYM_KP + k0 + kr) * PYM_M + 16 * w + col];
#pragma unroll
      for (int v = 0; v < 5; ++v) gt[i][v] = M::run(a, b[v], gt[i][v]);
    }
  }
  // the reference normal is constant over a face: lift the face's jumps, then scale
#pragma unroll
  for (int f = 0; f < 5; ++f) {
    typename M::V sf[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) sf[v] = typename M::V{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < (f == 0 ? 7 : 4); ++s) {
      const int k = pym_krow0(f) + 4 * s + kr;
      const T a = kAhead ? la[kAhead ? pym_krow0(f) / 4 + s : 0] : O.Lt[k * PYM_M + 16 * w + col];
#pragma unroll
      for (int v = 0; v < 5; ++v) sf[v] = M::run(a, W[JO + (k * 5 + v) * NE + col], sf[v]);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int v = 0; v < 5; ++v) gt[i][v] += K.nref[f][i] * sf[v];
  }
  T own[4][5];
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int v = 0; v < 5; ++v) own[q][v] = W[(min(16 * w + M::row(lane, q), PY_NSP - 1) * 5 + v) * NE + col];
  __syncthreads();                       // u and the jumps are read: the buffer takes the gradient
  T S[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) S[k] = SJ[k * NE + col];
  const T iJ = rcp(SJ[9 * NE + col]);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int pt = 16 * w + M::row(lane, q);
    if (pt >= PY_NSP) continue;
    T gp[15];
#pragma unroll
    for (int v = 0; v < 5; ++v)
#pragma unroll
      for (int j = 0; j < 3; ++j) {
        gp[v * 3 + j] = (S[j] * gt[0][v][q] + S[3 + j] * gt[1][v][q] + S[6 + j] * gt[2][v][q]) * iJ;
        W[(pt * 15 + v * 3 + j) * NE + col] = gp[v * 3 + j];
      }
    const PointFluxNS<T, DEV> pf(own[q], gp, gamma, mu, pr, R);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      T f4[4];
      pf.visc(S[3 * i], S[3 * i + 1], S[3 * i + 2], f4);
#pragma unroll
      for (int c = 0; c < 4; ++c) fv[pym_fv_index(e0, pt * 12 + i * 4 + c, col)] = f4[c];
    }
  }
  __syncthreads();
  // traces of the gradient and the common flux, one flux tile (face) after the other
  for (int ft = w; ft < PYM_FT; ft += NT / 64) {
    const int f = pym_face(ft);
    const int info = C.nbr_info[(int64_t)f * E + e];
    const int64_t en = C.nbr_elem[(int64_t)f * E + e];
    const bool left = (info >> 12) & 1, formed = left != (side_mode > 0);
    if (!__any(formed)) continue;
    // both sides' traces: FP64 loads them during the products, FP32 after (padding rows keep
    // in-bounds addresses)
    const int fb = info & 7, orient = (info >> 3) & 511;
    int fps[4], fpn[4];
    T uo[4][5], un[4][5];
    auto load_traces = [&] {
#pragma unroll
      for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          uo[q][v] = uf[((int64_t)fps[q] * 5 + v) * E + e];
          un[q][v] = uf[((int64_t)fpn[q] * 5 + v) * E + en];
        }
    };
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int fp = pym_fp(ft, M::row(lane, q));
      fps[q] = fp < 0 ? pym_off(f) : fp;
      fpn[q] = pym_off(fb) + C.perm[orient * C.perm_stride + fps[q] - pym_off(f)];
    }
    if constexpr (kAhead) load_traces();
    typename M::V gf[15];
#pragma unroll
    for (int c = 0; c < 15; ++c) gf[c] = typename M::V{0, 0, 0, 0};
#pragma unroll (sizeof(T) == 8 ? 14 : 7)
    for (int k0 = 0; k0 < PYM_KP; k0 += 4) {
      const int k = min(k0 + kr, PY_NSP - 1);
      const T a = O.It[(k0 + kr) * PYM_FM + 16 * ft + col];
#pragma unroll
      for (int c = 0; c < 15; ++c) gf[c] = M::run(a, W[(k * 15 + c) * NE + col], gf[c]);
    }
    if constexpr (!kAhead) load_traces();
    if (!formed) continue;
    T nv[3], nL[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) nv[j] = K.nref[f][0] * S[j] + K.nref[f][1] * S[3 + j] + K.nref[f][2] * S[6 + j];
    const T sl = fdiv(left ? T(1) : T(-1), fsqrt(nv[0] * nv[0] + nv[1] * nv[1] + nv[2] * nv[2]));
#pragma unroll
    for (int j = 0; j < 3; ++j) nL[j] = nv[j] * sl;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (pym_fp(ft, M::row(lane, q)) < 0) continue;
      T uL[5], uR[5], g[15], F[5], f5[5];
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        uL[v] = left ? uo[q][v] : un[q][v];
        uR[v] = left ? un[q][v] : uo[q][v];
      }
#pragma unroll
      for (int c = 0; c < 15; ++c) g[c] = gf[c][q];
      common_inviscid<T, DEV>(riemann, uL, uR, nL, gamma, R, F);
      viscous<T, DEV>(uo[q], g, nL[0], nL[1], nL[2], gamma, mu, pr, R, f5);
#pragma unroll
      for (int v = 0; v < 5; ++v) fc[pym_fc_index(e, fps[q] * 5 + v)] = F[v] - f5[v] + tau * (uL[v] - uR[v]);
    }
  }
}

// Corrected divergence (Euler; Navier--Stokes with what pyr_grad_mma left), R = -div / J.
template <typename T, bool DEV, bool NS>
__global__ void __launch_bounds__(PYM_NT) pyr_div_mma(const T* __restrict__ u, const T* __restrict__ uf,
                                                      const T* __restrict__ fv, const T* __restrict__ fc,
                                                      const T* __restrict__ geo, Conn C, PymOps<T> O, PyrK<T> K,
                                                      T* __restrict__ r, int64_t E, int64_t n, T gamma, int side_mode,
                                                      int riemann, RefState<T> R) {
  using M = Mma16<T>;
  constexpr int NE = PYM_NE, NT = PYM_NT, NTW = NT / 64, NFT = (PYM_FT + NTW - 1) / NTW;
  // f~ [(55 i + pt)*5 + v][el]; then the jumps of the normal flux [K row*5 + v][el] over it
  __shared__ T W[15 * PY_NSP * NE];
  static_assert(5 * PYM_KL <= 15 * PY_NSP, "jumps fit");
  __shared__ T SJ[10 * NE];
  const int t = threadIdx.x, w = t / 64, lane = t % 64, kr = lane / 16, col = lane % 16;
  const int64_t e0 = xcd_block() * NE, e = e0 + col;
  // connectivity of this lane's flux tiles, and the common fluxes formed by the gradient
  // kernel, read before anything waits
  int info[NFT];
  int64_t en[NFT];
#pragma unroll
  for (int a = 0; a < NFT; ++a) {
    const int ft = min(w + a * NTW, PYM_FT - 1);
    info[a] = C.nbr_info[(int64_t)pym_face(ft) * E + e];
    en[a] = C.nbr_elem[(int64_t)pym_face(ft) * E + e];
  }
  for (int i = t; i < 10 * NE; i += NT) SJ[i] = geo[(int64_t)(i / NE) * E + e0 + i % NE];
  __syncthreads();
#pragma unroll
  for (int j = 0; j < (PY_NSP * NE + NT - 1) / NT; ++j) {
    const int it = t + j * NT;
    if (it >= PY_NSP * NE) continue;
    const int el = it % NE, pt = it / NE;
    T wv[5], f4[12];
#pragma unroll
    for (int v = 0; v < 5; ++v) wv[v] = u[((int64_t)pt * 5 + v) * E + e0 + el];
    if constexpr (NS) {
#pragma unroll
      for (int k = 0; k < 12; ++k) f4[k] = fv[pym_fv_index(e0, pt * 12 + k, el)];
    }
    const PointInv<T, DEV> pin(wv, gamma, R);
#pragma unroll
    for (int i = 0; i < 3; ++i) {
      T f[5];
      pin.dir(SJ[(3 * i) * NE + el], SJ[(3 * i + 1) * NE + el], SJ[(3 * i + 2) * NE + el], f);
      if constexpr (NS) {
#pragma unroll
        for (int c = 0; c < 4; ++c) f[1 + c] -= f4[4 * i + c];
      }
#pragma unroll
      for (int v = 0; v < 5; ++v) W[((i * PY_NSP + pt) * 5 + v) * NE + el] = f[v];
    }
  }
  __syncthreads();
  T S[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) S[k] = SJ[k * NE + col];
  // the jumps F^C - n~ . (I f~) of this wave's flux tiles
  T jm[NFT][4][5];
#pragma unroll
  for (int a = 0; a < NFT; ++a) {
    const int ft = w + a * NTW;
    if (ft >= PYM_FT) continue;
    const int f = pym_face(ft);
    const bool left = (info[a] >> 12) & 1;
    const int fb = info[a] & 7, orient = (info[a] >> 3) & 511;
    T nv[3];
#pragma unroll
    for (int j = 0; j < 3; ++j) nv[j] = K.nref[f][0] * S[j] + K.nref[f][1] * S[3 + j] + K.nref[f][2] * S[6 + j];
    const T mag = fsqrt(nv[0] * nv[0] + nv[1] * nv[1] + nv[2] * nv[2]);
    const T fs = left ? mag : -mag;
    // common fluxes (NS: loads ahead of the products)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int fp = pym_fp(ft, M::row(lane, q));
      const int fo = fp < 0 ? pym_off(f) : fp;         // padding rows keep in-bounds addresses
      const int fpn = pym_off(fb) + C.perm[orient * C.perm_stride + fo - pym_off(f)];
      if constexpr (NS) {
        const bool mine = left != (side_mode > 0);
        const int64_t at = pym_fc_index(mine ? e : en[a], (mine ? fo : fpn) * 5);
#pragma unroll
        for (int v = 0; v < 5; ++v) jm[a][q][v] = fc[at + v * NE] * fs;
      } else {
        T uL[5], uR[5], nL[3], F[5];
        const T sl = fdiv(left ? T(1) : T(-1), mag);
#pragma unroll
        for (int j = 0; j < 3; ++j) nL[j] = nv[j] * sl;
#pragma unroll
        for (int v = 0; v < 5; ++v) {
          const T uo = uf[((int64_t)fo * 5 + v) * E + e], un = uf[((int64_t)fpn * 5 + v) * E + en[a]];
          uL[v] = left ? uo : un;
          uR[v] = left ? un : uo;
        }
        common_inviscid<T, DEV>(riemann, uL, uR, nL, gamma, R, F);
#pragma unroll
        for (int v = 0; v < 5; ++v) jm[a][q][v] = F[v] * fs;
      }
    }
    // normal trace of f~ (base: -f~_3)
    typename M::V acc[5];
#pragma unroll
    for (int v = 0; v < 5; ++v) acc[v] = typename M::V{0, 0, 0, 0};
    const int hd = f == 0 ? 2 : (f % 2 ? 1 : 0);       // the horizontal axis of the face's normal
    const T nh = f == 0 ? T(0) : K.nref[f][hd], nz = K.nref[f][2];
#pragma unroll
    for (int k0 = 0; k0 < PYM_KP; k0 += 4) {
      const int k = min(k0 + kr, PY_NSP - 1);
      const T o = O.It[(k0 + kr) * PYM_FM + 16 * ft + col];
#pragma unroll
      for (int v = 0; v < 5; ++v) {
        const T b = nh * W[((hd * PY_NSP + k) * 5 + v) * NE + col] + nz * W[((2 * PY_NSP + k) * 5 + v) * NE + col];
        acc[v] = M::run(o, b, acc[v]);
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int v = 0; v < 5; ++v) jm[a][q][v] = pym_fp(ft, M::row(lane, q)) < 0 ? T(0) : jm[a][q][v] - acc[v][q];
  }
  // D_i f~_i of point tile w
  typename M::V acc[5];
#pragma unroll
  for (int v = 0; v < 5; ++v) acc[v] = typename M::V{0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < 3; ++i) {
#pragma unroll 14
    for (int k0 = 0; k0 < PYM_KP; k0 += 4) {
      const int k = i * PY_NSP + min(k0 + kr, PY_NSP - 1);
      const T a = O.Dt[(i * PYM_KP + k0 + kr) * PYM_M + 16 * w + col];
#pragma unroll
      for (int v = 0; v < 5; ++v) acc[v] = M::run(a, W[(k * 5 + v) * NE + col], acc[v]);
    }
  }
  __syncthreads();                       // f~ is read: the buffer takes the jumps
#pragma unroll
  for (int a = 0; a < NFT; ++a) {
    const int ft = w + a * NTW;
    if (ft >= PYM_FT) continue;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int row = M::row(lane, q);
      if (ft == 1 && row >= 12) continue;              // the base's K rows end at 27
      const int k = (ft < 2 ? 16 * ft : 28 + 16 * (ft - 2)) + row;
#pragma unroll
      for (int v = 0; v < 5; ++v) W[(k * 5 + v) * NE + col] = jm[a][q][v];
    }
  }
  __syncthreads();
#pragma unroll
  for (int k0 = 0; k0 < PYM_KL; k0 += 4) {
    const T a = O.Lt[(k0 + kr) * PYM_M + 16 * w + col];
#pragma unroll
    for (int v = 0; v < 5; ++v) acc[v] = M::run(a, W[((k0 + kr) * 5 + v) * NE + col], acc[v]);
  }
  const T iJ = -rcp(SJ[9 * NE + col]);
  if (e >= n) return;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int pt = 16 * w + M::row(lane, q);
    if (pt >= PY_NSP) continue;
#pragma unroll
    for (int v = 0; v < 5; ++v) r[((int64_t)pt * 5 + v) * E + e] = acc[v][q] * iJ;
  }
}

}  // namespace frmi
