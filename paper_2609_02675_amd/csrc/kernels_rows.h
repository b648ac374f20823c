// kernels_rows.h -- the body iteration of joint scenes with a quad of lanes per
// body: lane k of the quad holds row k of the body's affine frame and its
// position component k (the fourth lane repeats the third, and is not read).
//
// Everything in an iteration but the rotation is separate by rows: component k of
// a bond point, a bond vector and its force, and row k of the block solve need
// nothing of the other rows.  The rotation's Newton steps take the other two rows
// (a row's cofactors are their cross product) and row 0's determinant from the
// quad by data-parallel primitives.  So a lane issues about a third of a body's
// instructions, and a body's chain of dependent ones, which is what a scene or
// batch with few waves waits for, shrinks with it.  With many waves the quad's
// idle fourth lane and its exchanges cost issue slots that one lane per body
// saves, so large batches keep kernels_tile.h.
//
//   k_resident_rows  steps of a small plain scene (k_resident_joints' arithmetic)
//   k_resident_ends  the same for bonds of any kind, in two phases
//   k_tile_rows      steps of a batch's tiles (k_tile_step's arithmetic)
//
// Each entry is formed by the operations of those kernels in their order, so the
// bits are theirs.
//
// Measured per step (K = 20), against one lane per body: eight-body chain 0.025 ->
// 0.011 ms (FP64 0.036 -> 0.018), chain of 60 0.026 -> 0.012, of 200 0.027 ->
// 0.020, 11 x 11 net of springs in FP64 0.068 -> 0.045; a batch of 64 chains 0.021
// -> 0.015 (FP64 0.028 -> 0.023).  An iteration is then about 1,200 cycles for 170
// instructions: LDS round trips, the exchanges and the reciprocals of three
// Newton steps, one after another.
#pragma once

#include "common.h"
#include "device_math.h"
#include "kernels_flat.h"
#include "kernels_resident.h"
#include "kernels_step.h"
#include "kernels_tile.h"

namespace pabd {

// x of lane J of this lane's quad
template <int J, typename U>
__device__ __forceinline__ U quad_from(U x) {
  return lane_of<J * 0x55>(x);
}

// component k of three, row k of a matrix; the fourth lane takes the third's (selects
// between values, so that no array needs memory to be indexed)
template <typename T>
__device__ __forceinline__ T pick(T x0, T x1, T x2, int k) {
  const T y = k == 1 ? x1 : x2;
  return k == 0 ? x0 : y;
}
template <typename T>
__device__ __forceinline__ void take_row(const T* A, int k, T* x) {
#pragma unroll
  for (int c = 0; c < 3; ++c) x[c] = pick(A[c], A[3 + c], A[6 + c], k);
}

// a body's record from its quad's rows: position words as given, hi apart
template <typename T>
__device__ __forceinline__ void gather_body(T hi, T lo, const T* x, T* q) {
  q[0] = quad_from<0>(hi);
  q[1] = quad_from<1>(hi);
  q[2] = quad_from<2>(hi);
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    q[3 + c] = quad_from<0>(x[c]);
    q[6 + c] = quad_from<1>(x[c]);
    q[9 + c] = quad_from<2>(x[c]);
  }
  if constexpr (sizeof(T) == 4) {
    q[12] = quad_from<0>(lo);
    q[13] = quad_from<1>(lo);
    q[14] = quad_from<2>(lo);
  }
}

// row k of the cofactor matrix of the quad's matrix (own row x); returns its
// determinant, row 0's, in every lane
template <typename T>
__device__ __forceinline__ T cofactor_row(const T* x, T* C) {
  T p[3], s[3];  // the rows after the own one, cyclically
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    p[c] = lane_of<0xC9>(x[c]);  // quad_perm 1 2 0 3
    s[c] = lane_of<0xD2>(x[c]);  // quad_perm 2 0 1 3
  }
  cross_rows(p, s, C);
  return quad_from<0>(dot_row(x, C));
}

template <typename T>
__device__ __forceinline__ void polar_plain_row(T* x, T* sigma, bool on) {
  T C[3];
  const T det = cofactor_row(x, C);
  const T s = *sigma;
  const T g = on ? rcp(s * s * det) : (T)0;
  *sigma = on ? (T)0.5 * s : s;
#pragma unroll
  for (int c = 0; c < 3; ++c) x[c] = fma(g, C[c], x[c]);
}

// polar_rotation of the quad's matrix, own row in place (the steps and the stopping
// rule of polar_fast); a lane whose first step was too large forms the whole
// matrix and goes on as the other kernels do
template <typename T>
__device__ __forceinline__ void polar_rows(T* x, int k, unsigned* counts, int body) {
  T C[3];
  const T det = cofactor_row(x, C);
  const bool ok = det > Eps<T>::det_floor;
  const bool unscaled = det > (T)0.5 && det < (T)1.5;
  const T zeta = unscaled || !ok ? (T)1 : rcp(cbrt(det));
  const T g = ok ? rcp(zeta * zeta * det) : (T)0;
  T sigma = ok ? (T)0.5 * zeta : (T)1;
#pragma unroll
  for (int c = 0; c < 3; ++c) x[c] = fma(g, C[c], x[c]);
  T C1[3];
  const T det1 = cofactor_row(x, C1);
  const T e = fma(sigma * sigma * sigma, det1, (T)-1);
  const bool one = ok && unscaled && e <= Eps<T>::polar_e_one;
  const bool two = ok && unscaled && !one && e <= Eps<T>::polar_e_three;
  const T g1 = one || two ? rcp(sigma * sigma * det1) : (T)0;
  sigma = one || two ? (T)0.5 * sigma : sigma;
#pragma unroll
  for (int c = 0; c < 3; ++c) x[c] = fma(g1, C1[c], x[c]);
  if (wave_any(two)) {
    polar_plain_row(x, &sigma, two);
    if constexpr (sizeof(T) == 8) {
      const bool three = two && e > Eps<T>::polar_e_two;
      if (wave_any(three)) polar_plain_row(x, &sigma, three);
    }
  }
#pragma unroll
  for (int c = 0; c < 3; ++c) x[c] *= sigma;
  if (wave_any(!(one || two))) {
    T X[9];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      X[c] = quad_from<0>(x[c]);
      X[3 + c] = quad_from<1>(x[c]);
      X[6 + c] = quad_from<2>(x[c]);
    }
    if (!(one || two)) {
      const int how = polar_finish(X, ok);
      if (k == 0) count_polar(counts, body, how);
      take_row(X, k, x);
    }
  }
}

// component of a bond's force, d the own component of its vector; rest: some lane of
// the wave has a rest length (wave-uniform)
template <typename T>
__device__ __forceinline__ T end_force_row(T kap, T phim, T d, bool rest) {
  T f = kap * d;
  if (rest) {
    const T D[3] = {quad_from<0>(d), quad_from<1>(d), quad_from<2>(d)};
    const T dn2 = dot_fused(D, D);
    if (phim != (T)0 && dn2 > (T)1e-24) f = fma(phim * rsqrt_(dn2), d, f);
  }
  return f;
}

// component k of the bond vector (bond_vec) from own row (hi, lo, a) and point xs to
// the partner's row po = (hi, a) and lo.  The world is a partner with c = 0 and
// A = I: its zeros and ones leave xo - c_s as bond_vec forms it.
template <typename T>
__device__ __forceinline__ T bond_row(T hi, T lo, const T* a, const T* xs, const T* po, T plo, const T* xo) {
  T u = po[0] - hi;
  u = fma(po[1], xo[0], u);
  u = fma(po[2], xo[1], u);
  u = fma(po[3], xo[2], u);
  u = fma(-a[0], xs[0], u);
  u = fma(-a[1], xs[1], u);
  u = fma(-a[2], xs[2], u);
  if constexpr (sizeof(T) == 4) u += plo - lo;
  return u;
}

// a quad's rows in LDS: (hi, a0, a1, a2) per lane, and in FP32 the low position word
template <typename T, int LANES>
struct RowLds {
  using R = Plane<T, 4, LANES>;
  T row[R::N];
  T lo[sizeof(T) == 4 ? LANES : 1];
  __device__ void put(int l, T hi, T low, const T* a) {
    const T x[4] = {hi, a[0], a[1], a[2]};
    R::put(row, l, x);
    if constexpr (sizeof(T) == 4) lo[l] = low;
  }
  __device__ void get(int l, T* x, T* low) const {
    R::get(row, l, x);
    if constexpr (sizeof(T) == 4) *low = lo[l];
  }
  // the world's rows in the quad from lane l0 on
  __device__ void put_world(int l0, int t) {
    if (t < 4) {
      const T a[3] = {(T)(t == 0), (T)(t == 1), (T)(t >= 2)};
      put(l0 + t, (T)0, (T)0, a);
    }
  }
};

// the global step of row k (solve_body) from the row's summed force terms (rc, ra)
template <typename T>
__device__ __forceinline__ void solve_row(const T* fac, const T* m, T shi, T slo, const T* sa, T hi, T lo, const T* a,
                                          T rc, T* ra, T* hn, T* ln, T* x) {
  constexpr bool F32 = sizeof(T) == 4;
  settle<1>(&rc);
  settle<3>(ra);
  // + M (s - q^k)
  const T dc = F32 ? slo - lo : shi - hi;  // within a step the high words agree
  const T d0 = sa[0] - a[0], d1 = sa[1] - a[1], d2 = sa[2] - a[2];
  rc = fma(m[0], dc, rc);
  ra[0] += fma(m[3], d2, fma(m[1], d0, m[2] * d1));
  ra[1] += fma(m[5], d2, fma(m[2], d0, m[4] * d1));
  ra[2] += fma(m[6], d2, fma(m[3], d0, m[5] * d1));
  // H^{-1} r
  const T qc = fma(fac[0], rc, -fma(fac[3], ra[2], fma(fac[1], ra[0], fac[2] * ra[1])));
  x[0] = a[0] + fma(fac[6], ra[2], fma(fac[5], ra[1], fma(fac[4], ra[0], -(fac[1] * rc))));
  x[1] = a[1] + fma(fac[8], ra[2], fma(fac[7], ra[1], fma(fac[5], ra[0], -(fac[2] * rc))));
  x[2] = a[2] + fma(fac[9], ra[2], fma(fac[8], ra[1], fma(fac[6], ra[0], -(fac[3] * rc))));
  *hn = F32 ? hi : hi + qc;
  *ln = F32 ? lo + qc : lo;
}

// nsteps steps of a plain scene of at most NT / 4 bodies whose bonds are all quadratic
template <typename T, int NT>
__global__ void __launch_bounds__(NT) k_resident_rows(View<T> v, int n, int nsteps) {
  constexpr int QR = Rec<T>::Q, NB = NT / 4;
  constexpr bool F32 = sizeof(T) == 4;
  __shared__ __align__(16) RowLds<T, NT + 4> lds[2];  // slot NB: the world
  __shared__ double red[2 * NB];
  const int t = threadIdx.x, b = t / 4, k = t % 4;
  const SceneDev& S = v.scenes[0];
  const int K = S.iters, step0 = S.step;
  const bool skip_local = (S.debug & 1) != 0;
  T qn[QR], vw[VW], m[MW], fac[FW], E[2][EW];
  // an end that is not there has no stiffness and the world for a partner, so
  // that the two register ends need no branches
  int ps[2] = {4 * NB + k, 4 * NB + k};
  int e0 = 0, ne = 0;
  bool free = false;
  lds[0].put_world(4 * NB, t);
  lds[1].put_world(4 * NB, t);
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int c = 0; c < EW; ++c) E[u][c] = (T)0;
  if (b < n) {
    load<T, QR>(v.qn + (size_t)QR * b, qn);
    load<T, VW>(v.vel + (size_t)VW * b, vw);
    load<T, MW>(v.mass + (size_t)MW * b, m);
    free = (v.flags[b] & F_PINNED) == 0;
    e0 = v.srow[b];
    ne = free ? v.srow_end[b] - e0 : 0;
    if (free) load<T, FW>(v.fac + (size_t)FW * b, fac);
#pragma unroll
    for (int u = 0; u < 2; ++u)
      if (u < ne) {
        const int j = v.se_partner[e0 + u];
        if (j >= 0) ps[u] = 4 * j + k;
        load<T, EW>(v.se + (size_t)EW * (e0 + u), E[u]);
      }
    if (!free) {  // a pinned body keeps q^n, in both buffers
      T a[3];
      take_row(qn + 3, k, a);
      const T hi = pick(qn[0], qn[1], qn[2], k), lo = F32 ? pick(qn[QR - 4], qn[QR - 3], qn[QR - 2], k) : (T)0;
      lds[0].put(t, hi, lo, a);
      lds[1].put(t, hi, lo, a);
    }
  }
  const bool rest[2] = {wave_any(E[0][7] != (T)0), wave_any(E[1][7] != (T)0)};
  const bool more = wave_any(ne > 2);
  double num = 0.0, den = 0.0;
  for (int st = 0; st < nsteps; ++st) {
    T hi = (T)0, lo = (T)0, a[3], shi = (T)0, slo = (T)0, sa[3];
    if (free) {
      T s[QR];
      resident_predict(S, qn, vw, s);
      shi = hi = pick(s[0], s[1], s[2], k);
      slo = lo = F32 ? pick(s[QR - 4], s[QR - 3], s[QR - 2], k) : (T)0;
      take_row(s + 3, k, sa);
#pragma unroll
      for (int c = 0; c < 3; ++c) a[c] = sa[c];
      lds[0].put(t, hi, lo, a);
    }
    __syncthreads();
    for (int it = 0; it < K; ++it) {
      const RowLds<T, NT + 4>& src = lds[it & 1];
      if (free) {
        T rc = (T)0, ra[3] = {(T)0, (T)0, (T)0};
        auto end = [&](const T* X, const T* po, T plo, bool rest) {
          const T d = bond_row(hi, lo, a, X, po, plo, X + 4);
          T f = end_force_row(X[3], X[7], d, rest);
          settle<1>(&f);
          rc += f;
#pragma unroll
          for (int c = 0; c < 3; ++c) ra[c] = fma(f, X[c], ra[c]);
        };
        T po[2][4], plo[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) src.get(ps[u], po[u], &plo[u]);
#pragma unroll
        for (int u = 0; u < 2; ++u) end(E[u], po[u], plo[u], rest[u]);
        if (more) {
          for (int u = 2; u < ne; ++u) {
            T X[EW], p[4], pl;
            load<T, EW>(v.se + (size_t)EW * (e0 + u), X);
            const int j = v.se_partner[e0 + u];
            src.get(4 * (j < 0 ? NB : j) + k, p, &pl);
            end(X, p, pl, true);
          }
        }
        T hn, ln, x[3];
        solve_row(fac, m, shi, slo, sa, hi, lo, a, rc, ra, &hn, &ln, x);
        if (!skip_local) polar_rows(x, k, v.polar, b);
        lds[(it + 1) & 1].put(t, hn, ln, x);
        if (it == K - 1) {
          T q0[QR], q1[QR];
          gather_body(hi, lo, a, q0);
          gather_body(hn, ln, x, q1);
          residual_terms(m, q1, q0, &num, &den);
        }
        hi = hn;
        lo = ln;
#pragma unroll
        for (int c = 0; c < 3; ++c) a[c] = x[c];
      }
      __syncthreads();
    }
    if (free) {
      T q[QR];
      gather_body(hi, lo, a, q);
      if constexpr (F32) q[QR - 1] = qn[QR - 1];
      resident_recover(q, qn, (T)(1.0 / S.h), vw, v.health);
#pragma unroll
      for (int c = 0; c < QR; ++c) qn[c] = q[c];
    }
  }
  if (free && k == 0) {
    store<T, QR>(v.qn + (size_t)QR * b, qn);
    store<T, VW>(v.vel + (size_t)VW * b, vw);
  }
  if (k == 0) {
    red[b] = num;
    red[NB + b] = den;
  }
  __syncthreads();
  resident_finish<NB>(red, red + NB, v.rho, &v.scenes[0].step, step0 + nsteps);
}

// nsteps steps of a plain scene of at most NT / 4 bodies and NT bond ends, of any
// kind.  An iteration has two phases: thread e forms the terms of end e, whose
// record and state it holds in registers, and puts them in LDS; then the quads add
// their bodies' ends in order and solve.  A body with five ends walks one end's
// chain instead of five.  VARIABLE: some weight or point moves within a step, so
// its body's block is inverted in every iteration.  Driven anchors pass from the
// thread of their entry to their ends through LDS; only a body whose own point is
// driven is factored again.  Us per step, one lane per body against this: slider
// crank 79 and 34, four-bar linkage 72 and 28 (FP64 79 and 34), 8 x 8 net of order 4
// 81 and 41.
template <typename T, int NT, bool VARIABLE>
__global__ void __launch_bounds__(NT) k_resident_ends(View<T> v, int n, int n_ends, int nsteps, DrivenTable dt) {
  constexpr int QR = Rec<T>::Q, NB = NT / 4;
  constexpr bool F32 = sizeof(T) == 4;
  __shared__ __align__(16) RowLds<T, NT> lds[2];
  __shared__ __align__(16) EndLds<T, NT> le;
  __shared__ T anchor[3 * NT];                    // per driven entry
  __shared__ int owner[NT], driver[NT];           // per end: its body, its driven entry (2 b: the partner's point, 2 b + 1: its own)
  __shared__ double red[2 * NB];
  const int t = threadIdx.x, b = t / 4, k = t % 4;
  const SceneDev& S = v.scenes[0];
  const int K = S.iters, step0 = S.step;
  const bool skip_local = (S.debug & 1) != 0;
  const T h2 = (T)(S.h * S.h), beta = (T)S.al_beta, ga = (T)S.al_gamma, ag = (T)(S.al_alpha * S.al_gamma);
  T qn[QR], vw[VW], m[MW], fac[FW];
  double bb[VARIABLE ? 10 : 1];
  int e0 = 0, ne = 0;
  bool free = false, var = false, own_driven = false;
  owner[t] = -1;
  driver[t] = -1;
  __syncthreads();
  for (int d = t; d < dt.n; d += NT) {
    if (dt.end_i[d] >= 0) driver[dt.end_i[d]] = 2 * d;
    if (dt.end_j[d] >= 0) driver[dt.end_j[d]] = 2 * d + 1;
  }
  if (b < n) {
    load<T, QR>(v.qn + (size_t)QR * b, qn);
    load<T, VW>(v.vel + (size_t)VW * b, vw);
    load<T, MW>(v.mass + (size_t)MW * b, m);
    const unsigned fl = v.flags[b];
    free = (fl & F_PINNED) == 0;
    var = (fl & F_VARIABLE) != 0;
    e0 = v.srow[b];
    ne = free ? v.srow_end[b] - e0 : 0;
    if (free) {
      load<T, FW>(v.fac + (size_t)FW * b, fac);
      if constexpr (VARIABLE) load<double, 10>(v.blk + 10 * (size_t)b, bb);
    }
    for (int u = k; u < ne; u += 4) owner[e0 + u] = 2 * b + (var ? 1 : 0);
    if (!free) {  // a pinned body keeps q^n, in both buffers
      T a[3];
      take_row(qn + 3, k, a);
      const T hi = pick(qn[0], qn[1], qn[2], k), lo = F32 ? pick(qn[QR - 4], qn[QR - 3], qn[QR - 2], k) : (T)0;
      lds[0].put(t, hi, lo, a);
      lds[1].put(t, hi, lo, a);
    }
  }
  __syncthreads();
  // this thread's end
  const bool end = t < n_ends && owner[t] >= 0;
  const bool end_var = end && (owner[t] & 1);
  const int eb = end ? owner[t] >> 1 : 0, drv = end ? driver[t] : -1;
  int ej = -1;
  T E[EW], al[4] = {(T)0, (T)0, (T)0, (T)0};
  if (end) {
    load<T, EW>(v.se + (size_t)EW * t, E);
    ej = v.se_partner[t];
    if (end_var) load<T, 4>(v.al + 4 * (size_t)t, al);
  }
  for (int u = 0; u < ne; ++u) own_driven = own_driven || (driver[e0 + u] >= 0 && (driver[e0 + u] & 1));
  double num = 0.0, den = 0.0;
  for (int st = 0; st < nsteps; ++st) {
    if (dt.n > 0) {
      for (int d = t; d < dt.n; d += NT)
        update_driven_entry(v, d, step0 + st, S, dt.end_i, dt.end_j, dt.param, anchor + 3 * d);
      __syncthreads();
      if (drv >= 0) {
        const T* x = anchor + 3 * (drv >> 1);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          E[c] = drv & 1 ? x[c] : E[c];
          E[4 + c] = drv & 1 ? E[4 + c] : x[c];
        }
      }
      if (own_driven) {
        if (k == 0) factor_body(v, dt.mass64, b);
        __threadfence_block();
        load<T, FW>(v.fac + (size_t)FW * b, fac);
        if constexpr (VARIABLE) load<double, 10>(v.blk + 10 * (size_t)b, bb);
      }
    }
    if (al[3] > (T)0) {  // augmented ends, warm start (Sec. 5.2.2)
      al[0] = fmax(ga * al[0], al[3]);
      al[1] = ag * al[1];
    }
    T hi = (T)0, lo = (T)0, a[3], shi = (T)0, slo = (T)0, sa[3];
    if (free) {
      T s[QR];
      resident_predict(S, qn, vw, s);
      shi = hi = pick(s[0], s[1], s[2], k);
      slo = lo = F32 ? pick(s[QR - 4], s[QR - 3], s[QR - 2], k) : (T)0;
      take_row(s + 3, k, sa);
#pragma unroll
      for (int c = 0; c < 3; ++c) a[c] = sa[c];
      lds[0].put(t, hi, lo, a);
    }
    __syncthreads();
    for (int it = 0; it < K; ++it) {
      const RowLds<T, NT>& src = lds[it & 1];
      if (end) {
        auto state = [&](int body, T* q) {
          T r[3][4], l[3];
#pragma unroll
          for (int c = 0; c < 3; ++c) src.get(4 * body + c, r[c], l + c);
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            q[c] = r[c][0];
#pragma unroll
            for (int i = 0; i < 3; ++i) q[3 + 3 * c + i] = r[c][1 + i];
            if constexpr (F32) q[12 + c] = l[c];
          }
        };
        T q[QR], qj[QR], f[4], g, x[4];
        state(eb, q);
        if (ej >= 0) state(ej, qj);
        const bool moves = end_terms(E, al, ej, q, qj, h2, beta, it == K - 1, f, &g, x, f + 3);
        x[3] = (T)(moves ? 1 : 0);
        le.put(t, f, x, g);
      }
      __syncthreads();
      if (free) {
        T rc = (T)0, ra[3] = {(T)0, (T)0, (T)0}, fk[FW];
        Block dB{};
        bool refactor = false;
        le.each(e0, ne, [&](const T* f, const T* x, T g) {
          const T fk = pick(f[0], f[1], f[2], k);
          T fr = g * fk;
          settle<1>(&fr);
          rc = fma(g, fk, rc);
#pragma unroll
          for (int c = 0; c < 3; ++c) ra[c] = fma(fr, x[c], ra[c]);
          if constexpr (VARIABLE) {
            add_moved(x[3] != (T)0, f[3], x, dB);
            refactor = refactor || x[3] != (T)0;
          }
        });
#pragma unroll
        for (int c = 0; c < 10; ++c) fk[c] = fac[c];
        if constexpr (VARIABLE) {
          if (refactor) refactored(bb, dB, fk);
        }
        T hn, ln, x[3];
        solve_row(fk, m, shi, slo, sa, hi, lo, a, rc, ra, &hn, &ln, x);
        if (!skip_local) polar_rows(x, k, v.polar, b);
        lds[(it + 1) & 1].put(t, hn, ln, x);
        if (it == K - 1) {
          T q0[QR], q1[QR];
          gather_body(hi, lo, a, q0);
          gather_body(hn, ln, x, q1);
          residual_terms(m, q1, q0, &num, &den);
        }
        hi = hn;
        lo = ln;
#pragma unroll
        for (int c = 0; c < 3; ++c) a[c] = x[c];
      }
      __syncthreads();
    }
    if (free) {
      T q[QR];
      gather_body(hi, lo, a, q);
      if constexpr (F32) q[QR - 1] = qn[QR - 1];
      resident_recover(q, qn, (T)(1.0 / S.h), vw, v.health);
#pragma unroll
      for (int c = 0; c < QR; ++c) qn[c] = q[c];
    }
  }
  if (free && k == 0) {
    store<T, QR>(v.qn + (size_t)QR * b, qn);
    store<T, VW>(v.vel + (size_t)VW * b, vw);
  }
  if (end_var) {
    store<T, 4>(v.al + 4 * (size_t)t, al);
    v.se[(size_t)EW * t + 7] = E[7];
  }
  if (k == 0) {
    red[b] = num;
    red[NB + b] = den;
  }
  __syncthreads();
  resident_finish<NB>(red, red + NB, v.rho, &v.scenes[0].step, step0 + nsteps);
}

// k_tile_step with a quad of lanes per body: nsteps steps of the batch's tiles of up
// to TB bodies, 4 TB threads each.  The state stays in registers from step to step
// and is stored where a scene's last step of the launch ends.
template <typename T, int TB>
__global__ void __launch_bounds__(4 * TB, sizeof(T) == 4 ? 3 : 2) k_tile_rows(View<T> v, TileTable tt, int nsteps) {
  constexpr int QR = Rec<T>::Q, NL = 4 * TB, MAXE = 2;
  constexpr bool F32 = sizeof(T) == 4;
  // q^k's rows (slot TB: the world) and the points of each body's first MAXE ends at
  // q^k (kernels_tile.h), double-buffered: one barrier per iteration
  __shared__ __align__(16) RowLds<T, NL + 4> lds[2];
  __shared__ T ly[2][MAXE * NL];
  using N = Plane<T, QR, TB>;
  __shared__ __align__(16) T ln[N::N];  // q^n through the iterations (each quad its own body's)
  __shared__ double red[2 * TB];
  const int t = threadIdx.x, b = t / 4, k = t % 4;
  lds[0].put_world(NL, t);
  lds[1].put_world(NL, t);
  const int ntiles = *tt.n_tiles;
  for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int first = tt.first[tile], nb = tt.count[tile], kmax = tt.kmax[tile];
    const int i = first + b;
    const int scn = b < nb ? v.bscene[i] : -1;
    const bool pinned = scn >= 0 && (v.flags[i] & F_PINNED);
    T qn[QR], vw[VW], m[MW], fac[FW];
    // per register end (as in k_tile_step): the own point, h^2 kappa, h^2 phi^-, the
    // partner's lane and the place of its mirror end's point.  An end that is not
    // there has no stiffness, the world for a partner and its own point for a mirror.
    T X[MAXE][3], kap[MAXE], phim[MAXE];
    int ps[MAXE], yo[MAXE];
    bool mirrored[MAXE];
#pragma unroll
    for (int u = 0; u < MAXE; ++u) {
      X[u][0] = X[u][1] = X[u][2] = kap[u] = phim[u] = (T)0;
      ps[u] = NL + k;
      yo[u] = u * NL + t;
      mirrored[u] = false;
    }
#pragma unroll
    for (int c = 0; c < QR; ++c) qn[c] = (T)0;
#pragma unroll
    for (int c = 0; c < MW; ++c) m[c] = (T)0;
    int e0 = 0, ne = 0, steps_total = 0, sstep = 0, iters = 0;
    if (scn >= 0) {
      const SceneDev& S = v.scenes[scn];
      steps_total = S.steps_total;
      sstep = S.step;
      iters = S.iters;
      load<T, QR>(v.qn + (size_t)QR * i, qn);
      e0 = v.srow[i];
      ne = v.srow_end[i] - e0;
      // a pinned body publishes its bond points too, for its partners
#pragma unroll
      for (int u = 0; u < MAXE; ++u) {
        if (u < ne) {
          T Eu[EW];
          load<T, EW>(v.se + (size_t)EW * (e0 + u), Eu);
          X[u][0] = Eu[0];
          X[u][1] = Eu[1];
          X[u][2] = Eu[2];
          kap[u] = Eu[3];
          phim[u] = Eu[7];
          const int p = v.se_partner[e0 + u];
          if (p >= 0) ps[u] = 4 * (p - first) + k;
          if (p >= 0 && !pinned) {
            // the mirror end: the end that is the n-th of this body towards p
            // pairs with the n-th end of p towards this body
            int rank = 0;
#pragma unroll
            for (int w = 0; w < u; ++w) rank += ps[w] == ps[u] ? 1 : 0;
            const int b0 = v.srow[p], b1 = min(v.srow_end[p], b0 + MAXE);
#pragma unroll
            for (int w = 0; w < MAXE; ++w)
              if (b0 + w < b1 && !mirrored[u] && v.se_partner[b0 + w] == i) {
                if (rank == 0) {
                  mirrored[u] = true;
                  yo[u] = w * NL + 4 * (p - first) + k;
                }
                --rank;
              }
          }
        }
      }
      if (!pinned) {
        load<T, VW>(v.vel + (size_t)VW * i, vw);
        load<T, MW>(v.mass + (size_t)MW * i, m);
        load<T, FW>(v.fac + (size_t)FW * i, fac);
      }
    }
    const bool mover = scn >= 0 && !pinned;
    const bool diag_pi = wave_all(!mover || (m[2] == (T)0 && m[3] == (T)0 && m[5] == (T)0));
    // wave-uniform: some lane takes register end u the long way, or has a rest length
    bool unmirrored[MAXE], rest[MAXE], long_way = mover && ne > MAXE;
#pragma unroll
    for (int u = 0; u < MAXE; ++u) {
      const bool lw = mover && u < ne && !mirrored[u];
      long_way = long_way || lw;
      unmirrored[u] = wave_any(lw);
      rest[u] = wave_any(mover && phim[u] != (T)0);
    }
    const bool more = wave_any(mover && ne > MAXE);
    // whether some lane of the tile reads a partner's rows after a step's first iteration
    const bool need_q = __syncthreads_or(long_way);
    for (int step = 0; step < nsteps; ++step) {
      const bool present = scn >= 0 && sstep < steps_total;
      const bool moving = present && !pinned;
      const int K = present ? iters : 0;
      // the residual is formed, and the state stored, on the launch's last step and on a
      // scene's own last step
      const bool final = present && (step == nsteps - 1 || sstep + 1 >= steps_total);
      T hi = (T)0, lo = (T)0, a[3], msc = (T)0, msa[3];
      N::put(ln, b, qn);
      {
        T q[QR], ms[QW];
#pragma unroll
        for (int c = 0; c < QR; ++c) q[c] = qn[c];
        if (moving) {
          const SceneDev& S = v.scenes[scn];
          const T h = (T)S.h;
          predict_rotation(qn + 3, vw + 3, h, q + 3);
          pos_add_lo(q, h * (vw[0] + h * (T)S.g0), h * (vw[1] + h * (T)S.g1), h * (vw[2] + h * (T)S.g2));
          mass_times(m, q, ms);
          msc = pick(ms[0], ms[1], ms[2], k);
          take_row(ms + 3, k, msa);
        }
        hi = pick(q[0], q[1], q[2], k);
        if constexpr (F32) lo = pick(q[12], q[13], q[14], k);
        take_row(q + 3, k, a);
      }
      double num = 0.0, den = 0.0;
      T dh[MAXE];  // FP32: hi of the partner minus hi of this body, per end
      for (int it = 0; it < kmax; ++it) {
        RowLds<T, NL + 4>& buf = lds[it & 1];
        T* ybuf = ly[it & 1];
        T ys[MAXE];
        // the point's part that moves within a step: in FP32 without the high word
#pragma unroll
        for (int u = 0; u < MAXE; ++u)
          ys[u] = fma(a[2], X[u][2], fma(a[1], X[u][1], fma(a[0], X[u][0], F32 ? lo : hi)));
        if (present) {
          if (it == 0 || need_q) buf.put(t, hi, lo, a);
#pragma unroll
          for (int u = 0; u < MAXE; ++u) ybuf[u * NL + t] = ys[u];
        }
        __syncthreads();
        if (moving && it < K) {
          T po[MAXE];
#pragma unroll
          for (int u = 0; u < MAXE; ++u) po[u] = ybuf[yo[u]];
          // r = M (s - q^k) + sum of the ends' J^T f (the forces carry h^2)
          T rc = fma(-m[0], F32 ? lo : hi, msc);
          T ra[3] = {fma(-m[1], a[0], msa[0]), fma(-m[4], a[1], msa[1]), fma(-m[6], a[2], msa[2])};
          if (!diag_pi) {
            ra[0] = fma(-m[3], a[2], fma(-m[2], a[1], ra[0]));
            ra[1] = fma(-m[5], a[2], fma(-m[2], a[0], ra[1]));
            ra[2] = fma(-m[5], a[1], fma(-m[3], a[0], ra[2]));
          }
          auto add = [&](const T* x, T f) {
            rc += f;
#pragma unroll
            for (int c = 0; c < 3; ++c) ra[c] = fma(f, x[c], ra[c]);
          };
#pragma unroll
          for (int u = 0; u < MAXE; ++u) {
            T d;
            if constexpr (F32) {
              if (it == 0) {
                T p[4], pl;
                buf.get(ps[u], p, &pl);
                dh[u] = p[0] - hi;
              }
              d = dh[u] + (po[u] - ys[u]);
            } else {
              d = po[u] - ys[u];
            }
            if (unmirrored[u]) {
              // an end anchored in the world, or whose mirror is not among the
              // partner's register ends: from the partner's rows and its record
              if (u < ne && !mirrored[u]) {
                T E[EW], p[4], pl;
                load<T, EW>(v.se + (size_t)EW * (e0 + u), E);
                buf.get(ps[u], p, &pl);
                d = bond_row(hi, lo, a, E, p, pl, E + 4);
              }
            }
            add(X[u], end_force_row(kap[u], phim[u], d, rest[u]));
          }
          if (more) {
            for (int e = e0 + MAXE; e < e0 + ne; ++e) {
              T E[EW], p[4], pl;
              load<T, EW>(v.se + (size_t)EW * e, E);
              const int j = v.se_partner[e];
              buf.get(j < 0 ? NL + k : 4 * (j - first) + k, p, &pl);
              add(E, end_force_row(E[3], E[7], bond_row(hi, lo, a, E, p, pl, E + 4), true));
            }
          }
          const bool last = it == K - 1 && final;
          T q0[QR];
          if (last) gather_body(hi, lo, a, q0);
          // q + H^{-1} r, each entry one fused chain from its own value (block_apply_add)
          T& c0 = F32 ? lo : hi;
          c0 = fma(fac[0], rc, fma(-fac[3], ra[2], fma(-fac[2], ra[1], fma(-fac[1], ra[0], c0))));
          a[0] = fma(fac[6], ra[2], fma(fac[5], ra[1], fma(fac[4], ra[0], fma(-fac[1], rc, a[0]))));
          a[1] = fma(fac[8], ra[2], fma(fac[7], ra[1], fma(fac[5], ra[0], fma(-fac[2], rc, a[1]))));
          a[2] = fma(fac[9], ra[2], fma(fac[8], ra[1], fma(fac[6], ra[0], fma(-fac[3], rc, a[2]))));
          polar_rows(a, k, v.polar, i);
          if (last) {
            constexpr int L = F32 ? 12 : 0;
            T q1[QR], dd[QW];
            gather_body(hi, lo, a, q1);
            const T cc[3] = {(T)pos_value(q0, 0), (T)pos_value(q0, 1), (T)pos_value(q0, 2)};
            den = m_norm2(m, cc, q0);
#pragma unroll
            for (int c = 0; c < 3; ++c) dd[c] = q1[L + c] - q0[L + c];
#pragma unroll
            for (int c = 0; c < 9; ++c) dd[3 + c] = q1[3 + c] - q0[3 + c];
            num = m_norm2(m, dd, dd);
          }
        }
      }
      if (moving) {
        T q[QR];
        gather_body(hi, lo, a, q);
        N::get(ln, b, qn);
        if constexpr (F32) q[QR - 1] = qn[QR - 1];
        resident_recover(q, qn, (T)(1.0 / v.scenes[scn].h), vw, v.health + scn);
#pragma unroll
        for (int c = 0; c < QR; ++c) qn[c] = q[c];
        if (final && k == 0) {
          store<T, QR>(v.qn + (size_t)QR * i, qn);
          store<T, VW>(v.vel + (size_t)VW * i, vw);
        }
      }
      // per-scene FP64 residual: pairwise sums over the scene's bodies by their index
      // within the scene, the same order wherever the scene sits in the tile
      if (k == 0) {
        red[b] = num;
        red[TB + b] = den;
      }
      const int loc = present && k == 0 ? i - v.scenes[scn].body_off : 1;
      // (this barrier also settles LDS for the next step or tile)
      if (__syncthreads_or(final)) {
        const int nbs = present ? v.scenes[scn].n_bodies : 0;
#pragma unroll
        for (int w = 1; w < TB; w <<= 1) {
          if ((loc & (2 * w - 1)) == 0 && loc + w < nbs) {
            red[b] += red[b + w];
            red[TB + b] += red[TB + b + w];
          }
          __syncthreads();
        }
      }
      if (present && loc == 0) {
        if (final) {
          const double x = red[b], y = red[TB + b];
          v.rho[scn] = y > 0.0 ? sqrt(x / y) : 0.0;
        }
        v.scenes[scn].step = sstep + 1;
      }
      if (present) ++sstep;
    }
  }
}

}  // namespace pabd
