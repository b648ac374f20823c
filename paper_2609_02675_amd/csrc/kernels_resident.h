// kernels_resident.h -- whole steps of one small scene in one workgroup: the
// prediction, the K global/local Jacobi iterations of Algorithm 1 and the
// velocity recovery of a plain handle's scene whose bodies fit the workgroup.
// The bodies exchange q^k through LDS and everything a step does not change
// stays in registers and LDS, so an iteration waits on no global load.
//
//   k_resident_joints   a scene of quadratic bonds, one lane per body: any number of
//                       steps in one launch (nothing is built between them)
//   k_resident_net      the same for bonds of any kind, in two phases: a lane per
//                       end, then a lane per body (smaller scenes: kernels_rows.h)
//   k_resident_contact  one step of a contact scene after its contact construction:
//                       four lanes per body form its ends' terms, then one lane
//                       per body solves
//
// Each iteration is made of the flat path's pieces in the same order, so a scene
// gives the same bits in the flat kernels, and its residual and step counter
// are kept here.
//
// What bounds them: the latency of one iteration (a barrier or two, the LDS round
// trip of a partner's state, the dependent arithmetic of its ends, block solve and
// rotation), not any throughput; the contact kernel with many waves and contacts is
// bound by their instruction issue on the one compute unit, so larger piles take the
// flat kernels (EngineT::resident).
//
// Measured per step, against one kernel that read records, masses, factors and the
// scene from memory in every iteration behind barriers of 16 waves (and took a
// launch per step): eight-body chain 0.044 -> 0.025 ms (FP64 0.066 -> 0.051),
// chain of 200 0.057 -> 0.027, of 500 0.075 -> 0.040, of 1,000 0.101 -> 0.085,
// 11 x 11 net of order 4 in FP64 0.164 -> 0.074 (0.090 with one lane walking a body's
// ends), 16 x 16 net of order 6 0.180 -> 0.070, pile of 16 boxes 0.118 -> 0.095, of 60
// 0.134 -> 0.111 with its contact construction, of 128 falling boxes 0.087 -> 0.051.
#pragma once

#include "common.h"
#include "device_math.h"
#include "kernels_flat.h"
#include "kernels_step.h"

namespace pabd {

// The largest workgroup: 1,024 threads in FP32, 512 in FP64, where the iteration
// needs more registers per lane.  A scene takes the smallest workgroup that holds
// its lanes: fewer waves meet at a barrier (one wave meets none), and up to 256
// threads each wave has a SIMD and its registers to itself.  HOLD: the
// workgroup's registers hold what a step does not change (not in the largest,
// whose lanes have 128 in FP32 and 256 in FP64: there every iteration reads it
// again, from the caches).
template <typename T>
struct Resident {
  static constexpr int NT = sizeof(T) == 4 ? 1024 : 512;
  static constexpr bool hold(int nt) { return nt < NT; }
};

// driven bonds of the scene (Sec. 5.3.3, read as in k_update_driven) and the FP64
// masses the refactor needs: a scene with driven bonds turns their anchors and
// refactors its bodies' blocks at the start of every step, as the flat path's
// k_update_driven and k_factor do
struct DrivenTable {
  int n;
  const int *end_i, *end_j;
  const double *param, *mass64;
};

// A record of R values per body in LDS for NB bodies, 16 bytes of a body beside
// the same 16 bytes of the next: neighbouring lanes read neighbouring words.
template <typename T, int R, int NB>
struct Plane {
  static constexpr int P = 16 / sizeof(T), N = R * NB;
  __device__ static void put(T* buf, int b, const T* x) {
#pragma unroll
    for (int c = 0; c < R / P; ++c) store<T, P>(buf + P * (c * NB + b), x + P * c);
  }
  __device__ static void get(const T* buf, int b, T* x) {
#pragma unroll
    for (int c = 0; c < R / P; ++c) load<T, P>(buf + P * (c * NB + b), x + P * c);
  }
};

// the scene's FP64 residual in a fixed order (a pairwise tree over the partials of
// NB bodies) and its step counter
template <int NB>
__device__ __forceinline__ void resident_finish(double* rn, double* rd, double* rho, int* step, int steps) {
  const int t = threadIdx.x;
  for (int w = NB / 2; w > 0; w >>= 1) {
    if (t < w) {
      rn[t] += rn[t + w];
      rd[t] += rd[t + w];
    }
    __syncthreads();
  }
  if (t == 0) {
    *rho = rd[0] > 0.0 ? sqrt(rn[0] / rd[0]) : 0.0;
    *step = steps;
  }
}

// the end of a body's step from q^K (in place: q^{n+1}) and q^n: velocities, health
template <typename T>
__device__ __forceinline__ void resident_recover(T* q, const T* qn, T ih, T* vw, int* health) {
  constexpr int QR = Rec<T>::Q;
  settle<QR>(q);
  recover_velocity(q, qn, ih, vw);
  bool finite = true;
#pragma unroll
  for (int c = 0; c < QR; ++c) finite = finite && isfinite(q[c]);
#pragma unroll
  for (int c = 0; c < 6; ++c) finite = finite && isfinite(vw[c]);
  if (!finite) atomicOr(health, 1);
  pos_renorm(q);
}

// the prediction (Algorithm 1) of a free body: s = q^0
template <typename T>
__device__ __forceinline__ void resident_predict(const SceneDev& S, const T* qn, const T* vw, T* s) {
  constexpr int QR = Rec<T>::Q;
  const T h = (T)S.h;
#pragma unroll
  for (int c = 0; c < QR; ++c) s[c] = qn[c];
  pos_add_lo(s, h * (vw[0] + h * (T)S.g0), h * (vw[1] + h * (T)S.g1), h * (vw[2] + h * (T)S.g2));
  predict_rotation(qn + 3, vw + 3, h, s + 3);
  settle<QR>(s);
}

// nsteps steps of a scene of at most NT bodies without contacts whose bonds are all
// quadratic.  The first two ends of a body are read once per launch, any further
// ones from global memory as they are needed.
template <typename T, int NT>
__global__ void __launch_bounds__(NT) k_resident_joints(View<T> v, int n, int nsteps) {
  constexpr int QR = Rec<T>::Q;
  constexpr bool HOLD = Resident<T>::hold(NT);
  using Q = Plane<T, QR, NT>;
  __shared__ __align__(16) T lq[2][Q::N];
  const int t = threadIdx.x;
  const SceneDev& S = v.scenes[0];
  const int K = S.iters, step0 = S.step;
  const bool skip_local = (S.debug & 1) != 0;
  const bool body = t < n;
  T qn[QR], vw[VW], m[MW], fac[FW], E[2][EW];
  int id[2];
  int e0 = 0, ne = 0;
  bool free = false;
  if (body) {
    load<T, QR>(v.qn + (size_t)QR * t, qn);
    load<T, VW>(v.vel + (size_t)VW * t, vw);
    free = (v.flags[t] & F_PINNED) == 0;
    e0 = v.srow[t];
    ne = free ? v.srow_end[t] - e0 : 0;
    if constexpr (HOLD) {
      load<T, MW>(v.mass + (size_t)MW * t, m);
      if (free) load<T, FW>(v.fac + (size_t)FW * t, fac);
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (u < ne) {
          id[u] = v.se_partner[e0 + u];
          load<T, EW>(v.se + (size_t)EW * (e0 + u), E[u]);
        }
    }
  }
  if (body && !free) {  // a pinned body keeps q^n, in both buffers
    Q::put(lq[0], t, qn);
    Q::put(lq[1], t, qn);
  }
  double num = 0.0, den = 0.0;
  for (int st = 0; st < nsteps; ++st) {
    T s[QR], q[QR];
    if (free) {
      if constexpr (!HOLD) {
        load<T, QR>(v.qn + (size_t)QR * t, qn);
        load<T, VW>(v.vel + (size_t)VW * t, vw);
      }
      resident_predict(S, qn, vw, s);
      Q::put(lq[0], t, s);
      if constexpr (!HOLD) store<T, QR>(v.s + (size_t)QR * t, s);
#pragma unroll
      for (int c = 0; c < QR; ++c) q[c] = s[c];
    }
    __syncthreads();
    for (int k = 0; k < K; ++k) {
      const T* src = lq[k & 1];
      T* dst = lq[(k + 1) & 1];
      if (free) {
        auto state = [&](int j, T* qj) { Q::get(src, j, qj); };
        T rb[QW];
#pragma unroll
        for (int c = 0; c < QW; ++c) rb[c] = (T)0;
        if constexpr (!HOLD) {
          quadratic_ends<T, 1>(v, e0, e0 + ne, q, state, rb);
        } else {
          T qj[2][QR];
#pragma unroll
          for (int u = 0; u < 2; ++u)
            if (u < ne && id[u] >= 0) state(id[u], qj[u]);
#pragma unroll
          for (int u = 0; u < 2; ++u)
            if (u < ne) quadratic_end(E[u], id[u], q, qj[u], rb);
          quadratic_ends<T, 1>(v, e0 + 2, e0 + ne, q, state, rb);
        }
        T fk[FW];
        if constexpr (HOLD) {
#pragma unroll
          for (int c = 0; c < 10; ++c) fk[c] = fac[c];
        } else {
          load<T, FW>(v.fac + (size_t)FW * t, fk);
          load<T, QR>(v.s + (size_t)QR * t, s);
          load<T, MW>(v.mass + (size_t)MW * t, m);
        }
        T qo[QR];
        solve_body(fk, s, m, rb, q, skip_local, v.polar, t, qo);
        if (k == K - 1) residual_terms(m, qo, q, &num, &den);
        settle<QR>(qo);
        Q::put(dst, t, qo);
#pragma unroll
        for (int c = 0; c < QR; ++c) q[c] = qo[c];
      }
      __syncthreads();
    }
    if (free) {
      if constexpr (!HOLD) load<T, QR>(v.qn + (size_t)QR * t, qn);
      resident_recover(q, qn, (T)(1.0 / S.h), vw, v.health);
      if constexpr (HOLD) {
#pragma unroll
        for (int c = 0; c < QR; ++c) qn[c] = q[c];
      } else {
        store<T, QR>(v.qn + (size_t)QR * t, q);
        store<T, VW>(v.vel + (size_t)VW * t, vw);
      }
    }
  }
  if constexpr (HOLD) {
    if (free) {
      store<T, QR>(v.qn + (size_t)QR * t, qn);
      store<T, VW>(v.vel + (size_t)VW * t, vw);
    }
  }
  double* red = reinterpret_cast<double*>(&lq[0][0]);  // the buffers are done with
  red[t] = num;
  red[NT + t] = den;
  __syncthreads();
  resident_finish<NT>(red, red + NT, v.rho, &v.scenes[0].step, step0 + nsteps);
}

// Per end of a two-phase iteration, in LDS: (force, weight), (point, 1 if weight or
// point moves within the step) and the force's factor (end_terms)
template <typename T, int NE>
struct EndLds {
  using P = Plane<T, 4, NE>;
  T f[P::N], x[P::N], g[NE];
  __device__ void put(int e, const T* fw, const T* xm, T scale) {
    P::put(f, e, fw);
    P::put(x, e, xm);
    g[e] = scale;
  }
  // add(f, x, g) of ends e0 .. e0 + ne in order, four ends' reads in flight
  template <typename Add>
  __device__ __forceinline__ void each(int e0, int ne, Add add) const {
    for (int u0 = 0; u0 < ne; u0 += 4) {
      T a[4][4], b[4][4], c[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int e = e0 + min(u0 + u, ne - 1);
        P::get(f, e, a[u]);
        P::get(x, e, b[u]);
        c[u] = g[e];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (u0 + u < ne) add(a[u], b[u], c[u]);
    }
  }
};

// The most ends of a scene in k_resident_net: what 160 KB of LDS hold beside q^k.
template <typename T>
constexpr int NET_ENDS = sizeof(T) == 4 ? 2560 : 1536;

// nsteps steps of a scene of at most NT bodies and NET_ENDS ends of any kind, without
// contacts.  An iteration has two phases: the threads form the terms of the ends,
// one end each, and put them in LDS; then one thread per body adds its ends in
// order and solves.  The first U ends of a thread stay in its registers, with their
// states; the rest come from global memory.  VARIABLE: some weight or point moves
// within a step, so its body's block is inverted in every iteration.  One thread
// per body for both phases walked its ends one after another; a quad of threads per
// body (k_resident_ends) inverts the block four times, which more than 64 bodies
// pay for in instructions.  Issue bounds it: about 1,100 FP64 instructions per body
// and iteration on two to eight waves.
template <typename T, int NT, bool VARIABLE>
__global__ void __launch_bounds__(NT) k_resident_net(View<T> v, int n, int n_ends, int nsteps, DrivenTable dt) {
  constexpr int QR = Rec<T>::Q, NE = NET_ENDS<T>, U = NT < 1024 ? 2 : 1;
  constexpr bool HOLD = NT < 1024;
  using Q = Plane<T, QR, NT>;
  __shared__ __align__(16) T lq[Q::N];
  __shared__ __align__(16) EndLds<T, NE> le;
  __shared__ short owner[NE];  // 2 b + 1 of a body with variable ends, 2 b of another; -1: pinned
  const int t = threadIdx.x;
  const SceneDev& S = v.scenes[0];
  const int K = S.iters, step0 = S.step;
  const bool skip_local = (S.debug & 1) != 0;
  const T h2 = (T)(S.h * S.h), beta = (T)S.al_beta, ga = (T)S.al_gamma, ag = (T)(S.al_alpha * S.al_gamma);
  T qn[QR], vw[VW], m[MW], fac[FW];
  double bb[VARIABLE ? 10 : 1];
  int e0 = 0, ne = 0;
  bool free = false;
  if (t < n) {
    load<T, QR>(v.qn + (size_t)QR * t, qn);
    load<T, VW>(v.vel + (size_t)VW * t, vw);
    const unsigned fl = v.flags[t];
    free = (fl & F_PINNED) == 0;
    e0 = v.srow[t];
    ne = v.srow_end[t] - e0;
    const short o = free ? (short)(2 * t + (fl & F_VARIABLE ? 1 : 0)) : (short)-1;
    for (int u = 0; u < ne; ++u) owner[e0 + u] = o;
    if (!free) Q::put(lq, t, qn);  // a pinned body keeps q^n
  }
  __syncthreads();
  // this thread's register ends
  int eo[U], ej[U];
  T E[U][EW], al[U][4];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int e = t + u * NT;
    eo[u] = e < n_ends ? owner[e] : -1;
    ej[u] = -1;
    al[u][0] = al[u][1] = al[u][2] = al[u][3] = (T)0;
    if (eo[u] >= 0) {
      load<T, EW>(v.se + (size_t)EW * e, E[u]);
      ej[u] = v.se_partner[e];
      if (eo[u] & 1) load<T, 4>(v.al + 4 * (size_t)e, al[u]);
    }
  }
  auto warm = [&](T* a) {  // augmented ends, warm start (Sec. 5.2.2)
    a[0] = fmax(ga * a[0], a[3]);
    a[1] = ag * a[1];
  };
  double num = 0.0, den = 0.0;
  for (int st = 0; st < nsteps; ++st) {
    if (dt.n > 0) {
      // driven anchors at this step's time, then every block of the scene
      // refactored (the same functions as the flat path's kernels)
      for (int b = t; b < dt.n; b += NT)
        update_driven_entry(v, b, step0 + st, S, dt.end_i, dt.end_j, dt.param);
      __syncthreads();
      if (free) factor_body(v, dt.mass64, t);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (eo[u] >= 0) {  // a slider's E[7] lives in the register
          T r[EW];
          load<T, EW>(v.se + (size_t)EW * (t + u * NT), r);
#pragma unroll
          for (int c = 0; c < 7; ++c) E[u][c] = r[c];
        }
    }
    if (free && (st == 0 || dt.n > 0) && HOLD) {
      load<T, MW>(v.mass + (size_t)MW * t, m);
      load<T, FW>(v.fac + (size_t)FW * t, fac);
      if constexpr (VARIABLE) load<double, 10>(v.blk + 10 * (size_t)t, bb);
    }
    if constexpr (VARIABLE) {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (al[u][3] > (T)0) warm(al[u]);
      for (int e = t + U * NT; e < n_ends; e += NT)
        if (owner[e] >= 0 && (owner[e] & 1)) {
          T a[4];
          load<T, 4>(v.al + 4 * (size_t)e, a);
          if (a[3] > (T)0) {
            warm(a);
            store<T, 4>(v.al + 4 * (size_t)e, a);
          }
        }
    }
    T s[QR], q[QR];
    if (free) {
      resident_predict(S, qn, vw, s);
      Q::put(lq, t, s);
      if constexpr (!HOLD) store<T, QR>(v.s + (size_t)QR * t, s);
#pragma unroll
      for (int c = 0; c < QR; ++c) q[c] = s[c];
    }
    __syncthreads();
    for (int k = 0; k < K; ++k) {
      auto terms = [&](int e, int o, int j, T* R, T* a) {
        T qi[QR], qj[QR], f[4], g, x[4];
        Q::get(lq, o >> 1, qi);
        if (j >= 0) Q::get(lq, j, qj);
        const bool moves = end_terms(R, a, j, qi, qj, h2, beta, k == K - 1, f, &g, x, f + 3);
        x[3] = (T)(moves ? 1 : 0);
        le.put(e, f, x, g);
      };
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (eo[u] >= 0) terms(t + u * NT, eo[u], ej[u], E[u], al[u]);
      for (int e = t + U * NT; e < n_ends; e += NT) {
        const int o = owner[e];
        if (o < 0) continue;
        T R[EW], a[4] = {(T)0, (T)0, (T)0, (T)0};
        load<T, EW>(v.se + (size_t)EW * e, R);
        if (VARIABLE && (o & 1)) load<T, 4>(v.al + 4 * (size_t)e, a);
        terms(e, o, v.se_partner[e], R, a);
        if constexpr (VARIABLE) {
          if (a[3] > (T)0)
            store<T, 4>(v.al + 4 * (size_t)e, a);
          else if (k == K - 1 && a[3] != (T)0)
            v.se[(size_t)EW * e + 7] = R[7];
        }
      }
      __syncthreads();
      if (free) {
        T rb[QW], fk[FW];
#pragma unroll
        for (int c = 0; c < QW; ++c) rb[c] = (T)0;
        Block dB{};
        bool refactor = false;
        le.each(e0, ne, [&](const T* f, const T* x, T g) {
          add_scaled(rb, x, g, f);
          if constexpr (VARIABLE) {
            add_moved(x[3] != (T)0, f[3], x, dB);
            refactor = refactor || x[3] != (T)0;
          }
        });
        if constexpr (HOLD) {
#pragma unroll
          for (int c = 0; c < 10; ++c) fk[c] = fac[c];
        } else {
          load<T, FW>(v.fac + (size_t)FW * t, fk);
          load<T, QR>(v.s + (size_t)QR * t, s);
          load<T, MW>(v.mass + (size_t)MW * t, m);
        }
        if constexpr (VARIABLE) {
          if (refactor) {
            if constexpr (!HOLD) load<double, 10>(v.blk + 10 * (size_t)t, bb);
            refactored(bb, dB, fk);
          }
        }
        T qo[QR];
        solve_body(fk, s, m, rb, q, skip_local, v.polar, t, qo);
        if (k == K - 1) residual_terms(m, qo, q, &num, &den);
        settle<QR>(qo);
        Q::put(lq, t, qo);
#pragma unroll
        for (int c = 0; c < QR; ++c) q[c] = qo[c];
      }
      __syncthreads();
    }
    if (free) {
      resident_recover(q, qn, (T)(1.0 / S.h), vw, v.health);
#pragma unroll
      for (int c = 0; c < QR; ++c) qn[c] = q[c];
    }
  }
  if (free) {
    store<T, QR>(v.qn + (size_t)QR * t, qn);
    store<T, VW>(v.vel + (size_t)VW * t, vw);
  }
  if constexpr (VARIABLE) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (eo[u] >= 0 && (eo[u] & 1)) {
        const size_t e = t + u * NT;
        store<T, 4>(v.al + 4 * e, al[u]);
        v.se[EW * e + 7] = E[u][7];
      }
  }
  double* red = reinterpret_cast<double*>(lq);  // the buffer is done with
  red[t] = num;
  red[NT + t] = den;
  __syncthreads();
  resident_finish<NT>(red, red + NT, v.rho, &v.scenes[0].step, step0 + nsteps);
}

// One step of a contact scene of at most NT / 4 bodies.  Thread t forms the terms
// of ends t % 4, t % 4 + 4, ... of body t / 4 (the first U contacts of them held in
// registers through the step) and the four lanes' sum goes to LDS; then thread
// b solves body b, with full waves instead of every fourth lane.  U is two, or one
// where two waves share a SIMD's registers in FP64 (a heap of 100 boxes, us per step: 260
// with two, which spill 184 bytes a lane, 193 with one and no spills).
template <typename T, int NT, bool GENERAL>
__global__ void __launch_bounds__(NT) k_resident_contact(View<T> v, int n, int ccap, DrivenTable dt) {
  constexpr int QR = Rec<T>::Q, W = ContactRec<T>::W, NB = NT / 4;
  constexpr int U = sizeof(T) == 8 && NT > 256 ? 1 : 2;
  using Q = Plane<T, QR, NB>;
  using M = Plane<T, MW, NB>;
  using F = Plane<T, FW, NB>;
  using D = Plane<double, 10, NB>;
  __shared__ __align__(16) T lq[Q::N], ls[Q::N], lm[M::N], lf[F::N], lr[F::N];
  __shared__ __align__(16) double lb[D::N], ld[D::N];
  __shared__ int lflag[NB];
  __shared__ double red[2 * NT];
  const int t = threadIdx.x, be = t / 4, sub = t % 4;
  const SceneDev& S = v.scenes[0];
  const int K = S.iters, step0 = S.step;
  const bool skip_local = (S.debug & 1) != 0;
  const bool body = t < n;          // this thread solves body t
  bool free = false;
  if constexpr (GENERAL) {
    if (dt.n > 0) {
      for (int b = t; b < dt.n; b += NT) update_driven_entry(v, b, step0, S, dt.end_i, dt.end_j, dt.param);
      __syncthreads();
      if (body && !(v.flags[t] & F_PINNED)) factor_body(v, dt.mass64, t);
      __syncthreads();
    }
  }
  if (body) {
    T q[QR];
    load<T, QR>(v.qn + (size_t)QR * t, q);
    free = (v.flags[t] & F_PINNED) == 0;
    if (free) {
      T vw[VW], s[QR], x[FW];
      load<T, VW>(v.vel + (size_t)VW * t, vw);
      resident_predict(S, q, vw, s);
      Q::put(lq, t, s);
      Q::put(ls, t, s);
      load<T, MW>(v.mass + (size_t)MW * t, x);
      M::put(lm, t, x);
      load<T, FW>(v.fac + (size_t)FW * t, x);
      F::put(lf, t, x);
      double b10[10];
      load<double, 10>(v.blk + 10 * (size_t)t, b10);
      D::put(lb, t, b10);
      if constexpr (GENERAL) {
        if (v.flags[t] & F_VARIABLE) {  // augmented ends, warm start (Sec. 5.2.2)
          const T ga = (T)S.al_gamma, ag = (T)(S.al_alpha * S.al_gamma);
          for (int e = v.srow[t]; e < v.srow_end[t]; ++e) {
            T* a = v.al + 4 * (size_t)e;
            if (!(a[3] > (T)0)) continue;
            a[0] = fmax(ga * a[0], a[3]);
            a[1] = ag * a[1];
          }
        }
      }
    } else {
      Q::put(lq, t, q);
    }
  }
  // the ends of body be
  int cnt = 0, e0 = 0, e1 = 0;
  bool var = false;
  const size_t base = (size_t)be * ccap;
  T C[U][W];
  int id[U];
  if (be < n) {
    const uint8_t fl = v.flags[be];
    var = (fl & F_VARIABLE) != 0;
    if (!(fl & F_PINNED)) {
      cnt = min(v.ccount[be], ccap);
      e0 = v.srow[be];
      e1 = v.srow_end[be];
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (sub + 4 * u < cnt) {
      id[u] = v.ce_partner[base + sub + 4 * u];
      load<T, W>(v.ce + (size_t)W * (base + sub + 4 * u), C[u]);
    }
  const T mu = (T)S.mu;
  __syncthreads();
  double num = 0.0, den = 0.0;
  for (int k = 0; k < K; ++k) {
    if (cnt > 0 || e0 < e1) {
      auto state = [&](int j, T* qj) { Q::get(lq, j, qj); };
      T q[QR], rb[FW];
      Q::get(lq, be, q);
#pragma unroll
      for (int c = 0; c < FW; ++c) rb[c] = (T)0;
      bool refactor = false;
      Block dB{};
      if constexpr (GENERAL)
        general_ends<T, 4>(v, S, e0 + sub, e1, var, k == K - 1, q, state, rb, dB, refactor);
      else
        quadratic_ends<T, 4>(v, e0 + sub, e1, q, state, rb);
      T qj[U][QR];
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (sub + 4 * u < cnt && id[u] >= 0) state(id[u], qj[u]);
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (sub + 4 * u < cnt) contact_end(C[u], id[u], q, qj[u], mu, rb, dB, refactor);
      for (int c = sub + 4 * U; c < cnt; c += 4) {
        const int j = v.ce_partner[base + c];
        T R[W], qc[QR];
        load<T, W>(v.ce + (size_t)W * (base + c), R);
        if (j >= 0) state(j, qc);
        contact_end(R, j, q, qc, mu, rb, dB, refactor);
      }
      sum_lanes<T, 4>(rb, dB, refactor);
      if (sub == 0) {
        F::put(lr, be, rb);
        lflag[be] = refactor ? 1 : 0;
        if (refactor) {
          const double d10[10] = {dB.a, dB.b0, dB.b1, dB.b2, dB.d00, dB.d01, dB.d02, dB.d11, dB.d12, dB.d22};
          D::put(ld, be, d10);
        }
      }
    } else if (be < n && sub == 0) {
      T rb[FW];
#pragma unroll
      for (int c = 0; c < FW; ++c) rb[c] = (T)0;
      F::put(lr, be, rb);
      lflag[be] = 0;
    }
    __syncthreads();
    if (free) {
      T q[QR], s[QR], m[MW], rb[FW], fac[FW], qo[QR];
      Q::get(lq, t, q);
      Q::get(ls, t, s);
      M::get(lm, t, m);
      F::get(lr, t, rb);
      if (lflag[t]) {
        double bb[10], d[10];
        D::get(lb, t, bb);
        D::get(ld, t, d);
        refactored(bb, Block{d[0], d[1], d[2], d[3], d[4], d[5], d[6], d[7], d[8], d[9]}, fac);
      } else {
        F::get(lf, t, fac);
      }
      solve_body(fac, s, m, rb, q, skip_local, v.polar, t, qo);
      if (k == K - 1) residual_terms(m, qo, q, &num, &den);
      Q::put(lq, t, qo);
    }
    __syncthreads();
  }
  if (free) {
    T q[QR], qn[QR], vw[VW];
    Q::get(lq, t, q);
    load<T, QR>(v.qn + (size_t)QR * t, qn);
    resident_recover(q, qn, (T)(1.0 / S.h), vw, v.health);
    store<T, QR>(v.qn + (size_t)QR * t, q);
    store<T, VW>(v.vel + (size_t)VW * t, vw);
  }
  red[t] = num;
  red[NT + t] = den;
  __syncthreads();
  resident_finish<NT>(red, red + NT, v.rho, &v.scenes[0].step, step0 + 1);
}

}  // namespace pabd
