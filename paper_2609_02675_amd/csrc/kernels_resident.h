// kernels_resident.h -- whole steps of one small scene in one workgroup: the
// prediction, the K global/local Jacobi iterations of Algorithm 1 and the
// velocity recovery of a plain handle's scene whose bodies fit the workgroup.
// The bodies exchange q^k through LDS and everything a step does not change
// stays in registers and LDS, so an iteration waits on no global load.
//
//   k_resident_joints   a scene without contacts, one lane per body: any number of
//                       steps in one launch (nothing is built between them)
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
// rotation), not any throughput; the contact kernel with more than four
// waves is bound by their instruction issue on the one compute unit, so larger
// piles take the flat kernels (EngineT::resident_max).
//
// Measured per step, against one kernel that read records, masses, factors and the
// scene from memory in every iteration behind barriers of 16 waves (and took a
// launch per step): eight-body chain 0.044 -> 0.025 ms (FP64 0.066 -> 0.051),
// chain of 200 0.057 -> 0.027, of 500 0.075 -> 0.040, of 1,000 0.101 -> 0.085,
// slider crank 0.106 -> 0.079, 11 x 11 net of order 4 in FP64 0.164 -> 0.090, pile
// of 16 boxes 0.118 -> 0.095, of 60 0.134 -> 0.111 with its contact construction.
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
  const int *scene, *end_i, *end_j;
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

// nsteps steps of a scene of at most NT bodies without contacts.  GENERAL: the scene
// has variable or driven bonds.  The first ends of a body (two; of a GENERAL scene
// as many as fit LDS, with their states) are read once per launch, or per step
// when driven bonds move them; any further ones from global memory as they are
// needed.
template <typename T, int NT, bool GENERAL>
__global__ void __launch_bounds__(NT) k_resident_joints(View<T> v, int n, int nsteps, DrivenTable dt) {
  constexpr int QR = Rec<T>::Q;
  constexpr bool HOLD = Resident<T>::hold(NT);
  using Q = Plane<T, QR, NT>;
  // ends per body held in LDS: what the buffers of q leave, at most 8
  constexpr int END_BYTES = 12 * sizeof(T) + 4;
  constexpr int ROOM = (150 * 1024 - 2 * Q::N * (int)sizeof(T)) / (NT * END_BYTES);
  constexpr int ME = !HOLD ? 0 : !GENERAL ? 2 : (ROOM < 8 ? ROOM : 8);
  constexpr int SLOTS = GENERAL && ME > 0 ? ME * NT : 1;
  using ES = Plane<T, EW, SLOTS>;
  using AS = Plane<T, 4, SLOTS>;
  __shared__ __align__(16) T lq[2][Q::N];
  __shared__ __align__(16) T le[GENERAL ? ES::N : 4], la[GENERAL ? AS::N : 4];
  __shared__ int lp[SLOTS];
  const int t = threadIdx.x;
  const SceneDev& S = v.scenes[0];
  const int K = S.iters, step0 = S.step;
  const bool skip_local = (S.debug & 1) != 0;
  const bool body = t < n;
  T qn[QR], vw[VW], m[MW], fac[FW], E[GENERAL ? 1 : 2][EW];
  double bb[GENERAL ? 10 : 1];
  int id[GENERAL ? 1 : 2];
  int e0 = 0, ne = 0;
  bool free = false, var = false;
  if (body) {
    load<T, QR>(v.qn + (size_t)QR * t, qn);
    load<T, VW>(v.vel + (size_t)VW * t, vw);
    if constexpr (HOLD) load<T, MW>(v.mass + (size_t)MW * t, m);
    const uint8_t fl = v.flags[t];
    free = (fl & F_PINNED) == 0;
    var = (fl & F_VARIABLE) != 0;
    e0 = v.srow[t];
    ne = free ? v.srow_end[t] - e0 : 0;
    if constexpr (HOLD) {
      if (free) load<T, FW>(v.fac + (size_t)FW * t, fac);
    }
    if constexpr (HOLD && GENERAL) {
      if (free) load<double, 10>(v.blk + 10 * (size_t)t, bb);
    } else if constexpr (HOLD) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
        if (u < ne) {
          id[u] = v.se_partner[e0 + u];
          load<T, EW>(v.se + (size_t)EW * (e0 + u), E[u]);
        }
    }
  }
  auto stage_ends = [&]() {
    if constexpr (GENERAL && ME > 0) {
      for (int u = 0; u < ME && u < ne; ++u) {
        T r[EW];
        load<T, EW>(v.se + (size_t)EW * (e0 + u), r);
        ES::put(le, u * NT + t, r);
        lp[u * NT + t] = v.se_partner[e0 + u];
      }
    }
  };
  stage_ends();
  if constexpr (GENERAL && ME > 0) {
    for (int u = 0; u < ME && u < ne; ++u) {
      T a[4] = {(T)0, (T)0, (T)0, (T)0};
      if (var) load<T, 4>(v.al + 4 * (size_t)(e0 + u), a);
      AS::put(la, u * NT + t, a);
    }
  }
  if (body && !free) {  // a pinned body keeps q^n, in both buffers
    Q::put(lq[0], t, qn);
    Q::put(lq[1], t, qn);
  }
  double num = 0.0, den = 0.0;
  for (int st = 0; st < nsteps; ++st) {
    if constexpr (GENERAL) {
      if (dt.n > 0) {
        // driven anchors at this step's time, then every block of the scene
        // refactored (the same functions as the flat path's kernels)
        for (int b = t; b < dt.n; b += NT)
          update_driven_entry(v, b, step0 + st, S, dt.end_i, dt.end_j, dt.param);
        __syncthreads();
        if (body && free) {
          factor_body(v, dt.mass64, t);
          if constexpr (HOLD) {
            load<T, FW>(v.fac + (size_t)FW * t, fac);
            load<double, 10>(v.blk + 10 * (size_t)t, bb);
          }
          // the anchors that moved; a slider's E[7] lives in LDS between steps
          for (int u = 0; u < ME && u < ne; ++u) {
            T r[EW], x[EW];
            load<T, EW>(v.se + (size_t)EW * (e0 + u), r);
            ES::get(le, u * NT + t, x);
            r[7] = x[7];
            ES::put(le, u * NT + t, r);
          }
        }
      }
    }
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
      if constexpr (GENERAL) {
        if (var) {  // augmented ends, warm start (Sec. 5.2.2), as in the flat path's prediction
          const T ga = (T)S.al_gamma, ag = (T)(S.al_alpha * S.al_gamma);
          for (int u = 0; u < ne; ++u) {
            T a[4];
            if (u < ME)
              AS::get(la, u * NT + t, a);
            else
              load<T, 4>(v.al + 4 * (size_t)(e0 + u), a);
            if (!(a[3] > (T)0)) continue;
            a[0] = fmax(ga * a[0], a[3]);
            a[1] = ag * a[1];
            if (u < ME)
              AS::put(la, u * NT + t, a);
            else
              store<T, 4>(v.al + 4 * (size_t)(e0 + u), a);
          }
        }
      }
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
        bool refactor = false;
        Block dB{};
        if constexpr (GENERAL) {
          for (int u = 0; u < ME && u < ne; ++u) {
            const int x = u * NT + t, j = lp[x];
            T R[EW], a[4], qj[QR];
            ES::get(le, x, R);
            AS::get(la, x, a);
            if (j >= 0) state(j, qj);
            general_end(R, a, j, q, qj, S, k == K - 1, rb, dB, refactor);
            if (a[3] > (T)0)
              AS::put(la, x, a);
            else if (k == K - 1 && a[3] != (T)0)
              ES::put(le, x, R);
          }
          if (ne > ME)
            general_ends<T, 1>(v, S, e0 + ME, e0 + ne, var, k == K - 1, q, state, rb, dB, refactor);
        } else if constexpr (!HOLD) {
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
        if constexpr (GENERAL) {
          if (refactor) {
            if constexpr (!HOLD) load<double, 10>(v.blk + 10 * (size_t)t, bb);
            refactored(bb, dB, fk);
          }
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
  if (free) {
    if constexpr (HOLD) {
      store<T, QR>(v.qn + (size_t)QR * t, qn);
      store<T, VW>(v.vel + (size_t)VW * t, vw);
    }
    if constexpr (GENERAL && ME > 0) {
      if (var)
        for (int u = 0; u < ME && u < ne; ++u) {
          T a[4], R[EW];
          AS::get(la, u * NT + t, a);
          ES::get(le, u * NT + t, R);
          store<T, 4>(v.al + 4 * (size_t)(e0 + u), a);
          v.se[(size_t)EW * (e0 + u) + 7] = R[7];
        }
    }
  }
  double* red = reinterpret_cast<double*>(&lq[0][0]);  // the buffers are done with
  red[t] = num;
  red[NT + t] = den;
  __syncthreads();
  resident_finish<NT>(red, red + NT, v.rho, &v.scenes[0].step, step0 + nsteps);
}

// One step of a contact scene of at most NT / 4 bodies.  Thread t forms the terms
// of ends t % 4, t % 4 + 4, ... of body t / 4 (the first two of them held in
// registers through the step) and the four lanes' sum goes to LDS; then thread
// b solves body b, with full waves instead of every fourth lane.
template <typename T, int NT, bool GENERAL>
__global__ void __launch_bounds__(NT) k_resident_contact(View<T> v, int n, int ccap, DrivenTable dt) {
  constexpr int QR = Rec<T>::Q, W = ContactRec<T>::W, NB = NT / 4, U = 2;
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
