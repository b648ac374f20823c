// kernels_flat.h -- the body iteration of the flat path (Algorithm 1's global
// and local step for one body) and the kernels that run it over a flat range
// of bodies:
//   k_iterate   one global + local iteration for every body (Jacobi: reads only
//               q^k, writes q^{k+1} to the other buffer), increment form:
//               dq = H^{-1} (M (s - q^k) + h^2 sum [w J^T (y_o - y_s) + phi^- J^T n
//                    + J^T f_contact]),  then A <- polar rotation (Sec. 4.2.2)
//   k_iterate_waves  the same over a batch's table of wavefronts (CL lanes per
//               body of a contact scene, one per body of any other scene)
// with the force terms of the variable ends (augmented, polynomial, slider) and
// of the contact ends.  The resident step kernel forms its iteration from the
// same pieces.
#pragma once

#include "common.h"
#include "contact_record.h"
#include "device_math.h"
#include "kernels_step.h"

namespace pabd {

// one augmented end (Sec. 5.2.2) with bond vector d = y_o - y_s at iterate k:
// h^2-scaled force and implicit weight of Psi = 1/2 kappa C^2 + lambda C, C = d - l
// (the multiplier's tension beyond kappa l joins the weight), then the
// multiplier and stiffness updates from C; a = (kappa, lambda, l, kappa_start)
template <typename T>
__device__ __forceinline__ T augmented_end(T* a, const T* d, T h2, T beta, T* f) {
  const T kap = a[0], lam = a[1], l = a[2];
  const T dn = sqrt(dot_fused(d, d));
  T w = kap, phim = lam - kap * l;
  if (phim > (T)0 && dn > (T)1e-12) {
    w += phim / dn;
    phim = (T)0;
  }
  const T sc = dn > (T)1e-12 ? phim / dn : (T)0;
  f[0] = h2 * (w + sc) * d[0];
  f[1] = h2 * (w + sc) * d[1];
  f[2] = h2 * (w + sc) * d[2];
  const T C = dn - l;
  a[1] = kap * C + lam;
  a[0] = kap + beta * fabs(C);
  return h2 * w;  // implicit weight (h^2-scaled) for the block
}

// one polynomial end, Psi = kappa / p (d - l)^p (p even, at most 12): phi =
// kappa (d - l)^{p-1} = kappa sum_k C(p-1, k) d^k (-l)^{p-1-k}; the terms with
// p-1-k even are >= 0 and form phi^+ (implicit weight phi^+ / d), the others
// phi^- (explicit) -- the split of Sec. 4.2.1; a = (kappa, 0, l, -p)
//
// The sums for one order, every coefficient known at compile time (all are
// whole numbers below 2^9, so forming them ahead changes no bit).
template <int P, typename T>
__device__ __forceinline__ void polynomial_sums(T l, T dn, T* w_out, T* phim_out) {
  T lp[P];  // l^j
  lp[0] = (T)1;
#pragma unroll
  for (int j = 1; j < P; ++j) lp[j] = lp[j - 1] * l;
  int binom = 1;
  T dk1 = (T)1, w = (T)0, phim = (T)0;  // dk1 = d^{k-1}
#pragma unroll
  for (int k = 0; k < P; ++k) {
    if (k > 0) binom = binom * (P - k) / k;
    const int j = P - 1 - k;
    if (j % 2 == 0) {
      if (k >= 1) w += (T)binom * dk1 * lp[j];
    } else {
      phim -= (T)binom * (k >= 1 ? dk1 * dn : (T)1) * lp[j];
    }
    if (k >= 1) dk1 *= dn;
    settle<1>(&dk1);
  }
  *w_out = w;
  *phim_out = phim;
}
template <typename T>
__device__ __forceinline__ T polynomial_end(const T* a, const T* d, T h2, T* f) {
  const T kap = a[0];
  T l = a[2];
  settle<1>(&l);  // no power of it taken ahead of a caller's loop
  const T dn = sqrt(dot_fused(d, d));
  T w = (T)0, phim = (T)0;
  switch ((int)(-a[3])) {
    case 2: polynomial_sums<2>(l, dn, &w, &phim); break;
    case 4: polynomial_sums<4>(l, dn, &w, &phim); break;
    case 6: polynomial_sums<6>(l, dn, &w, &phim); break;
    case 8: polynomial_sums<8>(l, dn, &w, &phim); break;
    case 10: polynomial_sums<10>(l, dn, &w, &phim); break;
    default: polynomial_sums<12>(l, dn, &w, &phim); break;
  }
  w *= kap;
  phim *= kap;
  const T sc = dn > (T)1e-12 ? phim / dn : (T)0;
  f[0] = h2 * (w + sc) * d[0];
  f[1] = h2 * (w + sc) * d[1];
  f[2] = h2 * (w + sc) * d[2];
  return h2 * w;
}

// one slider end (the point-on-line reading of the slider joint of Sec. 5.1).
// d0 = y_o - y_s is the record's bond vector (point side: from the point to the
// line's anchor on the partner; line side: from the own line anchor to the
// partner's point); g = A u is the line's world direction (u the unit axis in
// the line body's frame, A that body's iterate, or u itself for a world line).
// Sets d to the part of d0 across g -- on either side the vector from this end's
// point to the other, with the line-side point at the foot of the
// perpendicular -- and returns t = d0.g / g.g, the foot's distance along u from
// the line anchor as seen from the line side.
template <typename T>
__device__ __forceinline__ T slider_end(const T* d0, const T* A, const T* u, T* d) {
  T g[3];
#pragma unroll
  for (int r = 0; r < 3; ++r) g[r] = A ? dot_fused(A + 3 * r, u) : u[r];
  T t = dot_fused(d0, g) / dot_fused(g, g);
  settle<1>(&t);
#pragma unroll
  for (int r = 0; r < 3; ++r) d[r] = d0[r] - t * g[r];
  return t;
}

// contact end (reading of the paper's contact bond), d = y_o - y_s: stick force
// kappa d acting only while penetrating along n (n from the partner's surface
// towards the owner), tangential part clamped to mu times the normal part; kap
// is h^2 kappa, so the force comes out scaled by h^2 like the bonds'.
// Returns false when separated (no contribution, no implicit weight).
template <typename T>
__device__ __forceinline__ bool contact_end_force(T kap, T mu, const T* n, const T* d, T* f) {
  const T d0 = d[0], d1 = d[1], d2 = d[2];
  const T n0 = n[0], n1 = n[1], n2 = n[2];
  T dn = dot_fused(n, d);  // = -gap
  if (!(dn > (T)0)) return false;
  T fn = kap * dn;
  T t0 = kap * fma(-dn, n0, d0), t1 = kap * fma(-dn, n1, d1), t2 = kap * fma(-dn, n2, d2);
  T tn2 = fma(t2, t2, fma(t0, t0, t1 * t1));
  T lim = mu * fn;
  if (tn2 > lim * lim) {
    T sc = lim * rsqrt_(tn2);
    t0 *= sc;
    t1 *= sc;
    t2 *= sc;
  }
  f[0] = fma(fn, n0, t0);
  f[1] = fma(fn, n1, t1);
  f[2] = fma(fn, n2, t2);
  return true;
}

// residual partials of one body: |q_new - q|_M^2 and |q|_M^2
template <typename T>
__device__ __forceinline__ void residual_terms(const T* m, const T* qo, const T* q, double* num,
                                               double* den) {
  T dd[QW];
  pos_diff(qo, q, dd);
#pragma unroll
  for (int c = 3; c < QW; ++c) dd[c] = qo[c] - q[c];
  const T cc[3] = {(T)pos_value(q, 0), (T)pos_value(q, 1), (T)pos_value(q, 2)};
  *num = m_norm2(m, dd, dd);
  *den = m_norm2(m, cc, q);
}

// sum over the LPB consecutive lanes of a body (2, 4, 8 or 16, aligned): pairs,
// quads, then mirrored halves of eight and sixteen, whose lanes already agree
// within each half, so a mirrored lane stands for any lane of the other half.
// Every lane gets the same bits, since each partial sum is formed from the same
// two operands.
template <int LPB, typename U>
__device__ __forceinline__ U lane_sum(U x) {
  if constexpr (LPB >= 2) x += lane_of<0xB1>(x);    // quad_perm 1 0 3 2
  if constexpr (LPB >= 4) x += lane_of<0x4E>(x);    // quad_perm 2 3 0 1
  if constexpr (LPB >= 8) x += lane_of<0x141>(x);   // row_half_mirror
  if constexpr (LPB >= 16) x += lane_of<0x140>(x);  // row_mirror
  return x;
}

// The pieces of one Jacobi iteration of a body, shared by the flat kernels and
// the resident step so that both round alike: a static end (quadratic, or of any
// kind), a contact end, the sum across the lanes that share the body, and the
// solve with the local step.

// one quadratic static end
template <typename T>
__device__ __forceinline__ void quadratic_end(const T* E, int j, const T* q, const T* qj, T* rb) {
  T d[3], f[3];
  bond_vec<T>(q, E, j < 0 ? (const T*)nullptr : qj, E + 4, d);
  quad_end_force(E, d, f);
  settle<3>(f);
  add_JT(rb, E, f[0], f[1], f[2]);
  settle<QW>(rb);
}

// forces of the static ends e, e + LPB, ... below e1, quadratic ends only, two
// ends per round with both ends' loads (record and partner state) in flight
// together; each end's terms are added in end order.  state(j, qj) loads a
// partner's q^k.
template <typename T, int LPB, typename State>
__device__ __forceinline__ void quadratic_ends(const View<T>& v, int e, int e1, const T* q, State state, T* rb) {
  constexpr int QR = Rec<T>::Q;
  for (; e < e1; e += 2 * LPB) {
    const int eb = e + LPB;
    const bool hb = eb < e1;
    const int ja = v.se_partner[e];
    const int jb = hb ? v.se_partner[eb] : -1;
    T Ea[EW], Eb[EW], qa[QR], qb[QR];
    load<T, EW>(v.se + (size_t)EW * e, Ea);
    if (hb) load<T, EW>(v.se + (size_t)EW * eb, Eb);
    if (ja >= 0) state(ja, qa);
    if (jb >= 0) state(jb, qb);
    quadratic_end(Ea, ja, q, qa, rb);
    if (hb) quadratic_end(Eb, jb, q, qb, rb);
  }
}

// the terms of one static end of any kind, record E and, for a body with variable
// ends, its state a (else zeros), partner j (-1: the world) at qj: the force g f, the
// own point x it acts at and, for an end whose weight or point moves (then true is
// returned), its weight w in the block.  An augmented end's multiplier and
// stiffness move on in a, a slider's anchor, in the step's last iteration, in E[7].
template <typename T>
__device__ __forceinline__ bool end_terms(T* E, T* a, int j, const T* q, const T* qj, T h2, T beta, bool last, T* f,
                                          T* g, T* x, T* w) {
  const T kind = a[3];
  x[0] = E[0];
  x[1] = E[1];
  x[2] = E[2];
  *w = (T)0;
  *g = (T)1;
  // a slider end's line anchor sits t0 = E[7] along the axis from the given
  // one (a slider's rest length is 0, so E[7] holds no phi^-): the same line,
  // re-anchored near the point every step so that the bond vector, whose
  // across-axis part is the force, stays short (in FP32 a long one would lose
  // that part to rounding)
  T xs[3] = {E[0], E[1], E[2]}, xo[3] = {E[4], E[5], E[6]};
  if (kind == (T)AL_SLIDER_POINT) {
#pragma unroll
    for (int r = 0; r < 3; ++r) xo[r] = fma(E[7], a[r], xo[r]);
  } else if (kind == (T)AL_SLIDER_LINE) {
#pragma unroll
    for (int r = 0; r < 3; ++r) xs[r] = fma(E[7], a[r], xs[r]);
  }
  T d[3];
  bool moves = false;
  bond_vec<T>(q, xs, j < 0 ? (const T*)nullptr : qj, xo, d);
  settle<3>(d);
  if (kind == (T)AL_SLIDER_POINT) {
    // fixed weight at the own point (in the static block), drawn to the foot
    const T t = slider_end(d, j < 0 ? (const T*)nullptr : qj + 3, a, f);
    *g = E[3];
    if (last) E[7] = E[7] - t;  // the foot is -t from the anchor
  } else if (kind == (T)AL_SLIDER_LINE) {
    // the own point is the foot xf = x_s + t u, so its weight moves every iteration
    const T t = slider_end(d, q + 3, a, f);
#pragma unroll
    for (int r = 0; r < 3; ++r) x[r] = fma(t, a[r], xs[r]);
    *g = *w = E[3];
    moves = true;
    if (last) E[7] = E[7] + t;
  } else if (kind != (T)0) {
    *w = kind > (T)0 ? augmented_end(a, d, h2, beta, f) : polynomial_end(a, d, h2, f);
    moves = true;
  } else {
    quad_end_force(E, d, f);
  }
  settle<3>(f);
  settle<1>(g);
  settle<3>(x);
  settle<1>(w);
  return moves;
}

// an end's terms added: force (times 1 rounds to itself), and block change of an end
// that moves
template <typename T>
__device__ __forceinline__ void add_scaled(T* rb, const T* x, T g, const T* f) {
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    T y = g * f[r];
    settle<1>(&y);
    rb[r] = fma(g, f[r], rb[r]);
#pragma unroll
    for (int c = 0; c < 3; ++c) rb[3 + 3 * r + c] = fma(y, x[c], rb[3 + 3 * r + c]);
  }
  settle<QW>(rb);
}
template <typename T>
__device__ __forceinline__ void add_moved(bool moves, T w, const T* x, Block& dB) {
  if (moves) block_add_end(dB, (double)w, (double)x[0], (double)x[1], (double)x[2]);
  settle_block(dB);
}
template <typename T>
__device__ __forceinline__ void general_end(T* E, T* a, int j, const T* q, const T* qj, const SceneDev& S, bool last,
                                            T* rb, Block& dB, bool& refactor) {
  T f[3], g, x[3], w;
  const bool moves = end_terms(E, a, j, q, qj, (T)(S.h * S.h), (T)S.al_beta, last, f, &g, x, &w);
  add_scaled(rb, x, g, f);
  add_moved(moves, w, x, dB);
  refactor = refactor || moves;
}

// forces of the static ends e, e + LPB, ... below e1 of any kind, from global
// memory, one at a time: every end's terms are formed with the same operations
// in the same order as above.  var: the body owns variable ends; state(j, qj)
// loads the partner's q^k; `last`: the step's last iteration.
template <typename T, int LPB, typename State>
__device__ __forceinline__ void general_ends(const View<T>& v, const SceneDev& S, int e, int e1, bool var, bool last,
                                             const T* q, State state, T* rb, Block& dB, bool& refactor) {
  for (; e < e1; e += LPB) {
    const int j = v.se_partner[e];
    T E[EW], a[4] = {(T)0, (T)0, (T)0, (T)0}, qj[Rec<T>::Q];
    load<T, EW>(v.se + (size_t)EW * e, E);
    if (var) load<T, 4>(v.al + 4 * (size_t)e, a);
    if (j >= 0) state(j, qj);
    general_end(E, a, j, q, qj, S, last, rb, dB, refactor);
    if (a[3] > (T)0) {
      v.al[4 * (size_t)e] = a[0];
      v.al[4 * (size_t)e + 1] = a[1];
    } else if (last && (a[3] == (T)AL_SLIDER_POINT || a[3] == (T)AL_SLIDER_LINE)) {
      v.se[(size_t)EW * e + 7] = E[7];
    }
  }
}

// one contact end: record C, partner j (-1: a plane) at qj
template <typename T>
__device__ __forceinline__ void contact_end(const T* C, int j, const T* q, const T* qj, T mu, T* rb, Block& dB,
                                            bool& refactor) {
  T d[3], f[3], n[3], kap;
  bond_vec<T>(q, C, j < 0 ? nullptr : qj, C + 4, d);
  if constexpr (sizeof(T) == 4) {
    // h^2 kappa from the two q records, the normal from its octahedral form
    kap = fmax(q[Q_KAPPA], j < 0 ? (T)0 : qj[Q_KAPPA]);
    oct_decode(C[3], C[7], n);
  } else {
    kap = C[3];
    settle<1>(&kap);  // no product of the record's own values taken ahead of a caller's loop
    n[0] = C[8];
    n[1] = C[9];
    n[2] = C[10];
  }
  if (!contact_end_force(kap, mu, n, d, f)) return;
  add_JT(rb, C, f[0], f[1], f[2]);
  block_add_end(dB, (double)kap, (double)C[0], (double)C[1], (double)C[2]);
  settle<QW>(rb);
  settle_block(dB);
  refactor = true;
}

// the force terms and the block change summed over the lanes of a body
template <typename T, int LPB>
__device__ __forceinline__ void sum_lanes(T* rb, Block& dB, bool& refactor) {
  if constexpr (LPB > 1) {
#pragma unroll
    for (int c = 0; c < QW; ++c) rb[c] = lane_sum<LPB>(rb[c]);
    refactor = lane_sum<LPB>(refactor ? 1 : 0) > 0;
    if (refactor) {  // uniform across the body's lanes
      dB.a = lane_sum<LPB>(dB.a);
      dB.b0 = lane_sum<LPB>(dB.b0);
      dB.b1 = lane_sum<LPB>(dB.b1);
      dB.b2 = lane_sum<LPB>(dB.b2);
      dB.d00 = lane_sum<LPB>(dB.d00);
      dB.d01 = lane_sum<LPB>(dB.d01);
      dB.d02 = lane_sum<LPB>(dB.d02);
      dB.d11 = lane_sum<LPB>(dB.d11);
      dB.d12 = lane_sum<LPB>(dB.d12);
      dB.d22 = lane_sum<LPB>(dB.d22);
    }
  }
}

// the factor of H^k = H + dB from the static block bb (10 doubles)
template <typename T>
__device__ __forceinline__ void refactored(const double* bb, const Block& dB, T* fac) {
  const Block B{bb[0] + dB.a,   bb[1] + dB.b0,  bb[2] + dB.b1,  bb[3] + dB.b2,  bb[4] + dB.d00,
                bb[5] + dB.d01, bb[6] + dB.d02, bb[7] + dB.d11, bb[8] + dB.d12, bb[9] + dB.d22};
  double f64[10];
  block_inverse(B, f64);
#pragma unroll
  for (int c = 0; c < 10; ++c) fac[c] = (T)f64[c];
}

// global and local step of one body: qo = q^{k+1} from q = q^k, its summed force
// terms rb (scaled by h^2), s, masses and factor
template <typename T>
__device__ __forceinline__ void solve_body(const T* fac, const T* s, const T* m, const T* rb, const T* q,
                                           bool skip_local, unsigned* polar, int i, T* qo) {
  constexpr int QR = Rec<T>::Q;
  T r[QW];  // M (s - q^k) + h^2 sum (...)
#pragma unroll
  for (int c = 0; c < QW; ++c) r[c] = rb[c];
  settle<QW>(r);
  add_inertia(r, m, s, q);
  T dq[QW];
  block_apply(fac, r, dq);
#pragma unroll
  for (int c = 0; c < QR; ++c) qo[c] = q[c];
  pos_add_lo(qo, dq[0], dq[1], dq[2]);
  T Ah[9];
#pragma unroll
  for (int c = 0; c < 9; ++c) Ah[c] = q[3 + c] + dq[3 + c];
  if (skip_local) {
#pragma unroll
    for (int c = 0; c < 9; ++c) qo[3 + c] = Ah[c];
  } else {
    polar_rotation(Ah, qo + 3, polar, i);
  }
}

// One Jacobi iteration of the flat path for body i (Algorithm 1's global and
// local step; reads q^k of every body, writes q^{k+1} to the other buffer), LPB
// lanes per body.  A launch covers one iteration, and a kernel boundary leaves
// nothing in the caches nearest the compute units, so what a small scene waits
// for is the chain of loads that need one another's results.  The chain has two
// links: everything whose address follows from the body's index (its state,
// count of contact ends, factor, block, masses, the partner ids and records of
// its first ends -- slots beyond the count hold no end, but lie in the body's
// own range), then the partners' states.  `base` is the body's first contact
// slot.
//
// EARLY also loads what only the solve needs at the start, and the first U ends
// of every lane before the count is known: for launches with so few waves that
// latency decides.  Otherwise the solve's operands are loaded before the sum
// across the lanes and records only for ends that exist, in fewer registers, so
// that more waves hide one another's waits.
//
// MIXED: the lanes' bodies belong to several scenes (scene, K and sc are not given).
// The scenes' entries are two more links, beside the first of the chain: nothing
// waits for them before the ends (a wait ahead of everything took 2% more of a step).
//
// Measured (FP32, per step): a 1,000-box pile 0.251 -> 0.209 ms against the chain
// of six links it had (scene id, scene, ranges, partner ids, records and states,
// solve operands), a chain of 2,000 bodies 0.119 -> 0.103; the 125,000-block
// pile, bound by the bytes of its records (4.5 TB/s), unchanged at 64 us an
// iteration.
template <typename T, bool CONTACT, int LPB, int U, bool EARLY, bool MIXED = false>
__device__ __forceinline__ void iterate_flat(const View<T>& v, const SceneDev* scene, int k, int K, double* rh_num,
                                             double* rh_den, int i, int sub, size_t base, int ccap, int sc) {
  constexpr int QR = Rec<T>::Q, W = ContactRec<T>::W;
  const T* qs = v.q[k & 1];
  T* qd = v.q[(k + 1) & 1];
  T q[QR], s[QR], m[MW], fac[FW];
  double bb[10];
  if constexpr (MIXED) {
    sc = v.bscene[i];
    scene = v.scenes + sc;
  }
  const uint8_t flags = v.flags[i];
  const int e0 = v.srow[i], e1 = v.srow_end[i];
  load<T, QR>(qs + (size_t)QR * i, q);
  const SceneDev& S = *scene;
  bool live = true;  // this scene takes iteration k
  if constexpr (MIXED) {
    K = S.step < S.steps_total ? S.iters : 0;
    live = k < K;
  }
  int cnt = 0;
  int id[U];
  T C[U][W];
  if constexpr (CONTACT) {
    cnt = v.ccount[i];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int c = sub + u * LPB;
      const size_t slot = base + (c < ccap ? c : 0);
      id[u] = v.ce_partner[slot];
      if constexpr (EARLY) load<T, W>(v.ce + (size_t)W * slot, C[u]);
    }
  }
  auto solve_operands = [&]() {
    load<T, QR>(v.s + (size_t)QR * i, s);
    load<T, MW>(v.mass + (size_t)MW * i, m);
    load<T, FW>(v.fac + (size_t)FW * i, fac);
    if constexpr (CONTACT) {
#pragma unroll
      for (int c = 0; c < 5; ++c) {
        const double2 b2 = reinterpret_cast<const double2*>(v.blk + 10 * (size_t)i)[c];
        bb[2 * c] = b2.x;
        bb[2 * c + 1] = b2.y;
      }
    }
  };
  if constexpr (EARLY) solve_operands();
  const bool pinned = (flags & F_PINNED) != 0;
  T rb[QW];
#pragma unroll
  for (int c = 0; c < QW; ++c) rb[c] = (T)0;
  bool refactor = false;
  Block dB{};  // contact and augmented part of H^k - H (this lane's ends)
  const bool var = (flags & F_VARIABLE) != 0;
  const int eb = e0 + sub, ee = pinned || !live ? eb : e1;
  // a wave with a body that has variable ends takes the general loop, any
  // other wave the quadratic loop (a divergent wave would run both loops one
  // after the other)
  auto state = [&](int j, T* qj) { load<T, QR>(qs + (size_t)QR * j, qj); };
  if (wave_any(var && !pinned && live))
    general_ends<T, LPB>(v, S, eb, ee, var, k == K - 1, q, state, rb, dB, refactor);
  else
    quadratic_ends<T, LPB>(v, eb, ee, q, state, rb);
  if constexpr (CONTACT) {
    const T mu = (T)S.mu;
    cnt = pinned ? 0 : (cnt < ccap ? cnt : ccap);
    // U ends per lane and round (neighbouring lanes take neighbouring records):
    // a round's partner states go out at once
    for (int c0 = sub; c0 < cnt; c0 += U * LPB) {
      if (c0 != sub) {
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (EARLY && c0 + u * LPB < cnt) id[u] = v.ce_partner[base + c0 + u * LPB];
      }
      T qj[U][QR];
      int idn[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = c0 + u * LPB;
        if (c < cnt) {
          if (!EARLY || c0 != sub) load<T, W>(v.ce + (size_t)W * (base + c), C[u]);
          if (id[u] >= 0) load<T, QR>(qs + (size_t)QR * id[u], qj[u]);
        }
        if constexpr (!EARLY) {
          // the next round's partner ids during this one
          const int cn = c + U * LPB;
          idn[u] = cn < cnt ? v.ce_partner[base + cn] : -1;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (c0 + u * LPB < cnt) contact_end(C[u], id[u], q, qj[u], mu, rb, dB, refactor);
      if constexpr (!EARLY) {
#pragma unroll
        for (int u = 0; u < U; ++u) id[u] = idn[u];
      }
    }
  }
  if constexpr (!EARLY) solve_operands();
  sum_lanes<T, LPB>(rb, dB, refactor);
  // H^k changed: a contact penetrates, or a variable end's weight or point moved
  if (refactor) {
    if constexpr (!CONTACT) {
#pragma unroll
      for (int c = 0; c < 10; ++c) bb[c] = v.blk[10 * (size_t)i + c];
    }
    refactored(bb, dB, fac);
  }
  if (!live) return;
  if (pinned) {
    // a pinned body's residual shares stay zero (it never moves); written in
    // the first iteration, before the step's residual reduction reads them
    if (k == 0 && sub == 0) {
      v.r_num[i] = 0.0;
      v.r_den[i] = 0.0;
    }
    return;
  }
  if (sub != 0) return;
  T qo[QR];
  solve_body(fac, s, m, rb, q, (S.debug & 1) != 0, v.polar, i, qo);
  // q^{k+1} for the partners' next iteration; after the last iteration nothing
  // reads it (the body's step ends below)
  if (k < K - 1) store<T, QR>(qd + (size_t)QR * i, qo);
  if (k == K - 1 || rh_num) {
    double num, den;
    residual_terms(m, qo, q, &num, &den);
    if (k == K - 1) {
      v.r_num[i] = num;
      v.r_den[i] = den;
    }
    if (rh_num) {
      rh_num[(size_t)k * v.n + i] = num;
      rh_den[(size_t)k * v.n + i] = den;
    }
  }
  if (k == K - 1) {
    // the end of the body's step: velocity recovery (Sec. 4.4) from q^K and
    // q^n, the health bit, and q^{n+1} = q^K with its position folded back to
    // (hi, lo) (the resident kernel ends its scenes' steps itself)
    T q0[QR], vw[VW];
    load<T, QR>(v.qn + (size_t)QR * i, q0);
    // q^K as if read back from memory: the recovery's subtractions must not
    // fuse with the local step's last products, so that the flat path rounds
    // as the resident kernel does
    settle<QR>(qo);
    recover_velocity(qo, q0, (T)(1.0 / S.h), vw);
    bool finite = true;
#pragma unroll
    for (int c = 0; c < QR; ++c) finite = finite && isfinite(qo[c]);
#pragma unroll
    for (int c = 0; c < 6; ++c) finite = finite && isfinite(vw[c]);
    if (!finite) atomicOr(v.health + sc, 1);
    pos_renorm(qo);
    store<T, QR>(v.qn + (size_t)QR * i, qo);
    store<T, VW>(v.vel + (size_t)VW * i, vw);
  }
}

// Registers: the latency variant may take as many as one wave per SIMD leaves;
// the other at most what four waves per SIMD leave in FP32 (128), two in FP64.
template <typename T, bool EARLY>
struct FlatBounds {
  static constexpr int WAVES = EARLY ? 1 : (sizeof(T) == 4 ? 4 : 2);
};
// ends per lane and round: the latency variant sixteen per body and round (at
// most four per lane), the other two per lane
template <int LPB, bool EARLY>
struct FlatRound {
  static constexpr int U = EARLY ? (LPB >= 8 ? 2 : 4) : 2;
};

// the single scene of a plain handle, n bodies, ccap contact slots per body
template <typename T, bool CONTACT, int LPB, bool EARLY>
__global__ void __launch_bounds__(256, (FlatBounds<T, EARLY>::WAVES)) k_iterate(View<T> v, int k, int K, int ccap,
                                                                            double* rh_num, double* rh_den) {
  const int t = (int)(blockIdx.x * blockDim.x + threadIdx.x);
  const int i = t / LPB, sub = t % LPB;
  if (i >= v.n) return;
  iterate_flat<T, CONTACT, LPB, FlatRound<LPB, EARLY>::U, EARLY>(v, v.scenes, k, K, rh_num, rh_den, i, sub,
                                                               (size_t)i * ccap, ccap, 0);
}

// The same iteration over a batch's table of wavefronts: a wave covers 64 / CL
// bodies of a contact scene with CL lanes each (16 with the default four), or
// 64 bodies without contacts with one lane each: of one scene, or, where the batch
// holds many small ones (MIX_WAVES), of several, whose lanes look their scenes up.
// Waves past the table's count leave at once, so the grid can stay fixed while
// scenes come and go.
template <typename T, int CL, bool EARLY>
__global__ void __launch_bounds__(256, (FlatBounds<T, EARLY>::WAVES)) k_iterate_waves(View<T> v, int k,
                                                                                  const FlatWave* waves,
                                                                                  const int* n_waves) {
  const int w = (int)(blockIdx.x * (blockDim.x / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x / 64)));
  const int l = (int)(threadIdx.x & 63);
  if (w >= *n_waves) return;
  const FlatWave fw = waves[w];
  if (k >= fw.iters) return;
  if (fw.contact) {
    const int b = l / CL;
    if (b >= fw.count) return;
    iterate_flat<T, true, CL, FlatRound<CL, EARLY>::U, EARLY>(v, v.scenes + fw.scene, k, fw.iters, nullptr, nullptr,
                                                            fw.first + b, l % CL,
                                                            (size_t)fw.ce0 + (size_t)b * fw.ccap, fw.ccap, fw.scene);
  } else {
    if (l >= fw.count) return;
    if (fw.scene >= 0)
      iterate_flat<T, false, 1, 1, EARLY>(v, v.scenes + fw.scene, k, fw.iters, nullptr, nullptr, fw.first + l, 0, 0, 0,
                                          fw.scene);
    else
      iterate_flat<T, false, 1, 1, EARLY, true>(v, nullptr, k, 0, nullptr, nullptr, fw.first + l, 0, 0, 0, 0);
  }
}

}  // namespace pabd
