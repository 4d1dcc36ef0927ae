// rr_ray.hpp -- per-ray device helpers of the march kernels: crossing
// parameters (FP64), projections of the tidal tensor, the per-cell integral
// and the debug hash.
#pragma once

// Multiply-adds are fused only within one expression (explicit fma() calls
// and a * b + c written together), never across statements: the march is
// instantiated with and without the pass logic, and both instantiations must
// round every piece the same way.
#pragma clang fp contract(on)

#include "rr_internal.hpp"

namespace rr {

// Crossing parameter of plane x_a = P for a ray p(chi) = o + chi * n:
// chi = (P - o_a) * (1/n_a), FP64, never contracted.
__device__ __forceinline__ double tplane(double P, double o, double r) {
  return __dmul_rn(__dsub_rn(P, o), r);
}

// Slab of one axis holding the ray at chi (plane spacing hl):
// t_exit < chi <= t_entry, a point on a plane belongs to the slab the ray
// moves into.  Starts from floor((o + chi n) / hl) and corrects.
__device__ __forceinline__ int start_slab(double o, double n, double r, double chi, double hl) {
  if (n == 0.0) return (int)floor(o / hl);
  int m = (int)floor((o + chi * n) / hl);
  for (int it = 0; it < 8; ++it) {
    const double t0 = tplane((double)m * hl, o, r);
    const double t1 = tplane((double)(m + 1) * hl, o, r);
    const double texit = n > 0.0 ? t0 : t1;
    const double tentry = n > 0.0 ? t1 : t0;
    if (!(texit < chi)) {
      m += (n > 0.0) ? -1 : 1;
      continue;
    }
    if (!(chi <= tentry)) {
      m += (n > 0.0) ? 1 : -1;
      continue;
    }
    break;
  }
  return m;
}

// Exit parameter of slab m on one axis (-inf when the ray never crosses it).
__device__ __forceinline__ double texit_of(int m, double o, double n, double r, double hl) {
  if (n == 0.0) return -__builtin_inf();
  const int plane = n > 0.0 ? m : m + 1;
  return tplane((double)plane * hl, o, r);
}

// Projection coefficients P_ab so that Q = sum_ab P_ab T_ab (components
// xx, yy, zz, xy, xz, yz; off-diagonals already doubled).
//   kappa : tr T - n^T T n                    (Eqs. n1n1 + n2n2)
//   gamma1: e_phi^T T e_phi - e_theta^T T e_theta  (Eq. gamma1)
//   gamma2: 2 e_phi^T T e_theta               (Eq. gamma2, flat-sky mixed term)
__device__ inline void projection(int quantity, double dx, double dy, double dz, double* P) {
  if (quantity == RR_Q_KAPPA) {
    P[0] = 1.0 - dx * dx;
    P[1] = 1.0 - dy * dy;
    P[2] = 1.0 - dz * dz;
    P[3] = -2.0 * dx * dy;
    P[4] = -2.0 * dx * dz;
    P[5] = -2.0 * dy * dz;
    return;
  }
  const double st = sqrt(dx * dx + dy * dy);
  const double cp = st > 0.0 ? dx / st : 1.0;
  const double sp = st > 0.0 ? dy / st : 0.0;
  const double ct = dz;
  const double et[3] = {ct * cp, ct * sp, -st};
  const double ep[3] = {-sp, cp, 0.0};
  if (quantity == RR_Q_GAMMA1) {
    P[0] = ep[0] * ep[0] - et[0] * et[0];
    P[1] = ep[1] * ep[1] - et[1] * et[1];
    P[2] = ep[2] * ep[2] - et[2] * et[2];
    P[3] = 2.0 * (ep[0] * ep[1] - et[0] * et[1]);
    P[4] = 2.0 * (ep[0] * ep[2] - et[0] * et[2]);
    P[5] = 2.0 * (ep[1] * ep[2] - et[1] * et[2]);
  } else {
    P[0] = 2.0 * ep[0] * et[0];
    P[1] = 2.0 * ep[1] * et[1];
    P[2] = 2.0 * ep[2] * et[2];
    P[3] = 2.0 * (ep[0] * et[1] + ep[1] * et[0]);
    P[4] = 2.0 * (ep[0] * et[2] + ep[2] * et[0]);
    P[5] = 2.0 * (ep[1] * et[2] + ep[2] * et[1]);
  }
}

// Three-point Gauss-Legendre on [chi_B, chi_A], nodes at chi_B + L * c_k.
// The integrand g(chi) * Q(p(chi)) is a polynomial of degree <= 5 in chi
// (cubic trilinear field along a line times the quadratic lensing kernel), so
// the rule reproduces Eq. (Iclensing) exactly up to rounding.
struct GL3 {
  static constexpr double c0 = 0.11270166537925831148;  // (1 - sqrt(3/5)) / 2
  static constexpr double c1 = 0.5;
  static constexpr double c2 = 0.88729833462074168852;  // (1 + sqrt(3/5)) / 2
  static constexpr double w0 = 5.0 / 18.0;              // weights on [0, 1]
  static constexpr double w1 = 8.0 / 18.0;
  static constexpr double w2 = 5.0 / 18.0;
};

// Trilinear value from the eight corner values at local coords (ux, uy, uz),
// with the x-differences precomputed (corner v = ix + 2 iy + 4 iz).
template <typename R>
__device__ __forceinline__ R trilerp(const R* q, const R* dq, R ux, R uy, R uz) {
  const R a00 = fma(ux, dq[0], q[0]);
  const R a10 = fma(ux, dq[1], q[2]);
  const R a01 = fma(ux, dq[2], q[4]);
  const R a11 = fma(ux, dq[3], q[6]);
  const R b0 = fma(uy, a10 - a00, a00);
  const R b1 = fma(uy, a11 - a01, a01);
  return fma(uz, b1 - b0, b0);
}

// int_{chi_B}^{chi_A} g(chi) Q dchi for one cell.  uA/uB: local coordinates
// (cell units) of the entry and exit points; L = chi_A - chi_B; chiB;
// DB = chi_s - chi_B; inv_chis = 1/chi_s.
template <typename R>
__device__ __forceinline__ R cell_integral(const R* q, const R* uA, const R* uB, R L, R chiB, R DB,
                                           R inv_chis) {
  R dq[4];
  dq[0] = q[1] - q[0];
  dq[1] = q[3] - q[2];
  dq[2] = q[5] - q[4];
  dq[3] = q[7] - q[6];
  const R du0 = uA[0] - uB[0], du1 = uA[1] - uB[1], du2 = uA[2] - uB[2];
  R acc;
  {
    const R c = (R)GL3::c0;
    const R qk = trilerp(q, dq, fma(du0, c, uB[0]), fma(du1, c, uB[1]), fma(du2, c, uB[2]));
    const R chik = fma(L, c, chiB);
    const R gk = chik * fma(-L, c, DB);
    acc = (R)GL3::w0 * gk * qk;
  }
  {
    const R c = (R)GL3::c1;
    const R qk = trilerp(q, dq, fma(du0, c, uB[0]), fma(du1, c, uB[1]), fma(du2, c, uB[2]));
    const R chik = fma(L, c, chiB);
    const R gk = chik * fma(-L, c, DB);
    acc = fma((R)GL3::w1 * gk, qk, acc);
  }
  {
    const R c = (R)GL3::c2;
    const R qk = trilerp(q, dq, fma(du0, c, uB[0]), fma(du1, c, uB[1]), fma(du2, c, uB[2]));
    const R chik = fma(L, c, chiB);
    const R gk = chik * fma(-L, c, DB);
    acc = fma((R)GL3::w2 * gk, qk, acc);
  }
  return acc * L * inv_chis;
}

// The two integrals of the source-distance decomposition (Eq. Isources) over
// one cell: ma = int chi Q dchi and mb = int chi^2 Q dchi on [chi_B, chi_A]
// (degree <= 5 in chi: the three-point rule is exact).
template <typename R>
__device__ __forceinline__ void cell_moments(const R* q, const R* uA, const R* uB, R L, R chiB,
                                             R& ma, R& mb) {
  R dq[4];
  dq[0] = q[1] - q[0];
  dq[1] = q[3] - q[2];
  dq[2] = q[5] - q[4];
  dq[3] = q[7] - q[6];
  const R du0 = uA[0] - uB[0], du1 = uA[1] - uB[1], du2 = uA[2] - uB[2];
  const R cs[3] = {(R)GL3::c0, (R)GL3::c1, (R)GL3::c2};
  const R ws[3] = {(R)GL3::w0, (R)GL3::w1, (R)GL3::w2};
  R a = 0, b = 0;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const R c = cs[k];
    const R qk = trilerp(q, dq, fma(du0, c, uB[0]), fma(du1, c, uB[1]), fma(du2, c, uB[2]));
    const R chik = fma(L, c, chiB);
    const R wq = ws[k] * qk * chik;
    a += wq;
    b = fma(wq, chik, b);
  }
  ma = a * L;
  mb = b * L;
}

// Selects by lane masks held in pairs of scalar registers: a row of selects on
// VCC in the short encoding takes the SIMD 23 clocks each, this form 4.  Each
// statement opens with the two wait states due between a vector instruction
// that writes a mask (a compare, the reload of a spilled one) and a select that
// reads it: the compiler does not count them for hand-written statements, and
// inside one it can put nothing between.

// The entry face's values E and the exit face's X[0..2], in place: see
// shift_face (m01 = m0 | m1).
__device__ __forceinline__ void shift_words(float* E, float* X, unsigned long long m0,
                                            unsigned long long m1, unsigned long long m01,
                                            const float* F) {
  asm("s_nop 1\n\t"
      "v_cndmask_b32_e64 %0, %4, %2, %12\n\t"
      "v_cndmask_b32_e64 %0, %0, %1, %11\n\t"
      "v_cndmask_b32_e64 %1, %5, %3, %12\n\t"
      "v_cndmask_b32_e64 %1, %1, %8, %11\n\t"
      "v_cndmask_b32_e64 %4, %8, %6, %12\n\t"
      "v_cndmask_b32_e64 %4, %4, %5, %11\n\t"
      "v_cndmask_b32_e64 %5, %9, %7, %12\n\t"
      "v_cndmask_b32_e64 %5, %5, %10, %11\n\t"
      "v_cndmask_b32_e64 %2, %6, %8, %12\n\t"
      "v_cndmask_b32_e64 %2, %2, %3, %11\n\t"
      "v_cndmask_b32_e64 %3, %7, %9, %13\n\t"
      "v_cndmask_b32_e64 %6, %10, %7, %11"
      : "+&v"(E[0]), "+&v"(E[1]), "+&v"(E[2]), "+&v"(E[3]), "+&v"(X[0]), "+&v"(X[1]), "+&v"(X[2])
      : "v"(X[3]), "v"(F[0]), "v"(F[1]), "v"(F[2]), "s"(m0), "s"(m1), "s"(m01));
}

// x where the lane's bit of m is clear, 0 where it is set (y, z likewise).
__device__ __forceinline__ void clear_words(float& x, float& y, float& z, unsigned long long mx,
                                            unsigned long long my, unsigned long long mz) {
  asm("s_nop 1\n\t"
      "v_cndmask_b32_e64 %0, %0, 0, %3\n\t"
      "v_cndmask_b32_e64 %1, %1, 0, %4\n\t"
      "v_cndmask_b32_e64 %2, %2, 0, %5"
      : "+&v"(x), "+&v"(y), "+&v"(z)
      : "s"(mx), "s"(my), "s"(mz));
}

// The two halves of doubles.
template <int kN>
__device__ __forceinline__ void split_words(const double* v, float* lo, float* hi) {
#pragma unroll
  for (int c = 0; c < kN; ++c) {
    lo[c] = __int_as_float(__double2loint(v[c]));
    hi[c] = __int_as_float(__double2hiint(v[c]));
  }
}
template <int kN>
__device__ __forceinline__ void join_words(const float* lo, const float* hi, double* v) {
#pragma unroll
  for (int c = 0; c < kN; ++c) v[c] = __hiloint2double(__float_as_int(hi[c]), __float_as_int(lo[c]));
}

// f of a lane that has crossed one face, along axis 0 in the lanes of m0, axis 1
// in those of m1 and axis 2 in the others: 0 on that axis.
__device__ __forceinline__ void enter_cell(float* f, unsigned long long m0, unsigned long long m1) {
  clear_words(f[0], f[1], f[2], m0, m1, ~(m0 | m1));
}
__device__ __forceinline__ void enter_cell(double* f, unsigned long long m0,
                                           unsigned long long m1) {
  float lo[3], hi[3];
  split_words<3>(f, lo, hi);
  enter_cell(lo, m0, m1);
  enter_cell(hi, m0, m1);
  join_words<3>(lo, hi, f);
}

// Corner values q[i + 2 j] of one face and its bilinear coefficients
// q0 + cx x + cy y + cxy x y.
template <typename R>
struct Face {
  R q[4], cx, cy, cxy;
  Face() = default;
  __device__ __forceinline__ explicit Face(const R* v) {
#pragma unroll
    for (int c = 0; c < 4; ++c) q[c] = v[c];
    cx = q[1] - q[0];
    cy = q[2] - q[0];
    cxy = (q[3] - q[2]) - cx;
  }
  __device__ __forceinline__ R at(R x, R y) const {
    return fma(y, fma(x, cxy, cy), fma(x, cx, q[0]));
  }
};

template <typename R>
__device__ __forceinline__ void swap_faces(Face<R>& a, Face<R>& b) {
  const Face<R> t = a;
  a = b;
  b = t;
}

// The trilinear field along a piece from (xA, yA, zA) to (xB, yB, zB), with E
// and X the faces z = 0 and z = 1 of the cell.  On either face the bilinear
// value along the piece is, in t = (chi_A - chi) / L,
//   E(t) = E0 (1 - t) + E1 t - cE t (1 - t),  cE = cxy (xB - xA) (yB - yA),
// and 1 - z and z are linear in t, so
//   Q(t) = u0 (1 - t)^2 + m t (1 - t) + u1 t^2 - t (1 - t) (cA (1 - t) + cB t)
// with u0 and u1 the values at the two ends.  Against a quadratic kernel
// g = gA (1 - t) + gB t + K t (1 - t) its integral is a sum of five products
// (integrate_form): Eq. (Iclensing) exactly up to rounding, in about half the
// operations of a three-point Gauss rule, most of all between two faces of one
// axis (zA = 0, zB = 1), where u0 is the value the last cell ended with.  The
// three builders round every piece they share alike.
template <typename R>
struct PieceForm {
  R u0, m, u1, cA, cB;
};

// Value at the start of a piece (z = 0: exactly the entry face's).
template <typename R>
__device__ __forceinline__ R form_start(const Face<R>& e, const Face<R>& x, const R* fA) {
  return fma(fA[2], x.at(fA[0], fA[1]), ((R)1 - fA[2]) * e.at(fA[0], fA[1]));
}

template <typename R>
__device__ __forceinline__ PieceForm<R> form_general(const Face<R>& e, const Face<R>& x,
                                                     const R* fA, const R* fB) {
  const R eA = e.at(fA[0], fA[1]), eB = e.at(fB[0], fB[1]);
  const R xA = x.at(fA[0], fA[1]), xB = x.at(fB[0], fB[1]);
  const R dd = (fB[0] - fA[0]) * (fB[1] - fA[1]);
  const R cE = e.cxy * dd, cX = x.cxy * dd;
  const R zA = fA[2], zB = fB[2], wA = (R)1 - zA, wB = (R)1 - zB;
  PieceForm<R> f;
  f.u0 = fma(zA, xA, wA * eA);
  f.u1 = fma(zB, xB, wB * eB);
  f.m = fma(wA, eB, wB * eA) + fma(zA, xB, zB * xA);
  f.cA = fma(zA, cX, wA * cE);
  f.cB = fma(zB, cX, wB * cE);
  return f;
}

// A piece that ends on the exit face (zB = 1); u0 from form_start.
template <typename R>
__device__ __forceinline__ PieceForm<R> form_out(const Face<R>& e, const Face<R>& x, R u0, R xa,
                                                 R ya, R zA, R xb, R yb) {
  const R eB = e.at(xb, yb), xA = x.at(xa, ya), xB = x.at(xb, yb);
  const R dd = (xb - xa) * (yb - ya);
  const R cE = e.cxy * dd, cX = x.cxy * dd;
  const R wA = (R)1 - zA;
  PieceForm<R> f;
  f.u0 = u0;
  f.u1 = xB;
  const R we = wA * eB;   // rounded by itself, as in form_general with zB = 1
  f.m = we + fma(zA, xB, xA);
  f.cA = fma(zA, cX, wA * cE);
  f.cB = cX;
  return f;
}

// A piece from the entry face to the exit face (zA = 0, zB = 1).
template <typename R>
__device__ __forceinline__ PieceForm<R> form_through(const Face<R>& e, const Face<R>& x, R u0,
                                                     R xa, R ya, R xb, R yb) {
  const R dd = (xb - xa) * (yb - ya);
  PieceForm<R> f;
  f.u0 = u0;
  f.u1 = x.at(xb, yb);
  f.m = e.at(xb, yb) + x.at(xa, ya);
  f.cA = e.cxy * dd;
  f.cB = x.cxy * dd;
  return f;
}

// 12 int_0^1 g Q dt of a piece against the kernel gA (1 - t) + gB t + K t (1 - t).
template <typename R>
__device__ __forceinline__ R integrate_form(const PieceForm<R>& f, R gA, R gB, R K) {
  const R s = gA + gB;
  const R a = fma((R)0.6, K, s), b = fma((R)0.2, K, (R)0.4 * s);
  const R k20 = fma((R)2, gA, a), k02 = fma((R)2, gB, a), k11 = fma((R)0.4, K, s);
  const R h21 = fma((R)0.2, gA, b), h12 = fma((R)0.2, gB, b);
  return fma(f.u0, k20, fma(f.m, k11, fma(f.u1, k02, -fma(f.cA, h21, f.cB * h12))));
}

// The same with K = 0.
template <typename R>
__device__ __forceinline__ R integrate_form(const PieceForm<R>& f, R gA, R gB) {
  const R s = gA + gB, b = (R)0.4 * s;
  const R k20 = fma((R)2, gA, s), k02 = fma((R)2, gB, s);
  const R h21 = fma((R)0.2, gA, b), h12 = fma((R)0.2, gB, b);
  return fma(f.u0, k20, fma(f.m, s, fma(f.u1, k02, -fma(f.cA, h21, f.cB * h12))));
}

// 12 int_0^1 Q dt.
template <typename R>
__device__ __forceinline__ R integrate_constant(const PieceForm<R>& f) {
  return fma((R)4, f.u0 + f.u1, fma((R)2, f.m, -(f.cA + f.cB)));
}

// One face crossed, along axis 0 in the lanes of m0, axis 1 in those of m1 and
// axis 2 in the others: the four values of that face move to the entry side,
// the four of the new exit face F_j (j = i_a + 2 i_b over the two other axes
// a < b) come in.
__device__ __forceinline__ void shift_face(float* E, float* X, unsigned long long m0,
                                           unsigned long long m1, const float* F) {
  shift_words(E, X, m0, m1, m0 | m1, F);
  X[3] = F[3];
}
__device__ __forceinline__ void shift_face(double* E, double* X, unsigned long long m0,
                                           unsigned long long m1, const double* F) {
  float El[4], Eh[4], Xl[4], Xh[4], Fl[3], Fh[3];
  split_words<4>(E, El, Eh);
  split_words<4>(X, Xl, Xh);
  split_words<3>(F, Fl, Fh);
  shift_words(El, Xl, m0, m1, m0 | m1, Fl);
  shift_words(Eh, Xh, m0, m1, m0 | m1, Fh);
  join_words<4>(El, Eh, E);
  join_words<3>(Xl, Xh, X);
  X[3] = F[3];
}

// FNV-1a, 64 bit, over the 8 little-endian bytes of w.
__device__ __forceinline__ uint64_t fnv_word(uint64_t h, uint64_t w) {
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    h ^= (w >> (8 * b)) & 0xffull;
    h *= 0x100000001b3ull;
  }
  return h;
}
__device__ __forceinline__ uint64_t fnv_piece(uint64_t h, int64_t cell, double a, double b) {
  h = fnv_word(h, (uint64_t)cell);
  h = fnv_word(h, (uint64_t)__double_as_longlong(a));
  h = fnv_word(h, (uint64_t)__double_as_longlong(b));
  return h;
}
constexpr uint64_t kFnvOffset = 0xcbf29ce484222325ull;

struct LogRecord {
  int64_t cell;
  double chi_a, chi_b;
};

// Kahan step: (sum, comp) += x
__device__ __forceinline__ void kahan_add(float& sum, float& comp, float x) {
  const float y = __fsub_rn(x, comp);
  const float t = __fadd_rn(sum, y);
  comp = __fsub_rn(__fsub_rn(t, sum), y);
  sum = t;
}

// Position of the k-th 8 x 8 tile of a bundle's tiles_x x tiles_y tile grid
// in Z order (quadrants (0,0), (1,0), (0,1), (1,1) at every level of the
// enclosing power-of-two square, positions outside the grid skipped): tiles
// that are close in launch order are close on the sky, so the wavefronts
// working at the same time, and the ones that share a chiplet, gather from
// the same part of the field.  k is wavefront-uniform (scalar work).
__device__ __forceinline__ void zorder_tile(int64_t k, int W, int H, int& x, int& y) {
  int s = 1;
  while (s < W || s < H) s <<= 1;
  int x0 = 0, y0 = 0;
  while (s > 1) {
    const int h = s >> 1;
    const int64_t w0 = min(max(W - x0, 0), h), w1 = min(max(W - x0 - h, 0), h);
    const int64_t h0 = min(max(H - y0, 0), h), h1 = min(max(H - y0 - h, 0), h);
    s = h;
    if (k < w0 * h0) continue;
    k -= w0 * h0;
    if (k < w1 * h0) {
      x0 += h;
      continue;
    }
    k -= w1 * h0;
    if (k < w0 * h1) {
      y0 += h;
      continue;
    }
    k -= w0 * h1;
    x0 += h;
    y0 += h;
  }
  x = x0;
  y = y0;
}

// Position of a lane's ray in its 8 x 8 tile, Z order: each quad of lanes is a
// 2 x 2 block of the map.
__device__ __forceinline__ void zorder_lane(int lane, int& x, int& y) {
  x = (lane & 1) | ((lane >> 1) & 2) | ((lane >> 2) & 4);
  y = ((lane >> 1) & 1) | ((lane >> 2) & 2) | ((lane >> 3) & 4);
}

// Persistent launches: one work counter per chiplet (XCD).  Workgroups are
// dealt to the eight XCDs round-robin, so workgroup b runs on XCD b % 8; the
// tiles are split into eight contiguous ranges of the launch order, each
// chiplet drains its own range first (its L2 sees one compact part of the
// sky) and then helps with the others.  Returns the next tile, or -1 once
// every range is empty (every wavefront reaches that exit).
constexpr int kQueues = 8;
__device__ __forceinline__ int64_t next_tile(unsigned long long* queue, int64_t n_tiles, int& q,
                                             int& tried, int lane) {
  while (tried < kQueues) {
    const int64_t lo = n_tiles * q / kQueues, hi = n_tiles * (q + 1) / kQueues;
    unsigned long long t = 0;
    if (lane == 0) t = atomicAdd(queue + q, 1ull);
    t = __shfl(t, 0, 64);
    const int64_t k = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 32))
                                 << 32) |
                                (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)t));
    if (k < hi - lo) return lo + k;
    q = q + 1 == kQueues ? 0 : q + 1;
    ++tried;
  }
  return -1;
}

// Work assignment: global tile index -> (bundle, tile within it).
__device__ __forceinline__ int find_bundle(const DevBundle* b, int nb, int64_t tile) {
  int lo = 0, hi = nb - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (b[mid].tile_begin <= tile)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

}  // namespace rr
