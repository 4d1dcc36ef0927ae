// rr_march_uniform.hip -- cell-by-cell ray march through a uniform grid
// (Sec. III F, Eqs. rayposition - disttocross) with the per-cell lensing
// integral of the trilinear vertex reconstruction (Eqs. trilinear_int,
// Iclensing) and its accumulation along the ray (Eq. sumIc).
//
// Work decomposition: a wavefront owns an 8 x 8 tile of a bundle's ray map,
// so its 64 lanes start from neighbouring directions, visit neighbouring
// cells (coalesced, cache-friendly gathers) and take similar numbers of steps.
// Tiles are either mapped one per wavefront from the grid (XCD-striped so a
// chiplet's L2 sees a contiguous part of the sky) or pulled from a device
// queue by persistent workgroups.
#include <climits>
#include <type_traits>

#include "rr_ray.hpp"

namespace rr {
namespace {

// Vertex record at byte offset `off` of the tensor (6 components: three
// 8-byte accesses in FP32, three 16-byte accesses in FP64).  A 32-bit offset
// lets the load take the array base from scalar registers.
template <typename R, typename Off>
__device__ __forceinline__ void load_vertex(const R* __restrict__ tv, Off off, R* t) {
  const char* b = reinterpret_cast<const char*>(tv) + (uint64_t)off;
  if constexpr (sizeof(R) == 4) {
    const float2* p = reinterpret_cast<const float2*>(b);
    const float2 x = p[0], y = p[1], z = p[2];
    t[0] = x.x; t[1] = x.y; t[2] = y.x; t[3] = y.y; t[4] = z.x; t[5] = z.y;
  } else {
    const double2* p = reinterpret_cast<const double2*>(b);
    const double2 x = p[0], y = p[1], z = p[2];
    t[0] = x.x; t[1] = x.y; t[2] = y.x; t[3] = y.y; t[4] = z.x; t[5] = z.y;
  }
}

// Integrand modes: the tidal tensor with the trilinear integral, the tidal
// tensor at cell centres (NGP), Method A's (c delta, grad Phi) fields, the
// tidal tensor against the two source-distance moments chi and chi^2, and a
// vertex scalar with a constant kernel (ISW).
constexpr int kTidal = 0, kNgp = 1, kMethodA = 2, kSources = 3, kScalar = 4;

// The record at byte offset `off` and its value(s): Q = P : T (tidal modes),
// (c delta, n . grad Phi) with P[0..2] = n (Method A), or the scalar (ISW).
template <typename R, typename Off, int kMode>
__device__ __forceinline__ void load_record(const R* __restrict__ tv, Off off, R* t) {
  const char* b = reinterpret_cast<const char*>(tv) + (uint64_t)off;
  if constexpr (kMode == kScalar) {
    t[0] = *reinterpret_cast<const R*>(b);
  } else if constexpr (kMode == kMethodA) {
    if constexpr (sizeof(R) == 4) {
      const float4 x = *reinterpret_cast<const float4*>(b);
      t[0] = x.x; t[1] = x.y; t[2] = x.z; t[3] = x.w;
    } else {
      const double2* p = reinterpret_cast<const double2*>(b);
      const double2 x = p[0], y = p[1];
      t[0] = x.x; t[1] = x.y; t[2] = y.x; t[3] = y.y;
    }
  } else {
    load_vertex<R, Off>(tv, off, t);
  }
}
template <typename R, int kMode>
__device__ __forceinline__ void record_value(const R* t, const R* P, R& q, R& q2) {
  q2 = (R)0;
  if constexpr (kMode == kScalar) {
    q = t[0];
  } else if constexpr (kMode == kMethodA) {
    q = t[0];
    q2 = fma(P[2], t[3], fma(P[1], t[2], P[0] * t[1]));
  } else {
    R acc = P[0] * t[0];
#pragma unroll
    for (int c = 1; c < 6; ++c) acc = fma(P[c], t[c], acc);
    q = acc;
  }
}
template <typename R, typename Off, int kMode>
__device__ __forceinline__ R point_value(const R* __restrict__ tv, Off off, const R* P) {
  R t[6], q, q2;
  load_record<R, Off, kMode>(tv, off, t);
  record_value<R, kMode>(t, P, q, q2);
  return q;
}

// Records loaded ahead of an integral are not touched before it is done: an
// empty statement takes the sum and hands the loaded words on, so that the
// compiler neither waits for the loads early nor moves the integral past them.
template <int kWords, typename R>
__device__ __forceinline__ void after_sum(R* t, R sum) {
#pragma unroll
  for (int c = 0; c < kWords; ++c) asm volatile("" : "+v"(t[c]) : "v"(sum));
}

// The records of a face's corners c = i_a + 2 i_b (w0 the offset of corner 0,
// da and db the steps along its two axes), loaded ahead of their use.
template <typename R, typename Off, int kMode>
struct FaceRecords {
  static constexpr int kWords = kMode == 2 ? 4 : (kMode == 4 ? 1 : 6);
  R t[4][kWords];
  __device__ __forceinline__ void load(const R* __restrict__ tv, Off w0, Off da, Off db) {
    const Off w1 = w0 + da;
    load_record<R, Off, kMode>(tv, w0, t[0]);
    load_record<R, Off, kMode>(tv, w1, t[1]);
    load_record<R, Off, kMode>(tv, w0 + db, t[2]);
    load_record<R, Off, kMode>(tv, w1 + db, t[3]);
  }
  __device__ __forceinline__ void hold(R sum) {
#pragma unroll
    for (int c = 0; c < 4; ++c) after_sum<kWords>(t[c], sum);
  }
  // their values (one set, or Method A's two)
  __device__ __forceinline__ void project(const R* P, R* f, R* f2) const {
#pragma unroll
    for (int c = 0; c < 4; ++c) record_value<R, kMode>(t[c], P, f[c], f2[c]);
  }
};
template <typename R, typename Off, int kMode>
__device__ __forceinline__ void load_face(const R* __restrict__ tv, Off w0, Off da, Off db,
                                          const R* P, R* f, R* f2) {
  FaceRecords<R, Off, kMode> r;
  r.load(tv, w0, da, db);
  r.project(P, f, f2);
}

// The same four corners for a quad of lanes that share the face (FP32): lane i
// of the quad has loaded the record of corner i, and v_mfma_f32_4x4x1_16b
// (sixteen 4 x 4 outer products, one per quad) accumulates over the
// components f[i] = sum_c T_c(lane i) P_c(own lane): the rounding of the fma
// chain in record_value, component by component, with a quarter of its loads.
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <int kMode>
__device__ __forceinline__ void project_quad(const float* t, const float* P, float* f,
                                             float* f2) {
  const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  f32x4 d;
  if constexpr (kMode == kScalar) {
    d = __builtin_amdgcn_mfma_f32_4x4x1f32(t[0], 1.0f, zero, 0, 0, 0);
  } else if constexpr (kMode == kMethodA) {
    d = __builtin_amdgcn_mfma_f32_4x4x1f32(t[0], 1.0f, zero, 0, 0, 0);
    f32x4 g = zero;
#pragma unroll
    for (int c = 0; c < 3; ++c)
      g = __builtin_amdgcn_mfma_f32_4x4x1f32(t[c + 1], P[c], g, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) f2[i] = g[i];
  } else {
    d = zero;
#pragma unroll
    for (int c = 0; c < 6; ++c) d = __builtin_amdgcn_mfma_f32_4x4x1f32(t[c], P[c], d, 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) f[i] = d[i];
}

// x of lane 0 of the quad.
__device__ __forceinline__ uint32_t quad_first(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x00, 0xf, 0xf, false);
}
__device__ __forceinline__ uint64_t quad_first(uint64_t x) {
  return ((uint64_t)quad_first((uint32_t)(x >> 32)) << 32) | quad_first((uint32_t)x);
}

// The largest x of the quad.
__device__ __forceinline__ int quad_max(int x) {
  const int y = max(x, __builtin_amdgcn_update_dpp(0, x, 0xb1, 0xf, 0xf, false));
  return max(y, __builtin_amdgcn_update_dpp(0, y, 0x4e, 0xf, 0xf, false));
}

// One ray, in the ray's own frame: along each axis, corner bit 0 is the
// vertex layer of the face the ray enters through and bit 1 the layer of the
// face it leaves through, and the local coordinate f runs from 0 (entry face)
// to 1 (exit face).  The lattice axes are relabelled cyclically so that axis 2
// is the one the tile's rays run along (kz: the largest component of the
// tile's first direction); a cell's corners are its entry face E and its exit
// face X on that axis.  A crossing of one face keeps the four projected corner
// values of that face (they become the entry face of the next cell) and loads
// only the four of the new exit face; a crossing through an edge or a vertex
// reloads all eight.
//
// Per axis the lane keeps, in FP64, the crossing parameter of the exit plane
// (f = 1 - |n_a| (chi - t_exit) inside the slab) and its reciprocal
// direction, the exit plane's lattice coordinate, and the byte offsets of the
// wrapped entry and exit vertex layers (32 bit when the tensor is below
// 4 GiB): a corner's offset is the sum of one of them per axis.
//
// Most cells of a bundle are entered and left through faces of axis 2.  While
// every lane of the wavefront is about to leave its cell that way, the march
// runs a short loop of its own: no exit selection, no stepping of the other
// axes, the entry face's bilinear coefficients and the value at the entry
// point carried over from the last cell, and (FP32) one record per lane
// instead of four, shared within quads and projected on the matrix cores.
// Between runs every lane crosses one face at a time with the loads of the new
// face in flight during the integral; what neither covers (edges, ends of the
// window, sources) takes the cell of any kind at the bottom.  All three round a
// piece alike, so a ray's result depends neither on its neighbours nor on the
// launch.  Launches that follow every crossing (debug outputs, crossing limits)
// or may end at the edge of an open grid are instantiations without runs
// (kRun false, launch_off).
//
// What bounds it is VALU issue, with the address path of the gathers close
// behind (an FP32 operation on vector registers takes a SIMD 2.5 clocks, an
// FP64 one, a compare, a select, an integer minimum or a conversion 4.3, the
// 4 x 4 matrix instruction 8.6): 121 VALU instructions per crossing and
// wavefront (69 in the run, 175 in a step between runs) against 206 for one
// loop over cells of any kind with a three-point Gauss rule; address unit 76 %
// busy.  512^3, 2048^2 rays over 5 degrees: 0.80 ms per segment (1.12 before;
// 0.88 while lanes a layer of axis 2 apart were left so, see quad_max).
// Keeping the wavefront in one layer of axis 2 throughout (lanes that leave
// sideways cross first, the others wait) cost more than it saved: 150 VALU and
// 0.97 ms against 0.88.
template <typename R, bool kDebug, typename Off, int kMode, bool kPass, bool kRun>
__device__ void trace_one(const R* __restrict__ tv, const TraceArgs& a, const DevBundle& B,
                          int64_t ray, bool own) {
  const int64_t out = B.ray_offset + ray;
  const double dir[3] = {B.dir[3 * ray + 0], B.dir[3 * ray + 1], B.dir[3 * ray + 2]};
  // Only unit directions are traced: that bounds the number of crossings by
  // the chi window validated on the host, so every lane terminates.
  const double nrm2 = dir[0] * dir[0] + dir[1] * dir[1] + dir[2] * dir[2];
  if (!(fabs(nrm2 - 1.0) <= 1e-9)) {
    if (a.status && own) a.status[out] = RR_RAY_BAD_DIRECTION;
    return;
  }
  R P[6];
  if constexpr (kMode == kMethodA || kMode == kScalar) {
#pragma unroll
    for (int c = 0; c < 3; ++c) P[c] = (R)dir[c];
  } else {
    double Pd[6];
    projection(a.quantity, dir[0], dir[1], dir[2], Pd);
#pragma unroll
    for (int c = 0; c < 6; ++c) P[c] = (R)Pd[c];
  }

  const int n = a.n;
  constexpr Off kRec =
      (Off)((kMode == kMethodA ? 4 : (kMode == kScalar ? 1 : 6)) * sizeof(R));  // bytes per record
  // axis 2 of the frame is lattice axis kz, axes 0 and 1 the two after it
  int kz = fabs(dir[0]) > fabs(dir[2]) ? 0 : 2;
  kz = fabs(dir[1]) > fmax(fabs(dir[0]), fabs(dir[2])) ? 1 : kz;
  kz = __builtin_amdgcn_readfirstlane(kz);
  const double d[3] = {kz == 2 ? dir[0] : (kz == 0 ? dir[1] : dir[2]),
                       kz == 2 ? dir[1] : (kz == 0 ? dir[2] : dir[0]),
                       kz == 2 ? dir[2] : (kz == 0 ? dir[0] : dir[1])};
  const double o[3] = {kz == 2 ? a.o[0] : (kz == 0 ? a.o[1] : a.o[2]),
                       kz == 2 ? a.o[1] : (kz == 0 ? a.o[2] : a.o[0]),
                       kz == 2 ? a.o[2] : (kz == 0 ? a.o[0] : a.o[1])};
  const Off sx = kRec, sy = kRec * (Off)n, sz = kRec * (Off)n * (Off)n;
  const Off stride[3] = {kz == 2 ? sx : (kz == 0 ? sy : sz), kz == 2 ? sy : (kz == 0 ? sz : sx),
                         kz == 2 ? sz : (kz == 0 ? sx : sy)};
  const double lo = B.chi_lo;
  double chiA = B.chi_hi;
  // a later pass resumes on the face where the last one stopped
  if constexpr (kPass) {
    const double r0 = a.resume[out];
    if (!(r0 > lo)) return;             // done in an earlier pass
    chiA = fmin(r0, chiA);              // +inf before the first pass
    if (chiA <= a.pause_chi) return;    // starts in a later pass
  }
  double r[3], te[3];
  R absd[3];         // f(chi) = 1 - absd (chi - t_exit)
  double pp[3];      // lattice coordinate of the exit plane (unwrapped, replicated box)
  Off oE[3], oX[3];  // byte offsets of the entry and the exit vertex layer, wrapped into [0, n)
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    r[k] = (d[k] != 0.0) ? 1.0 / d[k] : 0.0;
    const int m = start_slab(o[k], d[k], r[k], chiA, 1.0);
    // n_a > 0: the march runs down the lattice, leaving through plane m;
    // otherwise up, leaving through plane m + 1 (never reached if n_a = 0)
    pp[k] = (double)(d[k] > 0.0 ? m : m + 1);
    if (d[k] != 0.0) {
      te[k] = tplane(pp[k], o[k], r[k]);
      absd[k] = (R)fabs(d[k]);
    } else {
      // never crossed: a slope of 1e-30 with an exit parameter (1 - f) 1e30
      // below reproduces the fixed coordinate f = o~ - m to rounding, and the
      // parameter is never the largest (chi_lo >= 0)
      te[k] = -(1.0 - (o[k] - (double)m)) * 1e30;
      absd[k] = (R)1e-30;
    }
    int lm = m % n;
    lm = lm < 0 ? lm + n : lm;                       // layer of plane m
    const int lp = lm + 1 == n ? 0 : lm + 1;         // layer of plane m + 1
    oE[k] = (Off)(d[k] > 0.0 ? lp : lm) * stride[k];
    oX[k] = (Off)(d[k] > 0.0 ? lm : lp) * stride[k];
  }
  R fA[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    fA[k] = (R)1 - absd[k] * (R)(chiA - te[k]);
    // on the entry face (a resumed ray, or a window that starts on a face)
    // the coordinate is 0, as when the march steps across that face
    if (kPass && d[k] != 0.0 && chiA == tplane(d[k] > 0.0 ? pp[k] + 1.0 : pp[k] - 1.0, o[k], r[k]))
      fA[k] = (R)0;
  }
  // axis 2 marched as a countdown: its exit layer's offset is (mx ^ up) + cx
  // with mx one stride less at every crossing and the last layer after 0
  const Off span2 = (Off)(n - 1) * stride[2];
  const bool down2 = d[2] > 0.0;
  const Off up = down2 ? (Off)0 : ~(Off)0;
  const Off cx = down2 ? (Off)0 : span2 + (Off)1;
  const double step2 = down2 ? -1.0 : 1.0;
  // whether the lanes of every quad march axis 2 in one sense: only then do
  // equally many crossings along it mean the same layer, and may a quad share
  // its records or wait for its slowest lane (rays of a bundle are free to
  // look either way).  A lane that is missing here never marches.
  const bool one_way = __ballot(quad_first((uint32_t)down2) == (uint32_t)down2) == ~0ull;

  constexpr bool kTwo = kMode == kMethodA;   // a second set of corner values (n . grad Phi)
  // corner values c = i_0 + 2 i_1 of the entry and the exit face of axis 2
  // (2: Method A's gradient set)
  R E[4], X[4], E2[4], X2[4];
  // all eight corners, in two halves so that at most four records are in
  // flight: this must not set the register budget of the whole march
  auto load_cell = [&] {
    const Off da = oX[0] - oE[0], db = oX[1] - oE[1];
    load_face<R, Off, kMode>(tv, oE[0] + oE[1] + oE[2], da, db, P, E, E2);
    __builtin_amdgcn_sched_barrier(0);
    load_face<R, Off, kMode>(tv, oE[0] + oE[1] + oX[2], da, db, P, X, X2);
  };
  if constexpr (kMode != kNgp) load_cell();

  const double chi_s = B.chi_s;
  // what multiplies a piece's integral (the forms give 12 times it, the
  // kernels of the lensing integrands chi_s times theirs).  FP32 keeps the part
  // that its rounding leaves out, which would be one relative error of up to
  // 6e-8 common to all pieces.
  const double form = kMode == kNgp ? 1.0 : 1.0 / 12.0;
  const double factor = kMode == kScalar || kMode == kSources ? a.kappa_scale * form
                                                              : a.kappa_scale * form / chi_s;
  const R scale = (R)factor, scale_rest = (R)(factor - (double)scale);
  auto scaled = [&](R x) {
    if constexpr (sizeof(R) == 4) return fma(x, scale, x * scale_rest);
    else return x * scale;
  };
  R sum;
  float comp = 0.0f;
  // source-distance moments: (sum, comp) integrate chi Q, (sum2, comp2)
  // chi^2 Q; the walk also stops at the next source distance src_j
  R sum2 = 0;
  float comp2 = 0.0f;
  int jn = 0;
  double src_j = -1.0;
  if constexpr (kMode == kSources) {
    if constexpr (sizeof(R) == 4) {
      const float4 m = reinterpret_cast<const float4*>(a.kappa)[out];
      sum = m.x; comp = m.y; sum2 = m.z; comp2 = m.w;
    } else {
      const double2 m = reinterpret_cast<const double2*>(a.kappa)[out];
      sum = m.x; sum2 = m.y;
    }
    // this window stops at the sources with chi_lo <= chi_s,j < chi_hi
    while (jn < a.n_src && !(a.src[jn] < chiA)) ++jn;
    src_j = jn < a.n_src ? a.src[jn] : -1.0;
  } else if constexpr (sizeof(R) == 4) {
    sum = reinterpret_cast<float*>(a.kappa)[out];
    if (a.kappa_comp) comp = a.kappa_comp[out];
  } else {
    sum = reinterpret_cast<double*>(a.kappa)[out];
  }
  uint64_t hv = kFnvOffset;
  int64_t count = 0;
  int32_t st = RR_RAY_OK;
  const int64_t maxc = a.max_crossings > 0 ? a.max_crossings : INT64_MAX;
  static_assert(!(kDebug && kRun), "runs keep no count, hash or log");
  // open grids: chi of the last plane whose crossing leads into a cell with a
  // whole stencil (cells 2 .. n - 3 on every axis)
  double open_halt = -INFINITY;
  if (!kRun && a.open) {
#pragma unroll
    for (int k = 0; k < 3; ++k)
      if (d[k] != 0.0)
        open_halt = fmax(open_halt, tplane(d[k] > 0.0 ? 2.0 : (double)(n - 2), o[k], r[k]));
  }

  // the kernel at chi: g times chi_s (tidal), chi (sources), both g and
  // dg/dchi times chi_s (Method A)
  auto kernel = [&](double chi, R& k0, R& k1) {
    const R c = (R)chi;
    k0 = c;
    k1 = 0;
    if constexpr (kMode == kTidal || kMode == kMethodA) {
      const R rest = (R)(chi_s - chi);
      k0 = c * rest;
      if constexpr (kMode == kMethodA) k1 = rest - c;
    }
  };
  // adds the piece of length L with the form q (q2: the gradient's), its
  // kernel values at both ends
  auto add_piece = [&](const PieceForm<R>& q, const PieceForm<R>& q2, R L, R gA, R gB, R hA, R hB,
                       R surface) {
    R ic, ic2 = 0;
    if constexpr (kMode == kScalar) {
      ic = integrate_constant(q) * scaled(L);
    } else if constexpr (kMode == kSources) {
      // the moments' kernels chi and chi^2 (curvature -L^2)
      const R Ls = scaled(L);
      ic = integrate_form(q, gA, gB) * Ls;
      ic2 = integrate_form(q, gA * gA, gB * gB, -(L * L)) * Ls;
    } else {
      R s = integrate_form(q, gA, gB, L * L);
      if constexpr (kMode == kMethodA) s += integrate_form(q2, hA, hB);
      ic = scaled(fma(s, L, surface));
    }
    if constexpr (sizeof(R) == 4) {
      kahan_add(sum, comp, ic);
      if constexpr (kMode == kSources) kahan_add(sum2, comp2, ic2);
    } else {
      sum += ic;
      if constexpr (kMode == kSources) sum2 += ic2;
    }
  };
  // Eq. (Iclensing_ngp): the cell-centre value times the integral of g over
  // the piece, L (g(mid) - L^2 / (12 chi_s)) with g(chi) = chi (chi_s - chi) / chi_s
  auto add_ngp = [&](R Qc, double chiB, R L) {
    const double mid = chiB + 0.5 * (chiA - chiB);
    const R gm = (R)mid * (R)(chi_s - mid) - L * L * (R)(1.0 / 12.0);
    const R ic = Qc * scaled(gm * L);
    if constexpr (sizeof(R) == 4) kahan_add(sum, comp, ic);
    else sum += ic;
  };
  R gA, hA;   // kernel values at chi_A
  kernel(chiA, gA, hA);

  // steps axis k: the exit layer becomes the entry layer, the next layer
  // along the march the exit layer
  auto next_layer = [&](int k) {
    const bool down = r[k] > 0.0;
    const Off top = (Off)(n - 1) * stride[k];
    pp[k] += down ? -1.0 : 1.0;
    te[k] = tplane(pp[k], o[k], r[k]);
    oE[k] = oX[k];
    const Off wrap_at = down ? (Off)0 : top, wrap_to = down ? top : (Off)0;
    const Off next = down ? oX[k] - stride[k] : oX[k] + stride[k];
    oX[k] = oX[k] == wrap_at ? wrap_to : next;
  };
  // offset of the record of the cell: the lower vertex layer on every axis
  auto cell_offset = [&] {
    Off low = 0;
#pragma unroll
    for (int k = 0; k < 3; ++k) low += r[k] > 0.0 ? oX[k] : oE[k];
    return low;
  };

  // what a debug launch writes of the piece that ends at chiB
  auto record_piece = [&](double chiB) {
    if constexpr (kDebug) {
      // cell id = vertex id of its lower corner
      const int64_t cell = (int64_t)(cell_offset() / kRec);
      if (a.hash) hv = fnv_piece(hv, cell, chiA, chiB);
      if (own && a.log && count < a.log_stride) {
        LogRecord* L0 = reinterpret_cast<LogRecord*>(a.log) + out * a.log_stride + count;
        L0->cell = cell;
        L0->chi_a = chiA;
        L0->chi_b = chiB;
      }
    }
  };

  for (;;) {
    if (!kRun && a.open) {
      bool outside = false;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const double m = r[k] > 0.0 ? pp[k] : pp[k] - 1.0;
        outside |= m < 2.0 || m > (double)(n - 3);
      }
      if (outside) {
        st = RR_RAY_OUT_OF_DOMAIN;
        break;
      }
    }
    // the walk stops at chi_lo, or at the next source distance above it; a
    // pass also before its boundary
    double stop = lo;
    if constexpr (kMode == kSources) stop = src_j >= lo ? src_j : lo;
    // (Method A's first piece carries a surface term)
    const bool first = kTwo && !(chiA < B.chi_hi);
    const unsigned long long all = __ballot(1);
    double halt = stop;
    if constexpr (kPass) halt = fmax(halt, a.pause_chi);
    if constexpr (!kRun) halt = fmax(halt, open_halt);
    while (__ballot(!first && (kRun || count < maxc)) == all) {
      const double side = fmax(te[0], te[1]);
      const double lim = fmax(side, halt);
      const Off w01 = oE[0] + oE[1];
      // one record per lane: all 64 lanes march (matrix instructions ignore
      // the execution mask), and the four lanes of every quad are in one cell
      // and share its frame
      bool run = kRun && __ballot(te[2] > lim) == all, part = true;
      if constexpr (kRun && sizeof(R) == 4 && kMode != kNgp) {
        run = run && one_way;
        if (run) {
          const Off w2 = oX[0] + oX[1];
          run = (__ballot(quad_first(w01) == w01) & __ballot(quad_first(w2) == w2)) == ~0ull;
          if (run) {
            // lanes of one column of cells, but in different layers of axis 2 (a
            // window that starts with a plane of axis 0 or 1 across a quad
            // leaves its lanes one crossing apart): those behind cross a face
            // alone, once, and the runs go on
            const int adv = down2 ? -(int)pp[2] : (int)pp[2];
            const bool behind = adv < quad_max(adv);
            run = __ballot(behind) == 0ull;
            part = run || behind;
          }
        }
      }
      if (run) {
        // ---- every lane leaves its cell through axis 2 alone
        if constexpr (!kRun) {
        } else if constexpr (kMode == kNgp) {
          do {
            const R Qc = point_value<R, Off, kMode>(tv, cell_offset(), P);
            add_ngp(Qc, te[2], (R)(chiA - te[2]));
            chiA = te[2];
            next_layer(2);
          } while (__ballot(te[2] > lim) == all);
        } else {
          const Off da = oX[0] - oE[0], db = oX[1] - oE[1];
          const Off off = w01 + ((threadIdx.x & 1) ? da : (Off)0) + ((threadIdx.x & 2) ? db : (Off)0);
          // countdown of the exit layer: its offset is (mx ^ up) + cx
          Off mx = (oX[2] - cx) ^ up;
          Face<R> fE(E), fX(X), gE, gX;
          R u0 = form_start(fE, fX, fA), v0 = 0;   // values at the entry point
          if constexpr (kTwo) {
            gE = Face<R>(E2);
            gX = Face<R>(X2);
            v0 = form_start(gE, gX, fA);
          }
          // one cell: entry face e, exit face x; the next exit face replaces e.
          // first: the entry point may lie inside the cell (zA > 0)
          auto step = [&](Face<R>& e, Face<R>& x, Face<R>& e2, Face<R>& x2, auto first) {
            mx = mx - stride[2] < span2 ? mx - stride[2] : span2;
            const Off nx = (mx ^ up) + cx;
            FaceRecords<R, Off, kMode> rec;
            if constexpr (sizeof(R) == 4)
              load_record<R, Off, kMode>(tv, off + nx, rec.t[0]);
            else
              rec.load(tv, w01 + nx, da, db);
            __builtin_amdgcn_sched_barrier(0);   // in flight during the integral
            const double chiB = te[2];
            const R L = (R)(chiA - chiB);
            const R xB = (R)1 - absd[0] * (R)(chiB - te[0]);
            const R yB = (R)1 - absd[1] * (R)(chiB - te[1]);
            R gB, hB;
            kernel(chiB, gB, hB);
            PieceForm<R> q, q2;
            if constexpr (first.value) {
              q = form_out(e, x, u0, fA[0], fA[1], fA[2], xB, yB);
              if constexpr (kTwo) q2 = form_out(e2, x2, v0, fA[0], fA[1], fA[2], xB, yB);
            } else {
              q = form_through(e, x, u0, fA[0], fA[1], xB, yB);
              if constexpr (kTwo) q2 = form_through(e2, x2, v0, fA[0], fA[1], xB, yB);
            }
            add_piece(q, q2, L, gA, gB, hA, hB, (R)0);
            u0 = q.u1;
            if constexpr (kTwo) v0 = q2.u1;
            gA = gB;
            hA = hB;
            fA[0] = xB;
            fA[1] = yB;
            chiA = chiB;
            pp[2] += step2;
            te[2] = tplane(pp[2], o[2], r[2]);
            if constexpr (sizeof(R) == 4) after_sum<rec.kWords>(rec.t[0], sum);
            else rec.hold(sum);
            R nf[4], nf2[4];
            if constexpr (sizeof(R) == 4)
              project_quad<kMode>(rec.t[0], P, nf, nf2);
            else
              rec.project(P, nf, nf2);
            e = Face<R>(nf);
            if constexpr (kTwo) e2 = Face<R>(nf2);
          };
          using no = std::false_type;
          step(fE, fX, gE, gX, std::true_type{});
          bool odd = true;
          for (;;) {
            if (__ballot(te[2] > lim) != all) break;
            step(fX, fE, gX, gE, no{});
            odd = false;
            if (__ballot(te[2] > lim) != all) break;
            step(fE, fX, gE, gX, no{});
            odd = true;
          }
          // after an odd number of cells the roles of the two faces are swapped
          if (odd) {
            swap_faces(fE, fX);
            if constexpr (kTwo) swap_faces(gE, gX);
          }
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            E[c] = fE.q[c];
            X[c] = fX.q[c];
            if constexpr (kTwo) {
              E2[c] = gE.q[c];
              X2[c] = gX.q[c];
            }
          }
          oX[2] = (mx ^ up) + cx;
          // the entry layer is the one before it
          const Off back = mx == span2 ? (Off)0 : mx + stride[2];
          oE[2] = (back ^ up) + cx;
        }
        fA[2] = (R)0;
      }
      // ---- every lane leaves its cell through one face (m0, m1: the lanes
      // that do through axis 0 or 1, the others through axis 2)
      const unsigned long long m2 = __ballot(te[2] > lim);
      const unsigned long long ms =
          __ballot(side > te[2]) & __ballot(side > halt) & __ballot(te[0] != te[1]);
      if ((m2 | ms) != all) break;
      if (part) {
        const double chiB = fmax(te[2], side);
        const unsigned long long m0 = ms & __ballot(te[0] > te[1]), m1 = ms & ~m0;
        R fB[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) fB[k] = (R)1 - absd[k] * (R)(chiB - te[k]);
        R ngp = 0;   // NGP: the value of the cell being left
        if constexpr (kMode == kNgp) ngp = point_value<R, Off, kMode>(tv, cell_offset(), P);
        record_piece(chiB);
        if constexpr (!kRun) ++count;
        const bool k2 = te[2] == chiB, k0 = te[0] == chiB, k1 = te[1] == chiB;
        if (k2) next_layer(2);
        if (k0) next_layer(0);
        if (k1) next_layer(1);
        // the four records of the new exit face, in flight during the integral
        FaceRecords<R, Off, kMode> rec;
        if constexpr (kMode != kNgp) {
          const Off w0 = (k0 ? oX[0] : oE[0]) + (k1 ? oX[1] : oE[1]) + (k2 ? oX[2] : oE[2]);
          rec.load(tv, w0, k0 ? oX[1] - oE[1] : oX[0] - oE[0], k2 ? oX[1] - oE[1] : oX[2] - oE[2]);
        }
        __builtin_amdgcn_sched_barrier(0);
        const R L = (R)(chiA - chiB);
        R gB, hB;
        kernel(chiB, gB, hB);
        if constexpr (kMode == kNgp) {
          add_ngp(ngp, chiB, L);
        } else {
          const PieceForm<R> q = form_general(Face<R>(E), Face<R>(X), fA, fB);
          PieceForm<R> q2 = q;
          if constexpr (kTwo) q2 = form_general(Face<R>(E2), Face<R>(X2), fA, fB);
          add_piece(q, q2, L, gA, gB, hA, hB, (R)0);
        }
        gA = gB;
        hA = hB;
        chiA = chiB;
#pragma unroll
        for (int k = 0; k < 3; ++k) fA[k] = fB[k];
        enter_cell(fA, m0, m1);
        if constexpr (kMode != kNgp) {
          rec.hold(sum);
          R F[4], F2[4];
          rec.project(P, F, F2);
          shift_face(E, X, m0, m1, F);
          if constexpr (kTwo) shift_face(E2, X2, m0, m1, F2);
        }
      }
    }
    // ---- one cell of any kind
    if constexpr (kPass) {
      if (chiA <= a.pause_chi) break;   // the rest of the window is a later pass's
    }
    if (count >= maxc) {
      st = RR_RAY_MAX_STEPS;
      break;
    }
    // exit point: chi_B = max(chi_lo, t_exit,x, t_exit,y, t_exit,z)
    double chiB = fmax(fmax(fmax(te[0], te[1]), te[2]), stop);
    if constexpr (kDebug) chiB = chiB == lo ? lo : chiB;   // the bits of chi_lo itself
    bool stepped[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) stepped[k] = te[k] == chiB;

    // local coordinates of the exit point; exactly 1 on the crossed faces
    R fB[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) fB[k] = (R)1 - absd[k] * (R)(chiB - te[k]);
    const R L = (R)(chiA - chiB);
    R gB, hB;
    kernel(chiB, gB, hB);
    if constexpr (kMode == kNgp) {
      add_ngp(point_value<R, Off, kMode>(tv, cell_offset(), P), chiB, L);
    } else {
      const PieceForm<R> q = form_general(Face<R>(E), Face<R>(X), fA, fB);
      PieceForm<R> q2 = q;
      R surface = 0;
      if constexpr (kTwo) {
        // Eq. (kappa2): c delta against g, n . grad Phi against dg/dchi, and the
        // step's surface term -[g n . grad Phi] at its first and last point
        q2 = form_general(Face<R>(E2), Face<R>(X2), fA, fB);
        if (chiA == B.chi_hi) surface -= (R)12 * gA * q2.u0;
        if (chiB == lo) surface += (R)12 * gB * q2.u1;
      }
      add_piece(q, q2, L, gA, gB, hA, hB, surface);
    }
    gA = gB;
    hA = hB;
    record_piece(chiB);
    ++count;
    if constexpr (kMode == kSources) {
      if (src_j == chiB) {
        // hand out the two integrals accumulated since the previous stop
        if (own) {
          double* pc = a.pieces + (out * a.n_src + jn) * 2;
          pc[0] = (double)sum - (double)comp;
          pc[1] = (double)sum2 - (double)comp2;
        }
        sum = 0; comp = 0.0f; sum2 = 0; comp2 = 0.0f;
        ++jn;
        src_j = jn < a.n_src ? a.src[jn] : -1.0;
      }
    }
    if (chiB == lo) {
      chiA = lo;
      break;
    }
    chiA = chiB;
    // step every axis whose exit plane is at chi_B
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      fA[k] = fB[k];
      if (stepped[k]) {
        fA[k] = (R)0;
        next_layer(k);
      }
    }
    if constexpr (kMode == kNgp) continue;   // one record per cell: nothing carried over
    const int n_stepped = (int)stepped[0] + (int)stepped[1] + (int)stepped[2];
    if (kMode == kSources && n_stepped == 0) continue;   // a source inside the cell: same corners
    if (n_stepped == 1) {
      // one face crossed (axis k): its four values stay, the new exit face
      // comes in, corners F_j (j = i_a + 2 i_b over the two other axes a < b)
      const bool k0 = stepped[0], k1 = stepped[1];
      const Off w0 = (k0 ? oX[0] : oE[0]) + (k1 ? oX[1] : oE[1]) +
                     (k0 || k1 ? oE[2] : oX[2]);
      const Off da = k0 ? oX[1] - oE[1] : oX[0] - oE[0];
      const Off db = k0 || k1 ? oX[2] - oE[2] : oX[1] - oE[1];
      R F[4], F2[4];
      load_face<R, Off, kMode>(tv, w0, da, db, P, F, F2);
      const unsigned long long m0 = __ballot(k0), m1 = __ballot(k1);
      shift_face(E, X, m0, m1, F);
      if constexpr (kTwo) shift_face(E2, X2, m0, m1, F2);
    } else {
      load_cell();
    }
  }
  // a ray that ended without reaching chi_lo or an error stopped at a pass boundary
  const bool paused = st == RR_RAY_OK && chiA > lo;
  if (!own) return;
  if (!(sum == sum) || sum - sum != (R)0) st = RR_RAY_NONFINITE;
  if constexpr (kMode == kSources) {
    if (!(sum2 == sum2) || sum2 - sum2 != (R)0) st = RR_RAY_NONFINITE;
    if constexpr (sizeof(R) == 4)
      reinterpret_cast<float4*>(a.kappa)[out] = make_float4(sum, comp, sum2, comp2);
    else
      reinterpret_cast<double2*>(a.kappa)[out] = make_double2(sum, sum2);
  } else if constexpr (sizeof(R) == 4) {
    reinterpret_cast<float*>(a.kappa)[out] = sum;
    if (a.kappa_comp) a.kappa_comp[out] = comp;
  } else {
    reinterpret_cast<double*>(a.kappa)[out] = sum;
  }
  // stopped at the pass boundary: the next pass starts on the face ahead
  if constexpr (kPass) a.resume[out] = paused ? chiA : -INFINITY;
  if (a.status) a.status[out] = st;
  if constexpr (kDebug) {
    if (a.hash) a.hash[out] = hv;
    if (a.count) a.count[out] = count;
  }
}

template <typename R, bool kDebug, typename Off, int kMode, bool kPass, bool kRun>
__device__ __forceinline__ void run_tile(const R* __restrict__ tv, const TraceArgs& a,
                                         int64_t tile, int lane) {
  const int b = find_bundle(a.bundles, a.n_bundles, tile);
  const DevBundle& B = a.bundles[b];
  int tx, ty;
  zorder_tile(tile - B.tile_begin, B.tiles_x, B.tiles_y, tx, ty);
  // lanes in Z order: a quad is a 2 x 2 block of rays.  At the ragged edge of
  // a map the lanes beyond it walk the map's last ray again and write nothing,
  // so that their quads stay whole.
  int ix, iy;
  zorder_lane(lane, ix, iy);
  ix += tx * 8;
  iy += ty * 8;
  const bool own = ix < B.nx && iy < B.ny;
  ix = min(ix, B.nx - 1);
  iy = min(iy, B.ny - 1);
  trace_one<R, kDebug, Off, kMode, kPass, kRun>(tv, a, B, (int64_t)iy * B.nx + ix, own);
}

// Wavefronts per SIMD that the register budget is held to: four (128 VGPRs)
// for FP32 with 32-bit offsets, three where 64-bit offsets would spill more
// under that cap; FP64 takes what it needs (three: 32 registers spilled, 24.0
// against 16.0 ms for five 512^3 segments).  Five (96 VGPRs, 14 spilled) gained
// nothing: 0.95 against 0.89 ms per 512^3 segment of 2048^2 rays; Method A,
// which spills at four (4 registers in a direct launch, 12 in a persistent one, 8
// in the direct one timed), took 8.4 ms for five segments against 8.8 at three
// (both pairs timed before the re-alignment of lanes a layer apart).  Without
// runs: four as well, and what they need for the others (FP32 at five 0.6 of the
// speed, FP64 at three 0.8 to 1).
template <typename R, typename Off, bool kRun>
constexpr int waves_per_simd() {
  if (!kRun) return sizeof(R) == 4 && sizeof(Off) == 4 ? 4 : 1;
  return sizeof(R) == 8 ? 1 : (sizeof(Off) == 4 ? 4 : 3);
}

// One wavefront per tile.  Workgroups are dealt round-robin to the 8 XCDs;
// remap so that XCD x gets the x-th contiguous slice of tiles.
template <typename R, bool kDebug, typename Off, int kMode, bool kPass, bool kRun>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(waves_per_simd<R, Off, kRun>())))
void march_uniform_kernel(const R* __restrict__ tv, TraceArgs a) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t nblk = gridDim.x;
  const int64_t blk = blockIdx.x;
  const int64_t per = (nblk + 7) / 8;
  const int64_t xcd = blk % 8, slot = blk / 8;
  const int64_t vblk = xcd * per + slot;
  // the tile is the same for the 64 lanes: keep it (and the bundle) scalar
  const int64_t tile = vblk * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane(wave);
  if (tile >= a.n_tiles) return;
  run_tile<R, kDebug, Off, kMode, kPass, kRun>(tv, a, tile, lane);
}

// Persistent workgroups: every wavefront pulls tiles from its chiplet's
// counter, then from the others', until all are drained (every wave reaches
// the exit test).  The tile is the same for the 64 lanes: it (and the
// bundle) stays scalar.
template <typename R, bool kDebug, typename Off, int kMode, bool kPass, bool kRun>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(waves_per_simd<R, Off, kRun>())))
void march_uniform_persistent(const R* __restrict__ tv, TraceArgs a) {
  const int lane = threadIdx.x & 63;
  int q = blockIdx.x % kQueues, tried = 0;
  for (;;) {
    const int64_t tile = next_tile(a.queue, a.n_tiles, q, tried, lane);
    if (tile < 0) break;
    run_tile<R, kDebug, Off, kMode, kPass, kRun>(tv, a, tile, lane);
  }
}

__global__ void queue_reset_kernel(unsigned long long* q) {
  if (threadIdx.x < kQueues) q[threadIdx.x] = 0ull;
}

__global__ __launch_bounds__(256) void fill_kernel(double* __restrict__ p, int64_t n, double v) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = v;
}

// kappa of every source (Eqs. Isources, Isources1) once the walk has reached
// the observer: the moment state holds what lies below the nearest source,
// and summing the pieces from the observer outwards gives int chi Q and
// int chi^2 Q below each source in turn, kappa_j = A_j - B_j / chi_s,j.
// FP64 throughout; one thread per ray, eight sources at a time staged through
// LDS so that pieces and kappa (ray-major) move as 128- and 64-byte runs: 245 ->
// 79 us for 1024^2 rays and ten sources, whose 252 MB take 53 us at the
// memory's copy rate.
constexpr int kPieceTile = 8;
// The integrals below the nearest source: the walk's moment state of ray r.
__device__ __forceinline__ void start_sums(const float* mom, int64_t r, double& A, double& B) {
  const float4 m = reinterpret_cast<const float4*>(mom)[r];
  A = (double)m.x - (double)m.y;
  B = (double)m.z - (double)m.w;
}
__device__ __forceinline__ void start_sums(const double* mom, int64_t r, double& A, double& B) {
  const double2 m = reinterpret_cast<const double2*>(mom)[r];
  A = m.x;
  B = m.y;
}
template <typename R>
__global__ __launch_bounds__(256) void kappa_from_pieces_kernel(const R* __restrict__ mom,
                                                                const double* __restrict__ pieces,
                                                                const double* __restrict__ src,
                                                                int ns, int64_t nr,
                                                                double* __restrict__ kappa) {
  // two doubles at any address that holds one: all that the caller promises
  typedef double pair_t __attribute__((ext_vector_type(2), aligned(8)));
  __shared__ double2 pc[256][kPieceTile + 1];
  const int64_t r0 = (int64_t)blockIdx.x * 256;
  const int rays = (int)(nr - r0 < 256 ? nr - r0 : 256);
  const int t = threadIdx.x;
  double A = 0.0, B = 0.0;
  if (t < rays) start_sums(mom, r0 + t, A, B);
  for (int j1 = ns; j1 > 0; j1 -= kPieceTile) {
    const int j0 = j1 > kPieceTile ? j1 - kPieceTile : 0;   // sources j0 .. j1 - 1
    __syncthreads();
    for (int e = t; e < 256 * kPieceTile; e += 256) {
      const int r = e / kPieceTile, j = j0 + e % kPieceTile;
      if (r < rays && j < j1) {
        const pair_t p = *reinterpret_cast<const pair_t*>(pieces + 2 * ((r0 + r) * ns + j));
        pc[r][e % kPieceTile] = make_double2(p.x, p.y);
      }
    }
    __syncthreads();
    for (int j = j1 - 1; j >= j0; --j) {
      const double2 p = pc[t][j - j0];
      pc[t][j - j0].x = A - B / src[j];
      A += p.x;
      B += p.y;
    }
    __syncthreads();
    for (int e = t; e < 256 * kPieceTile; e += 256) {
      const int r = e / kPieceTile, j = j0 + e % kPieceTile;
      if (r < rays && j < j1) kappa[(r0 + r) * ns + j] = pc[r][e % kPieceTile].x;
    }
  }
}

// The same for few sources, whose pieces lie close enough for one thread to read
// them in place (launch_kappa_from_pieces).
template <typename R>
__global__ __launch_bounds__(256) void kappa_from_few_pieces_kernel(
    const R* __restrict__ mom, const double* __restrict__ pieces, const double* __restrict__ src,
    int ns, int64_t nr, double* __restrict__ kappa) {
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= nr) return;
  double A, B;
  start_sums(mom, r, A, B);
  for (int j = ns - 1; j >= 0; --j) {
    kappa[r * ns + j] = A - B / src[j];
    A += pieces[(r * ns + j) * 2 + 0];
    B += pieces[(r * ns + j) * 2 + 1];
  }
}

template <typename R, bool kDebug, typename Off, int kMode, bool kPass, bool kRun>
hipError_t launch3(const void* tv, const TraceArgs& a, int persistent, int block, int grid_waves,
                   hipStream_t s) {
  const int wpb = block / 64;
  if (persistent) {
    const int blocks = (grid_waves + wpb - 1) / wpb;
    hipLaunchKernelGGL((march_uniform_persistent<R, kDebug, Off, kMode, kPass, kRun>), dim3(blocks), dim3(block), 0, s,
                       (const R*)tv, a);
  } else {
    int64_t blocks = (a.n_tiles + wpb - 1) / wpb;
    if (blocks == 0) return hipSuccess;
    blocks = (blocks + 7) / 8 * 8;   // the XCD remap is a bijection on multiples of 8
    hipLaunchKernelGGL((march_uniform_kernel<R, kDebug, Off, kMode, kPass, kRun>), dim3((unsigned)blocks), dim3(block),
                       0, s, (const R*)tv, a);
  }
  return hipGetLastError();
}

// Runs keep no count and test no domain, so launches with debug outputs, a
// crossing limit or an open grid cannot use them, and pay for the registers
// they hold where they are compiled in: 256^3 open grid, 1400^2 rays over 8
// degrees, Method A in FP64 2.95 ms with runs compiled in and each cell taken as
// one of any kind, 2.09 without runs and single faces crossed as between them;
// FP32 kappa off the axes 1.90 against 1.82.
template <typename R, typename Off, int kMode>
hipError_t launch_off(const void* tv, const TraceArgs& a, int persistent, int block,
                      int grid_waves, hipStream_t s) {
  const bool dbg = a.hash || a.log || a.count;
  const bool run = !a.open && a.max_crossings <= 0;
  // split marches never carry debug outputs (the host keeps those in one pass)
  if (a.resume)
    return run ? launch3<R, false, Off, kMode, true, true>(tv, a, persistent, block, grid_waves, s)
               : launch3<R, false, Off, kMode, true, false>(tv, a, persistent, block, grid_waves, s);
  if (dbg)
    return launch3<R, true, Off, kMode, false, false>(tv, a, persistent, block, grid_waves, s);
  return run ? launch3<R, false, Off, kMode, false, true>(tv, a, persistent, block, grid_waves, s)
             : launch3<R, false, Off, kMode, false, false>(tv, a, persistent, block, grid_waves, s);
}

template <typename R, int kMode>
hipError_t launch_mode(const void* tv, const TraceArgs& a, bool small, int persistent, int block,
                       int grid_waves, hipStream_t s) {
  return small ? launch_off<R, uint32_t, kMode>(tv, a, persistent, block, grid_waves, s)
               : launch_off<R, uint64_t, kMode>(tv, a, persistent, block, grid_waves, s);
}

template <typename R>
hipError_t launch(const void* tv, const TraceArgs& a, int persistent, int block, int grid_waves,
                  hipStream_t s) {
  // 32-bit byte offsets when the whole tensor is below 4 GiB
  const int words = a.mode == kMethodA ? 4 : (a.mode == kScalar ? 1 : 6);
  const bool small = (int64_t)a.n * a.n * a.n * (int64_t)(words * sizeof(R)) < (1ll << 32);
  switch (a.mode) {
    case kNgp: return launch_mode<R, kNgp>(tv, a, small, persistent, block, grid_waves, s);
    case kMethodA: return launch_mode<R, kMethodA>(tv, a, small, persistent, block, grid_waves, s);
    case kSources: return launch_mode<R, kSources>(tv, a, small, persistent, block, grid_waves, s);
    case kScalar: return launch_mode<R, kScalar>(tv, a, small, persistent, block, grid_waves, s);
    default: return launch_mode<R, kTidal>(tv, a, small, persistent, block, grid_waves, s);
  }
}

}  // namespace

hipError_t launch_march_uniform(int precision, const void* tv, const TraceArgs& a, int persistent,
                                int block, int grid_waves, hipStream_t s) {
  if (precision == RR_PREC_FP32_KAHAN) return launch<float>(tv, a, persistent, block, grid_waves, s);
  return launch<double>(tv, a, persistent, block, grid_waves, s);
}

namespace {
template <typename R>
hipError_t launch_pieces(const R* moments, const double* pieces, const double* src, int n_src,
                         int64_t n_rays, double* kappa, hipStream_t s) {
  const dim3 blocks((unsigned)((n_rays + 255) / 256));
  // 1024^2 rays, FP32, in place / through LDS: one source 12.0 us / 19.5, two 12.6 /
  // 21.6, three 19.8 / 22.5, four 31.0 / 24.5, five 51.4 / 27.3, eight 181 / 38
  if (n_src <= 3)
    hipLaunchKernelGGL(kappa_from_few_pieces_kernel<R>, blocks, dim3(256), 0, s, moments, pieces,
                       src, n_src, n_rays, kappa);
  else
    hipLaunchKernelGGL(kappa_from_pieces_kernel<R>, blocks, dim3(256), 0, s, moments, pieces, src,
                       n_src, n_rays, kappa);
  return hipGetLastError();
}
}  // namespace

hipError_t launch_kappa_from_pieces(int precision, const void* moments, const double* pieces,
                                    const double* src, int n_src, int64_t n_rays, double* kappa,
                                    hipStream_t s) {
  if (n_rays == 0) return hipSuccess;
  if (precision == RR_PREC_FP32_KAHAN)
    return launch_pieces((const float*)moments, pieces, src, n_src, n_rays, kappa, s);
  return launch_pieces((const double*)moments, pieces, src, n_src, n_rays, kappa, s);
}

hipError_t launch_fill(double* p, int64_t n, double v, hipStream_t s) {
  const int64_t blocks = (n + 255) / 256;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_queue_reset(unsigned long long* q, hipStream_t s) {
  hipLaunchKernelGGL(queue_reset_kernel, dim3(1), dim3(64), 0, s, q);
  return hipGetLastError();
}

}  // namespace rr
