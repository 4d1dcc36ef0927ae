// rr_tensor_uniform.hip -- tidal tensor at cell centres (Eq. tidalexample) fused
// with its interpolation to cell vertices (Sec. III H, regular vertices).
//
// Vertex (i,j,k) is the lower corner of cell (i,j,k) and takes the mean of the
// centre tensors of cells {i-1,i} x {j-1,j} x {k-1,k}.  Summing the centre
// stencils over those eight cells factorises per axis into
//   second difference summed over two cells: S f(i) = (f(i+1) - f(i)) - (f(i-1) - f(i-2))
//   first difference summed over two cells:  D f(i) = (f(i+1) - f(i-1)) + (f(i) - f(i-2))
//   plain sum over the two cells:            B f(i) = f(i-1) + f(i)
// so that   T_xx = (1/8) S_x B_y B_z Phi,   T_xy = (1/32) D_x D_y B_z Phi, ...
// Differences are always taken first on the raw potential (exact for
// neighbours within a factor two, Sterbenz), sums afterwards.
//
// The vertices built are a periodic box [o, o + size) of the lattice (the
// whole grid, or the part a set of rays can reach).
//
// Layout of the work: a workgroup owns a 64 x TY column of vertices in x-y
// and marches KZ vertices along z.  Each step stages one potential plane
// (plus a two-cell halo) in LDS; every thread reads its 4 x 4 patch of that
// plane once and keeps the per-plane partial stencils of the last four planes
// in registers, so each vertex costs 16 LDS reads and ~80 arithmetic
// operations.  Large grids and boxes take columns of 64 x 8 x 8 (512 threads) or
// 64 x 16 x 16 (1024 threads; staging with the halo reads 1.5 potential values per
// vertex) and, beyond the last-level cache, write the records with non-temporal
// stores; small ones take columns of 64 x 4 with 256 threads and ordinary
// stores, since the march reads them right away (launch_vt).
#include "rr_internal.hpp"

namespace rr {
namespace {

constexpr int TX = 64;                  // vertices per workgroup in x

__device__ inline int wrapi(int i, int n) {
  i %= n;
  return i < 0 ? i + n : i;
}

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

template <bool kNT>
__device__ inline void store_vertex(float* dst, const float* r) {
  f32x2* d = reinterpret_cast<f32x2*>(dst);
  const f32x2 a = {r[0], r[1]}, b = {r[2], r[3]}, c = {r[4], r[5]};
  if constexpr (kNT) {
    __builtin_nontemporal_store(a, d);
    __builtin_nontemporal_store(b, d + 1);
    __builtin_nontemporal_store(c, d + 2);
  } else {
    d[0] = a; d[1] = b; d[2] = c;
  }
}
template <bool kNT>
__device__ inline void store_vertex(double* dst, const double* r) {
  f64x2* d = reinterpret_cast<f64x2*>(dst);
  const f64x2 a = {r[0], r[1]}, b = {r[2], r[3]}, c = {r[4], r[5]};
  if constexpr (kNT) {
    __builtin_nontemporal_store(a, d);
    __builtin_nontemporal_store(b, d + 1);
    __builtin_nontemporal_store(c, d + 2);
  } else {
    d[0] = a; d[1] = b; d[2] = c;
  }
}

struct VertexBox {
  int ox, oy, oz;   // origin, wrapped into [0, n)
  int sx, sy, sz;   // extent, at most n
  int ntx, nty;     // workgroup tiles in x and y
};

template <typename In, typename Acc, int TY, int KZ, bool kNT, bool kRows>
__global__ __launch_bounds__(64 * TY) void vertex_tensor_uniform_kernel(const In* __restrict__ phi,
                                                                        Acc* __restrict__ tv,
                                                                        int n, int open,
                                                                        VertexBox V) {
  constexpr int RW = VertexRecord<Acc>::kWords;
  constexpr int NT = TX * TY;                 // threads
  constexpr int PX = TX + 3, PY = TY + 3;     // staged plane: halo 2 below, 1 above
  __shared__ Acc plane[2][PY * PX];
  // kRows: records leave through LDS, each wavefront (one row of 64 vertices)
  // writes its row with contiguous stores instead of three per lane at the stride
  // of a record.  512^3 FP64: 2.2 -> 1.8 ms, and 1.38 with the next plane read
  // ahead; 192^3 FP64 0.144 (64 x 4 x 32, per-lane stores) -> 0.073.  FP32 in
  // 64 x 16 columns keeps per-lane stores: there staging costs the second
  // workgroup per CU.
  __shared__ __align__(16) Acc rowbuf[kRows ? TY : 1][kRows ? TX * RW : 1];

  const int b = blockIdx.x;
  const int bx = b % V.ntx;
  const int by = (b / V.ntx) % V.nty;
  const int bz = b / (V.ntx * V.nty);
  // box-local origin of this workgroup's column; lattice indices wrap
  const int li0 = bx * TX, lj0 = by * TY, lk0 = bz * KZ;
  const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
  const bool mine = li0 + tx < V.sx && lj0 + ty < V.sy;
  int i = V.ox + li0 + tx, j = V.oy + lj0 + ty;
  i = i >= n ? i - n : i;
  j = j >= n ? j - n : j;
  const int64_t nn = (int64_t)n * n;
  // the wavefront's row of n_row vertices does not wrap
  int i_row = V.ox + li0;
  i_row = i_row >= n ? i_row - n : i_row;
  const int n_row = min(TX, V.sx - li0);
  const bool row_ok = kRows && i_row + n_row <= n;

  // per-plane partial stencils, history over planes (index 0 = oldest)
  Acc XX[2], YY[2], XY[2];     // planes k-1, k
  Acc Z[4][4];                 // raw Phi of the 2x2 column box, planes k-2..k+1
  Acc DX[4][2], DY[4][2];      // D_x on rows j-1, j and D_y on columns i-1, i, planes k-2..k+1

  // staging: each thread copies at most two elements of every plane; their
  // (wrapped) x-y offsets are fixed for the whole march
  constexpr int kStage = (PX * PY + NT - 1) / NT;
  int soff[kStage];
  bool sin_[kStage], sact[kStage];
#pragma unroll
  for (int u = 0; u < kStage; ++u) {
    const int e = threadIdx.x + NT * u;
    sact[u] = e < PX * PY;
    const int lx = e % PX, ly = e / PX;
    // unwrapped lattice coordinates (the open boundary pads outside [0, n))
    const int gx = V.ox + li0 - 2 + lx, gy = V.oy + lj0 - 2 + ly;
    sin_[u] = gx >= 0 && gy >= 0 && gx < n && gy < n;
    int wx = gx % n, wy = gy % n;
    wx = wx < 0 ? wx + n : wx;
    wy = wy < 0 ? wy + n : wy;
    soff[u] = wy * n + wx;
  }

  const int k0 = V.oz + lk0;                       // unwrapped
  const int k_end = k0 + min(KZ, V.sz - lk0);
  int slot = 0;
  int gz = (k0 - 2) % n;
  if (gz < 0) gz += n;
  // this thread's part of plane p (x fastest, wrapped or zero-padded), read
  // one plane ahead, so that the loads of plane p + 1 are in flight while
  // plane p is differenced and its vertices stored.  FP64 records written
  // with three per-lane stores each (vertex boxes) read each plane when it
  // is staged: there reading ahead was slower (3.3 against 2.2 ms for
  // 512^3); with their rows leaving through LDS it is faster (1.76 -> 1.38).
  constexpr bool kAhead = sizeof(Acc) == 4 || kRows;
  In pre[kStage];
  auto fetch = [&](int p, int gzp) {
    const bool zin = p >= 0 && p < n;
    const In* src = phi + (int64_t)gzp * nn;
#pragma unroll
    for (int u = 0; u < kStage; ++u) {
      if (!sact[u] || (open && !(sin_[u] && zin)))
        pre[u] = (In)0;
      else
        pre[u] = src[soff[u]];
    }
  };
  if constexpr (kAhead) fetch(k0 - 2, gz);
  for (int p = k0 - 2; p <= k_end; ++p, slot ^= 1) {
    Acc* pl = plane[slot];
    if constexpr (!kAhead) fetch(p, gz);
#pragma unroll
    for (int u = 0; u < kStage; ++u)
      if (sact[u]) pl[threadIdx.x + NT * u] = (Acc)pre[u];
    if (++gz == n) gz = 0;
    __syncthreads();
    if constexpr (kAhead) {
      if (p < k_end) fetch(p + 1, gz);
    }
    // 4x4 patch: rows y = j-2..j+1, columns x = i-2..i+1
    Acc q[4][4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < 4; ++c) q[r][c] = pl[(ty + r) * PX + (tx + c)];

    Acc dx[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) dx[r] = (q[r][3] - q[r][1]) + (q[r][2] - q[r][0]);
    const Acc sxx = ((q[1][3] - q[1][2]) - (q[1][1] - q[1][0])) +
                    ((q[2][3] - q[2][2]) - (q[2][1] - q[2][0]));
    const Acc syy = ((q[3][1] - q[2][1]) - (q[1][1] - q[0][1])) +
                    ((q[3][2] - q[2][2]) - (q[1][2] - q[0][2]));
    const Acc dxy = (dx[3] - dx[1]) + (dx[2] - dx[0]);
    const Acc dy1 = (q[3][1] - q[1][1]) + (q[2][1] - q[0][1]);
    const Acc dy2 = (q[3][2] - q[1][2]) + (q[2][2] - q[0][2]);

    // shift the z histories so that Z/DX/DY[0..3] hold planes p-3..p
#pragma unroll
    for (int h = 0; h < 3; ++h) {
#pragma unroll
      for (int c = 0; c < 4; ++c) Z[h][c] = Z[h + 1][c];
      DX[h][0] = DX[h + 1][0]; DX[h][1] = DX[h + 1][1];
      DY[h][0] = DY[h + 1][0]; DY[h][1] = DY[h + 1][1];
    }
    Z[3][0] = q[1][1]; Z[3][1] = q[1][2]; Z[3][2] = q[2][1]; Z[3][3] = q[2][2];
    DX[3][0] = dx[1]; DX[3][1] = dx[2];
    DY[3][0] = dy1; DY[3][1] = dy2;

    if (p >= k0 + 1 && lj0 + ty < V.sy) {
      // vertex k = p - 1: Z/DX/DY[0..3] are planes k-2..k+1; XX/YY/XY[0..1] are k-1, k
      const int k = p - 1 >= n ? p - 1 - n : p - 1;
      Acc rec[6];
      rec[0] = (XX[0] + XX[1]) * (Acc)0.125;
      rec[1] = (YY[0] + YY[1]) * (Acc)0.125;
      Acc zz = 0;
#pragma unroll
      for (int c = 0; c < 4; ++c) zz += (Z[3][c] - Z[2][c]) - (Z[1][c] - Z[0][c]);
      rec[2] = zz * (Acc)0.125;
      rec[3] = (XY[0] + XY[1]) * (Acc)0.03125;
      Acc xz = 0, yz = 0;
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        xz += (DX[3][c] - DX[1][c]) + (DX[2][c] - DX[0][c]);
        yz += (DY[3][c] - DY[1][c]) + (DY[2][c] - DY[0][c]);
      }
      rec[4] = xz * (Acc)0.03125;
      rec[5] = yz * (Acc)0.03125;
      if (open && (i < 2 || j < 2 || k < 2 || i > n - 2 || j > n - 2 || k > n - 2)) {
        const Acc nan = (Acc)__builtin_nan("");
#pragma unroll
        for (int c = 0; c < 6; ++c) rec[c] = nan;
      }
      if (row_ok) {
        // lanes write their records side by side in LDS, then read back
        // chunks of the row in order: 16 bytes in FP64, 8 in FP32, whose rows
        // start at any multiple of 8 (LDS operations of one wavefront complete
        // in order; the empty asm statements keep the compiler from moving the
        // accesses across each other)
        Acc* rb = rowbuf[kRows ? ty : 0];
        typedef Acc chunk_t __attribute__((ext_vector_type(2)));
        constexpr int kChunks = RW / 2;      // per record
        chunk_t* rc = reinterpret_cast<chunk_t*>(rb);
#pragma unroll
        for (int c = 0; c < kChunks; ++c) rc[tx * kChunks + c] = chunk_t{rec[2 * c], rec[2 * c + 1]};
        __asm__ volatile("" ::: "memory");
        chunk_t* dst =
            reinterpret_cast<chunk_t*>(tv + ((int64_t)k * nn + (int64_t)j * n + i_row) * RW);
#pragma unroll
        for (int m = tx; m < TX * kChunks; m += TX)
          if (m < n_row * kChunks) {
            if constexpr (kNT) __builtin_nontemporal_store(rc[m], dst + m);
            else dst[m] = rc[m];
          }
        __asm__ volatile("" ::: "memory");
      } else if (mine) {
        store_vertex<kNT>(tv + ((int64_t)k * nn + (int64_t)j * n + i) * RW, rec);
      }
    }
    // XX/YY/XY hold planes (p-2, p-1) during step p; push plane p
    XX[0] = XX[1]; YY[0] = YY[1]; XY[0] = XY[1];
    XX[1] = sxx; YY[1] = syy; XY[1] = dxy;
  }
}

// Cell-centre tensor (Eq. tidalexample, cell size 1) for the nearest-grid-point
// integral (Eq. Iclensing_ngp).  Second differences as differences of
// differences, mixed ones over the four diagonal neighbours; open grids leave
// the outer cell layer NaN (no stencil).
//
// Memory bound (4 bytes in, 24 out in FP32).  A wavefront owns a row of 64
// cells and marches kz cells along z, reading nine values of each plane and
// keeping three planes in registers; its records leave through LDS as
// contiguous stores.  One cell per thread, 19 gathered values each and three
// stores at the stride of a record took 171 us for 256^3 FP32 (2.8 TB/s of
// algorithmic traffic); this takes 94 us (5.0 TB/s);
// 512^3 1345 -> 926, FP64 256^3 368 -> 169.
template <typename In, typename Acc, bool kNT>
__global__ __launch_bounds__(256) void centre_tensor_uniform_kernel(const In* __restrict__ phi,
                                                                    Acc* __restrict__ tc, int n,
                                                                    int open, int kz) {
  typedef Acc chunk_t __attribute__((ext_vector_type(2)));
  __shared__ __align__(16) chunk_t rows[4][TX * 3];
  const int tx = threadIdx.x % TX, ty = threadIdx.x / TX;
  const int i0 = blockIdx.x * TX, j = blockIdx.y * 4 + ty, k0 = blockIdx.z * kz;
  if (j >= n) return;   // whole wavefronts
  const int64_t nn = (int64_t)n * n;
  const int n_row = min(TX, n - i0), i = min(i0 + tx, n - 1);
  const int xs[3] = {i == 0 ? n - 1 : i - 1, i, i + 1 == n ? 0 : i + 1};
  const int ys[3] = {(j == 0 ? n - 1 : j - 1) * n, j * n, (j + 1 == n ? 0 : j + 1) * n};
  In v[3][3];
  auto fetch = [&](int k) {
    const In* src = phi + (int64_t)(k < 0 ? k + n : (k >= n ? k - n : k)) * nn;
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int a = 0; a < 3; ++a) v[b][a] = src[ys[b] + xs[a]];
  };
  // planes k - 1, k, k + 1: the cell's cross (c, x-, x+, y-, y+); plane k also
  // the second differences and the mixed one in x and y
  Acc lo[5], mid[5], hi[5], txx = 0, tyy = 0, txy = 0;
  const int k_end = min(k0 + kz, n);
  auto take = [&](Acc* p) {
    p[0] = (Acc)v[1][1];
    p[1] = (Acc)v[1][0];
    p[2] = (Acc)v[1][2];
    p[3] = (Acc)v[0][1];
    p[4] = (Acc)v[2][1];
  };
  auto in_plane = [&](const Acc* p) {
    txx = (p[2] - p[0]) - (p[0] - p[1]);
    tyy = (p[4] - p[0]) - (p[0] - p[3]);
    txy = (((Acc)v[2][2] - (Acc)v[0][2]) - ((Acc)v[2][0] - (Acc)v[0][0])) * (Acc)0.25;
  };
  fetch(k0 - 1);
  take(lo);
  fetch(k0);
  take(mid);
  in_plane(mid);
  fetch(k0 + 1);
  for (int k = k0; k < k_end; ++k) {
    take(hi);
    Acc rec[6];
    rec[0] = txx;
    rec[1] = tyy;
    rec[2] = (hi[0] - mid[0]) - (mid[0] - lo[0]);
    rec[3] = txy;
    rec[4] = ((hi[2] - lo[2]) - (hi[1] - lo[1])) * (Acc)0.25;
    rec[5] = ((hi[4] - lo[4]) - (hi[3] - lo[3])) * (Acc)0.25;
    if (open && (i < 1 || j < 1 || k < 1 || i > n - 2 || j > n - 2 || k > n - 2)) {
#pragma unroll
      for (int u = 0; u < 6; ++u) rec[u] = (Acc)__builtin_nan("");
    }
    in_plane(hi);
    if (k + 1 < k_end) fetch(k + 2);   // in flight while the row is stored
#pragma unroll
    for (int u = 0; u < 5; ++u) {
      lo[u] = mid[u];
      mid[u] = hi[u];
    }
    // LDS operations of one wavefront complete in order; the empty statements
    // keep the compiler from moving the accesses across each other
    chunk_t* rc = rows[ty];
#pragma unroll
    for (int u = 0; u < 3; ++u) rc[tx * 3 + u] = chunk_t{rec[2 * u], rec[2 * u + 1]};
    __asm__ volatile("" ::: "memory");
    chunk_t* dst = reinterpret_cast<chunk_t*>(tc + ((int64_t)k * nn + (int64_t)j * n + i0) * 6);
#pragma unroll
    for (int m = tx; m < TX * 3; m += TX)
      if (m < n_row * 3) {
        if constexpr (kNT) __builtin_nontemporal_store(rc[m], dst + m);
        else dst[m] = rc[m];
      }
    __asm__ volatile("" ::: "memory");
  }
}

template <typename In, typename Acc>
hipError_t launch_ct(int n, int open, const void* phi, void* tc, hipStream_t s) {
  // cells along z per workgroup: 16, fewer where that leaves the chip short of
  // four workgroups per compute unit
  const int ntx = (n + TX - 1) / TX, nty = (n + 3) / 4;
  int kz = 16;
  while (kz > 2 && (int64_t)ntx * nty * ((n + kz - 1) / kz) < 1024) kz /= 2;
  const dim3 grid(ntx, nty, (n + kz - 1) / kz);
  // records beyond the last-level cache are stored past it
  if ((int64_t)n * n * n * 6 * (int64_t)sizeof(Acc) > (256ll << 20))
    hipLaunchKernelGGL((centre_tensor_uniform_kernel<In, Acc, true>), grid, dim3(256), 0, s,
                       (const In*)phi, (Acc*)tc, n, open, kz);
  else
    hipLaunchKernelGGL((centre_tensor_uniform_kernel<In, Acc, false>), grid, dim3(256), 0, s,
                       (const In*)phi, (Acc*)tc, n, open, kz);
  return hipGetLastError();
}

template <typename In, typename Acc, int TY, int KZ, bool kNT,
          bool kRows = kNT && (sizeof(Acc) == 8 || TY != 16)>
hipError_t launch_shape(const VertexBox& box, int n, int open, const void* phi, void* tv,
                        hipStream_t s) {
  VertexBox V = box;
  V.ntx = (V.sx + TX - 1) / TX;
  V.nty = (V.sy + TY - 1) / TY;
  const int ntz = (V.sz + KZ - 1) / KZ;
  const int64_t blocks = (int64_t)V.ntx * V.nty * ntz;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL((vertex_tensor_uniform_kernel<In, Acc, TY, KZ, kNT, kRows>),
                     dim3((unsigned)blocks), dim3(TX * TY), 0, s, (const In*)phi, (Acc*)tv, n,
                     open, V);
  return hipGetLastError();
}

template <typename In, typename Acc>
hipError_t launch_vt(int n, int open, const int* lo, const int* size, const void* phi, void* tv,
                     hipStream_t s) {
  VertexBox V;
  int o[3];
  for (int a = 0; a < 3; ++a) {
    o[a] = lo[a] % n;
    if (o[a] < 0) o[a] += n;
  }
  V.ox = o[0]; V.oy = o[1]; V.oz = o[2];
  V.sx = size[0]; V.sy = size[1]; V.sz = size[2];
  auto columns = [&](int ty, int kz) {
    return (int64_t)((V.sx + TX - 1) / TX) * ((V.sy + ty - 1) / ty) * ((V.sz + kz - 1) / kz);
  };
  // Boxes beyond 1/8 of the grid: rows stored through LDS, in columns of
  // 64 x 8 x 8 unless said otherwise.  They want enough columns (us, in 64 x 4 /
  // 64 x 8 x 8 columns): FP64 64^3, 64 columns, 10.2 / 13.5, 80^3, 200, 18.7 / 13.7;
  // FP32 128^3, 512, 17.0 / 14.7 but even or 1 to 3 % behind in a step of build and
  // march up to 136^3, 867; 144^3, 972, 27.7 / 30.7 with another potential each
  // time; 160^3, 1200, 31.1 / 29.4; FP32 boxes 125^2 x 250, 1024,
  // 27.6 / 35.2, 144^2 x 288, 1944, 45 / 51, 166^2 x 333, 2646, 79 / 72.
  const int64_t vertices = (int64_t)V.sx * V.sy * V.sz, grid = (int64_t)n * n * n;
  const int64_t rows_from = sizeof(Acc) == 8 ? 128 : (vertices == grid ? 1000 : 2200);
  if (8 * vertices > grid && columns(8, 8) >= rows_from) {
    // Records that the last-level cache holds beside the rest of a step are stored
    // into it: the march reads them next.  Whole steps of drawn maps, time of a
    // limit of 96 MiB over one of 160, and of 160 over 288: FP32 tensors of 96 to
    // 160 MiB 1.03, 160 to 224 MiB 0.97 (0.91 at worst), 224 to 288 MiB 0.98; FP64
    // 1.05 and 1.02.
    if (vertices * 6 * (int64_t)sizeof(Acc) <= (vertices == grid ? 160ll << 20 : 96ll << 20))
      return launch_shape<In, Acc, 8, 8, false, true>(V, n, open, phi, tv, s);
    // Whole rows that start on 64-byte lines fill them from any shape: there the
    // least halo, 64 x 16 x 16, wins on large grids (us, 64 x 16 x 16 / 8 x 8, each
    // build of another potential; FP32 240^3 102 / 101, 256^3 103 / 114, 288^3 152 /
    // 170, 328^3 225 / 277, 400^3 396 / 468, 480^3 665 / 809; FP64 176^3 71 / 67,
    // 208^3 117 / 123, 256^3 166 / 183, 320^3 330 / 368, 480^3 1177 / 1310, slabs of
    // 512^2 x 170 439 / 493), except on FP32 slabs (512^2 x 170 373 / 226).  Other
    // rows share their lines, which the longer bursts of the staged rows mend
    // (FP32 257^3 130 / 113, 333^3 258 / 242, 441^3 567 / 557, 500^3 805 / 741;
    // FP64 257^3 204 / 197, 333^3 423 / 417, 441^3 1025 / 968; boxes of 493 x 491 x
    // 250 in 500^3 FP32 542 / 372, FP64 795 / 758).
    const bool lines = n % (64 / sizeof(Acc) / 2) == 0;
    if constexpr (sizeof(Acc) == 4) {
      if (lines && vertices == grid && n >= 250)
        return launch_shape<In, Acc, 16, 16, true>(V, n, open, phi, tv, s);
    } else if (lines && (vertices == grid ? n >= 190 : V.sx == n && columns(16, 16) >= 2048)) {
      return launch_shape<In, Acc, 16, 16, true>(V, n, open, phi, tv, s);
    }
    return launch_shape<In, Acc, 8, 8, true>(V, n, open, phi, tv, s);
  }
  // Smaller boxes and grids: columns of 64 x 4, as deep as leaves the chip two
  // workgroups per compute unit: 64^3 FP64 29 -> 10 us, the vertex box of a
  // 512^3 cone's segment 22 -> 8 us.
  constexpr int64_t kFill = 512;
  if (columns(4, 32) >= kFill) return launch_shape<In, Acc, 4, 32, false>(V, n, open, phi, tv, s);
  if (columns(4, 8) >= kFill) return launch_shape<In, Acc, 4, 8, false>(V, n, open, phi, tv, s);
  return launch_shape<In, Acc, 4, 4, false>(V, n, open, phi, tv, s);
}

}  // namespace

// Vertices of the periodic box [lo, lo + size) (size[a] <= n; the host
// layer validates).
hipError_t launch_vertex_tensor_uniform(int precision, int dtype, int n, int open, const int* lo,
                                        const int* size, const void* phi, void* tv,
                                        hipStream_t s) {
  if (precision == RR_PREC_FP32_KAHAN) {
    if (dtype == RR_F32) return launch_vt<float, float>(n, open, lo, size, phi, tv, s);
    return launch_vt<double, float>(n, open, lo, size, phi, tv, s);
  }
  if (dtype == RR_F32) return launch_vt<float, double>(n, open, lo, size, phi, tv, s);
  return launch_vt<double, double>(n, open, lo, size, phi, tv, s);
}

hipError_t launch_centre_tensor_uniform(int precision, int dtype, int n, int open,
                                        const void* phi, void* tc, hipStream_t s) {
  if (precision == RR_PREC_FP32_KAHAN) {
    if (dtype == RR_F32) return launch_ct<float, float>(n, open, phi, tc, s);
    return launch_ct<double, float>(n, open, phi, tc, s);
  }
  if (dtype == RR_F32) return launch_ct<float, double>(n, open, phi, tc, s);
  return launch_ct<double, double>(n, open, phi, tc, s);
}

}  // namespace rr
