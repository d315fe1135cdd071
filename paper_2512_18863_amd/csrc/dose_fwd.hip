// dose_fwd.hip — forward kernels of the dose path (arXiv:2512.18863 §2.2.2-2.2.7).
//
// Per control-point batch the forward runs
//   k_raster      fluence map F [b][Nu][Nv]                  (§2.2.2, Eq. 4)
//   k_ca_depth    central-axis depth z [b][Nk]               (§2.2.4, Eq. 7)
//   k_march       primary P = F (SAD/d)^2 DD(W) [b][Nk][Nu][Nv] (§2.2.3-2.2.4, Eqs. 6-7)
//   conv          beam-frame dose Dfan = K_k (*) P_k         (§2.2.5-2.2.6, Eq. 8)
//   k_gather      dose += MU_b trilinear(Dfan_b)             (§2.2.7, Eq. 9)
// k_frame and k_transpose_rho prepare per-call constants.
#include <type_traits>

#include "taps.hpp"

namespace pdrt {

// ------------------------------------------------------------------ setup

template <typename T>
__global__ void k_frame(const T* __restrict__ gantry, int n_cp, T* __restrict__ frame) {
  int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= n_cp) return;
  double sn, cs;
  sincospi((double)gantry[b] / 180.0, &sn, &cs);
  frame[2 * b] = (T)sn;
  frame[2 * b + 1] = (T)cs;
}

template <typename T>
hipError_t launch_frame(const Geo<T>& g, const T* gantry, int n_cp, T* frame, hipStream_t s) {
  (void)g;
  hipLaunchKernelGGL(k_frame<T>, dim3((n_cp + 255) / 256), dim3(256), 0, s, gantry, n_cp, frame);
  return hipGetLastError();
}

struct HuTable {
  int n;
  float hu[16], rho[16];
};

// HU -> relative density: piecewise-linear calibration curve, clamped (§2.2).
__global__ void k_hu_to_density(long n, const float* __restrict__ hu, float* __restrict__ rho, HuTable t) {
  long q = (long)blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= n) return;
  float h = hu[q];
  float r;
  if (h <= t.hu[0]) {
    r = t.rho[0];
  } else if (h >= t.hu[t.n - 1]) {
    r = t.rho[t.n - 1];
  } else {
    int s = 0;
    while (h > t.hu[s + 1]) ++s;
    float f = (h - t.hu[s]) / (t.hu[s + 1] - t.hu[s]);
    r = t.rho[s] + f * (t.rho[s + 1] - t.rho[s]);
  }
  rho[q] = r;
}

hipError_t launch_hu_to_density(long n, const float* hu, float* rho, int n_pts, const float* hp, const float* rp,
                                hipStream_t s) {
  HuTable t;
  t.n = n_pts;
  for (int i = 0; i < n_pts; ++i) {
    t.hu[i] = hp[i];
    t.rho[i] = rp[i];
  }
  hipLaunchKernelGGL(k_hu_to_density, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, n, hu, rho, t);
  return hipGetLastError();
}

// rho [nz][ny][nx] -> rho_t [ny][nx][nz] (per y slice, a tiled 2-D transpose).
template <typename T>
__global__ void __launch_bounds__(256) k_transpose_rho(int nx, int ny, int nz, const T* __restrict__ rho,
                                                        T* __restrict__ rho_t) {
  __shared__ T tile[32][33];
  int x0 = blockIdx.x * 32, z0 = blockIdx.y * 32, y = blockIdx.z;
  int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 32 x 8
  for (int r = ty; r < 32; r += 8) {
    int z = z0 + r, x = x0 + tx;
    tile[r][tx] = (z < nz && x < nx) ? rho[((size_t)z * ny + y) * nx + x] : T(0);
  }
  __syncthreads();
  for (int r = ty; r < 32; r += 8) {
    int x = x0 + r, z = z0 + tx;
    if (x < nx && z < nz) rho_t[((size_t)y * nx + x) * nz + z] = tile[tx][r];
  }
}

template <typename T>
hipError_t launch_transpose_rho(const Geo<T>& g, const T* rho, T* rho_t, hipStream_t s) {
  dim3 grid((g.nx + 31) / 32, (g.nz + 31) / 32, g.ny);
  hipLaunchKernelGGL(k_transpose_rho<T>, grid, dim3(256), 0, s, g.nx, g.ny, g.nz, rho, rho_t);
  return hipGetLastError();
}

// ------------------------------------------------------------------ fluence

// Fluence map of one pixel (§2.2.2):
//   F = f(u; x1, x2) f(v; y1, y2) [tau S + (1 - tau) O],
//   S = sum_l w_l (row coverage by the leaf bank), O = sum_l w_l f(u; l_l, r_l).
template <typename T>
__global__ void __launch_bounds__(256) k_raster(Geo<T> g, const T* __restrict__ leaves, const T* __restrict__ jaws,
                                                T* __restrict__ F) {
  int b = blockIdx.y;
  int plane = g.Nu * g.Nv;
  int r = blockIdx.x * 256 + threadIdx.x;
  if (r >= plane) return;
  int i = r / g.Nv, j = r - i * g.Nv;
  T D = g.lat, iD = g.inv_lat;
  T u = (T(i) - g.cu) * D, v = (T(j) - g.cv) * D;
  const T* jw = jaws + 4 * b;
  const T* lv = leaves + (size_t)2 * g.L * b;
  T fx = overlap(u, jw[0], jw[1], D, iD);
  T fy = overlap(v, jw[2], jw[3], D, iD);
  T S = T(0), O = T(0);
  if (fx * fy != T(0)) {
    for (int l = 0; l < g.L; ++l) {
      T w = overlap(v, g.leaf_edges[l], g.leaf_edges[l + 1], D, iD);
      if (w > T(0)) {
        S += w;
        O += w * overlap(u, lv[l], lv[g.L + l], D, iD);
      }
    }
  }
  F[(size_t)b * plane + r] = fx * fy * (g.tau * S + (T(1) - g.tau) * O);
}

template <typename T>
hipError_t launch_raster(const Geo<T>& g, int nb, const T* leaves, const T* jaws, T* F, hipStream_t s) {
  dim3 grid((g.Nu * g.Nv + 255) / 256, nb);
  hipLaunchKernelGGL(k_raster<T>, grid, dim3(256), 0, s, g, leaves, jaws, F);
  return hipGetLastError();
}

// Rectangle of fluence pixels [u0, u1) x [v0, v1) of each control point outside
// which F and all its derivatives are exactly zero: a pixel carries fluence only
// if it overlaps the jaw opening (the factor f(u; x1, x2) f(v; y1, y2) of Eq. 4): pixel
// i overlaps [a, b] iff fa < i < fb, with a thousandth of a pixel for rounding (indices
// stay below 2^12, so theirs is below 2^-11), widened by (du, dv) pixels for the reach
// of the fluence corrections.  A non-finite jaw gives the whole plane.
template <typename T>
__device__ __forceinline__ void pixel_range(T a, T b, T c, int N, int d, T inv_lat, int* lo, int* hi) {
  const T fa = a * inv_lat + c - T(0.5), fb = b * inv_lat + c + T(0.5);
  if (!(fa == fa) || !(fb == fb) || !(fabs(fa) < T(1e8)) || !(fabs(fb) < T(1e8))) {
    *lo = 0;
    *hi = N;
    return;
  }
  int l = (int)floor(fa - T(1e-3)) + 1 - d, u = (int)ceil(fb + T(1e-3)) + d;
  l = max(l, 0);
  u = min(u, N);
  *lo = l;
  *hi = u > l ? u : l;
}

template <typename T>
__global__ void k_aperture_box(Geo<T> g, int nb, const T* __restrict__ jaws, int du, int dv, int* __restrict__ box) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= nb) return;
  const T* jw = jaws + 4 * b;
  int u0, u1, v0, v1;
  pixel_range(jw[0], jw[1], g.cu, g.Nu, du, g.inv_lat, &u0, &u1);
  pixel_range(jw[2], jw[3], g.cv, g.Nv, dv, g.inv_lat, &v0, &v1);
  box[4 * b] = u0;
  box[4 * b + 1] = u1;
  box[4 * b + 2] = v0;
  box[4 * b + 3] = v1;
}

template <typename T>
hipError_t launch_aperture_box(const Geo<T>& g, int nb, const T* jaws, int du, int dv, int* box, hipStream_t s) {
  hipLaunchKernelGGL(k_aperture_box<T>, dim3((nb + 63) / 64), dim3(64), 0, s, g, nb, jaws, du, dv, box);
  return hipGetLastError();
}

// ------------------------------------------------------------------ depth

// Central-axis depth (§2.2.4, Eq. 7): one wavefront per control point samples
// 64 consecutive planes at a time and turns them into the running integral with
// an inclusive wavefront prefix sum plus the carry of the previous chunk.
template <typename T>
__global__ void __launch_bounds__(64) k_ca_depth(Geo<T> g, const T* __restrict__ frame, const T* __restrict__ rho_t,
                                                 T* __restrict__ z) {
  int b = blockIdx.x;
  int lane = threadIdx.x;
  T sn = frame[2 * b], cs = frame[2 * b + 1];
  T carry = T(0) * (sn + cs);  // (an angle that is NaN leaves a NaN depth)
  for (int k0 = 0; k0 < g.Nk; k0 += 64) {
    int k = k0 + lane;
    T val = T(0);
    if (k < g.Nk) {
      T e = g.e0 + T(k) * g.dstep;
      T X = g.iso_ix + (-e * sn) * g.inv_sx;
      T Y = g.iso_iy + (e * cs) * g.inv_sy;
      val = sample_rho(rho_t, g.nx, g.ny, g.nz, X, Y, g.iso_iz) * g.dstep;
    }
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      T o = __shfl_up(val, off, 64);
      if (lane >= off) val += o;
    }
    if (k < g.Nk) z[(size_t)b * g.Nk + k] = carry + val;
    carry += __shfl(val, 63, 64);
  }
}

template <typename T>
hipError_t launch_ca_depth(const Geo<T>& g, int nb, const T* frame, const T* rho_t, T* z, hipStream_t s) {
  hipLaunchKernelGGL(k_ca_depth<T>, dim3(nb), dim3(64), 0, s, g, frame, rho_t, z);
  return hipGetLastError();
}

// ------------------------------------------------------------------ ray march

// Ray (u_i, v_j) meets plane k at
//   q - iso = (d_k - SAD) b + (d_k / SAD)(u e_u + v e_v);
// the density is sampled trilinearly there, and the water-equivalent depth of
// Eq. 7 is the inclusive sum W_k = sum_{k' <= k} rho(q_k') ds, ds = Dd sqrt(1 +
// (u^2 + v^2)/SAD^2); the primary is P_k = F (SAD / d_k)^2 DD(W_k).
// MARCH_ADJOINT instead accumulates A = sum_k H_k (SAD / d_k)^2 DD(W_k) (the
// adjoint of the primary w.r.t. F); MARCH_GEOMETRY stores the aperture-independent
// factor G_k = (SAD / d_k)^2 DD(W_k) itself (rounded to E), so that P = F G later.
enum { MARCH_PRIMARY = 0, MARCH_ADJOINT = 1, MARCH_GEOMETRY = 2 };

// ---- serial form
//
// One thread per divergent ray (i, j) walks its Nk planes in order with a
// compensated running sum; eight planes' density loads are in flight at a time.
// Lanes run along v, i.e. along patient z, so the z-fastest density copy is read
// almost contiguously.  With a box (the aperture rectangle of each control point,
// given when the convolution honours it) rays outside it are skipped: the
// convolution never reads P there, and the adjoint's A there is written as 0
// (the parameter gradients only read it inside).
// One ray (i, j) of control point b.
template <typename T, int MODE, typename E>
__device__ __forceinline__ void march_ray(const Geo<T>& g, int b, int i, int j, const T* __restrict__ frame,
                                          const T* __restrict__ rho_t, const T* __restrict__ F,
                                          const T* __restrict__ zca, const T* tab, E* __restrict__ vol,
                                          T* __restrict__ A) {
  const int plane = g.Nu * g.Nv;
  const int r = i * g.Nv + j;
  E* vb = vol + (size_t)b * g.Nk * plane + r;
  T Fv = T(1);
  if (MODE == MARCH_PRIMARY) {
    Fv = F[(size_t)b * plane + r];
    if (Fv == T(0)) {
      for (int k = 0; k < g.Nk; ++k) vb[(size_t)k * plane] = E(0);
      return;
    }
  }
  T sn = frame[2 * b], cs = frame[2 * b + 1];
  T u = (T(i) - g.cu) * g.lat, v = (T(j) - g.cv) * g.lat;
  T ucs = u * cs, usn = u * sn;
  T ds = g.dstep * dsqrt(T(1) + (u * u + v * v) * (g.inv_sad * g.inv_sad));
  const T* zb = zca + (size_t)b * g.Nk;
  T W = T(0) * (sn + cs), c = T(0), acc = T(0);  // (an angle that is NaN leaves a NaN depth)
  // one step of the march: the water-equivalent depth Wk of plane k, then the
  // primary (or its adjoint, or the factor itself) at that plane
  auto step = [&](int k, T Wk) {
    const T e = g.e0 + T(k) * g.dstep;
    const T gk = T(1) + e * g.inv_sad;
    const T geo = dd_lookup(tab, g.n_dd, g.inv_dd_step, Wk) / (gk * gk);
    if (MODE == MARCH_ADJOINT)
      acc = fma(T(vb[(size_t)k * plane]), geo, acc);
    else if (MODE == MARCH_PRIMARY)
      vb[(size_t)k * plane] = Fv * geo;
    else
      vb[(size_t)k * plane] = E(geo);
  };
  if (g.wepl_mode == PDRT_WEPL_PER_RAY) {
#pragma unroll 8
    for (int k = 0; k < g.Nk; ++k) {
      const T e = g.e0 + T(k) * g.dstep;
      const T gk = T(1) + e * g.inv_sad;
      const T X = g.iso_ix + (-e * sn + gk * ucs) * g.inv_sx;
      const T Y = g.iso_iy + (e * cs + gk * usn) * g.inv_sy;
      const T Z = g.iso_iz + (gk * v) * g.inv_sz;
      const T rho = sample_rho(rho_t, g.nx, g.ny, g.nz, X, Y, Z);
      const T y = rho * ds - c;  // Kahan-compensated running sum
      const T t = W + y;
      c = (t - W) - y;
      W = t;
      step(k, W);
    }
  } else {
    for (int k = 0; k < g.Nk; ++k) step(k, zb[k]);
  }
  if (MODE == MARCH_ADJOINT) A[(size_t)b * plane + r] = acc;
}

template <typename T>
__device__ __forceinline__ void kahan_add(T& S, T& c, T x) {
  const T y = x - c;
  const T t = S + y;
  c = (t - S) - y;
  S = t;
}

// Density fetch of plane k on a ray, and its term of the depth integral (rounded by
// itself, so that the scan and march_ray_segments add the same bits).
template <typename T>
__device__ __forceinline__ RhoFetch<T> ray_fetch(const Geo<T>& g, const T* __restrict__ rho_t, int k, T sn, T cs, T ucs,
                                                 T usn, T v) {
  const T e = g.e0 + T(k) * g.dstep;
  const T gk = T(1) + e * g.inv_sad;
  const T X = g.iso_ix + (-e * sn + gk * ucs) * g.inv_sx;
  const T Y = g.iso_iy + (e * cs + gk * usn) * g.inv_sy;
  const T Z = g.iso_iz + (gk * v) * g.inv_sz;
  return rho_fetch(rho_t, g.nx, g.ny, g.nz, X, Y, Z);
}

template <typename T>
__device__ __forceinline__ T ray_term(const RhoFetch<T>& r, T ds) {
  const T rho = rho_combine(r);
  {
#pragma clang fp contract(off)
    return rho * ds;
  }
}

// Ray (i, j) in the order of the segmented scan below, for launches with more rays than
// the scan is the faster for: beside the running sum from the carry a segment's own sum
// is kept, and joins the carry where the segment ends.
template <typename T, int MODE, typename E>
__device__ __forceinline__ void march_ray_segments(const Geo<T>& g, int b, int i, int j, const T* __restrict__ frame,
                                                   const T* __restrict__ rho_t, const T* __restrict__ F,
                                                   const T* __restrict__ zca, const T* tab, E* __restrict__ vol,
                                                   T* __restrict__ A) {
  constexpr int U = 4;  // planes fetched at once
  const int plane = g.Nu * g.Nv;
  const int r = i * g.Nv + j;
  E* vb = vol + (size_t)b * g.Nk * plane + r;
  const T Fv = MODE == MARCH_PRIMARY ? F[(size_t)b * plane + r] : T(1);
  const T sn = frame[2 * b], cs = frame[2 * b + 1];
  const T u = (T(i) - g.cu) * g.lat, v = (T(j) - g.cv) * g.lat;
  const T ucs = u * cs, usn = u * sn;
  const T ds = g.dstep * dsqrt(T(1) + (u * u + v * v) * (g.inv_sad * g.inv_sad));
  const T* zb = zca + (size_t)b * g.Nk;
  const bool per_ray = g.wepl_mode == PDRT_WEPL_PER_RAY;
  const int nseg = march_segments(g.Nk);
  int w = 0, ke = g.Nk / nseg;
  T C = T(0) * (sn + cs), cC = T(0);  // carry (an angle that is NaN leaves a NaN depth)
  T W = C, cW = T(0), S = T(0), cS = T(0), acc = T(0), total = T(0);
  for (int k0 = 0; k0 < g.Nk; k0 += U) {
    T y[U];
    if (per_ray) {
      RhoFetch<T> fr[U];
#pragma unroll
      for (int s = 0; s < U; ++s) fr[s] = ray_fetch(g, rho_t, min(k0 + s, g.Nk - 1), sn, cs, ucs, usn, v);
#pragma unroll
      for (int s = 0; s < U; ++s) y[s] = ray_term(fr[s], ds);
    }
#pragma unroll
    for (int s = 0; s < U; ++s) {
      const int k = k0 + s;
      if (k >= g.Nk) break;
      if (k == ke) {  // the next segment
        kahan_add(C, cC, S - cS);
        W = C, cW = cC, S = T(0), cS = T(0);
        total += acc;
        acc = T(0);
        ++w;
        ke = (g.Nk * (w + 1)) / nseg;
      }
      T Wk;
      if (per_ray) {
        kahan_add(S, cS, y[s]);
        kahan_add(W, cW, y[s]);
        Wk = W;
      } else {
        Wk = zb[k];
      }
      const T e = g.e0 + T(k) * g.dstep;
      const T gk = T(1) + e * g.inv_sad;
      const T geo = dd_lookup(tab, g.n_dd, g.inv_dd_step, Wk) / (gk * gk);
      if (MODE == MARCH_ADJOINT)
        acc = fma(T(vb[(size_t)k * plane]), geo, acc);
      else if (MODE == MARCH_PRIMARY)
        vb[(size_t)k * plane] = Fv * geo;
      else
        vb[(size_t)k * plane] = E(geo);
    }
  }
  if (MODE == MARCH_ADJOINT) A[(size_t)b * plane + r] = total + acc;
}

// Workgroups of a march: block q of n of control point b.  Fluence corrections widen the
// largest rectangle, and with it the grid, by up to the blur's radius, and openings are
// often much smaller, so that half of the workgroups have none.  Control points then run
// fastest, and those workgroups come last: with rays fastest they fell on the same compute
// units for every control point and left those idle (60 of 31 x 33 rays and 99 planes in a
// grid of 45 x 45, march and adjoint as a scan: 0.069 + 0.083 ms, now 0.043 + 0.053).
// Uncorrected plans keep rays fastest (60 openings of 24 x 24 mm in 120 mm limits, march:
// 0.053 ms, 0.056 with control points fastest).
template <typename T>
__host__ __device__ bool march_cp_first(const Geo<T>& g, const int* box) {
  return box && g.fcorr;
}

struct MarchBlock {
  int b, q, n;
  template <typename T>
  __device__ MarchBlock(const Geo<T>& g, const int* box) {
    const bool cf = march_cp_first(g, box);
    b = cf ? blockIdx.x : blockIdx.y, q = cf ? blockIdx.y : blockIdx.x, n = cf ? gridDim.y : gridDim.x;
  }
};

// Without a box, one thread per ray of the plane; with a box, the blocks of control
// point b walk only the rays of control point b's rectangle (grid-stride),
// so no lanes idle on rays outside it.  (In adjoint mode A outside the box is
// cleared beforehand.)  SEG: the scan's order.
template <typename T, int MODE, typename E, bool SEG>
__global__ void __launch_bounds__(256) k_march_serial(Geo<T> g, const T* __restrict__ frame, const T* __restrict__ rho_t,
                                               const T* __restrict__ F, const T* __restrict__ zca,
                                               const T* __restrict__ dd, E* __restrict__ vol, T* __restrict__ A,
                                               const int* __restrict__ box) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* tab = reinterpret_cast<T*>(smem_raw);
  for (int q = threadIdx.x; q < g.n_dd; q += 256) tab[q] = dd[q];
  __syncthreads();
  const MarchBlock mb(g, box);
  const int b = mb.b;
  auto march = [&](int i, int j) {
    if constexpr (SEG) march_ray_segments<T, MODE, E>(g, b, i, j, frame, rho_t, F, zca, tab, vol, A);
    else march_ray<T, MODE, E>(g, b, i, j, frame, rho_t, F, zca, tab, vol, A);
  };
  if (box) {
    const int* bx = box + 4 * b;
    const int bw = bx[3] - bx[2], area = bx[1] > bx[0] && bw > 0 ? (bx[1] - bx[0]) * bw : 0;
    for (int rr = mb.q * 256 + threadIdx.x; rr < area; rr += mb.n * 256) {
      const int li = rr / bw;
      march(bx[0] + li, bx[2] + rr - li * bw);
    }
  } else {
    const int r = mb.q * 256 + threadIdx.x;
    if (r < g.Nu * g.Nv) march(r / g.Nv, r % g.Nv);
  }
}

// ---- segmented scan (launches of few rays, or MARCH_SCAN)
//
// The inclusive sum as a segmented scan across the wavefronts of a workgroup.
// The workgroup takes 64 rays (lanes along v, so that neighbouring lanes read
// neighbouring z of the z-fastest density copy) and its NW wavefronts take
// consecutive segments of the Nk planes: each wavefront samples its segment
// (samples kept in registers, MARCH_SEG planes per pass) and forms the segment's
// compensated sum; the segment sums go through LDS and each wavefront adds those
// of the segments before its own in plane order (its carry); it then rescans its
// segment from the carry, giving W_k for its planes, and applies the depth dose.
// In adjoint mode the wavefronts' partial sums of H_k (SAD/d_k)^2 DD(W_k) are
// added in LDS in segment order.  Every sum runs in a fixed order.
//
// With a box (the aperture rectangle of each control point, given when the
// convolution honours it) only the rays inside it are marched: the convolution
// never reads P outside it, and the adjoint's A there is written as 0 beforehand
// (the parameter gradients only read it inside).
constexpr int MARCH_SEG = kMarchSeg;           // planes per wavefront and pass
constexpr int MARCH_MAXW = kMarchMaxSegments;  // wavefronts per workgroup

template <typename T, int MODE, typename E>
__global__ void __launch_bounds__(64 * MARCH_MAXW) k_march_scan(Geo<T> g, const T* __restrict__ frame,
                                                           const T* __restrict__ rho_t, const T* __restrict__ F,
                                                           const T* __restrict__ zca, const T* __restrict__ dd,
                                                           E* __restrict__ vol, T* __restrict__ A,
                                                           const int* __restrict__ box) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  T* seg = reinterpret_cast<T*>(smem_raw);  // [2][MARCH_MAXW][64]: segment sums and compensations
  T* tab = seg + 2 * MARCH_MAXW * 64;       // depth-dose table [n_dd]
  const int nw = blockDim.x >> 6;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  for (int q = tid; q < g.n_dd; q += blockDim.x) tab[q] = dd[q];
  __syncthreads();
  const MarchBlock mb(g, box);
  const int b = mb.b;
  const int plane = g.Nu * g.Nv;
  int u0 = 0, nu = g.Nu, v0 = 0, nv = g.Nv;
  if (box) {
    const int* bx = box + 4 * b;
    u0 = bx[0], v0 = bx[2];
    nu = max(0, bx[1] - bx[0]), nv = max(0, bx[3] - bx[2]);
  }
  const int area = nu * nv;
  const int kb = (g.Nk * w) / nw, ke = (g.Nk * (w + 1)) / nw;  // this wavefront's planes
  const bool per_ray = g.wepl_mode == PDRT_WEPL_PER_RAY;
  const bool keep = ke - kb <= MARCH_SEG;  // one pass holds the whole segment
  const T sn = frame[2 * b], cs = frame[2 * b + 1];
  const T* zb = zca + (size_t)b * g.Nk;
  for (int grp = mb.q; grp * 64 < area; grp += mb.n) {
    const int rr = grp * 64 + lane;
    const bool valid = rr < area;
    const int li = valid ? rr / nv : 0;
    const int i = u0 + li, j = v0 + (valid ? rr - li * nv : 0);
    const int r = i * g.Nv + j;
    const T u = (T(i) - g.cu) * g.lat, v = (T(j) - g.cv) * g.lat;
    const T ucs = u * cs, usn = u * sn;
    const T ds = g.dstep * dsqrt(T(1) + (u * u + v * v) * (g.inv_sad * g.inv_sad));
    // samples rho ds of planes k0 .. k0 + MARCH_SEG - 1 (zero past the segment),
    // four planes' corner loads issued together before they are combined
    T y[MARCH_SEG];
    auto sample_pass = [&](int k0) {
#pragma unroll
      for (int s0 = 0; s0 < MARCH_SEG; s0 += 4) {
        RhoFetch<T> fr[4];
#pragma unroll
        for (int s1 = 0; s1 < 4; ++s1)
          fr[s1] = ray_fetch(g, rho_t, min(k0 + s0 + s1, g.Nk - 1), sn, cs, ucs, usn, v);
#pragma unroll
        for (int s1 = 0; s1 < 4; ++s1)
          y[s0 + s1] = k0 + s0 + s1 < ke ? ray_term(fr[s1], ds) : T(0);
      }
    };
    T S = T(0), cS = T(0);
    if (per_ray) {
      for (int k0 = kb; k0 < ke; k0 += MARCH_SEG) {
        sample_pass(k0);
#pragma unroll
        for (int s2 = 0; s2 < MARCH_SEG; ++s2)
          if (k0 + s2 < ke) kahan_add(S, cS, y[s2]);
      }
      seg[w * 64 + lane] = S;
      seg[(MARCH_MAXW + w) * 64 + lane] = cS;
    }
    __syncthreads();
    // carry: the sums of the segments before this one, in plane order
    T W = T(0) * (sn + cs), cW = T(0);  // (an angle that is NaN leaves a NaN depth)
    if (per_ray)
      for (int w2 = 0; w2 < w; ++w2) kahan_add(W, cW, seg[w2 * 64 + lane] - seg[(MARCH_MAXW + w2) * 64 + lane]);
    T Fv = T(1);
    if (MODE == MARCH_PRIMARY && valid) Fv = F[(size_t)b * plane + r];
    E* vb = vol + (size_t)b * g.Nk * plane + r;
    T acc = T(0);
    for (int k0 = kb; k0 < ke; k0 += MARCH_SEG) {
      if (per_ray && !keep) sample_pass(k0);
#pragma unroll
      for (int s2 = 0; s2 < MARCH_SEG; ++s2) {
        const int k = k0 + s2;
        if (k < ke) {
          T Wk;
          if (per_ray) {
            kahan_add(W, cW, y[s2]);
            Wk = W;
          } else {
            Wk = zb[k];
          }
          const T e = g.e0 + T(k) * g.dstep;
          const T gk = T(1) + e * g.inv_sad;
          const T geo = dd_lookup(tab, g.n_dd, g.inv_dd_step, Wk) / (gk * gk);
          if (valid) {
            if (MODE == MARCH_ADJOINT)
              acc = fma(T(vb[(size_t)k * plane]), geo, acc);
            else if (MODE == MARCH_PRIMARY)
              vb[(size_t)k * plane] = Fv * geo;
            else
              vb[(size_t)k * plane] = E(geo);
          }
        }
      }
    }
    if (MODE == MARCH_ADJOINT) {
      __syncthreads();
      seg[w * 64 + lane] = acc;
      __syncthreads();
      if (w == 0 && valid) {
        T a = T(0);
        for (int w2 = 0; w2 < nw; ++w2) a += seg[w2 * 64 + lane];
        A[(size_t)b * plane + r] = a;
      }
    }
    __syncthreads();  // the segment sums are reused by the next group
  }
}

template <typename T>
__global__ void k_fill_zero(size_t n, T* __restrict__ p) {
  for (size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (size_t)gridDim.x * blockDim.x)
    p[q] = T(0);
}

// Rays of a control point to be marched: those of the largest jaw rectangle the field
// limit allows (the plane minus the kernel halo), widened by the fluence corrections;
// without a box the whole plane.  `margin`: pixels on each side more, for the grid (a
// turned rectangle has two, and a workgroup left over costs less than a second round;
// the walk is grid-stride, so that larger rectangles, from jaws beyond the field limit,
// are covered all the same).
template <typename T>
int march_rays(const Geo<T>& g, const int* box, int margin) {
  if (!box) return g.Nu * g.Nv;
  const int du = margin - g.h + (g.fcorr ? g.conv_du : 0), dv = margin - g.h + (g.fcorr ? g.conv_dv : 0);
  return max(1, min(g.Nu, g.Nu + 2 * du)) * max(1, min(g.Nv, g.Nv + 2 * dv));
}

// The scan's wavefronts per workgroup: segments of at most MARCH_SEG planes where
// eight wavefronts suffice (Nk <= 256), else eight segments of several passes.
template <typename T, int MODE, typename E>
hipError_t launch_march_mode(const Geo<T>& g, int nb, const T* frame, const T* rho_t, const T* F, const T* z,
                             const T* dd, E* vol, T* A, hipStream_t s, const int* box) {
  const int rays = march_rays(g, box, 3);
  const auto grid_of = [&](int blocks) {
    return march_cp_first(g, box) ? dim3(nb, min(blocks, 65535)) : dim3(blocks, nb);
  };
  const dim3 serial = grid_of((rays + 255) / 256);
  if (g.march_scan == MARCH_SERIAL) {
    hipLaunchKernelGGL((k_march_serial<T, MODE, E, false>), serial, dim3(256), g.n_dd * sizeof(T), s, g, frame, rho_t,
                       F, z, dd, vol, A, box);
    return hipGetLastError();
  }
  // Geometry cache of 60 control points of 89 x 89 x 183 nodes: 0.31 ms (scan 0.58); the march
  // and its adjoint of 90 with fluence corrections (n = 31, 59 x 59): 0.21 + 0.31 ms (scan
  // 0.39 + 0.57).  The same bits.
  // With boxes only the rays of the largest rectangle are known here, and openings often hold
  // half of them or less: counted as half (12 control points of 24 x 24 mm openings in
  // 120 mm limits, corrected and turned, n = 61 at 5 mm: 0.038 + 0.049 ms as a scan, 0.050 +
  // 0.073 by threads).
  const long waves = (long)(march_rays(g, box, 0) + 63) / 64 * nb / (box ? 2 : 1);
  if (g.march_scan == MARCH_SEGMENTS && !march_scan_wins(waves, g.Nk)) {
    hipLaunchKernelGGL((k_march_serial<T, MODE, E, true>), serial, dim3(256), g.n_dd * sizeof(T), s, g, frame, rho_t,
                       F, z, dd, vol, A, box);
    return hipGetLastError();
  }
  const int nw = march_segments(g.Nk);
  const size_t lds = sizeof(T) * (2 * MARCH_MAXW * 64 + (size_t)g.n_dd);
  if (lds > 64 * 1024) return hipErrorInvalidConfiguration;
  const dim3 grid = grid_of((rays + 63) / 64);
  hipLaunchKernelGGL((k_march_scan<T, MODE, E>), grid, dim3(64 * nw), lds, s, g, frame, rho_t, F, z, dd, vol, A,
                     box);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_march(const Geo<T>& g, int nb, const T* frame, const T* rho_t, const T* F, const T* z, const T* dd,
                        T* P, hipStream_t s, const int* box) {
  return launch_march_mode<T, MARCH_PRIMARY, T>(g, nb, frame, rho_t, F, z, dd, P, (T*)nullptr, s, box);
}

template <typename E>
hipError_t launch_march_geometry(const Geo<float>& g, int nb, const float* frame, const float* rho_t, const float* z,
                                 const float* dd, E* G, hipStream_t s) {
  return launch_march_mode<float, MARCH_GEOMETRY, E>(g, nb, frame, rho_t, (const float*)nullptr, z, dd, G,
                                                     (float*)nullptr, s, (const int*)nullptr);
}
template hipError_t launch_march_geometry<float>(const Geo<float>&, int, const float*, const float*, const float*,
                                                 const float*, float*, hipStream_t);
template hipError_t launch_march_geometry<__bf16>(const Geo<float>&, int, const float*, const float*, const float*,
                                                  const float*, __bf16*, hipStream_t);

template <typename T>
hipError_t launch_march_adj(const Geo<T>& g, int nb, const T* frame, const T* rho_t, const T* z, const T* dd,
                            const T* H, T* A, hipStream_t s, const int* box) {
  if (box) {
    const size_t n = (size_t)nb * g.Nu * g.Nv;
    hipLaunchKernelGGL(k_fill_zero<T>, dim3((unsigned)((n + 255) / 256 < 2048 ? (n + 255) / 256 : 2048)), dim3(256), 0,
                       s, n, A);
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;
  }
  return launch_march_mode<T, MARCH_ADJOINT, T>(g, nb, frame, rho_t, (const T*)nullptr, z, dd, const_cast<T*>(H), A,
                                                s, box);
}

// ------------------------------------------------------------------ kernel taps

template <typename T>
__device__ void build_taps(const Geo<T>& g, int k, T zk, T* K, int tid, int nthreads) {
  TapParams<T> tp = tap_params(g, k, zk);
  int n = g.n_taps, h = g.h;
  for (int idx = tid; idx < n * n; idx += nthreads) K[idx] = tap_value(tp, idx / n - h, idx % n - h);
}

// ------------------------------------------------------------------ direct conv

// Zero-padded per-plane convolution Dfan_k = K_k (*) P_k (§2.2.6, Eq. 8) on the
// vector ALUs.  A block owns a 48 (u) x 32 (v) output tile of one plane; the
// input tile with its halo and the plane's taps are staged in LDS.  Each thread
// owns 6 outputs along u and slides a 6-deep register window down the tap rows,
// so each tap costs 6 FMAs per LDS load.  Used for the FP64 path and for small
// kernels.
constexpr int DC_COLS = 32, DC_RG = 8, DC_R = 6, DC_ROWS = DC_RG * DC_R;

template <typename T>
__global__ void __launch_bounds__(256) k_conv_direct(Geo<T> g, const T* __restrict__ zca, const T* __restrict__ in,
                                                     T* __restrict__ out) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int n = g.n_taps, h = g.h;
  const int pitch = DC_COLS + 2 * h;
  const int rows = DC_ROWS + 2 * h + DC_R;  // DC_R spare rows for the window prefetch
  T* tile = reinterpret_cast<T*>(smem_raw);
  T* K = tile + rows * pitch;
  const int k = blockIdx.y, b = blockIdx.z;
  const int tiles_v = (g.Nv + DC_COLS - 1) / DC_COLS;
  const int i0 = (blockIdx.x / tiles_v) * DC_ROWS, j0 = (blockIdx.x % tiles_v) * DC_COLS;
  const int plane = g.Nu * g.Nv;
  const T* src = in + ((size_t)b * g.Nk + k) * plane;
  const int tid = threadIdx.x;
  for (int idx = tid; idx < rows * pitch; idx += 256) {
    int rr = idx / pitch, cc = idx - rr * pitch;
    int i = i0 - h + rr, j = j0 - h + cc;
    T val = T(0);
    if (rr < DC_ROWS + 2 * h && i >= 0 && i < g.Nu && j >= 0 && j < g.Nv) val = src[(size_t)i * g.Nv + j];
    tile[idx] = val;
  }
  build_taps(g, k, zca[(size_t)b * g.Nk + k], K, tid, 256);
  __syncthreads();
  const int tx = tid % DC_COLS, ty = tid / DC_COLS;
  const int rbase = ty * DC_R;
  T acc[DC_R];
#pragma unroll
  for (int r = 0; r < DC_R; ++r) acc[r] = T(0);
  for (int q = 0; q < n; ++q) {
    const T* col = tile + rbase * pitch + tx + q;
    T w[DC_R];
#pragma unroll
    for (int r = 0; r < DC_R; ++r) w[r] = col[r * pitch];
    for (int p0 = 0; p0 < n; p0 += DC_R) {
#pragma unroll
      for (int s = 0; s < DC_R; ++s) {
        int p = p0 + s;
        if (p < n) {
          T t = K[p * n + q];
#pragma unroll
          for (int r = 0; r < DC_R; ++r) acc[r] += t * w[(r + s) % DC_R];
          w[s] = col[(p + DC_R) * pitch];
        }
      }
    }
  }
  T* dst = out + ((size_t)b * g.Nk + k) * plane;
  int j = j0 + tx;
#pragma unroll
  for (int r = 0; r < DC_R; ++r) {
    int i = i0 + rbase + r;
    if (i < g.Nu && j < g.Nv) dst[(size_t)i * g.Nv + j] = acc[r];
  }
}

template <typename T>
size_t conv_direct_lds(const Geo<T>& g) {
  int pitch = DC_COLS + 2 * g.h, rows = DC_ROWS + 2 * g.h + DC_R;
  return sizeof(T) * ((size_t)rows * pitch + (size_t)g.n_taps * g.n_taps);
}

template <typename T>
hipError_t launch_conv_direct(const Geo<T>& g, int nb, const T* z, const T* in, T* out, hipStream_t s) {
  size_t lds = conv_direct_lds(g);
  if (lds > 160 * 1024) return hipErrorInvalidConfiguration;
  {
    hipError_t e = ensure_lds_limit((const void*)k_conv_direct<T>, 160 * 1024);
    if (e != hipSuccess) return e;
  }
  int tiles = ((g.Nu + DC_ROWS - 1) / DC_ROWS) * ((g.Nv + DC_COLS - 1) / DC_COLS);
  dim3 grid(tiles, g.Nk, nb);
  hipLaunchKernelGGL(k_conv_direct<T>, grid, dim3(256), lds, s, g, z, in, out);
  return hipGetLastError();
}

// ------------------------------------------------------------------ gather

// Back-projection and MU-weighted sum (§2.2.7, Eq. 9):
// dose(x, y, z) += sum_b MU_b trilinear(Dfan_b at the voxel's beam-frame position).
//
// A voxel column (x, y) meets one beam-frame cell (k, i) per control point, the same
// for all its z, so the lookup separates: the column's four rows (k, i), (k, i + 1),
// (k + 1, i), (k + 1, i + 1) are first blended into one row over j, which its z then
// read at j0 and j0 + 1.  One wavefront owns a column and ZS z per lane (lanes along
// z): its lanes load the four rows coalesced (lanes along j), blend them with the
// corner weights and park the blended row in LDS; every z then takes two
// neighbouring words of it.  A control point whose fan misses the column is skipped.
// Against eight loads and eight weighted adds per voxel and control point this is 4
// Nv / nz of each, and reads whole cache lines.  180 control points at 128^3 (89-wide
// planes, 1.04 GB of Dfan): 0.41 ms (2.6 TB/s; eight loads per voxel: 0.92 ms); 90 at
// 128 x 128 x 96 (43-wide): 0.084 ms (0.33).  Latency of the loads bounds it.
//
// A column's z reach a window of the row only, nz s_z / lat pixels at the axis.  Where
// that takes fewer 64-wide pieces than the plane (thin grids under wide planes) the
// wavefront loads and blends the window alone (WIN): 60 control points, 16 slices of
// 224 x 224 under 191-wide planes 0.30 ms (whole rows 0.82, eight loads per voxel 0.40).
//
// The terms are summed in control-point order, in FP64 for the FP32 path (an exact
// sum of FP32 terms to 53 bits, two instructions a term where the compensated FP32
// sum takes seven) and with Neumaier compensation for the FP64 path; across batches
// the running sum lives in `dose` and `comp`.
//
// A block's four wavefronts cover a 2 x 2 patch of columns: neighbouring columns read
// mostly the same beam-frame rows.  Workgroups are numbered so that each of the
// eight XCDs (which receive workgroups round robin) walks a contiguous range of
// patches and they share one L2.

// One control point's terms of a voxel column, its fan reaching the column.
template <typename T>
struct GatherCol {
  T w[4];      // corner (dk, di) = (c >> 1, c & 1): in-grid mask x (1 - wk or wk) x (1 - wi or wi)
  int off[4];  // element offset of the corner's row (clamped into the grid)
  T q, m;      // SAD / d, which scales z into the lateral coordinate j; MU
  int b;       // control point within the batch
  int jb;      // first pixel of the window (WIN)
};

constexpr int GATHER_CHUNK = 64;  // control points examined at once, one per lane
constexpr int GATHER_PAD = 2;     // zero words on each side of a blended row

// A wavefront-uniform value moved to a scalar register (so that addresses built from
// it use the scalar base of a global load).
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Running sum over control points.
template <typename T>
struct GatherSum;

template <>
struct GatherSum<float> {
  double s = 0.0;
  __device__ void add(float v) { s += (double)v; }
  // the sum's 64 bits, split over two words, carried between batches
  __device__ void load(float a, float c) {
    s = __hiloint2double(__float_as_int(a), __float_as_int(c));
  }
  __device__ void store(float* a, float* c) const {
    *a = __int_as_float(__double2hiint(s));
    *c = __int_as_float(__double2loint(s));
  }
  __device__ float value(float calib) const { return calib * (float)s; }
};

template <>
struct GatherSum<double> {
  double s = 0.0, c = 0.0;
  __device__ void add(double v) {
    const double t = s + v;
    c += fabs(s) >= fabs(v) ? (s - t) + v : (v - t) + s;
    s = t;
  }
  __device__ void load(double a, double b) { s = a, c = b; }
  __device__ void store(double* a, double* b) const { *a = s, *b = c; }
  __device__ double value(double calib) const { return calib * (s + c); }
};

// JS: ceil(Nv / 64), or 0 for a loop over wider planes, or (WIN) the 64-wide pieces of the
// window; ZS: z per lane; PX x PY: the block's patch of columns; U: control points in flight.
template <typename T, int JS, int ZS, int PX, int PY, int U, bool WIN>
__global__ void __launch_bounds__(64 * PX * PY) k_gather(Geo<T> g, int nb, int first, int last, int win, int zc, int xc, int yc,
                                                         const T* __restrict__ frame, const T* __restrict__ mu,
                                                         const T* __restrict__ Dfan, T* __restrict__ dose,
                                                         T* __restrict__ comp) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  constexpr int NW = PX * PY;
  const int nblk = zc * xc * yc;
  const int per_xcd = (nblk + 7) / 8;
  const int w = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (w >= nblk) return;
  const int zq = w % zc, xq = (w / zc) % xc, yq = w / (zc * xc);
  const int lane = threadIdx.x & 63;
  const int wave = uniform(threadIdx.x >> 6);
  const int x = xq * PX + wave % PX, y = yq * PY + wave / PX;
  if (x >= g.nx || y >= g.ny) return;  // (wavefronts are independent: no barriers below)
  const int z0 = zq * 64 * ZS + lane;
  const int js = JS ? JS : (g.Nv + 63) / 64;
  const int pitch = 64 * js + 2 * GATHER_PAD;
  GatherCol<T>* cols = reinterpret_cast<GatherCol<T>*>(smem_raw) + wave * GATHER_CHUNK;
  T* rows = reinterpret_cast<T*>(smem_raw + NW * GATHER_CHUNK * sizeof(GatherCol<T>)) + (size_t)wave * U * pitch;
  for (int q = lane; q < U * pitch; q += 64) rows[q] = T(0);  // the words beside j = 0 .. Nv - 1 stay zero

  GatherSum<T> sum[ZS];
  T tz[ZS];
#pragma unroll
  for (int s = 0; s < ZS; ++s) {
    const int z = z0 + 64 * s;
    tz[s] = g.rel_oz + T(z) * g.sz;
    if (!first && z < g.nz) {
      const size_t vox = ((size_t)z * g.ny + y) * g.nx + x;
      sum[s].load(dose[vox], comp[vox]);
    }
  }
  const int plane = g.Nu * g.Nv;
  const size_t cp_elems = (size_t)g.Nk * plane;
  const T tx = g.rel_ox + T(x) * g.sx, ty = g.rel_oy + T(y) * g.sy;
  bool bad = false;  // a non-finite MU makes every voxel NaN, also those its fan misses
  for (int b0 = 0; b0 < nb; b0 += GATHER_CHUNK) {
    // this lane's control point: its cell (k, i) and weights; those that reach the
    // column are listed in control-point order
    const int b = b0 + lane;
    bool hit = false;
    GatherCol<T> col;
    if (b < nb) {
      const T sn = frame[2 * b], cs = frame[2 * b + 1], m = mu[b];
      bad |= !(m - m == T(0));
      // voxel_to_fan without the z part (the fused products spelt out: the learned
      // correction's BF16 layers turn a dose's last bits into differences of 2.5e-5)
      const T ev = fma(cs, ty, -sn * tx);
      const T q = T(1) / (T(1) + ev * g.inv_sad);
      const T u = fma(cs, tx, sn * ty) * q;
      const T fkv = (ev - g.e0) * g.inv_dstep, fiv = u * g.inv_lat + g.cu;
      const T fk = dfloor(fkv), fi = dfloor(fiv);
      const bool in_ki = (fk >= T(-1)) & (fk < T(g.Nk)) & (fi >= T(-1)) & (fi < T(g.Nu));
      hit = !((fk < T(-1)) | (fk >= T(g.Nk)) | (fi < T(-1)) | (fi >= T(g.Nu)));  // (a NaN angle is not skipped)
      const int k0 = in_ki ? (int)fk : 0, i0 = in_ki ? (int)fi : 0;
      const T wk = fkv - fk, wi = fiv - fi;
      col.q = q;
      col.m = m;
      col.b = b;
      if constexpr (WIN) {
        // one pixel before the first z's, for rounding; from the zero beside the plane on
        const T fj = dfloor((g.rel_oz + T(zq * 64 * ZS) * g.sz) * q * g.inv_lat + g.cv);
        col.jb = min(max((int)fj - 1, -1), g.Nv);
      }
#pragma unroll
      for (int dk = 0; dk < 2; ++dk)
#pragma unroll
        for (int di = 0; di < 2; ++di) {
          const int kk = k0 + dk, ii = i0 + di;
          const bool ok = (kk >= 0) & (kk < g.Nk) & (ii >= 0) & (ii < g.Nu);
          const T wkk = dk ? wk : T(1) - wk, wii = di ? wi : T(1) - wi;
          col.w[2 * dk + di] = ok ? wkk * wii : T(0);
          col.off[2 * dk + di] = min(max(kk, 0), g.Nk - 1) * plane + min(max(ii, 0), g.Nu - 1) * g.Nv;
        }
    }
    const unsigned long long mask = __ballot(hit);
    if (hit) cols[__popcll(mask & ((1ull << lane) - 1ull))] = col;
    const int n = __popcll(mask);
    __builtin_amdgcn_wave_barrier();

    // UU listed control points: all their row loads, then the blended rows, then the z
    auto take = [&](int e0, auto uu) {
      constexpr int UU = decltype(uu)::value;
      if constexpr (JS > 0) {
        T v[UU][JS][4];
#pragma unroll
        for (int u = 0; u < UU; ++u) {
          const GatherCol<T>& c = cols[e0 + u];
          const T* base = Dfan + (size_t)uniform(c.b) * cp_elems;
#pragma unroll
          for (int cc = 0; cc < 4; ++cc) {
            const T* row = base + uniform(c.off[cc]);
#pragma unroll
            for (int s = 0; s < JS; ++s) {
              // (lanes past the window read its last pixel again)
              const int j = WIN ? max(uniform(c.jb) + min(64 * s + lane, win - 1), 0) : 64 * s + lane;
              v[u][s][cc] = row[(unsigned)min(j, g.Nv - 1)];
            }
          }
        }
#pragma unroll
        for (int u = 0; u < UU; ++u) {
          const GatherCol<T>& c = cols[e0 + u];
#pragma unroll
          for (int s = 0; s < JS; ++s) {
            T r = T(0);
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) r += c.w[cc] * v[u][s][cc];
            if constexpr (WIN) {
              const int j = uniform(c.jb) + 64 * s + lane;
              rows[u * pitch + GATHER_PAD + 64 * s + lane] = j >= 0 && j < g.Nv ? r : T(0);
            } else if (64 * s + lane < g.Nv) {
              rows[u * pitch + GATHER_PAD + 64 * s + lane] = r;
            }
          }
        }
      } else {
        const GatherCol<T>& c = cols[e0];
        const T* base = Dfan + (size_t)uniform(c.b) * cp_elems;
        for (int j = lane; j < g.Nv; j += 64) {
          T r = T(0);
#pragma unroll
          for (int cc = 0; cc < 4; ++cc) r += c.w[cc] * base[uniform(c.off[cc]) + j];
          rows[GATHER_PAD + j] = r;
        }
      }
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int u = 0; u < UU; ++u) {
        const T q = cols[e0 + u].q, m = cols[e0 + u].m;
        const T* row = rows + u * pitch + GATHER_PAD;
#pragma unroll
        for (int s = 0; s < ZS; ++s) {
          const T fjv = tz[s] * q * g.inv_lat + g.cv;
          const T fj = dfloor(fjv), wj = fjv - fj;
          // outside the plane both words are zero
          int j = min(max((int)fj, -GATHER_PAD), g.Nv);
          if constexpr (WIN) j = min(max(j - uniform(cols[e0 + u].jb), -GATHER_PAD), 64 * JS);
          const T lo = row[j], hi = row[j + 1];
          sum[s].add(m * (lo + wj * (hi - lo)));
        }
      }
      __builtin_amdgcn_wave_barrier();
    };
    int e = 0;
    for (; e + U <= n; e += U) take(e, std::integral_constant<int, U>());
    if constexpr (U > 1)
      for (; e < n; ++e) take(e, std::integral_constant<int, 1>());
  }
  const bool any_bad = __ballot(bad) != 0;  // (over the whole wavefront, before lanes past nz drop out)
#pragma unroll
  for (int s = 0; s < ZS; ++s) {
    const int z = z0 + 64 * s;
    if (z >= g.nz) continue;
    const size_t vox = ((size_t)z * g.ny + y) * g.nx + x;
    if (any_bad) sum[s].add(T(__builtin_nanf("")));
    if (last)
      dose[vox] = sum[s].value(g.calib);
    else
      sum[s].store(dose + vox, comp + vox);
  }
}

template <typename T, int JS, int ZS, bool WIN>
static hipError_t launch_gather_cfg(const Geo<T>& g, int nb, int first, int last, int win, const T* frame, const T* mu,
                                    const T* Dfan, T* dose, T* comp, hipStream_t s) {
  // Two control points in flight: four need more registers and lose more to the lower
  // occupancy than they hide (128^3: 0.58 ms against 0.43); one: 0.40, but 0.11 against
  // 0.09 on the 43-wide planes.  2 x 2 patches of independent wavefronts: 0.41 against
  // 0.43 with 4 x 4 (192 x 192 x 128: 0.51 against 0.56).
  constexpr int PX = 2, PY = 2, U = JS == 0 || sizeof(T) == 8 ? 1 : 2;
  const int zc = (g.nz + 64 * ZS - 1) / (64 * ZS), xc = (g.nx + PX - 1) / PX, yc = (g.ny + PY - 1) / PY;
  const long nblk = (long)zc * xc * yc;
  if (nblk > 0x7ffffff0L) return hipErrorInvalidConfiguration;
  const int js = JS ? JS : (g.Nv + 63) / 64;
  const size_t lds = (size_t)PX * PY * (GATHER_CHUNK * sizeof(GatherCol<T>) + U * (64 * js + 2 * GATHER_PAD) * sizeof(T));
  if (lds > 160 * 1024) return hipErrorInvalidConfiguration;
  const void* kern = (const void*)k_gather<T, JS, ZS, PX, PY, U, WIN>;
  {
    hipError_t e = ensure_lds_limit(kern, (int)lds);
    if (e != hipSuccess) return e;
  }
  const int grid = (int)((nblk + 7) / 8 * 8);
  hipLaunchKernelGGL((k_gather<T, JS, ZS, PX, PY, U, WIN>), dim3(grid), dim3(64 * PX * PY), lds, s, g, nb, first, last,
                     win, zc, xc, yc, frame, mu, Dfan, dose, comp);
  return hipGetLastError();
}

template <typename T, int JS, bool WIN>
static hipError_t launch_gather_js(const Geo<T>& g, int nb, int first, int last, int win, const T* frame, const T* mu,
                                   const T* Dfan, T* dose, T* comp, hipStream_t s) {
  if (g.nz <= 64) return launch_gather_cfg<T, JS, 1, WIN>(g, nb, first, last, win, frame, mu, Dfan, dose, comp, s);
  if (g.nz <= 128) return launch_gather_cfg<T, JS, 2, WIN>(g, nb, first, last, win, frame, mu, Dfan, dose, comp, s);
  return launch_gather_cfg<T, JS, 3, WIN>(g, nb, first, last, win, frame, mu, Dfan, dose, comp, s);
}

// Pixels of the window that a wavefront's z reach, largest next to the source
// (columns reached lie at most a plane outside the planes): the step between the first
// and last z, a pixel at each end for the cells' two sides and one for rounding.
template <typename T>
static int gather_window(const Geo<T>& g) {
  const double d = 1.0 + ((double)g.e0 - (double)g.dstep) * (double)g.inv_sad;  // SAD / d at its largest
  if (!(d > 1e-3)) return 1 << 20;
  const int nzw = min(g.nz, g.nz <= 64 ? 64 : g.nz <= 128 ? 128 : 192);
  const double span = (double)(nzw - 1) * (double)g.sz * (double)g.inv_lat / d * (1.0 + 1e-5);
  return span < 1e6 ? (int)span + 6 : 1 << 20;
}

template <typename T>
hipError_t launch_gather(const Geo<T>& g, int nb, int first, int last, const T* frame, const T* mu, const T* Dfan,
                         T* dose, T* comp, hipStream_t s) {
  if ((long)g.Nk * g.Nu * g.Nv > 0x7fffffffL) return hipErrorInvalidConfiguration;  // 32-bit corner offsets
  const int js = (g.Nv + 63) / 64, win = gather_window(g);
  if ((win + 63) / 64 < js) {
    switch ((win + 63) / 64) {
      case 1: return launch_gather_js<T, 1, true>(g, nb, first, last, win, frame, mu, Dfan, dose, comp, s);
      case 2: return launch_gather_js<T, 2, true>(g, nb, first, last, win, frame, mu, Dfan, dose, comp, s);
      case 3: return launch_gather_js<T, 3, true>(g, nb, first, last, win, frame, mu, Dfan, dose, comp, s);
      case 4: return launch_gather_js<T, 4, true>(g, nb, first, last, win, frame, mu, Dfan, dose, comp, s);
      default: break;
    }
  }
  switch (js) {
    case 1: return launch_gather_js<T, 1, false>(g, nb, first, last, 0, frame, mu, Dfan, dose, comp, s);
    case 2: return launch_gather_js<T, 2, false>(g, nb, first, last, 0, frame, mu, Dfan, dose, comp, s);
    case 3: return launch_gather_js<T, 3, false>(g, nb, first, last, 0, frame, mu, Dfan, dose, comp, s);
    case 4: return launch_gather_js<T, 4, false>(g, nb, first, last, 0, frame, mu, Dfan, dose, comp, s);
    default: return launch_gather_js<T, 0, false>(g, nb, first, last, 0, frame, mu, Dfan, dose, comp, s);
  }
}

#define PDRT_INST(T)                                                                                         \
  template hipError_t launch_frame<T>(const Geo<T>&, const T*, int, T*, hipStream_t);                        \
  template hipError_t launch_transpose_rho<T>(const Geo<T>&, const T*, T*, hipStream_t);                     \
  template hipError_t launch_raster<T>(const Geo<T>&, int, const T*, const T*, T*, hipStream_t);             \
  template hipError_t launch_aperture_box<T>(const Geo<T>&, int, const T*, int, int, int*, hipStream_t);     \
  template hipError_t launch_ca_depth<T>(const Geo<T>&, int, const T*, const T*, T*, hipStream_t);           \
  template hipError_t launch_march<T>(const Geo<T>&, int, const T*, const T*, const T*, const T*, const T*, T*, \
                                      hipStream_t, const int*);                                              \
  template hipError_t launch_march_adj<T>(const Geo<T>&, int, const T*, const T*, const T*, const T*, const T*, \
                                          T*, hipStream_t, const int*);                                      \
  template hipError_t launch_conv_direct<T>(const Geo<T>&, int, const T*, const T*, T*, hipStream_t);        \
  template hipError_t launch_gather<T>(const Geo<T>&, int, int, int, const T*, const T*, const T*, T*, T*,    \
                                       hipStream_t);

PDRT_INST(float)
PDRT_INST(double)

}  // namespace pdrt
