// conv_adj.hip — the adjoint per-plane lateral convolution (arXiv:2512.18863 §2.2.6,
// Eq. 8) on the CDNA4 BF16 matrix instructions, in FP32 (operands as three BF16 pieces)
// or with BF16 operands, for outputs that are needed
// inside the aperture rectangle only (the parameter gradients read them there).
//
// out[i][j] = sum_{p,q} K[p][q] in[i+p][j+q] = sum_{p >= 0} sum_c K[p][c - j] S_p[i][c],
//   S_p[i][c] = in[i+p][c] + in[i-p][c]   (the taps are even in p; row 0 counts half),
// a product per tap row p with M = 16 output columns j, N = 16 output rows i and K = 32
// plane columns c (a group):
//   A[m][k] = K[p][c_k - j_m] (from the extended tap row), B[k][n] = S_p[i_n][c_k].
// The window of plane rows and columns that a piece of T x CB output tiles reads sits
// in LDS in FP32; a wavefront forms S_p in FP32 and splits it, like the taps, exactly
// into three BF16 pieces (conv_fwd_reg.hip: six exact piece products per product, what is
// left out, FP32 sums; error of the output against FP64 on the 128^3 plan 7.1e-7 on FP32
// matrix instructions, 1.6e-7 now, with fluence corrections and collimator rotation 9.9e-7
// and 2.6e-7).  Folding the two rows first halves the matrix work; the split is
// done in the vector unit, which the matrix instructions leave free.
//
// One workgroup per (control point, plane) item and piece; a rectangle's pieces have equal
// numbers of tiles.  Its wavefronts share the (column group, tap row) pairs evenly, each
// for all T x CB tiles, so a split feeds CB tiles and a tap run T.  Their sums are added in LDS in wavefront order, one row of
// tiles at a time.  (Wavefronts come in multiples of four: a workgroup of six, two on
// two of the SIMDs, kept a second one off the compute unit.)
//
// A lane's K entries of a group are columns 4 kk + 0..3 and 16 + 4 kk + 0..3 (A and B
// agree), so that its image reads are two 16-byte reads at n P + 4 kk words, free of
// bank conflicts for a pitch P of 8 (mod 16) words.
//
// What bounds it: vector instructions, 52 per S_p fragment beside 12 to 24 matrix
// instructions of 16 cycles.  FP32 against the windowed kernel on FP32 matrix
// instructions (conv_mfma.hip, which remains for h > 31): 180 control points at 128^3 (n
// = 61, 27 x 27 outputs) 1.34 to 1.39 ms by clock (1.61), at 224 x 224 x 105 (n = 55, 41 x
// 41) 3.5 ms (5.8), at 192 x 192 x 128 (n = 31) 0.88 ms (1.15), 90 at 128 x 128 x 96 (n =
// 15) 0.13 ms (0.22); 90 with fluence corrections and collimator rotation (up to 99 x 99)
// 6.5 ms (9.1 by regions).  BF16: 1.8 ms on the second (2.9), 0.086 on the fourth (0.14),
// 3.8 on the last (13).
#include <type_traits>

#include "conv_common.hpp"

namespace pdrt {

namespace {

typedef float f32x4a __attribute__((ext_vector_type(4)));
typedef unsigned u32x4a __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8a __attribute__((ext_vector_type(8)));
typedef float f32x4ua __attribute__((ext_vector_type(4), aligned(4)));

__host__ __device__ inline int adj_img_rows(int T, int h) { return 16 * T + 2 * h; }

// NP pieces per operand: 3 (FP32) or 1 (BF16; the rows are then not folded).
template <int NP, int T, int CB>
__global__ void __launch_bounds__(512, T <= 2 ? 5 : T == 3 ? 4 : 2) k_conv_adj(Geo<float> g, int pitch, const int4* __restrict__ box,
                                                      const float* __restrict__ zca, const float* __restrict__ in,
                                                      float* __restrict__ out) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int h = g.h, h1 = h + 1;
  const int CS = h1 * NP * kRegW;
  unsigned* taps = reinterpret_cast<unsigned*>(smem_raw);
  float* img = reinterpret_cast<float*>(taps + reg_tap_words(h, NP));
  f32x4a* sums = reinterpret_cast<f32x4a*>(img);  // [wavefront][CB][64], once the image is no longer read
  const int NT = blockDim.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = NT >> 6;
  const int bk = blockIdx.x;
  const int b = bk / g.Nk, k = bk - b * g.Nk;
  const int Nu = g.Nu, Nv = g.Nv;
  const size_t plane = (size_t)Nu * Nv;
  const int4 bx = box[b];
  const int r0 = max(bx.x, 0), r1 = min(bx.y, Nu), c0 = max(bx.z, 0), c1 = min(bx.w, Nv);
  if (r1 <= r0 || c1 <= c0) return;
  // pieces of equal numbers of tiles, tr x tc
  const int nr = (r1 - r0 + 15) / 16, nc = (c1 - c0 + 15) / 16;
  const int npi = (nr + T - 1) / T, npj = (nc + CB - 1) / CB;
  int tr = nr, tc = nc;
  if (npi > 1) tr = (nr + npi - 1) / npi;
  if (npj > 1) tc = (nc + npj - 1) / npj;
  if ((int)blockIdx.y >= npi * npj) return;
  const float* src = in + (size_t)bk * plane;
  float* dst = out + (size_t)bk * plane;
  const int n = lane & 15, kk = lane >> 4;
  clear_tap_rows(taps, h, NP, tid, NT);
  bool built = false;

  for (int pp = blockIdx.y; pp < npi * npj; pp += gridDim.y) {
    const int I = r0 + 16 * tr * (pp / npj), J = c0 + 16 * tc * (pp % npj);
    const int I1 = min(I + 16 * tr, r1), J1 = min(J + 16 * tc, c1);
    // the window: plane rows I - h + [0, 16 tr + 2 h), zero outside the plane, and columns
    // [wc0, wc1), zero up to the end of their last group; a four-column group that starts
    // inside a row may read up to three words past its end (the next row, or after the
    // batch's last row the workspace that follows)
    const int wc0 = max(0, J - h), wc1 = min(Nv, J1 + h);
    const int ng = (wc1 - wc0 + 31) / 32, gw = 8 * ng;
    for (RectWalk w(tid, NT, gw); w.r < 16 * tr + 2 * h; w.next(gw)) {
      const int r = w.r, q = w.c;
      const int pr = I - h + r, pc = wc0 + 4 * q;
      f32x4a v = {0.f, 0.f, 0.f, 0.f};
      if (pr >= 0 && pr < Nu && pc < wc1) {
        const f32x4ua x = *reinterpret_cast<const f32x4ua*>(src + (size_t)pr * Nv + pc);
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = pc + c < wc1 ? x[c] : 0.f;
      }
      *reinterpret_cast<f32x4a*>(img + r * pitch + 4 * q) = v;
    }
    if (!built) {
      lds_barrier();  // the rows are cleared
      build_tap_rows<NP>(g, k, zca[bk], taps, tid, NT, 0.5f);
      built = true;
    }
    lds_barrier();

    f32x4a acc[T][CB];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int c = 0; c < CB; ++c) acc[t][c] = f32x4a{0.f, 0.f, 0.f, 0.f};
    // all the pairs (gq, p), p fastest, of this wavefront, for TT x CC tiles
    auto products = [&](auto tt, auto cb) {
      constexpr int TT = decltype(tt)::value, CC = decltype(cb)::value;
      const int ua = ng * h1 * wave / nw, uz = ng * h1 * (wave + 1) / nw;
      for (int gq = ua / h1; gq * h1 < uz; ++gq) {
        const int pa = max(ua - gq * h1, 0), pz = min(uz - gq * h1, h1);
        // tap runs of the lane: four taps each for columns 4 kk and 16 + 4 kk of the group, a
        // run that meets no tap moved to the zeros beside them.  (Word offsets into the rows,
        // not pointers: pointers kept in an array lost their address space with one column of
        // tiles, and generic loads took the place of LDS reads, 0.57 against 0.20 ms for 90
        // control points of 98 planes, n = 61.)
        int run[CC][2];
#pragma unroll
        for (int c = 0; c < CC; ++c)
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            int x = kRegOff + wc0 + 32 * gq + 16 * e + 4 * kk - (J + 16 * c + n);
            const int x0 = kRegOff - h - 5, x1 = kRegOff + h + 1;
            if (x < x0 + 1) x = x0 + ((x ^ x0) & 1);
            if (x > x1) x = x1 + ((x ^ x1) & 1);
            run[c][e] = ((x & 1) ? CS : 0) + (x >> 1) + pa * NP * kRegW;
          }
        const float* up = img + (n + h + pa) * pitch + 32 * gq + 4 * kk;
        const float* dn = img + (n + h - pa) * pitch + 32 * gq + 4 * kk;
#pragma unroll 1
        for (int p = pa; p < pz; ++p) {
          u32x4a A[CC][NP];
#pragma unroll
          for (int c = 0; c < CC; ++c)
#pragma unroll
            for (int i = 0; i < NP; ++i)
              A[c][i] = u32x4a{taps[run[c][0] + i * kRegW], taps[run[c][0] + i * kRegW + 1],
                               taps[run[c][1] + i * kRegW], taps[run[c][1] + i * kRegW + 1]};
#pragma unroll
          for (int t = 0; t < TT; ++t) {
            // FP32: the pieces of the folded rows; BF16: the rows i + p and i - p rounded
            // one by one, so that every input is rounded by itself
            constexpr int NB = NP == 3 ? 3 : 2;
            u32x4a B[NB];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              const f32x4a x = *reinterpret_cast<const f32x4a*>(up + 16 * t * pitch + 16 * e),
                           y = *reinterpret_cast<const f32x4a*>(dn + 16 * t * pitch + 16 * e);
#pragma unroll
              for (int w = 0; w < 2; ++w) {
                if constexpr (NP == 3) {
                  unsigned u[NP];
                  reg_pieces2<NP>(x[2 * w] + y[2 * w], x[2 * w + 1] + y[2 * w + 1], u);
#pragma unroll
                  for (int i = 0; i < NP; ++i) B[i][2 * e + w] = u[i];
                } else {
                  unsigned u[1];
                  reg_pieces2<1>(x[2 * w], x[2 * w + 1], u);
                  B[0][2 * e + w] = u[0];
                  reg_pieces2<1>(y[2 * w], y[2 * w + 1], u);
                  B[1][2 * e + w] = u[0];
                }
              }
            }
            // (piece of A, piece of B), smallest products first
            constexpr int np = NP == 3 ? 6 : 2, qa[6] = {2, 0, 1, 1, 0, 0}, qb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
            for (int i = 0; i < np; ++i)
#pragma unroll
              for (int c = 0; c < CC; ++c)
                acc[t][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                    __builtin_bit_cast(bf16x8a, A[c][NP == 3 ? qa[i] : 0]),
                    __builtin_bit_cast(bf16x8a, B[NP == 3 ? qb[i] : i]), acc[t][c], 0, 0, 0);
          }
          up += pitch;
          dn -= pitch;
#pragma unroll
          for (int c = 0; c < CC; ++c) {
            run[c][0] += NP * kRegW;
            run[c][1] += NP * kRegW;
          }
        }
      }
    };
    // a rectangle (or its last piece) one row or column of tiles smaller leaves them out,
    // and one of an opening far inside the field limits takes the least square that holds it
    typedef std::integral_constant<int, T> FT;
    typedef std::integral_constant<int, (T > 1 ? T - 1 : 1)> ST;
    typedef std::integral_constant<int, CB> FC;
    typedef std::integral_constant<int, (CB > 1 ? CB - 1 : 1)> SC;
    typedef std::integral_constant<int, 1> One;
    typedef std::integral_constant<int, 2> Two;
    const bool st = I1 - I <= 16 * (T - 1), sc = J1 - J <= 16 * (CB - 1);
    const int side = max(I1 - I, J1 - J);
    if (T > 2 && side <= 16) {
      products(One(), One());
    } else if (T > 3 && side <= 32) {
      products(Two(), Two());
    } else if (st) {
      if (sc) products(ST(), SC());
      else products(ST(), FC());
    } else {
      if (sc) products(FT(), SC());
      else products(FT(), FC());
    }
    // the wavefronts' sums, one row of tiles at a time; lane (n, kk) holds output row n
    // and columns 4 kk + e of a tile
#pragma unroll
    for (int t = 0; t < T; ++t) {
      lds_barrier();
#pragma unroll
      for (int c = 0; c < CB; ++c) sums[(wave * CB + c) * 64 + lane] = acc[t][c];
      lds_barrier();
      for (int c = wave; c < CB; c += nw) {
        f32x4a v = sums[c * 64 + lane];
        for (int w = 1; w < nw; ++w) v += sums[(w * CB + c) * 64 + lane];
        const int i = I + 16 * t + n, j = J + 16 * c + 4 * kk;
        if (i < min(I + 16 * tr, Nu)) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (j + e < min(J + 16 * tc, Nv)) dst[(size_t)i * Nv + j + e] = v[e];
        }
      }
    }
    lds_barrier();  // the next piece's window overwrites the sums
  }
}

// LDS of a workgroup for pieces of n x n tiles, and its wavefronts: four for small
// kernels and for pieces of four where two workgroups fit a compute unit.
int adj_pitch(const Geo<float>& g, int n) { return (min(g.Nv, 16 * n + 2 * g.h) + 31) / 32 * 32 + 8; }
size_t adj_lds(const Geo<float>& g, int np, int n) {
  const size_t img = sizeof(float) * (size_t)adj_img_rows(n, g.h) * adj_pitch(g, n), red = (size_t)8 * n * 1024;
  return sizeof(unsigned) * (size_t)reg_tap_words(g.h, np) + (img > red ? img : red);
}
bool adj_two_fit(const Geo<float>& g, int np, int n) { return adj_lds(g, np, n) <= 80 * 1024; }
int adj_waves(const Geo<float>& g, int np, int n) { return g.h <= 16 || (n == 4 && adj_two_fit(g, np, n)) ? 4 : 8; }

// Estimated time of a rectangle of side `side` pixels in pieces of n x n tiles: column
// groups over all pieces x time of a (group, tap row) pair, measured relative to pieces of
// two: three 1.45 and four 2.8 (BF16: 1.25, 1.55), pieces that are a tile smaller than their
// kernel 0.7 of that (BF16 pieces of four: all of it), and where FP32 windows leave one
// workgroup to a compute unit 1.75 (pieces of four, which have few wavefronts anyway, 1.1).
double adj_cost(const Geo<float>& g, int np, int n, double side) {
  const int blocks = max(1, (int)ceil(side / 16.0)), m = (blocks + n - 1) / n, tiles = (blocks + m - 1) / m;
  const double c0 = 0.5 * (g.Nv - side);  // the rectangle's first column
  double groups = 0.0;
  for (int j = 0; j < m; ++j) {
    const double a = fmax(0.0, c0 + 16 * tiles * j - g.h);
    const double b = fmin(g.Nv, fmin(c0 + 16 * tiles * (j + 1), c0 + side) + g.h);
    groups += fmax(1.0, ceil((b - a) / 32.0 - 1e-9));
  }
  const double pair[5] = {0.0, 0.0, 1.0, np == 3 ? 1.45 : 1.25, np == 3 ? 2.8 : 1.55};
  double cost = m * groups * pair[n];
  if (tiles < n && (np == 3 || n < 4)) cost *= 0.7;
  if (np == 3 && !adj_two_fit(g, np, n)) cost *= n < 4 ? 1.75 : 1.1;
  return cost;
}

// Tiles per side of a piece for rectangles that are usually of side `usual` and at most
// `most` pixels: one piece up to three tiles; above, the least of both sides' times (a
// rectangle at the limits may take a row of tiles more, and with it more pieces), weighed
// as fits best 650 shapes of 13 to 61 taps and 7 to 97 pixels with and without corrections
// and rotation, openings at the limits and up to a tenth inside: 1 : 0.7, BF16 1 : 1.  FP32,
// 75 planes each:
//   60 control points, n = 13, 57 x 57 pixels  0.136 ms in pieces of 2, 0.164 of 3, 0.156 of 4
//   20, n = 13, 121 x 121                      0.168, 0.148, 0.191
//   60, n = 45, 57 x 57                        0.53, 0.58, 0.46
//   60, n = 61, 57 x 57                        0.66, 1.03, 0.76
//   40, n = 55, 103 x 103 (corrections)        1.24, 1.74, 1.17
int adj_tiles(const Geo<float>& g, int np, double usual, double most) {
  const int blocks = (int)ceil(most / 16.0);
  if (blocks <= 3) return max(1, blocks);
  int best = 2;
  double least = 1e30;
  for (int n = 2; n <= 4; ++n) {
    const double cost = adj_cost(g, np, n, usual) + (np == 3 ? 0.7 : 1.0) * adj_cost(g, np, n, most);
    if (cost < least) {
      least = cost;
      best = n;
    }
  }
  return best;
}

template <int NP, int N>
hipError_t launch_adj_cfg(const Geo<float>& g, int nb, int pieces, const int4* box, const float* z, const float* in,
                          float* out, hipStream_t s) {
  const size_t lds = adj_lds(g, NP, N);
  if (lds > 160 * 1024) return hipErrorInvalidConfiguration;
  const void* kern = (const void*)k_conv_adj<NP, N, N>;
  {
    hipError_t e = ensure_lds_limit(kern, (int)lds);
    if (e != hipSuccess) return e;
  }
  const long n_items = (long)nb * g.Nk;
  if (n_items > 0x7fffffffL) return hipErrorInvalidConfiguration;
  hipLaunchKernelGGL((k_conv_adj<NP, N, N>), dim3((unsigned)n_items, pieces), dim3(64 * adj_waves(g, NP, N)), lds, s, g,
                     adj_pitch(g, N), box, z, in, out);
  return hipGetLastError();
}

template <int NP>
hipError_t launch_adj_np(const Geo<float>& g, int nb, const int4* box, const float* z, const float* in, float* out,
                         hipStream_t s) {
  // the largest rectangle that jaws inside the field limits give, widened by fluence
  // corrections and collimator rotation, sets the number of workgroups per item (a larger
  // one has them take several pieces); the usual one, of openings a little inside the
  // limits and angles short of the diagonal, the pieces' size
  const int half_u = (g.Nu - 1) / 2 - g.h, half_v = (g.Nv - 1) / 2 - g.h;  // field limit in pixels
  const int fu = 2 * (half_u > 0 ? half_u : 0) + 1, fv = 2 * (half_v > 0 ? half_v : 0) + 1;
  const int br = min(g.Nu, fu + 2 * g.conv_du), bc = min(g.Nv, fv + 2 * g.conv_dv);
  const bool turned = g.conv_du != g.box_du || g.conv_dv != g.box_dv;
  const double open = turned ? 0.9 : 0.95, wide = turned ? 1.4 : 2.0;
  const double ur = fmin(g.Nu, open * fu + wide * g.conv_du), uc = fmin(g.Nv, open * fv + wide * g.conv_dv);
  const int n = adj_tiles(g, NP, fmax(ur, uc), br > bc ? br : bc);
  const int pieces = ((br + 16 * n - 1) / (16 * n)) * ((bc + 16 * n - 1) / (16 * n));
  switch (n) {
    case 1: return launch_adj_cfg<NP, 1>(g, nb, pieces, box, z, in, out, s);
    case 2: return launch_adj_cfg<NP, 2>(g, nb, pieces, box, z, in, out, s);
    case 3: return launch_adj_cfg<NP, 3>(g, nb, pieces, box, z, in, out, s);
    default: return launch_adj_cfg<NP, 4>(g, nb, pieces, box, z, in, out, s);
  }
}

}  // namespace

bool conv_adj_supported(const Geo<float>& g) { return g.h >= 1 && g.h <= kRegMaxH; }

hipError_t launch_conv_adj(const Geo<float>& g, int nb, const float* z, const float* in, float* out, hipStream_t s,
                           const int* box, bool bf16) {
  if (!conv_adj_supported(g) || !box) return hipErrorInvalidConfiguration;
  const int4* bx = reinterpret_cast<const int4*>(box);
  return bf16 ? launch_adj_np<1>(g, nb, bx, z, in, out, s) : launch_adj_np<3>(g, nb, bx, z, in, out, s);
}

}  // namespace pdrt
