// net_wgrad.hip — weight and bias gradients of the network's 3 x 3 x 3
// convolutions on the matrix cores,
//   dW[co][tap][ci] = sum_p dY'[p][co] X[p + o(tap)][ci],  dY' = dY * [Y > 0],
//   db[co] = sum_p dY'[p][co].
//
// For one tap this is a product over positions: v_mfma_f32_16x16x32_bf16 with M =
// 16 output channels, N = 16 input channels and K = 32 consecutive positions along
// w.  Tensors are channels-last, so a lane's eight consecutive positions of one
// channel are strided in memory: the operands are transposed on their way into LDS
// (a thread loads eight positions x eight channels, swaps half-words in registers
// and stores eight 16-byte runs), and the three shifts along w are taken from six
// words of a row by word alignment.
//
// A workgroup of three wavefronts, one per tap plane td, owns NCI tiles of 16 input
// channels and all (up to 16 CO_T) output channels, and walks the position tiles of
// its split: 32 (w) x 4 (h) outputs, three planes of six input rows with the halo.
// Each wavefront reads every staged input row once and uses it for the three h
// shifts and three w shifts (9 taps), 36 CO_T NCI matrix instructions per tile.
// Positions outside the volume are staged as zero.  Splits are contiguous tile
// ranges; their partial sums are added in split order, so results do not depend on
// scheduling.
//
// What bounds it: staging (loads and transposes between two barriers), covered by
// the other workgroups on the compute unit.  The ten layers of the 128^3 network
// take 1.3 ms (264 GFLOP, 200 TFLOP/s); one thread per (tap, co, ci) summing its
// positions on the vector ALUs, the kernel that remains for unaligned buffers and
// other channel counts, took 130 ms.
#include "pdrt_internal.hpp"

namespace pdrt {

namespace {

typedef float wf32x4 __attribute__((ext_vector_type(4)));
typedef unsigned wu32x4 __attribute__((ext_vector_type(4)));
typedef unsigned wu32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 wbf16x8 __attribute__((ext_vector_type(8)));

constexpr int WG_W = 32, WG_H = 4;        // output positions per tile
constexpr int WG_XR = WG_H + 2;           // staged input rows per plane
constexpr int WG_P = 40;                  // row pitch in positions: input row element x is position w0 - 2 + x
constexpr int WG_PW = WG_P / 2;           // ... in words
constexpr int WG_NT = 192;                // three wavefronts

// (lo half-words of a and b) or (hi half-words), a first.
__device__ __forceinline__ unsigned lo_pair(unsigned a, unsigned b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ unsigned hi_pair(unsigned a, unsigned b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// v[i] holds channels 0..7 of position i; row c of the result holds positions 0..7
// of channel c, stored at dst + c * pitch words.
__device__ __forceinline__ void store_transposed(const wu32x4 (&v)[8], unsigned* dst, int pitch) {
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    wu32x4 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const unsigned a = v[2 * j][c / 2], b = v[2 * j + 1][c / 2];
      r[j] = (c & 1) ? hi_pair(a, b) : lo_pair(a, b);
    }
    *reinterpret_cast<wu32x4*>(dst + c * pitch) = r;
  }
}

// The half-words of g whose counterpart in y is a positive BF16 number.
__device__ __forceinline__ unsigned relu_mask(unsigned g, unsigned y) {
  const float lo = __uint_as_float(y << 16), hi = __uint_as_float(y & 0xffff0000u);
  return (lo > 0.f ? g & 0xffffu : 0u) | (hi > 0.f ? g & 0xffff0000u : 0u);
}

template <int CO_T, int NCI>
__global__ void __launch_bounds__(WG_NT) k_conv3d_wgrad_mfma(Vol v, int C1, int C2, const __bf16* __restrict__ X1,
                                                             const __bf16* __restrict__ X2, int Cout,
                                                             const __bf16* __restrict__ dY,
                                                             const __bf16* __restrict__ Yact,
                                                             float* __restrict__ part, float* __restrict__ partb) {
  // [3 planes][WG_XR rows][16 NCI channels][WG_PW] and [WG_H rows][16 CO_T channels][WG_PW] words
  __shared__ __align__(16) unsigned xs[3 * WG_XR * 16 * NCI * WG_PW];
  __shared__ __align__(16) unsigned ys[WG_H * 16 * CO_T * WG_PW];
  const int tid = threadIdx.x, lane = tid & 63;
  const int td = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = lane & 15, kq = lane >> 4;
  const int Cin = C1 + C2, c0 = 16 * NCI * blockIdx.y, split = blockIdx.x, nsplit = gridDim.x;
  const int tw = (v.W + WG_W - 1) / WG_W, th = (v.H + WG_H - 1) / WG_H;
  const long tiles = (long)tw * th * v.D;
  const long ta = tiles * split / nsplit, tb = tiles * (split + 1) / nsplit;
  const bool bias = td == 1 && blockIdx.y == 0;

  wf32x4 acc[9][NCI][CO_T], accb[CO_T];
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int a = 0; a < NCI; ++a)
#pragma unroll
      for (int c = 0; c < CO_T; ++c) acc[t][a][c] = wf32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < CO_T; ++c) accb[c] = wf32x4{0.f, 0.f, 0.f, 0.f};

  for (long tile = ta; tile < tb; ++tile) {
    const int w0 = (int)(tile % tw) * WG_W;
    const int h0 = (int)((tile / tw) % th) * WG_H;
    const int d0 = (int)(tile / ((long)tw * th));
    __syncthreads();  // the previous tile is no longer read
    // input: unit = (plane, row, block of 8 positions, group of 8 channels), channels fastest
    for (int u = tid; u < 3 * WG_XR * 5 * 2 * NCI; u += WG_NT) {
      const int cg = u % (2 * NCI), wb = (u / (2 * NCI)) % 5, row = (u / (10 * NCI)) % WG_XR, pl = u / (10 * NCI * WG_XR);
      const int dd = d0 + pl - 1, hh = h0 + row - 1, c = c0 + 8 * cg;
      wu32x4 x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = wu32x4{0u, 0u, 0u, 0u};
      if (dd >= 0 && dd < v.D && hh >= 0 && hh < v.H && c < Cin) {
        const bool first = c < C1;
        const int stride = first ? C1 : C2;
        const __bf16* src = (first ? X1 + c : X2 + (c - C1)) + (size_t)((long)dd * v.H + hh) * v.W * stride;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int w = w0 - 2 + 8 * wb + i;
          if (w >= 0 && w < v.W) x[i] = *reinterpret_cast<const wu32x4*>(src + (size_t)w * stride);
        }
      }
      store_transposed(x, xs + ((pl * WG_XR + row) * 16 * NCI + 8 * cg) * WG_PW + 4 * wb, WG_PW);
    }
    // output gradient, masked by the activation: unit = (row, block of 8 positions, group of 8 channels)
    for (int u = tid; u < WG_H * 4 * 2 * CO_T; u += WG_NT) {
      const int cg = u % (2 * CO_T), wb = (u / (2 * CO_T)) % 4, row = u / (8 * CO_T);
      const int hh = h0 + row, c = 8 * cg;
      wu32x4 x[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) x[i] = wu32x4{0u, 0u, 0u, 0u};
      if (hh < v.H && c < Cout) {
        const size_t base = (size_t)((long)d0 * v.H + hh) * v.W * Cout + c;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int w = w0 + 8 * wb + i;
          if (w < v.W) x[i] = *reinterpret_cast<const wu32x4*>(dY + base + (size_t)w * Cout);
        }
        if (Yact) {
          wu32x4 y[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const int w = w0 + 8 * wb + i;
            y[i] = wu32x4{0u, 0u, 0u, 0u};
            if (w < v.W) y[i] = *reinterpret_cast<const wu32x4*>(Yact + base + (size_t)w * Cout);
          }
#pragma unroll
          for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) x[i][e] = relu_mask(x[i][e], y[i][e]);
        }
      }
      store_transposed(x, ys + (row * 16 * CO_T + 8 * cg) * WG_PW + 4 * wb, WG_PW);
    }
    __syncthreads();
    wu32x4 A[WG_H][CO_T];
#pragma unroll
    for (int r = 0; r < WG_H; ++r)
#pragma unroll
      for (int c = 0; c < CO_T; ++c)
        A[r][c] = *reinterpret_cast<const wu32x4*>(ys + ((r * CO_T + c) * 16 + m) * WG_PW + 4 * kq);
    if (bias) {
      const wu32x4 ones = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
#pragma unroll
      for (int r = 0; r < WG_H; ++r)
#pragma unroll
        for (int c = 0; c < CO_T; ++c)
          accb[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(wbf16x8, A[r][c]),
                                                            __builtin_bit_cast(wbf16x8, ones), accb[c], 0, 0, 0);
    }
    // input row r serves output rows r - th, th = 0..2 (input row 0 is h0 - 1)
#pragma unroll
    for (int r = 0; r < WG_XR; ++r) {
#pragma unroll
      for (int a = 0; a < NCI; ++a) {
        // words 0..5: positions w0 - 2 + 8 kq + 0..11; w shift tw starts at element tw + 1
        const unsigned* p = xs + ((td * WG_XR + r) * 16 * NCI + 16 * a + m) * WG_PW + 4 * kq;
        const wu32x4 q = *reinterpret_cast<const wu32x4*>(p);
        const wu32x2 q2 = *reinterpret_cast<const wu32x2*>(p + 4);
        const unsigned s01 = __builtin_amdgcn_alignbit(q[1], q[0], 16), s12 = __builtin_amdgcn_alignbit(q[2], q[1], 16),
                       s23 = __builtin_amdgcn_alignbit(q[3], q[2], 16), s34 = __builtin_amdgcn_alignbit(q2[0], q[3], 16),
                       s45 = __builtin_amdgcn_alignbit(q2[1], q2[0], 16);
        const wu32x4 B[3] = {wu32x4{s01, s12, s23, s34}, wu32x4{q[1], q[2], q[3], q2[0]}, wu32x4{s12, s23, s34, s45}};
#pragma unroll
        for (int t = 0; t < 3; ++t) {
          const int o = r - t;  // output row
          if (o < 0 || o >= WG_H) continue;
#pragma unroll
          for (int s = 0; s < 3; ++s)
#pragma unroll
            for (int c = 0; c < CO_T; ++c)
              acc[3 * t + s][a][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                  __builtin_bit_cast(wbf16x8, A[o][c]), __builtin_bit_cast(wbf16x8, B[s]), acc[3 * t + s][a][c], 0, 0, 0);
        }
      }
    }
  }
  // lane (n = m, kq) of a tile holds input channel n and output channels 4 kq + e
#pragma unroll
  for (int t = 0; t < 9; ++t)
#pragma unroll
    for (int a = 0; a < NCI; ++a)
#pragma unroll
      for (int c = 0; c < CO_T; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int co = 16 * c + 4 * kq + e, ci = c0 + 16 * a + m;
          if (co < Cout && ci < Cin) part[(((size_t)split * Cout + co) * 27 + 9 * td + t) * Cin + ci] = acc[t][a][c][e];
        }
  if (bias && partb && m == 0)
#pragma unroll
    for (int c = 0; c < CO_T; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int co = 16 * c + 4 * kq + e;
        if (co < Cout) partb[(size_t)split * Cout + co] = accb[c][e];
      }
}

// dW and db: outputs [0, n) sum part[k][i], outputs [n, n + nb) sum partb[k][i - n],
// both over the splits k.  A block owns 32 outputs; eight threads per output each add
// a contiguous range of splits in order, then the eight sums are added in order.
__global__ void __launch_bounds__(256) k_reduce_wgrad(int nsplit, size_t n, const float* __restrict__ part,
                                                      float* __restrict__ dW, int nb, const float* __restrict__ partb,
                                                      float* __restrict__ db) {
  __shared__ float red[8][32];
  const int l = threadIdx.x & 31, seg = threadIdx.x >> 5;
  const size_t i = (size_t)blockIdx.x * 32 + l;
  const bool w = i < n, b = !w && i < n + nb;
  const float* p = w ? part + i : partb + (i - n);
  const size_t stride = w ? n : nb;
  const int ka = (int)((long)nsplit * seg / 8), kb = (int)((long)nsplit * (seg + 1) / 8);
  float s = 0.f;
  if (w || b) {
#pragma unroll 8
    for (int k = ka; k < kb; ++k) s += p[k * stride];
  }
  red[seg][l] = s;
  __syncthreads();
  if (seg != 0 || !(w || b)) return;
#pragma unroll
  for (int q = 1; q < 8; ++q) s += red[q][l];
  (w ? dW[i] : db[i - n]) = s;
}

template <int CO_T, int NCI>
hipError_t launch_mfma(Vol v, int C1, int C2, const __bf16* X1, const __bf16* X2, int Cout, const __bf16* dY,
                       const __bf16* Yact, int ns, float* part, float* partb, hipStream_t s) {
  const int groups = (C1 + C2 + 16 * NCI - 1) / (16 * NCI);
  hipLaunchKernelGGL((k_conv3d_wgrad_mfma<CO_T, NCI>), dim3(ns, groups), dim3(WG_NT), 0, s, v, C1, C2, X1, X2, Cout, dY,
                     Yact, part, partb);
  return hipGetLastError();
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

// 16-byte loads of eight channels: every tensor 16-byte aligned, Cout a multiple of 8
// (C1 and C2 always are).  Other calls take the scalar kernel.
bool conv3d_wgrad_mfma_ok(const __bf16* X1, const __bf16* X2, int Cout, const __bf16* dY, const __bf16* Yact) {
  return Cout % 8 == 0 && Cout <= 64 && aligned16(X1) && aligned16(X2) && aligned16(dY) && aligned16(Yact);
}

// The splits that leave room for their bias sums in a workspace of nsplit splits'
// weight sums; 0 for nsplit == 1 (the bias is then summed by itself).
int conv3d_wgrad_splits(int Cin, int nsplit) { return (int)((size_t)nsplit * 27 * Cin / (27 * Cin + 1)); }

// db may be null: no bias sums (and no room for them needed).
hipError_t launch_conv3d_wgrad_mfma(Vol v, int C1, int C2, const __bf16* X1, const __bf16* X2, int Cout,
                                    const __bf16* dY, const __bf16* Yact, int ns, float* part, float* dW, float* db,
                                    hipStream_t s) {
  const int Cin = C1 + C2, nci = (Cin + 15) / 16;
  const size_t n = (size_t)Cout * 27 * Cin;
  float* partb = db ? part + ns * n : nullptr;
  hipError_t e;
  // tiles of input channels per workgroup: as many as keep its sums in registers
  // (9 NCI CO_T tiles of four registers, at most 144)
  if (Cout <= 16)
    e = nci >= 3 ? launch_mfma<1, 3>(v, C1, C2, X1, X2, Cout, dY, Yact, ns, part, partb, s)
        : nci == 2 ? launch_mfma<1, 2>(v, C1, C2, X1, X2, Cout, dY, Yact, ns, part, partb, s)
                   : launch_mfma<1, 1>(v, C1, C2, X1, X2, Cout, dY, Yact, ns, part, partb, s);
  else if (Cout <= 32)
    e = nci >= 2 ? launch_mfma<2, 2>(v, C1, C2, X1, X2, Cout, dY, Yact, ns, part, partb, s)
                 : launch_mfma<2, 1>(v, C1, C2, X1, X2, Cout, dY, Yact, ns, part, partb, s);
  else
    e = launch_mfma<4, 1>(v, C1, C2, X1, X2, Cout, dY, Yact, ns, part, partb, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_reduce_wgrad, dim3((unsigned)((n + Cout + 31) / 32)), dim3(256), 0, s, ns, n, part, dW,
                     db ? Cout : 0, partb, db);
  return hipGetLastError();
}

}  // namespace pdrt
