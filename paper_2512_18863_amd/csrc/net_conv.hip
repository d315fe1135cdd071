// net_conv.hip — forward and data gradient of the network's 3 x 3 x 3 convolutions.
//
// Implicit GEMM on v_mfma_f32_16x16x32_bf16 over a tile of 16 (w) x 8 (h) x TD (d)
// output positions per workgroup of NW wavefronts.  The input tile with its one-voxel
// halo is read from global memory once and kept in LDS, where every position's 27
// neighbours are then read.  A holds 16 output channels, B 16 positions along w, K runs
// over (tap, input channel) in steps of 32, the channel fastest, so a lane's eight K
// entries are eight channels of one neighbour: one 16-byte read.  The data gradient is
// the same product with the taps mirrored, K over (tap, output channel), the ReLU mask
// applied while the tile is staged.
//
// The products are the small part: 16 channels at 128^3 have 14 K steps per tile.  What
// the rest of the design takes out:
//  - vector instructions: the channel count is a template parameter and K unrolled, so a
//    tap is a constant LDS offset.  Where a step's halves fall into two taps (16, 48 or
//    80 channels) the lanes of the second half carry the distance in their address;
//  - weight reads: a fragment's 16 rows lie a row apart, 64 bytes of each, and every
//    wavefront would fetch them again.  They come in chunks of four K steps, a row's
//    256 bytes at a time, through LDS, the next chunk under way during this one's products;
//  - LDS bank conflicts (half of the LDS cycles with positions as padded rows): planes of
//    eight channels, see tile_plane;
//  - narrow stores: channels as the rows of the result leave four consecutive channels of
//    a position in a lane, one 8-byte store instead of four of 2 bytes.
// All forward and data-gradient calls of the network at 128^3: 2.31 -> 0.89 ms (with K
// unrolled alone 1.21).  16 -> 16 channels forward 0.121 -> 0.05 ms (0.03 to move its
// 134 MB), 48 -> 16 0.434 -> 0.138 (0.05 for 268 MB), 96 -> 32 at 64^3 0.217 -> 0.060.
// It is now bound by staging and products taking turns in the two or three
// workgroups that a compute unit holds.
#include "conv_common.hpp"
#include "pdrt_internal.hpp"

namespace pdrt {

typedef float nf32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 nbf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 nbf16x8 __attribute__((ext_vector_type(8)));
typedef short ni16x8 __attribute__((ext_vector_type(8)));

constexpr int CT_W = 16, CT_H = 8;                  // output tile (w, h)
constexpr int CT_HW = CT_W + 2, CT_HH = CT_H + 2;   // with halo

struct ConvIO {
  const __bf16* a1;      // input, channels [0, c1)
  const __bf16* a2;      // input, channels [c1, c1 + c2) (may be null when c2 == 0)
  int c1, c2;
  const __bf16* mask;    // optional (c2 == 0): a1 counts only where mask > 0
  const __bf16* w;       // weights [N][Kp], K = 27 (c1 + c2) padded to a multiple of 32
  const float* bias;     // optional
  int relu;
  __bf16* o1;            // output channels [0, n1)
  __bf16* o2;            // output channels [n1, N)
  int n1;
  int wide;              // o1 and o2 are 8-byte aligned
};

// Offset of a tap's position in the staged tile, from the tile's first corner.
template <bool MIR>
__host__ __device__ constexpr int tap_pos(int tap) {
  const int t = MIR ? 26 - tap : tap;
  return ((t / 9) * CT_HH + (t / 3) % 3) * CT_HW + t % 3;
}

// The staged tile in LDS (elements): planes of eight channels, [position][8], a multiple
// of 256 bytes apart.  A wavefront reads 16 neighbouring positions of two planes for
// each half of a K step: whichever lanes the LDS serves together, they meet every bank once.
// Pairs of planes are shifted against each other, for the writes that stage a position's
// channels side by side.
constexpr int tile_plane(int TD) { return (CT_HW * CT_HH * (TD + 2) + 15) / 16 * 16 * 8; }
constexpr int tile_pair(int C, int TD) { return 2 * tile_plane(TD) + (C > 16 ? 16 / (C / 8) * 8 : 0); }

// x where m > 0, else 0 (BF16: the sign, zero and NaN told from the bits).
__device__ __forceinline__ nbf16x8 relu_mask(nbf16x8 x, nbf16x8 m) {
  const ni16x8 zero = ni16x8{}, inf = zero + (short)0x7f80;
  const ni16x8 p = __builtin_elementwise_max(__builtin_bit_cast(ni16x8, m), zero);
  const ni16x8 keep = ((zero - p) >> 15) & ~((inf - p) >> 15);  // all ones where 0 < m <= inf
  return __builtin_bit_cast(nbf16x8, (ni16x8)(__builtin_bit_cast(ni16x8, x) & keep));
}

template <int C, int NT, bool MIR, int TD, int NW>
__global__ void __launch_bounds__(64 * NW) k_conv3d(Vol v, ConvIO io) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  constexpr int N = NT * 16, CG = C / 8, PL = tile_plane(TD), PAIR = tile_pair(C, TD), KP = (27 * C + 31) / 32 * 32, NS = KP / 32;
  constexpr int POS = CT_HW * CT_HH * (TD + 2), TOT = POS * CG, R = CT_H * TD / NW;  // R rows per wavefront
  constexpr int U = 3;                      // loads of a thread in flight while staging
  constexpr int Q = 4;                      // K steps per weight chunk: 256 bytes of a weight row
  constexpr int WP = (N * 4 * Q + 64 * NW - 1) / (64 * NW);  // 16-byte pieces of a chunk per thread
  __bf16* tin = reinterpret_cast<__bf16*>(smem_raw);   // planes of eight channels, [POS][8]
  __bf16* tw = tin + CG / 2 * PAIR;                    // [2][Q][NT][64][8] weight chunks
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tiles_w = (v.W + CT_W - 1) / CT_W, tiles_h = (v.H + CT_H - 1) / CT_H;
  // workgroups are dealt round-robin to the eight XCDs: each takes a run of neighbouring
  // tiles, whose halos then meet in its L2
  const int nt8 = gridDim.x >> 3, bid = blockIdx.x;
  const int tile = bid < 8 * nt8 ? (bid & 7) * nt8 + (bid >> 3) : bid;
  const int w0 = (tile % tiles_w) * CT_W;
  const int h0 = ((tile / tiles_w) % tiles_h) * CT_H;
  const int d0 = (tile / (tiles_w * tiles_h)) * TD;
  const int m = lane & 15, kq = lane >> 4;

  // A chunk of the weights: read a row's 256 bytes by 16 neighbouring lanes, kept as the
  // lanes of the matrix instruction take it; the slot of a row is folded with the piece's
  // place in the row, so that neither the writes nor the reads meet in a bank.
  nbf16x8 wp[WP];
  auto fetch_w = [&](int c) {
#pragma unroll
    for (int j = 0; j < WP; ++j) {
      const int i = tid + 64 * NW * j, n = i / (4 * Q), k = 32 * Q * c + 8 * (i % (4 * Q));
      if (WP * 64 * NW == N * 4 * Q || n < N)
        wp[j] = *reinterpret_cast<const nbf16x8*>(io.w + n * KP + (k < KP ? k : KP - 8));
    }
  };
  auto store_w = [&](int c) {
#pragma unroll
    for (int j = 0; j < WP; ++j) {
      const int i = tid + 64 * NW * j, n = i / (4 * Q), kp = i % (4 * Q);
      __bf16* to = tw + ((((c & 1) * Q + kp / 4) * NT + n / 16) * 64 + (kp & 3) * 16 + ((n & 15) ^ kp)) * 8;
      if (WP * 64 * NW == N * 4 * Q || n < N) *reinterpret_cast<nbf16x8*>(to) = wp[j];
    }
  };
  fetch_w(0);

  // stage the input tile with halo (zero outside the volume), 8 channels per load
  for (int i0 = 0; i0 < TOT; i0 += 64 * NW * U) {
    nbf16x8 x[U], mk[U];
    bool in[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int idx = i0 + 64 * NW * u + tid, pos = idx / CG, c = 8 * (idx - pos * CG);
      const int pw = pos % CT_HW, pr = pos / CT_HW, ph = pr % CT_HH, pd = pr / CT_HH;
      const int ww = w0 - 1 + pw, hh = h0 - 1 + ph, dd = d0 - 1 + pd;
      in[u] = idx < TOT && (unsigned)ww < (unsigned)v.W && (unsigned)hh < (unsigned)v.H && (unsigned)dd < (unsigned)v.D;
      const size_t q = in[u] ? (size_t)((dd * v.H + hh) * v.W + ww) : 0;
      const __bf16* p = c < io.c1 ? io.a1 + q * io.c1 + c : io.a2 + q * io.c2 + (c - io.c1);
      x[u] = *reinterpret_cast<const nbf16x8*>(p);
      if (MIR && io.mask) mk[u] = *reinterpret_cast<const nbf16x8*>(io.mask + q * io.c1 + c);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int idx = i0 + 64 * NW * u + tid, pos = idx / CG, g = idx - pos * CG;
      nbf16x8 y = in[u] ? x[u] : nbf16x8{};
      if (MIR && io.mask) y = relu_mask(y, mk[u]);
      if (idx < TOT) *reinterpret_cast<nbf16x8*>(tin + (g >> 1) * PAIR + (g & 1) * PL + 8 * pos) = y;
    }
  }

  // this wavefront's R position rows, consecutive along h: (h, d) of row r is (hr + r, dz)
  const int hr = (R * wave) % CT_H, dz = (R * wave) / CT_H;
  const int a0 = 8 * ((dz * CT_HH + hr) * CT_HW + m) + (kq & 1) * PL;
  // the lanes of a step's second half: the next 16 channels, or the first of the next
  // tap, which lies along w, h or d
  const int up = kq >= 2 ? 1 : 0, hop = up * (C / 16 - 1) * PAIR, dir = MIR ? -8 : 8;
  const int ac = a0 + up * PAIR;
  const int aw = a0 - hop + up * dir;
  const int ah = a0 - hop + up * dir * (CT_HW - 2);
  const int ad = a0 - hop + up * dir * ((CT_HH - 2) * CT_HW - 2);
  nf32x4 acc[R][NT];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[r][t] = nf32x4{0.f, 0.f, 0.f, 0.f};
  nbf16x8 a[2][R];
  auto load_a = [&](int st, nbf16x8 (&x)[R]) {
    const int k0 = 32 * st, tl = k0 / C, tu = (k0 + 16) / C;
    const int base = (tu > 26 ? a0 : tl == tu ? ac : tu % 3 ? aw : tu % 9 ? ah : ad) + 8 * tap_pos<MIR>(tl) +
                     k0 % C / 16 * PAIR;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      x[r] = *reinterpret_cast<const nbf16x8*>(tin + base + 8 * r * CT_HW);
      if (tu > 26) x[r] = kq < 2 ? x[r] : nbf16x8{};  // K padding past the 27 taps reads as zero
    }
  };
  nbf16x8 b[2][NT];
  int slot[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) slot[q] = (kq * 16 + (m ^ (4 * q + kq))) * 8;
  auto load_b = [&](int st, nbf16x8 (&x)[NT]) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
      x[t] = *reinterpret_cast<const nbf16x8*>(tw + (st % (2 * Q) * NT + t) * 512 + slot[st % Q]);
  };
  store_w(0);
  __syncthreads();  // the tile and the first chunk are staged
  load_a(0, a[0]);
  load_b(0, b[0]);
#pragma unroll
  for (int st = 0; st < NS; ++st) {
    // the next chunk's weights are under way while this chunk's products run
    if (st % Q == 0 && st + Q < NS) fetch_w(st / Q + 1);
    if ((st + 1) % Q == 0 && st + 1 < NS) {
      store_w((st + 1) / Q);  // (its buffer's last reads were waited for at the barrier before)
      lds_barrier();
    }
    if (st + 1 < NS) {  // the next step's operands, under way while this step's products run
      load_a(st + 1, a[(st + 1) & 1]);
      load_b(st + 1, b[(st + 1) & 1]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int t = 0; t < NT; ++t)
        acc[r][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[st & 1][t], a[st & 1][r], acc[r][t], 0, 0, 0);
  }
  // write: lane m holds position w0 + m, channels 4 kq .. 4 kq + 3 of each 16
  const int ww = w0 + m, dd = d0 + dz;
  if (ww >= v.W || dd >= v.D) return;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int co = 16 * t + 4 * kq;
    nf32x4 bb = nf32x4{0.f, 0.f, 0.f, 0.f};
    if (io.bias)
#pragma unroll
      for (int e = 0; e < 4; ++e) bb[e] = io.bias[co + e];
    const bool first = co < io.n1;  // (n1 is a multiple of 8)
    __bf16* out = first ? io.o1 + co : io.o2 + (co - io.n1);
    const int pitch = first ? io.n1 : N - io.n1;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int hh = h0 + hr + r;
      if (hh >= v.H) break;
      nbf16x4 y;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float s = acc[r][t][e] + bb[e];
        if (io.relu) s = s > 0.f ? s : 0.f;
        y[e] = (__bf16)s;
      }
      __bf16* o = out + (size_t)((dd * v.H + hh) * v.W + ww) * pitch;
      if (io.wide) {
        *reinterpret_cast<nbf16x4*>(o) = y;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = y[e];
      }
    }
  }
}

constexpr size_t conv3d_lds(int C, int NT, int TD) {
  return (size_t)2 * (C / 16) * tile_pair(C, TD) + 8192 * NT;
}

template <int C, int NT, bool MIR>
static hipError_t launch_shape(Vol v, const ConvIO& io, hipStream_t s) {
  // Tile depth and wavefronts, ms per call at 128^3 (level 0) and 64^3, (depth,
  // wavefronts) = (4, 4) / (2, 4) / (4, 8) / (2, 8):
  //   16 -> 16 forward      0.046 / 0.048 / 0.047 / 0.051   one weight fragment a step: rows of positions reuse it
  //   16 -> 32 (64^3)       0.0154 / 0.0165 / 0.0135 / 0.0155
  //   48 -> 16 forward      0.213 / 0.155 / 0.152 / 0.138   the deep tile leaves one workgroup per compute unit
  //   16 -> 48 gradient     0.188 / 0.140 / 0.154 / 0.139
  //   32 -> 32 (64^3)       0.0268 / 0.0219 / 0.0227 / 0.0203
  //   96 -> 32 (64^3)       - / 0.076 / - / 0.060           and hides its staging by the number of wavefronts
  constexpr int NW = C == 16 && NT == 1 ? 4 : 8;
  constexpr int want = C == 16 && NT <= 2 ? 4 : 2;
  constexpr int TD = conv3d_lds(C, NT, want) <= 160 * 1024 ? want : 1;
  constexpr size_t lds = conv3d_lds(C, NT, TD);
  static_assert(lds <= 160 * 1024, "the staged tile and two weight chunks fit LDS");
  if (lds > 64 * 1024) {
    hipError_t e = ensure_lds_limit((const void*)k_conv3d<C, NT, MIR, TD, NW>, 160 * 1024);
    if (e != hipSuccess) return e;
  }
  const unsigned tiles = (unsigned)(((v.W + CT_W - 1) / CT_W) * ((v.H + CT_H - 1) / CT_H) * ((v.D + TD - 1) / TD));
  hipLaunchKernelGGL((k_conv3d<C, NT, MIR, TD, NW>), dim3(tiles), dim3(64 * NW), lds, s, v, io);
  return hipGetLastError();
}

template <int C, bool MIR>
static hipError_t launch_nt(Vol v, const ConvIO& io, int n, hipStream_t s) {
  switch (n / 16) {
    case 1: return launch_shape<C, 1, MIR>(v, io, s);
    case 2: return launch_shape<C, 2, MIR>(v, io, s);
    case 4: return launch_shape<C, 4, MIR>(v, io, s);
    default: break;
  }
  if constexpr (MIR) {
    if (n == 48) return launch_shape<C, 3, MIR>(v, io, s);
    if (n == 96) return launch_shape<C, 6, MIR>(v, io, s);
  }
  return hipErrorInvalidValue;
}

static int wide_ok(const __bf16* o1, const __bf16* o2) { return (((uintptr_t)o1 | (uintptr_t)o2) & 7) == 0; }

hipError_t launch_conv3d_fwd(Vol v, int C1, int C2, const __bf16* X1, const __bf16* X2, int Cout,
                             const __bf16* Wt, const float* bias, int relu, __bf16* Y, hipStream_t s) {
  ConvIO io{X1, X2, C1, C2, nullptr, Wt, bias, relu, Y, nullptr, Cout, wide_ok(Y, nullptr)};
  switch (C1 + C2) {
    case 16: return launch_nt<16, false>(v, io, Cout, s);
    case 32: return launch_nt<32, false>(v, io, Cout, s);
    case 48: return launch_nt<48, false>(v, io, Cout, s);
    case 64: return launch_nt<64, false>(v, io, Cout, s);
    case 80: return launch_nt<80, false>(v, io, Cout, s);
    case 96: return launch_nt<96, false>(v, io, Cout, s);
    default: return hipErrorInvalidConfiguration;
  }
}

hipError_t launch_conv3d_dgrad(Vol v, int Cout, const __bf16* dY, const __bf16* Yact, int Cin, const __bf16* Wd,
                               int C1, __bf16* dX1, __bf16* dX2, hipStream_t s) {
  ConvIO io{dY, nullptr, Cout, 0, Yact, Wd, nullptr, 0, dX1, dX2, C1, wide_ok(dX1, dX2)};
  switch (Cout) {
    case 16: return launch_nt<16, true>(v, io, Cin, s);
    case 32: return launch_nt<32, true>(v, io, Cin, s);
    case 48: return launch_nt<48, true>(v, io, Cin, s);
    case 64: return launch_nt<64, true>(v, io, Cin, s);
    default: return hipErrorInvalidConfiguration;
  }
}

}  // namespace pdrt
