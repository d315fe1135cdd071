// conv_fwd_reg.hip — the forward per-plane lateral convolution (arXiv:2512.18863
// §2.2.6, Eq. 8) on the CDNA4 matrix cores, in FP32 or with BF16 operands (FP32
// sums), for an input that vanishes outside the aperture rectangle (the primary
// P = F G).
//
// out[i][j] = sum_{p,q} K[p][q] in[i+p][j+q], with in zero outside the box
// [r0, r1) x [c0, c1).  Split by tap row p and by box row r:
//   Y_p[r][j] = sum_c K[p][c - j] in[r][c],   out[r - p][j] += Y_p[r][j],
// and since K[-p][.] = K[p][.] the same product also gives out[r + p][j] += Y_p[r][j].
// The input is small (the box) and the output large (the box and the kernel's
// reach around it), so the box stays in registers for the whole plane and only
// the Toeplitz band of tap row p is read from LDS.  v_mfma_f32_16x16x32_bf16 with
// M = 16 output columns j, N = 16 box rows r and K = 32 box columns c (a group):
//   A[m][k] = K[p][c_k - j_m] (from the extended tap row),
//   B[k][n] = in[r_n][c_k] (registers, loaded once per plane).
//
// FP32 operands are split exactly into three BF16 pieces, x = x0 + x1 + x2 (each the
// rounded remainder of the ones before: 8 significant bits and a sign each, 24 in
// all), and a product takes the six piece products down to x0 y2, x2 y0 and x1 y1,
// smallest first, every product exact, the sums in FP32.  Of the three left out, x1 y2
// and x2 y1 are up to 2^-25 of the product each and x2 y2 2^-34: 2^-24 together at most,
// the rounding of one FP32 product, and 2^-27.5 in the root mean square.  Six BF16
// instructions of K = 32 take 96 cycles where the eight FP32 instructions of K = 4 take
// 256, and fewer roundings enter a sum (an instruction rounds four times).  Error of the
// convolution's output against FP64, root mean square over that of the output, FP32
// instructions -> six products: 128^3 plan 1.51e-7 -> 1.40e-7, with fluence corrections
// and collimator rotation 5.2e-6 -> 3.0e-7.  (The dose, which rounds in other steps too:
// 1.41e-7 -> 1.50e-7 on the plan.)  The third piece of a number below about 2^-109 is
// subnormal and lost: such operands keep 16 bits or fewer (a loss scaled by 1e-36 has its
// gradients within 2.8e-6 in place of 3.4e-7).  A non-finite input makes outputs
// non-finite as far as its column group is multiplied: the strips that the group reaches,
// and for the first group of a box of one chunk every strip.
//
// The product's box rows lie along the lanes of each 16-lane row of the result, so
// moving it by p rows is a DPP row shift within those 16 lanes: the part that stays
// in a 16-row output block is one shift, the part that crosses into the neighbouring
// block the complementary one; lanes shifted in from outside the row read zero.
// Each wavefront owns one 16-column strip of the output and keeps its rows (the
// box rows and two blocks above and below, for h <= 31) in registers over all tap
// rows, then stores them; the rest of the plane (outside the strips) is written
// with zeros.  A box of more rows than one chunk holds is walked chunk by chunk down
// the strip (CARRY): the chunk's rows are stored, and the four blocks that the next one
// adds to stay in the registers.  Column chunks are loaded only where the strip is in
// their reach.  (Where jaws inside the field limits give one row chunk, registers are
// not kept for more: a box beyond the limits adds its chunks' strips into a cleared plane
// with atomic adds, each address by its own wavefront only, in chunk order.)  20 control
// points of 75 planes, 121 x 121 boxes, n = 13: 0.15 ms (0.88 with every chunk loaded for
// every strip and atomic adds).
//
// One small workgroup per (control point, plane) item: its wavefronts take the strips
// in turn, and the many workgroups of a compute unit overlap each other's taps, loads
// and stores.  (Eight wavefronts per workgroup, or persistent workgroups with a second
// buffer of taps and a barrier per plane, were slower: 1.23 to 1.37 against 1.07 ms on
// the 128^3 plan, 4.3 against 3.4 ms on the 224 x 224 x 105 one.)
//
// Work skipped: column groups of which no column lies within h of the strip (one
// uniform branch per group and tap row; inside a group the band's zero taps are
// multiplied).  The products of skipped groups are exact zeros.  The sum of every
// output runs over p = 0, 1, ..., h in order, within a tap row over the box's row
// blocks, and within a product over the box columns (deterministic).
//
// What bounds it: the vector instructions of the row shifts (16 per product) beside
// the matrix instructions (the two overlap: 16 cycles of matrix unit and about 7 of
// issue per product).  180 control points at 128^3 (n = 61, 27 x 27 boxes, 32940
// planes): FP32 0.94 to 1.02 ms by clock (1.91 on FP32 matrix instructions), BF16 0.53 ms
// (0.65); 224 x 224 x 105 (n = 55, 41 x 41): 3.2 ms (6.3); 90 control points with fluence
// corrections and collimator rotation (n = 61, up to 99 x 99): 4.9 ms (24.9; 6.1 with every
// column group loaded for every strip and strips added by atomics).
#include "conv_common.hpp"

namespace pdrt {

typedef float f32x4r __attribute__((ext_vector_type(4)));
typedef unsigned u32x4r __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8r __attribute__((ext_vector_type(8)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));  // four floats at any word address

constexpr int kRegQB = 2;    // output blocks of 16 rows above and below a row chunk
constexpr int kRegGW = 32;   // columns per group (one uniform branch each)
static_assert(16 * (kRegQB - 1) + 15 == kRegMaxH, "the blocks reach the largest half-width");

// Lane i takes lane i + S (LEFT) or i - S of its 16-lane row; 0 where that lane lies
// outside the row.  1 <= S <= 15.  (Each component is copied to a scalar before its
// bits are reinterpreted: this compiler turns __builtin_bit_cast of a vector element
// v[e] into a cast of v[0].)
template <int S, bool LEFT>
__device__ __forceinline__ f32x4r row_shift(const f32x4r& v) {
  constexpr int ctrl = LEFT ? 0x100 + S : 0x110 + S;  // row_shl:S / row_shr:S
  f32x4r r;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float x = v[e];
    r[e] = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), ctrl, 0xf, 0xf, false));
  }
  return r;
}

// Tap row P's products Y[t] of the box's row blocks t, added to the strip's output
// blocks O p rows up and down (block kRegQB + t holds the rows of box block t).
template <int P, int T, int NB>
__device__ __forceinline__ void reg_add_shifted(const f32x4r (&Y)[T], f32x4r (&O)[NB]) {
  constexpr int S = P & 15, Q = P >> 4, c = kRegQB;
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const f32x4r y = Y[t];
    if constexpr (P == 0) {
      O[c + t] += y;
    } else if constexpr (S == 0) {
      O[c + t - Q] += y;  // rows r - P
      O[c + t + Q] += y;  // rows r + P
    } else {
      // rows r - P: box lanes n >= S land in block t - Q at lane n - S, the others in
      // block t - Q - 1 at lane n - S + 16
      O[c + t - Q] += row_shift<S, true>(y);
      O[c + t - Q - 1] += row_shift<16 - S, false>(y);
      // rows r + P: lanes n + S < 16 land in block t + Q at lane n + S, the others in
      // block t + Q + 1 at lane n + S - 16
      O[c + t + Q] += row_shift<S, false>(y);
      O[c + t + Q + 1] += row_shift<16 - S, true>(y);
    }
  }
}

// NP pieces per operand (1: BF16, 3: FP32); aaddr[u] is the lane's run of group u in
// the first piece of row 0.
template <int NP, int T, int SU>
struct RegOps {
  typedef u32x4r AOp[NP][SU];
  typedef u32x4r BOp[NP][T][SU];
  template <int P>
  static __device__ __forceinline__ void load_row(const unsigned* const (&aaddr)[SU], AOp& A) {
#pragma unroll
    for (int u = 0; u < SU; ++u) {
      const unsigned* a = aaddr[u] + P * NP * kRegW;
#pragma unroll
      for (int i = 0; i < NP; ++i)
        A[i][u] = u32x4r{a[i * kRegW], a[i * kRegW + 1], a[i * kRegW + 2], a[i * kRegW + 3]};
    }
  }
  // Y[t] = sum over the groups of A B[t]
  static __device__ __forceinline__ void multiply(const AOp& A, unsigned umask, const BOp& B, f32x4r (&Y)[T]) {
    // (piece of A, piece of B), smallest products first
    constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
    constexpr int i0 = NP == 3 ? 0 : 5;
    auto mul = [&](int i, int u, int t, const f32x4r& c) {
      return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8r, A[pa[i]][u]),
                                                     __builtin_bit_cast(bf16x8r, B[pb[i]][t][u]), c, 0, 0, 0);
    };
    // group 0 always runs and starts the chains from zero (out of reach its A is
    // zero); the others run when their bit of umask is set and accumulate in place
#pragma unroll
    for (int i = i0; i < 6; ++i)
#pragma unroll
      for (int t = 0; t < T; ++t) Y[t] = mul(i, 0, t, i == i0 ? f32x4r{0.f, 0.f, 0.f, 0.f} : Y[t]);
#pragma unroll
    for (int u = 1; u < SU; ++u)
      if (umask & (1u << u)) {
#pragma unroll
        for (int i = i0; i < 6; ++i)
#pragma unroll
          for (int t = 0; t < T; ++t) Y[t] = mul(i, u, t, Y[t]);
      }
  }
};

// The next tap row's operand is read while a row's products run where registers allow
// it at the same occupancy (128^3 plan, T = 2: 1.07 ms with, 1.09 without and five
// wavefronts per SIMD; T = 3: 3.7 ms with, 3.4 without and three).
__host__ __device__ constexpr bool reg_read_ahead(int T) { return T <= 2; }

// Tap rows P, P + 1, ..., h; A holds row P's operand when reading ahead.
template <int NP, int P, int T, int SU, int NB>
__device__ __forceinline__ void reg_tap_rows(int h, const unsigned* const (&aaddr)[SU], unsigned umask,
                                             const typename RegOps<NP, T, SU>::AOp& A,
                                             const typename RegOps<NP, T, SU>::BOp& B, f32x4r (&O)[NB]) {
  typedef RegOps<NP, T, SU> Ops;
  if constexpr (P <= kRegMaxH) {
    if (P > h) return;
    typename Ops::AOp next;
    f32x4r Y[T];
    if constexpr (reg_read_ahead(T)) {
      Ops::template load_row<P + 1>(aaddr, next);  // (past the last row: the spare one, not used)
      Ops::multiply(A, umask, B, Y);
    } else {
      Ops::template load_row<P>(aaddr, next);
      Ops::multiply(next, umask, B, Y);
    }
    reg_add_shifted<P, T, NB>(Y, O);
    reg_tap_rows<NP, P + 1, T, SU, NB>(h, aaddr, umask, next, B, O);
  }
}

// Wavefronts per SIMD the registers are kept for.
__host__ __device__ constexpr int reg_waves(int np, int T) {
  return np == 3 ? (T == 1 ? 6 : T == 2 ? 5 : T == 3 ? 3 : 2) : (T <= 2 ? 7 : T == 3 ? 4 : T == 4 ? 3 : 2);
}

// T: row blocks of 16 box rows per chunk; SU: column groups per chunk (boxes larger
// than a chunk are taken chunk by chunk); CARRY: several row chunks expected.  LDS: the
// tap rows.
template <int NP, int T, int SU, bool CARRY>
__global__ void __launch_bounds__(512, reg_waves(NP, T)) k_conv_fwd_reg(Geo<float> g, const int4* __restrict__ box,
                                                                        const float* __restrict__ zca,
                                                                        const float* __restrict__ in,
                                                                        float* __restrict__ out) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  typedef RegOps<NP, T, SU> Ops;
  constexpr int GW = kRegGW;
  constexpr int NB = T + 2 * kRegQB;
  const int h = g.h, h1 = h + 1;
  const int CS = h1 * NP * kRegW;  // words from the first copy of the rows to the second
  unsigned* lds = reinterpret_cast<unsigned*>(smem_raw);
  const int NT = blockDim.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = NT >> 6;
  const int bk = blockIdx.x;
  const int b = bk / g.Nk, k = bk - b * g.Nk;
  const int Nu = g.Nu, Nv = g.Nv;
  const size_t plane = (size_t)Nu * Nv;
  float* dst = out + (size_t)bk * plane;
  const float* src = in + (size_t)bk * plane;
  const int n = lane & 15, kk = lane >> 4;
  const int4 bx = box[b];
  const int r0 = max(bx.x, 0), r1 = min(bx.y, Nu), c0 = max(bx.z, 0), c1 = min(bx.w, Nv);
  if (r1 <= r0 || c1 <= c0) {
    for (size_t i = tid; i < plane; i += NT) dst[i] = 0.f;
    return;
  }
  const int cw0 = max(0, c0 - h), cw1 = min(Nv, c1 + h);  // columns in reach
  const int njt = (cw1 - cw0 + 15) / 16;
  const int nrc = (r1 - r0 + 16 * T - 1) / (16 * T), ncc = (c1 - c0 + GW * SU - 1) / (GW * SU);

  // B fragments of a box chunk whose first row and column are R and C: lane (n, kk) holds
  // in[R + 16 t + n][C + 32 u + 8 kk .. + 7] as pairs of each piece.  Each run of four
  // columns is one four-word load from a row inside the box (rows past it and runs past
  // its last column read the box's first row or column and are cleared); a run that
  // starts inside the box may read up to three words past its last column, i.e. past the
  // end of the row into the next one (or, after the batch's last row, into the workspace
  // that follows the convolution's input).
  typename Ops::BOp B;
  auto run4 = [&](int r, int c) {
    const f32x4u x = *reinterpret_cast<const f32x4u*>(src + (size_t)(r < r1 ? r : r0) * Nv + (c < c1 ? c : c0));
    f32x4r v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = (r < r1 && c + e < c1) ? x[e] : 0.f;
    return v;
  };
  auto load_b = [&](int R, int C, int t, int u) {
    const int r = R + 16 * t + n, c = C + GW * u + 8 * kk;
    const f32x4r x[2] = {run4(r, c), run4(r, c + 4)};
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      unsigned v[NP];
      reg_pieces2<NP>(x[w / 2][2 * (w & 1)], x[w / 2][2 * (w & 1) + 1], v);
#pragma unroll
      for (int i = 0; i < NP; ++i) B[i][t][u][w] = v[i];
    }
  };
  const bool single = nrc == 1 && ncc == 1;
  if (single && wave < njt) {  // in flight while the taps are built
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int u = 0; u < SU; ++u) load_b(r0, c0, t, u);
  }

  clear_tap_rows(lds, h, NP, tid, NT);
  lds_barrier();
  build_tap_rows<NP>(g, k, zca[bk], lds, tid, NT, 1.f);
  // zeros outside the strips' window [wr0, wr1) x [cw0, cw0 + 16 njt); where strips are
  // added, in the whole plane (the barrier below orders them)
  const bool store = CARRY || nrc == 1;
  const int wr0 = store ? r0 - 16 * kRegQB : 0, wr1 = store ? r0 + 16 * (T * nrc + kRegQB) : 0;
  {
    // whole rows above and below the window (two contiguous ranges), then the
    // columns left and right of it in the rows between
    const int zr0 = min(max(wr0, 0), Nu), zr1 = min(max(wr1, zr0), Nu);
    const int cz1 = min(Nv, cw0 + 16 * njt);
    const int top = zr0 * Nv, nfull = top + (Nu - zr1) * Nv;
    for (int d = tid; d < nfull; d += NT) dst[d < top ? d : zr1 * Nv + (d - top)] = 0.f;
    const int side = cw0 + (Nv - cz1), nside = (zr1 - zr0) * side;
    for (int d = tid; d < nside; d += NT) {
      const int rr = d / side, cc = d - rr * side;
      dst[(size_t)(zr0 + rr) * Nv + (cc < cw0 ? cc : cz1 + (cc - cw0))] = 0.f;
    }
  }
  if (store) lds_barrier();
  else __syncthreads();

  for (int jt = wave; jt < njt; jt += nw) {
    const int J = cw0 + 16 * jt;  // the strip's first output column
    f32x4r O[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) O[q] = f32x4r{0.f, 0.f, 0.f, 0.f};
    for (int rc = 0; rc < nrc; ++rc) {
      const int R = r0 + 16 * T * rc;
      if constexpr (!CARRY) {
#pragma unroll
        for (int q = 0; q < NB; ++q) O[q] = f32x4r{0.f, 0.f, 0.f, 0.f};
      }
      for (int cc = 0; cc < ncc; ++cc) {
        const int C = c0 + GW * SU * cc;
        const int nsu = min(SU, (c1 - C + GW - 1) / GW);
        // column groups with a column within h of the strip [J, J + 16)
        const int lo = J - h - C - (GW - 1), hi = J + 15 + h - C;
        const int ua = lo <= 0 ? 0 : (lo + GW - 1) / GW;
        const int ub = min(nsu - 1, hi >= 0 ? hi / GW : -1);
        if (ua > ub) continue;
        if (!single) {  // the groups in reach; zeros in the others (group 0 is multiplied always)
#pragma unroll
          for (int u = 0; u < SU; ++u) {
            if (u >= ua && u <= ub) {
#pragma unroll
              for (int t = 0; t < T; ++t) load_b(R, C, t, u);
            } else {
#pragma unroll
              for (int t = 0; t < T; ++t)
#pragma unroll
                for (int i = 0; i < NP; ++i) B[i][t][u] = u32x4r{0u, 0u, 0u, 0u};
            }
          }
        }
        // A of group u in tap row p starts at x = C + 32 u + 8 kk - J - m + kRegOff (m
        // the lane's output column), moved to a run of zeros where it meets no tap
        // (so group 0 runs also out of reach; the others are skipped)
        const unsigned* aaddr[SU];
#pragma unroll
        for (int u = 0; u < SU; ++u) {
          int x = C + GW * u + 8 * kk - J - n + kRegOff;
          const int x0 = kRegOff - h - 9, x1 = kRegOff + h + 1;
          if (x < x0 + 1) x = x0 + ((x ^ x0) & 1);
          if (x > x1) x = x1 + ((x ^ x1) & 1);
          aaddr[u] = lds + ((x & 1) ? CS : 0) + (x >> 1);
        }
        const unsigned umask = __builtin_amdgcn_readfirstlane((2u << ub) - (1u << ua));  // bits ua .. ub
        typename Ops::AOp A;
        if constexpr (reg_read_ahead(T)) Ops::template load_row<0>(aaddr, A);
        reg_tap_rows<NP, 0, T, SU, NB>(h, aaddr, umask, A, B, O);
      }
      // the strip's rows R - 16 kRegQB + 16 q + n and columns J + 4 kk + e that lie in
      // the plane; only this wavefront writes them (CARRY: the four lower blocks stay for the
      // next chunk, which stores them again: a test for the last chunk costs the registers
      // of a second copy)
#pragma unroll
      for (int q = 0; q < NB; ++q) {
        const int row = R - 16 * kRegQB + 16 * q + n;
        if (row >= 0 && row < Nu) {
          float* o = dst + (size_t)row * Nv + J + 4 * kk;
          if (store && J + 4 * kk + 3 < Nv) {
            *reinterpret_cast<f32x4u*>(o) = O[q];  // the lane's four consecutive columns
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float v = O[q][e];
              if (J + 4 * kk + e < Nv) {
                if (store) o[e] = v;
                else unsafeAtomicAdd(o + e, v);
              }
            }
          }
        }
      }
      if constexpr (CARRY) {
#pragma unroll
        for (int q = 0; q < NB; ++q) O[q] = q + T < NB ? O[q + T] : f32x4r{0.f, 0.f, 0.f, 0.f};
      }
    }
  }
}

static size_t reg_lds(int h, bool bf) { return sizeof(unsigned) * (size_t)reg_tap_words(h, bf ? 1 : 3); }

bool conv_fwd_reg_supported(const Geo<float>& g, bool bf16) {
  return g.h >= 1 && g.h <= kRegMaxH && reg_lds(g.h, bf16) <= 160 * 1024;
}

template <int NP, int T, int SU, bool CARRY = false>
static hipError_t launch_reg_cfg(const Geo<float>& g, int nb, const int4* box, const float* z, const float* in,
                                 float* out, hipStream_t s) {
  const size_t lds = reg_lds(g.h, NP == 1);
  const void* kern = (const void*)k_conv_fwd_reg<NP, T, SU, CARRY>;
  {
    hipError_t e = ensure_lds_limit(kern, (int)lds);
    if (e != hipSuccess) return e;
  }
  const long n_items = (long)nb * g.Nk;
  if (n_items > 0x7fffffffL) return hipErrorInvalidConfiguration;
  // few items: eight wavefronts share an item's strips (214 planes: 0.044 against 0.052
  // ms); else two for the short loops of small kernels (90 control points, n = 15: 0.095
  // against 0.117 ms), four for larger ones (180, n = 61: 1.07 against 1.26 ms)
  const int nw = n_items <= 2 * device_cus() ? 8 : g.h <= 16 ? 2 : 4;
  hipLaunchKernelGGL((k_conv_fwd_reg<NP, T, SU, CARRY>), dim3((unsigned)n_items), dim3(64 * nw), lds, s, g, box, z, in,
                     out);
  return hipGetLastError();
}

template <int NP>
static hipError_t launch_reg_np(const Geo<float>& g, int nb, const int4* box, const float* z, const float* in,
                                float* out, hipStream_t s, int ch, int chunks) {
  if (chunks > 1) {
    switch (ch) {
      case 4: return launch_reg_cfg<NP, 4, 2, true>(g, nb, box, z, in, out, s);
      case 5: return launch_reg_cfg<NP, 5, 2, true>(g, nb, box, z, in, out, s);
      default: return launch_reg_cfg<NP, 6, 2, true>(g, nb, box, z, in, out, s);
    }
  }
  switch (ch) {
    case 1: return launch_reg_cfg<NP, 1, 1>(g, nb, box, z, in, out, s);
    case 2: return launch_reg_cfg<NP, 2, 1>(g, nb, box, z, in, out, s);
    case 3: return launch_reg_cfg<NP, 3, 2>(g, nb, box, z, in, out, s);
    case 4: return launch_reg_cfg<NP, 4, 2>(g, nb, box, z, in, out, s);
    case 5: return launch_reg_cfg<NP, 5, 2>(g, nb, box, z, in, out, s);
    default: return launch_reg_cfg<NP, 6, 2>(g, nb, box, z, in, out, s);
  }
}

// The chunk shape from the largest rectangle that jaws inside the field limits give,
// widened by fluence corrections and collimator rotation: one row chunk of up to six
// blocks, else equal chunks; columns beyond two groups come in column chunks, summed in
// registers.  (n = 61, 40 control points of 75 planes, 81 x 81 boxes: 0.68 ms with six
// blocks, 0.72 in two chunks of three, 0.94 of four; all columns at once leave one
// wavefront per SIMD.)
hipError_t launch_conv_fwd_reg(const Geo<float>& g, int nb, const float* z, const float* in, float* out,
                               hipStream_t s, const int* box, bool bf16) {
  if (!conv_fwd_reg_supported(g, bf16) || !box) return hipErrorInvalidConfiguration;
  const int4* bx = reinterpret_cast<const int4*>(box);
  const int half_u = (g.Nu - 1) / 2 - g.h, half_v = (g.Nv - 1) / 2 - g.h;  // field limit in pixels
  const int br = min(g.Nu, 2 * (half_u > 0 ? half_u : 0) + 1 + 2 * g.conv_du);
  const int bc = min(g.Nv, 2 * (half_v > 0 ? half_v : 0) + 1 + 2 * g.conv_dv);
  const int blocks = ((br > bc ? br : bc) + 15) / 16, chunks = (blocks + 5) / 6;
  const int ch = (blocks + chunks - 1) / chunks;
  return bf16 ? launch_reg_np<1>(g, nb, bx, z, in, out, s, ch, chunks)
              : launch_reg_np<3>(g, nb, bx, z, in, out, s, ch, chunks);
}

}  // namespace pdrt
