// Implicit-GEMM forward convolution of fp32 data on bf16 MFMA, without losing
// a bit of either operand: every fp32 value is the exact sum of three bf16
// parts (8 + 8 + 8 significand bits, each the rounded remainder of the last),
// and a product is taken as the six part products that reach above 2^-24 of
// it (hh; hm, mh; hl, mm, lh -- the other three are below 2^-24 together).
// Included by the instantiation files (conv_b3*.hip).
//
// Why: fp32 MFMA has a sixteenth of the bf16 rate on this chip, so six bf16
// MFMAs in place of one fp32 MFMA are 2.67 times as fast at the peaks.  And
// the sums are more exact: the hh products go to an accumulator of their own,
// which rounds once per 32 rows of the reduction where the fp32 MFMA rounds
// every two, and the five small products (2^-8 of hh and less) to a second
// one, added at the end.  Against 64-bit sums, random data, 4608 rows: 3.5e-7
// (fp32 MFMA: 8.7e-7); 64 rows: 4.1e-8 (1.0e-7).
//
// What bounds it: power, then instruction issue.  v_mfma_f32_16x16x32_bf16 is
// used because the 32x32x16 form, which reads and writes twice the
// accumulators per product, ran the chip into its power limit (MFMAs alone on
// random data: 229 against 372 TFLOPS of fp32 products).  Splitting an operand
// takes 6 vector instructions per element, half a one of them for the check of
// lost bits below, so the split is done once per work-group for the filter
// (through LDS) and once per wave for the patches, and is spread between the
// MFMAs.
//
// Range.  bf16 has no bits below 2^-133, so an operand under 2^-110 may have no
// exact parts; and an infinity has no finite remainder.  The split itself tells:
// the third part is the upper half of its fp32 value, and a set bit in the lower
// half is a lost one.  A wave with a finished sum that is not finite, or nonzero
// and under 2^-86 (part products may have fallen below the fp32 range), computes
// its part again on fp32 MFMA, straight from memory.  So does one in whose patches
// a bit was lost.  Where only the filter lost some (weights that training let
// decay), they are worth at most Kg * 2^-133 of the largest patch element, and the
// waves of the largest tiles (eight side by side) look first whether their sums
// are above that (least_safe).  The others stage NaN for a filter column that lost
// bits instead, so that its sums are computed again: the barrier and the code for
// the look take 2% of the smaller tiles' time in every call, and 8% of the
// resident-filter kernel's; of the largest tiles' none to 1%.
// Time, 512 channels at 28x28, N = 64 (1700 us on fp32 MFMA): 925 us; 1150 with a
// lost bit in the filter, 1200 with an infinity in x, 3060 where every sum is
// computed again.  128 -> 512 channels, 1x1 at 28x28, N = 32 (36): 24, 49, 25 and 49.
#pragma once

#include "conv_kernel.h"

namespace mg3m {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// W floats at byte offset voff + soff (voff is what the buffer's bound is
// checked against).
template <int W>
__device__ __forceinline__ void bload_w(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, float (&v)[W]) {
  static_assert(W == 1 || W == 2 || W == 4, "one load");
  if constexpr (W == 4) {
    const f32x4 x = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = x[i];
  } else if constexpr (W == 2) {
    const f32x2 x = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
    v[0] = x[0];
    v[1] = x[1];
  } else {
    v[0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
  }
}
template <int W>
__device__ __forceinline__ void bstore_w(__amdgpu_buffer_rsrc_t r, unsigned voff, unsigned soff, const float (&v)[W]) {
  if constexpr (W == 4)
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, f32x4{v[0], v[1], v[2], v[3]}), r, voff, soff, 0);
  else if constexpr (W == 2)
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, f32x2{v[0], v[1]}), r, voff, soff, 0);
  else
    bstore1(r, voff, soff, v[0]);
}

// Two values in three bf16 parts each, packed in pairs.  What is left for the
// third part has at most eight significant bits: its lower half is zero unless
// it reaches below bf16's last bit, 2^-133.  lost collects these halves.
__device__ __forceinline__ void split2(float a, float b, unsigned (&o)[3], unsigned& lost) {
#pragma unroll
  for (int p = 0; p < 3; ++p) {
    o[p] = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2));
    if (p < 2) {
      a -= __builtin_bit_cast(float, o[p] << 16);
      b -= __builtin_bit_cast(float, o[p] & 0xffff0000u);
    }
  }
  lost |= __builtin_bit_cast(unsigned, a) | __builtin_bit_cast(unsigned, b);
}
__device__ __forceinline__ bool lost_bits(unsigned lost) { return (unsigned short)lost != 0; }

// The largest of a wave's values, in every lane.
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v = fmaxf(v, __shfl_xor(v, d));
  return v;
}
// The smallest sum of Kg products that lost bits of the filter reach by no more
// than 2^-25 of it, with patch elements of at most `largest`.
__device__ __forceinline__ float least_safe(float largest, int Kg) { return largest * ((float)Kg * 0x1p-108f); }

// Formed here, not sunk to the block of their use (the next stage).
__device__ __forceinline__ void pin3(unsigned (&o)[3], unsigned& lost) {
  asm volatile("" : "+v"(o[0]), "+v"(o[1]), "+v"(o[2]), "+v"(lost));
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>): the
// indices are constants in f, so register arrays stay in registers.
template <class F, int... I>
__device__ __forceinline__ void static_for_seq(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_seq(f, std::make_integer_sequence<int, N>{});
}

// Geometry.  The WN waves stand side by side along the columns, each with all
// MT rows and WTN columns, as 16x16 blocks; KT is a multiple of 32, the depth
// of one MFMA (KS of them per stage).
template <int MT, int NT, int KT, int WN>
struct B3Cfg {
  static constexpr int T = WN * 64;
  static constexpr int WTN = NT / WN;
  static constexpr int TM = MT / 16, TN = WTN / 16, KS = KT / 32;
  // A thread stages AR consecutive rows of one filter column, UA times.
  static constexpr int A_ROWS = KT * MT / T;
  static constexpr int AR = A_ROWS < 8 ? A_ROWS : 8;
  static constexpr int UA = A_ROWS / AR;
  static_assert(KT % 32 == 0 && KT * MT % T == 0 && T % MT == 0 && (AR == 2 || AR == 4 || AR == 8) &&
                A_ROWS % AR == 0, "filter stage split");
  static_assert(TN == 1 || TN == 2 || TN == 4, "columns per lane");
  // A stage in LDS: for each part, 16-byte chunks of eight consecutive rows of
  // one filter column, [KT / 8][MT].
  static constexpr int PLANE = KT / 8 * MT;
  static constexpr int STAGE = 3 * PLANE;
  static constexpr int LDS_CHUNKS = 2 * STAGE;
  static_assert(LDS_CHUNKS * 16 == lds_bytes_for_b3(TileDesc{MT, NT, KT, 1, WN, 0, 0.0}), "LDS size model");
};

// How the operands are addressed (kernel variants; plan.cpp chooses).
//  kB3Slab   C % KT == 0: a stage is one filter tap over KT channels (taps
//            inside channel slabs, as the fp32 one-tap kernels), its tap in
//            scalar registers; HWCN, N % 4 == 0: a lane's TN columns are one load.
//  kB3SlabW  the same stages in NCHW on the [R][S][C][K] filter copy: 16 lanes
//            along the output pixels, a load per column.
//  kB3Group  C % 8 == 0: the reduction runs tap by tap over groups of eight
//            channels, four groups to a k-step, so each lane group has a tap and
//            channels of its own.  HWCN, N % 4 == 0, columns as kB3Slab.
//  kB3GroupN the same for any N: a load per column.
//  kB3GroupC the same for N == 1: a group's channels are contiguous, two 16-byte
//            loads per column.
//  kB3Row    any C: the reduction runs tap by tap over single channels, each row
//            of the stage with a tap and channel of its own, stepped one row
//            after another as they are loaded.  HWCN, N % 4 == 0, columns as
//            kB3Slab.
//  kB3RowN   the same for any N: a load per column.
// (enum B3Load, mg3m_internal.h)
constexpr bool b3_vec(int ld) { return ld == kB3Slab || ld == kB3Group || ld == kB3Row; }   // a lane's columns are consecutive
constexpr bool b3_rows(int ld) { return ld >= kB3Row; }

// Position of a lane (or thread) in the reduction of the group and row
// variants: tap (r, s) and channel group (row variants: channel) g of the G
// per tap; moved by `step` at a time, given in the mixed radix of (R, S, G).
struct GroupStep {
  int dr, ds, dg, G;
  __device__ void init(const KArgs& a, int G_, int step) {
    G = G_;
    ds = step / G;
    dg = step - ds * G;
    dr = ds / a.S;
    ds -= dr * a.S;
  }
};
struct GroupPos {
  int r, s, g;
  __device__ void init(const KArgs& a, int G, int group) {
    const int tap = group / G;
    g = group - tap * G;
    r = tap / a.S;
    s = tap - r * a.S;
  }
  __device__ void advance(const KArgs& a, const GroupStep& st) {
    g += st.dg;
    s += st.ds;
    r += st.dr;
    if (g >= st.G) { g -= st.G; ++s; }
    if (s >= a.S) { s -= a.S; ++r; }
  }
  __device__ void next(const KArgs& a, int G) {
    if (++g == G) { g = 0; ++s; }
    if (s == a.S) { s = 0; ++r; }
  }
};

// Stage order: taps inside channel slabs, as the fp32 one-tap kernels.
struct TapPos {
  int r, s, c0;
  __device__ void init(const KArgs& a, int kt, int KT) {
    const int rs = a.R * a.S, slab = kt / rs, tap = kt - slab * rs;
    c0 = slab * KT;
    r = tap / a.S;
    s = tap - r * a.S;
  }
  // to the next stage if `more` (selects, not branches: the main loop's body
  // stays one basic block, which the interleaving below needs)
  __device__ void advance(const KArgs& a, int KT, bool more) {
    const int s1 = s + (more ? 1 : 0);
    const bool ws = s1 == a.S;
    const int r1 = r + (ws ? 1 : 0);
    const bool wr = r1 == a.R;
    s = ws ? 0 : s1;
    r = wr ? 0 : r1;
    c0 += wr ? KT : 0;
  }
};

// Smallest magnitude (as float bits) that a finished sum may have without
// being computed again: 2^-86.
constexpr unsigned kB3TinyBits = 0x14800000u;

// One tile's product over the k-tiles [kt0, kt0 + nk), handed to store(acc,
// m0, n0, wave's first column in the tile, g4, q): acc[i][j][e] is row 16*i +
// 4*g4 + e, and column TN*q + j of the wave (b3_vec) or 16*j + q.
//
// KW > 1: the stages are shared out among KW groups of WN waves, each with LDS
// buffers of its own, and the first group adds up their sums (through LDS) and
// stores.  For layers with too few tiles to give every SIMD a second wave, which
// otherwise wait out the loads, splits and barriers of every stage: 64 channels,
// 3x3 on 56x56, N = 4 (196 tiles): 17.4 us with one group, 13.9 with two, 14.9 with
// four; 2048 channels, 1x1 on 7x7, N = 32 (200 tiles): 51, 36 and 31.
// The smallest layers take 16x16 or 32x32 tiles with sixteen or eight groups, and
// no second launch for split tiles: 256 channels, 3x3 on 14x14, one image: 13.2 us
// split over 256 work-groups and summed by another kernel, 11.3 this way.
template <int LD, int MT, int NT, int KT, int WN, int KW, class Store>
__device__ __forceinline__ void tile_product_b3(const KArgs& a, u32x4* lds0, int t0, int tile, int kt00, int nk_all,
                                                Store&& store) {
  using C = B3Cfg<MT, NT, KT, WN>;
  constexpr int TM = C::TM, TN = C::TN, KS = C::KS;
  constexpr bool kGroups = b3_groups(LD), kRows = b3_rows(LD), kVec = b3_vec(LD);   // kGroups: kRows too
  constexpr int NB = kVec ? 1 : TN;      // patch addresses per lane
  constexpr bool kLook = KW == 1 && WN == 8;      // lost bits of the filter: look before computing again
  static_assert(!kGroups || (KS == 1 && C::UA == 1), "one group of eight rows, or a part of it, per thread");
  // this group's stages: nk of them from kt0; every group runs `loops`, as the
  // barriers are common
  const int kg = KW > 1 ? __builtin_amdgcn_readfirstlane(t0 / C::T) : 0, t = KW > 1 ? t0 - kg * C::T : t0;
  u32x4* const lds = lds0 + kg * C::LDS_CHUNKS;
  const int loops = KW > 1 ? (nk_all + KW - 1) / KW : nk_all;
  const int nk = KW > 1 ? min(loops, nk_all - kg * loops) : nk_all;      // (none or less: all its columns are out of range)
  const int kt0 = nk > 0 ? kt00 + kg * loops : kt00;
  const int m0 = (tile % a.tiles_m) * MT, n0 = (tile / a.tiles_m) * NT;
  const int wn = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
  const int g4 = lane >> 4, q = lane & 15;
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes);
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(a.w, a.w_bytes);

  // filter: thread t takes column m0 + t % MT, AR rows of the stage from AR*(t / MT)
  const int am = m0 + t % MT, ak = t / MT * C::AR;
  const bool am_ok = am < a.Mg;
  unsigned* const aslot = reinterpret_cast<unsigned*>(lds) + 4 * ((ak >> 3) * MT + t % MT) + (ak & 7) / 2;
  // patches: this lane's TN columns, and rows 8*g4 .. 8*g4+7 of each 32: its
  // part of the MFMA's operand, so the patches never go through LDS (no other
  // wave of the group needs them)
  int ih0[NB], iw0[NB];
  unsigned bbase[NB];                // bytes to the column's pixel at tap (0, 0); wraps below zero at the border
  bool col_ok[NB];
  const unsigned C4 = 4u * (unsigned)(LD == kB3SlabW ? a.H * a.W : a.N);   // bytes between channels
  const unsigned tap_w4 = LD == kB3SlabW ? 4u : 4u * (unsigned)(a.C * a.N), tap_h4 = (unsigned)a.W * tap_w4;
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    const int n = n0 + wn * C::WTN + (kVec ? q * TN : 16 * j + q);
    col_ok[j] = n < a.Ng;
    int pix, b;
    if constexpr (LD == kB3SlabW) { const int hw = a.Ho * a.Wo; b = n / hw; pix = n - b * hw; }
    else if constexpr (LD == kB3GroupC) { b = 0; pix = n; }
    else { pix = n / a.N; b = n - pix * a.N; }
    const int ho = pix / a.Wo;
    ih0[j] = ho * a.sh - a.ph;
    iw0[j] = (pix - ho * a.Wo) * a.sw - a.pw;
    if constexpr (LD == kB3SlabW) bbase[j] = 4u * (unsigned)(((b * a.C + 8 * g4) * a.H + ih0[j]) * a.W + iw0[j]);
    else bbase[j] = 4u * (unsigned)(((ih0[j] * a.W + iw0[j]) * a.C + (kGroups ? 0 : 8 * g4)) * a.N + b);
  }
  const unsigned K4 = 4u * (unsigned)a.K;

  float fa[C::UA][C::AR];            // loaded, not yet split
  float fb[8][TN];
  u32x4 bf[2][TN][3];                // patch fragments of this k-step and the next
  unsigned ap[C::UA][C::AR / 2][3];  // split filter rows on their way to LDS
  unsigned lost = 0;                 // lower halves of this thread's third parts (split2)

  // Where the next loads go.  Patches are loaded two k-steps ahead, the filter
  // two stages ahead.
  TapPos pa, pb;
  GroupPos ga, gb;
  GroupStep gst;
  unsigned av, bv[NB], as = 0, bs = 0;
  int arow = 0;
  unsigned brow = 0;                 // row variants: the thread's first filter row, and the bytes to the lane's row
  bool blive = true;
  const int G = kRows ? a.C : a.C >> 3;
  auto start_a = [&](int kt) {
    if constexpr (kRows) arow = kt * KT + ak;
    else if constexpr (kGroups) ga.init(a, G, kt * (KT / 8) + (ak >> 3));
    else pa.init(a, kt, KT);
  };
  auto start_b = [&](int kt) {
    if constexpr (kGroups) gb.init(a, G, kRows ? kt * KT + 8 * g4 : kt * (KT / 8) + g4);
    else pb.init(a, kt, KT);
  };
  auto advance_a = [&](bool more) {
    if constexpr (kRows) arow += KT;
    else if constexpr (kGroups) ga.advance(a, gst);
    else pa.advance(a, KT, more);
  };
  auto advance_b = [&](bool more) {
    if constexpr (kGroups) gb.advance(a, gst);
    else pb.advance(a, KT, more);
  };
  auto place_a = [&]() {
    if constexpr (kRows) {
      av = 4u * (unsigned)(arow * a.K + am);
    } else if constexpr (kGroups) {
      const int c = 8 * ga.g + (ak & 7);
      const bool ok = am_ok & (ga.r < a.R);
      const unsigned at = 4u * (unsigned)(((ga.r * a.S + ga.s) * a.C + c) * a.K + am);
      av = ok ? at : kOOB;
    } else {
      av = am_ok ? 4u * (unsigned)(am + ak * a.K) : kOOB;
      as = (unsigned)((pa.r * a.S + pa.s) * a.C + pa.c0) * K4;
    }
  };
  auto place_b = [&](bool live, int ks) {
    if constexpr (kRows) {
      brow = (unsigned)gb.r * tap_h4 + (unsigned)gb.s * tap_w4 + (unsigned)gb.g * C4;
      blive = live;
      return;
    }
    const int r = kGroups ? gb.r : pb.r, s = kGroups ? gb.s : pb.s;
    const unsigned off = (unsigned)r * tap_h4 + (unsigned)s * tap_w4 + (kGroups ? 8u * (unsigned)gb.g * C4 : 0u);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const bool ok = live & col_ok[j] & ((unsigned)(ih0[j] + r) < (unsigned)a.H) &
                      ((unsigned)(iw0[j] + s) < (unsigned)a.W) & (!kGroups || r < a.R);
      const unsigned at = bbase[j] + off;
      bv[j] = ok ? at : kOOB;
    }
    if constexpr (!kGroups) bs = (unsigned)(pb.c0 + 32 * ks) * C4;
  };
  auto load_a = [&](int u, int i) {
    float v[1];
    if constexpr (kRows) bload_w<1>(wr, am_ok & (arow + i < a.Kg) ? av : kOOB, (unsigned)i * K4, v);
    else if constexpr (kGroups) bload_w<1>(wr, av, (unsigned)i * K4, v);
    else bload_w<1>(wr, av, as + (unsigned)(u * (C::T / MT) * C::AR + i) * K4, v);
    fa[u][i] = v[0];
  };
  auto load_b = [&](int i) {
    const unsigned rowC4 = C4 * (unsigned)i;
    if constexpr (kRows) {
      // the row's address, then on to the next row: channels and the taps of
      // one filter row follow each other in x, the next filter row is W - S
      // pixels on
      const bool live = blive & (gb.r < a.R);
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const bool ok = live & col_ok[j] & ((unsigned)(ih0[j] + gb.r) < (unsigned)a.H) &
                        ((unsigned)(iw0[j] + gb.s) < (unsigned)a.W);
        const unsigned at = bbase[j] + brow;
        if constexpr (kVec) {
          bload_w<TN>(xr, ok ? at : kOOB, 0u, fb[i]);
        } else {
          float v[1];
          bload_w<1>(xr, ok ? at : kOOB, 0u, v);
          fb[i][j] = v[0];
        }
      }
      const int r0 = gb.r;
      gb.next(a, G);
      brow += C4 + (gb.r != r0 ? tap_h4 - (unsigned)a.S * tap_w4 : 0u);
    } else if constexpr (LD == kB3GroupC) {
      // rows i .. i+3 at once
      if (i % 4 == 0) {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          float v[4];
          bload_w<4>(xr, bv[j], 4u * (unsigned)i, v);
#pragma unroll
          for (int e = 0; e < 4; ++e) fb[i + e][j] = v[e];
        }
      }
    } else if constexpr (kVec) {
      bload_w<TN>(xr, bv[0], bs + rowC4, fb[i]);
    } else {
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        float v[1];
        bload_w<1>(xr, bv[j], bs + rowC4, v);
        fb[i][j] = v[0];
      }
    }
  };

  // The split work in pieces of two rows of one column.
  constexpr int ITB = 4 * TN;                          // per k-step
  constexpr int ITA = C::UA * C::AR / 2;               // per stage
  static_assert(ITA % KS == 0, "the filter's pieces spread evenly over the k-steps");
  constexpr int IT = ITB + ITA / KS;
  auto split_b = [&](int it, int nxt) {
    const int p = it / TN, j = it % TN;
    unsigned o[3];
    split2(fb[2 * p][j], fb[2 * p + 1][j], o, lost);
    pin3(o, lost);
#pragma unroll
    for (int k = 0; k < 3; ++k) bf[nxt][j][k][p] = o[k];
  };
  auto split_a = [&](int it, int buf) {
    const int u = it / (C::AR / 2), p = it % (C::AR / 2);
    split2(fa[u][2 * p], fa[u][2 * p + 1], ap[u][p], lost);
    pin3(ap[u][p], lost);
    if (p == C::AR / 2 - 1) {
      // a lost bit, in these rows or met earlier: NaN in their place
      if constexpr (!kLook) ap[u][p][0] = lost_bits(lost) ? ~0u : ap[u][p][0];
      unsigned* const d = aslot + buf * C::STAGE * 4 + u * (C::T / MT) * C::AR / 8 * MT * 4;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        if constexpr (C::AR == 8)
          *reinterpret_cast<u32x4*>(d + k * C::PLANE * 4) = u32x4{ap[u][0][k], ap[u][1][k], ap[u][2][k], ap[u][3][k]};
        else if constexpr (C::AR == 4)
          *reinterpret_cast<u32x2*>(d + k * C::PLANE * 4) = u32x2{ap[u][0][k], ap[u][1][k]};
        else
          d[k * C::PLANE * 4] = ap[u][0][k];
      }
    }
  };
  auto reload_b = [&](int it) {
    if (it % TN != TN - 1) return;
    const int p = it / TN;
    if constexpr (LD == kB3GroupC) {
      if (p % 2 == 1) load_b(2 * p - 2);
    } else {
      load_b(2 * p);
      load_b(2 * p + 1);
    }
  };
  auto reload_a = [&](int it) {
    load_a(it / (C::AR / 2), 2 * (it % (C::AR / 2)));
    load_a(it / (C::AR / 2), 2 * (it % (C::AR / 2)) + 1);
  };

  f32x4 acc[TM][TN], lo[TM][TN];
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = lo[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  clear();

  // One k-step: its NM MFMAs, row block by row block; each block's filter
  // fragments are read from LDS as the block before it uses a part for the
  // last time (part h has three products, m two, l one).  Between the MFMAs,
  // in even steps: the split of the next k-step's patches and of a KS-th of
  // the next stage's filter, and into the registers that this frees the loads
  // of the k-step (stage) after it.
  constexpr int PER = TN * 6, NM = TM * PER;
  const int abase = g4 * MT + q;
  auto kstep = [&](auto buf_c, auto ks_c) {
    constexpr int buf = decltype(buf_c)::value, ks = decltype(ks_c)::value, cur = (buf * KS + ks) & 1;
    const u32x4* const As = lds + buf * C::STAGE + ks * 4 * MT;
    bf16x8 av[3];
    auto read = [&](int i, int p) { av[p] = __builtin_bit_cast(bf16x8, As[p * C::PLANE + i * 16 + abase]); };
    read(0, 0);
    read(0, 1);
    read(0, 2);
    constexpr int PA[6] = {0, 0, 0, 1, 1, 2}, PX[6] = {0, 1, 2, 1, 0, 0};
    static_for<IT>([&](auto ic) {
      constexpr int it = decltype(ic)::value;
      constexpr int ma = it * NM / IT, mb = (it + 1) * NM / IT;
      if constexpr (it < ITB) split_b(it, cur ^ 1);
      else split_a(ks * (ITA / KS) + it - ITB, buf ^ 1);
      static_for<mb - ma>([&](auto mc) {
        constexpr int m = ma + decltype(mc)::value, i = m / PER, k = m % PER / TN, j = m % TN;
        f32x4& d = k == 0 ? acc[i][j] : lo[i][j];
        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[PA[k]], __builtin_bit_cast(bf16x8, bf[cur][j][PX[k]]), d, 0, 0, 0);
        if constexpr (i + 1 < TM && j == TN - 1 && (k == 2 || k == 4 || k == 5)) read(i + 1, PA[k]);
      });
      // alternate them one MFMA to a few vector instructions: two waves per
      // SIMD alone do not fill the MFMA pipe if each runs its split in a block
      static_for<mb - ma>([&](auto) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, (12 + mb - ma - 1) / (mb - ma > 0 ? mb - ma : 1), 0);
      });
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (it < ITB) reload_b(it);
      else reload_a(ks * (ITA / KS) + it - ITB);
    });
    __builtin_amdgcn_sched_barrier(0);
  };
  // The buffer that the previous stage consumed, filled with NaN (debug build).
  auto poison = [&](int buf) {
    if constexpr (MG3M_LDS_POISON != 0) {
      for (int i = t; i < C::STAGE; i += C::T) lds[buf * C::STAGE + i] = u32x4{~0u, ~0u, ~0u, ~0u};
      __syncthreads();
    }
  };

  // Stages go in pairs, one per LDS buffer, KS k-steps each.  Past the last
  // one the patch columns are out of range and the filter address stays.
  if constexpr (kGroups) gst.init(a, G, kRows ? KT - 8 : KT / 8);   // rows: eight are stepped by their loads
  start_a(kt0);
  start_b(kt0);
  place_a();
#pragma unroll
  for (int it = 0; it < ITA; ++it) reload_a(it);
  place_b(KW == 1 || nk > 0, 0);
#pragma unroll
  for (int it = 0; it < ITB; ++it) reload_b(it);
#pragma unroll
  for (int it = 0; it < ITA; ++it) split_a(it, 0);
#pragma unroll
  for (int it = 0; it < ITB; ++it) split_b(it, 0);
  advance_a(nk > 1);
  place_a();
#pragma unroll
  for (int it = 0; it < ITA; ++it) reload_a(it);
  if constexpr (KS == 1) advance_b(nk > 1);
  place_b(KS > 1 ? KW == 1 || nk > 0 : nk > 1, KS > 1 ? 1 : 0);
#pragma unroll
  for (int it = 0; it < ITB; ++it) reload_b(it);
  __syncthreads();
  auto stage = [&](int it, auto buf_c) {
    constexpr int buf = decltype(buf_c)::value;
    poison(buf ^ 1);
    advance_a(it + 2 < nk);
    place_a();
    static_for<KS>([&](auto ks_c) {
      // k-step ks of stage it loads the patches two k-steps on
      constexpr int ks = decltype(ks_c)::value, step = ks + 2;
      if constexpr (step % KS == 0) advance_b(it + step / KS < nk);
      place_b(it + step / KS < nk, step % KS);
      __builtin_amdgcn_sched_barrier(0);
      kstep(buf_c, ks_c);
    });
    __syncthreads();
  };
  for (int it = 0; it < loops; it += 2) {
    stage(it, std::integral_constant<int, 0>{});
    if (it + 1 < loops) stage(it + 1, std::integral_constant<int, 1>{});
  }
  // (the last stage's barrier: the buffers are free)
  unsigned* const note = reinterpret_cast<unsigned*>(lds0 + KW * C::LDS_CHUNKS) - 16;
  const bool wave_lost = kLook && __ballot(lost_bits(lost)) != 0;
  if (kLook && (g4 | q) == 0) note[wn] = wave_lost;
  // the first group's wave answers for the patches of all groups
  if (KW > 1 && lost_bits(lost)) lo[0][0][0] = __builtin_nanf("");
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      acc[i][j] += lo[i][j];
      if (KW > 1 && kg > 0) lds0[((kg - 1) * TM * TN + i * TN + j) * C::T + t] = __builtin_bit_cast(u32x4, acc[i][j]);
    }
  static_assert((KW - 1) * TM * TN * C::T <= KW * C::LDS_CHUNKS, "the groups' sums fit the buffers");
  if constexpr (KW > 1 || kLook) __syncthreads();
  // a wave of the work-group has met a lost bit
  const bool met = kLook && __ballot(q < WN && note[q] != 0) != 0;
  if constexpr (KW > 1) {
    if (kg > 0) return;
#pragma unroll
    for (int g = 1; g < KW; ++g)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] += __builtin_bit_cast(f32x4, lds0[((g - 1) * TM * TN + i * TN + j) * C::T + t]);
  }
  unsigned tiny = 0xffffffffu;
  float big = 0.f;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        big += __builtin_fabsf(acc[i][j][e]);                    // infinite or NaN if any is
        tiny = min(tiny, __builtin_bit_cast(unsigned, acc[i][j][e]) * 2u - 1u);   // zeros wrap to the maximum
      }
  bool again = !(big < __builtin_inff()) | (tiny < kB3TinyBits * 2u - 1u) | (KW == 1 && !kLook && lost_bits(lost));
  bool compute = __ballot(again) != 0;
  if (MG3M_LDS_POISON == 0 && (compute | met)) {
    // This wave's patches again, straight from memory: with the filter in the
    // second pass, on fp32 MFMA (step k of 32 rows takes rows 8*g + k of each
    // lane group g, the rows that the lanes' patches hold); in the first, if that
    // is not needed anyway, for whether it is.  One loop for both: two take four
    // registers.
#pragma unroll 1
    for (;;) {
      unsigned lost_b = 0;
      big = 0.f;
      if (compute) clear();
      start_b(kt00);
      for (int it = 0; it < nk_all; ++it) {
#pragma unroll 1
        for (int ks = 0; ks < KS; ++ks) {
          place_b(true, ks);
#pragma unroll
          for (int k = 0; k < ITB; ++k) reload_b(k);
          if (!compute) {
#pragma unroll
            for (int i = 0; i < 8; i += 2)
#pragma unroll
              for (int j = 0; j < TN; ++j) {
                unsigned o[3];
                big = fmaxf(big, fmaxf(__builtin_fabsf(fb[i][j]), __builtin_fabsf(fb[i + 1][j])));
                split2(fb[i][j], fb[i + 1][j], o, lost_b);
              }
            continue;
          }
          // the lane group's first filter row
          const int row = kRows ? (kt00 + it) * KT + 8 * g4
                          : kGroups ? (gb.r * a.S + gb.s) * a.C + 8 * gb.g
                                  : (pb.r * a.S + pb.s) * a.C + pb.c0 + 32 * ks + 8 * g4;
          const unsigned fv = 4u * (unsigned)(row * a.K + m0 + q);
          // all loads of the 32 rows in flight at once
          float f[8][TM][1];
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const bool row_ok = kRows ? row + k < a.Kg : !kGroups || gb.r < a.R;
#pragma unroll
            for (int i = 0; i < TM; ++i)
              bload_w<1>(wr, row_ok & (m0 + i * 16 + q < a.Mg) ? fv + 64u * i : kOOB, (unsigned)k * K4, f[k][i]);
          }
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int k = 0; k < 8; ++k)
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
              for (int j = 0; j < TN; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[k][i][0], fb[k][j], acc[i][j], 0, 0, 0);
        }
        advance_b(it + 1 < nk_all);
      }
      if (compute) break;
      const unsigned safe = __builtin_bit_cast(unsigned, least_safe(wave_max(big), a.Kg));
      again = lost_bits(lost_b) | (tiny < safe * 2u - 1u);
      // a sum of nothing but lost parts is zero (opaque: or its bounds are formed
      // ahead of the loop, in every call)
      int rows = a.Mg - m0, cols = a.Ng - n0 - wn * C::WTN;
      asm volatile("" : "+s"(rows), "+s"(cols));
      rows -= 4 * g4;
      cols -= kVec ? q * TN : q;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e)
            again |= (acc[i][j][e] == 0.f) & (16 * i + e < rows) & ((kVec ? j : 16 * j) < cols);
      compute = __ballot(again) != 0;
      if (!compute) break;
    }
  }
  store(acc, m0, n0, wn * C::WTN, g4, q);
}

// A lane's finished rows (16*i + e from row_l on) of SW columns from n on
// (accumulator columns u .. u+SW-1) to y, with the fused output stage.  Rows
// and columns outside y go to the out-of-range offset.
template <int LAYOUT, int TM, int TN, int SW, bool FUSE>
__device__ __forceinline__ void store_cols_b3(const KArgs& a, __amdgpu_buffer_rsrc_t yr, __amdgpu_buffer_rsrc_t ar,
                                              bool has_add, f32x4 (&acc)[TM][TN], int u, int row_l, int n) {
  unsigned rs4 = 4u * (unsigned)a.mstride;
  asm volatile("" : "+s"(rs4));
  const int rows_left = a.Mg - row_l;
  const bool col_ok = n < a.Ng;
  const unsigned voff = 4u * (unsigned)(out_colbase<LAYOUT>(a, n) + row_l * a.mstride);
  auto offset = [&](int i, int e) {
    const bool ok = col_ok & (i * 16 + e < rows_left);
    return ok ? voff + (unsigned)(i * 16 + e) * rs4 : kOOB;
  };
  if constexpr (FUSE) {
    // every load of add is in flight before the first is used (they fit the
    // registers that the small products' sums leave).  Loaded one by one, each
    // waited for the store before it, which may go to the same memory:
    // 64 -> 256 channels at 56x56, N = 64: 228 us, now 112 (one form's 128x128
    // tiles).
    if (has_add) {
      float d[TM][4][SW];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) bload_w<SW>(ar, offset(i, e), 0u, d[i][e]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int j = 0; j < SW; ++j) acc[i][u + j][e] += d[i][e][j];
    }
    if (a.relu != 0) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int j = 0; j < SW; ++j)
            if (acc[i][u + j][e] < 0.f) acc[i][u + j][e] = 0.f;     // NaN kept
    }
  }
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float v[SW];
#pragma unroll
      for (int j = 0; j < SW; ++j) v[j] = acc[i][u + j][e];
      bstore_w<SW>(yr, offset(i, e), 0u, v);
    }
}

// Schedule and tails as conv_igemm_f32: whole tiles grouped per XCD, then the
// tail work-groups, whose pieces (split, or stream-K runs of up to two) leave
// tile-local partials for the tail reduction.
template <int LD, int MT, int NT, int KT, int WN, int KW, bool FUSE>
__global__ __launch_bounds__(KW * WN * 64) __attribute__((amdgpu_waves_per_eu(KW > 2 ? 4 : 2)))
void conv_igemm_b3(KArgs a) {
  using C = B3Cfg<MT, NT, KT, WN>;
  constexpr int TM = C::TM, TN = C::TN;
  constexpr bool kVec = b3_vec(LD);
  constexpr int NS = kVec ? 1 : TN, SW = kVec ? TN : 1;      // stores per row, and their width
  __shared__ __attribute__((aligned(16))) u32x4 lds[KW * C::LDS_CHUNKS];

  // One call of the product for whole tiles and pieces: a second copy of its
  // code would cost registers, scalar ones above all.
  const bool whole = (int)blockIdx.x < a.dp_tiles;
  const int w = whole ? 0 : tail_wg(a, blockIdx.x - a.dp_tiles);
  TailRun run = whole ? TailRun{0, 0} : tail_run(a, w);
  for (;;) {
    int rel = 0, kt0 = 0, nk = a.k_tiles, tile = xcd_group(blockIdx.x, a.dp_tiles);
    if (!whole) {
      tail_piece(a, run, &rel, &kt0, &nk);
      tile = a.dp_tiles + rel;
    }
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    tile_product_b3<LD, MT, NT, KT, WN, KW>(
        a, lds, t, tile, kt0, nk, [&](f32x4 (&acc)[TM][TN], int m0, int n0, int wcol, int g4, int q) {
          if (!whole) {
            const __amdgpu_buffer_rsrc_t pr = make_rsrc(a.ws + tail_slot(w, rel) * (MT * NT), MT * NT * 4);
            const unsigned lane_b = 4u * (unsigned)(4 * g4 * NT + wcol + (kVec ? q * TN : q));
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
              for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int u = 0; u < NS; ++u) {
                  float v[SW];
#pragma unroll
                  for (int j = 0; j < SW; ++j) v[j] = acc[i][u + j][e];
                  bstore_w<SW>(pr, lane_b, 4u * ((i * 16 + e) * NT + 16 * u), v);
                }
            return;
          }
          const __amdgpu_buffer_rsrc_t yr = make_rsrc(a.y, a.y_bytes);
          const bool has_add = FUSE && a.add != nullptr;
          const __amdgpu_buffer_rsrc_t ar = make_rsrc(has_add ? a.add : a.y, a.y_bytes);
#pragma unroll
          for (int u = 0; u < NS; ++u)
            store_cols_b3<LD == kB3SlabW ? kNCHW : kHWCN, TM, TN, SW, FUSE>(
                a, yr, ar, has_add, acc, u, m0 + 4 * g4, n0 + wcol + (kVec ? q * TN : 16 * u + q));
        });
    run.it += nk;
    if (whole || run.it >= run.end) return;
    __syncthreads();   // the next piece restages the LDS buffers
  }
}

template <int LD, bool FUSE, int TI>
constexpr KernelFn b3_kernel_at() {
  constexpr TileDesc d = kTilesB3[TI];
  if constexpr (b3_built(LD, TI)) return &conv_igemm_b3<LD, d.mt, d.nt, d.kt, d.wn, d.wm, FUSE>;
  else return nullptr;
}
template <int LD, bool FUSE, int... TI>
KernelFn pick_b3(int tile, std::integer_sequence<int, TI...>) {
  KernelFn fn = nullptr;
  ((fn = (tile == TI ? b3_kernel_at<LD, FUSE, TI>() : fn)), ...);
  return fn;
}
template <int LD, bool FUSE>
KernelFn b3_kernel_for_tile(int tile) {
  return pick_b3<LD, FUSE>(tile, std::make_integer_sequence<int, kNumTilesB3>{});
}

}  // namespace mg3m
