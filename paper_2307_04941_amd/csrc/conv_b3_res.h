// 1x1 convolutions on bf16 part products, persistent, with the filter resident
// in LDS.  Included by conv_b3_res.hip.
//
// Why: these layers have few reduction steps per tile (2 to 8 stages of 32 to
// 64 rows), so the tile kernel (conv_b3.h) spends more time on the start and
// the end of its tiles than between, and splits every filter element again for
// every 64 columns.  Here a work-group splits a 64-row filter tile once, keeps
// its parts in LDS, and its waves then walk the columns on their own, 32 at a
// time: no barrier, no second split, the patches of the next columns in flight
// while these are stored, and a wave's stores under the other waves' MFMAs.
#pragma once

#include "conv_b3.h"

namespace mg3m {

template <bool FUSE>
__global__ __launch_bounds__(kB3ResWaves * 64)
void conv_igemm_b3_res(KArgs a) {
  constexpr int WV = kB3ResWaves, MT = 64, TM = 4, TN = 2, WTN = 16 * TN;
  // [C / 8][part][MT] chunks of eight consecutive rows of one filter column
  __shared__ __attribute__((aligned(16))) u32x4 lds[kB3ResMaxC / 8 * 3 * MT];
  int t = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6), lane = t & 63;
  const int g4 = lane >> 4, q = lane & 15;
  const int chunks = a.C >> 3, nk = a.C >> 5;
  const unsigned K4 = 4u * (unsigned)a.K, C4 = 4u * (unsigned)a.N;
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, a.x_bytes);
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(a.w, a.w_bytes);
  const __amdgpu_buffer_rsrc_t yr = make_rsrc(a.y, a.y_bytes);
  const bool has_add = FUSE && a.add != nullptr;
  const __amdgpu_buffer_rsrc_t ar = make_rsrc(has_add ? a.add : a.y, a.y_bytes);

  // Work-group i runs on XCD i % 8.  Each XCD takes a contiguous eighth of the
  // column blocks for all filter tiles (its L2 then serves the patches'
  // re-reads), dealt out in equal runs of (filter tile, column block).
  const int blocks = (a.Ng + WTN - 1) / WTN;
  const int xcd = (int)(blockIdx.x & 7), loc = (int)(blockIdx.x >> 3), cnt = (int)(gridDim.x >> 3);
  const int cb0 = (int)((long long)blocks * xcd >> 3), nb = (int)((long long)blocks * (xcd + 1) >> 3) - cb0;
  const long long units = (long long)a.tiles_m * nb;
  long long u = units * loc / cnt;
  const long long u_end = units * (loc + 1) / cnt;

  float fb[8][TN];
  u32x4 bf[2][TN][3];
  f32x4 acc[TM][TN], lo[TM][TN];
  unsigned lost = 0;                 // lower halves of the patches' third parts (split2)
  auto clear = [&]() {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = lo[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  // byte offset of this lane's columns (row 8*g4) in column block cb
  auto place = [&](int cb, bool live) {
    const int n = cb * WTN + q * TN;
    const int pix = n / a.N, b = n - pix * a.N, ho = pix / a.Wo;
    const int ih = ho * a.sh - a.ph, iw = (pix - ho * a.Wo) * a.sw - a.pw;
    const bool ok = live & (n < a.Ng) & ((unsigned)ih < (unsigned)a.H) & ((unsigned)iw < (unsigned)a.W);
    const unsigned at = 4u * (unsigned)(((ih * a.W + iw) * a.C + 8 * g4) * a.N + b);
    return ok ? at : kOOB;
  };
  auto split_b = [&](int it, int nxt) {
    const int p = it / TN, j = it % TN;
    unsigned o[3];
    split2(fb[2 * p][j], fb[2 * p + 1][j], o, lost);
    pin3(o, lost);
#pragma unroll
    for (int k = 0; k < 3; ++k) bf[nxt][j][k][p] = o[k];
  };
  const u32x4* const Al = lds + g4 * 3 * MT + q;
  // One step of 32 rows: its 48 MFMAs, and between them the split of the next
  // step's patches and the loads of the one after (at voff + soff).
  constexpr int IT = 4 * TN, PER = TN * 6, NM = TM * PER;
  auto kstep = [&](auto cur_c, int ks, unsigned voff, unsigned soff) {
    constexpr int cur = decltype(cur_c)::value;
    const u32x4* const As = Al + ks * (4 * 3 * MT);
    bf16x8 av[3];
    auto read = [&](int i, int p) { av[p] = __builtin_bit_cast(bf16x8, As[p * MT + i * 16]); };
    read(0, 0);
    read(0, 1);
    read(0, 2);
    constexpr int PA[6] = {0, 0, 0, 1, 1, 2}, PX[6] = {0, 1, 2, 1, 0, 0};
    static_for<IT>([&](auto ic) {
      constexpr int it = decltype(ic)::value;
      constexpr int ma = it * NM / IT, mb = (it + 1) * NM / IT;
      split_b(it, cur ^ 1);
      static_for<mb - ma>([&](auto mc) {
        constexpr int m = ma + decltype(mc)::value, i = m / PER, k = m % PER / TN, j = m % TN;
        f32x4& d = k == 0 ? acc[i][j] : lo[i][j];
        d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[PA[k]], __builtin_bit_cast(bf16x8, bf[cur][j][PX[k]]), d, 0, 0, 0);
        if constexpr (i + 1 < TM && j == TN - 1 && (k == 2 || k == 4 || k == 5)) read(i + 1, PA[k]);
      });
      static_for<mb - ma>([&](auto) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, (12 + mb - ma - 1) / (mb - ma), 0);
      });
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (it % TN == TN - 1) {
        constexpr int p = it / TN;
        bload_w<TN>(xr, voff, soff + C4 * (2 * p), fb[2 * p]);
        bload_w<TN>(xr, voff, soff + C4 * (2 * p + 1), fb[2 * p + 1]);
      }
    });
    __builtin_amdgcn_sched_barrier(0);
  };

  while (u < u_end) {
    const int tm = (int)(u / nb), m0 = tm * MT;
    const int first = (int)(u - (long long)tm * nb);
    const int last = (int)min((long long)nb, first + (u_end - u));      // column blocks [first, last) of the XCD's
    u += last - first;
    int cb = cb0 + first + wave;
    const int cb_end = cb0 + last;
    // the first patches, then the filter tile
    unsigned bv = place(cb, cb < cb_end);
#pragma unroll
    for (int i = 0; i < 8; ++i) bload_w<TN>(xr, bv, C4 * (unsigned)i, fb[i]);
    if constexpr (MG3M_LDS_POISON != 0) {
      for (int i = t; i < kB3ResMaxC / 8 * 3 * MT; i += WV * 64) lds[i] = u32x4{~0u, ~0u, ~0u, ~0u};
      __syncthreads();
    }
    {
      constexpr int UA = kB3ResMaxC / 8 / WV;
      float fa[UA][8];
      const int m = m0 + lane;
#pragma unroll
      for (int r = 0; r < UA; ++r) {
        const int c8 = wave + r * WV;
        const unsigned at = (c8 < chunks) & (m < a.Mg) ? 4u * (unsigned)(c8 * 8 * a.K + m) : kOOB;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          float v[1];
          bload_w<1>(wr, at, (unsigned)i * K4, v);
          fa[r][i] = v[0];
        }
      }
#pragma unroll
      for (int r = 0; r < UA; ++r) {
        const int c8 = wave + r * WV;
        if (c8 >= chunks) break;
        unsigned o[4][3], lost_a = 0;
#pragma unroll
        for (int p = 0; p < 4; ++p) split2(fa[r][2 * p], fa[r][2 * p + 1], o[p], lost_a);
        o[0][0] = lost_bits(lost_a) ? ~0u : o[0][0];      // a lost bit: NaN in its place
#pragma unroll
        for (int k = 0; k < 3; ++k) lds[(c8 * 3 + k) * MT + lane] = u32x4{o[0][k], o[1][k], o[2][k], o[3][k]};
      }
    }
    lost = 0;
    static_for<IT>([&](auto ic) { split_b(decltype(ic)::value, 0); });
#pragma unroll
    for (int i = 0; i < 8; ++i) bload_w<TN>(xr, bv, C4 * (unsigned)(32 + i), fb[i]);
    __syncthreads();

    for (; cb < cb_end; cb += WV) {
      unsigned lost_here = 0;
      clear();
      for (int ks = 0; ks < nk; ks += 2) {
        // the loads are two steps ahead: in the last two, the next block's
        const bool end = ks + 2 == nk;
        if (end) bv = place(cb + WV, cb + WV < cb_end);
        const unsigned soff = end ? 0u : C4 * (unsigned)(32 * (ks + 2));
        __builtin_amdgcn_sched_barrier(0);
        kstep(std::integral_constant<int, 0>{}, ks, bv, soff);
        // this block's patches are all split; from here on the next block's
        lost_here = lost;
        lost = end ? 0u : lost;
        kstep(std::integral_constant<int, 1>{}, ks + 1, bv, soff + 32u * C4);
      }
      unsigned tiny = 0xffffffffu;
      float big = 0.f;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          acc[i][j] += lo[i][j];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            big += __builtin_fabsf(acc[i][j][e]);
            tiny = min(tiny, __builtin_bit_cast(unsigned, acc[i][j][e]) * 2u - 1u);
          }
        }
      const bool again = !(big < __builtin_inff()) | (tiny < kB3TinyBits * 2u - 1u) | lost_bits(lost_here);
      if (MG3M_LDS_POISON == 0 && __ballot(again) != 0) {
        // this block again on fp32 MFMA, straight from memory (tile_product_b3)
        clear();
        const unsigned v0 = place(cb, true);
#pragma unroll 1
        for (int ks = 0; ks < nk; ++ks) {
          const unsigned fv = 4u * (unsigned)((32 * ks + 8 * g4) * a.K + m0 + q);
#pragma unroll
          for (int k0 = 0; k0 < 8; k0 += 4) {
            float xv[4][TN], f[4][TM][1];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              bload_w<TN>(xr, v0, C4 * (unsigned)(32 * ks + k0 + k), xv[k]);
#pragma unroll
              for (int i = 0; i < TM; ++i)
                bload_w<1>(wr, m0 + i * 16 + q < a.Mg ? fv + 64u * i : kOOB, (unsigned)(k0 + k) * K4, f[k][i]);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
              for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
                  acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[k][i][0], xv[k][j], acc[i][j], 0, 0, 0);
          }
        }
      }
      store_cols_b3<kHWCN, TM, TN, TN, FUSE>(a, yr, ar, has_add, acc, 0, m0 + 4 * g4, cb * WTN + q * TN);
    }
    __syncthreads();   // every wave is done with the filter tile
  }
}

}  // namespace mg3m
