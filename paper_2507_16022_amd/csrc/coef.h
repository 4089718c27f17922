// First half of the coefficient route for split precisions: the raw
// accumulators of every pair of the listed 64 x 64 tiles, stored for the
// kernels that bound and marginalise them.
//
// An accumulator is complete when its m group's chunks (or its (h|h) block)
// are, so it is stored there and then and a wave needs one group's at a time:
// 64 x 32 pairs per wave in 2 x 32 accumulator registers (the fused kernel
// holds all 240 of a tile's 32 x 32 pairs until its epilogue, one wave per
// SIMD).  A workgroup of two waves takes a tile, with two stages of 16 KB in
// LDS; four workgroups share a CU, so one's loads, barriers and stores run
// beside the products of the others, and a chunk's loads have the products of
// two waves to arrive in.  64 x 32 pairs per wave read 12 KB from LDS for 24
// products (32 x 32: 8 KB for 12, the LDS rate's limit).  A list short enough
// to leave half of the workgroups idle is taken in halves of 32 rows instead,
// which halves the time of its one round.
//
// Launches that the host knows to be of few tiles leave each workgroup most of a CU,
// and then two stages wait for loads at every step, and the loads issued in front
// of the products keep the matrix cores waiting.  So more stages and the loads
// between the products: up to 128 tiles in halves (every half its own CU), up to
// 512 by four waves of 32 x 32 pairs each (two halves on a CU would load 24 KB per
// chunk, as fast as a CU's share of L2 gives it; a tile 16).  ln L matrices of one
// phase, five modes, before and now: 512 bins, 200 tiles 0.139 -> 0.114 ms, 500
// tiles 0.227 -> 0.191; 1700 bins, one tile 0.242 -> 0.187, 200 tiles 0.324 ->
// 0.238; 256 bins, 256 tiles 0.109 -> 0.093.  (The fused kernel, four waves and
// eight stages, one workgroup per CU: 0.117, 0.227, 0.201, 0.227, 0.097.)
//
// 2048 tiles of 5-mode, 256-bin operands take 0.30 ms (0.36 to 0.38 in the
// fused kernel), if neighbouring tiles run together: with the list in the
// order in which it was written half of the reads missed L2 and it took as
// long as before.
#pragma once

#include "fused.h"

namespace dotpe {

// bytes of a chunk of 32 bm rows: A hi, A lo (2 KB per 32 rows each), B hi, B lo
// (4 KB each)
constexpr int coef_stage(int bm) { return bm * 4096 + 8192; }
struct CoefTile {
  static constexpr int NT = 128;
  static constexpr int HALF_NS = 3, FEW_NS = 6;      // stages of half a tile
  static constexpr int MID_NS = 4;                   // of a tile by four waves
  static constexpr int LDS_BYTES = HALF_NS * coef_stage(1);
  static constexpr int FEW_BYTES = FEW_NS * coef_stage(1);
  static constexpr int MID_BYTES = MID_NS * coef_stage(2);
  static_assert(2 * coef_stage(2) <= LDS_BYTES && 4 * LDS_BYTES <= 160 * 1024, "four workgroups per CU");
  static_assert(2 * MID_BYTES <= 160 * 1024, "two workgroups per CU");
};

// Work item q, by a workgroup of NW waves, 32 BM x 32 pairs each, with NS stages:
// the tile (NW BM = 4) or the 32 rows `half` of it (NW BM = 2).
template <int PREC, int G, int NW, int BM, int NS>
__device__ __forceinline__ void coef_item(const FusedArgs& a, unsigned char* smem, int64_t q, int half) {
  static_assert(PREC != kFP64, "split precisions only");
  static_assert((NW == 2 && (BM == 1 || BM == 2)) || (NW == 4 && BM == 1), "a tile or half of one");
  typedef typename Pol<PREC>::Acc Acc;
  typedef __attribute__((address_space(1))) const unsigned char gbyte;
  typedef __attribute__((address_space(3))) void lvoid;
  constexpr int NRT = (G == 1) ? 1 : kMaxNR;
  constexpr int NCO = 2 * G + NRT, NPT = 64 * 64;
  constexpr int ES = 2;                      // bytes per operand element
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ndh = a.n_chunks;                // (d|h) chunks (groups of a multiple of 4), then NRT (h|h) blocks
  const int nk = ndh + NRT;
  constexpr int RB = NW * BM / 2;            // 32-row blocks
  constexpr int STAGE = coef_stage(RB), ALO = 2048 * RB, BHI = 2 * ALO, BLO = BHI + 4096;
  const int wm = NW == 4 ? wave >> 1 : 0, wn = wave & 1;      // the wave's rows and columns

  // fragments of one chunk: A blocks [bm][slice] and this wave's B block
  struct Frag {
    uint4 ah[BM][2], al[BM][2], bh[2], bl[2];
  };
  constexpr int NF = 4 * BM + 4;
  Frag fr0, fr1;
  auto frag = [&](auto pi) -> Frag& {
    if constexpr (decltype(pi)::value % 2 == 0) return fr0;
    else return fr1;
  };
  // byte offset of the stage after one at `at`
  auto after = [](unsigned at) { return at == (NS - 1) * STAGE ? 0u : at + STAGE; };
  // read k (0 .. NF - 1) of a chunk's fragments from the stage at `at`
  auto read_k = [&](Frag& f, unsigned at, int k) {
    const unsigned char* st = smem + at + lane * 16;
    const int x = k % (2 * BM);
    if (k < 2 * BM) f.al[x >> 1][x & 1] = *(const uint4*)(st + ALO + (2 * wm + x) * 1024);
    else if (k < 4 * BM) f.ah[x >> 1][x & 1] = *(const uint4*)(st + (2 * wm + x) * 1024);
    else if (k < 4 * BM + 2) f.bh[k & 1] = *(const uint4*)(st + BHI + (2 * wn + (k & 1)) * 1024);
    else f.bl[k & 1] = *(const uint4*)(st + BLO + (2 * wn + (k & 1)) * 1024);
  };
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };

  const int64_t t = coef_tile(a, q);
  const int64_t row0 = t / a.n_tiles_n * 64 + 32 * half, col0 = t % a.n_tiles_n * 64;
  float* cf = (float*)a.coef + (q - a.work0) * (int64_t)(NCO * NPT) + (half + wm) * 32 * 64 + 32 * wn +
              (lane & 31);

  // ---- operand streams, 1 KB pieces as they sit in HBM (fragment order): of
  // every chunk slices 0 and 1 of its 32-row blocks, hi and lo.  Rows past the
  // subset re-read the last row (their pairs are never used); columns run to the
  // padded sample count.  A stream is one (A hi, B lo, ..) of a 32-row block: its
  // source steps by one chunk (2 KB), and to the (h|h) operand after the last
  // (d|h) chunk; the immediate offset of the second load applies to the global and
  // the LDS address alike.  The asm saves and restores M0 and waits the state an
  // M0 write needs. ----
  auto blk = [](int64_t i, int64_t K) { return (i >> 5) * (K >> 5) * 1024 + (i & 31) * 8; };
  struct Stream {
    gbyte *p, *hh;         // next chunk, first (h|h) block
  };
  auto stream = [&](bool is_a, int block, bool is_lo) {
    const int r = 32 * block + (lane & 31);
    const int64_t in_chunk = (lane >> 5) * 256;
    Stream t;
    if (is_a) {
      const int64_t ie = min(row0 + r, a.n_sub - 1);
      const int64_t i = a.sub_idx ? a.sub_idx[ie] : a.sub0 + ie;
      t.p = (gbyte*)(is_lo ? a.A1 : a.A0) + (blk(i, a.K2) + in_chunk) * ES;
      t.hh = (gbyte*)(is_lo ? a.Ah1 : a.Ah0) + (blk(ie, a.KH) + in_chunk) * ES;
    } else {
      const int64_t e = col0 + r;
      t.p = (gbyte*)(is_lo ? a.B1 : a.B0) + (blk(e, a.K2) + in_chunk) * ES;
      t.hh = (gbyte*)(is_lo ? a.Bh1 : a.Bh0) + (blk(e, a.KH) + in_chunk) * ES;
    }
    return t;
  };
  auto next = [&](Stream& t, int c) {
    t.p += 1024 * ES;
    if (__builtin_expect(c + 1 == ndh, 0)) t.p = t.hh;
  };
  // Parts of a wave's loads, an M0 value each.  BM = 2: wave 0 loads A, wave 1 B,
  // hi of both blocks, then lo.  Half a tile: each wave one part of A, then its
  // block of B, hi and lo.  Four waves: a stream of A and one of B each.
  constexpr int PARTS = NW == 2 && BM == 1 ? 3 : 2, PER = BM, LPW = 2 * PARTS * PER;
  Stream str[PARTS * PER];
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lvoid*)smem);
  unsigned place[PARTS];
  if constexpr (BM == 2) {
#pragma unroll
    for (int t = 0; t < 4; ++t) str[t] = stream(wave == 0, t & 1, t >= 2);
    place[0] = lds0 + wave * BHI;
    place[1] = place[0] + ALO;
  } else if constexpr (NW == 2) {
    str[0] = stream(true, 0, wave == 1);
    str[1] = stream(false, wave, false);
    str[2] = stream(false, wave, true);
    place[0] = lds0 + wave * ALO;
    place[1] = lds0 + BHI + wave * 2048;
    place[2] = lds0 + BLO + wave * 2048;
  } else {
    str[0] = stream(true, wn, wm);
    str[1] = stream(false, wn, wm);
    place[0] = lds0 + wm * ALO + wn * 2048;
    place[1] = lds0 + BHI + wm * (BLO - BHI) + wn * 2048;
  }
  // part t of the loads of the next chunk (c), into the stage at st
  auto issue_part = [&](int c, unsigned st, auto ti) {
    constexpr int t = decltype(ti)::value;
    unsigned m0_saved;
    if constexpr (PER == 2)
      __asm__ __volatile__(
          "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
          "global_load_lds_dwordx4 %2, off\n\t"
          "global_load_lds_dwordx4 %2, off offset:1024\n\t"
          "global_load_lds_dwordx4 %3, off offset:2048\n\t"
          "global_load_lds_dwordx4 %3, off offset:3072\n\ts_mov_b32 m0, %0"
          : "=&s"(m0_saved)
          : "s"(__builtin_amdgcn_readfirstlane(place[t] + st)), "v"(str[2 * t].p), "v"(str[2 * t + 1].p - 2048)
          : "memory");
    else
      __asm__ __volatile__(
          "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
          "global_load_lds_dwordx4 %2, off\n\t"
          "global_load_lds_dwordx4 %2, off offset:1024\n\ts_mov_b32 m0, %0"
          : "=&s"(m0_saved)
          : "s"(__builtin_amdgcn_readfirstlane(place[t] + st)), "v"(str[t].p)
          : "memory");
#pragma unroll
    for (int q = 0; q < PER; ++q) next(str[PER * t + q], c);
  };
  auto issue = [&](int c, unsigned st) {
    static_for<PARTS>([&](auto ti) { issue_part(c, st, ti); });
  };

  // workgroup barrier with at most n (0 .. NS - 1) of the wave's chunks in flight:
  // the loads complete in order, and a store among them only makes it wait longer
  auto barrier = [&](int n) {
    static_for<NS>([&](auto qi) {
      constexpr int q = decltype(qi)::value;
      if (n == q) pipeline_barrier<q * LPW>();
    });
  };
  unsigned cur_st = 0;         // the stage of chunk j

  // Step j (fragment parity P = j mod 2): once every wave's loads of chunk j + 1
  // have landed (up to j + NS - 1 may stay in flight) and every wave has read
  // chunk j's fragments, chunk j + NS goes into that stage; the products of chunk j
  // (mf(f, k) issues product k of NMF) have the reads of chunk j + 1 between them,
  // and with more than two stages the loads as well (in front of the products they
  // keep the matrix cores waiting where no other wave shares the SIMD).
  auto step = [&](int j, auto pi, auto nmf, auto ahead, auto&& mf) {
    constexpr int P = decltype(pi)::value % 2, NMF = decltype(nmf)::value;
    constexpr int NR = decltype(ahead)::value ? NF : 0;
    Frag& cur = frag(std::integral_constant<int, P>{});
    Frag& nxt = frag(std::integral_constant<int, P + 1>{});
    if constexpr (NR > 0) {
      if constexpr (NS == 2) pipeline_barrier<0>();
      else if (j + NS <= nk) pipeline_barrier<(NS - 2) * LPW>();
      else barrier(nk - 2 - j);
      fence();
      if constexpr (NS == 2) {
        if (j + NS < nk) issue(j + NS, cur_st);
        fence();
      }
    }
    const unsigned nxt_st = after(cur_st);
    static_for<(NMF > NR ? NMF : NR)>([&](auto ti) {
      constexpr int x = decltype(ti)::value;
      if constexpr (x < NMF) mf(cur, x);
      if constexpr (x < NR) read_k(nxt, nxt_st, x);
      if constexpr (NS > 2 && NR > 0 && x >= NMF - 4 && x < NMF - 4 + PARTS) {
        fence();
        if (j + NS < nk) issue_part(j + NS, cur_st, std::integral_constant<int, x - (NMF - 4)>{});
        fence();
      }
    });
    cur_st = nxt_st;
  };

  __syncthreads();       // (the last tile's stages are no longer read)
  static_for<NS>([&](auto ci) {
    if (decltype(ci)::value < nk) issue(decltype(ci)::value, decltype(ci)::value * STAGE);
  });
  barrier(min(NS, nk) - 1);     // chunk 0 has landed
  static_for<NF>([&](auto ki) { read_k(fr0, 0, decltype(ki)::value); });

  // component c of the wave's pairs from block bm's accumulator
  auto store = [&](int c, int bm, const Acc& v) {
#pragma unroll
    for (int e = 0; e < 16; ++e)
      cf[c * NPT + (32 * bm + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)) * 64] = v[e];
  };

  // ---- (d|h), a group at a time.  With A = [hr | hi] and B_re = [Br | -Bi]
  // by slice, re += A B_re and im += A B_im, B_im = [Bi | Br] = [-(B_re
  // slice 1) | B_re slice 0]; 3 split products per real product, the smaller
  // ones first, re and im alternating (each accumulator's products in the
  // fused kernel's order, so their sums are its sums). ----
  int ch = 0;
  static_for<G>([&](auto gi) {
    constexpr int g = decltype(gi)::value;
    Acc re[BM], im[BM];
    const int gend = a.mt.gk0[g + 1];
    auto dh = [&](auto pi, auto first) {
      const Frag& f = frag(pi);
      auto neg = [](const uint4& x) {
        return make_uint4(x.x ^ 0x80008000u, x.y ^ 0x80008000u, x.z ^ 0x80008000u, x.w ^ 0x80008000u);
      };
      const uint4 nbh = neg(f.bh[1]), nbl = neg(f.bl[1]);
      step(ch, pi, std::integral_constant<int, 12 * BM>{}, std::true_type{}, [&](const Frag& f, int x) {
        const int bm = x % BM, k = x / BM;
        if constexpr (decltype(first)::value) {
          if (k == 0) re[bm] = Acc{};
          if (k == 1) im[bm] = Acc{};
        }
        switch (k) {
          case 0: mma<PREC>(re[bm], f.al[bm][0], f.bh[0]); break;
          case 1: mma<PREC>(im[bm], f.al[bm][0], nbh); break;
          case 2: mma<PREC>(re[bm], f.ah[bm][0], f.bl[0]); break;
          case 3: mma<PREC>(im[bm], f.ah[bm][0], nbl); break;
          case 4: mma<PREC>(re[bm], f.ah[bm][0], f.bh[0]); break;
          case 5: mma<PREC>(im[bm], f.ah[bm][0], nbh); break;
          case 6: mma<PREC>(re[bm], f.al[bm][1], f.bh[1]); break;
          case 7: mma<PREC>(im[bm], f.al[bm][1], f.bh[0]); break;
          case 8: mma<PREC>(re[bm], f.ah[bm][1], f.bl[1]); break;
          case 9: mma<PREC>(im[bm], f.ah[bm][1], f.bl[0]); break;
          case 10: mma<PREC>(re[bm], f.ah[bm][1], f.bh[1]); break;
          default: mma<PREC>(im[bm], f.ah[bm][1], f.bh[0]); break;
        }
      });
      ++ch;
    };
    constexpr std::integral_constant<int, 0> even{};
    constexpr std::integral_constant<int, 1> odd{};
    dh(even, std::true_type{});
    dh(odd, std::false_type{});
    while (ch < gend) {
      dh(even, std::false_type{});
      dh(odd, std::false_type{});
    }
#pragma unroll
    for (int bm = 0; bm < BM; ++bm) {
      store(2 * g, bm, re[bm]);
      store(2 * g + 1, bm, im[bm]);
    }
  });
  // ---- (h|h) block r: the real product of the row and column operands ----
  static_for<NRT>([&](auto ri) {
    constexpr int r = decltype(ri)::value;
    Acc h[BM] = {};
    step(ndh + r, ri, std::integral_constant<int, 6 * BM>{}, std::bool_constant<(r + 1 < NRT)>{},
         [&](const Frag& f, int x) {
           const int bm = x % BM, sl = x / (3 * BM);
           switch ((x / BM) % 3) {
             case 0: mma<PREC>(h[bm], f.al[bm][sl], f.bh[sl]); break;
             case 1: mma<PREC>(h[bm], f.ah[bm][sl], f.bl[sl]); break;
             default: mma<PREC>(h[bm], f.ah[bm][sl], f.bh[sl]); break;
           }
         });
#pragma unroll
    for (int bm = 0; bm < BM; ++bm) store(2 * G + r, bm, h[bm]);
  });
}

// n tiles in halves, the two of a tile on one XCD; 2 n at most the workgroups
template <int PREC, int G, int NS>
__device__ __forceinline__ void coef_halves(const FusedArgs& a, unsigned char* smem, int64_t n, int64_t wg_id,
                                            int64_t wg_count) {
  const int64_t part = (n + 7) / 8, y = wg_id / 8;
  int64_t at = wg_id / 2, half = wg_id & 1;
  if (16 * part <= wg_count) {
    at = y / 2 < part ? wg_id % 8 * part + y / 2 : n;
    half = y & 1;
  }
  if (at < n) coef_item<PREC, G, 2, 1, NS>(a, smem, a.work0 + at, (int)half);
}

template <int PREC, int G>
__device__ __forceinline__ void coef_pass(const FusedArgs& a, int64_t wg_id, int64_t wg_count) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int64_t end = min(a.work0 + a.coef_tiles, coef_work_count(a));
  const int64_t n = end - a.work0;
  if (2 * n <= wg_count) {
    // a list that leaves half of the workgroups idle
    coef_halves<PREC, G, CoefTile::HALF_NS>(a, smem, n, wg_id, wg_count);
    return;
  }
#pragma unroll 1
  for (int64_t q0 = a.work0; q0 < end; q0 += wg_count) {
    const int64_t at = coef_place(wg_id, wg_count, min(wg_count, end - q0));
    if (at < 0) break;
    coef_item<PREC, G, 2, 2, 2>(a, smem, q0 + at, 0);
  }
}

template <int PREC, int G>
__global__ __launch_bounds__(CoefTile::NT, 2) void k_coef(FusedArgs a) {
  coef_pass<PREC, G>(a, blockIdx.x, gridDim.x);
}

// Launches that the host knows to be of few tiles: in halves where each then has
// a CU; up to two tiles per CU by four waves each.
constexpr int64_t kCoefFew = 128, kCoefMid = 512;
template <int PREC, int G>
__global__ __launch_bounds__(CoefTile::NT, 1) void k_coef_few(FusedArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int64_t n = min(a.work0 + a.coef_tiles, coef_work_count(a)) - a.work0;
  coef_halves<PREC, G, CoefTile::FEW_NS>(a, smem, n, blockIdx.x, gridDim.x);
}
template <int PREC, int G>
__global__ __launch_bounds__(2 * CoefTile::NT, 2) void k_coef_mid(FusedArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int64_t n = min(a.work0 + a.coef_tiles, coef_work_count(a)) - a.work0;
  const int64_t at = coef_place(blockIdx.x, gridDim.x, n);
  if (at >= 0) coef_item<PREC, G, 4, 1, CoefTile::MID_NS>(a, smem, a.work0 + at, 0);
}
// the most tiles that a launch may have to take
inline int64_t coef_most(const FusedArgs& a) {
  const int64_t left = (a.work_list ? a.n_work_list : a.n_tiles) - a.work0;
  return left < a.coef_tiles ? left : a.coef_tiles;
}

// one chunk's first half of several events
template <int PREC, int G>
__global__ __launch_bounds__(CoefTile::NT, 2) void k_coef_packed(PackLaunch p) {
  int64_t blk, nblk;
  int q;
  const int e = pack_locate(p, blockIdx.x, &blk, &nblk, &q);
  FusedArgs a = pack_args(p, e, q);
  a.work0 = p.chunk * a.coef_tiles;
  coef_pass<PREC, G>(a, blk, nblk);
}

}  // namespace dotpe
