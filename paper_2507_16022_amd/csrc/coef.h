// First half of the coefficient route for split precisions: the raw
// accumulators of every pair of the listed 64 x 64 tiles, stored for the
// kernels that bound and marginalise them.
//
// An accumulator is complete when its m group's chunks (or its (h|h) block)
// are, so it is stored there and then and a wave needs one group's at a time:
// 32 x 32 pairs per wave in 32 accumulator registers (the fused kernel holds all
// 240 until its epilogue, one wave per SIMD).  A workgroup of four waves takes a
// tile, with four stages of 16 KB in LDS, and two share a CU: a chunk's loads have
// the products of three others to arrive in, and sit between them (in front of
// them they kept the matrix cores waiting).  An event of at most 128 tiles is taken
// in halves of 32 rows by two waves each, with six stages (more halves than CUs
// would load 24 KB per chunk and CU, all that a CU's share of L2 gives it; a tile
// 16).
//
// ln L matrices of one phase, five modes, in ms by tiles; in brackets the fused
// kernel (four waves, eight stages, one workgroup per CU), then 64 x 32 pairs per
// wave with two stages and four workgroups per CU (what this replaced), now:
//   256 bins: 64 tiles (0.094, 0.070) 0.061, 256 (0.097, 0.109) 0.093, 600 (0.257,
//     0.242) 0.182, 4096 (1.27, 1.24) 1.18
//   1700 bins: 1 (0.201, 0.242) 0.187, 200 (0.227, 0.324) 0.238, 1024 (0.93, 1.01)
//     0.88, 4096 (3.59, 4.12) 3.47
// Neighbouring tiles have to run together: with the list in the order in which it
// was written half of the reads missed L2.
#pragma once

#include "fused.h"

namespace dotpe {

// bytes of a chunk of 32 rb rows: A hi, A lo (2 KB per 32 rows each), B hi, B lo
// (4 KB each)
constexpr int coef_stage(int rb) { return rb * 4096 + 8192; }
struct CoefTile {
  static constexpr int NT = 256, NS = 4;             // a tile by four waves
  static constexpr int HALF_NT = 128, HALF_NS = 6;   // half of one by two
  static constexpr int LDS_BYTES = NS * coef_stage(2), HALF_BYTES = HALF_NS * coef_stage(1);
  static_assert(LDS_BYTES <= 64 * 1024, "no attribute, two workgroups per CU");
};

// Work item q, by a workgroup of NW waves, 32 x 32 pairs each, with NS stages: the
// tile (four waves) or the 32 rows `half` of it (two).
template <int PREC, int G, int NW, int NS>
__device__ __forceinline__ void coef_item(const FusedArgs& a, unsigned char* smem, int64_t q, int half) {
  static_assert(PREC != kFP64, "split precisions only");
  static_assert(NW == 2 || NW == 4, "a tile or half of one");
  typedef typename Pol<PREC>::Acc Acc;
  typedef __attribute__((address_space(1))) const unsigned char gbyte;
  typedef __attribute__((address_space(3))) void lvoid;
  constexpr int NRT = (G == 1) ? 1 : kMaxNR;
  constexpr int NCO = 2 * G + NRT, NPT = 64 * 64;
  constexpr int ES = 2;                      // bytes per operand element
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ndh = a.n_chunks;                // (d|h) chunks (groups of a multiple of 4), then NRT (h|h) blocks
  const int nk = ndh + NRT;
  constexpr int STAGE = coef_stage(NW / 2), ALO = 1024 * NW, BHI = 2 * ALO, BLO = BHI + 4096;
  const int wm = wave >> 1, wn = wave & 1;   // the wave's rows (of a tile) and columns

  // fragments of one chunk, [slice]
  struct Frag {
    uint4 ah[2], al[2], bh[2], bl[2];
  };
  constexpr int NF = 8;
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
    const int sl = k & 1;
    if (k < 2) f.al[sl] = *(const uint4*)(st + ALO + (2 * wm + sl) * 1024);
    else if (k < 4) f.ah[sl] = *(const uint4*)(st + (2 * wm + sl) * 1024);
    else if (k < 6) f.bh[sl] = *(const uint4*)(st + BHI + (2 * wn + sl) * 1024);
    else f.bl[sl] = *(const uint4*)(st + BLO + (2 * wn + sl) * 1024);
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
  // A wave's loads: a tile's waves have a stream of A and one of B each; of half a
  // tile's each has one part of A and its block of B, hi and lo.
  constexpr int NSTR = NW == 4 ? 2 : 3, LPW = 2 * NSTR;
  Stream str[NSTR];
  unsigned place[NSTR];        // its LDS address in stage 0
  const unsigned lds0 = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lvoid*)smem);
  if constexpr (NW == 4) {
    str[0] = stream(true, wn, wm);
    str[1] = stream(false, wn, wm);
    place[0] = lds0 + wm * ALO + wn * 2048;
    place[1] = lds0 + BHI + wm * (BLO - BHI) + wn * 2048;
  } else {
    str[0] = stream(true, 0, wn);
    str[1] = stream(false, wn, false);
    str[2] = stream(false, wn, true);
    place[0] = lds0 + wn * ALO;
    place[1] = lds0 + BHI + wn * 2048;
    place[2] = lds0 + BLO + wn * 2048;
  }
  // stream t of the next chunk (c), into the stage at st
  auto issue_part = [&](int c, unsigned st, auto ti) {
    constexpr int t = decltype(ti)::value;
    unsigned m0_saved;
    __asm__ __volatile__(
        "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
        "global_load_lds_dwordx4 %2, off\n\t"
        "global_load_lds_dwordx4 %2, off offset:1024\n\ts_mov_b32 m0, %0"
        : "=&s"(m0_saved)
        : "s"(__builtin_amdgcn_readfirstlane(place[t] + st)), "v"(str[t].p)
        : "memory");
    str[t].p += 1024 * ES;
    if (__builtin_expect(c + 1 == ndh, 0)) str[t].p = str[t].hh;
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
  // chunk j's fragments, the products of chunk j (mf(f, k) issues product k of NMF)
  // with the reads of chunk j + 1 and then the loads of chunk j + NS, into the
  // stage of chunk j, between them.
  auto step = [&](int j, auto pi, auto nmf, auto ahead, auto&& mf) {
    constexpr int P = decltype(pi)::value % 2, NMF = decltype(nmf)::value;
    constexpr int NR = decltype(ahead)::value ? NF : 0;
    Frag& cur = frag(std::integral_constant<int, P>{});
    Frag& nxt = frag(std::integral_constant<int, P + 1>{});
    if constexpr (NR > 0) {
      if (j + NS <= nk) pipeline_barrier<(NS - 2) * LPW>();
      else barrier(nk - 2 - j);
      fence();
    }
    const unsigned nxt_st = after(cur_st);
    static_for<(NMF > NR ? NMF : NR)>([&](auto ti) {
      constexpr int x = decltype(ti)::value;
      if constexpr (x < NMF) mf(cur, x);
      if constexpr (x < NR) read_k(nxt, nxt_st, x);
      if constexpr (NR > 0 && x >= NMF - 4 && x < NMF - 4 + NSTR) {
        fence();
        if (j + NS < nk) issue_part(j + NS, cur_st, std::integral_constant<int, x - (NMF - 4)>{});
        fence();
      }
    });
    cur_st = nxt_st;
  };

  __syncthreads();       // (the last tile's stages are no longer read)
  static_for<NS>([&](auto ci) {
    constexpr int c = decltype(ci)::value;
    if (c < nk) static_for<NSTR>([&](auto ti) { issue_part(c, c * STAGE, ti); });
  });
  barrier(min(NS, nk) - 1);     // chunk 0 has landed
  static_for<NF>([&](auto ki) { read_k(fr0, 0, decltype(ki)::value); });

  // component c of the wave's pairs from its accumulator
  auto store = [&](int c, const Acc& v) {
#pragma unroll
    for (int e = 0; e < 16; ++e)
      cf[c * NPT + (8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)) * 64] = v[e];
  };

  // ---- (d|h), a group at a time.  With A = [hr | hi] and B_re = [Br | -Bi]
  // by slice, re += A B_re and im += A B_im, B_im = [Bi | Br] = [-(B_re
  // slice 1) | B_re slice 0]; 3 split products per real product, the smaller
  // ones first, re and im alternating (each accumulator's products in the
  // fused kernel's order, so their sums are its sums). ----
  int ch = 0;
  static_for<G>([&](auto gi) {
    constexpr int g = decltype(gi)::value;
    Acc re, im;
    const int gend = a.mt.gk0[g + 1];
    auto dh = [&](auto pi, auto first) {
      const Frag& f = frag(pi);
      auto neg = [](const uint4& x) {
        return make_uint4(x.x ^ 0x80008000u, x.y ^ 0x80008000u, x.z ^ 0x80008000u, x.w ^ 0x80008000u);
      };
      const uint4 nbh = neg(f.bh[1]), nbl = neg(f.bl[1]);
      step(ch, pi, std::integral_constant<int, 12>{}, std::true_type{}, [&](const Frag& f, int k) {
        if constexpr (decltype(first)::value) {
          if (k == 0) re = Acc{};
          if (k == 1) im = Acc{};
        }
        switch (k) {
          case 0: mma<PREC>(re, f.al[0], f.bh[0]); break;
          case 1: mma<PREC>(im, f.al[0], nbh); break;
          case 2: mma<PREC>(re, f.ah[0], f.bl[0]); break;
          case 3: mma<PREC>(im, f.ah[0], nbl); break;
          case 4: mma<PREC>(re, f.ah[0], f.bh[0]); break;
          case 5: mma<PREC>(im, f.ah[0], nbh); break;
          case 6: mma<PREC>(re, f.al[1], f.bh[1]); break;
          case 7: mma<PREC>(im, f.al[1], f.bh[0]); break;
          case 8: mma<PREC>(re, f.ah[1], f.bl[1]); break;
          case 9: mma<PREC>(im, f.ah[1], f.bl[0]); break;
          case 10: mma<PREC>(re, f.ah[1], f.bh[1]); break;
          default: mma<PREC>(im, f.ah[1], f.bh[0]); break;
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
    store(2 * g, re);
    store(2 * g + 1, im);
  });
  // ---- (h|h) block r: the real product of the row and column operands ----
  static_for<NRT>([&](auto ri) {
    constexpr int r = decltype(ri)::value;
    Acc h = {};
    step(ndh + r, ri, std::integral_constant<int, 6>{}, std::bool_constant<(r + 1 < NRT)>{},
         [&](const Frag& f, int x) {
           const int sl = x / 3;
           switch (x % 3) {
             case 0: mma<PREC>(h, f.al[sl], f.bh[sl]); break;
             case 1: mma<PREC>(h, f.ah[sl], f.bl[sl]); break;
             default: mma<PREC>(h, f.ah[sl], f.bh[sl]); break;
           }
         });
    store(2 * G + r, h);
  });
}

// the chunk's tiles, the workgroups in turn
template <int PREC, int G>
__device__ __forceinline__ void coef_pass(const FusedArgs& a, int64_t wg_id, int64_t wg_count) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int64_t end = min(a.work0 + a.coef_tiles, coef_work_count(a));
#pragma unroll 1
  for (int64_t q0 = a.work0; q0 < end; q0 += wg_count) {
    const int64_t at = coef_place(wg_id, wg_count, min(wg_count, end - q0));
    if (at < 0) break;
    coef_item<PREC, G, 4, CoefTile::NS>(a, smem, q0 + at, 0);
  }
}

template <int PREC, int G>
__global__ __launch_bounds__(CoefTile::NT, 2) void k_coef(FusedArgs a) {
  coef_pass<PREC, G>(a, blockIdx.x, gridDim.x);
}

// Launches of few tiles, in halves: two workgroups for each of the most tiles that
// the launch may have to take (known to the host), the two of a tile on one XCD.
constexpr int64_t kCoefFew = 128;
inline int64_t coef_most(const FusedArgs& a) {
  const int64_t left = (a.work_list ? a.n_work_list : a.n_tiles) - a.work0;
  return left < a.coef_tiles ? left : a.coef_tiles;
}
template <int PREC, int G>
__global__ __launch_bounds__(CoefTile::HALF_NT, 1) void k_coef_few(FusedArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int64_t n = min(a.work0 + a.coef_tiles, coef_work_count(a)) - a.work0;
  const int64_t wg_id = blockIdx.x, part = (n + 7) / 8, y = wg_id / 8;
  int64_t at = wg_id / 2, half = wg_id & 1;
  if (16 * part <= (int64_t)gridDim.x) {
    at = y / 2 < part ? wg_id % 8 * part + y / 2 : n;
    half = y & 1;
  }
  if (at < n) coef_item<PREC, G, 2, CoefTile::HALF_NS>(a, smem, a.work0 + at, (int)half);
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
