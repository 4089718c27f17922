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
// 2048 tiles of 5-mode, 256-bin operands take 0.30 ms (0.36 to 0.38 in the
// fused kernel), if neighbouring tiles run together: with the list in the
// order in which it was written half of the reads missed L2 and it took as
// long as before.
#pragma once

#include "fused.h"

namespace dotpe {

struct CoefTile {
  static constexpr int NT = 128;
  static constexpr int STAGE = 16384;      // a chunk of A hi, A lo, B hi, B lo: 4 KB each
  static constexpr int LDS_BYTES = 2 * STAGE;
};

// One tile (BM = 2) or the 32 rows `half` of one (BM = 1) of work item q, by
// a workgroup of two waves, 32 BM x 32 pairs each.
template <int PREC, int G, int BM>
__device__ __forceinline__ void coef_item(const FusedArgs& a, unsigned char* smem, int64_t q, int half) {
  static_assert(PREC != kFP64, "split precisions only");
  typedef typename Pol<PREC>::Acc Acc;
  typedef __attribute__((address_space(1))) const unsigned char gbyte;
  typedef __attribute__((address_space(3))) void lvoid;
  constexpr int NRT = (G == 1) ? 1 : kMaxNR;
  constexpr int NCO = 2 * G + NRT, NPT = 64 * 64;
  constexpr int ES = 2;                      // bytes per operand element
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ndh = a.n_chunks;                // (d|h) chunks (groups of a multiple of 4), then NRT (h|h) blocks
  const int nk = ndh + NRT;
  const unsigned lds_wave =
      __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lvoid*)smem) + wave * 8192;

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
  // read k (0 .. NF - 1) of a chunk's fragments from stage P
  auto read_k = [&](Frag& f, auto pi, int k) {
    const unsigned char* st = smem + (decltype(pi)::value % 2) * CoefTile::STAGE + lane * 16;
    const int x = k % (2 * BM);
    if (k < 2 * BM) f.al[x >> 1][x & 1] = *(const uint4*)(st + 4096 + x * 1024);
    else if (k < 4 * BM) f.ah[x >> 1][x & 1] = *(const uint4*)(st + x * 1024);
    else if (k < 4 * BM + 2) f.bh[k & 1] = *(const uint4*)(st + 8192 + (2 * wave + (k & 1)) * 1024);
    else f.bl[k & 1] = *(const uint4*)(st + 12288 + (2 * wave + (k & 1)) * 1024);
  };
  auto fence = [] { __builtin_amdgcn_sched_barrier(0); };

  const int64_t t = coef_tile(a, q);
  const int64_t row0 = t / a.n_tiles_n * 64 + 32 * half, col0 = t % a.n_tiles_n * 64;
  float* cf = (float*)a.coef + (q - a.work0) * (int64_t)(NCO * NPT) + half * 32 * 64 + 32 * wave +
              (lane & 31);

  // ---- operand streams: wave 0 loads A, wave 1 B; of every chunk slices 0
  // and 1 of its 32-row blocks (A: BM, B: two), hi and lo, 1 KB each as it
  // sits in HBM (fragment order).  Rows past the subset re-read the last row
  // (their pairs are never used); columns run to the padded sample count. ----
  gbyte *p_hi[2] = {}, *p_lo[2] = {}, *h_hi[2] = {}, *h_lo[2] = {};
  auto blk = [](int64_t i, int64_t K) { return (i >> 5) * (K >> 5) * 1024 + (i & 31) * 8; };
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int r = 32 * b + (lane & 31);
    const int64_t in_chunk = (lane >> 5) * 256;
    if (wave == 0) {
      if (b >= BM) continue;
      const int64_t ie = min(row0 + r, a.n_sub - 1);
      const int64_t i = a.sub_idx ? a.sub_idx[ie] : a.sub0 + ie;
      const int64_t od = (blk(i, a.K2) + in_chunk) * ES, oh = (blk(ie, a.KH) + in_chunk) * ES;
      p_hi[b] = (gbyte*)a.A0 + od;
      p_lo[b] = (gbyte*)a.A1 + od;
      h_hi[b] = (gbyte*)a.Ah0 + oh;
      h_lo[b] = (gbyte*)a.Ah1 + oh;
    } else {
      const int64_t e = col0 + r;
      const int64_t od = (blk(e, a.K2) + in_chunk) * ES, oh = (blk(e, a.KH) + in_chunk) * ES;
      p_hi[b] = (gbyte*)a.B0 + od;
      p_lo[b] = (gbyte*)a.B1 + od;
      h_hi[b] = (gbyte*)a.Bh0 + oh;
      h_lo[b] = (gbyte*)a.Bh1 + oh;
    }
  }
  // the loads of the next chunk (c), into stage c mod 2: the immediate offset
  // applies to the global and the LDS address alike, so those of one array
  // share an M0 value.  The asm saves and restores M0 and waits the state an M0
  // write needs.
  auto issue = [&](int c) {
    const unsigned st = lds_wave + (unsigned)((c & 1) * CoefTile::STAGE);
    unsigned m0_saved;
    if (BM == 2 || wave == 1) {
      __asm__ __volatile__(
          "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
          "global_load_lds_dwordx4 %3, off\n\t"
          "global_load_lds_dwordx4 %3, off offset:1024\n\t"
          "global_load_lds_dwordx4 %4, off offset:2048\n\t"
          "global_load_lds_dwordx4 %4, off offset:3072\n\t"
          "s_mov_b32 m0, %2\n\ts_nop 0\n\t"
          "global_load_lds_dwordx4 %5, off\n\t"
          "global_load_lds_dwordx4 %5, off offset:1024\n\t"
          "global_load_lds_dwordx4 %6, off offset:2048\n\t"
          "global_load_lds_dwordx4 %6, off offset:3072\n\ts_mov_b32 m0, %0"
          : "=&s"(m0_saved)
          : "s"(__builtin_amdgcn_readfirstlane(st)), "s"(__builtin_amdgcn_readfirstlane(st + 4096)),
            "v"(p_hi[0]), "v"(p_hi[1] - 2048), "v"(p_lo[0]), "v"(p_lo[1] - 2048)
          : "memory");
    } else {
      __asm__ __volatile__(
          "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
          "global_load_lds_dwordx4 %3, off\n\t"
          "global_load_lds_dwordx4 %3, off offset:1024\n\t"
          "s_mov_b32 m0, %2\n\ts_nop 0\n\t"
          "global_load_lds_dwordx4 %4, off\n\t"
          "global_load_lds_dwordx4 %4, off offset:1024\n\ts_mov_b32 m0, %0"
          : "=&s"(m0_saved)
          : "s"(__builtin_amdgcn_readfirstlane(st)), "s"(__builtin_amdgcn_readfirstlane(st + 4096)),
            "v"(p_hi[0]), "v"(p_lo[0])
          : "memory");
    }
    // the sources step by one chunk (2 KB), and to the (h|h) operands after
    // the last (d|h) chunk
    const bool to_hh = c + 1 == ndh;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      p_hi[b] = to_hh ? h_hi[b] : p_hi[b] + 1024 * ES;
      p_lo[b] = to_hh ? h_lo[b] : p_lo[b] + 1024 * ES;
    }
  };

  // Step j (stage and fragment parity P = j mod 2): once every wave's loads
  // of chunk j + 1 have landed and every wave has read chunk j's fragments,
  // chunk j + 2 goes into that stage; then the products of chunk j (mf(f, k)
  // issues product k of NMF) with the reads of chunk j + 1 between them.
  auto step = [&](int j, auto pi, auto nmf, auto ahead, auto&& mf) {
    constexpr int P = decltype(pi)::value % 2, NMF = decltype(nmf)::value;
    constexpr int NR = decltype(ahead)::value ? NF : 0;
    Frag& cur = frag(std::integral_constant<int, P>{});
    Frag& nxt = frag(std::integral_constant<int, P + 1>{});
    if constexpr (NR > 0) {
      pipeline_barrier<0>();
      fence();
      if (j + 2 < nk) issue(j + 2);
      fence();
    }
    static_for<(NMF > NR ? NMF : NR)>([&](auto ti) {
      constexpr int x = decltype(ti)::value;
      if constexpr (x < NMF) mf(cur, x);
      if constexpr (x < NR) read_k(nxt, std::integral_constant<int, P + 1>{}, x);
    });
  };

  __syncthreads();       // (the last tile's stages are no longer read)
  issue(0);
  issue(1);
  pipeline_barrier<4 * BM>();   // chunk 0 has landed
  static_for<NF>([&](auto ki) { read_k(fr0, std::integral_constant<int, 0>{}, decltype(ki)::value); });

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

template <int PREC, int G>
__device__ __forceinline__ void coef_pass(const FusedArgs& a, int64_t wg_id, int64_t wg_count) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int64_t end = min(a.work0 + a.coef_tiles, coef_work_count(a));
  const int64_t n = end - a.work0;
  if (2 * n <= wg_count) {
    // a list that leaves half of the workgroups idle: half a tile each, the
    // halves of a tile on one XCD
    const int64_t part = (n + 7) / 8, y = wg_id / 8;
    int64_t at = wg_id / 2, half = wg_id & 1;
    if (16 * part <= wg_count) {
      at = y / 2 < part ? wg_id % 8 * part + y / 2 : n;
      half = y & 1;
    }
    if (at < n) coef_item<PREC, G, 1>(a, smem, a.work0 + at, (int)half);
    return;
  }
#pragma unroll 1
  for (int64_t q0 = a.work0; q0 < end; q0 += wg_count) {
    const int64_t at = coef_place(wg_id, wg_count, min(wg_count, end - q0));
    if (at < 0) break;
    coef_item<PREC, G, 2>(a, smem, q0 + at, 0);
  }
}

template <int PREC, int G>
__global__ __launch_bounds__(CoefTile::NT, 2) void k_coef(FusedArgs a) {
  coef_pass<PREC, G>(a, blockIdx.x, gridDim.x);
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
