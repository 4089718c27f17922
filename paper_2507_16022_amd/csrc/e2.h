// Second half of the coefficient route of an evidence pass.  The first half
// (k_coef; for FP64 banks the fused kernel in mode kCoef) has stored the raw
// accumulators of every pair of the chunk's tiles; this kernel bounds (E1) and
// evaluates (E2: per-phase distance marginalisation, eq. lnl_dist_marginalized,
// and the phase average) every pair and writes each tile's partial.  Apart from
// the accumulators it holds a handful of doubles per lane, so several waves share
// every SIMD and hide the latency of the distance rule's table reads, which the
// fused kernel, one wave per SIMD, cannot.  The (i, e) matrix of ln L is written
// by the same kernel without the cut and the sums.
#pragma once

#include "fused.h"

namespace dotpe {

// Per-row and per-column scalars of a tile into LDS, as the fused kernel
// forms them: rowd [TM][4] (ln w_i, row scale, (h|h) row scale, bank row),
// cold [TN][3] (ln w_e, column scale, (h|h) column scale), rowq [TM][2]
// (row scale^2 / (h|h) row scale, ln w_i).  Threads 0 .. TM + TN - 1 write.
template <int PREC, int TM, int TN>
__device__ __forceinline__ void e2_scalars(const FusedArgs& a, int64_t row0, int64_t col0,
                                           double* rowd, double* cold, double* rowq) {
  const int tid = threadIdx.x;
  if (tid < TM) {
    double rv0 = 0.0, rv1 = 1.0, rv2 = 1.0, rv3 = -1.0;
    const int64_t ie = row0 + tid;
    if (ie < a.n_sub) {
      const int64_t i = a.sub_idx ? a.sub_idx[ie] : a.sub0 + ie;
      rv0 = a.ln_w_bank ? a.ln_w_bank[i] : 0.0;
      rv1 = PREC == kFP64 ? 1.0 : a.row_scale[i];
      rv2 = PREC == kFP64 ? 1.0 : a.ah_scale[ie];
      rv3 = (double)i;
    }
    rowd[tid * 4] = rv0; rowd[tid * 4 + 1] = rv1; rowd[tid * 4 + 2] = rv2; rowd[tid * 4 + 3] = rv3;
    rowq[tid * 2] = rv1 * rv1 / rv2;
    rowq[tid * 2 + 1] = rv0;
  } else if (tid < TM + TN) {
    double cv0 = 0.0, cv1 = 1.0, cv2 = 1.0;
    const int64_t e = col0 + (tid - TM);
    if (e < a.n_ext) {
      cv0 = a.ln_w_ext ? a.ln_w_ext[e] : 0.0;
      cv1 = PREC == kFP64 ? 1.0 : a.col_scale[e];
      cv2 = PREC == kFP64 ? 1.0 : a.bh_scale[e];
    }
    cold[(tid - TM) * 3] = cv0; cold[(tid - TM) * 3 + 1] = cv1; cold[(tid - TM) * 3 + 2] = cv2;
  }
}

// The stored accumulators of one pair and the quantities E1 and E2 take
// from them.
template <typename AT, int G, int NRT>
struct PairCoef {
  AT x[2 * G], sv[NRT];
  template <int NPT>
  __device__ __forceinline__ void load(const AT* cf, int p) {
#pragma unroll
    for (int c = 0; c < 2 * G; ++c) x[c] = cf[c * NPT + p];
#pragma unroll
    for (int c = 0; c < NRT; ++c) sv[c] = cf[(2 * G + c) * NPT + p];
  }
  // E1: the certified bound on lnL^ML, the same arithmetic as the fused
  // kernel's epilogue on the same accumulators; true when the pair is
  // bounded (below thr_f), with the bound and ln w_ie in FP32
  __device__ __forceinline__ bool bounded(const double* rowq, const double* cold, int tr, int tc,
                                          float thr_f, float& bound, float& lw) const {
    float U0 = 0.f;
#pragma unroll
    for (int g = 0; g < G; ++g) {
      const float xr = (float)x[2 * g], xi = (float)x[2 * g + 1];
      U0 += __builtin_amdgcn_sqrtf(xr * xr + xi * xi);
    }
    const float s0 = (float)sv[0];
    float sabs = 0.f;
#pragma unroll
    for (int d = 1; d < (NRT + 1) / 2; ++d) {
      const float sr = (float)sv[2 * d - 1], si = (float)sv[2 * d];
      sabs += 2.f * __builtin_amdgcn_sqrtf(sr * sr + si * si);
    }
    const float lo0 = (s0 - sabs) - 2e-5f * (fabsf(s0) + sabs);
    const double colq = cold[tc * 3 + 1] * cold[tc * 3 + 1] / cold[tc * 3 + 2];
    const float qf = (float)(rowq[tr * 2] * colq);
    bound = qf * (U0 * U0) * __builtin_amdgcn_rcpf(2.f * lo0) * 1.001f + 1e-3f;
    lw = (float)(rowq[tr * 2 + 1] + cold[tc * 3]);
    return lo0 > 0.f && bound < thr_f;
  }
  // E2 inputs: X_g and the (h|h) phase coefficients at d0, ln w_ie
  __device__ __forceinline__ void unscale(const double* rowd, const double* cold, int tr, int tc,
                                          double2 (&X)[G], double& S0, double (&Sr)[kMaxND],
                                          double (&Si)[kMaxND], double& lnw) const {
    const double sx = rowd[tr * 4 + 1] * cold[tc * 3 + 1];
    const double sh = rowd[tr * 4 + 2] * cold[tc * 3 + 2];
#pragma unroll
    for (int g = 0; g < G; ++g) X[g] = make_double2(sx * (double)x[2 * g], sx * (double)x[2 * g + 1]);
    S0 = sh * (double)sv[0];
#pragma unroll
    for (int d = 0; d < kMaxND; ++d) { Sr[d] = 0.0; Si[d] = 0.0; }
#pragma unroll
    for (int d = 1; d < (NRT + 1) / 2; ++d) {
      Sr[d] = sh * (double)sv[2 * d - 1];
      Si[d] = sh * (double)sv[2 * d];
    }
    lnw = rowd[tr * 4] + cold[tc * 3];
  }
};

// The pairs that E1 leaves, a wave's batch of up to 64 at a time, in three
// steps, each with the lanes full whatever the cut leaves:
//  - a pair per lane: which phases the cut keeps (a mask), the cut phases'
//    bounds and the largest lnL^ML, from the pair's coefficients in registers
//    and the phase table in scalar registers;
//  - a kept phase per lane, the pairs' phases in order: the distance rule.  Its
//    table reads are bound by the rate at which a CU's L1 serves gathered
//    lines (64 lanes at random: ~150 cycles per load of 16 bytes, within a few
//    lines: ~25), and the phases of one pair fall into few lines;
//  - a pair per lane: the running sum over its kept phases, in order.
// Where a posterior is broad, one pair in ten survives E1 and one phase in
// ten of a survivor the cut: with a lane per pair of the tile and every phase
// in its loop (as before), the wave took each step that any lane needed.  At
// 30011 x 3001 pairs and 32 phases a pass with every phase kept went from 52.4
// to 36.1 ms (8.0e10 triples/s, its FP64 instructions 60% of the cycles), at
// 8192 x 4096 pairs with 11% and 7% kept this kernel from 5.1 to 2.0 ms.  (A
// phase per lane throughout, with scans for the running sums, took 45 ms and
// 6.4 ms.)
//
// Slot of a pair in its wave's batch: the accumulators, the pair's place in
// the tile (in the last element before the scales), and the two scales as
// doubles (FP32 accumulators; FP64 ones carry none).  An odd number of
// 16-byte units, so that consecutive slots start in different banks.
template <typename AT, int NCO>
struct PairSlot {
  static constexpr int U = 16 / (int)sizeof(AT);
  static constexpr int CP = (NCO + 1 + U - 1) / U * U;
  static constexpr int UNITS = CP / U + (sizeof(AT) == 4 ? 1 : 0);
  static constexpr int STRIDE = (UNITS | 1) * U;
};

// Kept phases per wave and turn of the distance rule: as LDS allows three
// workgroups per CU.  FP64 slots of four m groups are larger: 192 leave room for
// three (64 x 20000 pairs, 32 phases, all kept: this kernel 0.98 ms with 256 and
// two workgroups, 0.76 with 192), but not beside the phase table of 64 phases and
// more (3000 x 3000, 128 phases a call of 21.3 ms with 256, 23.3 with 192), nor is
// a third used by an event of two tiles per CU (64 x 64 pairs 0.56 against 0.61
// ms a call).
// Split banks: 512, and 384 in a pass of three or four m groups whose phase table
// would not fit beside that three times (MANY: 520 tiles of 100 phases, all kept,
// an evidence call of 4.78 ms with 512 and two workgroups per CU, 3.58 with 384;
// 1920 tiles 10.3 and 8.9; but 256 tiles, which two per CU take in one round, 2.41
// and 2.55).
template <int PREC, int G, bool MANY = false>
__host__ __device__ constexpr int e2_turn(int n_phi, bool few_tiles) {
  return PREC != kFP64 ? (MANY ? 384 : 512) : G == kMaxG && n_phi < 64 && !few_tiles ? 192 : 256;
}
template <int PREC, int G>
constexpr bool e2_many(int n_phi, bool few_tiles) { return PREC != kFP64 && G >= 3 && n_phi > 78 && !few_tiles; }
__host__ __device__ constexpr bool e2_few(int64_t n_tiles) { return n_tiles <= 512; }
constexpr int kE2Waves = 4;
// bytes of its dynamic LDS: the phase table, then for FP64 per wave a turn's
// ln Lbar and places (those of split banks, whose turns have one length, at fixed
// addresses)
template <int PREC, int G>
constexpr size_t e2_lds(int n_phi, bool few_tiles) {
  const size_t turn = PREC == kFP64 ? e2_turn<PREC, G>(n_phi, few_tiles) : 0;
  return sizeof(double) * kMaxM * (size_t)n_phi * 2 + kE2Waves * turn * (sizeof(double) + sizeof(uint16_t));
}

// MODE kEvidence: the second half of an evidence pass; kEval: every pair's
// ln L (and largest lnL^ML, and triples) of the tiles from work0 on.
template <int PREC, int G, int MODE, bool MANY = false>
__device__ __forceinline__ void e2_pass(const FusedArgs& a, bool few_tiles, int64_t wg_id, int64_t wg_count) {
  typedef Tile<PREC> TL;
  typedef typename std::conditional<PREC == kFP64, double, float>::type AT;
  constexpr bool EVAL = MODE == kEval;
  constexpr int NRT = (G == 1) ? 1 : kMaxNR;
  constexpr int NCO = 2 * G + NRT;
  constexpr int TM = TL::TM, TN = TL::TN, NPT = TM * TN, NT = 256, NW = kE2Waves, NK = NPT / NT;
  static_assert(NT == 64 * NW && NPT % NT == 0 && (TN == 64 || TN == 32), "whole rows per wave");
  constexpr int PARTS = EVAL ? kEvalParts : 1;
  static_assert(NK % PARTS == 0, "whole turns per part");
  typedef PairSlot<AT, NCO> SL;
  extern __shared__ __align__(16) double lds_cs[];     // [kMaxM][n_phi][2]
  __shared__ DistParams dp;
  __shared__ double rowd[TM * 4], cold[TN * 3], rowq[TM * 2], red[NW * kNPart];
  __shared__ __align__(16) AT slots[NW][64 * SL::STRIDE];
  // sums of the waves' e^(ln p - m) by row and by column, m the wave's largest
  // ln p so far
  __shared__ double rsum[TM], csum[NW][TN], wmax[NW];
  __shared__ unsigned long long tile_lnp_max;
  static_assert(kMaxPhi <= 256, "a phase in 8 bits");

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_phi = a.n_phi;
  for (int t = tid; t < kMaxM * n_phi * 2; t += NT) lds_cs[t] = a.phase_cs[t];
  static_assert(sizeof(DistParams) % 4 == 0, "DistParams words");
  for (int t = tid; t < (int)(sizeof(DistParams) / 4); t += NT)
    ((unsigned*)&dp)[t] = ((const unsigned*)a.dist.prm)[t];
  // the phase table again, for wave-uniform reads
  typedef const double __attribute__((address_space(4))) cdouble;
  cdouble* cs_u = (cdouble*)(uintptr_t)a.phase_cs;
  // the cut as the fused kernel's epilogue applies it
  const bool on = !EVAL && cut_on(a);
  const double thr_ml = on ? __longlong_as_double(a.state[3]) - a.cut_delta : -INFINITY;
  const double thr2 = 2.0 * thr_ml;
  const float thr_f = (float)thr_ml;
  const int64_t end = min(a.work0 + a.coef_tiles, coef_work_count(a));
  AT* const my_slots = slots[wave];
  // per wave ln Lbar of the turn's kept phases, and their slot << 8 | phase
  const int CH = e2_turn<PREC, G, MANY>(n_phi, few_tiles);
  constexpr int FIX = PREC == kFP64 ? 1 : e2_turn<PREC, G, MANY>(0, false);
  __shared__ double val_fix[NW][FIX];
  __shared__ uint16_t ent_fix[NW][FIX];
  double* const val = lds_cs + kMaxM * n_phi * 2;
  double* const my_val = PREC == kFP64 ? val + wave * CH : val_fix[wave];
  uint16_t* const my_ent = PREC == kFP64 ? (uint16_t*)(val + NW * CH) + wave * CH : ent_fix[wave];

  // a pair's coefficients and scales from its slot
  struct Coef {
    double2 X[G];
    double S0, Sr[kMaxND], Si[kMaxND], sx, sh;
    int place;
  };
  auto read_slot = [&](int s, Coef& c) {
    const AT* q = my_slots + s * SL::STRIDE;
    AT v[SL::CP];
#pragma unroll
    for (int u = 0; u < SL::CP; u += SL::U) {
      typedef AT VT __attribute__((ext_vector_type(SL::U)));
      const VT w = *(const VT*)(q + u);
#pragma unroll
      for (int x = 0; x < SL::U; ++x) v[u + x] = w[x];
    }
#pragma unroll
    for (int g = 0; g < G; ++g) c.X[g] = make_double2((double)v[2 * g], (double)v[2 * g + 1]);
    c.S0 = (double)v[2 * G];
#pragma unroll
    for (int d = 0; d < kMaxND; ++d) { c.Sr[d] = 0.0; c.Si[d] = 0.0; }
#pragma unroll
    for (int d = 1; d < (NRT + 1) / 2; ++d) {
      c.Sr[d] = (double)v[2 * G + 2 * d - 1];
      c.Si[d] = (double)v[2 * G + 2 * d];
    }
    c.place = *(const int*)(q + SL::CP - 1);
    if constexpr (PREC == kFP64) {
      c.sx = c.sh = 1.0;
    } else {
      const double2 w = *(const double2*)(q + SL::CP);
      c.sx = w.x;
      c.sh = w.y;
    }
  };
  auto wave_sync = [] {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };

  for (int64_t w = wg_id; w < (end - a.work0) * PARTS; w += wg_count) {
    const int64_t q = a.work0 + w / PARTS;
    const int part = (int)(w % PARTS);
    const int64_t t = coef_tile(a, q);
    const int64_t tm = t / a.n_tiles_n, tn = t % a.n_tiles_n;
    const int64_t row0 = tm * TM, col0 = tn * TN;
    e2_scalars<PREC, TM, TN>(a, row0, col0, rowd, cold, rowq);
    if (tid == 0) tile_lnp_max = 0ull;
    if (tid < TM) rsum[tid] = 0.0;
    if (lane < TN) csum[wave][lane] = 0.0;
    __syncthreads();
    const double thr_topk_glob = EVAL ? 0.0 : order_value(a.state[1]) - a.topk_window;
    const int rows_in = (int)min((int64_t)TM, a.n_sub - row0);
    const int cols_in = (int)min((int64_t)TN, a.n_ext - col0);
    const AT* cf = (const AT*)a.coef + (q - a.work0) * (int64_t)(NCO * NPT);
    EvAcc ev;
    ev.init();
    int n_pairs_i = 0, n_bounded_i = 0;
    double wm = -INFINITY;
    const int k1 = (part + 1) * (NK / PARTS);
    int k = part * (NK / PARTS);
#pragma unroll 1
    for (;;) {
      // fill the batch: consecutive pairs of a row per wave, coalesced
      // component reads; a turn whose survivors do not fit is read again for
      // the next batch (held in registers instead, or asked for a turn ahead,
      // it was 5% slower)
      int used = 0;
#pragma unroll 1
      for (; k < k1 && used < 64; ++k) {
        const int p = k * NT + tid, tr = p / TN, tc = p % TN;
        const bool in = tr < rows_in && tc < cols_in;
        PairCoef<AT, G, NRT> pc;
        pc.template load<NPT>(cf, p);
        float bound = 0.f, lw = 0.f;
        const bool bounded = on && pc.bounded(rowq, cold, tr, tc, thr_f, bound, lw) && in;
        const bool live = in && !bounded;
        const unsigned long long lv = __ballot(live);
        const int n_live = (int)__popcll(lv);
        if (used + n_live > 64) break;
        n_pairs_i += in ? 1 : 0;
        if (on) {
          ev.drop.add(bounded ? lw + bound : -INFINITY);
          ev.max_bound = bounded ? fmaxf(ev.max_bound, lw + bound) : ev.max_bound;
          n_bounded_i += bounded ? 1 : 0;
        }
        if (live) {
          AT* o = my_slots + SL::STRIDE * (used + (int)__builtin_amdgcn_mbcnt_hi(
                                                      (unsigned)(lv >> 32),
                                                      __builtin_amdgcn_mbcnt_lo((unsigned)lv, 0u)));
#pragma unroll
          for (int c = 0; c < 2 * G; ++c) o[c] = pc.x[c];
#pragma unroll
          for (int c = 0; c < NRT; ++c) o[2 * G + c] = pc.sv[c];
          *(int*)(o + SL::CP - 1) = p;
          if constexpr (PREC != kFP64)
            *(double2*)(o + SL::CP) = make_double2(rowd[tr * 4 + 1] * cold[tc * 3 + 1],
                                                   rowd[tr * 4 + 2] * cold[tc * 3 + 2]);
        }
        used += n_live;
      }
      if (!used) break;
      wave_sync();
      const bool act = lane < used;
      int tr, tc, ob = 0;
      double lnw, mn = 0.0, md = 1.0;
      LsePh lse;
      lse.init();
      {
        const int place = *(const int*)(my_slots + (act ? lane : 0) * SL::STRIDE + SL::CP - 1);
        tr = place / TN;
        tc = place % TN;
        lnw = rowd[tr * 4] + cold[tc * 3];
      }
      // phases in blocks of 32, or of 16 where all are kept: 64 pairs then fill
      // two turns, and half of the lanes have a pair in each turn's sums
      const int blk = on ? 32 : 16;
#pragma unroll 1
      for (int o0 = 0; o0 < n_phi; o0 += blk) {
        const int no = min(blk, n_phi - o0);
        unsigned mask = act ? (no == 32 ? ~0u : (1u << no) - 1u) : 0u;
        // a pair per lane
        if (!EVAL || a.ml_out) {
          Coef c;
          read_slot(act ? lane : 0, c);
          unsigned keeps = 0u;
#pragma unroll 1
          for (int b = 0; b < no; ++b) {
            double dh, hh;
            phase_dh_hh<G>(a.mt.gm, n_phi, cs_u, c.X, c.S0, c.Sr, c.Si, o0 + b, dh, hh);
            dh *= c.sx;
            hh *= c.sh;
            const bool pos = dh > 0.0 && hh > 0.0;
            const double dh2 = dh * dh;
            const bool more = pos && dh2 * md > mn * hh;
            mn = more ? dh2 : mn;
            md = more ? hh : md;
            if (on) {
              // lnL^ML >= thr  <=>  dh > 0 and dh^2 >= 2 thr hh (no division)
              const bool keep = thr_ml <= 0.0 || (dh > 0.0 && dh2 >= thr2 * hh);
              keeps |= keep ? 1u << b : 0u;
              double ml = 0.0;
              if (pos) ml = hh > 0x1p-900 && hh < 0x1p900 ? dh2 * dr_rcp(2.0 * hh) : dh2 / (2.0 * hh);
              const float x = (float)(lnw + ml - a.ln_nphi);
              // (the rounding margin keeps it a bound)
              ev.drop.add(act && !keep ? x + fabsf(x) * 1e-6f + 1e-5f : -INFINITY);
            }
          }
          if (on) mask &= keeps;
        }
        // the kept phases' places, pair by pair
        const int cnt = __popc(mask);
        if (!EVAL) ev.n_marg += cnt;
        int incl = cnt;
        incl += (int)dpp_mov<0x111, 0xF>(0u, (unsigned)incl);   // row_shr:1, 2, 4, 8
        incl += (int)dpp_mov<0x112, 0xF>(0u, (unsigned)incl);
        incl += (int)dpp_mov<0x114, 0xF>(0u, (unsigned)incl);
        incl += (int)dpp_mov<0x118, 0xF>(0u, (unsigned)incl);
        incl += (int)dpp_mov<0x142, 0xA>(0u, (unsigned)incl);   // row_bcast:15, 31
        incl += (int)dpp_mov<0x143, 0xC>(0u, (unsigned)incl);
        const int off = incl - cnt, total = __builtin_amdgcn_readlane(incl, 63);
        int at = off;
        const unsigned inv_no = (65536u + no - 1) / no;
#pragma unroll 1
        for (int c0 = 0; c0 < total; c0 += CH) {
          const int c1 = min(c0 + CH, total);
          const int lo = at;
          if (on) {
            while (mask && at < c1) {
              my_ent[at - c0] = (uint16_t)(lane << 8 | (o0 + __builtin_ctz(mask)));
              mask &= mask - 1u;
              ++at;
            }
            wave_sync();
          } else {
            at = max(at, min(off + cnt, c1));
          }
          // a kept phase per lane
#pragma unroll 1
          for (int e0 = c0; e0 < c1; e0 += 64) {
            const int e = e0 + lane, ec = min(e, c1 - 1);
            int src, o;
            if (on) {
              const unsigned en = my_ent[ec - c0];
              src = (int)(en >> 8);
              o = (int)(en & 255u);
            } else {
              src = (int)((unsigned)ec * inv_no >> 16);      // ec / no (ec < 2^10, no <= 16)
              o = o0 + ec - src * no;
            }
            Coef c;
            read_slot(src, c);
            double dh, hh, v;
            phase_dh_hh<G>(a.mt.gm, n_phi, (const double*)lds_cs, c.X, c.S0, c.Sr, c.Si, o, dh, hh);
            dh *= c.sx;
            hh *= c.sh;
            if (EVAL && a.trip_out && e < c1) {
              const size_t to = (((size_t)(row0 + c.place / TN) * a.n_ext + (col0 + c.place % TN)) *
                                     n_phi + o) * 2;
              a.trip_out[to] = dh;
              a.trip_out[to + 1] = hh;
            }
            if (!dr_ln_marg_try(dh, hh, a.r0, a.dist.tab, dp.ghx, dp.ghw, v))
              v = dr_ln_marg(dh, hh, a.r0, a.dist.tab, dp.ghx, dp.ghw);
            if (e < c1) my_val[e - c0] = v;
          }
          wave_sync();
          // a pair per lane: its phases of this turn, in order
          int jb = -1;
          for (int j = lo; j < at; ++j) jb = lse.add(my_val[j - c0]) ? j : jb;
          if (jb >= 0) ob = on ? my_ent[jb - c0] & 255 : o0 + jb - off;
          wave_sync();
        }
      }
      const bool have = act && lse.m != -INFINITY;
      const double lnl = have ? lse.m + log(lse.s) - a.ln_nphi : -INFINITY;
      if (EVAL) {
        if (act) {
          const size_t to = (size_t)(row0 + tr) * a.n_ext + (col0 + tc);
          a.lnl_out[to] = lnl;
          if (a.ml_out) a.ml_out[to] = mn / (2.0 * md);
        }
        continue;
      }
      if (act) ev.ml_max = fmax(ev.ml_max, mn / (2.0 * md));
      const double lnp = lnw + lnl;
      const double mx = wave_max(have ? lnp : -INFINITY);
      // top-k candidates within the window of the running maxima: with the cut
      // on, when a batch gathers its pairs from many rows, its own maximum is
      // one of them; else each lane adds its own in turn
      double tmax = -INFINITY;
      if (on) {
        unsigned long long prev = 0ull;
        if (lane == 0 && mx > -INFINITY) prev = atomicMax(&tile_lnp_max, order_bits(mx));
        tmax = fmax(mx, order_value((unsigned long long)__shfl((long long)prev, 0, 64)));
      }
      if (have) {
        if (!on) {
          const unsigned long long own = order_bits(lnp);
          const unsigned long long prev = atomicMax(&tile_lnp_max, own);
          tmax = order_value(prev > own ? prev : own);
        }
        append_candidate(a, lnp >= fmax(thr_topk_glob, tmax - a.topk_window), lnp, rowd[tr * 4 + 3],
                         (double)(col0 + tc), ob);
      }
      // the row and column sums, a row of the batch at a time (a fixed order;
      // a row belongs to one wave)
      const bool sums = have && lnp != -INFINITY;
      unsigned long long todo = __ballot(sums);
      if (!todo) continue;
      if (mx > wm) {
        const double f = wm == -INFINITY ? 0.0 : exp(wm - mx);
        ev.p.s *= f;
        ev.p.s2 *= f * f;
        ev.p.s3 *= f * f;
        if (lane < TN) csum[wave][lane] *= f;
        if (lane < TM && (lane * TN / 64) % NW == wave) rsum[lane] *= f;
        wm = mx;
        wave_sync();
      }
      const double ex = sums ? exp(lnp - wm) : 0.0;
      ev.p.s += ex;
      ev.p.s2 = fma(ex, ex, ev.p.s2);
      ev.p.s3 = fma(ex * ex, sums ? lse.sq_ratio() : 0.0, ev.p.s3);
      while (todo) {
        const int r = __builtin_amdgcn_readlane(tr, __builtin_ctzll(todo));
        const bool mine = sums && tr == r;
        todo &= ~__ballot(mine);
        const double sum = wave_reduce(mine ? ex : 0.0, 0.0, [](double x, double y) { return x + y; });
        if (lane == 63) rsum[r] += sum;
        if (mine) csum[wave][tc] += ex;
        wave_sync();
      }
    }
    if (EVAL) {
      __syncthreads();
      continue;
    }
    if (lane == 0) wmax[wave] = wm;
    // (every lane's sums are relative to wm)
    auto add_d = [](double x, double y) { return x + y; };
    ev.p.s = wave_reduce(ev.p.s, 0.0, add_d);
    ev.p.s2 = wave_reduce(ev.p.s2, 0.0, add_d);
    ev.p.s3 = wave_reduce(ev.p.s3, 0.0, add_d);
    ev.p.m = lane == 63 ? wm : -INFINITY;
    tile_partial<NW>(a, ev, n_pairs_i, n_bounded_i, red, &tile_lnp_max, t);
    // (the sums and the tile maximum are final: tile_partial has a barrier)
    // relative to the tile maximum
    {
      const unsigned long long mb = tile_lnp_max;
      const double mxp = mb == 0ull ? -INFINITY : order_value(mb);
      auto rel = [&](int w) { return wmax[w] == -INFINITY ? 0.0 : exp(wmax[w] - mxp); };
      double* rc = a.rowcol + t * 128;
      if (tid < TM) {
        rc[tid] = rsum[tid] * rel((tid * TN / 64) % NW);
      } else if (tid < TM + TN) {
        double sum = 0.0;
        for (int w = 0; w < NW; ++w) sum += csum[w][tid - TM] * rel(w);
        rc[64 + tid - TM] = sum;
      }
    }
    __syncthreads();   // the tile's scalars and reduction area are reused
  }
}

template <int PREC, int G, int MODE, bool MANY = false>
__global__ __launch_bounds__(256, 3) void k_e2_tiles(FusedArgs a) {
  e2_pass<PREC, G, MODE, MANY>(a, e2_few(a.n_tiles), blockIdx.x, gridDim.x);
}

// one chunk's second half of several events
template <int PREC, int G, bool MANY>
__global__ __launch_bounds__(256, 3) void k_e2_tiles_packed(PackLaunch p) {
  int64_t blk, nblk;
  int q;
  const int e = pack_locate(p, blockIdx.x, &blk, &nblk, &q);
  FusedArgs a = pack_args(p, e, q);
  a.work0 = p.chunk * a.coef_tiles;
  e2_pass<PREC, G, kEvidence, MANY>(a, false, blk, nblk);
}

// ---------------------------------------------------------------------------
// Posterior sampling (Sec. III B: resampling by the probabilistic weights;
// Sec. V B).  A systematic draw over the pairs' weights p_ie has been placed
// in tiles (by the tiles' masses from the evidence pass); here each listed
// tile is evaluated again and its draws resolved: the pair by the running
// sum of its weights in index order, then the phase o with probability
// proportional to Lbar_ieo, then the distance from its posterior given that
// triple.
// ---------------------------------------------------------------------------

// D drawn from its posterior given (dh, hh) at d0 with the prior
// proportional to D^2 on (0, D_max] (the integrand of eq.
// lnl_dist_marginalized): in x = ln u, u = d0 / D >= u0 = d0 / D_max, the
// density is proportional to u^-3 exp(dh u - hh u^2 / 2).  Its CDF on NG
// points uniform in x over [ln u0, ln u_hi] (u_hi past the peak by 12
// widths and at least 100 u0) by the trapezoid rule, inverted at `uni` by
// linear interpolation within the cell.  Every lane of the wave takes part
// and gets the result.
__device__ inline double draw_distance(double dh, double hh, double u0, double d0, double uni,
                                       int lane) {
  constexpr int NG = 4096, PER = NG / 64;
  const double us = hh > 0.0 ? fmax(u0, dh / hh) : u0;
  const double sg = hh > 0.0 ? 1.0 / sqrt(hh) : 0.0;
  const double uhi = fmax(100.0 * u0, us + 12.0 * sg);
  const double x0 = log(u0), hx = (log(uhi) - x0) / (NG - 1);
  auto lg = [&](int j) {
    const double x = x0 + hx * j, u = exp(x);
    return -3.0 * x + dh * u - 0.5 * hh * u * u;
  };
  double mx = -INFINITY;
  for (int q = 0; q < PER; ++q) mx = fmax(mx, lg(lane * PER + q));
  mx = wave_max(mx);
  // this lane's cells j = lane * PER .. lane * PER + PER - 1 (the last one
  // stops at NG - 2)
  double part = 0.0, fprev = exp(lg(lane * PER) - mx);
  for (int q = 0; q < PER; ++q) {
    const int j = lane * PER + q;
    if (j + 1 >= NG) break;
    const double fn = exp(lg(j + 1) - mx);
    part += 0.5 * hx * (fprev + fn);
    fprev = fn;
  }
  double pre = part;      // inclusive prefix over lanes
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double v = __shfl_up(pre, off, 64);
    if (lane >= off) pre += v;
  }
  const double total = __shfl(pre, 63, 64);
  const double target = uni * total;
  const unsigned long long hit = __ballot(pre > target && part > 0.0);
  const int src = hit ? __ffsll((long long)hit) - 1 : 63;
  double x = x0 + hx * (NG - 1);
  if (hit) {
    // the PER = 64 cells of lane src, one per lane: the first whose running
    // sum exceeds the target
    static_assert(PER == 64, "a cell per lane");
    const int j = src * PER + lane;
    const bool in = j + 1 < NG;
    const double cell = in ? 0.5 * hx * (exp(lg(j) - mx) + exp(lg(j + 1) - mx)) : 0.0;
    double run = cell;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const double v = __shfl_up(run, off, 64);
      if (lane >= off) run += v;
    }
    const double before = __shfl(pre - part, src, 64);
    const unsigned long long cross = __ballot(in && before + run > target);
    if (cross) {
      const int c = __ffsll((long long)cross) - 1;
      const double xc = x0 + hx * (j + (target - (before + run - cell)) / cell);
      x = __shfl(xc, c, 64);
    }
  }
  return d0 / exp(x);
}

// The listed tiles' pairs: ln p of every pair as the evidence pass evaluated
// it (-inf where it was cut), a pair per thread, to sample_lnp [item][NPT].
// Few tiles are drawn (tens, where the posterior is narrow), so a tile is
// spread over NPT / 256 workgroups; with a workgroup per tile that also
// resolved the tile's draws, 4096 draws in ~30 tiles kept ~30 of the 256 CUs
// busy: a call took 34 ms at 65536 x 4096 pairs, 1.7 ms with the pairs, the
// running sums and the draws in kernels of their own.
template <int PREC, int G>
__global__ __launch_bounds__(256, 3) void k_sample_pairs(FusedArgs a) {
  typedef Tile<PREC> TL;
  typedef typename std::conditional<PREC == kFP64, double, float>::type AT;
  constexpr int NRT = (G == 1) ? 1 : kMaxNR;
  constexpr int NCO = 2 * G + NRT;
  constexpr int TM = TL::TM, TN = TL::TN, NPT = TM * TN, NT = 256, PARTS = NPT / NT;
  __shared__ DistParams dp;
  __shared__ double lds_cs[kMaxM * kMaxPhi * 2];
  __shared__ double rowd[TM * 4], cold[TN * 3], rowq[TM * 2];
  const int tid = threadIdx.x;
  for (int t = tid; t < kMaxM * a.n_phi * 2; t += NT) lds_cs[t] = a.phase_cs[t];
  for (int t = tid; t < (int)(sizeof(DistParams) / 4); t += NT)
    ((unsigned*)&dp)[t] = ((const unsigned*)a.dist.prm)[t];
  const bool on = cut_on(a);
  const double thr_ml = on ? __longlong_as_double(a.state[3]) - a.cut_delta : -INFINITY;
  const float thr_f = (float)thr_ml;
  const int64_t end = (min(a.work0 + a.coef_tiles, a.n_work_list) - a.work0) * PARTS;
  for (int64_t w = blockIdx.x; w < end; w += gridDim.x) {
    const int64_t item = w / PARTS;
    const int p = (int)(w % PARTS) * NT + tid, tr = p / TN, tc = p % TN;
    const int64_t t = a.work_list[a.work0 + item];
    const int64_t row0 = t / a.n_tiles_n * TM, col0 = t % a.n_tiles_n * TN;
    __syncthreads();   // (the scalars of the block's last item are no longer read)
    e2_scalars<PREC, TM, TN>(a, row0, col0, rowd, cold, rowq);
    __syncthreads();
    double lnp = -INFINITY;
    if (row0 + tr < a.n_sub && col0 + tc < a.n_ext) {
      PairCoef<AT, G, NRT> pc;
      pc.template load<NPT>((const AT*)a.coef + item * (int64_t)(NCO * NPT), p);
      float bound, lw;
      if (!(on && pc.bounded(rowq, cold, tr, tc, thr_f, bound, lw))) {
        double2 X[G];
        double S0, Sr[kMaxND], Si[kMaxND], lnw;
        pc.unscale(rowd, cold, tr, tc, X, S0, Sr, Si, lnw);
        EvAcc ev;
        ev.init();
        LsePh lse;
        lse.init();
        double best = -INFINITY, mlmax = 0.0;
        int ob = 0;
        pair_phases<kEvidence, G, true>(a, lds_cs, dp, X, S0, Sr, Si, lnw, thr_ml, 0, 1, ev, lse, best,
                                        ob, mlmax);
        if (lse.m != -INFINITY) lnp = lnw + (lse.m + log(lse.s) - a.ln_nphi);
      }
    }
    a.sample_lnp[item * NPT + p] = lnp;
  }
}

// Running sums of each listed tile's pair weights e^(ln p - m) in index
// order (m: the tile's largest ln p in the evidence pass), for the draws to
// search: chunks of 64 by lane scans, then the chunks' totals in order.
template <int NPT>
__global__ __launch_bounds__(256) void k_sample_cum(FusedArgs a) {
  constexpr int NC = NPT / 64, PER = NC / 4;
  __shared__ double tot[NC];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t item = blockIdx.x;
  const double pm = a.partials[a.work_list[a.work0 + item] * kNPart];
  const double* v = a.sample_lnp + item * NPT;
  double pre[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int c = wave * PER + q;
    const double x = v[c * 64 + lane];
    pre[q] = x == -INFINITY ? 0.0 : exp(x - pm);
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const double y = __shfl_up(pre[q], off, 64);
      if (lane >= off) pre[q] += y;
    }
    if (lane == 63) tot[c] = pre[q];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double run = 0.0;
    for (int c = 0; c < NC; ++c) {
      const double x = tot[c];
      tot[c] = run;
      run += x;
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int c = wave * PER + q;
    a.sample_cum[item * NPT + c * 64 + lane] = tot[c] + pre[q];
  }
}

// The draws, a wave per draw: the pair by the running sums of its tile, the
// phase by those of the pair's Lbar_ieo, the distance from its posterior.
template <int PREC, int G>
__global__ __launch_bounds__(256) void k_sample_draws(FusedArgs a) {
  typedef Tile<PREC> TL;
  typedef typename std::conditional<PREC == kFP64, double, float>::type AT;
  constexpr int NRT = (G == 1) ? 1 : kMaxNR;
  constexpr int NCO = 2 * G + NRT;
  constexpr int TM = TL::TM, TN = TL::TN, NPT = TM * TN;
  __shared__ DistParams dp;
  __shared__ double lds_cs[kMaxM * kMaxPhi * 2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int t = tid; t < kMaxM * a.n_phi * 2; t += 256) lds_cs[t] = a.phase_cs[t];
  for (int t = tid; t < (int)(sizeof(DistParams) / 4); t += 256)
    ((unsigned*)&dp)[t] = ((const unsigned*)a.dist.prm)[t];
  __syncthreads();
  const double thr_ml = cut_on(a) ? __longlong_as_double(a.state[3]) - a.cut_delta : -INFINITY;
  const int64_t s = long_grid_wg() * 4 + wave;
  if (s >= a.n_samples) return;
  const int64_t item = (int64_t)a.sample_item[s] - a.work0;
  if (item < 0 || item >= a.coef_tiles) return;   // another chunk's
  const int64_t t = a.work_list[a.work0 + item];
  const int64_t row0 = t / a.n_tiles_n * TM, col0 = t % a.n_tiles_n * TN;
  const double pm = a.partials[t * kNPart];
  // the pair: the draw's residual mass within the tile against the running
  // sums (the first that exceeds it; a pair with weight)
  const double r = a.sample_res[s] * exp(a.final_out[9] - pm);
  const double* cum = a.sample_cum + item * NPT;
  const double* lnp = a.sample_lnp + item * NPT;
  int lo = 0, hi = NPT;
  while (lo < hi) {
    const int mid = (lo + hi) / 2;
    if (cum[mid] > r) hi = mid;
    else lo = mid + 1;
  }
  int sel = lo;
  while (sel < NPT && lnp[sel] == -INFINITY) ++sel;
  if (sel == NPT) {                // rounding past the tile's total: its last pair
    for (sel = NPT - 1; sel >= 0 && lnp[sel] == -INFINITY;) --sel;
    if (sel < 0) return;           // (a tile with mass always has a pair)
  }
  const int tr = sel / TN, tc = sel % TN;
  const int64_t ie = row0 + tr, e = col0 + tc;
  const int64_t i = a.sub_idx ? a.sub_idx[ie] : a.sub0 + ie;
  const AT* cf = (const AT*)a.coef + item * (int64_t)(NCO * NPT);
  PairCoef<AT, G, NRT> pc;
  pc.template load<NPT>(cf, sel);
  const double rowd[4] = {a.ln_w_bank ? a.ln_w_bank[i] : 0.0, PREC == kFP64 ? 1.0 : a.row_scale[i],
                          PREC == kFP64 ? 1.0 : a.ah_scale[ie], (double)i};
  const double cold[3] = {a.ln_w_ext ? a.ln_w_ext[e] : 0.0, PREC == kFP64 ? 1.0 : a.col_scale[e],
                          PREC == kFP64 ? 1.0 : a.bh_scale[e]};
  double2 X[G];
  double S0, Sr[kMaxND], Si[kMaxND], lnw;
  pc.unscale(rowd, cold, 0, 0, X, S0, Sr, Si, lnw);
  // the phase: probability Lbar_ieo over the phases kept by the cut
  double v_o[2], dh_o[2], hh_o[2];
  for (int h = 0; h < 2; ++h) {
    const int o = lane + 64 * h;
    v_o[h] = -INFINITY;
    dh_o[h] = 0.0;
    hh_o[h] = 0.0;
    if (o < a.n_phi) {
      phase_dh_hh<G>(a.mt.gm, a.n_phi, lds_cs, X, S0, Sr, Si, o, dh_o[h], hh_o[h]);
      const bool keep = thr_ml <= 0.0 || (dh_o[h] > 0.0 && dh_o[h] * dh_o[h] >= 2.0 * thr_ml * hh_o[h]);
      if (keep) v_o[h] = dr_ln_marg(dh_o[h], hh_o[h], a.r0, a.dist.tab, dp.ghx, dp.ghw);
    }
  }
  const double vmax = wave_max(fmax(v_o[0], v_o[1]));
  const double w0 = v_o[0] == -INFINITY ? 0.0 : exp(v_o[0] - vmax);
  const double w1 = v_o[1] == -INFINITY ? 0.0 : exp(v_o[1] - vmax);
  double pre0 = w0, pre1 = w1;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const double y0 = __shfl_up(pre0, off, 64), y1 = __shfl_up(pre1, off, 64);
    if (lane >= off) { pre0 += y0; pre1 += y1; }
  }
  const double tot0 = __shfl(pre0, 63, 64);
  const double tot = tot0 + __shfl(pre1, 63, 64);
  const double target = sm64_uniform(a.seed, 2 * (uint64_t)s) * tot;
  const unsigned long long h0 = __ballot(w0 > 0.0 && pre0 > target);
  const unsigned long long h1 = __ballot(w1 > 0.0 && tot0 + pre1 > target);
  int osel;
  if (h0) osel = __ffsll((long long)h0) - 1;
  else if (h1) osel = 64 + __ffsll((long long)h1) - 1;
  else {   // rounding past the total: the last kept phase
    const unsigned long long k0 = __ballot(w0 > 0.0), k1 = __ballot(w1 > 0.0);
    osel = k1 ? 64 + 63 - __clzll((long long)k1) : 63 - __clzll((long long)k0);
  }
  const int src = osel & 63, hs = osel >> 6;
  const double dh = __shfl(hs ? dh_o[1] : dh_o[0], src, 64);
  const double hh = __shfl(hs ? hh_o[1] : hh_o[0], src, 64);
  const double v = __shfl(hs ? v_o[1] : v_o[0], src, 64);
  const double D = draw_distance(dh, hh, a.r0, a.d0, sm64_uniform(a.seed, 2 * (uint64_t)s + 1), lane);
  if (lane == 0) {
    double* out = a.samples + 6 * s;
    out[0] = rowd[3];
    out[1] = (double)e;
    out[2] = (double)osel;
    out[3] = D;
    out[4] = lnp[sel];
    out[5] = lnw + v - a.ln_nphi;
  }
}

}  // namespace dotpe
