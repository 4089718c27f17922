// Weighted Gram sums of single bank rows: G_kcc' = sum_b w_kb h_cb conj(h_c'b)
// (c <= c') of one row for a few detectors, by 16 lanes in FP64 from the
// row-major split bank (four rows per wave, so that a load takes whole lines
// of each).  The lanes take four consecutive bins at a time (8 bytes of every
// array and part; two where the accumulators leave no room for four bins'
// values), form the NC^2 real products of a bin once and weight them for KD
// detectors; the KD NC^2 sums are reduced over the lanes together, ~7
// instructions per sum and row of lanes (a full wave sum each, a wave per row,
// took ~30 and more time than the products).
#pragma once

#include "fused.h"

namespace dotpe {

// real sums per detector: re of every pair c <= c', im of every pair c < c'
constexpr int gram_vals(int nc) { return nc * nc; }
// detectors per pass: as many as the accumulators of a pass leave room for
constexpr int gram_dets(int nc) { return nc <= 5 ? 3 : 1; }

// Sums over the 16 lanes of a row of lanes of v[0 .. N): each step pairs the
// values, a lane keeping one of a pair and adding the other half's share of it,
// so the registers halve while they add.  Afterwards lane l of the row holds in
// v[g], g < (N + 15) / 16, the sum of value 16 g + gram_value(l).
__device__ __forceinline__ int gram_value(int l) {
  return ((l & 1) << 3) | ((l & 2) << 1) | ((l & 4) >> 1) | ((l & 8) >> 3);
}
// the value of lane ^ 4: row_shl:4 into the lower four lanes of each eight,
// row_shr:4 into the upper four
__device__ __forceinline__ unsigned dpp_xor4(unsigned v) {
  const unsigned x = __builtin_amdgcn_update_dpp(0u, v, 0x104, 0xF, 0x5, false);
  return __builtin_amdgcn_update_dpp(x, v, 0x114, 0xF, 0xA, false);
}
constexpr int kDppXor4 = -4;
// one step: N values to (N + 1) / 2, the partner lane by the DPP control CTRL
// (or kDppXor4); partners own the same bits of earlier steps
template <int N, int CTRL>
__device__ __forceinline__ void gram_halve(double* v, bool upper) {
#pragma unroll
  for (int g = 0; g < (N + 1) / 2; ++g) {
    const double a = v[2 * g], b = 2 * g + 1 < N ? v[2 * g + 1] : 0.0;
    const double own = upper ? b : a, other = upper ? a : b;
    if constexpr (CTRL == kDppXor4) {
      const unsigned long long o = (unsigned long long)__double_as_longlong(other);
      const unsigned lo = dpp_xor4((unsigned)o), hi = dpp_xor4((unsigned)(o >> 32));
      v[g] = own + __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
    } else {
      v[g] = own + dpp_mov<CTRL, 0xF>(0.0, other);
    }
  }
}
template <int N>
__device__ __forceinline__ void gram_reduce(double (&v)[N], int lane) {
  constexpr int N1 = (N + 1) / 2, N2 = (N1 + 1) / 2, N3 = (N2 + 1) / 2;
  gram_halve<N, 0x128>(v, lane & 8);     // row_ror:8: lane ^ 8
  gram_halve<N1, 0x141>(v, lane & 4);    // row_half_mirror: lane ^ 7
  gram_halve<N2, 0x4E>(v, lane & 2);     // quad_perm 2,3,0,1: lane ^ 2
  gram_halve<N3, 0xB1>(v, lane & 1);     // quad_perm 1,0,3,2: lane ^ 1
}

// A bank value hi + lo.  lo may start far below hi's last place, so the sum can
// take more than a float's 24 bits: about one FP16 value in six loses some of
// them, up to 2^-24 of the value, a quarter of what the split leaves out.
// WHOLE: every bit.  (The kernel that stages rows in LDS keeps them as floats;
// rows it would stage are rounded here as there, longer ones are whole on both.)
template <bool WHOLE>
__device__ __forceinline__ double gram_join(float hi, float lo) {
  return WHOLE ? (double)hi + (double)lo : (double)(hi + lo);
}

// v += the Gram sums of the row whose hi and lo parts (conj(h), row-major, n_bp
// bins per channel) start at r0, r1, for the detectors w[0 .. KD) (rows of n_b
// weights; nk of them valid), this lane's bins.  v: per detector re of (c, c'
// >= c) row by row, then im of (c, c' > c).
template <int PREC, int NC, int KD, bool WHOLE>
__device__ __forceinline__ void gram_row(const void* r0, const void* r1, int n_b, int n_bp, const double* w,
                                         int nk, int l16, double (&v)[KD * gram_vals(NC)]) {
  typedef typename std::conditional<PREC == kFP16X2, _Float16, __bf16>::type H;
  constexpr int NV = gram_vals(NC), NP = NC * (NC + 1) / 2;
  constexpr int BL = KD * NV > 64 ? 2 : 4;       // bins per lane and turn
  struct alignas(2 * BL) HB {
    H x[BL];
  };
  for (int b0 = BL * l16; b0 < n_b; b0 += 16 * BL) {
    HB rh[NC], rl[NC], ih[NC], il[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int o = (c * (n_bp / kChunk) + b0 / kChunk) * 32 + b0 % kChunk;
      rh[c] = *(const HB*)((const H*)r0 + o);
      rl[c] = *(const HB*)((const H*)r1 + o);
      ih[c] = *(const HB*)((const H*)r0 + o + 16);
      il[c] = *(const HB*)((const H*)r1 + o + 16);
    }
#pragma unroll
    for (int j = 0; j < BL; ++j) {
      if (b0 + j >= n_b) break;
      double wk[KD];
#pragma unroll
      for (int k = 0; k < KD; ++k) wk[k] = k < nk ? w[k * n_b + b0 + j] : 0.0;
      double hr[NC], hi[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        hr[c] = gram_join<WHOLE>((float)rh[c].x[j], (float)rl[c].x[j]);
        hi[c] = -gram_join<WHOLE>((float)ih[c].x[j], (float)il[c].x[j]);
      }
      int p = 0, q = NP;
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int c2 = c; c2 < NC; ++c2) {
          const double x = hr[c] * hr[c2] + hi[c] * hi[c2];
#pragma unroll
          for (int k = 0; k < KD; ++k) v[k * NV + p] += wk[k] * x;
          ++p;
          if (c2 > c) {
            const double y = hi[c] * hr[c2] - hr[c] * hi[c2];
#pragma unroll
            for (int k = 0; k < KD; ++k) v[k * NV + q] += wk[k] * y;
            ++q;
          }
        }
    }
  }
}

// place of real sum u (0 .. NC^2) of a detector in its NP complex pairs stored
// (re, im) in row order of c <= c': 2 pair + part
template <int NC>
__device__ __forceinline__ int gram_place(int u) {
  constexpr int NP = NC * (NC + 1) / 2;
  if (u < NP) return 2 * u;
  int q = u - NP, c = 0;             // im of the q-th pair with c < c'
  while (q >= NC - 1 - c) {
    q -= NC - 1 - c;
    ++c;
  }
  // pairs before row c, then (c, c), then (c, c + 1 + q)
  return 2 * (c * NC - c * (c - 1) / 2 + 1 + q) + 1;
}

// The Gram sums of one row per 16 lanes for n_det detectors to out [n_det][NP]
// (re, im), times scale (the row's); every lane takes part, those of a row past
// the end with live = false.  (The im of c = c' is zero.)
template <int PREC, int NC, bool WHOLE>
__device__ __forceinline__ void gram_row_all(const void* r0, const void* r1, int n_b, int n_bp,
                                             const double* w, int n_det, double scale, int lane, double* out,
                                             bool live) {
  constexpr int KD = gram_dets(NC), NV = gram_vals(NC), NP = NC * (NC + 1) / 2;
  const int l16 = lane & 15;
  for (int k0 = 0; k0 < n_det; k0 += KD) {
    double v[KD * NV];
#pragma unroll
    for (int q = 0; q < KD * NV; ++q) v[q] = 0.0;
    const int nk = min(KD, n_det - k0);
    gram_row<PREC, NC, KD, WHOLE>(r0, r1, n_b, n_bp, w + (int64_t)k0 * n_b, nk, l16, v);
    gram_reduce(v, lane);
    if (!live) continue;
#pragma unroll
    for (int g = 0; g < (KD * NV + 15) / 16; ++g) {
      const int t = 16 * g + gram_value(l16);
      const int k = t / NV, u = t % NV;
      if (t < KD * NV && k < nk) out[(k0 + k) * 2 * NP + gram_place<NC>(u)] = scale * v[g];
    }
    // im of the diagonal
    for (int t = l16; t < nk * NC; t += 16) {
      const int k = t / NC, c = t % NC;
      out[(k0 + k) * 2 * NP + 2 * (c * NC - c * (c - 1) / 2) + 1] = 0.0;
    }
  }
}

}  // namespace dotpe
