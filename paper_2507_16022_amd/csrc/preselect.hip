// Kernels of the intrinsic pre-selection (Sec. IV D; App. B eqs. dh_itop,
// x_ML, single_det_ML); the arithmetic is laid out in preselect.h.
//
// The per-channel inner products Y_ikc(t) are one complex matrix product
// per channel on the matrix cores: the bank rows (the split operand the
// evidence pass reads) against one data operand whose rows are the
// (detector, time) grid points, the same for every channel.  A workgroup
// takes 32 bank rows and one detector, a wave 32 grid times; its epilogue
// forms the polarisation projections for every phase, applies the 2x2
// pseudo-inverse and keeps the maximum, and the workgroup writes the
// per-row maximum for its detector.
#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>

#include "gram.h"
#include "preselect.h"

namespace dotpe {
namespace {

template <int PREC>
__device__ __forceinline__ void store_split(void* p0, void* p1, int64_t o, double x) {
  if constexpr (PREC == kFP16X2) {
    const _Float16 hi = (_Float16)x;
    ((_Float16*)p0)[o] = hi;
    ((_Float16*)p1)[o] = (_Float16)(x - (double)hi);
  } else {
    const __bf16 hi = (__bf16)(float)x;
    ((__bf16*)p0)[o] = hi;
    ((__bf16*)p1)[o] = (__bf16)(float)(x - (double)(float)hi);
  }
}

// bank row of entry q of the rows
__device__ __forceinline__ int64_t pre_row(const PreArgs& a, int64_t q) {
  return a.rows ? a.rows[q] : a.row0 + q;
}

// w_kb d_kb exp(2 pi i f_b t) with f_b t reduced to a fraction of a cycle in FP64
__device__ __forceinline__ double2 pre_data(const PreArgs& a, int k, int b, double t) {
  const double x = a.f[b] * t;
  double sn, cn;
  sincospi(2.0 * (x - floor(x)), &sn, &cn);
  const double2 d = a.d[(int64_t)k * a.n_b + b];
  const double w = a.w[(int64_t)k * a.n_b + b];
  return make_double2(w * (d.x * cn - d.y * sn), w * (d.x * sn + d.y * cn));
}

// Data operand: row r = k n_t + j holds w_kb d_kb exp(2 pi i f_b t_kj) (bins
// past n_b zero), scaled by 2^-e_r so that its largest component lies in
// [2^13, 2^14) (col_scale[r] = 2^e_r), stored [Re | -Im] by slice in hi + lo.
template <int PREC>
__global__ __launch_bounds__(256) void k_pre_build_B(PreArgs a) {
  const int64_t r = blockIdx.x;
  const int k = (int)(r / a.n_t), j = (int)(r % a.n_t);
  const double t = a.t0[k] + j * a.dt;
  __shared__ double red[256];
  double mx = 0.0;
  for (int b = threadIdx.x; b < a.n_b; b += blockDim.x) {
    const double2 v = pre_data(a, k, b, t);
    mx = fmax(mx, fmax(fabs(v.x), fabs(v.y)));
  }
  red[threadIdx.x] = mx;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + s]);
    __syncthreads();
  }
  mx = red[0];
  const int ex = (mx > 0.0 && isfinite(mx)) ? ilogb(mx) - 13 : 0;
  if (threadIdx.x == 0) a.col_scale[r] = ldexp(1.0, ex);
  for (int b = threadIdx.x; b < a.n_bp; b += blockDim.x) {
    double br = 0.0, bi = 0.0;
    if (b < a.n_b) {
      const double2 v = pre_data(a, k, b, t);
      br = ldexp(v.x, -ex);
      bi = ldexp(v.y, -ex);
    }
    const int64_t base = (int64_t)(b / kChunk) * 32 + (b % kChunk);
    store_split<PREC>((void*)a.B0, (void*)a.B1, op_index<PREC>(r, base, a.K2p), br);
    store_split<PREC>((void*)a.B0, (void*)a.B1, op_index<PREC>(r, base + 16, a.K2p), -bi);
  }
}

// G_ikcc' = sum_b w_kb h_icb conj(h_ic'b) (c <= c') from the split bank
// values (h = conj(A) 2^e_i) in FP64, a wave per row, its lanes over the bins
// (b = lane mod 64), the sums over the lanes in the order of wave_reduce.  The
// pseudo-inverse below divides by H's smaller eigenvalue, down to 1e-10 of the
// larger one, so the last bits of G reach the results: products, sums and
// their order are fixed.  A pass over the row per detector and a full wave sum
// per output took 1.95 ms per 2^18 rows of five channels and three detectors;
// one pass for three detectors, and sums that share the lane steps (gram.h),
// 1.2 ms, against 0.56 ms to read the rows.
template <int PREC, int NC>
__global__ __launch_bounds__(256, 2) void k_pre_gram(PreArgs a) {
  typedef typename std::conditional<PREC == kFP16X2, _Float16, __bf16>::type H;
  constexpr int NP = NC * (NC + 1) / 2, KD = gram_dets(NC), N = KD * 2 * NP;
  constexpr int N1 = (N + 1) / 2, N2 = (N1 + 1) / 2, N3 = (N2 + 1) / 2, N4 = (N3 + 1) / 2;
  const int lane = threadIdx.x & 63;
  const int64_t q = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (q >= a.n_chunk) return;
  const int64_t i = pre_row(a, a.chunk0 + q);
  const H* r0 = (const H*)a.R0 + i * a.K2;
  const H* r1 = (const H*)a.R1 + i * a.K2;
  const double s2 = a.row_scale[i] * a.row_scale[i];
  for (int k0 = 0; k0 < a.n_det; k0 += KD) {
    const int nk = min(KD, a.n_det - k0);
    double v[N];                     // per detector (re, im) of the pairs
#pragma unroll
    for (int t = 0; t < N; ++t) v[t] = 0.0;
    for (int b = lane; b < a.n_b; b += 64) {
      // (every load asked for before the first is used: the compiler
      // otherwise waits for each channel in turn, 0.61 against 0.36 ms per
      // 2^15 rows of six channels and three detectors)
      H xr[NC][2], xi[NC][2];          // hi, lo
      const H* p0 = r0 + b / kChunk * 32 + b % kChunk;
      const H* p1 = r1 + b / kChunk * 32 + b % kChunk;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        xr[c][0] = p0[c * 2 * a.n_bp];
        xr[c][1] = p1[c * 2 * a.n_bp];
        xi[c][0] = p0[c * 2 * a.n_bp + 16];
        xi[c][1] = p1[c * 2 * a.n_bp + 16];
      }
      __builtin_amdgcn_sched_barrier(0);
      double hr[NC], hi[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        hr[c] = (double)(float)xr[c][0] + (double)(float)xr[c][1];
        hi[c] = -((double)(float)xi[c][0] + (double)(float)xi[c][1]);
      }
      double w[KD];
#pragma unroll
      for (int k = 0; k < KD; ++k) w[k] = k < nk ? a.w[(int64_t)(k0 + k) * a.n_b + b] : 0.0;
      int p = 0;
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int c2 = c; c2 < NC; ++c2, ++p) {
          const double x = hr[c] * hr[c2] + hi[c] * hi[c2], y = hi[c] * hr[c2] - hr[c] * hi[c2];
#pragma unroll
          for (int k = 0; k < KD; ++k) {
            v[(k * NP + p) * 2] += w[k] * x;
            v[(k * NP + p) * 2 + 1] += w[k] * y;
          }
        }
    }
    // wave_reduce's tree: lanes ^ 1, quads, halves of a row, rows, pairs of rows
    gram_halve<N, 0xB1>(v, lane & 1);
    gram_halve<N1, 0x4E>(v, lane & 2);
    gram_halve<N2, kDppXor4>(v, lane & 4);
    gram_halve<N3, 0x128>(v, lane & 8);
    double* out = (double*)(a.gram + (q * a.n_det + k0) * NP);
#pragma unroll
    for (int g = 0; g < N4; ++g) {
      v[g] += __shfl_xor(v[g], 16, 64);
      v[g] += __shfl_xor(v[g], 32, 64);
      const int t = 16 * g + (lane & 15);     // (the steps took the lane's bits in order)
      if (lane < 16 && t < nk * 2 * NP) out[t] = s2 * v[g];
    }
  }
}

__device__ __forceinline__ uint4 ld16(const void* base, int64_t elem) {
  return *(const uint4*)((const uint16_t*)base + elem);
}
__device__ __forceinline__ uint4 neg16(const uint4& x) {
  return make_uint4(x.x ^ 0x80008000u, x.y ^ 0x80008000u, x.z ^ 0x80008000u, x.w ^ 0x80008000u);
}

// One phase of one (row, time): the projections b+ and bx and the form
// a1 (c b+ + s bx)^2 + a2 (-s b+ + c bx)^2, q = (c, s, a1, a2), in FP32 with
// every rounding written out, so that the paths below agree bit for bit.
__device__ __forceinline__ float pre_form(float bp, float bx, const float4& q) {
#pragma clang fp contract(off)
  const float u = __builtin_fmaf(bp, q.x, bx * q.y), v = __builtin_fmaf(bx, q.x, -(bp * q.y));
  return __builtin_fmaf(u, q.z * u, v * (q.w * v));
}
__device__ __forceinline__ float pre_term(float cn, float sn, float re, float im) {
#pragma clang fp contract(off)
  return __builtin_fmaf(cn, re, -(sn * im));
}

// Phase grids with a power of two of at least four phases: the table's
// entries for o, n - o, n / 2 + o and n / 2 - o are the same numbers up to
// sign (2 (m o mod n) / n is exact, and so is the reduction of its cosine and
// sine), so the four phases share their products: seven operations per
// channel and polarisation instead of twelve.  Negating a factor negates the
// rounded result, so every sum is the one the plain loop forms.
__host__ __device__ constexpr bool pre_fours(int n) { return n >= 4 && (n & (n - 1)) == 0; }
// groups of four phases (o = 0 .. n / 4) or single phases, as the forms are stored
__host__ __device__ constexpr int pre_slots(int n) { return pre_fours(n) ? n + 4 : n; }
// phase o's place: group g = 0 .. n / 4 holds g, n - g, n / 2 + g, n / 2 - g
__device__ __forceinline__ int pre_slot(int o, int n) {
  if (!pre_fours(n)) return o;
  if (o <= n / 4) return 4 * o;
  if (o < n / 2) return 4 * (n / 2 - o) + 3;
  return o <= 3 * n / 4 ? 4 * (o - n / 2) + 2 : 4 * (n - o) + 1;
}
// channels per phase in the FP32 phase table, padded so that two channels'
// (cos, sin) are one aligned 16-byte read
constexpr int pre_ncp(int nc) { return (nc + 1) / 2 * 2; }

// The maximum of pre_form over the phase grid for one (row, time): w = (conj(K_c+)
// Y re, im, conj(K_cx) Y re, im) per channel, cs [phase][pre_ncp(NC)] (cos,
// sin) (m_c phi), qf the row's forms by pre_slot, sg +1 for even m, -1 for odd.
template <int NC, bool FOURS>
__device__ __forceinline__ float pre_best(int n, const float (&sg)[NC], const float2* cs, const float4* qf,
                                          const float (&wpr)[NC], const float (&wpi)[NC],
                                          const float (&wxr)[NC], const float (&wxi)[NC]) {
  constexpr int NCP = pre_ncp(NC);
  float best = 0.f;
  struct Cs {
    float2 v[NCP];
  };
  auto load_cs = [&](int o) {
    Cs c;
    const float4* p = (const float4*)(cs + o * NCP);
#pragma unroll
    for (int q = 0; q < NCP / 2; ++q) {
      const float4 x = p[q];
      c.v[2 * q] = make_float2(x.x, x.y);
      c.v[2 * q + 1] = make_float2(x.z, x.w);
    }
    return c;
  };
  if constexpr (FOURS) {
    auto pair = [&](int g) {         // g = 0 or n / 4: two phases
      const Cs k = load_cs(g);
      const float4 q0 = qf[4 * g], q2 = qf[4 * g + 2];
      float p0, p2, x0, x2;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        const float tp = pre_term(k.v[c].x, k.v[c].y, wpr[c], wpi[c]);
        const float tx = pre_term(k.v[c].x, k.v[c].y, wxr[c], wxi[c]);
        p0 = c ? p0 + tp : tp;
        x0 = c ? x0 + tx : tx;
        p2 = c ? __builtin_fmaf(sg[c], tp, p2) : sg[c] * tp;
        x2 = c ? __builtin_fmaf(sg[c], tx, x2) : sg[c] * tx;
      }
      best = fmaxf(best, fmaxf(pre_form(p0, x0, q0), pre_form(p2, x2, q2)));
    };
    pair(0);
    pair(n / 4);
    // the next group's table entries and forms are read while one is
    // evaluated (held by the pins: the reads would otherwise move to their
    // uses, an LDS latency per group in front of its arithmetic)
    struct Group {
      Cs k;
      float4 q[4];
    };
    auto load = [&](int g) {
      Group r;
      r.k = load_cs(g);
#pragma unroll
      for (int u = 0; u < 4; ++u) r.q[u] = qf[4 * g + u];
      return r;
    };
    auto hold = [&](Group& r) {
#pragma unroll
      for (int c = 0; c < NCP; ++c) __asm__ __volatile__("" : "+v"(r.k.v[c].x), "+v"(r.k.v[c].y));
#pragma unroll
      for (int u = 0; u < 4; ++u)
        __asm__ __volatile__("" : "+v"(r.q[u].x), "+v"(r.q[u].y), "+v"(r.q[u].z), "+v"(r.q[u].w));
    };
    auto eval = [&](const Group& r) {
      float p0, p1, p2, p3, x0, x1, x2, x3;
#pragma unroll
      for (int c = 0; c < NC; ++c) {
#pragma clang fp contract(off)
        const float cn = r.k.v[c].x, sp = r.k.v[c].y * wpi[c], sx = r.k.v[c].y * wxi[c];
        const float tp = __builtin_fmaf(cn, wpr[c], -sp), tx = __builtin_fmaf(cn, wxr[c], -sx);
        const float up = __builtin_fmaf(cn, wpr[c], sp), ux = __builtin_fmaf(cn, wxr[c], sx);
        p0 = c ? p0 + tp : tp;
        x0 = c ? x0 + tx : tx;
        p1 = c ? p1 + up : up;
        x1 = c ? x1 + ux : ux;
        p2 = c ? __builtin_fmaf(sg[c], tp, p2) : sg[c] * tp;
        x2 = c ? __builtin_fmaf(sg[c], tx, x2) : sg[c] * tx;
        p3 = c ? __builtin_fmaf(sg[c], up, p3) : sg[c] * up;
        x3 = c ? __builtin_fmaf(sg[c], ux, x3) : sg[c] * ux;
      }
      best = fmaxf(best, fmaxf(pre_form(p0, x0, r.q[0]), pre_form(p2, x2, r.q[2])));
      best = fmaxf(best, fmaxf(pre_form(p1, x1, r.q[1]), pre_form(p3, x3, r.q[3])));
    };
    // groups 1 .. n / 4 - 1, an odd number of them, in turns of two
    Group even = load(1);
    for (int g = 1; g < n / 4; g += 2) {
      Group odd = load(g + 1);
      eval(even);
      hold(odd);
      if (g + 1 < n / 4) {
        even = load(g + 2);
        eval(odd);
        hold(even);
      }
    }
    return best;
  }
  for (int o = 0; o < n; ++o) {
    const Cs k = load_cs(o);
    float bp = 0.f, bx = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      bp += pre_term(k.v[c].x, k.v[c].y, wpr[c], wpi[c]);
      bx += pre_term(k.v[c].x, k.v[c].y, wxr[c], wxi[c]);
    }
    best = fmaxf(best, pre_form(bp, bx, qf[o]));
  }
  return best;
}

// K_c+ and K_cx / i of the chunk's rows, [n_chunk][NC], a thread each
template <int NC>
__global__ __launch_bounds__(256) void k_pre_factors(PreArgs a) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= a.n_chunk * NC) return;
  const int c = (int)(t % NC);
  const double ci = a.cos_iota[a.chunk0 + t / NC];
  const double yn = swsh_m2(a.l[c], -a.m[c], ci), yp = swsh_m2(a.l[c], a.m[c], ci);
  const double sg = (a.l[c] & 1) ? -1.0 : 1.0;
  a.factors[t] = make_double2(0.5 * (yn + sg * yp), 0.5 * (yn - sg * yp));
}

// bytes of k_preselect's dynamic LDS
constexpr size_t pre_lds_bytes(int nc, int n_phi, bool shared) {
  return sizeof(double) * ((size_t)kMaxM * n_phi * 2 + 64 * nc + 32 * (size_t)pre_slots(n_phi) * 2 +
                           (kPreMaxT / 32) * 32) +
         (shared ? (size_t)2 * nc * 4096 : 0);
}

// FOURS: pre_fours(n_phi); SHARED: the waves share the bank rows through LDS
template <int PREC, int NC, bool FOURS, bool SHARED>
__global__ __launch_bounds__(64 * kPreMaxT / 32, (SHARED && NC <= 5) || NC <= 3 ? 2 : 1) void k_preselect(PreArgs a) {
  typedef typename Pol<PREC>::Acc Acc;
  extern __shared__ __align__(16) double pls[];
  const int n_phi = a.n_phi;
  constexpr int NCP = pre_ncp(NC);
  static_assert(NCP * sizeof(float2) <= kMaxM * 2 * sizeof(double), "csf fits the place of cs");
  const int slots = pre_slots(n_phi);
  double* cs = pls;                          // [kMaxM][n_phi][2] cos, sin of m phi_o
  float2* csf = (float2*)pls;                // after the products: [n_phi][NCP] cos, sin of m_c phi_o in FP32
  double* kp = cs + kMaxM * n_phi * 2;       // [32][NC] K_c+
  double* kx = kp + 32 * NC;                 // [32][NC] K_cx / i
  float* qf = (float*)(kx + 32 * NC);        // [32][slots][4] H^+ / 2 as (cos, sin, a1, a2), by pre_slot
  double* red = (double*)(qf + 32 * slots * 4);   // [NW][32]
  unsigned char* stage = (unsigned char*)(red + (kPreMaxT / 32) * 32);   // SHARED: [2][NC][4][1 KB]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nt = blockDim.x;
  // workgroup -> (row block, detector): consecutive ids go to the XCDs in
  // turn; each XCD takes a contiguous range with the detectors of one row
  // block next to each other, so that its L2 serves the bank rows to all of
  // them (the grid is a multiple of 8)
  const int64_t wg = (int64_t)(blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
  const int k = (int)(wg % a.n_det);
  const int64_t rb0 = a.chunk0 + wg / a.n_det * 32;          // first row of the block
  if (rb0 >= a.chunk0 + a.n_chunk) return;
  // the A stages' loads: slice u = 4 c + (0 hi 0, 1 hi 1, 2 lo 0, 3 lo 1) of a
  // chunk by wave u mod (number of waves), 1 KB each.  M0 carries the LDS
  // address; the asm saves and restores it and waits the state an M0 write
  // needs.
  typedef __attribute__((address_space(1))) const unsigned char gbyte;
  typedef __attribute__((address_space(3))) void lvoid;
  const int h = lane >> 5, nj = a.n_bp / kChunk;    // chunks: a multiple of 4 (bins padded to 64)
  const int64_t ia = pre_row(a, min(rb0 + (lane & 31), a.n_rows - 1));   // (rows past the end re-read the last)
  const int64_t abase = ((ia >> 5) * (a.K2 >> 5)) * 1024 + h * 256 + (ia & 31) * 8;
  const unsigned lds_stage = __builtin_amdgcn_readfirstlane((unsigned)(uintptr_t)(lvoid*)stage);
  const int wave_u = __builtin_amdgcn_readfirstlane(wave), nw = nt >> 6;
  auto issue = [&](int j) {
    for (int u = wave_u; u < 4 * NC; u += nw) {
      const int64_t o = abase + (int64_t)((u >> 2) * nj + j) * 1024 + (u & 1) * 512;
      gbyte* p = (gbyte*)((u & 2) ? a.A1 : a.A0) + 2 * o;
      const unsigned m0v = lds_stage + (unsigned)((j & 1) * (NC * 4096) + u * 1024);
      unsigned m0_saved;
      __asm__ __volatile__(
          "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
          "global_load_lds_dwordx4 %2, off\n\ts_mov_b32 m0, %0"
          : "=&s"(m0_saved)
          : "s"(__builtin_amdgcn_readfirstlane(m0v)), "v"(p)
          : "memory");
    }
  };
  if constexpr (SHARED) issue(0);
  const int rows_in = (int)min((int64_t)32, a.chunk0 + a.n_chunk - rb0);

  for (int t = tid; t < kMaxM * n_phi; t += nt) {
    const int mm = t / n_phi + 1, o = t % n_phi;
    sincospi(2.0 * (double)((mm * o) % n_phi) / n_phi, &cs[2 * t + 1], &cs[2 * t]);
  }
  for (int t = tid; t < 32 * NC; t += nt) {
    const double2 f = t / NC < rows_in ? a.factors[(rb0 - a.chunk0) * NC + t] : make_double2(0.0, 0.0);
    kp[t] = f.x;
    kx[t] = f.y;
  }
  __syncthreads();
  // H_pp'(row, o) from the Gram matrix, then its pseudo-inverse / 2 (an
  // eigen-direction with eigenvalue below 1e-10 of the largest dropped) in
  // eigen-form: b^T H^+ b / 2 = a1 (c b+ + s bx)^2 + a2 (-s b+ + c bx)^2, a
  // sum of non-negative terms, so the epilogue may evaluate it in FP32
  constexpr int NP = NC * (NC + 1) / 2;
  for (int t = tid; t < 32 * n_phi; t += nt) {
    const int rr = t / n_phi, o = t % n_phi;
    double h00 = 0.0, h01 = 0.0, h11 = 0.0;
    if (rr < rows_in) {
      const double2* g = a.gram + ((rb0 + rr - a.chunk0) * a.n_det + k) * NP;
      int p = 0;
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int c2 = c; c2 < NC; ++c2, ++p) {
          const double2 G = g[p];
          const int dm = a.m[c] - a.m[c2];
          double cd = 1.0, sd = 0.0;
          if (dm != 0) {
            const int ad = dm < 0 ? -dm : dm;
            cd = cs[((ad - 1) * n_phi + o) * 2];
            sd = dm < 0 ? -cs[((ad - 1) * n_phi + o) * 2 + 1] : cs[((ad - 1) * n_phi + o) * 2 + 1];
          }
          // exp(-i dm phi) G_cc'; the (c', c) term is its conjugate
          const double re = cd * G.x + sd * G.y, im = cd * G.y - sd * G.x;
          const double pa = kp[rr * NC + c], pb = kp[rr * NC + c2];
          const double xa = kx[rr * NC + c], xb = kx[rr * NC + c2];
          const double f = (c == c2) ? 1.0 : 2.0;
          h00 += f * pa * pb * re;
          h11 += f * xa * xb * re;
          h01 += (c == c2) ? pa * xb * im : (pa * xb - pb * xa) * im;
        }
    }
    double ec = 1.0, es = 0.0, a1 = 0.0, a2 = 0.0;
    const double df = 0.5 * (h00 - h11);
    const double lp = 0.5 * (h00 + h11) + sqrt(df * df + h01 * h01);
    if (lp > 0.0) {
      // eigenvector of the larger eigenvalue, then the smaller one as det / lp
      const double vx = df >= 0.0 ? lp - h11 : h01, vy = df >= 0.0 ? h01 : lp - h00;
      const double nn = sqrt(vx * vx + vy * vy);
      if (nn > 0.0) {
        ec = vx / nn;
        es = vy / nn;
      }
      a1 = 0.5 / lp;
      const double lm = (h00 * h11 - h01 * h01) / lp;
      a2 = lm > 1e-10 * lp ? 0.5 / lm : 0.0;
    }
    *(float4*)(qf + 4 * (rr * slots + pre_slot(o, n_phi))) =
        make_float4((float)ec, (float)es, (float)a1, (float)a2);
  }

  // ---- Y_ikc for this wave's 32 grid times, every channel ----
  const int64_t rbB = (int64_t)k * a.n_t + 32 * wave + (lane & 31);
  const int64_t bbase = ((rbB >> 5) * (a.K2p >> 5)) * 1024 + h * 256 + (rbB & 31) * 8;
  Acc acc[NC][2];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    acc[c][0] = Acc{};
    acc[c][1] = Acc{};
  }
  // SHARED: the waves of the workgroup (grid times) share the bank rows: a bin
  // chunk's A slices of every channel (hi, lo of both slices, NC x 4 KB) go straight
  // into one of two LDS stages, shared out over the waves, while the chunk
  // before is multiplied (each of four waves reading A from global memory for
  // itself moved four times the bytes through the L1s: 5.5 of 7.8 ms per 2^18
  // rows).
  // B is the wave's own: registers, a chunk ahead.  Two waves per SIMD (256
  // registers: 160 accumulators at five channels), so that one's epilogue,
  // all VALU, runs under another's products.
  struct FB {
    uint4 h0, h1, l0, l1;
  };
  auto load_b = [&](FB& f, int j) {
    const int64_t bo = bbase + (int64_t)j * 1024;
    f.h0 = ld16(a.B0, bo);
    f.h1 = ld16(a.B0, bo + 512);
    f.l0 = ld16(a.B1, bo);
    f.l1 = ld16(a.B1, bo + 512);
  };
  // A = [Re conj h | Im conj h], B_re = [Br | -Bi], B_im = [Bi | Br]: 3 split
  // products per real product
  auto products = [&](Acc& re, Acc& im, const FB& b, const uint4& nh1, const uint4& nl1, const uint4& h0,
                      const uint4& h1, const uint4& l0, const uint4& l1) {
    mma<PREC>(re, l0, b.h0);  mma<PREC>(im, l0, nh1);
    mma<PREC>(re, h0, b.l0);  mma<PREC>(im, h0, nl1);
    mma<PREC>(re, h0, b.h0);  mma<PREC>(im, h0, nh1);
    mma<PREC>(re, l1, b.h1);  mma<PREC>(im, l1, b.h0);
    mma<PREC>(re, h1, b.l1);  mma<PREC>(im, h1, b.l0);
    mma<PREC>(re, h1, b.h1);  mma<PREC>(im, h1, b.h0);
  };
  FB b0, b1;
  load_b(b0, 0);
  if constexpr (SHARED) {
    auto compute = [&](int j, const FB& b) {
      const uint4 nh1 = neg16(b.h1), nl1 = neg16(b.l1);
      const unsigned char* st = stage + (j & 1) * (NC * 4096) + lane * 16;
      static_for<NC>([&](auto ci) {
        constexpr int c = decltype(ci)::value;
        const uint4 h0 = *(const uint4*)(st + c * 4096), h1 = *(const uint4*)(st + c * 4096 + 1024);
        const uint4 l0 = *(const uint4*)(st + c * 4096 + 2048), l1 = *(const uint4*)(st + c * 4096 + 3072);
        products(acc[c][0], acc[c][1], b, nh1, nl1, h0, h1, l0, l1);
      });
    };
    for (int j = 0; j < nj; j += 2) {
      // chunk j has landed (every wave's part), and every wave is done with j - 1
      pipeline_barrier<0>();
      issue(j + 1);
      load_b(b1, j + 1);
      compute(j, b0);
      pipeline_barrier<0>();
      if (j + 2 < nj) {
        issue(j + 2);
        load_b(b0, j + 2);
      }
      compute(j + 1, b1);
    }
  } else {
    // each wave's own loads, a chunk ahead in registers (one wave per SIMD)
    struct FA {
      uint4 v[NC][4];      // hi 0, hi 1, lo 0, lo 1
    };
    auto load_a = [&](FA& f, int j) {
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int u = 0; u < 4; ++u)
          f.v[c][u] = ld16((u & 2) ? a.A1 : a.A0, abase + (int64_t)(c * nj + j) * 1024 + (u & 1) * 512);
    };
    auto compute = [&](const FA& f, const FB& b) {
      const uint4 nh1 = neg16(b.h1), nl1 = neg16(b.l1);
#pragma unroll
      for (int c = 0; c < NC; ++c)
        products(acc[c][0], acc[c][1], b, nh1, nl1, f.v[c][0], f.v[c][1], f.v[c][2], f.v[c][3]);
    };
    FA f0, f1;
    load_a(f0, 0);
    for (int j = 0; j < nj; j += 2) {
      load_a(f1, j + 1);
      load_b(b1, j + 1);
      compute(f0, b0);
      if (j + 2 < nj) {
        load_a(f0, j + 2);
        load_b(b0, j + 2);
      }
      compute(f1, b1);
    }
  }
  __syncthreads();   // (the forms in qf are complete, cs is no longer read)
  for (int t = tid; t < n_phi * NC; t += nt) {
    const int o = t / NC, c = t % NC;
    double sn, cn;
    sincospi(2.0 * (double)((a.m[c] * o) % n_phi) / n_phi, &sn, &cn);
    csf[o * NCP + c] = make_float2((float)cn, (float)sn);
  }
  __syncthreads();

  // ---- epilogue: polarisation projections, 2x2 form, maximum ----
  // (in FP32: the accumulators are FP32 and the form is a sum of squares)
  const double csc = a.col_scale[rbB];
  float sg[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) sg[c] = (a.m[c] & 1) ? -1.f : 1.f;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int rr = 8 * (r >> 2) + 4 * h + (r & 3);
    const float sc = (float)((rr < rows_in ? a.row_scale[pre_row(a, rb0 + rr)] : 0.0) * csc);
    float wpr[NC], wpi[NC], wxr[NC], wxi[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const float yr = sc * acc[c][0][r], yi = sc * acc[c][1][r];
      const float pk = (float)kp[rr * NC + c], xk = (float)kx[rr * NC + c];
      wpr[c] = pk * yr;     // conj(K_c+) Y
      wpi[c] = pk * yi;
      wxr[c] = xk * yi;     // conj(K_cx) Y = -i (K_cx / i) Y
      wxi[c] = -xk * yr;
    }
    const float bestf = pre_best<NC, FOURS>(n_phi, sg, csf, (const float4*)(qf + 4 * rr * slots), wpr, wpi, wxr,
                                     wxi);
    if (a.ml_t && rr < rows_in)
      a.ml_t[((rb0 + rr) * a.n_det + k) * a.n_t + 32 * wave + (lane & 31)] = (double)bestf;
    // the maximum over the 32 times of this half wave (non-negative values),
    // complete in its last lane
    float m = bestf;
    m = fmaxf(m, dpp_mov<0xB1, 0xF>(0.f, m));
    m = fmaxf(m, dpp_mov<0x4E, 0xF>(0.f, m));
    m = fmaxf(m, dpp_mov<0x141, 0xF>(0.f, m));
    m = fmaxf(m, dpp_mov<0x140, 0xF>(0.f, m));
    m = fmaxf(m, dpp_mov<0x142, 0xA>(0.f, m));
    if ((lane & 31) == 31) red[wave * 32 + rr] = (double)m;
  }
  __syncthreads();
  if (tid < rows_in) {
    double m = red[tid];
    for (int w = 1; w < nt / 64; ++w) m = fmax(m, red[w * 32 + tid]);
    a.ml_det[(rb0 + tid) * a.n_det + k] = m;
  }
}

// incoherent sums over detectors (fixed order), and their maximum
__global__ __launch_bounds__(256) void k_pre_final(PreArgs a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  double v = -INFINITY;
  if (i < a.n_rows) {
    v = 0.0;
    for (int k = 0; k < a.n_det; ++k) v += a.ml_det[i * a.n_det + k];
    a.lnl[i] = v;
  }
  const double m = wave_max(v);
  // (most waves cannot raise the maximum: a read, maybe stale, spares the atomic)
  if ((threadIdx.x & 63) == 0 && m > -INFINITY && order_bits(m) > a.state[0])
    atomicMax((unsigned long long*)&a.state[0], (unsigned long long)order_bits(m));
}

// selection: rows with lnl >= max - delta, in row order (blocks of 1024
// rows, 4 consecutive per thread)
__device__ __forceinline__ unsigned pre_flags(const PreArgs& a, int64_t r0) {
  const double thr = order_value(a.state[0]) - a.delta;
  unsigned f = 0;
  for (int q = 0; q < 4; ++q) {
    const int64_t i = r0 + q;
    if (i < a.n_rows && a.lnl[i] >= thr) f |= 1u << q;
  }
  return f;
}

__global__ __launch_bounds__(256) void k_pre_count(PreArgs a) {
  __shared__ int sc[256];
  const unsigned f = pre_flags(a, (int64_t)blockIdx.x * 1024 + 4 * threadIdx.x);
  sc[threadIdx.x] = __popc(f);
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) sc[threadIdx.x] += sc[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) a.counts[blockIdx.x] = sc[0];
}

__global__ __launch_bounds__(256) void k_pre_scan(PreArgs a, int64_t nb) {
  // each thread a contiguous range of blocks, a scan of the ranges' totals
  __shared__ int64_t sh[256];
  const int t = threadIdx.x;
  const int64_t per = (nb + 255) / 256, lo = min(nb, t * per), hi = min(nb, lo + per);
  int64_t n = 0;
  for (int64_t b = lo; b < hi; ++b) n += a.counts[b];
  sh[t] = n;
  __syncthreads();
  for (int k = 1; k < 256; k <<= 1) {
    const int64_t v = t >= k ? sh[t - k] : 0;
    __syncthreads();
    sh[t] += v;
    __syncthreads();
  }
  int64_t run = sh[t] - n;
  for (int64_t b = lo; b < hi; ++b) {
    a.offsets[b] = run;
    run += a.counts[b];
  }
  if (t == 255) a.state[1] = (uint64_t)sh[255];
}

__global__ __launch_bounds__(256) void k_pre_write(PreArgs a) {
  __shared__ int sc[256];
  const int64_t r0 = (int64_t)blockIdx.x * 1024 + 4 * threadIdx.x;
  const unsigned f = pre_flags(a, r0);
  sc[threadIdx.x] = __popc(f);
  __syncthreads();
  // inclusive scan (Hillis-Steele)
  for (int s = 1; s < 256; s <<= 1) {
    const int v = threadIdx.x >= s ? sc[threadIdx.x - s] : 0;
    __syncthreads();
    sc[threadIdx.x] += v;
    __syncthreads();
  }
  int64_t pos = a.offsets[blockIdx.x] + sc[threadIdx.x] - __popc(f);
  for (int q = 0; q < 4; ++q)
    if (f & (1u << q)) a.selected[pos++] = a.row0 + r0 + q;
}

// Whether the waves of a workgroup share the bank rows through LDS (else each
// wave reads them for itself, a chunk ahead in registers).  Shared, with two to
// five channels, the kernel runs two waves per SIMD, which pays when the LDS of
// its stages and forms leaves room for six of the eight on a CU: five channels,
// 2^15 rows, three detectors, 128 times, 32 phases 0.95 against 1.20 ms a call
// (64 times 0.94 against 0.84; 128 phases, one workgroup per CU, 2.46 against
// 2.42; 32 times, one wave per workgroup and nothing to share, 0.97 against
// 0.67).  One channel has few loads to share (0.44 either way, 0.42 against 0.38
// at 64 times), and six or seven leave one wave per SIMD on both paths, where
// the barriers cost what the shared loads save (seven channels, 64 times: 2.39
// against 1.78).  With eight the registers do not hold a chunk ahead (120
// spilled), so shared from three waves on a CU (96 times 2.62 against 3.20).
constexpr bool pre_shared(int nc, int n_t, int n_phi) {
  if (n_t < 64 || nc == 1 || nc == 6 || nc == 7) return false;
  const int room = nc <= 5 ? 8 : 4, want = nc <= 5 ? 6 : 3;
  const int waves = n_t / 32 * (int)(160 * 1024 / pre_lds_bytes(nc, n_phi, true));
  return (waves < room ? waves : room) >= want;
}

template <int PREC, int NC, bool FOURS, bool SHARED>
hipError_t launch_pre_grid(const PreArgs& a, hipStream_t s) {
  static std::once_flag attr_once;
  std::call_once(attr_once, [&] {
    if (hipFuncSetAttribute((const void*)k_preselect<PREC, NC, FOURS, SHARED>,
                            hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)pre_lds_bytes(NC, kMaxPhi, SHARED)) != hipSuccess)
      (void)hipGetLastError();
  });
  const dim3 grid((unsigned)(((a.n_chunk + 31) / 32 * a.n_det + 7) / 8 * 8));
  hipLaunchKernelGGL((k_preselect<PREC, NC, FOURS, SHARED>), grid, dim3(64 * (a.n_t / 32)),
                     pre_lds_bytes(NC, a.n_phi, SHARED), s, a);
  return hipGetLastError();
}

template <int PREC, int NC>
hipError_t launch_pre_main(const PreArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((k_pre_factors<NC>), dim3((unsigned)((a.n_chunk * NC + 255) / 256)), dim3(256), 0, s,
                     a);
  hipLaunchKernelGGL((k_pre_gram<PREC, NC>), dim3((unsigned)((a.n_chunk + 3) / 4)), dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (pre_shared(NC, a.n_t, a.n_phi))
    return pre_fours(a.n_phi) ? launch_pre_grid<PREC, NC, true, true>(a, s)
                              : launch_pre_grid<PREC, NC, false, true>(a, s);
  return pre_fours(a.n_phi) ? launch_pre_grid<PREC, NC, true, false>(a, s)
                            : launch_pre_grid<PREC, NC, false, false>(a, s);
}

template <int PREC>
hipError_t launch_pre_nc(const PreArgs& a, hipStream_t s) {
  switch (a.n_c) {
    case 1: return launch_pre_main<PREC, 1>(a, s);
    case 2: return launch_pre_main<PREC, 2>(a, s);
    case 3: return launch_pre_main<PREC, 3>(a, s);
    case 4: return launch_pre_main<PREC, 4>(a, s);
    case 5: return launch_pre_main<PREC, 5>(a, s);
    case 6: return launch_pre_main<PREC, 6>(a, s);
    case 7: return launch_pre_main<PREC, 7>(a, s);
    case 8: return launch_pre_main<PREC, 8>(a, s);
  }
  return hipErrorInvalidValue;
}

template <int PREC>
hipError_t run_all(PreArgs a, hipStream_t s) {
  hipLaunchKernelGGL(k_pre_build_B<PREC>, dim3((unsigned)(a.n_det * a.n_t)), dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  for (int64_t c0 = 0; c0 < a.n_rows; c0 += a.chunk_rows) {
    a.chunk0 = c0;
    a.n_chunk = std::min<int64_t>(a.chunk_rows, a.n_rows - c0);
    if ((e = launch_pre_nc<PREC>(a, s)) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_pre_final, dim3((unsigned)((a.n_rows + 255) / 256)), dim3(256), 0, s, a);
  const int64_t nb = (a.n_rows + 1023) / 1024;
  hipLaunchKernelGGL(k_pre_count, dim3((unsigned)nb), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_pre_scan, dim3(1), dim3(256), 0, s, a, nb);
  hipLaunchKernelGGL(k_pre_write, dim3((unsigned)nb), dim3(256), 0, s, a);
  return hipGetLastError();
}

template <int PREC>
hipError_t run_series(PreArgs a, hipStream_t s) {
  if (a.n_rows > a.chunk_rows) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_pre_build_B<PREC>, dim3((unsigned)(a.n_det * a.n_t)), dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  a.chunk0 = 0;
  a.n_chunk = a.n_rows;
  return launch_pre_nc<PREC>(a, s);
}

}  // namespace

hipError_t preselect_series_launch(int prec, PreArgs a, hipStream_t s) {
  if (prec == kFP16X2) return run_series<kFP16X2>(a, s);
  if (prec == kBF16X2) return run_series<kBF16X2>(a, s);
  return hipErrorInvalidValue;
}

hipError_t preselect_launch(int prec, PreArgs a, hipStream_t s) {
  if (prec == kFP16X2) return run_all<kFP16X2>(a, s);
  if (prec == kBF16X2) return run_all<kBF16X2>(a, s);
  return hipErrorInvalidValue;
}

}  // namespace dotpe
