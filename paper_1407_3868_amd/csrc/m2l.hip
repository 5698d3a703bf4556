// Row a1: the all-pairs free-space M2L, its forms for one and for many
// right-hand sides, and the FMM's near field (the same pair translation).
// Layouts as in kernels.hip.
#include <atomic>
#include <cmath>

#include "kernels.h"

namespace mpsl {

namespace {

constexpr int kThreads = 128;

inline int cdiv(int64_t a, int64_t b) { return static_cast<int>((a + b - 1) / b); }

// Row a1: all-pairs free-space M2L (Graf's addition theorem).
// One lane per target l; every lane of the grid walks the same source chunk,
// so the source's coefficients are wave-uniform and live in scalar registers.
// Per pair: H_0, H_1 and e^{i phi} from the pair table, the upward recurrence
// H_{q+1} = (2q/z) H_q - H_{q-1}, e^{iq phi} by repeated multiplication,
// h_q = H_q e^{iq phi}, h_{-q} = (-1)^q H_q e^{-iq phi}, and the Toeplitz
// product alpha_{n'} += sum_nu h_{nu - n'} beta_nu consumed in the order the
// recurrence produces h_q.
//
// m2l_block adds the contribution of source slots [V0, V1] to output slots
// [O0, O1].  FP32 does everything in one call (33 accumulators, 66 scalar
// registers of beta at p = 16).  FP64 splits the outputs over two lanes and
// the source coefficients over two calls: 17 accumulators and at most 68
// scalar registers of beta, at the cost of re-running the recurrence.
template <typename T, int p, int O0, int O1, int V0, int V1, bool MIRROR>
__device__ __forceinline__ void m2l_block(cx<T> (&acc)[O1 - O0 + 1], const cv_t<T> *__restrict__ bm, cx<T> h0,
                                          cx<T> h1, cx<T> t, T two_over_z) {
  constexpr int QA = V1 - O0, QB = O1 - V0;
  constexpr int QMAX = (QA > QB ? QA : QB) < 2 * p ? (QA > QB ? QA : QB) : 2 * p;
  cx<T> bv[V1 - V0 + 1];
#pragma unroll
  for (int v = V0; v <= V1; ++v) bv[v - V0] = ld<T>(bm[MIRROR ? 2 * p - v : v]);
#pragma unroll
  for (int v = (V0 > O0 ? V0 : O0); v <= (V1 < O1 ? V1 : O1); ++v) cmac(acc[v - O0], h0, bv[v - V0]);
  cx<T> hprev = h0, hcur = h1, tq = t;
#pragma unroll
  for (int q = 1; q <= QMAX; ++q) {
    if (q >= 2) {
      const cx<T> hn = static_cast<T>(q - 1) * two_over_z * hcur - hprev;
      hprev = hcur;
      hcur = hn;
      tq = tq * t;
    }
    // alpha_{v-q} += h_q beta_v for v - q in [O0, O1]
    if ((V1 < O1 + q ? V1 : O1 + q) >= (V0 > O0 + q ? V0 : O0 + q)) {
      const cx<T> hp = hcur * tq;
#pragma unroll
      for (int v = (V0 > O0 + q ? V0 : O0 + q); v <= (V1 < O1 + q ? V1 : O1 + q); ++v)
        cmac(acc[v - q - O0], hp, bv[v - V0]);
    }
    // alpha_{v+q} += h_{-q} beta_v for v + q in [O0, O1]
    if ((V1 < O1 - q ? V1 : O1 - q) >= (V0 > O0 - q ? V0 : O0 - q)) {
      cx<T> hm = hcur * conj(tq);
      if (q & 1) hm = mk<T>(-hm.re, -hm.im);
#pragma unroll
      for (int v = (V0 > O0 - q ? V0 : O0 - q); v <= (V1 < O1 - q ? V1 : O1 - q); ++v)
        cmac(acc[v + q - O0], hm, bv[v - V0]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Mirror identity: with reversed indices (alpha~_k = alpha_{-k},
// beta~_nu = beta_{-nu}) the translation keeps its Toeplitz form with
// h~_q = h_{-q} = H_q e^{iq(pi - phi)}, i.e. e^{i phi} -> -conj(e^{i phi}).
// MIRROR = true computes output slots 2p - [O0, O1] that way.
template <typename T, int p, int O0, int O1, int SPLIT, bool MIRROR>
__device__ __forceinline__ void m2l_body(const cv_t<T> *__restrict__ pairs, const cv_t<T> *__restrict__ beta,
                                         cv_t<T> *__restrict__ part, int n, int m0, int m1, int l) {
  constexpr int P = 2 * p + 1;
  constexpr int NO = O1 - O0 + 1;
  const bool valid = l < n;
  const int lc = valid ? l : n - 1;
  cx<T> acc[NO];
#pragma unroll
  for (int i = 0; i < NO; ++i) acc[i] = mk<T>(0, 0);
  if (m0 < m1) {
    const cv_t<T> *pe = pairs + 4 * (static_cast<int64_t>(m0) * n + lc);
    cv_t<T> a0 = pe[0], a1 = pe[1], a2 = pe[2], a3 = pe[3];
    for (int m = m0; m < m1; ++m) {
      cx<T> h0 = ld<T>(a0), h1 = ld<T>(a1);
      cx<T> t = ld<T>(a2);
      if (MIRROR) t.re = -t.re;
      const T two_over_z = a3.x;
      if (m + 1 < m1) {  // prefetch the next source's pair entry
        pe += 4 * static_cast<int64_t>(n);
        a0 = pe[0];
        a1 = pe[1];
        a2 = pe[2];
        a3 = pe[3];
      }
      if (!valid) h0 = h1 = mk<T>(0, 0);
      const cv_t<T> *bm = beta + static_cast<int64_t>(m) * P;
      if (SPLIT) {  // source coefficients in two halves, one scalar-register set each
        m2l_block<T, p, O0, O1, 0, p, MIRROR>(acc, bm, h0, h1, t, two_over_z);
        __builtin_amdgcn_sched_barrier(0);
        m2l_block<T, p, O0, O1, p + 1, P - 1, MIRROR>(acc, bm, h0, h1, t, two_over_z);
        __builtin_amdgcn_sched_barrier(0);
      } else {
        m2l_block<T, p, O0, O1, 0, P - 1, MIRROR>(acc, bm, h0, h1, t, two_over_z);
      }
    }
  }
  if (valid) {
#pragma unroll
    for (int i = 0; i < NO; ++i) part[static_cast<int64_t>(l) * P + (MIRROR ? 2 * p - O0 - i : O0 + i)] = st(acc[i]);
  }
}

// grid: (target blocks, source chunks); part[chunk][n][P].  Two variants:
//  whole  (HALF = -1): one lane holds all P accumulators of its target;
//  halves (HALF = 0, 1, two launches): output slots [0, p] and, through the
//         mirror identity, [p+1, 2p], at most p+1 accumulators per lane and
//         more waves per SIMD, for twice the recurrence work.  The two halves
//         are separate kernels: in one kernel the compiler merges the bodies
//         and doubles the live registers.
// FP64 always takes the source coefficients in two scalar-register halves.
// The launcher runs the variant the autotuner picked (default: whole).
template <typename T, int p, int HALF>
__global__ __launch_bounds__(kThreads) void k_m2l(const cv_t<T> *__restrict__ pairs,
                                                  const cv_t<T> *__restrict__ beta,
                                                  cv_t<T> *__restrict__ part, int n, int chunk_len,
                                                  int64_t bstride, int64_t pstride) {
  constexpr int P = 2 * p + 1;
  const int l = blockIdx.x * kThreads + threadIdx.x;
  const int c = blockIdx.y;
  beta += blockIdx.z * bstride;  // right-hand side
  part += blockIdx.z * pstride;
  const int m0 = c * chunk_len;
  const int m1 = min(n, m0 + chunk_len);
  cv_t<T> *o = part + static_cast<int64_t>(c) * n * P;
  constexpr int SPLIT = std::is_same<T, double>::value ? 1 : 0;
  if (HALF == 0) m2l_body<T, p, 0, p, SPLIT, false>(pairs, beta, o, n, m0, m1, l);
  else if (HALF == 1) m2l_body<T, p, 0, p - 1, SPLIT, true>(pairs, beta, o, n, m0, m1, l);
  else m2l_body<T, p, 0, P - 1, SPLIT, false>(pairs, beta, o, n, m0, m1, l);
}

// FMM near field: the same pair translation restricted to padded neighbour
// lists.  One lane per target in leaf-box order; each lane walks its own
// list of sources (pair entries [j][i][4] as in the all-pairs table, source
// coefficients loaded per lane), and every wave loops to the longest list
// among its 64 targets (padding entries are zeros).  HALF as in k_m2l: -1
// all outputs; 0 / 1 output slots [0, p] / (mirror) [p+1, 2p] in two
// launches, which keeps FP64 within the register file.
template <typename T, int p, int HALF>
__global__ __launch_bounds__(kThreads) void k_fmm_near(const cv_t<T> *__restrict__ pairs,
                                                       const int *__restrict__ src, const int *__restrict__ perm,
                                                       const int *__restrict__ wave_cnt,
                                                       const cv_t<T> *__restrict__ beta, cv_t<T> *__restrict__ out,
                                                       int n, int kc) {
  constexpr int P = 2 * p + 1;
  const int i = blockIdx.x * kThreads + threadIdx.x;
  // list entries [j_lo, j_hi) of this chunk into partial slot blockIdx.y
  const int kw = __builtin_amdgcn_readfirstlane(wave_cnt[i >> 6]);
  const int j_lo = blockIdx.y * kc, j_hi = min(kw, j_lo + kc);
  out += static_cast<int64_t>(blockIdx.y) * n * P;
  const bool valid = i < n;
  const int ic = valid ? i : n - 1;
  constexpr bool MIRROR = HALF == 1;
  constexpr int O1 = HALF == 0 ? p : (HALF == 1 ? p - 1 : P - 1);  // outputs [0, O1]
  cx<T> acc[O1 + 1];
#pragma unroll
  for (int k = 0; k <= O1; ++k) acc[k] = mk<T>(0, 0);
  constexpr int SPLIT = std::is_same<T, double>::value ? 1 : 0;
  for (int j = j_lo; j < j_hi; ++j) {
    const int64_t e = static_cast<int64_t>(j) * n + ic;
    const cv_t<T> *pe = pairs + 4 * e;
    cx<T> h0 = ld<T>(pe[0]), h1 = ld<T>(pe[1]);
    cx<T> t = ld<T>(pe[2]);
    if (MIRROR) t.re = -t.re;
    const T two_over_z = pe[3].x;
    if (!valid) h0 = h1 = mk<T>(0, 0);
    const cv_t<T> *bm = beta + static_cast<int64_t>(src[e]) * P;
    if (SPLIT) {
      m2l_block<T, p, 0, O1, 0, p, MIRROR>(acc, bm, h0, h1, t, two_over_z);
      __builtin_amdgcn_sched_barrier(0);
      m2l_block<T, p, 0, O1, p + 1, P - 1, MIRROR>(acc, bm, h0, h1, t, two_over_z);
      __builtin_amdgcn_sched_barrier(0);
    } else {
      m2l_block<T, p, 0, O1, 0, P - 1, MIRROR>(acc, bm, h0, h1, t, two_over_z);
    }
  }
  if (valid) {
    const int64_t o = static_cast<int64_t>(perm[i]) * P;
#pragma unroll
    for (int k = 0; k <= O1; ++k) out[o + (MIRROR ? 2 * p - k : k)] = st(acc[k]);
  }
}


// ---------------------------------------------------------------------------
// Row a1 on the matrix cores, one right-hand side, FP64.  The translation
// alpha_{n'} = sum_q h_q beta_{n'+q} (q = nu - n', |q| <= 2p) is a product
// with the source coefficients in shifted form: with slots s' = n' + p,
// A_m[s'][q] = beta_m[s' + q] (zero where s' + q leaves [0, 2p]) and
// B[(m, q)][l] = h_q of the pair (m -> l),
//   alpha_l[s'] = sum_{m, q} A_m[s'][q] B[(m, q)][l],
// a GEMM with M = output slots, N = targets and K = (source, q).  A 4x4x4 MFMA
// (four blocks) takes four sources at one q and four output slots for 16
// targets: lane i runs the Hankel recurrence of the pair (source i / 16 of the
// group -> target i % 16) and supplies its h_q as the B operand; A, four
// consecutive coefficients from slot 4 R + q of the lane's source, is read from
// LDS, which holds the coefficients of kM2lBatch sources as (re, im, re + im)
// with zero padding.  Complex products take three real MFMAs (Gauss):
// P1 = sum Ar Br, P2 = sum Ai Bi, P3 = sum (Ar + Ai)(Br + Bi); re = P1 - P2,
// im = P3 - P1 - P2.  Their rounding is relative to the product of the moduli,
// not to the smaller of an entry's real and imaginary part; against extended
// precision the error is that of four products (70 particles, p = 8, 12, 14:
// 7.0, 5.6 and 2.8e-15, vector form 7.0, 5.6 and 2.7).  For even p the last slot runs on the vector units
// (2p + 1 = 4 NR + 1).
//
// Bound by the matrix cores and the vector units in turn: FP64 MFMAs and
// vector instructions do not overlap on this chip (a 4x4x4 costs 16.5 cycles, an
// FP64 multiply-add beside it 4.4 more), so the work is the sum of both.  Why
// 4x4x4: only |s' + q - p| <= p of a block's rows count, and blocks of four
// slots waste 9 % of them where 16-slot blocks wasted 31 % (p = 16: 864 x 16.5
// cycles per 64 pairs instead of 288 x 65), at the same rate per operation.
// 3001 particles, p = 16: 1.40 -> 1.22 ms; 1000, p = 12: 146 us on the vector
// units -> 83 us.
// NT = 2 target tiles per wave share the A reads, which would take all of the
// LDS bandwidth for one.
constexpr int kM2lWaves = 4;
constexpr int kM2lBatch = 16;

template <int p, int NT>
__global__ __launch_bounds__(64 * kM2lWaves, 2) void k_m2l_f64(const double2 *__restrict__ pairs,
                                                               const double2 *__restrict__ beta,
                                                               double2 *__restrict__ part, int n, int chunk_len,
                                                               int64_t bstride, int64_t pstride) {
  constexpr int P = 2 * p + 1;
  constexpr bool VROW = P % 4 == 1 && P > 1;  // slot 2p on the vector units
  constexpr int NR = VROW ? P / 4 : (P + 3) / 4;
  // row of a source: slots -3 .. 2p + 3 + the padded rows' overhang; a stride of
  // 4 mod 32 entries puts the four sources of one read in different banks
  constexpr int LR0 = P + 8;
  constexpr int LR = LR0 + ((4 - LR0) % 32 + 32) % 32;
  constexpr int SB = kM2lBatch;
  __shared__ double sa[3][SB][LR];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const int c = blockIdx.y;
  beta += blockIdx.z * bstride;
  part += blockIdx.z * pstride;
  const int m0 = c * chunk_len;
  const int m1 = min(n, m0 + chunk_len);
  const int lt0 = (blockIdx.x * kM2lWaves + w) * 16 * NT;

  for (int e = threadIdx.x; e < 3 * SB * LR; e += 64 * kM2lWaves) (&sa[0][0][0])[e] = 0.0;

  double acc[NT][NR][3];
  cx<double> zc[NT];
#pragma unroll
  for (int tt = 0; tt < NT; ++tt) {
#pragma unroll
    for (int R = 0; R < NR; ++R) acc[tt][R][0] = acc[tt][R][1] = acc[tt][R][2] = 0.0;
    zc[tt] = mk(0.0, 0.0);
  }
  // pair entries of the first group (source m0 + g)
  double2 pa[NT][4];
  auto load_pairs = [&](int m) {
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) {
      const int l = lt0 + tt * 16 + r;
      if (m < m1 && l < n) {
        const double2 *pe = pairs + 4 * (static_cast<int64_t>(m) * n + l);
#pragma unroll
        for (int k = 0; k < 4; ++k) pa[tt][k] = pe[k];
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) pa[tt][k] = make_double2(0.0, 0.0);
      }
    }
  };
  load_pairs(m0 + g);

  for (int mb = m0; mb < m1; mb += SB) {
    const int sb = min(SB, m1 - mb);
    __syncthreads();  // previous batch consumed (and the zero fill done)
    for (int e = threadIdx.x; e < SB * P; e += 64 * kM2lWaves) {
      const int s = e / P, v = e - s * P;
      const double2 b = s < sb ? beta[static_cast<int64_t>(mb + s) * P + v] : make_double2(0.0, 0.0);
      sa[0][s][v + 3] = b.x;
      sa[1][s][v + 3] = b.y;
      sa[2][s][v + 3] = b.x + b.y;
    }
    __syncthreads();
    // a wave whose targets all lie past the last particle (the grid's tail)
    // stages its share of the batch and meets the barriers, but multiplies nothing
    for (int g0 = 0; g0 < sb && lt0 < n; g0 += 4) {
      const int s = g0 + g;  // this lane's source within the batch
      cx<double> hp[NT], hc[NT], t[NT], tq[NT];
      double tz[NT];
#pragma unroll
      for (int tt = 0; tt < NT; ++tt) {
        hp[tt] = ld<double>(pa[tt][0]);
        hc[tt] = ld<double>(pa[tt][1]);
        t[tt] = ld<double>(pa[tt][2]);
        tq[tt] = t[tt];
        tz[tt] = pa[tt][3].x;
      }
      load_pairs(mb + s + 4);  // next group's entries in flight
      const double *ar = &sa[0][s][3 + (lane & 3)], *ai = &sa[1][s][3 + (lane & 3)], *as = &sa[2][s][3 + (lane & 3)];
      const double *vr = &sa[0][s][3], *vi = &sa[1][s][3];
#pragma unroll
      for (int q = 0; q <= 2 * p; ++q) {
        cx<double> hq[NT], hm[NT];
        double sq[NT], sm[NT];
#pragma unroll
        for (int tt = 0; tt < NT; ++tt) {
          if (q == 0) {
            hq[tt] = hm[tt] = hp[tt];  // H_0
          } else {
            if (q >= 2) {
              // not a running sum of 2 / z: its roundings add up to four times the error of h_32
              const double f = (q - 1) * tz[tt];  // 2 (q - 1) / z
              const cx<double> hn = mk(fma(f, hc[tt].re, -hp[tt].re), fma(f, hc[tt].im, -hp[tt].im));
              hp[tt] = hc[tt];
              hc[tt] = hn;
              tq[tt] = tq[tt] * t[tt];
            }
            // h_q = H_q e^{iq phi}, h_{-q} = (-1)^q H_q e^{-iq phi}: two shared products
            const double a = hc[tt].re * tq[tt].re, d = hc[tt].re * tq[tt].im;
            hq[tt] = mk(fma(-hc[tt].im, tq[tt].im, a), fma(hc[tt].im, tq[tt].re, d));
            hm[tt] = q & 1 ? mk(fma(-hc[tt].im, tq[tt].im, -a), fma(-hc[tt].im, tq[tt].re, d))
                           : mk(fma(hc[tt].im, tq[tt].im, a), fma(hc[tt].im, tq[tt].re, -d));
          }
          if (VROW) cmac(zc[tt], hm[tt], mk(vr[2 * p - q], vi[2 * p - q]));
          sq[tt] = hq[tt].re + hq[tt].im;
          sm[tt] = hm[tt].re + hm[tt].im;
        }
        // q: blocks with 4 R <= 2 p - q; -q: blocks with 4 R + 3 >= q
#pragma unroll
        for (int R = 0; R < NR; ++R) {
          if (4 * R <= 2 * p - q) {
            const double xr = ar[4 * R + q], xi = ai[4 * R + q], xs = as[4 * R + q];
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) {
              acc[tt][R][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(xr, hq[tt].re, acc[tt][R][0], 0, 0, 0);
              acc[tt][R][1] = __builtin_amdgcn_mfma_f64_4x4x4f64(xi, hq[tt].im, acc[tt][R][1], 0, 0, 0);
              acc[tt][R][2] = __builtin_amdgcn_mfma_f64_4x4x4f64(xs, sq[tt], acc[tt][R][2], 0, 0, 0);
            }
          }
          if (q > 0 && 4 * R + 3 >= q) {
            const double xr = ar[4 * R - q], xi = ai[4 * R - q], xs = as[4 * R - q];
#pragma unroll
            for (int tt = 0; tt < NT; ++tt) {
              acc[tt][R][0] = __builtin_amdgcn_mfma_f64_4x4x4f64(xr, hm[tt].re, acc[tt][R][0], 0, 0, 0);
              acc[tt][R][1] = __builtin_amdgcn_mfma_f64_4x4x4f64(xi, hm[tt].im, acc[tt][R][1], 0, 0, 0);
              acc[tt][R][2] = __builtin_amdgcn_mfma_f64_4x4x4f64(xs, sm[tt], acc[tt][R][2], 0, 0, 0);
            }
          }
        }
        // one q step at a time keeps the live registers to one step's operands
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  // lane i holds slot 4 R + i / 16 of target i % 16
  double2 *o = part + static_cast<int64_t>(c) * n * P;
#pragma unroll
  for (int tt = 0; tt < NT; ++tt) {
    const int l = lt0 + tt * 16 + r;
    cx<double> z = zc[tt];
    z.re += __shfl_xor(z.re, 16);
    z.im += __shfl_xor(z.im, 16);
    z.re += __shfl_xor(z.re, 32);
    z.im += __shfl_xor(z.im, 32);
    if (l >= n) continue;
    if (VROW && g == 0) o[static_cast<int64_t>(l) * P + 2 * p] = st(z);
#pragma unroll
    for (int R = 0; R < NR; ++R) {
      const int row = 4 * R + g;
      const double p1 = acc[tt][R][0], p2 = acc[tt][R][1], p3 = acc[tt][R][2];
      if (row < P - (VROW ? 1 : 0)) o[static_cast<int64_t>(l) * P + row] = make_double2(p1 - p2, p3 - p1 - p2);
    }
  }
}

// ---------------------------------------------------------------------------
// Row a1 in FP32 on the bf16 matrix cores, one right-hand side: the same
// product of shifted source coefficients and pair Hankel values as above,
//   alpha_l[s'] = sum_{m, q} A_m[s'][q] h_q(m -> l),  A_m[s'][q] = beta_m[s' + q]
// (slots s' = n' + p), with every FP32 operand split into three bf16 parts,
// x = x1 + x2 + x3 (rounding to nearest leaves 9 more bits to each next part, so
// the 24 bits of x fit), and the six products whose parts' weights reach 2^-18
// (11, 12, 21, 22, 13, 31) accumulated in FP32; the three left out are below
// 2^-26 of the product, less than the rounding of one FP32 multiply.  The split
// is exact where the last bit of x stays above the smallest bf16 subnormal,
// 2^-133, and x1 rounds to a finite number, below 3.39e38.  Coefficients reach
// below that range (high orders of small particles, vectors of small norm), so
// those of a batch are scaled by 2^24, which brings every FP32 number into it,
// and the pairs' Hankel values by 2^-24 (they are far above it, and their
// recurrence is linear): the products stay as they were.  A batch with a
// coefficient of 2^100 or more takes 2^-4 and 2^4 (BfScale).
// Complex products take four real ones (no operand sums), each in its own
// accumulators.  The matrix cores' bf16 sums do not round to nearest, so a
// long chain of them drifts (chunks of 316 sources: 5.9e-7 relative error of a
// 5000-particle matvec, of 40: 4.5e-7); after every batch of sources they are
// added to running FP32 sums and start again from zero.
//
// Why: an FP32 MFMA and FP32 vector instructions do not overlap on this chip (a
// 16x16x4 costs 32.4 cycles, a multiply-add beside it 3.3 .. 4.9 more), and
// the FP32 matrix kernel spent 288 of them and ~1000 vector instructions per
// group of 64 pairs.  Six bf16 MFMAs at 16x the rate replace one: 288 of 16
// cycles with the four-product form, and ~1280 vector instructions (the
// recurrence, the products with e^{iq phi}, the splitting), in turn as well
// where a wave issues its MFMAs back to back.  Interleaving them one to three
// did not help (each instruction then takes 5.3 cycles), nor did dot products
// for the remainders (they share the matrix pipe).  5000 particles, p = 16:
// 1.96 -> 1.55 ms; the matvec's error against 64 bits 4.6e-7 -> 4.0e-7.
//
// Layout.  One wave per 16 targets; a 16x16x32 MFMA takes four sources and
// eight consecutive q: lane i runs the recurrence of the pair (source i / 16
// of the group -> target i % 16) and its eight h_q are its B operand.  q goes
// in octets, {8j + 1 .. 8j + 8} and {-8j .. -8j - 7}.  The A operand of output
// rows 16 b + r and an octet is eight consecutive coefficients from slot
// r + 1 + 8 t, with t = 2 b + j or 2 b - j - 1: the LDS holds every source's
// parts zero-padded and in four copies, shifted by 0 .. 3 entries, so that each
// lane reads its eight with two aligned 8-byte reads.  For 2 p + 1 = 16 NB + 1
// (p = 8, 16) the last row runs on the vector units.
constexpr int kM2lBfWaves = 4;
constexpr int kM2lBfBatch = 8;                       // sources staged at a time
constexpr int kBfRow = 80;                           // entries of one shifted copy (64 used), 2 bytes each
constexpr int kBfSrc = 6 * 4 * kBfRow + 32;          // entries per source: [part][re, im][copy], bank offset
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The power of two by which coefficients are multiplied before their split, and
// its inverse for the Hankel values they meet.
struct BfScale {
  float up, down;
};
__device__ __forceinline__ bool bf_big(float2 b) {  // also true for a NaN
  return !(fabsf(b.x) < 0x1p100f && fabsf(b.y) < 0x1p100f);
}
__device__ __forceinline__ BfScale bf_scale(bool big) {
  return big ? BfScale{0x1p-4f, 0x1p4f} : BfScale{0x1p24f, 0x1p-24f};
}

// Eight FP32 values as three bf16 parts (round to nearest; the remainders are
// exact within the range above).
struct Split8 {
  bf8 v[3];
};
__device__ __forceinline__ Split8 split8(const float (&x)[8]) {
  Split8 o;
#pragma unroll
  for (int i = 0; i < 8; i += 2) {
    f32x2 r = {x[i], x[i + 1]};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const bf2 h = __builtin_convertvector(r, bf2);
      o.v[k][i] = h[0];
      o.v[k][i + 1] = h[1];
      if (k < 2) r = r - __builtin_convertvector(h, f32x2);
    }
  }
  return o;
}

template <int p, int NT>
__global__ __launch_bounds__(64 * kM2lBfWaves, NT == 1 ? 3 : 2) void k_m2l_bf(const float2 *__restrict__ pairs,
                                                             const float2 *__restrict__ beta,
                                                             float2 *__restrict__ part, int n, int chunk_len,
                                                             int64_t bstride, int64_t pstride) {
  static_assert(p >= 1 && p <= 16, "two 16-row blocks");
  constexpr int P = 2 * p + 1;
  constexpr bool VROW = P % 16 == 1 && P > 1;  // slot 2p on the vector units
  constexpr int NB = (P - (VROW ? 1 : 0) + 15) / 16;
  constexpr int NJ = (2 * p + 7) / 8;          // octets of q > 0
  constexpr int NM = (P - (VROW ? 1 : 0) + 7) / 8;  // octets of q <= 0 that the matrix rows need
  constexpr int NO = NJ > NM ? NJ : NM;
  static_assert(NO <= 4, "octets");
  // The matrix cores' sums are rounded downwards, so the errors of one source
  // after another add up (700 particles, p = 4: 1.2 times the vector form's error).
  // Up to p = 7, where that shows most, each octet's products start from zero, are
  // added to acc rounded to nearest, and every second group of four sources is
  // multiplied negated (0.9 times; 2000 particles, p = 7: 127 -> 131 us a matvec;
  // with two row blocks the registers spill, 12 % at p = 10).  From p = 9 every
  // second batch is negated (p = 10: 1.02 -> 1.00 times); with a row on the vector
  // units neither (p = 8: 1.02 times with or without; p = 16: 5 % slower).
  constexpr bool RN = NB == 1 && !VROW, ALT = !VROW;
  constexpr int SB = kM2lBfBatch;
  typedef float v4 __attribute__((ext_vector_type(4)));
  __shared__ __align__(16) __bf16 sa[SB * kBfSrc];
  __shared__ float2 sv[VROW ? SB : 1][VROW ? P : 1];
  __shared__ v4 run[kM2lBfWaves][NT * NB * 2][64];  // sums over the batches, each lane its own entries
  __shared__ int sbig[kM2lBfWaves];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const int c = blockIdx.y;
  beta += blockIdx.z * bstride;
  part += blockIdx.z * pstride;
  const int m0 = c * chunk_len;
  const int m1 = min(n, m0 + chunk_len);
  const int lt0 = (blockIdx.x * kM2lBfWaves + w) * 16 * NT;

  for (int e = threadIdx.x; e < SB * kBfSrc / 8; e += 64 * kM2lBfWaves)
    reinterpret_cast<float4 *>(sa)[e] = make_float4(0.f, 0.f, 0.f, 0.f);

  v4 acc[NT][NB][4];  // Ar Br, Ai Bi, Ar Bi, Ai Br
  cx<float> zc[NT];
#pragma unroll
  for (int tt = 0; tt < NT; ++tt) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int k = 0; k < 4; ++k) acc[tt][b][k] = v4{0, 0, 0, 0};
    zc[tt] = mk(0.f, 0.f);
  }
#pragma unroll
  for (int x = 0; x < NT * NB * 2; ++x) run[w][x][lane] = v4{0, 0, 0, 0};
  float2 pa[NT][4];
  auto load_pairs = [&](int m) {
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) {
      const int l = lt0 + tt * 16 + r;
      if (m < m1 && l < n) {
        const float2 *pe = pairs + 4 * (static_cast<int64_t>(m) * n + l);
#pragma unroll
        for (int k = 0; k < 4; ++k) pa[tt][k] = pe[k];
      } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) pa[tt][k] = make_float2(0.f, 0.f);
      }
    }
  };
  load_pairs(m0 + g);

  for (int mb = m0; mb < m1; mb += SB) {
    const int sb = min(SB, m1 - mb);
    constexpr int NL = (SB * P + 64 * kM2lBfWaves - 1) / (64 * kM2lBfWaves);
    float2 bl[NL];
    bool big = false;
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int e = threadIdx.x + 64 * kM2lBfWaves * i;
      bl[i] = e < sb * P ? beta[static_cast<int64_t>(mb) * P + e] : make_float2(0.f, 0.f);
      big |= bf_big(bl[i]);
    }
    big = __any(big);
    if (lane == 0) sbig[w] = big;
    __syncthreads();  // previous batch consumed (and the zero fill done)
    static_assert(kM2lBfWaves == 4, "flags of four waves");
    const BfScale sc = bf_scale((sbig[0] | sbig[1] | sbig[2] | sbig[3]) != 0);
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int e = threadIdx.x + 64 * kM2lBfWaves * i;
      if (e < SB * P) {
        const int s = e / P, v = e - s * P;
        float x[2] = {bl[i].x * sc.up, bl[i].y * sc.up};
        if (VROW) sv[s][v] = make_float2(x[0], x[1]);
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const __bf16 h = static_cast<__bf16>(x[j]);
            x[j] -= static_cast<float>(h);
            __bf16 *o = sa + s * kBfSrc + (2 * k + j) * 4 * kBfRow + v + 15;  // copy u holds slot v at v + 15 - u
#pragma unroll
            for (int u = 0; u < 4; ++u) o[u * kBfRow - u] = h;
          }
      }
    }
    __syncthreads();
    // a wave whose targets all lie past the last particle (the grid's tail)
    // stages its share of the batch and meets the barriers, but multiplies nothing
    for (int g0 = 0; g0 < sb && lt0 < n; g0 += 4) {
      const int s = g0 + g;  // this lane's source within the batch
      const float sg = ALT && (RN ? g0 / 4 : mb / SB) & 1 ? -1.f : 1.f, down = sg * sc.down;
      float2 pc[NT][4];
#pragma unroll
      for (int tt = 0; tt < NT; ++tt)
#pragma unroll
        for (int k = 0; k < 4; ++k) pc[tt][k] = pa[tt][k];
      load_pairs(mb + s + 4);  // next group's entries in flight
      // entry r + 16 + 8 t of the zero-padded row starts at copy r % 4, entry 4 (r / 4) + 16 + 8 t
      const __bf16 *as = sa + s * kBfSrc + (r & 3) * kBfRow + (r & ~3) + 16;
      auto frag = [&](int k, int i, int tt) {
        const bf4 *a = reinterpret_cast<const bf4 *>(as + (2 * k + i) * 4 * kBfRow + 8 * tt);
        const bf4 lo = a[0], hi = a[1];
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      };
#pragma unroll
      for (int tt = 0; tt < NT; ++tt) {
        cx<float> hp = down * ld<float>(pc[tt][0]), hc = down * ld<float>(pc[tt][1]);
        const cx<float> t = ld<float>(pc[tt][2]);
        cx<float> tq = t;
        const float tz = pc[tt][3].x;
        // products of one octet (B parts br, bi) with the fragments t0 + 2 b of the blocks [b0, b1)
        auto mul = [&](const Split8 &br, const Split8 &bi, int t0, auto b0c, auto b1c) {
          constexpr int b0 = decltype(b0c)::value, b1 = decltype(b1c)::value;
          if constexpr (b0 < b1) {
            constexpr int ka[6] = {0, 0, 1, 0, 1, 2}, kb[6] = {2, 1, 1, 0, 0, 0};
            bf8 ar[NB][3], ai[NB][3];
#pragma unroll
            for (int b = b0; b < b1; ++b)
#pragma unroll
              for (int k = 0; k < 3; ++k) {
                ar[b][k] = frag(k, 0, t0 + 2 * b);
                ai[b][k] = frag(k, 1, t0 + 2 * b);
              }
            v4 sum[NB][4];
#pragma unroll
            for (int b = b0; b < b1; ++b)
#pragma unroll
              for (int k = 0; k < 4; ++k) sum[b][k] = RN ? v4{0, 0, 0, 0} : acc[tt][b][k];
#pragma unroll
            for (int x = 0; x < 6; ++x)
#pragma unroll
              for (int b = b0; b < b1; ++b) {
                sum[b][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar[b][ka[x]], br.v[kb[x]], sum[b][0], 0, 0, 0);
                sum[b][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ai[b][ka[x]], bi.v[kb[x]], sum[b][1], 0, 0, 0);
                sum[b][2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar[b][ka[x]], bi.v[kb[x]], sum[b][2], 0, 0, 0);
                sum[b][3] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ai[b][ka[x]], br.v[kb[x]], sum[b][3], 0, 0, 0);
              }
#pragma unroll
            for (int b = b0; b < b1; ++b)
#pragma unroll
              for (int k = 0; k < 4; ++k) acc[tt][b][k] = RN ? acc[tt][b][k] + sg * sum[b][k] : sum[b][k];
          }
        };
        float pr[8], pi[8], nr[8], ni[8];  // h_{8j+1 ..} and h_{-8j-7 ..}
        auto octet = [&](auto jc) {
          constexpr int j = decltype(jc)::value;
          // q = 8 j .. 8 j + 8; the last one's h_{-q} opens the next octet
#pragma unroll
          for (int u = 0; u <= 8; ++u) {
            const int q = 8 * j + u;
            if (u == 0 && j > 0) continue;  // done at the end of the previous octet
            cx<float> hq = mk(0.f, 0.f), hm = mk(0.f, 0.f);
            if (q == 0) {
              hm = hp;  // H_0
            } else if (q <= 2 * p) {
              if (q >= 2) {
                const cx<float> hn = static_cast<float>(q - 1) * tz * hc - hp;
                hp = hc;
                hc = hn;
                tq = tq * t;
              }
              // h_q = H_q e^{iq phi}, h_{-q} = (-1)^q H_q e^{-iq phi}: two shared products
              const float a = hc.re * tq.re, d = hc.re * tq.im;
              hq = mk(fmaf(-hc.im, tq.im, a), fmaf(hc.im, tq.re, d));
              hm = q & 1 ? mk(fmaf(-hc.im, tq.im, -a), fmaf(-hc.im, tq.re, d))
                         : mk(fmaf(hc.im, tq.im, a), fmaf(hc.im, tq.re, -d));
            }
            if (VROW && q <= 2 * p) cmac(zc[tt], hm, ld<float>(sv[s][VROW ? 2 * p - q : 0]));
            if (u > 0) {
              pr[u - 1] = hq.re;
              pi[u - 1] = hq.im;
            }
            if (u == 8) {  // opens the next octet of q <= 0, after this one is used
              const Split8 br = split8(nr), bi = split8(ni);
              // q <= 0: block b needs q >= -16 b - 15, fragment t = 2 b - j - 1
              mul(br, bi, -j - 1, std::integral_constant<int, (j < NM ? (j / 2 < NB ? j / 2 : NB) : NB)>{},
                  std::integral_constant<int, NB>{});
              nr[7] = hm.re;
              ni[7] = hm.im;
            } else {
              nr[7 - u] = hm.re;
              ni[7 - u] = hm.im;
            }
          }
          // q > 0: block b needs q <= 2 p - 16 b, fragment t = 2 b + j
          constexpr int top = 8 * j + 1 <= 2 * p ? (2 * p - 8 * j - 1) / 16 + 1 : 0;
          if constexpr (top > 0) {
            const Split8 br = split8(pr), bi = split8(pi);
            mul(br, bi, j, std::integral_constant<int, 0>{}, std::integral_constant<int, (top < NB ? top : NB)>{});
          }
          __builtin_amdgcn_sched_barrier(0);
        };
        octet(std::integral_constant<int, 0>{});
        if constexpr (NO > 1) octet(std::integral_constant<int, 1>{});
        if constexpr (NO > 2) octet(std::integral_constant<int, 2>{});
        if constexpr (NO > 3) octet(std::integral_constant<int, 3>{});
      }
    }
    // the batch's products into the running sums (rounded to nearest)
    const float bsg = ALT && !RN && (mb / SB) & 1 ? -1.f : 1.f;
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        v4 *s = &run[w][(tt * NB + b) * 2][lane];
        s[0] = s[0] + bsg * (acc[tt][b][0] - acc[tt][b][1]);
        s[64] = s[64] + bsg * (acc[tt][b][2] + acc[tt][b][3]);
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[tt][b][k] = v4{0, 0, 0, 0};
      }
  }
  float2 *o = part + static_cast<int64_t>(c) * n * P;
#pragma unroll
  for (int tt = 0; tt < NT; ++tt) {
    const int l = lt0 + tt * 16 + r;
    cx<float> z = zc[tt];
    z.re += __shfl_xor(z.re, 16);
    z.im += __shfl_xor(z.im, 16);
    z.re += __shfl_xor(z.re, 32);
    z.im += __shfl_xor(z.im, 32);
    if (l >= n) continue;
    if (VROW && g == 0) o[static_cast<int64_t>(l) * P + 2 * p] = st(z);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      const v4 *s = &run[w][(tt * NB + b) * 2][lane];
      const v4 re = s[0], im = s[64];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = 16 * b + 4 * g + j;
        if (row < P - (VROW ? 1 : 0)) o[static_cast<int64_t>(l) * P + row] = make_float2(re[j], im[j]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Row a1 for many right-hand sides on the matrix cores (FP32): per pair the
// Toeplitz translation T^{ml}[n'][nu] = h_{nu-n'} is built once and applied to
// the coefficients of 64 right-hand sides as a GEMM  alpha_l[n'][r] +=
// sum_nu T[n'][nu] beta_m[nu][r]  with 16x16x4 MFMA (M = n', K = nu, N = r),
// complex products in three real MFMAs (Gauss).  One wave per target, kMrhsWaves
// targets per block, grid.y source chunks, grid.z groups of 64 right-hand
// sides.  Lanes 0..7 of each wave run the Hankel recurrences of 8 sources
// at a time (from the pair table, as in k_m2l) into zero-padded LDS rows;
// the A operand is read from there.  The B operand, beta transposed to
// [m][nu][r] (r fastest, zero rows and columns as padding), is staged per
// source in LDS for all waves of the block, double-buffered: the next
// source's loads are in flight during the current source's MFMAs.
//
// The error grows with the length of the sums.  With one row block (p <= 7) they
// are added to running ones every `run` batches, so that a chunk's length
// costs no accuracy (700 particles, 16 right-hand sides, p = 1: 1.08 -> 0.99 times
// the error of twelve chunks; every batch would cost 4 %).
constexpr int kMrhsWaves = 8;
constexpr int kMrhsBatch = 8;

template <int p>
__global__ __launch_bounds__(64 * kMrhsWaves) void k_m2l_mrhs(const float2 *__restrict__ pairs,
                                                              const float2 *__restrict__ bt,
                                                              float2 *__restrict__ part, int n, int chunk_len,
                                                              int nrhs, int r_pad, int64_t pstride, int run) {
  constexpr int P = 2 * p + 1;
  constexpr int MT = (P + 15) / 16;
  constexpr int KP = (P + 3) / 4 * 4;
  constexpr int NT = 4;                      // 64 right-hand sides per block
  constexpr bool RUN = MT == 1;              // running sums: registers for them
  constexpr int OFF = 16 * MT - 1;           // H index of q = k - row is q + OFF
  constexpr int HQ = KP + OFF;               // zero outside |q| <= 2p
  constexpr int BE = KP * 64;                // B entries of one source
  constexpr int BL = (BE + 64 * kMrhsWaves - 1) / (64 * kMrhsWaves);  // loads per thread
  __shared__ float2 H[kMrhsWaves][kMrhsBatch][HQ];
  __shared__ float2 Bs[2][KP][64];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int l = blockIdx.x * kMrhsWaves + w;
  const int c = blockIdx.y;
  const int r0 = blockIdx.z * 64;
  const int m0 = c * chunk_len;
  const int m1 = min(n, m0 + chunk_len);
  typedef float v4 __attribute__((ext_vector_type(4)));
  // Gauss: P1 = sum Ar Br, P2 = sum Ai Bi, P3 = sum (Ar + Ai)(Br + Bi)
  v4 P1[MT][NT], P2[MT][NT], P3[MT][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) P1[mt][ct] = P2[mt][ct] = P3[mt][ct] = v4{0, 0, 0, 0};
  v4 Sr[NT], Si[NT];  // RUN: running sums
#pragma unroll
  for (int ct = 0; ct < NT; ++ct) Sr[ct] = Si[ct] = v4{0, 0, 0, 0};
  const int col = lane & 15, kq = lane >> 4;
  // B of source m: rows k (zero rows k >= P in bt), 64 right-hand sides
  float2 pre[BL];
  auto load_b = [&](int m) {
#pragma unroll
    for (int i = 0; i < BL; ++i) {
      const int e = threadIdx.x + 64 * kMrhsWaves * i;
      pre[i] = (m < m1 && e < BE) ? bt[(static_cast<int64_t>(m) * KP + e / 64) * r_pad + r0 + (e & 63)]
                                  : make_float2(0.f, 0.f);
    }
  };
  auto store_b = [&](int buf) {
#pragma unroll
    for (int i = 0; i < BL; ++i) {
      const int e = threadIdx.x + 64 * kMrhsWaves * i;
      if (e < BE) Bs[buf][e / 64][e & 63] = pre[i];
    }
  };
  load_b(m0);
  int it = 0;
  for (int mb = m0; mb < m1; mb += kMrhsBatch) {
    const int sb = min(kMrhsBatch, m1 - mb);
    for (int i = lane; i < kMrhsBatch * HQ; i += 64) H[w][i / HQ][i % HQ] = make_float2(0.f, 0.f);
    __syncthreads();
    if (lane < sb) {  // h_q of pair (mb + lane -> l), q = -2p..2p
      const int m = mb + lane;
      float2 *h = H[w][lane] + OFF;
      if (l < n && m != l) {
        const float2 *pe = pairs + 4 * (static_cast<int64_t>(m) * n + l);
        cx<float> hp = ld<float>(pe[0]), hc = ld<float>(pe[1]);
        const cx<float> t = ld<float>(pe[2]);
        const float tz = pe[3].x;
        h[0] = st(hp);
        cx<float> tq = t;
        for (int q = 1; q <= 2 * p; ++q) {
          if (q >= 2) {
            const cx<float> hn = static_cast<float>(q - 1) * tz * hc - hp;
            hp = hc;
            hc = hn;
            tq = tq * t;
          }
          h[q] = st(hc * tq);
          cx<float> hm = hc * conj(tq);
          if (q & 1) hm = mk<float>(-hm.re, -hm.im);
          h[-q] = st(hm);
        }
      }
    }
    for (int s = 0; s < sb; ++s, ++it) {
      const int buf = it & 1;
      store_b(buf);          // B of source mb + s (loaded one iteration ahead)
      __syncthreads();
      load_b(mb + s + 1);    // next source's B in flight during the MFMAs
      const float2 *hrow = H[w][s];
#pragma unroll
      for (int k0 = 0; k0 < KP; k0 += 4) {
        const int k = k0 + kq;
        float br[NT], bi[NT], bs[NT];
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
          const float2 bv = Bs[buf][k][ct * 16 + col];
          br[ct] = bv.x;
          bi[ct] = bv.y;
          bs[ct] = bv.x + bv.y;
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const float2 a = hrow[k - (mt * 16 + col) + OFF];
          const float as = a.x + a.y;
#pragma unroll
          for (int ct = 0; ct < NT; ++ct) {
            P1[mt][ct] = mfma4<float>::mac(a.x, br[ct], P1[mt][ct]);
            P2[mt][ct] = mfma4<float>::mac(a.y, bi[ct], P2[mt][ct]);
            P3[mt][ct] = mfma4<float>::mac(as, bs[ct], P3[mt][ct]);
          }
        }
      }
    }
    if constexpr (RUN) {
      if (((mb - m0) / kMrhsBatch + 1) % run == 0 || mb + kMrhsBatch >= m1) {
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
          Sr[ct] += P1[0][ct] - P2[0][ct];
          Si[ct] += P3[0][ct] - P1[0][ct] - P2[0][ct];
          P1[0][ct] = P2[0][ct] = P3[0][ct] = v4{0, 0, 0, 0};
        }
      }
    }
    __syncthreads();
  }
  if (l >= n) return;
  // result register j of lane i: row 4 (i / 16) + j, column i % 16
  const int64_t len = static_cast<int64_t>(n) * P;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int ct = 0; ct < NT; ++ct)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = mt * 16 + 4 * kq + j;
        const int r = r0 + ct * 16 + col;
        const float p1 = P1[mt][ct][j], p2 = P2[mt][ct][j], p3 = P3[mt][ct][j];
        if (row < P && r < nrhs)
          part[r * pstride + c * len + static_cast<int64_t>(l) * P + row] =
              RUN ? make_float2(Sr[ct][j], Si[ct][j]) : make_float2(p1 - p2, p3 - p1 - p2);
      }
}

// ---------------------------------------------------------------------------
// Row a1 for many right-hand sides on the bf16 matrix cores (FP32 operands in
// three bf16 parts and the six largest products of parts, scaled as in k_m2l_bf
// by one power of two per source and 64 right-hand sides), for 16 < 2p + 1 <= 32: per pair one 16x16x32 MFMA step covers all
// source orders.  alpha_l[n'][r] += sum_nu T[n'][nu] beta_m[nu][r] with
// T[n'][nu] = h_{nu - n'} (M = n' in two 16-row blocks, K = nu, N = r in four
// 16-column tiles); complex products in four real ones, re and im in one
// accumulator each (the imaginary part of T negated in registers).
//
// One wave per target, kMrhsWaves targets per block, grid.y source chunks,
// grid.z groups of 64 right-hand sides.  Lanes 0..7 run the Hankel recurrences
// of 8 sources at a time into FP32 rows; per source each lane splits one h_q
// and stores its parts in four copies, shifted by 0 .. 3 entries, from which
// the A operand (eight consecutive q, ending at a lane's row) is read with
// aligned 8-byte reads.  B, beta transposed as for the FP32 form, is split while
// it is staged, four source orders of one right-hand side per thread, once per
// source for all waves of the block, double-buffered, between the MFMAs.  (Split
// beforehand, the parts were 1.5 to 2.4 times the size of the transposed beta,
// which a context's memory budget may not have; the matvec of the case below
// took 8.46 ms with them, 8.54 ms without.)  The matrix cores' bf16 sums do not
// round to nearest, so they are added to running FP32 sums after every batch of
// 8 sources and start again from zero.
//
// Bound by the matrix cores: 192 MFMAs of 16 cycles per pair and 64 right-hand
// sides, where the FP32 form above needs 3 MT KP NT / 4 = 168 of 32.4 (p = 12).
// 64 right-hand sides, 2000 particles, p = 12: 10.9 -> 8.0 ms (MFMAs 66 % of the
// cycles), the batch's error against 64 bits 1.3e-6 -> 1.0e-6.
template <int p>
__global__ __launch_bounds__(64 * kMrhsWaves) void k_m2l_mrhs_bf(const float2 *__restrict__ pairs,
                                                                 const float2 *__restrict__ bt,
                                                                 float2 *__restrict__ part, int n, int chunk_len,
                                                                 int nrhs, int r_pad, int64_t pstride) {
  constexpr int P = 2 * p + 1;
  static_assert(P > 16 && P <= 32, "two row blocks, one K step");
  constexpr int MT = 2, NT = 4;
  constexpr int OFF = 31;                    // row entry of h_q is q + OFF
  constexpr int KP = (P + 3) / 4 * 4;        // rows of bt per source
  constexpr int PR = 6 * 64 * 32;            // B entries of one source
  static_assert(4 * kMrhsWaves == 32, "four source orders per wave");
  typedef float v4 __attribute__((ext_vector_type(4)));
  __shared__ float2 H[kMrhsWaves][kMrhsBatch][65];
  __shared__ __align__(16) __bf16 Hs[2][kMrhsWaves][6][4][kBfRow];
  __shared__ __align__(16) __bf16 Bs[2][PR];  // [part, re / im][nu / 8][r][nu % 8]: a read's 16 columns are contiguous
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int l = blockIdx.x * kMrhsWaves + w;
  const int c = blockIdx.y;
  const int r0 = blockIdx.z * 64;
  const int m0 = c * chunk_len;
  const int m1 = min(n, m0 + chunk_len);
  const int col = lane & 15, kq = lane >> 4;
  v4 acc[MT][NT][2];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) acc[mt][ct][0] = acc[mt][ct][1] = v4{0, 0, 0, 0};
  float2 pre[4];  // this thread's source orders 4 w .. 4 w + 3 of right-hand side r0 + lane
  auto load_b = [&](int m) {
    const int64_t mc = min(m, n - 1);  // past the chunk: loaded, never used
#pragma unroll
    for (int i = 0; i < 4; ++i)
      pre[i] = 4 * w + i < P ? bt[(mc * KP + 4 * w + i) * r_pad + r0 + lane] : make_float2(0.f, 0.f);
  };
  auto store_b = [&](int buf, int j) {  // real (j = 0) or imaginary parts
    {
      f32x2 x[2];
#pragma unroll
      for (int i = 0; i < 2; ++i)
        x[i] = j ? f32x2{pre[2 * i].y, pre[2 * i + 1].y} : f32x2{pre[2 * i].x, pre[2 * i + 1].x};
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        bf2 h[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          h[i] = __builtin_convertvector(x[i], bf2);
          if (k < 2) x[i] = x[i] - __builtin_convertvector(h[i], f32x2);
        }
        *reinterpret_cast<bf4 *>(&Bs[buf][(((2 * k + j) * 4 + w / 2) * 64 + lane) * 8 + w % 2 * 4]) =
            __builtin_shufflevector(h[0], h[1], 0, 1, 2, 3);
      }
    }
  };
  // sums of the sources since the last flush into the running ones
  v4 run[MT][NT][2];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) run[mt][ct][0] = run[mt][ct][1] = v4{0, 0, 0, 0};
  auto flush = [&]() {
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int ct = 0; ct < NT; ++ct)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          run[mt][ct][i] += acc[mt][ct][i];
          acc[mt][ct][i] = v4{0, 0, 0, 0};
        }
  };
  load_b(m0);
  int it = 0;
  for (int mb = m0; mb < m1; mb += kMrhsBatch) {
    const int sb = min(kMrhsBatch, m1 - mb);
    // each wave fills its own rows (one wave's LDS accesses stay in order)
    for (int i = lane; i < kMrhsBatch * 64; i += 64) H[w][i / 64][i % 64] = make_float2(0.f, 0.f);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (lane < sb) {  // h_q of pair (mb + lane -> l), q = -2p..2p
      const int m = mb + lane;
      float2 *h = H[w][lane] + OFF;
      if (l < n && m != l) {
        const float2 *pe = pairs + 4 * (static_cast<int64_t>(m) * n + l);
        // times the inverse of the source's power of two
        const float down = bt[(static_cast<int64_t>(m) * KP + KP - 1) * r_pad + r0].x;
        cx<float> hp = down * ld<float>(pe[0]), hc = down * ld<float>(pe[1]);
        const cx<float> t = ld<float>(pe[2]);
        const float tz = pe[3].x;
        h[0] = st(hp);
        cx<float> tq = t;
        for (int q = 1; q <= 2 * p; ++q) {
          if (q >= 2) {
            const cx<float> hn = static_cast<float>(q - 1) * tz * hc - hp;
            hp = hc;
            hc = hn;
            tq = tq * t;
          }
          h[q] = st(hc * tq);
          cx<float> hm = hc * conj(tq);
          if (q & 1) hm = mk<float>(-hm.re, -hm.im);
          h[-q] = st(hm);
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // parts of the h of source s of the batch: copy u holds entry x at x + 3 - u
    auto split_h = [&](int s, int buf) {
      const float2 h = H[w][s][lane];
      float x[2] = {h.x, h.y};
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const __bf16 b = static_cast<__bf16>(x[i]);
          x[i] -= static_cast<float>(b);
#pragma unroll
          for (int u = 0; u < 4; ++u) Hs[buf][w][2 * k + i][u][lane + 3 - u] = b;
        }
    };
    split_h(0, it & 1);
    if (it == 0) {
      store_b(0, 0);
      store_b(0, 1);
    }
    for (int s = 0; s < sb; ++s, ++it) {
      const int buf = it & 1;
      __syncthreads();       // B and the parts of h of this source stored
      load_b(mb + s + 1);    // the next source's, beside the MFMAs
      if (s + 1 < sb) split_h(s + 1, buf ^ 1);
      const __bf16 *bs = Bs[buf] + (kq * 64 + col) * 8;
      bf8 ar[MT][3], ai[MT][3], an[MT][3];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        // h_{nu - n'} for nu = 8 kq + 0 .. 7, n' = 16 mt + col: entries from x0
        const int x0 = 8 * kq - 16 * mt - col + OFF + 3;
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          const bf4 *a = reinterpret_cast<const bf4 *>(&Hs[buf][w][2 * k][x0 & 3][x0 & ~3]);
          const bf4 *b = reinterpret_cast<const bf4 *>(&Hs[buf][w][2 * k + 1][x0 & 3][x0 & ~3]);
          ar[mt][k] = __builtin_shufflevector(a[0], a[1], 0, 1, 2, 3, 4, 5, 6, 7);
          ai[mt][k] = __builtin_shufflevector(b[0], b[1], 0, 1, 2, 3, 4, 5, 6, 7);
          an[mt][k] = __builtin_bit_cast(bf8, __builtin_bit_cast(u32x4, ai[mt][k]) ^ 0x80008000u);
        }
      }
#pragma unroll
      for (int ct = 0; ct < NT; ++ct) {
        bf8 br[3], bi[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
          br[k] = *reinterpret_cast<const bf8 *>(bs + (2 * k) * 64 * 32 + ct * 16 * 8);
          bi[k] = *reinterpret_cast<const bf8 *>(bs + (2 * k + 1) * 64 * 32 + ct * 16 * 8);
        }
        constexpr int ka[6] = {0, 0, 1, 0, 1, 2}, kb[6] = {2, 1, 1, 0, 0, 0};
#pragma unroll
        for (int x = 0; x < 6; ++x) {
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            acc[mt][ct][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar[mt][ka[x]], br[kb[x]], acc[mt][ct][0], 0, 0, 0);
            acc[mt][ct][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ar[mt][ka[x]], bi[kb[x]], acc[mt][ct][1], 0, 0, 0);
          }
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) {
            acc[mt][ct][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(an[mt][ka[x]], bi[kb[x]], acc[mt][ct][0], 0, 0, 0);
            acc[mt][ct][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ai[mt][ka[x]], br[kb[x]], acc[mt][ct][1], 0, 0, 0);
          }
        }
        if (ct == 1 || ct == 2) store_b(buf ^ 1, ct - 1);  // last read two sources ago
      }
    }
    flush();
  }
  if (l >= n) return;
  const int64_t len = static_cast<int64_t>(n) * P;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int ct = 0; ct < NT; ++ct)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = mt * 16 + 4 * kq + j, r = r0 + ct * 16 + col;
        if (row < P && r < nrhs)
          part[r * pstride + c * len + static_cast<int64_t>(l) * P + row] =
              make_float2(run[mt][ct][0][j], run[mt][ct][1][j]);
      }
}

// beta [r][m][P] -> bt [m][KP][r_pad] (r fastest; zero rows k >= P and
// zero columns r >= nrhs), FP32: one block per source and 64 right-hand sides,
// through LDS.  With scale (the bf16 form, which has its own zeros) the
// coefficients are multiplied by the power of two for their split, and the last
// row, KP - 1 >= P, holds its inverse.
template <int P>
__global__ __launch_bounds__(256) void k_rhs_transpose(const float2 *__restrict__ x, float2 *__restrict__ bt, int n,
                                                       int nrhs, int r_pad, bool scale) {
  constexpr int KP = (P + 3) / 4 * 4;
  static_assert(KP > P, "a spare row");
  __shared__ float2 t[P][65];
  const int64_t m = blockIdx.x;
  const int r0 = blockIdx.y * 64;
  bool big = false;
  for (int e = threadIdx.x; e < 64 * P; e += 256) {
    const int r = e / P, k = e - r * P;
    const float2 v = r0 + r < nrhs ? x[((r0 + r) * static_cast<int64_t>(n) + m) * P + k] : make_float2(0.f, 0.f);
    t[k][r] = v;
    big |= bf_big(v);
  }
  big = __syncthreads_or(big);
  const BfScale sc = scale ? bf_scale(big) : BfScale{1.f, 0.f};
  float2 *o = bt + m * KP * r_pad + r0;
  for (int e = threadIdx.x; e < 64 * KP; e += 256) {
    const int k = e / 64, r = e % 64;
    o[static_cast<int64_t>(k) * r_pad + r] = k < P ? make_float2(sc.up * t[k][r].x, sc.up * t[k][r].y)
                                                   : make_float2(k == KP - 1 ? sc.down : 0.f, 0.f);
  }
}

// ---------------------------------------------------------------------------
// Dispatch over the expansion order.
#define MPSL_P_CASES(X) \
  X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(17) \
  X(18) X(19) X(20)

}  // namespace

#define LAUNCH_CHECK(ctx)                                                          \
  do {                                                                             \
    hipError_t e_ = hipGetLastError();                                             \
    if (e_ != hipSuccess) return set_err(ctx, MPSL_EHIP, std::string("kernel launch: ") + hipGetErrorString(e_)); \
  } while (0)

// The matrix-core forms win from order 4 (FP64) and 6 (FP32) on (matvecs, one lane
// per target and matrix cores, us: FP32 p = 6, 1000 and 5000 particles 59 and 54,
// 704 and 641; p = 16 187 and 116, 3168 and 1781; FP64 p = 4 61 and 50, 536 and
// 542; p = 8 111 and 81, 1363 and 1193).  Below, the padding to 16 or 4 rows costs
// more than the vector units' work, once there are pairs enough for its one lane
// per target to fill the chip: FP32 p <= 5 from 1e6 pairs on (p = 4: 500 particles
// with one right-hand side 43 and 27, 1000 47 and 47, 2000 90 and 103, 5000 396
// and 493, 3000 with eight 973 and 1296), FP64 p <= 3 from 3e7 (p = 3: 1400 with
// eight 249 and 256, 3000 with 15 1734 and 1940, 5000 with two 791 and 840).
// FP64 takes 32 targets per wave up to p = 12 (they share the coefficient reads;
// at p = 16 the registers spill, 1245 against 1215 us at 3001 particles) once that
// leaves enough waves (p = 12, 16 and 32 targets: 300 particles 41.7 and 44.2 us,
// 600 71.2 and 71.0, 1000 130 and 125).
int m2l_default_variant(const mpsl_ctx *ctx, int prec, int nrhs) {
  if (ctx->p > kM2LMfmaMaxP) return kM2LWhole;
  const double pairs = static_cast<double>(ctx->n) * ctx->n * nrhs;
  if (prec == MPSL_FP64) {
    if (ctx->p <= 3 && pairs >= 3e7) return kM2LWhole;
    return ctx->p <= 12 && ctx->n >= 768 ? kM2LMfmaWide : kM2LMfma;
  }
  return ctx->p <= 5 && pairs >= 1e6 ? kM2LWhole : kM2LMfma;
}

static int m2l_variant(const mpsl_ctx *ctx, int prec, int nrhs) {
  int v = ctx->tune[prec == MPSL_FP64 ? 0 : 1].variant;
  if (v < 0) v = m2l_default_variant(ctx, prec, nrhs);
  if (v >= kM2LMfma && ctx->p > kM2LMfmaMaxP) v = kM2LWhole;
  return v;
}

// Source chunks of the matrix-core forms.  A compute unit works through its
// share of the blocks at a fixed rate, so a launch takes about
//   ceil(blocks / units) x (groups of four sources per chunk) x t_group
// (t_group: 260 P cycles FP32, 525 P FP64 per 16 targets and wave, measured), a
// sixth more while a unit has one block only, plus the writing and summing of
// the chunks' partials at HBM rate; the best of up to 128 counts.  (5000
// particles FP32: 42 chunks and 1.49 ms, as 125, which left 3x the partials to
// sum; 1000 particles FP64, p = 12: 63 chunks, 83 us.)  Right-hand sides multiply
// the blocks and the partials, and neither one nor several of them get more
// partial slots than m2l_slot_bound: partials of 20000 particles would take more
// memory than all other work buffers.  (1400 particles, 15 right-hand sides,
// FP64, p = 16: dividing the count of one left a single chunk, 330 blocks on 256
// units, 6.40 ms; the rule's count 3.98.  250 particles, 32 right-hand sides,
// FP64, p = 5: one chunk, 128 blocks, 163 us; the rule's count 90.)
static int m2l_slot_bound(const mpsl_ctx *ctx, int from) {
  // about 2560 blocks of 128 lanes, from order `from` on 10240 of 64
  const int n = static_cast<int>(ctx->n);
  if (ctx->p < from) return std::max(1, std::min(cdiv(2560, cdiv(n, kThreads)), n));
  return cdiv(n, m2l_mfma_chunk_len(n, std::max(1, std::min(cdiv(10240, cdiv(n, 64)), n))));
}

static int m2l_mfma_chunks(const mpsl_ctx *ctx, int prec, int nt, int nrhs) {
  const int n = static_cast<int>(ctx->n), P = 2 * ctx->p + 1;
  const int bpc = cdiv(n, 64 * nt) * nrhs, units = std::max(1, ctx->n_cu);
  // a context's partials hold one right-hand side of either precision
  const int slots = m2l_slot_bound(ctx, nrhs > 1 && prec == MPSL_FP64 ? 15 : 12) / nrhs;
  const int cmax = std::max(1, std::min(std::min(128, slots), cdiv(n, 4)));
  const bool f64 = prec == MPSL_FP64;
  const double t_group = (f64 ? 525.0 : 260.0) * P * nt / 2.3e3;                        // us
  const double t_slot = 2.0 * nrhs * n * P * (f64 ? sizeof(double2) : sizeof(float2)) / 4.5e6;  // us
  double best = 1e300;
  int bc = 1;
  for (int c = 1; c <= cmax; ++c) {
    const int groups = m2l_mfma_chunk_len(n, c) / 4;
    if (cdiv(n, 4 * groups) != c) continue;  // trailing chunks empty
    const int rounds = cdiv(static_cast<int64_t>(bpc) * c, units);
    const double t = rounds * groups * t_group * (rounds == 1 ? 1.17 : 1.0) + c * t_slot;
    if (t < best) {
      best = t;
      bc = c;
    }
  }
  return bc;
}

int chunks_m2l(const mpsl_ctx *ctx, int prec, int nrhs) {
  // the right-hand sides already multiply the grid: a count set for one is shared
  const int tuned = ctx->tune[prec == MPSL_FP64 ? 0 : 1].chunks;
  if (tuned > 0) return std::max(1, static_cast<int>(std::min<int64_t>(tuned, ctx->n)) / nrhs);
  if (ctx->m2l_chunks > 0) return std::max(1, static_cast<int>(std::min<int64_t>(ctx->m2l_chunks, ctx->n)) / nrhs);
  const int v = m2l_variant(ctx, prec, nrhs);
  if (v >= kM2LMfma) return m2l_mfma_chunks(ctx, prec, v == kM2LMfmaWide ? 2 : 1, nrhs);
  // one lane per target: about 2560 blocks of 128 lanes
  const int64_t c = std::max<int64_t>(1, std::min<int64_t>(cdiv(2560, cdiv(ctx->n, kThreads)), ctx->n));
  return std::max(1, static_cast<int>(c) / nrhs);
}

// Sources per chunk of the matrix-core M2L: each MFMA step takes a group of
// four sources, so a chunk length that is not a multiple of 4 leaves a part
// of one group's matrix work on zeros in every chunk (39 sources: 2.5 %
// of the launch at 5000 particles); trailing chunks may come out empty and
// then write zero partials.
int m2l_mfma_chunk_len(int n, int chunks) { return (cdiv(n, chunks) + 3) / 4 * 4; }

template <typename T>
static int launch_m2l_t(mpsl_ctx *ctx, const void *beta, void *part, int chunks, int variant, int nrhs,
                        int64_t pstride) {
  const int n = static_cast<int>(ctx->n);
  const int chunk_len = cdiv(n, chunks);
  const bool f64 = std::is_same<T, double>::value;
  const dim3 grid(cdiv(n, kThreads), chunks, nrhs);
  const auto *pairs = static_cast<const cv_t<T> *>(f64 ? ctx->gt.pair64.p : ctx->gt.pair32.p);
  const auto *b = static_cast<const cv_t<T> *>(beta);
  auto *o = static_cast<cv_t<T> *>(part);
  const int64_t bs = ctx->n * static_cast<int64_t>(2 * ctx->p + 1);
  if (variant == kM2LMfma || variant == kM2LMfmaWide) {
    if (ctx->p > kM2LMfmaMaxP) return set_err(ctx, MPSL_EUNSUPPORTED, "matrix-core M2L needs p <= 16");
    const int nt = variant == kM2LMfma ? 1 : 2;
    static_assert(kM2lWaves == kM2lBfWaves, "one grid for both precisions");
    const dim3 g(cdiv(n, 16 * nt * kM2lWaves), chunks, nrhs);
    const dim3 blk(64 * kM2lWaves);
    const int cl = m2l_mfma_chunk_len(n, chunks);
    switch (ctx->p) {
#define X(PP)                                                                                        \
  case PP:                                                                                           \
    if constexpr (PP <= kM2LMfmaMaxP) {                                                              \
      if constexpr (std::is_same<T, float>::value) {                                                 \
        if (nt == 1)                                                                                 \
          hipLaunchKernelGGL((k_m2l_bf<PP, 1>), g, blk, 0, ctx->stream, pairs, b, o, n, cl, bs, pstride); \
        else                                                                                         \
          hipLaunchKernelGGL((k_m2l_bf<PP, 2>), g, blk, 0, ctx->stream, pairs, b, o, n, cl, bs, pstride); \
      } else {                                                                                       \
        if (nt == 1)                                                                                 \
          hipLaunchKernelGGL((k_m2l_f64<PP, 1>), g, blk, 0, ctx->stream, pairs, b, o, n, cl, bs, pstride); \
        else                                                                                         \
          hipLaunchKernelGGL((k_m2l_f64<PP, 2>), g, blk, 0, ctx->stream, pairs, b, o, n, cl, bs, pstride); \
      }                                                                                              \
    }                                                                                                \
    break;
      MPSL_P_CASES(X)
#undef X
      default: return set_err(ctx, MPSL_EUNSUPPORTED, "expansion order outside 1..20");
    }
    LAUNCH_CHECK(ctx);
    return MPSL_OK;
  }
  switch (ctx->p) {
#define X(PP)                                                                                               \
  case PP:                                                                                                  \
    if (variant == kM2LHalves) {                                                                            \
      hipLaunchKernelGGL((k_m2l<T, PP, 0>), grid, dim3(kThreads), 0, ctx->stream, pairs, b, o, n, chunk_len, \
                         bs, pstride);                                                                      \
      hipLaunchKernelGGL((k_m2l<T, PP, 1>), grid, dim3(kThreads), 0, ctx->stream, pairs, b, o, n, chunk_len, \
                         bs, pstride);                                                                      \
    } else {                                                                                                \
      hipLaunchKernelGGL((k_m2l<T, PP, -1>), grid, dim3(kThreads), 0, ctx->stream, pairs, b, o, n,           \
                         chunk_len, bs, pstride);                                                           \
    }                                                                                                       \
    break;
    MPSL_P_CASES(X)
#undef X
    default: return set_err(ctx, MPSL_EUNSUPPORTED, "expansion order outside 1..20");
  }
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

int launch_m2l(mpsl_ctx *ctx, int prec, const void *beta, void *part, int chunks, int variant, int nrhs,
               int64_t pstride) {
  if (variant < 0) variant = m2l_variant(ctx, prec, nrhs);  // tuned or default; matrix cores up to p = 16
  return prec == MPSL_FP64 ? launch_m2l_t<double>(ctx, beta, part, chunks, variant, nrhs, pstride)
                           : launch_m2l_t<float>(ctx, beta, part, chunks, variant, nrhs, pstride);
}

// bf16 parts where one K step holds all orders (p = 8 .. 15; at p = 16 the 33
// orders would pad to 64), else the FP32 form.
static constexpr bool mrhs_bf(int p) { return p >= 8 && p <= 15; }

// Blocks of the many-right-hand-side M2L resident per compute unit (occupancy
// query, cached per order; 1 if the query fails).
static int mrhs_resident(int p) {
  static std::atomic<int> cache[kMaxP + 1];
  if (p < kMinP || p > kMaxP) return 1;
  int r = cache[p].load(std::memory_order_relaxed);
  if (r > 0) return r;
  const void *fn = nullptr;
  switch (p) {
#define X(PP)                                                                     \
  case PP:                                                                        \
    if constexpr (mrhs_bf(PP)) fn = reinterpret_cast<const void *>(&k_m2l_mrhs_bf<PP>); \
    else fn = reinterpret_cast<const void *>(&k_m2l_mrhs<PP>);                    \
    break;
    MPSL_P_CASES(X)
#undef X
  }
  int nb = 0;
  if (!fn || hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, 64 * kMrhsWaves, 0) != hipSuccess || nb < 1) {
    (void)hipGetLastError();
    nb = 1;
  }
  cache[p].store(nb, std::memory_order_relaxed);
  return nb;
}

// The most source chunks: about 1024 blocks' worth, of no less than one batch.
static int mrhs_most(const mpsl_ctx *ctx, int nrhs) {
  const int64_t blocks = static_cast<int64_t>(cdiv(ctx->n, kMrhsWaves)) * cdiv(nrhs, 64);
  return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(cdiv(1024, blocks), cdiv(ctx->n, kMrhsBatch))));
}

// Source chunks: all blocks carry the same work, so of the counts up to mrhs_most
// one whose blocks fill the last round of the resident slots within 3 % of the
// best.  Of these the bf16 form, one block per unit, takes the smallest (2000
// particles, 64 right-hand sides, p = 12, 250 blocks: one chunk), the FP32 form
// the largest: shorter sums, and blocks that the units finish at different
// times (p = 4, two per unit, 16 right-hand sides: four chunks 2.65 ms, two 2.70,
// five, which leave the third round half empty, 2.64; 500 particles: eight
// 0.206, sixteen 0.221).
int chunks_m2l_mrhs(const mpsl_ctx *ctx, int nrhs) {
  const int64_t blocks = static_cast<int64_t>(cdiv(ctx->n, kMrhsWaves)) * cdiv(nrhs, 64);
  const int hi = mrhs_most(ctx, nrhs);
  const int64_t slots = static_cast<int64_t>(std::max(1, ctx->n_cu)) * mrhs_resident(ctx->p);
  auto cost = [&](int c) { return static_cast<double>(cdiv(blocks * c, slots)) / c; };
  double best = 1e300;
  for (int c = 1; c <= hi; ++c) best = std::min(best, cost(c));
  int pick = hi;
  for (int c = hi; c >= 1; --c)
    if (cost(c) <= 1.03 * best) {
      pick = c;
      if (!mrhs_bf(ctx->p)) break;
    }
  return pick;
}

int launch_m2l_mrhs(mpsl_ctx *ctx, const void *beta, void *part, int chunks, int nrhs, int64_t pstride) {
  const int n = static_cast<int>(ctx->n);
  const int P = 2 * ctx->p + 1;
  const int KP = (P + 3) / 4 * 4;
  const int64_t rows = static_cast<int64_t>(n) * KP;
  const int r_pad = 64 * cdiv(nrhs, 64);
  int rc = dev_alloc(ctx, ctx->bt, static_cast<size_t>(rows) * r_pad * sizeof(float2));
  if (rc) return rc;
  switch (ctx->p) {
#define X(PP)                                                                                                \
  case PP:                                                                                                   \
    hipLaunchKernelGGL(k_rhs_transpose<2 * PP + 1>, dim3(n, r_pad / 64), dim3(256), 0, ctx->stream,          \
                       static_cast<const float2 *>(beta), static_cast<float2 *>(ctx->bt.p), n, nrhs, r_pad,  \
                       mrhs_bf(PP));                                                                         \
    break;
    MPSL_P_CASES(X)
#undef X
    default: return set_err(ctx, MPSL_EUNSUPPORTED, "expansion order outside 1..20");
  }
  LAUNCH_CHECK(ctx);
  const int chunk_len = cdiv(n, chunks);
  // as many batches as the shortest chunk has
  const int run = std::max(1, cdiv(n, mrhs_most(ctx, nrhs)) / kMrhsBatch);
  const dim3 grid(cdiv(n, kMrhsWaves), chunks, r_pad / 64);
  const auto *pairs = static_cast<const float2 *>(ctx->gt.pair32.p);
  const auto *bt = static_cast<const float2 *>(ctx->bt.p);
  auto *pp = static_cast<float2 *>(part);
  switch (ctx->p) {
#define X(PP)                                                                                                      \
  case PP:                                                                                                         \
    if constexpr (mrhs_bf(PP))                                                                                     \
      hipLaunchKernelGGL((k_m2l_mrhs_bf<PP>), grid, dim3(64 * kMrhsWaves), 0, ctx->stream, pairs, bt, pp, n,       \
                         chunk_len, nrhs, r_pad, pstride);                                                         \
    else                                                                                                           \
      hipLaunchKernelGGL((k_m2l_mrhs<PP>), grid, dim3(64 * kMrhsWaves), 0, ctx->stream, pairs, bt, pp, n,          \
                         chunk_len, nrhs, r_pad, pstride, run);                                                    \
    break;
    MPSL_P_CASES(X)
#undef X
    default: return set_err(ctx, MPSL_EUNSUPPORTED, "expansion order outside 1..20");
  }
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

template <typename T>
static int launch_fmm_near_t(mpsl_ctx *ctx, const void *beta, void *out) {
  const FmmPlan &f = ctx->fmm;
  const int n = static_cast<int>(ctx->n);
  const bool f64 = std::is_same<T, double>::value;
  const auto *pairs = static_cast<const cv_t<T> *>(f64 ? f.near64.p : f.near32.p);
  const auto *src = static_cast<const int *>(f.near_src.p);
  const auto *perm = static_cast<const int *>(f.perm.p);
  const auto *wave = static_cast<const int *>(f.near_wave.p);
  const auto *b = static_cast<const cv_t<T> *>(beta);
  auto *o = static_cast<cv_t<T> *>(out);
  const int kc = cdiv(f.near_k, f.near_chunks);
  const dim3 grid(cdiv(n, kThreads), f.near_chunks);
  // FP64: two output halves (register pressure); FP32: one launch
  switch (ctx->p) {
#define X(PP)                                                                                                    \
  case PP:                                                                                                       \
    if constexpr (std::is_same<T, double>::value) {                                                              \
      hipLaunchKernelGGL((k_fmm_near<T, PP, 0>), grid, dim3(kThreads), 0, ctx->stream, pairs, src, perm, wave, b, \
                         o, n, kc);                                                                              \
      hipLaunchKernelGGL((k_fmm_near<T, PP, 1>), grid, dim3(kThreads), 0, ctx->stream, pairs, src, perm, wave, b, \
                         o, n, kc);                                                                              \
    } else {                                                                                                     \
      hipLaunchKernelGGL((k_fmm_near<T, PP, -1>), grid, dim3(kThreads), 0, ctx->stream, pairs, src, perm, wave,   \
                         b, o, n, kc);                                                                           \
    }                                                                                                            \
    break;
    MPSL_P_CASES(X)
#undef X
    default: return set_err(ctx, MPSL_EUNSUPPORTED, "expansion order outside 1..20");
  }
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

int launch_fmm_near(mpsl_ctx *ctx, int prec, const void *beta, void *out) {
  return prec == MPSL_FP64 ? launch_fmm_near_t<double>(ctx, beta, out) : launch_fmm_near_t<float>(ctx, beta, out);
}

}  // namespace mpsl
