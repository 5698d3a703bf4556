// Device kernels of the layered-medium multiple-scattering matvec.
//
// Layouts (row-major, complex interleaved):
//   beta, alpha, x, y   [n][P]                 P = 2p + 1, slot n + p
//   part                [chunk][n][P]          partial local expansions
//   E (M2S factors)     [2][n][ns]             side 0: upper interface, 1: lower
//   F (S2L factors)     [2][ns][n]
//   W (M2S order sums)  [2][ns][P]
//   Up (S2L coeffs)     [2][ns][P]
//   spec, sigma         [2][ns]                FP64
#include <atomic>
#include <cmath>

#include "kernels.h"

namespace mpsl {

namespace {

constexpr int kThreads = 128;

inline int cdiv(int64_t a, int64_t b) { return static_cast<int>((a + b - 1) / b); }

// complex exp(a + i b) in FP64
__device__ inline cx<double> cexp_d(double a, double b) {
  double s, c;
  sincos(b, &s, &c);
  const double e = exp(a);
  return {e * c, e * s};
}

// ---------------------------------------------------------------------------
// Row a0: plane-wave factors of every (particle, node) pair.
//   E+[m][q] = e^{-i lam x_m + g2 y_m}          E-[m][q] = e^{-i lam x_m - g2 (d + y_m)}
//   F+[q][l] = e^{ i lam x_l + g2 y_l}          F-[q][l] = e^{ i lam x_l - g2 (y_l + d)}
__global__ void k_geom_tables(const double2 *__restrict__ xy, const double2 *__restrict__ lam,
                              const double2 *__restrict__ g2, int n, int ns, double d,
                              double2 *__restrict__ E, double2 *__restrict__ F,
                              float2 *__restrict__ E32, float2 *__restrict__ F32) {
  const int64_t idx = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  const int64_t tot = static_cast<int64_t>(n) * ns;
  if (idx >= tot) return;
  const int m = static_cast<int>(idx / ns);
  const int q = static_cast<int>(idx % ns);
  const double x = xy[m].x, y = xy[m].y;
  const double lr = lam[q].x, li = lam[q].y, gr = g2[q].x, gi = g2[q].y;
  const cx<double> ep = cexp_d(li * x + gr * y, -lr * x + gi * y);
  const cx<double> em = cexp_d(li * x - gr * (d + y), -lr * x - gi * (d + y));
  const cx<double> fp = cexp_d(-li * x + gr * y, lr * x + gi * y);
  const cx<double> fm = cexp_d(-li * x - gr * (y + d), lr * x - gi * (y + d));
  const int64_t e0 = static_cast<int64_t>(m) * ns + q;
  const int64_t f0 = static_cast<int64_t>(q) * n + m;
  E[e0] = st(ep);
  E[tot + e0] = st(em);
  F[f0] = st(fp);
  F[tot + f0] = st(fm);
  E32[e0] = make_float2(static_cast<float>(ep.re), static_cast<float>(ep.im));
  E32[tot + e0] = make_float2(static_cast<float>(em.re), static_cast<float>(em.im));
  F32[f0] = make_float2(static_cast<float>(fp.re), static_cast<float>(fp.im));
  F32[tot + f0] = make_float2(static_cast<float>(fm.re), static_cast<float>(fm.im));
}

// ---------------------------------------------------------------------------
// Row a0 (pairs): per ordered pair (m -> l) the Hankel functions H_0, H_1 of
// z = k2 |x_l - x_m|, the direction e^{i phi} = (x_l - x_m)/|x_l - x_m| and
// 2/z, computed once per geometry in FP64 and stored source-major
// [m][l][4] = {H_0, H_1, e^{i phi}, (2/z, 0)} in FP64 and FP32.  The self
// pair l == m holds zeros.
__global__ void k_pair_tables(const double2 *__restrict__ xy, int n, double k2, double2 *__restrict__ t64,
                              float2 *__restrict__ t32) {
  const int64_t idx = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (idx >= static_cast<int64_t>(n) * n) return;
  const int m = static_cast<int>(idx / n);
  const int l = static_cast<int>(idx % n);
  double2 e[4] = {make_double2(0.0, 0.0), make_double2(0.0, 0.0), make_double2(0.0, 0.0),
                  make_double2(0.0, 0.0)};
  if (l != m) {
    const double dx = xy[l].x - xy[m].x, dy = xy[l].y - xy[m].y;
    const double rho = sqrt(dx * dx + dy * dy);
    const double z = k2 * rho;
    e[0] = make_double2(j0(z), y0(z));
    e[1] = make_double2(j1(z), y1(z));
    e[2] = make_double2(dx / rho, dy / rho);
    e[3] = make_double2(2.0 / z, 0.0);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    t64[4 * idx + k] = e[k];
    t32[4 * idx + k] = make_float2(static_cast<float>(e[k].x), static_cast<float>(e[k].y));
  }
}

// M2S partials to spectra, and for the matvec on to the S2L coefficients: per
// block 16 nodes, both sides, eight lanes per (node, side) taking every eighth
// particle chunk (FP64 sums, added in order).  With spec the sums are stored
// there; without, the block applies the reflection map (row b2) and writes
// Up[s][q][n] = c_q sigma_s U[s][q][n] in the matvec's precision: one launch
// for what were three, each a few microseconds of latency (5000 particles,
// 1024 nodes, FP32: 15.4 + 4.6 + 4.7 us; 20000: 28.3 us for the sums alone,
// whose lanes walked up to 109 chunks in series).
constexpr int kNodeBlock = 16, kNodeLanes = 8;
// c_q sigma_s(q) from the spectra of both sides of node q (reflection map).
__device__ inline cx<double> node_density(const double2 *__restrict__ R, const double2 *__restrict__ cq, int q, int s,
                                          cx<double> pp, cx<double> pm) {
  return ld<double>(cq[q]) * (ld<double>(R[4 * q + 2 * s]) * pp + ld<double>(R[4 * q + 2 * s + 1]) * pm);
}

template <typename T>
__global__ __launch_bounds__(2 * kNodeBlock *kNodeLanes) void k_nodes(
    const cv_t<T> *__restrict__ part, int ns, int chunks, const double2 *__restrict__ R,
    const double2 *__restrict__ cq, const double2 *__restrict__ U, int P, double2 *__restrict__ spec,
    cv_t<T> *__restrict__ Up) {
  __shared__ double2 sum[kNodeLanes][2][kNodeBlock];
  __shared__ double2 val[2][kNodeBlock];
  const int tid = threadIdx.x, qi = tid % kNodeBlock, s = tid / kNodeBlock & 1, cl = tid / (2 * kNodeBlock);
  const int64_t r = blockIdx.y;
  const int q0 = blockIdx.x * kNodeBlock, q = q0 + qi;
  double re = 0.0, im = 0.0;
  if (q < ns) {
    const cv_t<T> *p = part + (2 * r + s) * chunks * static_cast<int64_t>(ns) + q;
#pragma unroll 4
    for (int c = cl; c < chunks; c += kNodeLanes) {
      const cv_t<T> v = p[static_cast<int64_t>(c) * ns];
      re += static_cast<double>(v.x);
      im += static_cast<double>(v.y);
    }
  }
  sum[cl][s][qi] = make_double2(re, im);
  __syncthreads();
  if (cl == 0) {
    cx<double> v = mk(0.0, 0.0);
#pragma unroll
    for (int c = 0; c < kNodeLanes; ++c) v = v + ld<double>(sum[c][s][qi]);
    if (spec) {
      if (q < ns) spec[(2 * r + s) * ns + q] = st(v);
    } else {
      sum[0][s][qi] = st(v);
    }
  }
  if (spec) return;  // uniform over the grid
  __syncthreads();
  if (cl == 0) {
    const int qc = min(q, ns - 1);
    val[s][qi] = st(node_density(R, cq, qc, s, ld<double>(sum[0][0][qi]), ld<double>(sum[0][1][qi])));
  }
  __syncthreads();
  const int cnt = min(kNodeBlock, ns - q0) * P;
  for (int i = tid; i < 2 * cnt; i += 2 * kNodeBlock * kNodeLanes) {
    const int side = i >= cnt ? 1 : 0, e = i - side * cnt;
    const int64_t base = static_cast<int64_t>(side) * ns * P + static_cast<int64_t>(q0) * P + e;
    const cx<double> v = ld<double>(val[side][e / P]) * ld<double>(U[base]);
    Up[2 * r * ns * P + base] = st(mk(static_cast<T>(v.re), static_cast<T>(v.im)));
  }
}

// ---------------------------------------------------------------------------
// Row b2: middle-layer densities per node from the particle spectra and the
// point source:  [s+; s-] = R [P+; P-] + g [f+; f-],  g = e^{-i lam x_s - g1 y_s}.
__global__ void k_reflect(const double2 *__restrict__ spec, const double2 *__restrict__ R,
                          const double2 *__restrict__ sf, const double2 *__restrict__ lam,
                          const double2 *__restrict__ g1, int ns, int has_src, double xs, double ys,
                          double2 *__restrict__ sigma) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= ns) return;
  sigma += 2 * static_cast<int64_t>(ns) * blockIdx.y;  // right-hand side
  if (spec) spec += 2 * static_cast<int64_t>(ns) * blockIdx.y;
  cx<double> pp = mk(0.0, 0.0), pm = mk(0.0, 0.0);
  if (spec) {
    pp = ld<double>(spec[q]);
    pm = ld<double>(spec[ns + q]);
  }
  cx<double> sp = ld<double>(R[4 * q + 0]) * pp + ld<double>(R[4 * q + 1]) * pm;
  cx<double> sm = ld<double>(R[4 * q + 2]) * pp + ld<double>(R[4 * q + 3]) * pm;
  if (has_src) {
    const double lr = lam[q].x, li = lam[q].y, gr = g1[q].x, gi = g1[q].y;
    const cx<double> g = cexp_d(li * xs - gr * ys, -lr * xs - gi * ys);
    sp = sp + ld<double>(sf[2 * q + 0]) * g;
    sm = sm + ld<double>(sf[2 * q + 1]) * g;
  }
  sigma[q] = st(sp);
  sigma[ns + q] = st(sm);
}

// S2L coefficient tables: Up[s][q][n] = c_q sigma_s[q] U[s][q][n].
__global__ void k_s2l_coef(const double2 *__restrict__ sigma, const double2 *__restrict__ cq,
                           const double2 *__restrict__ U, int ns, int P, int nrhs, double2 *__restrict__ Up64,
                           float2 *__restrict__ Up32) {
  const int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  const int64_t per = 2LL * ns * P;
  if (i >= per * nrhs) return;
  const int64_t r = i / per, k = i % per;
  const int s = static_cast<int>(k / (static_cast<int64_t>(ns) * P));
  const int q = static_cast<int>((k / P) % ns);
  const cx<double> v = ld<double>(cq[q]) * ld<double>(sigma[(2 * r + s) * ns + q]) * ld<double>(U[k]);
  Up64[i] = st(v);
  Up32[i] = make_float2(static_cast<float>(v.re), static_cast<float>(v.im));
}


// ---------------------------------------------------------------------------
// Sum of the partial slots of one entry by four neighbouring lanes: lane g
// takes the slots g, g + 4, ..., eight loads in flight, and the four sums are
// added by two exchanges (a fixed order; every lane of the four gets the sum).
// One lane per entry left small problems waiting for their loads in series
// (1000 particles, p = 12, FP64: 25000 lanes, 384 slots, 35 us).  FP32 slots
// are added in pairs and the pairs in FP64: 8 % off the error of FP32 matvecs of 50
// to 3000 particles on average; every slot converted cost the matvec of 100
// particles 1.2 us, pairs nothing that shows.
constexpr int kSumLanes = 4;
template <typename T>
__device__ __forceinline__ cx<T> sum_slots(const cv_t<T> *part, int slots, int64_t len, int g) {
  double re[2] = {0, 0}, im[2] = {0, 0};
  auto add = [&](const cv_t<T> *v) {
#pragma unroll
    for (int u = 0; u < 8; u += 2) {
      re[u / 2 & 1] += v[u].x + v[u + 1].x;
      im[u / 2 & 1] += v[u].y + v[u + 1].y;
    }
  };
  int c = g;
  for (; c + 7 * kSumLanes < slots; c += 8 * kSumLanes) {
    cv_t<T> v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[(c + u * kSumLanes) * len];
    add(v);
  }
  cv_t<T> v[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) v[u] = c + u * kSumLanes < slots ? part[(c + u * kSumLanes) * len] : st(mk<T>(0, 0));
  add(v);
  cx<double> s = mk(re[0] + re[1], im[0] + im[1]);
#pragma unroll
  for (int o = 1; o < kSumLanes; o <<= 1) {
    s.re += __shfl_xor(s.re, o);
    s.im += __shfl_xor(s.im, o);
  }
  return mk<T>(static_cast<T>(s.re), static_cast<T>(s.im));
}

// out[i] = sum_c part[c len + i] (out may be the first slot), for right-hand side
// blockIdx.y with both buffers `stride` entries further on
template <typename T>
__global__ __launch_bounds__(256) void k_sum_parts(const cv_t<T> *part, int slots, int64_t len,
                                                   cv_t<T> *out, int64_t stride) {
  part += blockIdx.y * stride;
  out += blockIdx.y * stride;
  const int64_t t = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  const int64_t i = t / kSumLanes;
  if (i >= len) return;
  const int g = static_cast<int>(t % kSumLanes);
  const cx<T> s = sum_slots<T>(part + i, slots, len, g);
  if (g == 0) out[i] = st(s);
}

// Row a2 on the matrix cores: y^l = x^l - e^{-in psi_l} sum_n' S[n][n'] e^{in' psi_l} alpha^l_{n'},
// alpha the sum of `slots` partial buffers per right-hand side.  One block
// per tile of 16 particles: all lanes sum the partials of the tile's
// expansions (a contiguous range of 16 P entries; HBM-bound where the slots
// are many) and rotate them into LDS as B[K = n'][N = particle]; wave w < MT
// then multiplies row tile w of the shared S (A[M = n][K = n'], zero-padded to
// 16 MT x KP) by B with 16x16x4 MFMA, the complex product as four real
// chains (re += Sr Br - Si Bi, im += Sr Bi + Si Br); the result goes back
// through LDS for coalesced stores.  With more than kSapplyFew slots four lanes
// sum an entry, in blocks of 512; else one, in blocks of 256 (the strides are
// constants: read from the launch, they cost the step by itself 0.1 to 0.3 us).
//   (MFMA operand layout: mfma4 in common.h.)
constexpr int kSapplyFew = 8;

template <typename T, int p, int nthr>
__global__ __launch_bounds__(nthr) void k_sapply(const cv_t<T> *__restrict__ x,
                                                           const cv_t<T> *__restrict__ alpha, int slots,
                                                           const cv_t<T> *__restrict__ S,
                                                           const cv_t<T> *__restrict__ rot, int n,
                                                           cv_t<T> *__restrict__ y, int64_t astride,
                                                           const int32_t *__restrict__ types, int ntypes) {
  constexpr int P = 2 * p + 1;
  constexpr int MT = (P + 15) / 16;   // row tiles of S
  constexpr int KP = (P + 3) / 4 * 4; // K padded to the MFMA depth
  static_assert(MT <= 4, "one wave per row tile");
  {  // right-hand side
    const int64_t off = static_cast<int64_t>(blockIdx.y) * n * P;
    if (x) x += off;
    y += off;
    alpha += blockIdx.y * astride;
  }
  __shared__ T Sre[MT * 16][KP], Sim[MT * 16][KP];
  __shared__ T Bre[KP][16], Bim[KP][16];
  __shared__ cx<T> Yt[16 * P];
  __shared__ int32_t tt[16];  // particle types of the tile (-1 past the end)
  const int tid = threadIdx.x;
  const int l0 = blockIdx.x * 16;
  for (int i = tid; i < KP * 16; i += nthr) {
    Bre[i / 16][i % 16] = 0;
    Bim[i / 16][i % 16] = 0;
  }
  if (tid < 16) tt[tid] = (l0 + tid < n) ? (types ? types[l0 + tid] : 0) : -1;
  __syncthreads();
  const int cnt = min(16, n - l0) * P;  // entries of the tile
  const int64_t base = static_cast<int64_t>(l0) * P;
  const int64_t len = static_cast<int64_t>(n) * P;
  if constexpr (nthr == 256) {  // few slots: one lane per entry, summed in FP64
    for (int i = tid; i < cnt; i += nthr) {
      cx<double> z = mk<double>(alpha[base + i].x, alpha[base + i].y);
#pragma unroll 4
      for (int c = 1; c < slots; ++c) {
        const cv_t<T> v = alpha[c * len + base + i];
        z.re += v.x;
        z.im += v.y;
      }
      const cx<T> s = mk<T>(static_cast<T>(z.re), static_cast<T>(z.im)) * ld<T>(rot[base + i]);
      Bre[i % P][i / P] = s.re;
      Bim[i % P][i / P] = s.im;
    }
  } else {
    for (int t = tid; t < cnt * kSumLanes; t += nthr) {
      const int i = t / kSumLanes, g = t % kSumLanes;
      const cx<T> s = sum_slots<T>(alpha + base + i, slots, len, g) * ld<T>(rot[base + i]);
      if (g == 0) {
        Bre[i % P][i / P] = s.re;
        Bim[i % P][i / P] = s.im;
      }
    }
  }
  const int w = tid >> 6, lane = tid & 63;
  const int row = w * 16 + (lane & 15);
  const int col = lane & 15;
  typename mfma4<T>::v4 are = {0, 0, 0, 0}, aim = {0, 0, 0, 0};
  // several particle types: one pass per type present in the tile, with the
  // other columns of B masked out, so each column meets its own matrix
  const int nt = types ? ntypes : 1;
  for (int t = 0; t < nt; ++t) {
    if (types) {
      bool present = false;
      for (int c = 0; c < 16; ++c) present |= (tt[c] == t);
      if (!present) continue;  // uniform over the block
    }
    __syncthreads();  // B written (first pass) or the previous S consumed
    const cv_t<T> *St = S + static_cast<int64_t>(t) * P * P;
    for (int i = tid; i < MT * 16 * KP; i += nthr) {
      const int r = i / KP, c = i % KP;
      const cx<T> v = (r < P && c < P) ? ld<T>(St[r * P + c]) : mk<T>(0, 0);
      Sre[r][c] = v.re;
      Sim[r][c] = v.im;
    }
    __syncthreads();
    if (w < MT) {
      const bool on = !types || tt[col] == t;
#pragma unroll
      for (int k0 = 0; k0 < KP; k0 += 4) {
        const int k = k0 + (lane >> 4);
        const T sr = Sre[row][k], si = Sim[row][k];
        const T br = on ? Bre[k][col] : T(0), bi = on ? Bim[k][col] : T(0);
        are = mfma4<T>::mac(sr, br, are);
        are = mfma4<T>::mac(-si, bi, are);
        aim = mfma4<T>::mac(sr, bi, aim);
        aim = mfma4<T>::mac(si, br, aim);
      }
    }
  }
  if (w < MT) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int nn = w * 16 + mfma4<T>::row(lane, j);
      if (nn < P) Yt[col * P + nn] = mk<T>(are[j], aim[j]);
    }
  }
  __syncthreads();
  for (int i = tid; i < cnt; i += nthr) {
    cx<T> r = conj(ld<T>(rot[base + i])) * Yt[i];
    if (x) r = ld<T>(x[base + i]) - r;
    y[base + i] = st(r);
  }
}

// ---------------------------------------------------------------------------
// Row b1 on the matrix cores: M2S as a GEMM over the particles of a chunk,
//   G[q][nu] = sum_{m in chunk c} E[s][m][q] beta[m][nu]   (M = node, N = order,
// K = particle), then part[r][s][c][q] = sum_nu W[s][q][nu] G[q][nu] in the
// epilogue (a reduction over the 16 lanes that hold one node's orders).  One
// wave per 16 nodes; lane i supplies A[i % 16][i / 16] = E of node q0 + i % 16
// for particle m0 + i / 16 (16 consecutive nodes: coalesced) and
// B[i / 16][i % 16] = beta of that particle and order.  Complex products take
// three real MFMAs (Gauss: P1 = sum Ar Br, P2 = sum Ai Bi, P3 = sum (Ar + Ai)
// (Br + Bi); re = P1 - P2, im = P3 - P1 - P2).
constexpr int kM2sWaves = 4;
// Steps of the M2S and S2L products whose operands are in flight.  In FP64 they
// read an entry of 16 bytes per particle, node and side from HBM, and one step
// ahead left the matrix cores waiting (1000 particles, 25216 nodes, p = 12: M2S
// 336 us, S2L 349 us, 2.3 TB/s; two steps 274 and 298, four 265 and 281).  In
// FP32 one step ahead is enough, and loading past the end of a chunk costs
// more than it gives (20000 particles, 1024 nodes, p = 16: S2L 123 us with one
// step, fetched only where there is one, 143 with two).
template <typename T> constexpr int gemm_depth() { return sizeof(T) == 8 ? 4 : 1; }
// NODES: the matvec with one chunk (few particles) takes both sides of a node
// group in one block and goes on to the S2L coefficients, which saves the
// launch of k_nodes (16 particles, p = 8, FP64, matvec: 23.6 -> 21.7 us).
template <typename T, int p, bool NODES>
__global__ __launch_bounds__(64 * kM2sWaves) void k_m2s_mfma(
    const cv_t<T> *__restrict__ E, const cv_t<T> *__restrict__ beta, const cv_t<T> *__restrict__ W,
    cv_t<T> *__restrict__ part, int n, int ns, int chunk_len, int chunks, const double2 *__restrict__ R,
    const double2 *__restrict__ cq, const double2 *__restrict__ U, cv_t<T> *__restrict__ Up) {
  constexpr int kGroups = kM2sWaves / 2;  // node groups of a NODES block
  __shared__ double2 nsum[NODES ? kGroups : 1][2][16], nval[NODES ? kGroups : 1][2][16];
  constexpr int P = 2 * p + 1;
  constexpr int NT = OrderSplit<P>::NT, NV = OrderSplit<P>::NV;
  typedef typename mfma4<T>::v4 v4;
  const int c = blockIdx.y;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int s = NODES ? w & 1 : blockIdx.z & 1;           // side
  const int r = NODES ? blockIdx.z : blockIdx.z >> 1;     // right-hand side
  beta += static_cast<int64_t>(r) * n * P;
  const int q0 = (NODES ? blockIdx.x * kGroups + (w >> 1) : blockIdx.x * kM2sWaves + w) * 16;
  if (!NODES && q0 >= ns) return;  // the whole wave lies past the last node (no barriers below)
  const int m0 = c * chunk_len;
  const int m1 = min(n, m0 + chunk_len);
  const int qi = q0 + (lane & 15);
  const int qic = min(qi, ns - 1);
  const int kr = lane >> 4;
  const cv_t<T> *Es = E + static_cast<int64_t>(s) * n * ns;
  v4 P1[NT], P2[NT], P3[NT];
  cx<T> vr[NV > 0 ? NV : 1];
#pragma unroll
  for (int t = 0; t < NT; ++t) P1[t] = P2[t] = P3[t] = v4{0, 0, 0, 0};
#pragma unroll
  for (int v = 0; v < (NV > 0 ? NV : 1); ++v) vr[v] = mk<T>(0, 0);
  if (m0 < m1) {
    // operands of particle group mb (loads clamped into range, zeros selected
    // past the chunk), those of the next gemm_depth groups in flight while the
    // current one multiplies
    struct Ops {
      cv_t<T> a, b[NT], bv[NV > 0 ? NV : 1];
    };
    auto fetch = [&](int mb, Ops &o) {
      const int mc = min(mb + kr, m1 - 1);
      o.a = Es[static_cast<int64_t>(mc) * ns + qic];
#pragma unroll
      for (int t = 0; t < NT; ++t) o.b[t] = beta[static_cast<int64_t>(mc) * P + min(t * 16 + (lane & 15), P - 1)];
#pragma unroll
      for (int v = 0; v < NV; ++v) o.bv[v] = beta[static_cast<int64_t>(mc) * P + 16 * NT + v];
    };
    constexpr int U = gemm_depth<T>();
    Ops nx[U];
#pragma unroll
    for (int u = 0; u < U; ++u) fetch(m0 + 4 * u, nx[u]);
    for (int mb = m0; mb < m1; mb += 4 * U) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const Ops cu = nx[u];
        if (U > 1 || mb + 4 < m1) fetch(mb + 4 * (U + u), nx[u]);
        const bool mv = mb + 4 * u + kr < m1;
        const T zr = mv ? cu.a.x : T(0), zi = mv ? cu.a.y : T(0), zs = zr + zi;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const bool cv = t * 16 + (lane & 15) < P;  // padded tile (long remainders only)
          const T br = cv ? cu.b[t].x : T(0), bi = cv ? cu.b[t].y : T(0);
          P1[t] = mfma4<T>::mac(zr, br, P1[t]);
          P2[t] = mfma4<T>::mac(zi, bi, P2[t]);
          P3[t] = mfma4<T>::mac(zs, br + bi, P3[t]);
        }
#pragma unroll
        for (int v = 0; v < NV; ++v) cmac(vr[v], mk<T>(zr, zi), ld<T>(cu.bv[v]));
      }
    }
  }
  // vector-unit orders: sum over the four particles of each node (lane
  // groups); lane i then holds node q0 + i % 16
#pragma unroll
  for (int v = 0; v < NV; ++v) {
    vr[v].re += __shfl_xor(vr[v].re, 16);
    vr[v].im += __shfl_xor(vr[v].im, 16);
    vr[v].re += __shfl_xor(vr[v].re, 32);
    vr[v].im += __shfl_xor(vr[v].im, 32);
  }
  // epilogue: contract each node's orders with W, reduce over the 16 lanes
  // holding that node's columns, one lane per node stores
  const cv_t<T> *Ws = W + static_cast<int64_t>(s) * ns * P;
  cv_t<T> *o = part + ((2 * static_cast<int64_t>(r) + s) * chunks + c) * ns;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int row = mfma4<T>::row(lane, j);
    const int q = q0 + row;
    const int qc = min(q, ns - 1);
    cx<T> acc = mk<T>(0, 0);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int col = t * 16 + (lane & 15);
      const T p1 = P1[t][j], p2 = P2[t][j], p3 = P3[t][j];
      if (col < P) cmac(acc, mk<T>(p1 - p2, p3 - p1 - p2), ld<T>(Ws[static_cast<int64_t>(qc) * P + col]));
    }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) {
      acc.re += __shfl_xor(acc.re, off, 16);
      acc.im += __shfl_xor(acc.im, off, 16);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {  // node q's remainder orders live in lane `row`
      const cx<T> g = mk<T>(__shfl(vr[v].re, row), __shfl(vr[v].im, row));
      cmac(acc, g, ld<T>(Ws[static_cast<int64_t>(qc) * P + 16 * NT + v]));
    }
    if constexpr (NODES) {
      if ((lane & 15) == 0) nsum[w >> 1][s][row] = make_double2(acc.re, acc.im);
    } else {
      if ((lane & 15) == 0 && q < ns) o[q] = st(acc);
    }
  }
  if constexpr (NODES) {
    const int tid = threadIdx.x, b0 = blockIdx.x * kGroups * 16;
    __syncthreads();
    if (tid < 32 * kGroups) {
      const int g = tid / 32, sd = tid / 16 % 2, qi = tid % 16;
      nval[g][sd][qi] = st(node_density(R, cq, min(b0 + 16 * g + qi, ns - 1), sd, ld<double>(nsum[g][0][qi]),
                                        ld<double>(nsum[g][1][qi])));
    }
    __syncthreads();
    const int cnt = min(16 * kGroups, ns - b0) * P;
    for (int i = tid; i < 2 * cnt; i += 64 * kM2sWaves) {
      const int sd = i >= cnt ? 1 : 0, e = i - sd * cnt, node = e / P;
      const int64_t base = static_cast<int64_t>(sd) * ns * P + static_cast<int64_t>(b0) * P + e;
      const cx<double> v = ld<double>(nval[node / 16][sd][node % 16]) * ld<double>(U[base]);
      Up[2 * static_cast<int64_t>(r) * ns * P + base] = st(mk(static_cast<T>(v.re), static_cast<T>(v.im)));
    }
  }
}

// ---------------------------------------------------------------------------
// Row b3 on the matrix cores: S2L as a GEMM over the nodes of both interfaces,
//   part[c][l][n] = sum_{side, q in chunk c} F[side][q][l] Up[side][q][n]
// (M = particle, N = order, K = node).  One wave per 16 MT particles (MT
// tiles of 16) and all order tiles; lane i supplies A[i % 16][i / 16] = F of
// particle l0 + 16 t + i % 16 at node q0 + i / 16 (16 consecutive particles
// per node: coalesced) and B[i / 16][i % 16] = the S2L coefficient of that
// node and order, loaded once for the MT particle tiles; complex products
// take three real MFMAs (Gauss), and a remainder of one or two orders runs on
// the vector units (OrderSplit).
constexpr int kS2lWaves = 4;
// particle tiles per wave: two in FP32 (the coefficient loads shared by
// both); one in FP64, where a second tile's accumulators would leave one
// wave per SIMD
template <typename T> constexpr int s2l_tiles() { return sizeof(T) == 4 ? 2 : 1; }
template <typename T, int p, int MT>
__global__ __launch_bounds__(64 * kS2lWaves) void k_s2l_mfma(const cv_t<T> *__restrict__ F,
                                                             const cv_t<T> *__restrict__ Up,
                                                             cv_t<T> *__restrict__ part, int n, int ns,
                                                             int chunk_len, int64_t pstride) {
  constexpr int P = 2 * p + 1;
  constexpr int NT = OrderSplit<P>::NT, NV = OrderSplit<P>::NV;
  typedef typename mfma4<T>::v4 v4;
  Up += 2 * static_cast<int64_t>(ns) * P * blockIdx.z;  // right-hand side
  part += blockIdx.z * pstride;
  const int c = blockIdx.y;
  const int q0 = c * chunk_len;
  const int q1 = min(ns, q0 + chunk_len);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int l0 = (blockIdx.x * kS2lWaves + w) * 16 * MT;
  if (l0 >= n) return;  // the whole wave lies past the last particle (no barriers below)
  const int kr = lane >> 4;
  int li[MT];
  bool lv[MT];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    li[m] = l0 + 16 * m + (lane & 15);
    lv[m] = li[m] < n;
  }
  v4 P1[MT][NT], P2[MT][NT], P3[MT][NT];
  cx<T> vr[MT][NV > 0 ? NV : 1];
#pragma unroll
  for (int m = 0; m < MT; ++m) {
#pragma unroll
    for (int t = 0; t < NT; ++t) P1[m][t] = P2[m][t] = P3[m][t] = v4{0, 0, 0, 0};
#pragma unroll
    for (int v = 0; v < (NV > 0 ? NV : 1); ++v) vr[m][v] = mk<T>(0, 0);
  }
  if (q0 < q1) {
    // operands of node group qb (loads clamped into range, zeros selected
    // outside it), those of the next gemm_depth groups in flight while the
    // current one multiplies
    struct Ops {
      cv_t<T> a[MT], b[NT], bv[NV > 0 ? NV : 1];
    };
    auto fetch = [&](int side, int qb, Ops &o) {
      const int q = qb + kr;
      const int qc = min(q, q1 - 1);
      const cv_t<T> *f = F + (side * static_cast<int64_t>(ns) + qc) * n;
#pragma unroll
      for (int m = 0; m < MT; ++m) o.a[m] = f[lv[m] ? li[m] : n - 1];
      const cv_t<T> *u = Up + (side * static_cast<int64_t>(ns) + qc) * P;
#pragma unroll
      for (int t = 0; t < NT; ++t) o.b[t] = u[min(t * 16 + (lane & 15), P - 1)];
#pragma unroll
      for (int v = 0; v < NV; ++v) o.bv[v] = u[16 * NT + v];
    };
    constexpr int U = gemm_depth<T>();
    const int half = (q1 - q0 + 3) / 4;  // steps per side
    Ops nx[U];
    auto fetch_step = [&](int i, Ops &o) {
      const int side = i >= half ? 1 : 0;
      fetch(side, q0 + 4 * (i - side * half), o);
    };
#pragma unroll
    for (int u = 0; u < U; ++u) fetch_step(u, nx[u]);
    for (int i = 0; i < 2 * half; i += U) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const Ops cu = nx[u];
        if (U > 1 || i + 1 < 2 * half) fetch_step(i + u + U, nx[u]);
        const int x = i + u >= half ? i + u - half : i + u;
        const bool qv = i + u < 2 * half && q0 + 4 * x + kr < q1;
        T br[NT], bi[NT], bs[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const bool cv = qv && (t * 16 + (lane & 15)) < P;
          br[t] = cv ? cu.b[t].x : T(0);
          bi[t] = cv ? cu.b[t].y : T(0);
          bs[t] = br[t] + bi[t];
        }
#pragma unroll
        for (int m = 0; m < MT; ++m) {
          const T zr = (qv && lv[m]) ? cu.a[m].x : T(0), zi = (qv && lv[m]) ? cu.a[m].y : T(0), zs = zr + zi;
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            P1[m][t] = mfma4<T>::mac(zr, br[t], P1[m][t]);
            P2[m][t] = mfma4<T>::mac(zi, bi[t], P2[m][t]);
            P3[m][t] = mfma4<T>::mac(zs, bs[t], P3[m][t]);
          }
#pragma unroll
          for (int v = 0; v < NV; ++v) cmac(vr[m][v], mk<T>(zr, zi), ld<T>(cu.bv[v]));
        }
      }
    }
  }
  cv_t<T> *o = part + static_cast<int64_t>(c) * n * P;
#pragma unroll
  for (int m = 0; m < MT; ++m) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int col = t * 16 + (lane & 15);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int l = l0 + 16 * m + mfma4<T>::row(lane, j);
        const T p1 = P1[m][t][j], p2 = P2[m][t][j], p3 = P3[m][t][j];
        if (l < n && col < P) o[static_cast<int64_t>(l) * P + col] = st(mk<T>(p1 - p2, p3 - p1 - p2));
      }
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {  // sum over the four node lanes of each particle
      cx<T> z = vr[m][v];
      z.re += __shfl_xor(z.re, 16);
      z.im += __shfl_xor(z.im, 16);
      z.re += __shfl_xor(z.re, 32);
      z.im += __shfl_xor(z.im, 32);
      if (lane < 16 && lv[m]) o[static_cast<int64_t>(li[m]) * P + 16 * NT + v] = st(z);
    }
  }
}

// ---------------------------------------------------------------------------
// GMRES helpers, FP64 complex.
constexpr int kDotBlocks = 64;
constexpr int kRed = 256;

// V holds the basis in FP64 (double2) or, for the mixed-precision solve, FP32
// (float2); products and sums are FP64 either way.  Each block takes one
// slice of w and kDotVecs basis vectors, so every w element is loaded once
// for kDotVecs products (w would otherwise be re-read from L2 once per
// vector: at a basis of several hundred vectors that traffic exceeded V's).
// Sums: per thread, then across the wave by xor shuffles, then the four
// waves in order (deterministic).
constexpr int kDotVecs = 8;
template <typename TV>
__global__ __launch_bounds__(kRed) void k_dotc_part(const TV *__restrict__ V, int64_t ld_v, int k,
                                                    const double2 *__restrict__ w, int64_t len,
                                                    double2 *__restrict__ part, const int32_t *__restrict__ skip) {
  if (skip && *skip) return;  // the pass is not needed (k_dotc_final writes zeros)
  const int j0 = blockIdx.y * kDotVecs;
  const int nv = min(kDotVecs, k - j0);
  const int b = blockIdx.x;
  double re[kDotVecs], im[kDotVecs];
#pragma unroll
  for (int u = 0; u < kDotVecs; ++u) re[u] = im[u] = 0.0;
  for (int64_t i = b * static_cast<int64_t>(kRed) + threadIdx.x; i < len;
       i += static_cast<int64_t>(kRed) * gridDim.x) {
    const double2 c = w[i];
#pragma unroll
    for (int u = 0; u < kDotVecs; ++u) {
      if (u < nv) {
        const TV a = V[(j0 + u) * ld_v + i];
        const double ax = a.x, ay = a.y;
        re[u] += ax * c.x + ay * c.y;
        im[u] += ax * c.y - ay * c.x;
      }
    }
  }
  __shared__ double sr[kRed / 64][kDotVecs], si[kRed / 64][kDotVecs];
  const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int u = 0; u < kDotVecs; ++u) {
    double r = re[u], m = im[u];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      r += __shfl_xor(r, o);
      m += __shfl_xor(m, o);
    }
    if (lane == 0) {
      sr[wv][u] = r;
      si[wv][u] = m;
    }
  }
  __syncthreads();
  if (threadIdx.x < nv) {
    const int u = threadIdx.x;
    double r = 0.0, m = 0.0;
#pragma unroll
    for (int v = 0; v < kRed / 64; ++v) {
      r += sr[v][u];
      m += si[v][u];
    }
    part[(j0 + u) * gridDim.x + b] = make_double2(r, m);
  }
}

// Sums of the partials, one wave per value (one lane per value took its 64
// loads one after another: 5.9 us).
__global__ __launch_bounds__(256) void k_dotc_final(const double2 *__restrict__ part, int k, int nb,
                                                    double2 *__restrict__ h, const int32_t *__restrict__ skip) {
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (j >= k) return;
  const bool off = skip && *skip;
  double re = 0.0, im = 0.0;
  if (!off)
    for (int b = lane; b < nb; b += 64) {
      const double2 v = part[j * nb + b];
      re += v.x;
      im += v.y;
    }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    re += __shfl_xor(re, o);
    im += __shfl_xor(im, o);
  }
  if (lane == 0) h[j] = make_double2(re, im);
}

// w -= V h; with sq also the block's share of ||w||^2 (w is at hand: a dot
// product of its own read it back in two launches of 5.4 and 1.6 us).
template <typename TV>
__global__ __launch_bounds__(kRed) void k_gemv_sub(const TV *__restrict__ V, int64_t ld_v, int k,
                                                   const double2 *__restrict__ h, double2 *__restrict__ w,
                                                   int64_t len, double *__restrict__ sq,
                                                   const int32_t *__restrict__ skip) {
  if (skip && *skip) return;  // the whole grid
  const int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  double n2 = 0.0;
  if (i < len) {
    cx<double> acc = ld<double>(w[i]);
    int j = 0;
    for (; j + 8 <= k; j += 8) {  // eight loads in flight per lane
      TV a[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) a[u] = V[(j + u) * ld_v + i];
#pragma unroll
      for (int u = 0; u < 8; ++u) acc = acc - mk<double>(a[u].x, a[u].y) * ld<double>(h[j + u]);
    }
    for (; j < k; ++j) {
      const TV a = V[j * ld_v + i];
      acc = acc - mk<double>(a.x, a.y) * ld<double>(h[j]);
    }
    w[i] = st(acc);
    n2 = acc.re * acc.re + acc.im * acc.im;
  }
  if (!sq) return;
  __shared__ double red[kRed / 64];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) n2 += __shfl_xor(n2, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = n2;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = red[0];
#pragma unroll
    for (int v = 1; v < kRed / 64; ++v) s += red[v];
    sq[blockIdx.x] = s;
  }
}

// nrm = ||w||^2 from the shares of k_gemv_sub (skip: the pass was not needed and
// nrm stays).  With flag, whether the second Gram-Schmidt pass is needed, which
// is when the first cancelled much of the vector (Daniel, Gragg, Kaufman and
// Stewart): flag = ||w after||^2 >= eta2 ||w before||^2.
__global__ __launch_bounds__(kRed) void k_norm_final(const double *__restrict__ sq, int nb,
                                                     double2 *__restrict__ nrm, const int32_t *__restrict__ skip,
                                                     const double2 *__restrict__ before, double eta2,
                                                     int32_t *__restrict__ flag) {
  if (skip && *skip) return;
  __shared__ double red[kRed / 64];
  double n2 = 0.0;
  for (int b = threadIdx.x; b < nb; b += kRed) n2 += sq[b];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) n2 += __shfl_xor(n2, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = n2;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = red[0];
#pragma unroll
    for (int v = 1; v < kRed / 64; ++v) s += red[v];
    nrm[0] = make_double2(s, 0.0);
    if (flag) flag[0] = s >= eta2 * before->x ? 1 : 0;
  }
}

__global__ __launch_bounds__(kRed) void k_proj_fix(double2 *__restrict__ h, const double2 *__restrict__ q, int k) {
  __shared__ double sr[kRed], si[kRed];
  double re = 0.0, im = 0.0;
  for (int i = threadIdx.x; i < k; i += kRed) {  // q^H h
    re += q[i].x * h[i].x + q[i].y * h[i].y;
    im += q[i].x * h[i].y - q[i].y * h[i].x;
  }
  sr[threadIdx.x] = re;
  si[threadIdx.x] = im;
  __syncthreads();
  for (int o = kRed / 2; o > 0; o >>= 1) {
    if (threadIdx.x < o) {
      sr[threadIdx.x] += sr[threadIdx.x + o];
      si[threadIdx.x] += si[threadIdx.x + o];
    }
    __syncthreads();
  }
  const double ar = sr[0], ai = si[0];
  for (int i = threadIdx.x; i < k; i += kRed) {
    const double2 qi = q[i];
    h[i].x -= qi.x * ar - qi.y * ai;
    h[i].y -= qi.x * ai + qi.y * ar;
  }
}

__global__ void k_scale_to32(float2 *__restrict__ v, const double2 *__restrict__ src, int64_t len, double s) {
  const int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (i >= len) return;
  const double2 a = src[i];
  v[i] = make_float2(static_cast<float>(s * a.x), static_cast<float>(s * a.y));
}

__global__ void k_scale(double2 *__restrict__ v, const double2 *__restrict__ src, int64_t len, double s) {
  const int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (i >= len) return;
  const double2 a = src[i];
  v[i] = make_double2(s * a.x, s * a.y);
}

__global__ void k_axpy_c(double2 *__restrict__ y, const double2 *__restrict__ x, int64_t len,
                         double ar, double ai) {
  const int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (i >= len) return;
  const cx<double> r = ld<double>(y[i]) + mk(ar, ai) * ld<double>(x[i]);
  y[i] = st(r);
}

// Deterministic pseudo-random fill in [-1, 1) (tuning input with realistic
// operand switching; zero operands run faster and mislead the tuner).
__global__ void k_fill_hash(double *__restrict__ v, int64_t len, uint32_t seed) {
  const int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (i >= len) return;
  uint32_t h = static_cast<uint32_t>(i) * 2654435761u ^ seed;
  h ^= h >> 16;
  h *= 2246822519u;
  h ^= h >> 13;
  h *= 3266489917u;
  h ^= h >> 16;
  v[i] = static_cast<double>(h) * (2.0 / 4294967296.0) - 1.0;
}
__global__ void k_fill_hash32(float *__restrict__ v, int64_t len, uint32_t seed) {
  const int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (i >= len) return;
  uint32_t h = static_cast<uint32_t>(i) * 2654435761u ^ seed;
  h ^= h >> 16;
  h *= 2246822519u;
  h ^= h >> 13;
  h *= 3266489917u;
  h ^= h >> 16;
  v[i] = static_cast<float>(static_cast<double>(h) * (2.0 / 4294967296.0) - 1.0);
}

__global__ void k_to32(const double2 *__restrict__ a, float2 *__restrict__ b, int64_t len) {
  const int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (i < len) b[i] = make_float2(static_cast<float>(a[i].x), static_cast<float>(a[i].y));
}
__global__ void k_to64(const float2 *__restrict__ a, double2 *__restrict__ b, int64_t len) {
  const int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (i < len) b[i] = make_double2(static_cast<double>(a[i].x), static_cast<double>(a[i].y));
}

// ---------------------------------------------------------------------------
// Dispatch over the expansion order.
#define MPSL_P_CASES(X) \
  X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(17) \
  X(18) X(19) X(20)

}  // namespace

// Chunk count for a launch of bpc blocks per chunk whose blocks all carry the
// same work.  With `slots` blocks resident at once on the whole chip
// (compute units x blocks per unit), B blocks run in ceil(B / slots) waves,
// and each block holds 1/c of the work, so the launch takes about
// ceil(bpc c / slots) / c; of the counts in [lo, hi] the smallest within 3 %
// of the best is taken (fewer partial slots to sum).  At 5000 particles and
// 26816 nodes the FP32 S2L's 26 chunks made 1040 blocks for 1024 slots, a
// second wave of 16 blocks (0.82 ms; 50 chunks, 2000 blocks: about 0.63 ms).
static int balanced_chunks(int64_t bpc, int64_t slots, int lo, int hi) {
  lo = std::max(1, lo);
  hi = std::max(lo, hi);
  slots = std::max<int64_t>(1, slots);
  auto cost = [&](int c) { return static_cast<double>((bpc * c + slots - 1) / slots) / c; };
  double best = 1e300;
  for (int c = lo; c <= hi; ++c) best = std::min(best, cost(c));
  for (int c = lo; c <= hi; ++c)
    if (cost(c) <= 1.03 * best) return c;
  return lo;
}

// Blocks of the matrix-core S2L kernel resident per compute unit (occupancy
// query, cached per precision and order; 1 if the query fails).
template <typename T>
static int s2l_resident(int p) {
  static std::atomic<int> cache[kMaxP + 1];
  if (p < kMinP || p > kMaxP) return 1;
  int r = cache[p].load(std::memory_order_relaxed);
  if (r > 0) return r;
  constexpr int MT = s2l_tiles<T>();
  const void *fn = nullptr;
  switch (p) {
#define X(PP) \
  case PP: fn = reinterpret_cast<const void *>(&k_s2l_mfma<T, PP, MT>); break;
    MPSL_P_CASES(X)
#undef X
  }
  int nb = 0;
  if (!fn || hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, 64 * kS2lWaves, 0) != hipSuccess || nb < 1) {
    (void)hipGetLastError();
    nb = 1;
  }
  cache[p].store(nb, std::memory_order_relaxed);
  return nb;
}

int chunks_s2l(const mpsl_ctx *ctx, int nrhs, int prec) {
  if (ctx->somm.active) {  // the interpolated S2L: chunks of coarse nodes, one slot each
    const int tb = cdiv(ctx->n, 128) * nrhs;
    const int c0 = std::max(1, std::min(64, std::min(cdiv(1024, tb), 2 * ctx->somm.nc)));
    // fewer where the blocks (64 particles) would give some compute units a
    // second one and others not: with 256 units and one right-hand side that is
    // 257 to 448 particles, where the cap of 64 chunks binds, and nowhere else
    // (300 particles, FP64: 64 chunks 15.8 us, 51 12.9)
    const int64_t nb = static_cast<int64_t>(cdiv(ctx->n, 64)) * nrhs;
    return nb * c0 > ctx->n_cu && nb * c0 < 2 * ctx->n_cu ? static_cast<int>(ctx->n_cu / nb) : c0;
  }
  if (ctx->s2l_chunks > 0) return std::min(ctx->s2l_chunks, ctx->ns);
  // about 1024 blocks of 128 lanes' worth of particles, at least 8 nodes per
  // chunk; on long contours raised by up to 2x to fill the last wave of
  // blocks (fewer chunks would enlarge the coefficient rows that the resident
  // blocks read at once: at 26816 nodes 19 FP64 chunks ran slower than 26,
  // 29 faster).  Short contours keep it: each chunk adds a partial slot of n P
  // entries to write and sum, about what the better fill gains at 1024 nodes.
  const int tb = cdiv(ctx->n, kThreads) * nrhs;
  const int cmax = std::max(1, ctx->ns / 8);
  const int c0 = std::min(cdiv(1024, tb), cmax);
  if (ctx->ns < 4096) return std::max(1, c0);
  const bool f64 = prec == MPSL_FP64;
  const int64_t bpc =
      static_cast<int64_t>(cdiv(ctx->n, 16 * kS2lWaves * (f64 ? s2l_tiles<double>() : s2l_tiles<float>()))) * nrhs;
  const int64_t slots = static_cast<int64_t>(ctx->n_cu) * (f64 ? s2l_resident<double>(ctx->p) : s2l_resident<float>(ctx->p));
  return balanced_chunks(bpc, slots, std::max(1, c0), std::min(2 * c0, cmax));
}

// Blocks of the matrix-core M2S kernel resident per compute unit (occupancy
// query, cached per precision and order; 1 if the query fails).
template <typename T>
static int m2s_resident(int p) {
  static std::atomic<int> cache[kMaxP + 1];
  if (p < kMinP || p > kMaxP) return 1;
  int r = cache[p].load(std::memory_order_relaxed);
  if (r > 0) return r;
  const void *fn = nullptr;
  switch (p) {
#define X(PP) \
  case PP: fn = reinterpret_cast<const void *>(&k_m2s_mfma<T, PP, false>); break;
    MPSL_P_CASES(X)
#undef X
  }
  int nb = 0;
  if (!fn || hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, 64 * kM2sWaves, 0) != hipSuccess || nb < 1) {
    (void)hipGetLastError();
    nb = 1;
  }
  cache[p].store(nb, std::memory_order_relaxed);
  return nb;
}

// M2S chunks with at most by_n of them for the particles' sake.
static int m2s_count(const mpsl_ctx *ctx, int nrhs, int prec, int64_t by_n) {
  const int qb = cdiv(ctx->ns, kThreads) * 2 * nrhs;
  const int c0 = static_cast<int>(
      std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(cdiv(2048, qb), by_n), ctx->n)));
  // short contours: lowered by up to half to the count whose blocks fill
  // whole waves of the resident slots (1024 nodes, 5000 particles: 63 chunks
  // made 2016 blocks for 1792 FP32 slots; 55 make 1760).  Long contours run
  // many waves already and keep it (3 to 20 chunks within 0.5 % at 26816 nodes).
  if (ctx->ns >= 4096) return c0;
  const bool f64 = prec == MPSL_FP64;
  const int64_t bpc = static_cast<int64_t>(cdiv(ctx->ns, 16 * kM2sWaves)) * 2 * nrhs;
  const int64_t slots = static_cast<int64_t>(ctx->n_cu) * (f64 ? m2s_resident<double>(ctx->p) : m2s_resident<float>(ctx->p));
  return balanced_chunks(bpc, slots, std::max(1, c0 / 2), c0);
}

int m2s_part_chunks(const mpsl_ctx *ctx, int nrhs, int prec) {
  if (ctx->m2s_chunks > 0) return static_cast<int>(std::min<int64_t>(ctx->m2s_chunks, ctx->n));
  // about 2048 node-group x chunk tasks, but at least 80 particles per chunk:
  // shorter chunks spend more on the epilogue and on summing the partials
  // than they gain in parallelism (1024 nodes, 5000 particles: 256 -> 63
  // chunks, M2S and partial sum 75 -> about 45 us in FP32).
  return m2s_count(ctx, nrhs, prec, cdiv(ctx->n, 80));
}

int chunks_m2s(const mpsl_ctx *ctx, int nrhs, int prec) {
  const int base = m2s_part_chunks(ctx, nrhs, prec);
  if (ctx->m2s_chunks > 0) return base;
  // Up to 16 chunks 32 particles will do: their steps are a serial chain (512
  // nodes, p = 16, whole matvec, chunks of 80 and 32: 203 particles 48.9 and 44.9
  // us in FP64, 35.6 and 34.2 in FP32; 500: 79.8 and 76.4, 59.9 and 56.5).  One
  // chunk to 48, which needs no k_nodes (p = 8, FP64, one and two chunks: 16
  // particles 21.7 and 23.6 us, 48: 24.4 and 25.4, 64: 25.4 and 25.6).  The
  // partials of these chunks lie in the S2L coefficient table of the other
  // precision (m2s_partials), which takes 2P of them in FP32 and P / 2 in FP64.
  if (ctx->n <= 48) return base;
  const int P = 2 * ctx->p + 1, most = std::min(16, prec == MPSL_FP64 ? P / 2 : 2 * P);
  return std::max(base, std::min(most, m2s_count(ctx, nrhs, prec, std::max(cdiv(ctx->n, 80), std::min(16, cdiv(ctx->n, 32))))));
}

// Where the M2S writes its partials: m2s_part, sized for m2s_part_chunks, or with
// more chunks the S2L coefficients of the other precision, which nothing reads
// between the M2S and the end of the node sums.
static void *m2s_partials(const mpsl_ctx *ctx, int nrhs, int prec, int chunks) {
  if (chunks <= m2s_part_chunks(ctx, nrhs, prec)) return ctx->m2s_part.p;
  return prec == MPSL_FP64 ? ctx->Up32.p : ctx->Up64.p;
}

#define LAUNCH_CHECK(ctx)                                                          \
  do {                                                                             \
    hipError_t e_ = hipGetLastError();                                             \
    if (e_ != hipSuccess) return set_err(ctx, MPSL_EHIP, std::string("kernel launch: ") + hipGetErrorString(e_)); \
  } while (0)

int launch_geom_tables(mpsl_ctx *ctx) {
  const int64_t tot = ctx->n * static_cast<int64_t>(ctx->ns);
  const int threads = 256;
  hipLaunchKernelGGL(k_geom_tables, dim3(cdiv(tot, threads)), dim3(threads), 0, ctx->stream,
                     static_cast<const double2 *>(ctx->gt.xy.p), static_cast<const double2 *>(ctx->ct.lam.p),
                     static_cast<const double2 *>(ctx->ct.gw.p) + ctx->ns,  // g2 stored after g1
                     static_cast<int>(ctx->n), ctx->ns, ctx->d, static_cast<double2 *>(ctx->gt.E64.p),
                     static_cast<double2 *>(ctx->gt.F64.p), static_cast<float2 *>(ctx->gt.E32.p),
                     static_cast<float2 *>(ctx->gt.F32.p));
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

int launch_pair_tables(mpsl_ctx *ctx) {
  const int64_t tot = ctx->n * ctx->n;
  hipLaunchKernelGGL(k_pair_tables, dim3(cdiv(tot, 256)), dim3(256), 0, ctx->stream,
                     static_cast<const double2 *>(ctx->gt.xy.p), static_cast<int>(ctx->n), ctx->k2.real(),
                     static_cast<double2 *>(ctx->gt.pair64.p), static_cast<float2 *>(ctx->gt.pair32.p));
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

// nodes: with one chunk, on to the S2L coefficients.
template <typename T>
static int launch_m2s_t(mpsl_ctx *ctx, const void *beta, int nrhs, bool nodes = false) {
  const int n = static_cast<int>(ctx->n);
  const bool f64 = std::is_same<T, double>::value;
  const int prec = f64 ? MPSL_FP64 : MPSL_FP32;
  const int chunks = chunks_m2s(ctx, nrhs, prec);
  const int chunk_len = cdiv(n, chunks);
  const dim3 grid = nodes ? dim3(cdiv(ctx->ns, 8 * kM2sWaves), 1, nrhs)
                          : dim3(cdiv(ctx->ns, 16 * kM2sWaves), chunks, 2 * nrhs);
  const auto *E = static_cast<const cv_t<T> *>(f64 ? ctx->gt.E64.p : ctx->gt.E32.p);
  const auto *W = static_cast<const cv_t<T> *>(f64 ? ctx->ct.W64.p : ctx->ct.W32.p);
  const auto *b = static_cast<const cv_t<T> *>(beta);
  auto *part = static_cast<cv_t<T> *>(m2s_partials(ctx, nrhs, prec, chunks));
  const auto *R = static_cast<const double2 *>(ctx->ct.R.p), *cq = static_cast<const double2 *>(ctx->ct.cq.p),
             *U = static_cast<const double2 *>(ctx->ct.U64.p);
  auto *Up = static_cast<cv_t<T> *>(f64 ? ctx->Up64.p : ctx->Up32.p);
  const dim3 blk(64 * kM2sWaves);
  switch (ctx->p) {
#define X(PP)                                                                                                       \
  case PP:                                                                                                          \
    if (nodes)                                                                                                      \
      hipLaunchKernelGGL((k_m2s_mfma<T, PP, true>), grid, blk, 0, ctx->stream, E, b, W, part, n, ctx->ns,           \
                         chunk_len, chunks, R, cq, U, Up);                                                          \
    else                                                                                                            \
      hipLaunchKernelGGL((k_m2s_mfma<T, PP, false>), grid, blk, 0, ctx->stream, E, b, W, part, n, ctx->ns,          \
                         chunk_len, chunks, R, cq, U, Up);                                                          \
    break;
    MPSL_P_CASES(X)
#undef X
    default: return set_err(ctx, MPSL_EUNSUPPORTED, "expansion order outside 1..20");
  }
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

template <typename T>
static int launch_nodes_t(mpsl_ctx *ctx, void *spec, int nrhs) {
  const bool f64 = std::is_same<T, double>::value;
  const int prec = f64 ? MPSL_FP64 : MPSL_FP32;
  const int chunks = chunks_m2s(ctx, nrhs, prec);
  hipLaunchKernelGGL(k_nodes<T>, dim3(cdiv(ctx->ns, kNodeBlock), nrhs), dim3(2 * kNodeBlock * kNodeLanes), 0,
                     ctx->stream, static_cast<const cv_t<T> *>(m2s_partials(ctx, nrhs, prec, chunks)), ctx->ns, chunks,
                     static_cast<const double2 *>(ctx->ct.R.p), static_cast<const double2 *>(ctx->ct.cq.p),
                     static_cast<const double2 *>(ctx->ct.U64.p), 2 * ctx->p + 1, static_cast<double2 *>(spec),
                     static_cast<cv_t<T> *>(f64 ? ctx->Up64.p : ctx->Up32.p));
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

int launch_m2s(mpsl_ctx *ctx, int prec, const void *beta, void *spec, int nrhs) {
  if (ctx->somm.active) return launch_m2s_interp(ctx, prec, beta, spec, nrhs);
  if (prec == MPSL_FP64) {
    const int rc = launch_m2s_t<double>(ctx, beta, nrhs);
    return rc ? rc : launch_nodes_t<double>(ctx, spec, nrhs);
  }
  const int rc = launch_m2s_t<float>(ctx, beta, nrhs);
  return rc ? rc : launch_nodes_t<float>(ctx, spec, nrhs);
}

int launch_m2s_coef(mpsl_ctx *ctx, int prec, const void *beta, int nrhs) {
  if (ctx->somm.active) {
    int rc = launch_m2s_interp(ctx, prec, beta, ctx->spec.p, nrhs);
    if (!rc) rc = launch_reflect(ctx, ctx->spec.p, nullptr, ctx->sigma.p, nrhs);
    return rc ? rc : launch_s2l_coef(ctx, ctx->sigma.p, nrhs);
  }
  if (chunks_m2s(ctx, nrhs, prec) == 1)
    return prec == MPSL_FP64 ? launch_m2s_t<double>(ctx, beta, nrhs, true) : launch_m2s_t<float>(ctx, beta, nrhs, true);
  if (prec == MPSL_FP64) {
    const int rc = launch_m2s_t<double>(ctx, beta, nrhs);
    return rc ? rc : launch_nodes_t<double>(ctx, nullptr, nrhs);
  }
  const int rc = launch_m2s_t<float>(ctx, beta, nrhs);
  return rc ? rc : launch_nodes_t<float>(ctx, nullptr, nrhs);
}

int launch_reflect(mpsl_ctx *ctx, const void *spec, const double *src, void *sigma, int nrhs) {
  const int ns = ctx->ns;
  hipLaunchKernelGGL(k_reflect, dim3(cdiv(ns, 256), nrhs), dim3(256), 0, ctx->stream,
                     static_cast<const double2 *>(spec), static_cast<const double2 *>(ctx->ct.R.p),
                     static_cast<const double2 *>(ctx->ct.srcfac.p), static_cast<const double2 *>(ctx->ct.lam.p),
                     static_cast<const double2 *>(ctx->ct.gw.p), ns, src ? 1 : 0, src ? src[0] : 0.0,
                     src ? src[1] - ctx->yint[0] : 0.0, static_cast<double2 *>(sigma));
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

int launch_s2l_coef(mpsl_ctx *ctx, const void *sigma, int nrhs) {
  if (ctx->somm.active) {  // the interpolated S2L reads the densities directly
    ctx->somm.sigma = sigma;
    return MPSL_OK;
  }
  const int P = 2 * ctx->p + 1;
  const int64_t tot = 2LL * ctx->ns * P * nrhs;
  hipLaunchKernelGGL(k_s2l_coef, dim3(cdiv(tot, 256)), dim3(256), 0, ctx->stream,
                     static_cast<const double2 *>(sigma), static_cast<const double2 *>(ctx->ct.cq.p),
                     static_cast<const double2 *>(ctx->ct.U64.p), ctx->ns, P, nrhs,
                     static_cast<double2 *>(ctx->Up64.p), static_cast<float2 *>(ctx->Up32.p));
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

template <typename T>
static int launch_s2l_t(mpsl_ctx *ctx, void *part, int chunks, int nrhs, int64_t pstride) {
  const int n = static_cast<int>(ctx->n);
  const int chunk_len = cdiv(ctx->ns, chunks);
  constexpr int MT = s2l_tiles<T>();
  const dim3 grid(cdiv(n, 16 * MT * kS2lWaves), chunks, nrhs);
  const bool f64 = std::is_same<T, double>::value;
  const auto *F = static_cast<const cv_t<T> *>(f64 ? ctx->gt.F64.p : ctx->gt.F32.p);
  const auto *Up = static_cast<const cv_t<T> *>(f64 ? ctx->Up64.p : ctx->Up32.p);
  auto *o = static_cast<cv_t<T> *>(part);
  switch (ctx->p) {
#define X(PP) \
  case PP: hipLaunchKernelGGL((k_s2l_mfma<T, PP, MT>), grid, dim3(64 * kS2lWaves), 0, ctx->stream, F, Up, o, n, ctx->ns, chunk_len, pstride); break;
    MPSL_P_CASES(X)
#undef X
    default: return set_err(ctx, MPSL_EUNSUPPORTED, "expansion order outside 1..20");
  }
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

int launch_s2l(mpsl_ctx *ctx, int prec, void *part, int chunks, int nrhs, int64_t pstride) {
  if (ctx->somm.active) return launch_s2l_interp(ctx, prec, part, chunks, nrhs, pstride);
  return prec == MPSL_FP64 ? launch_s2l_t<double>(ctx, part, chunks, nrhs, pstride)
                           : launch_s2l_t<float>(ctx, part, chunks, nrhs, pstride);
}

int launch_sum_parts(mpsl_ctx *ctx, int prec, const void *part, int chunks, void *alpha, int nrhs, int64_t stride) {
  const int64_t len = ctx->n * static_cast<int64_t>(2 * ctx->p + 1);
  const dim3 grid(cdiv(len * kSumLanes, 256), nrhs);
  if (prec == MPSL_FP64)
    hipLaunchKernelGGL(k_sum_parts<double>, grid, dim3(256), 0, ctx->stream, static_cast<const double2 *>(part), chunks,
                       len, static_cast<double2 *>(alpha), stride);
  else
    hipLaunchKernelGGL(k_sum_parts<float>, grid, dim3(256), 0, ctx->stream, static_cast<const float2 *>(part), chunks,
                       len, static_cast<float2 *>(alpha), stride);
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

template <typename T>
static int launch_sapply_t(mpsl_ctx *ctx, const void *x, const void *alpha, int slots, void *y, int nrhs,
                           int64_t astride) {
  const int n = static_cast<int>(ctx->n);
  const bool f64 = std::is_same<T, double>::value;
  const auto *S = static_cast<const cv_t<T> *>(f64 ? ctx->S64.p : ctx->S32.p);
  const auto *rot = static_cast<const cv_t<T> *>(f64 ? ctx->gt.rot64.p : ctx->gt.rot32.p);
  const dim3 grid(cdiv(n, 16), nrhs);
  const auto *xx = static_cast<const cv_t<T> *>(x);
  const auto *aa = static_cast<const cv_t<T> *>(alpha);
  auto *yy = static_cast<cv_t<T> *>(y);
  // per-particle types only when several prototypes and a typed geometry
  const bool typed = ctx->n_types > 1 && !ctx->ptype.empty();
  const int32_t *ty = typed ? static_cast<const int32_t *>(ctx->types_dev.p) : nullptr;
  const int nt = typed ? ctx->n_types : 1;
  switch (ctx->p) {
#define X(PP) \
  case PP:                                                                                                         \
    if (slots > kSapplyFew)                                                                                        \
      hipLaunchKernelGGL((k_sapply<T, PP, 512>), grid, dim3(512), 0, ctx->stream, xx, aa, slots, S, rot, n, yy,    \
                         astride, ty, nt);                                                                         \
    else                                                                                                           \
      hipLaunchKernelGGL((k_sapply<T, PP, 256>), grid, dim3(256), 0, ctx->stream, xx, aa, slots, S, rot, n, yy,    \
                         astride, ty, nt);                                                                         \
    break;
    MPSL_P_CASES(X)
#undef X
    default: return set_err(ctx, MPSL_EUNSUPPORTED, "expansion order outside 1..20");
  }
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

// Bytes of partials that a tile block of k_sapply sums without help.
constexpr size_t kSapplySumBytes = 64 * 1024;

int launch_sapply(mpsl_ctx *ctx, int prec, const void *x, void *alpha, int slots, void *y, int nrhs, int64_t astride) {
  // The tile blocks of k_sapply sum the partials themselves where they fill
  // the chip or have little to sum; else a launch of its own spreads the sums
  // over more compute units (203 particles, p = 16, FP32, 83 slots: 42.7 us per
  // matvec with the extra launch, 49.2 us without; 1000, p = 12, FP64, 384
  // slots: 207 and 249 us; 20000, p = 16, FP32, 16 slots: 1040 us without it,
  // 1060 us with).
  const size_t esz = prec == MPSL_FP64 ? sizeof(double2) : sizeof(float2);
  const size_t tile = 16 * (2 * ctx->p + 1) * esz * slots;
  if (slots > 1 && tile > kSapplySumBytes && static_cast<int64_t>(cdiv(ctx->n, 16)) * nrhs < ctx->n_cu) {
    if (const int rc = launch_sum_parts(ctx, prec, alpha, slots, alpha, nrhs, astride)) return rc;
    slots = 1;
  }
  return prec == MPSL_FP64 ? launch_sapply_t<double>(ctx, x, alpha, slots, y, nrhs, astride)
                           : launch_sapply_t<float>(ctx, x, alpha, slots, y, nrhs, astride);
}

int launch_proj_fix(mpsl_ctx *ctx, void *h, const void *q, int k) {
  hipLaunchKernelGGL(k_proj_fix, dim3(1), dim3(kRed), 0, ctx->stream, static_cast<double2 *>(h),
                     static_cast<const double2 *>(q), k);
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

size_t dotc_scratch_bytes(int k) { return static_cast<size_t>(std::max(k, 1)) * kDotBlocks * sizeof(double2); }

int launch_dotc_multi(mpsl_ctx *ctx, const void *V, int64_t ld_v, int k, const void *w, int64_t len,
                      void *h_out, const int32_t *skip, int v_prec) {
  if (ctx->scal.bytes < dotc_scratch_bytes(k))
    return set_err(ctx, MPSL_EINVAL, "reduction scratch too small for " + std::to_string(k) + " dot products");
  auto *scr = static_cast<double2 *>(ctx->scal.p);
  const dim3 grid(kDotBlocks, cdiv(k, kDotVecs));
  if (v_prec == MPSL_FP32)
    hipLaunchKernelGGL(k_dotc_part<float2>, grid, dim3(kRed), 0, ctx->stream, static_cast<const float2 *>(V), ld_v,
                       k, static_cast<const double2 *>(w), len, scr, skip);
  else
    hipLaunchKernelGGL(k_dotc_part<double2>, grid, dim3(kRed), 0, ctx->stream, static_cast<const double2 *>(V), ld_v,
                       k, static_cast<const double2 *>(w), len, scr, skip);
  LAUNCH_CHECK(ctx);
  hipLaunchKernelGGL(k_dotc_final, dim3(cdiv(k, 4)), dim3(256), 0, ctx->stream, scr, k, kDotBlocks,
                     static_cast<double2 *>(h_out), skip);
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

static int gemv_sub(mpsl_ctx *ctx, const void *V, int64_t ld_v, int k, const void *h, void *w, int64_t len,
                    double *sq, const int32_t *skip, int v_prec) {
  const dim3 grid(cdiv(len, kRed));
  if (v_prec == MPSL_FP32)
    hipLaunchKernelGGL(k_gemv_sub<float2>, grid, dim3(kRed), 0, ctx->stream, static_cast<const float2 *>(V), ld_v, k,
                       static_cast<const double2 *>(h), static_cast<double2 *>(w), len, sq, skip);
  else
    hipLaunchKernelGGL(k_gemv_sub<double2>, grid, dim3(kRed), 0, ctx->stream, static_cast<const double2 *>(V), ld_v,
                       k, static_cast<const double2 *>(h), static_cast<double2 *>(w), len, sq, skip);
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

int launch_gemv_sub(mpsl_ctx *ctx, const void *V, int64_t ld_v, int k, const void *h, void *w, int64_t len,
                    const int32_t *skip, int v_prec) {
  return gemv_sub(ctx, V, ld_v, k, h, w, len, nullptr, skip, v_prec);
}

size_t gemv_norm_scratch_bytes(int64_t len) { return static_cast<size_t>(cdiv(len, kRed)) * sizeof(double); }

int launch_gemv_norm(mpsl_ctx *ctx, const void *V, int64_t ld_v, int k, const void *h, void *w, int64_t len,
                     void *nrm, const int32_t *skip, int v_prec, const void *before, double eta2, int32_t *flag) {
  if (ctx->scal.bytes < gemv_norm_scratch_bytes(len))
    return set_err(ctx, MPSL_EINVAL, "reduction scratch too small for the norm");
  auto *sq = static_cast<double *>(ctx->scal.p);
  const int rc = gemv_sub(ctx, V, ld_v, k, h, w, len, sq, skip, v_prec);
  if (rc) return rc;
  hipLaunchKernelGGL(k_norm_final, dim3(1), dim3(kRed), 0, ctx->stream, sq, cdiv(len, kRed),
                     static_cast<double2 *>(nrm), skip, static_cast<const double2 *>(before), eta2, flag);
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

int launch_scale_to_fp32(mpsl_ctx *ctx, void *v32, int64_t len, double s, const void *src) {
  hipLaunchKernelGGL(k_scale_to32, dim3(cdiv(len, 256)), dim3(256), 0, ctx->stream, static_cast<float2 *>(v32),
                     static_cast<const double2 *>(src), len, s);
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

int launch_scale(mpsl_ctx *ctx, void *v, int64_t len, double s, const void *src) {
  hipLaunchKernelGGL(k_scale, dim3(cdiv(len, 256)), dim3(256), 0, ctx->stream, static_cast<double2 *>(v),
                     static_cast<const double2 *>(src), len, s);
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

int launch_axpy_c(mpsl_ctx *ctx, void *y, const void *x, int64_t len, double a_re, double a_im) {
  hipLaunchKernelGGL(k_axpy_c, dim3(cdiv(len, 256)), dim3(256), 0, ctx->stream, static_cast<double2 *>(y),
                     static_cast<const double2 *>(x), len, a_re, a_im);
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

int launch_to_fp32(mpsl_ctx *ctx, const void *x64, void *x32, int64_t len) {
  hipLaunchKernelGGL(k_to32, dim3(cdiv(len, 256)), dim3(256), 0, ctx->stream, static_cast<const double2 *>(x64),
                     static_cast<float2 *>(x32), len);
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

int launch_fill_hash(mpsl_ctx *ctx, int prec, void *v, int64_t n_complex, uint32_t seed) {
  const int64_t len = 2 * n_complex;
  if (prec == MPSL_FP64)
    hipLaunchKernelGGL(k_fill_hash, dim3(cdiv(len, 256)), dim3(256), 0, ctx->stream, static_cast<double *>(v), len, seed);
  else
    hipLaunchKernelGGL(k_fill_hash32, dim3(cdiv(len, 256)), dim3(256), 0, ctx->stream, static_cast<float *>(v), len, seed);
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

int launch_to_fp64(mpsl_ctx *ctx, const void *x32, void *x64, int64_t len) {
  hipLaunchKernelGGL(k_to64, dim3(cdiv(len, 256)), dim3(256), 0, ctx->stream, static_cast<const float2 *>(x32),
                     static_cast<double2 *>(x64), len);
  LAUNCH_CHECK(ctx);
  return MPSL_OK;
}

}  // namespace mpsl
