// M2S and S2L by tile-local interpolation in lambda (Sections 5.2.1, 5.3).
//
// The direct transforms couple every particle m with every contour node q
// through e^{-i lam_q x_m +- g2_q y_m} (M2S) and e^{i lam_q x_l +- g2_q y_l}
// (S2L).  With the particles grouped in tiles of centre (x_T, y_T) the factor
// splits into a tile part e^{-+i lam x_T +- g2 y_T} and a local part whose
// phase is at most |lam| times the tile size: together with the order weights
// (powers of (lam -+ g2)/k2) the local part is smooth in lambda away from
// lam = +-k2.  Per tile it is evaluated at kSommNc Chebyshev nodes of each
// lambda-interval of length L_I on the contour's lines and interpolated to the
// contour nodes in barycentric form; nodes within d_dir of +-k2 and the nodes
// of the vertical segment are their own coarse nodes (interpolation weight 1).
//
//   M2S: G[T][c]   = sum_{m in T} local_m(c) (beta_m . W(c))
//        spec[q]   = sum_T E_T(q) sum_k L[q][k] G[T][c0(q) + k]
//   S2L: B[T][c]   = sum_{q in run(c)} L[q][k(c)] c_q sigma(q) E'_T(q)
//        alpha_l[n] = sum_c local_l(c) B[T(l)][c] Z_n(c)
//
// Exponentials are evaluated in FP64 (their phases reach |lam| times the strip
// width); sums run in the matvec precision.  The paper's NUFFT forms
// (Sections 5.2.2, 5.3.1) reach the same O(N + N_S) scaling with FFT grids;
// interpolation keeps every step a dense loop.
#include <algorithm>
#include <cmath>
#include <map>

#include "kernels.h"

namespace mpsl {

namespace {

constexpr double kTileW = 8.0, kTileH = 4.0, kIntervalL = 1.0, kDirect = 0.3;

// the expansion orders instantiated (1..20)
#define SOMM_P_CASES(X) \
  X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(17) X(18) X(19) X(20)

template <typename T> __device__ inline cx<T> cvt(cx<double> v) { return {static_cast<T>(v.re), static_cast<T>(v.im)}; }
template <typename T> __device__ inline cx<double> up(cx<T> v) { return {static_cast<double>(v.re), static_cast<double>(v.im)}; }

// M2S, step 2, interval nodes, on the matrix cores: per interval
//   H[T][q] = sum_k G[T][c0 + k] L[q][k]      (M = tile, N = node, K = 24)
//   spec[q] = sum_T e^{-i lam_q x_T + g2_q yy_T} H[T][q]
// One wave per 16 nodes of a block's run of kSiFineNodes (from fblk), the slots
// of trow in steps of 16: lane i supplies G of one slot for A (complex, two
// real MFMAs; the next step's loads are in flight) and B[i / 16][i % 16] = L of
// node i % 16 (loaded once).  The result rows a lane holds are one aligned
// group of four slots, neighbours in one row of tiles, so their factors take
// one exponential and three multiplies by e^{-i lam w} with no divergence
// (walked down the tile columns, which are a few tiles high, nearly every tile
// took an exponential: 5003 particles, 570 tiles, 30528 nodes, FP32, with the
// direct nodes 212 us, now 129; 300 particles, 36 tiles, FP64: 25 -> 14).
// The multiplies are in FP64 in both precisions: in FP32 their roundings doubled
// the error of M2S over gaps of four tiles (1.6 -> 3.0e-7), at the same speed.
// Each lane sums per step in the matvec precision and across steps in FP64;
// the four row groups are added at the end.
//
// The first blocks take the direct nodes (their own coarse node,
// weight 1): kSiDirNodes nodes per block, the tiles shared by kSiDirSplit lanes
// per node (as a launch of its own with four shares per node, 34 blocks on 256
// compute units, they took 80 us of the case above).
constexpr int kSiFineSplit = 4;   // waves per block
constexpr int kSiFineNodes = 64;  // nodes per block (16 per wave)
constexpr int kSiDirNodes = 8;
constexpr int kSiDirSplit = 64 * kSiFineSplit / kSiDirNodes;
template <typename T>
__device__ void si_fine_dir(const cv_t<T> *__restrict__ G, const double2 *__restrict__ lam,
                            const double2 *__restrict__ g2, const double2 *__restrict__ txy,
                            const int *__restrict__ dir, int db, int ndir, int ns, int nT, int nc, double d,
                            double2 *__restrict__ spec) {
  __shared__ double2 red[kSiDirSplit][kSiDirNodes];
  const int j = threadIdx.x / kSiDirNodes, ql = threadIdx.x - j * kSiDirNodes;
  const int i = db * kSiDirNodes + ql;
  const bool act = i < ndir;
  const int q = act ? dir[2 * i] : 0, c = act ? dir[2 * i + 1] : 0;
  const int s = blockIdx.y & 1, r = blockIdx.y >> 1;
  const double lr = lam[q].x, li = lam[q].y, gr = g2[q].x, gi = g2[q].y;
  const cv_t<T> *Gs = G + ((static_cast<int64_t>(r) * 2 + s) * nT) * nc + c;
  cx<double> acc = mk(0.0, 0.0);
  if (act) {
    for (int t = j; t < nT; t += kSiDirSplit) {
      const double xT = txy[t].x, yT = txy[t].y;
      const double yy = s == 0 ? yT : -(d + yT);
      acc = acc + up<T>(cexpT<T>(li * xT + gr * yy, -lr * xT + gi * yy)) * up<T>(ld<T>(Gs[static_cast<int64_t>(t) * nc]));
    }
  }
  red[j][ql] = st(acc);
  __syncthreads();
  if (j == 0 && act) {
    cx<double> sum = ld<double>(red[0][ql]);
#pragma unroll
    for (int u = 1; u < kSiDirSplit; ++u) sum = sum + ld<double>(red[u][ql]);
    spec[(static_cast<int64_t>(r) * 2 + s) * ns + q] = st(sum);
  }
}

// Slot of A row r, so that result register j of lane group g is slot 4 g + j.
template <typename T> __device__ inline int slot_of_row(int r) { return sizeof(T) == 4 ? r : 4 * (r & 3) + (r >> 2); }

// SPARSE: slots of tiles that stand apart, each with its own exponential.
template <typename T, bool SPARSE>
__global__ __launch_bounds__(64 * kSiFineSplit) void k_si_fine(
    const cv_t<T> *__restrict__ G, const double2 *__restrict__ lam, const double2 *__restrict__ g2,
    const double2 *__restrict__ txy, const int2 *__restrict__ trow, const double2 *__restrict__ tgrp,
    const int *__restrict__ ivl, const int *__restrict__ fperm, const int *__restrict__ fblk, const double *__restrict__ Lw,
    const int *__restrict__ dir, int nfb, int ndir, int ns, int nT, int nrow, int nc, double d, double tile_w,
    double2 *__restrict__ spec) {
  static_assert(kSiFineNodes == 16 * kSiFineSplit, "16 nodes per wave");
  static_assert(kSommNc == 24, "six K steps of four columns");
  typedef typename mfma4<T>::v4 v4;
  const int nd = static_cast<int>(gridDim.x) - nfb;
  if (static_cast<int>(blockIdx.x) < nd) {  // the whole block
    si_fine_dir<T>(G, lam, g2, txy, dir, blockIdx.x, ndir, ns, nT, nc, d, spec);
    return;
  }
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  // XCD-aware order: blocks are dealt to the 8 XCDs round-robin, so block b
  // takes run x q + min(x, rem) + b / 8 (x = b % 8) and each XCD works
  // through consecutive runs of the same intervals
  const int bi = blockIdx.x - nd, xq = nfb / 8, xr = nfb % 8, x = bi % 8;
  const int fb = x * xq + min(x, xr) + bi / 8;
  const int iv = fblk[2 * fb], off = fblk[2 * fb + 1] + 16 * w;
  const int f0 = ivl[4 * iv], nf = ivl[4 * iv + 1], c0 = ivl[4 * iv + 2];
  if (off >= nf) return;  // the whole wave lies past the interval's nodes (no barriers below)
  const int s = blockIdx.y & 1, rr = blockIdx.y >> 1;
  const bool qv = off + r < nf;
  const int q = fperm[f0 + (qv ? off + r : off)];
  T bl[6];  // B operand of the six K steps: L[q][4 ks + g]
#pragma unroll
  for (int ks = 0; ks < 6; ++ks) bl[ks] = qv ? static_cast<T>(Lw[static_cast<int64_t>(q) * kSommNc + 4 * ks + g]) : T(0);
  const double lr = lam[q].x, li = lam[q].y, gr = g2[q].x, gi = g2[q].y;
  const cx<double> Fd = cexpT<double>(li * tile_w, -lr * tile_w);
  const cv_t<T> *Gs = G + ((static_cast<int64_t>(rr) * 2 + s) * nT) * nc + c0 + g;
  const int sa = slot_of_row<T>(r);
  struct Ops {
    cv_t<T> a[6];
    bool av;
    double2 tc;   // centre of the first tile of this lane's group of slots
    int4 t01, t23;  // the group's (tile, step) pairs
  };
  auto tile = [&](int tb) { return trow[min(tb + sa, nrow - 1)].x; };
  auto fetch = [&](int tb, int ta, Ops &o) {  // ta: tile of this lane's A row
    o.av = tb + sa < nrow && ta >= 0;
    const cv_t<T> *Ga = Gs + static_cast<int64_t>(ta >= 0 ? ta : 0) * nc;
#pragma unroll
    for (int ks = 0; ks < 6; ++ks) o.a[ks] = Ga[4 * ks];
    const int gi = min(tb / 4 + g, nrow / 4 - 1);  // nrow is a multiple of 4
    if (!SPARSE) o.tc = tgrp[gi];
    o.t01 = reinterpret_cast<const int4 *>(trow)[2 * gi];
    o.t23 = reinterpret_cast<const int4 *>(trow)[2 * gi + 1];
  };
  Ops nx;
  fetch(0, tile(0), nx);
  int tn = tile(16);
  cx<double> acc = mk(0.0, 0.0);
  for (int tb = 0; tb < nrow; tb += 16) {
    const Ops cu = nx;
    if (tb + 16 < nrow) {
      fetch(tb + 16, tn, nx);
      tn = tile(tb + 32);
    }
    v4 hr = v4{0, 0, 0, 0}, hi = v4{0, 0, 0, 0};
#pragma unroll
    for (int ks = 0; ks < 6; ++ks) {
      const cx<T> a = cu.av ? ld<T>(cu.a[ks]) : mk<T>(0, 0);
      hr = mfma4<T>::mac(a.re, bl[ks], hr);
      hi = mfma4<T>::mac(a.im, bl[ks], hi);
    }
    if (tb + 4 * g < nrow) {
      const int tj[4] = {cu.t01.x, cu.t01.z, cu.t23.x, cu.t23.z}, kj[4] = {cu.t01.y, cu.t01.w, cu.t23.y, cu.t23.w};
      cx<T> blk = mk<T>(0, 0);
      if constexpr (SPARSE) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const double2 tc = txy[max(tj[j], 0)];
          const double yy = s == 0 ? tc.y : -(d + tc.y);
          const cx<T> E = cexpT<T>(li * tc.x + gr * yy, -lr * tc.x + gi * yy);
          if (tj[j] >= 0) cmac(blk, E, mk<T>(hr[j], hi[j]));
        }
      } else {
        const double yy = s == 0 ? cu.tc.y : -(d + cu.tc.y);
        const cx<T> E0 = cexpT<T>(li * cu.tc.x + gr * yy, -lr * cu.tc.x + gi * yy);
        cx<double> E = up<T>(E0);
        cmac(blk, E0, mk<T>(hr[0], hi[0]));
#pragma unroll
        for (int j = 1; j < 4; ++j) {
          if (tj[j] >= 0) {
            E = E * Fd;
            for (int v = 1; v < kj[j]; ++v) E = E * Fd;
            cmac(blk, cvt<T>(E), mk<T>(hr[j], hi[j]));
          }
        }
      }
      acc = acc + up<T>(blk);
    }
  }
  acc.re += __shfl_xor(acc.re, 16);
  acc.im += __shfl_xor(acc.im, 16);
  acc.re += __shfl_xor(acc.re, 32);
  acc.im += __shfl_xor(acc.im, 32);
  if (g == 0 && qv) spec[(static_cast<int64_t>(rr) * 2 + s) * ns + q] = st(acc);
}

// Sum of the node-chunk partials of k_si_coarseB into B[rhs, side][t][c],
// c < nci, in chunk order (the first nsum blocks), and S2L step 1 for the
// direct nodes, one lane per (direct node, tile), in the blocks after them.
template <typename T>
__global__ __launch_bounds__(256) void k_si_coarseB_fin(
    const cv_t<T> *__restrict__ Bp, int nchunk, int64_t rows, int nci, int nsum, const double2 *__restrict__ sigma,
    const double2 *__restrict__ cq, const double2 *__restrict__ lam, const double2 *__restrict__ g2,
    const double2 *__restrict__ txy, const int *__restrict__ dir, int ndir, int ns, int nT, int nc, double d,
    cv_t<T> *__restrict__ B) {
  if (static_cast<int>(blockIdx.x) < nsum) {
    const int64_t e = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
    if (e >= rows * nci) return;
    const int64_t row = e / nci;  // (rhs, side, tile)
    const int c = static_cast<int>(e - row * nci);
    const int64_t plane = rows * nci;
    cx<T> a = ld<T>(Bp[e]);
#pragma unroll 4
    for (int cz = 1; cz < nchunk; ++cz) a = a + ld<T>(Bp[cz * plane + e]);
    B[row * nc + c] = st(a);
    return;
  }
  const int per = (ndir + 255) / 256;  // blocks per row
  const int64_t b = blockIdx.x - nsum;
  const int64_t row = b / per;  // (rhs, side, tile)
  const int i = static_cast<int>(b - row * per) * 256 + threadIdx.x;
  const int t = static_cast<int>(row % nT), rs = static_cast<int>(row / nT), s = rs & 1;
  if (i >= ndir) return;
  sigma += static_cast<int64_t>(rs >> 1) * 2 * ns;
  const int q = dir[2 * i], c = dir[2 * i + 1];
  const double xT = txy[t].x, yT = txy[t].y;
  const double yy = s == 0 ? yT : -(yT + d);
  const double lr = lam[q].x, li = lam[q].y, gr = g2[q].x, gi = g2[q].y;
  const cx<T> v = cvt<T>(ld<double>(cq[q]) * ld<double>(sigma[s * ns + q])) *
                  cexpT<T>(-li * xT + gr * yy, lr * xT + gi * yy);
  B[row * nc + c] = st(v);
}

inline int cdv(int64_t a, int64_t b) { return static_cast<int>((a + b - 1) / b); }

// S2L, step 2 on the matrix cores: alpha_l[n] = sum_c e_l(c) Z_n(c) with
// e_l(c) = e^{i lam_c dx_l + sg g2_c dy_l} B[T(l)][c] is a GEMM with M =
// particle, N = order, K = (side, coarse node).  Each 16x16x4 MFMA takes 16
// particles and four coarse nodes: lane i forms e for (particle i % 16, node
// i / 16) — one FP64 exponential per (particle, node), as before — and loads
// Z_n(c) for (node i / 16, order i % 16) as the B operand.  Complex products in
// three real MFMAs (Gauss).  One wave per 16 particles, kSiAlphaWaves waves per
// block; blockIdx.y takes a chunk of the (side, coarse node) pairs and writes
// its own partial slot.
constexpr int kSiAlphaWaves = 4;

// The orders past the last full tile are summed on the vector units where that
// is cheaper (OrderSplit: the 33rd order of p = 16 took a tile of its own), and
// the operands of the next step are in flight (5003 particles, FP32: 165 us,
// now 112; 300 particles, FP64, p = 8, one wave per SIMD: 25 us, now 16).
template <typename T, int p>
__global__ __launch_bounds__(64 * kSiAlphaWaves) void k_si_alpha_mfma(
    const cv_t<T> *__restrict__ B, const double2 *__restrict__ xy, const int *__restrict__ ptile,
    const double2 *__restrict__ txy, const double2 *__restrict__ lamc, const double2 *__restrict__ gc,
    const cv_t<T> *__restrict__ Zc, int n, int nT, int nc, int chunk_len, cv_t<T> *__restrict__ part,
    int64_t pstride) {
  constexpr int P = 2 * p + 1;
  constexpr int NT = OrderSplit<P>::NT, NV = OrderSplit<P>::NV;
  typedef typename mfma4<T>::v4 v4;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const int ch = blockIdx.y, rr = blockIdx.z;
  const int k0 = ch * chunk_len, k1 = min(2 * nc, k0 + chunk_len);
  const int lw = (blockIdx.x * kSiAlphaWaves + w) * 16;  // first particle of this wave
  if (lw >= n) return;                                    // the whole wave (no barriers below)
  const int l = lw + r;                                   // this lane's particle (A row)
  const bool valid = l < n;
  const int lc = valid ? l : 0;
  const int t = ptile[lc];
  const double dx = xy[lc].x - txy[t].x, dy = xy[lc].y - txy[t].y;
  const cv_t<T> *Bt = B + (2 * static_cast<int64_t>(rr) * nT + t) * nc;
  const int64_t bside = static_cast<int64_t>(nT) * nc;
  v4 acc[NT > 0 ? NT : 1][3];
  cx<T> vr[NV > 0 ? NV : 1];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int k = 0; k < 3; ++k) acc[nt][k] = v4{0, 0, 0, 0};
#pragma unroll
  for (int v = 0; v < NV; ++v) vr[v] = mk<T>(0, 0);
  struct Ops {
    double2 lm, gm;
    cv_t<T> b, z[NT > 0 ? NT : 1], zv[NV > 0 ? NV : 1];
  };
  auto fetch = [&](int kk, Ops &o) {  // loads clamped into range, zeros selected past the chunk
    const int k = min(kk + g, k1 - 1);
    const int s = k >= nc ? 1 : 0, c = k - s * nc;
    o.lm = lamc[c];
    o.gm = gc[c];
    o.b = Bt[s * bside + c];
    const cv_t<T> *z = Zc + (static_cast<int64_t>(s) * nc + c) * P;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) o.z[nt] = z[min(nt * 16 + r, P - 1)];
#pragma unroll
    for (int v = 0; v < NV; ++v) o.zv[v] = z[16 * NT + v];
  };
  Ops nx;
  if (k0 < k1) fetch(k0, nx);
  for (int kk = k0; kk < k1; kk += 4) {
    const Ops cu = nx;
    if (kk + 4 < k1) fetch(kk + 4, nx);
    const int k = kk + g;  // this lane's coarse node (K index)
    // e^{i lam_c dx + sg g2_c dy} B[T][c]
    const double sy = k < nc ? dy : -dy;
    const cx<T> e = cexpT<T>(-cu.lm.y * dx + cu.gm.x * sy, cu.lm.x * dx + cu.gm.y * sy) * ld<T>(cu.b);
    const bool kv = k < k1 && valid;
    const cx<T> a = kv ? e : mk<T>(0, 0);
    const T as = a.re + a.im;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const bool ov = k < k1 && nt * 16 + r < P;  // padded tile (long remainders only)
      const T zr = ov ? cu.z[nt].x : T(0), zi = ov ? cu.z[nt].y : T(0);
      acc[nt][0] = mfma4<T>::mac(a.re, zr, acc[nt][0]);
      acc[nt][1] = mfma4<T>::mac(a.im, zi, acc[nt][1]);
      acc[nt][2] = mfma4<T>::mac(as, zr + zi, acc[nt][2]);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) cmac(vr[v], a, ld<T>(cu.zv[v]));
  }
  // result register j of lane i: particle lw + row(i, j), order nt * 16 + i % 16
  cv_t<T> *out = part + rr * pstride + static_cast<int64_t>(ch) * n * P;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int o = nt * 16 + r;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int pl = lw + mfma4<T>::row(lane, j);
      if (pl < n && o < P) {
        const T p1 = acc[nt][0][j], p2 = acc[nt][1][j], p3 = acc[nt][2][j];
        out[static_cast<int64_t>(pl) * P + o] = st(mk<T>(p1 - p2, p3 - p1 - p2));
      }
    }
  }
#pragma unroll
  for (int v = 0; v < NV; ++v) {  // over the four nodes of a step
    vr[v].re += __shfl_xor(vr[v].re, 16);
    vr[v].im += __shfl_xor(vr[v].im, 16);
    vr[v].re += __shfl_xor(vr[v].re, 32);
    vr[v].im += __shfl_xor(vr[v].im, 32);
    if (g == 0 && valid) out[static_cast<int64_t>(l) * P + 16 * NT + v] = st(vr[v]);
  }
}

// M2S, step 1 (FP32): one lane per (tile, coarse node), blockIdx.z = 2 rhs + side.
// (5003 particles, 570 tiles, p = 16: 139 us.  The matrix-core form below takes
// 175 there: tiles of about 9 particles leave 7 of its 16 rows empty.  With the
// weights held in registers over a run of tiles, 93 instead of 48 registers and
// half the waves, the scalar loads of the particles show: 183.)
template <int p>
__global__ __launch_bounds__(256) void k_si_tileG(const float2 *__restrict__ beta, const double2 *__restrict__ xy,
                                                  const int *__restrict__ perm, const int *__restrict__ tstart,
                                                  const double2 *__restrict__ txy, const double2 *__restrict__ lamc,
                                                  const double2 *__restrict__ gc, const float2 *__restrict__ Wc,
                                                  int n, int nT, int nc, float2 *__restrict__ G) {
  constexpr int P = 2 * p + 1;
  const int c = blockIdx.x * 256 + threadIdx.x;
  const int t = blockIdx.y;
  const int s = blockIdx.z & 1, r = blockIdx.z >> 1;
  if (c >= nc) return;
  beta += static_cast<int64_t>(r) * n * P;
  const double lr = lamc[c].x, li = lamc[c].y, gr = gc[c].x, gi = gc[c].y;
  const float2 *W = Wc + (static_cast<int64_t>(s) * nc + c) * P;
  cx<float> w[P];
#pragma unroll
  for (int j = 0; j < P; ++j) w[j] = ld<float>(W[j]);
  const double sg = s == 0 ? 1.0 : -1.0;
  const double xT = txy[t].x, yT = txy[t].y;
  cx<float> acc = mk<float>(0, 0);
  for (int k = tstart[t]; k < tstart[t + 1]; ++k) {
    const int m = perm[k];
    const double dx = xy[m].x - xT, dy = xy[m].y - yT;
    // e^{-i lam dx + sg g2 dy}
    const cx<float> e = cexpT<float>(li * dx + sg * gr * dy, -lr * dx + sg * gi * dy);
    const float2 *b = beta + static_cast<int64_t>(m) * P;
    cx<float> bw = mk<float>(0, 0);
#pragma unroll
    for (int j = 0; j < P; ++j) cmac(bw, ld<float>(b[j]), w[j]);
    cmac(acc, e, bw);
  }
  G[((static_cast<int64_t>(r) * 2 + s) * nT + t) * nc + c] = st(acc);
}

// M2S, step 1 in FP64 on the matrix cores: per tile, D[m][c] = sum_n beta_m[n] W_n(c)
// is a GEMM with M = the tile's particles (16 at a time), N = coarse nodes, K =
// orders; then G[T][c] = sum_m e_m(c) D[m][c] with the local factor
// e_m(c) = e^{-i lam_c dx_m + sg g2_c dy_m}, one exponential per (particle,
// node), summed over the lane's rows and across the four row groups.  One wave
// per 16 coarse nodes, kSiAlphaWaves waves per block; a wave keeps its nodes'
// weights in registers and takes the tiles of blockIdx.y's run one after
// another.  Result register q holds the particles 4 q .. 4 q + 3 of the step:
// registers past the tile's last particle take no exponential.
// grid: (node blocks, runs of tiles, 2 rhs + side).
template <int p>
__global__ __launch_bounds__(64 * kSiAlphaWaves) void k_si_tileG_mfma(
    const double2 *__restrict__ beta, const double2 *__restrict__ xy, const int *__restrict__ perm,
    const int *__restrict__ tstart, const double2 *__restrict__ txy, const double2 *__restrict__ lamc,
    const double2 *__restrict__ gc, const double2 *__restrict__ Wc, int n, int nT, int nc, int run,
    double2 *__restrict__ G) {
  constexpr int P = 2 * p + 1;
  constexpr int KS = (P + 3) / 4;
  typedef double T;
  typedef mfma4<T>::v4 v4;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const int s = blockIdx.z & 1, rr = blockIdx.z >> 1;
  const int c0 = (blockIdx.x * kSiAlphaWaves + w) * 16;
  if (c0 >= nc) return;  // the whole wave (no barriers below)
  const int c = c0 + r;  // this lane's coarse node (B column, output)
  const bool cv = c < nc;
  const int cc = cv ? c : nc - 1;
  beta += static_cast<int64_t>(rr) * n * P;
  const double2 *W = Wc + (static_cast<int64_t>(s) * nc + cc) * P;
  cx<T> z[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const int j = 4 * ks + g;  // order (K index) of this lane
    z[ks] = j < P ? ld<T>(W[j]) : mk<T>(0, 0);
  }
  const double sg = s == 0 ? 1.0 : -1.0;
  const double lr = lamc[cc].x, li = lamc[cc].y, gr = sg * gc[cc].x, gi = sg * gc[cc].y;
  const int t1 = min(nT, (static_cast<int>(blockIdx.y) + 1) * run);
  for (int t = blockIdx.y * run; t < t1; ++t) {
    const double xT = txy[t].x, yT = txy[t].y;
    const int m0 = tstart[t], m1 = tstart[t + 1];
    cx<double> acc = mk(0.0, 0.0);
    for (int mb = m0; mb < m1; mb += 16) {
      const int ma = mb + r < m1 ? perm[mb + r] : -1;
      const double2 *b = beta + static_cast<int64_t>(ma < 0 ? 0 : ma) * P;
      double2 av[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) av[ks] = b[min(4 * ks + g, P - 1)];  // its weight past P is zero
      double px[4], py[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = perm[min(mb + 4 * q + g, m1 - 1)];
        px[q] = xy[m].x - xT;
        py[q] = xy[m].y - yT;
      }
      v4 d0 = v4{0, 0, 0, 0}, d1 = v4{0, 0, 0, 0}, d2 = v4{0, 0, 0, 0};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bool ov = ma >= 0 && 4 * ks + g < P;
        const cx<T> a = ov ? ld<T>(av[ks]) : mk<T>(0, 0);
        d0 = mfma4<T>::mac(a.re, z[ks].re, d0);
        d1 = mfma4<T>::mac(a.im, z[ks].im, d1);
        d2 = mfma4<T>::mac(a.re + a.im, z[ks].re + z[ks].im, d2);
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        if (mb + 4 * q + g < m1) {
          const cx<T> e = cexpT<T>(li * px[q] + gr * py[q], -lr * px[q] + gi * py[q]);
          const double p1 = d0[q], p2 = d1[q], p3 = d2[q];
          acc = acc + e * mk(p1 - p2, p3 - p1 - p2);
        }
      }
    }
    acc.re += __shfl_xor(acc.re, 16);
    acc.im += __shfl_xor(acc.im, 16);
    acc.re += __shfl_xor(acc.re, 32);
    acc.im += __shfl_xor(acc.im, 32);
    if (g == 0 && cv) G[((static_cast<int64_t>(rr) * 2 + s) * nT + t) * nc + c] = st(acc);
  }
}

// S2L, step 1 for the Chebyshev intervals on the matrix cores:
// B[T][k] = sum_q V_T(q) L[q][k] with V_T(q) = c_q sigma(q) e^{i lam_q x_T + sg g2_q y_T}
// is a GEMM with M = tile, N = interpolation column k (24, two 16-column
// tiles), K = the interval's fine nodes.  A wave takes 16 RB slots of trow as
// RB row blocks: lane i owns slots tw + RB (i % 16) + b, b < RB, neighbours in
// one row of tiles (rows start at multiples of four slots), and forms their V
// for node i / 16 of the step as the A operand of row block b: one exponential
// for the first, then one complex multiply by e^{i lam w} (modulus ~1, table
// Fx) per tile.  L[q][k] for (node i / 16, column i % 16) is the B operand,
// shared by the row blocks; complex A times real B in two real MFMAs; the next
// step's node values are in flight.  Blocks are single waves: blocks of four
// had waves without tiles, which left whole SIMDs idle.  Rows that did not start
// at a multiple of four made most steps take an exponential for two or three
// of the row blocks (all three: 5003 particles, 570 tiles, FP32: 157 us -> 101;
// 300 particles, 36 tiles, FP64: 47 -> 25).
// grid: (interval, waves of 16 RB slots, chunk
// of the interval's nodes + nchunk * (2 rhs + side)); chunk cz writes its own
// partial slot Bp[cz][rhs, side][t][k], k over the intervals' coarse nodes
// (which come first in the coarse-node order), summed in order by
// k_si_coarseB_fin.
template <typename T> constexpr int coarse_rb() { return sizeof(T) == 4 ? 4 : 2; }
template <typename T, bool SPARSE>
__global__ __launch_bounds__(64) void k_si_coarseB_mfma(
    const double2 *__restrict__ sigma, const double2 *__restrict__ cq, const double2 *__restrict__ lam,
    const double2 *__restrict__ g2, const double2 *__restrict__ Fx, const double2 *__restrict__ txy,
    const int2 *__restrict__ trow, const int *__restrict__ ivl, const int *__restrict__ fperm,
    const double *__restrict__ Lw, int ns, int nT, int nrow, int nci, int nchunk, double d,
    cv_t<T> *__restrict__ Bp) {
  constexpr int RB = coarse_rb<T>();
  typedef typename mfma4<T>::v4 v4;
  const int lane = threadIdx.x;
  const int r = lane & 15, g = lane >> 4;
  const int iv = blockIdx.x;
  const int tw = blockIdx.y * 16 * RB;  // first slot of this wave
  const int cz = blockIdx.z % nchunk, rs = blockIdx.z / nchunk;
  const int s = rs & 1, rr = rs >> 1;
  const int f0 = ivl[4 * iv], nf = ivl[4 * iv + 1], c0 = ivl[4 * iv + 2];
  const int cl = (nf + nchunk - 1) / nchunk;  // 32-bit: a 64-bit division costs more than a step
  const int i0 = min(cz * cl, nf), i1 = min(i0 + cl, nf);
  sigma += static_cast<int64_t>(rr) * 2 * ns;
  // this lane's tiles (-1: none), the centre of the first, and the steps between them
  int tb[RB], kst[RB];
#pragma unroll
  for (int b = 0; b < RB; ++b) {
    const int o = tw + RB * r + b;
    const int2 e = o < nrow ? trow[o] : make_int2(-1, 0);
    tb[b] = e.x;
    kst[b] = e.y;
  }
  double xb[SPARSE ? RB : 1], yb[SPARSE ? RB : 1];  // of the others in a SPARSE list as well
#pragma unroll
  for (int b = 0; b < (SPARSE ? RB : 1); ++b) {
    const double2 tc = txy[tb[b] >= 0 ? tb[b] : 0];
    xb[b] = tc.x;
    yb[b] = s == 0 ? tc.y : -(tc.y + d);
  }
  v4 acc[RB][2][2];
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) acc[b][nt][0] = acc[b][nt][1] = v4{0, 0, 0, 0};
  struct Ops {
    double2 lm, gm, cw, sw, fx;
    double l[2];
  };
  auto node = [&](int i) { return fperm[f0 + (i + g < i1 ? i + g : i0)]; };
  auto fetch = [&](int q, Ops &o) {
    o.lm = lam[q];
    o.gm = g2[q];
    o.cw = cq[q];
    o.sw = sigma[s * ns + q];
    o.fx = Fx[q];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) o.l[nt] = Lw[static_cast<int64_t>(q) * kSommNc + min(nt * 16 + r, kSommNc - 1)];
  };
  Ops nx;
  int qn = 0;
  if (i0 < i1) {
    fetch(node(i0), nx);
    qn = node(i0 + 4);
  }
  for (int i = i0; i < i1; i += 4) {
    const Ops cu = nx;
    if (i + 4 < i1) {
      fetch(qn, nx);
      qn = node(i + 8);
    }
    const bool kv = i + g < i1;  // this lane's node (K index)
    const cx<T> u = kv ? cvt<T>(ld<double>(cu.cw) * ld<double>(cu.sw)) : mk<T>(0, 0);
    const cx<T> fx = cvt<T>(ld<double>(cu.fx));
    T lq[2];
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) lq[nt] = (kv && nt * 16 + r < kSommNc) ? static_cast<T>(cu.l[nt]) : T(0);
    const auto wave = [&](int b) {
      return cexpT<T>(-cu.lm.y * xb[b] + cu.gm.x * yb[b], cu.lm.x * xb[b] + cu.gm.y * yb[b]);
    };
    cx<T> E = wave(0);
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      if (b > 0) {
        if constexpr (SPARSE) {
          E = wave(b);
        } else {
          E = E * fx;
          for (int v = 1; v < kst[b]; ++v) E = E * fx;
        }
      }
      const cx<T> v = kv && tb[b] >= 0 ? u * E : mk<T>(0, 0);
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) {
        acc[b][nt][0] = mfma4<T>::mac(v.re, lq[nt], acc[b][nt][0]);
        acc[b][nt][1] = mfma4<T>::mac(v.im, lq[nt], acc[b][nt][1]);
      }
    }
  }
  // result register j of lane i in row block b: tile trow[tw + RB row(i, j) + b], column nt * 16 + i % 16
  cv_t<T> *o = Bp + (static_cast<int64_t>(cz) * (gridDim.z / nchunk) + rs) * nT * static_cast<int64_t>(nci) + c0;
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      const int k = nt * 16 + r;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int os = tw + RB * mfma4<T>::row(lane, j) + b;
        const int t = os < nrow ? trow[os].x : -1;
        if (t >= 0 && k < kSommNc)
          o[static_cast<int64_t>(t) * nci + k] = st(mk<T>(acc[b][nt][0][j], acc[b][nt][1][j]));
      }
    }
}

template <typename T>
int ensure_G(mpsl_ctx *ctx, int nrhs) {
  const SommPlan &pl = ctx->somm;
  return dev_alloc(ctx, ctx->somm.G, 2ull * nrhs * pl.nT * pl.nc * sizeof(cv_t<T>));
}

template <typename T>
int m2s_interp_t(mpsl_ctx *ctx, const void *beta, void *spec, int nrhs) {
  SommPlan &pl = ctx->somm;
  int rc = ensure_G<T>(ctx, nrhs);
  if (rc) return rc;
  const bool f64 = std::is_same<T, double>::value;
  auto *G = static_cast<cv_t<T> *>(pl.G.p);
  const int n = static_cast<int>(ctx->n);
  // FP64: runs of tiles so that the launch has about 2048 blocks (a longer run
  // reads the weights less often)
  const int nbc = cdv(pl.nc, f64 ? 16 * kSiAlphaWaves : 256);
  const int run = f64 ? cdv(pl.nT, std::min<int64_t>(pl.nT, cdv(2048, 2ll * nrhs * nbc))) : 1;
  const dim3 g1(nbc, cdv(pl.nT, run), 2 * nrhs);
  const auto *xy = static_cast<const double2 *>(ctx->gt.xy.p);
  const auto *perm = static_cast<const int *>(pl.perm.p), *tstart = static_cast<const int *>(pl.tstart.p);
  const auto *lamc = static_cast<const double2 *>(pl.lamc.p), *gc = static_cast<const double2 *>(pl.gc.p);
  const auto *txy = static_cast<const double2 *>(pl.txy.p);
  switch (ctx->p) {
#define X(PP)                                                                                                      \
  case PP:                                                                                                         \
    if (f64)                                                                                                       \
      hipLaunchKernelGGL(k_si_tileG_mfma<PP>, g1, dim3(64 * kSiAlphaWaves), 0, ctx->stream,                       \
                         static_cast<const double2 *>(beta), xy, perm, tstart, txy, lamc, gc,                       \
                         static_cast<const double2 *>(pl.Wc64.p), n, pl.nT, pl.nc, run,                             \
                         static_cast<double2 *>(pl.G.p));                                                           \
    else                                                                                                           \
      hipLaunchKernelGGL(k_si_tileG<PP>, g1, dim3(256), 0, ctx->stream, static_cast<const float2 *>(beta), xy,     \
                         perm, tstart, txy, lamc, gc, static_cast<const float2 *>(pl.Wc32.p), n, pl.nT, pl.nc,      \
                         static_cast<float2 *>(pl.G.p));                                                            \
    break;
    SOMM_P_CASES(X)
#undef X
    default: return set_err(ctx, MPSL_EUNSUPPORTED, "expansion order outside 1..20");
  }
  const auto *lam = static_cast<const double2 *>(ctx->ct.lam.p);
  const auto *g2 = static_cast<const double2 *>(ctx->ct.gw.p) + ctx->ns;  // g2 stored after g1
  const int nfine = pl.nfb + cdv(pl.ndir, kSiDirNodes);
  if (nfine > 0)
    hipLaunchKernelGGL((pl.sparse ? k_si_fine<T, true> : k_si_fine<T, false>), dim3(nfine, 2 * nrhs),
                       dim3(64 * kSiFineSplit), 0, ctx->stream, G, lam, g2, txy,
                       static_cast<const int2 *>(pl.trow.p), static_cast<const double2 *>(pl.tgrp.p),
                       static_cast<const int *>(pl.ivl.p), static_cast<const int *>(pl.fperm.p),
                       static_cast<const int *>(pl.fblk.p),
                       static_cast<const double *>(pl.Lw.p), static_cast<const int *>(pl.dir.p), pl.nfb, pl.ndir,
                       ctx->ns, pl.nT, pl.nrow, pl.nc, ctx->d, pl.tile_w, static_cast<double2 *>(spec));
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_err(ctx, MPSL_EHIP, std::string("interpolated M2S: ") + hipGetErrorString(e));
  return MPSL_OK;
}

template <typename T>
int s2l_interp_t(mpsl_ctx *ctx, void *part, int chunks, int nrhs, int64_t pstride) {
  SommPlan &pl = ctx->somm;
  if (!pl.sigma) return set_err(ctx, MPSL_ESTATE, "interpolated S2L without densities");
  int rc = ensure_G<T>(ctx, nrhs);
  if (rc) return rc;
  const bool f64 = std::is_same<T, double>::value;
  const auto *Zc = static_cast<const cv_t<T> *>(f64 ? pl.Zc64.p : pl.Zc32.p);
  auto *B = static_cast<cv_t<T> *>(pl.G.p);
  const auto *sig = static_cast<const double2 *>(pl.sigma);
  const auto *cq = static_cast<const double2 *>(ctx->ct.cq.p);
  const auto *lam = static_cast<const double2 *>(ctx->ct.lam.p);
  const auto *g2 = static_cast<const double2 *>(ctx->ct.gw.p) + ctx->ns;
  const auto *txy = static_cast<const double2 *>(pl.txy.p);
  const int nci = kSommNc * pl.nint;
  const int64_t rows = 2ll * nrhs * pl.nT;
  int nchunk = 1, nsum = 0;
  if (pl.nint > 0) {
    // node chunks so that the waves fill the chip once (7 per SIMD in FP32), with no
    // more partials than 2048 blocks of four waves over the tiles would write
    const int tb = cdv(pl.nrow, 16 * coarse_rb<T>());
    const int64_t per = static_cast<int64_t>(pl.nint) * 2 * nrhs;
    const int most = std::min(16, cdv(2048, per * cdv(pl.nT, 64 * coarse_rb<T>())));
    nchunk = std::max(1, std::min(most, static_cast<int>(28 * ctx->n_cu / (per * tb))));
    if ((rc = dev_alloc(ctx, pl.Bp, static_cast<size_t>(nchunk) * rows * nci * sizeof(cv_t<T>)))) return rc;
    nsum = cdv(rows * nci, 256);
    hipLaunchKernelGGL((pl.sparse ? k_si_coarseB_mfma<T, true> : k_si_coarseB_mfma<T, false>),
                       dim3(pl.nint, tb, nchunk * 2 * nrhs), dim3(64), 0, ctx->stream, sig, cq, lam, g2, static_cast<const double2 *>(pl.Fx.p), txy,
                       static_cast<const int2 *>(pl.trow.p), static_cast<const int *>(pl.ivl.p),
                       static_cast<const int *>(pl.fperm.p), static_cast<const double *>(pl.Lw.p), ctx->ns, pl.nT,
                       pl.nrow, nci, nchunk, ctx->d, static_cast<cv_t<T> *>(pl.Bp.p));
  }
  const int64_t nfin = nsum + rows * cdv(pl.ndir, 256);
  if (nfin > 0)
    hipLaunchKernelGGL(k_si_coarseB_fin<T>, dim3(static_cast<unsigned>(nfin)), dim3(256), 0, ctx->stream,
                       static_cast<const cv_t<T> *>(pl.Bp.p), nchunk, rows, nci, nsum, sig, cq, lam, g2, txy,
                       static_cast<const int *>(pl.dir.p), pl.ndir, ctx->ns, pl.nT, pl.nc, ctx->d, B);
  const int n = static_cast<int>(ctx->n);
  const int chunk_len = cdv(2 * static_cast<int64_t>(pl.nc), chunks);
  const dim3 g2d(cdv(n, 16 * kSiAlphaWaves), chunks, nrhs);
  auto *o = static_cast<cv_t<T> *>(part);
  switch (ctx->p) {
#define X(PP)                                                                                                       \
  case PP:                                                                                                          \
    hipLaunchKernelGGL((k_si_alpha_mfma<T, PP>), g2d, dim3(64 * kSiAlphaWaves), 0, ctx->stream, B,                 \
                       static_cast<const double2 *>(ctx->gt.xy.p), static_cast<const int *>(pl.ptile.p), txy,       \
                       static_cast<const double2 *>(pl.lamc.p), static_cast<const double2 *>(pl.gc.p), Zc, n,       \
                       pl.nT, pl.nc, chunk_len, o, pstride);                                                         \
    break;
    SOMM_P_CASES(X)
#undef X
    default: return set_err(ctx, MPSL_EUNSUPPORTED, "expansion order outside 1..20");
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return set_err(ctx, MPSL_EHIP, std::string("interpolated S2L: ") + hipGetErrorString(e));
  return MPSL_OK;
}

}  // namespace

int launch_m2s_interp(mpsl_ctx *ctx, int prec, const void *beta, void *spec, int nrhs) {
  return prec == MPSL_FP64 ? m2s_interp_t<double>(ctx, beta, spec, nrhs) : m2s_interp_t<float>(ctx, beta, spec, nrhs);
}

int launch_s2l_interp(mpsl_ctx *ctx, int prec, void *part, int chunks, int nrhs, int64_t pstride) {
  return prec == MPSL_FP64 ? s2l_interp_t<double>(ctx, part, chunks, nrhs, pstride)
                           : s2l_interp_t<float>(ctx, part, chunks, nrhs, pstride);
}

void somm_free(mpsl_ctx *ctx) {
  SommPlan &pl = ctx->somm;
  DBuf *b[] = {&pl.perm, &pl.tstart, &pl.txy, &pl.ptile, &pl.lamc, &pl.gc, &pl.Wc64, &pl.Wc32, &pl.Zc64,
               &pl.Zc32, &pl.Lw, &pl.ivl, &pl.fperm, &pl.dir, &pl.G, &pl.Bp, &pl.fblk,
               &pl.trow, &pl.tgrp, &pl.Fx};
  for (DBuf *x : b) dev_free(*x);
  pl.active = false;
  pl.sigma = nullptr;
}

// Tiles, intervals, coarse nodes and interpolation weights (host, FP64).
int somm_build(mpsl_ctx *ctx) {
  somm_free(ctx);
  SommPlan &pl = ctx->somm;
  if (ctx->somm_method != MPSL_SOMM_INTERP) return MPSL_OK;
  const int64_t n = ctx->n;
  const int ns = ctx->ns, p = ctx->p, P = 2 * p + 1;
  pl.tile_w = kTileW;
  pl.L_I = kIntervalL;
  pl.d_dir = kDirect;
  // tiles of the particle bounding box
  double x0 = 1e300, y0 = 1e300;
  for (int64_t m = 0; m < n; ++m) {
    x0 = std::min(x0, ctx->xy[2 * m]);
    y0 = std::min(y0, ctx->xy[2 * m + 1]);
  }
  std::map<std::pair<int64_t, int64_t>, int> tiles;
  std::vector<std::pair<int64_t, int64_t>> key(n);
  for (int64_t m = 0; m < n; ++m) {
    key[m] = {static_cast<int64_t>(std::floor((ctx->xy[2 * m] - x0) / kTileW)),
              static_cast<int64_t>(std::floor((ctx->xy[2 * m + 1] - y0) / kTileH))};
    tiles.emplace(key[m], 0);
  }
  int id = 0;
  std::vector<double2> txy;
  for (auto &kv : tiles) {
    kv.second = id++;
    txy.push_back(make_double2(x0 + (kv.first.first + 0.5) * kTileW, y0 + (kv.first.second + 0.5) * kTileH));
  }
  pl.nT = id;
  // slots: tiles in row-major order as (tile, tile widths from the slot before),
  // in groups of four that start anew (padded with (-1, 0)) where a row ends or
  // a gap is wider than four tiles
  std::vector<int2> trow;
  {
    std::vector<std::pair<std::pair<int64_t, int64_t>, int>> byrow;
    for (const auto &kv : tiles) byrow.push_back({{kv.first.second, kv.first.first}, kv.second});
    std::sort(byrow.begin(), byrow.end());
    for (size_t i = 0; i < byrow.size(); ++i) {
      int64_t step = 0;
      if (i > 0 && byrow[i].first.first == byrow[i - 1].first.first) step = byrow[i].first.second - byrow[i - 1].first.second;
      if (step < 1 || step > 4) {
        step = 0;
        while (trow.size() % 4) trow.push_back(make_int2(-1, 0));
      }
      trow.push_back(make_int2(byrow[i].second, static_cast<int>(step)));
    }
    while (trow.size() % 4) trow.push_back(make_int2(-1, 0));
  }
  // tiles that stand apart (more than two padding slots per tile, and a step of
  // the transforms full of them) stay without the padding and take an exponential
  // each (matvec, 1000 tiles five widths apart, 8192 nodes, p = 8, FP64 1281 us with
  // the padding and 809 without, FP32 564 and 365)
  pl.sparse = tiles.size() >= 16 && trow.size() > 3 * tiles.size();
  if (pl.sparse) {
    trow.clear();
    for (const auto &kv : tiles) trow.push_back(make_int2(kv.second, 0));
    while (trow.size() % 4) trow.push_back(make_int2(-1, 0));
  }
  pl.nrow = static_cast<int>(trow.size());
  std::vector<double2> tgrp;
  for (size_t i = 0; i < trow.size(); i += 4) tgrp.push_back(txy[trow[i].x]);
  std::vector<int> ptile(n), tstart(pl.nT + 1, 0), perm(n);
  for (int64_t m = 0; m < n; ++m) {
    ptile[m] = tiles[key[m]];
    ++tstart[ptile[m] + 1];
  }
  for (int t = 0; t < pl.nT; ++t) tstart[t + 1] += tstart[t];
  {
    std::vector<int> fill(tstart.begin(), tstart.end() - 1);
    for (int64_t m = 0; m < n; ++m) perm[fill[ptile[m]]++] = static_cast<int>(m);
  }
  // contour nodes: direct near +-k2 and on the vertical segment, intervals elsewhere
  const double k2r = ctx->k2.real();
  std::vector<char> direct(ns, 0);
  for (int q = 0; q < ns; ++q) {
    const double tr = ctx->lam[q].real();
    direct[q] = (std::fabs(tr) < 1e-14) || (std::fabs(std::fabs(tr) - k2r) < kDirect);
  }
  std::vector<std::vector<int>> groups;
  for (int q = 0; q < ns;) {
    if (direct[q]) {
      ++q;
      continue;
    }
    const double a = ctx->lam[q].real(), im = ctx->lam[q].imag();
    std::vector<int> g{q};
    int e = q + 1;
    while (e < ns && !direct[e] && ctx->lam[e].imag() == im && (ctx->lam[e].real() > 0) == (a > 0) &&
           std::fabs(ctx->lam[e].real() - a) <= kIntervalL)
      g.push_back(e++);
    if (static_cast<int>(g.size()) <= kSommNc)
      for (int x : g) direct[x] = 1;
    else
      groups.push_back(g);
    q = e;
  }
  // coarse nodes: kSommNc Chebyshev nodes per interval, then one per direct node
  std::vector<zc> lamc;
  std::vector<int> ivl, fperm, dir;
  std::vector<double> Lw(static_cast<size_t>(ns) * kSommNc, 0.0);
  double xs[kSommNc], bw[kSommNc];
  for (int j = 0; j < kSommNc; ++j) {
    xs[j] = std::cos((2 * j + 1) * M_PI / (2.0 * kSommNc));
    bw[j] = ((j & 1) ? -1.0 : 1.0) * std::sin((2 * j + 1) * M_PI / (2.0 * kSommNc));
  }
  for (const auto &g : groups) {
    double a = 1e300, c = -1e300;
    for (int q : g) {
      a = std::min(a, ctx->lam[q].real());
      c = std::max(c, ctx->lam[q].real());
    }
    const double im = ctx->lam[g[0]].imag();
    const int c0 = static_cast<int>(lamc.size());
    double tc[kSommNc];
    for (int j = 0; j < kSommNc; ++j) {
      tc[j] = 0.5 * (a + c) + 0.5 * (c - a) * xs[j];
      lamc.emplace_back(tc[j], im);
    }
    ivl.push_back(static_cast<int>(fperm.size()));
    ivl.push_back(static_cast<int>(g.size()));
    ivl.push_back(c0);
    ivl.push_back(0);
    for (int q : g) {
      fperm.push_back(q);
      const double t = ctx->lam[q].real();
      double *L = &Lw[static_cast<size_t>(q) * kSommNc];
      int hit = -1;
      double sum = 0.0;
      for (int j = 0; j < kSommNc; ++j) {
        const double dd = t - tc[j];
        if (dd == 0.0) hit = j;
        L[j] = (dd == 0.0) ? 0.0 : bw[j] / dd;
        sum += L[j];
      }
      if (hit >= 0) {
        for (int j = 0; j < kSommNc; ++j) L[j] = (j == hit) ? 1.0 : 0.0;
      } else {
        for (int j = 0; j < kSommNc; ++j) L[j] /= sum;
      }
    }
  }
  pl.nint = static_cast<int>(groups.size());
  // blocks of the interval-node M2S step: (interval, first node) per run of kSiFineNodes
  std::vector<int> fblk;
  for (int iv = 0; iv < pl.nint; ++iv)
    for (int o = 0; o < ivl[4 * iv + 1]; o += kSiFineNodes) {
      fblk.push_back(iv);
      fblk.push_back(o);
    }
  pl.nfb = static_cast<int>(fblk.size() / 2);
  for (int q = 0; q < ns; ++q)
    if (direct[q]) {
      const int c = static_cast<int>(lamc.size());
      lamc.push_back(ctx->lam[q]);
      Lw[static_cast<size_t>(q) * kSommNc] = 1.0;
      dir.push_back(q);
      dir.push_back(c);
    }
  pl.ndir = static_cast<int>(dir.size() / 2);
  pl.nc = static_cast<int>(lamc.size());
  // coarse-node tables
  std::vector<zc> gc(pl.nc), Wc(2ull * pl.nc * P), Zc(2ull * pl.nc * P);
  for (int c = 0; c < pl.nc; ++c) {
    gc[c] = gamma_branch(lamc[c], ctx->k2);
    order_weights(lamc[c], gc[c], ctx->k2, p, &Wc[static_cast<size_t>(c) * P],
                  &Wc[(static_cast<size_t>(pl.nc) + c) * P], &Zc[static_cast<size_t>(c) * P],
                  &Zc[(static_cast<size_t>(pl.nc) + c) * P]);
  }
  auto upload = [&](DBuf &b, const void *src, size_t bytes) -> int {
    int rc = dev_alloc(ctx, b, bytes > 0 ? bytes : 16);  // an empty table keeps a valid, unused allocation
    if (rc) return rc;
    if (bytes > 0) MPSL_HIP_TRY(ctx, hipMemcpy(b.p, src, bytes, hipMemcpyHostToDevice));
    return MPSL_OK;
  };
  std::vector<float2> Wc32(Wc.size()), Zc32(Zc.size());
  for (size_t i = 0; i < Wc.size(); ++i) {
    Wc32[i] = make_float2(static_cast<float>(Wc[i].real()), static_cast<float>(Wc[i].imag()));
    Zc32[i] = make_float2(static_cast<float>(Zc[i].real()), static_cast<float>(Zc[i].imag()));
  }
  int rc;
  if ((rc = upload(pl.perm, perm.data(), perm.size() * sizeof(int))) ||
      (rc = upload(pl.tstart, tstart.data(), tstart.size() * sizeof(int))) ||
      (rc = upload(pl.txy, txy.data(), txy.size() * sizeof(double2))) ||
      (rc = upload(pl.ptile, ptile.data(), ptile.size() * sizeof(int))) ||
      (rc = upload(pl.lamc, lamc.data(), lamc.size() * sizeof(double2))) ||
      (rc = upload(pl.gc, gc.data(), gc.size() * sizeof(double2))) ||
      (rc = upload(pl.Wc64, Wc.data(), Wc.size() * sizeof(double2))) ||
      (rc = upload(pl.Wc32, Wc32.data(), Wc32.size() * sizeof(float2))) ||
      (rc = upload(pl.Zc64, Zc.data(), Zc.size() * sizeof(double2))) ||
      (rc = upload(pl.Zc32, Zc32.data(), Zc32.size() * sizeof(float2))) ||
      (rc = upload(pl.Lw, Lw.data(), Lw.size() * sizeof(double))) ||
      (rc = upload(pl.ivl, ivl.data(), ivl.size() * sizeof(int))) ||
      (rc = upload(pl.fperm, fperm.data(), fperm.size() * sizeof(int))) ||
      (rc = upload(pl.dir, dir.data(), dir.size() * sizeof(int))) ||
      (rc = upload(pl.fblk, fblk.data(), fblk.size() * sizeof(int))) ||
      (rc = upload(pl.tgrp, tgrp.data(), tgrp.size() * sizeof(double2))) ||
      (rc = upload(pl.trow, trow.data(), trow.size() * sizeof(int2))))
    return rc;

  {  // e^{i lam_q w} per contour node
    std::vector<double2> fx(ns);
    for (int q = 0; q < ns; ++q) {
      const zc v = std::exp(zc(0.0, 1.0) * ctx->lam[q] * kTileW);
      fx[q] = make_double2(v.real(), v.imag());
    }
    if ((rc = upload(pl.Fx, fx.data(), fx.size() * sizeof(double2)))) return rc;
  }
  pl.active = true;
  return MPSL_OK;
}

}  // namespace mpsl

extern "C" int mpsl_get_somm_info(const mpsl_ctx *ctx, int *active, int *tiles, int *intervals, int *coarse_nodes,
                                  int *direct_nodes) {
  if (!ctx) return MPSL_EINVAL;
  if (!ctx->tables_ok) return MPSL_ESTATE;
  const mpsl::SommPlan &pl = ctx->somm;
  if (active) *active = pl.active ? 1 : 0;
  if (tiles) *tiles = pl.active ? pl.nT : 0;
  if (intervals) *intervals = pl.active ? pl.nint : 0;
  if (coarse_nodes) *coarse_nodes = pl.active ? pl.nc : 0;
  if (direct_nodes) *direct_nodes = pl.active ? pl.ndir : 0;
  return MPSL_OK;
}
