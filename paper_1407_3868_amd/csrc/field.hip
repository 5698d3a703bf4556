// Row a7: total field at receivers (eq. (36)), FP64.
//
// u = the layer's plane waves, a sum over the contour nodes, plus the point
// source in the top layer or the particles' multipoles in the particle layer.
//
// Bound by the vector units: per (receiver, particle) the Hankel functions of
// orders 0 .. p and one complex product each, per (receiver, node) two complex
// exponentials.  One lane per receiver alone leaves the chip empty (4096
// receivers are 64 waves, 27.4 ms at 5000 particles, p = 16, 1024 nodes), so
// the particles and the nodes are cut into chunks, a block per (256 receivers,
// chunk), and the partial sums added in a fixed order.
#include <cmath>

#include "kernels.h"

namespace mpsl {

namespace {

inline int cdiv(int64_t a, int64_t b) { return static_cast<int>((a + b - 1) / b); }

constexpr int kFieldThreads = 256;

__device__ inline cx<double> cdivz(cx<double> a, cx<double> b) {
  const double s = 1.0 / (b.re * b.re + b.im * b.im);
  return {(a.re * b.re + a.im * b.im) * s, (a.im * b.re - a.re * b.im) * s};
}

// sqrt(lam^2 - k^2), Re >= 0, and Im <= 0 on Re == 0
__device__ inline cx<double> gamma_dev(cx<double> lam, double k) {
  const cx<double> z = mk(lam.re - k, lam.im) * mk(lam.re + k, lam.im);
  const double r = hypot(z.re, z.im);
  const double s = sqrt(0.5 * (r + fabs(z.re)));
  if (s == 0.0) return {0.0, 0.0};
  const double t = 0.5 * fabs(z.im) / s;
  cx<double> g = z.re >= 0.0 ? mk(s, copysign(t, z.im)) : mk(t, copysign(s, z.im));
  if (g.re == 0.0 && g.im > 0.0) g.im = -g.im;
  return g;
}

__device__ inline cx<double> refl(cx<double> za, cx<double> zb) { return cdivz(za - zb, za + zb); }

// Plane-wave amplitudes of every layer per contour node, from the interface
// conditions outward from the particle layer c (the recursion of layers.hip on
// the device: the host loop over the nodes took longer than the field kernel).
// A[j]: downgoing wave at the top interface of layer j, B[j]: upgoing wave at
// its bottom, both times w / (4 pi gamma_j); gl[j]: gamma of layer j.  stack:
// kappa[L] (weight of du/dy), thickness[L], k[L].  gw: gamma of the top, the
// particle and the bottom layer and the weights, as the tables hold them.
// While the recursions run, A[j] and B[j] of a layer above the particle layer
// hold its generalized transmission and reflection, and B[j] of one below it
// its generalized reflection.
__global__ void k_field_amp(const double2 *__restrict__ lam, const double2 *__restrict__ gw,
                            const double2 *__restrict__ spec, const double2 *__restrict__ sigma,
                            const double *__restrict__ stack, int L, int c, int ns, double xs, double ys,
                            double2 *__restrict__ gl, double2 *__restrict__ A, double2 *__restrict__ B) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= ns) return;
  const double *kap = stack, *thick = stack + L, *kk = stack + 2 * L;
  const cx<double> lm = ld<double>(lam[q]);
  const auto at = [&](int j) { return static_cast<int64_t>(j) * ns + q; };
  for (int j = 0; j < L; ++j) {
    const int t = j == 0 ? 0 : j == c ? 1 : j == L - 1 ? 2 : -1;
    gl[at(j)] = t >= 0 ? gw[at(t)] : st(gamma_dev(lm, kk[j]));
  }
  const auto g = [&](int j) { return ld<double>(gl[at(j)]); };
  const auto e = [&](int j) {
    const cx<double> v = g(j);
    return cexpT<double>(-v.re * thick[j], -v.im * thick[j]);
  };
  {  // above: layer 1 under the top half-space, then one finite layer at a time
    cx<double> ru = refl(kap[1] * g(1), kap[0] * g(0));
    cx<double> tau = cdivz(2.0 * kap[0] * g(1), kap[0] * g(0) + kap[1] * g(1));
    for (int j = 1; j < c; ++j) {
      A[at(j)] = st(tau);
      B[at(j)] = st(ru);
      const cx<double> za = kap[j] * g(j), zb = kap[j + 1] * g(j + 1), ej = e(j);
      const cx<double> r = refl(zb, za), t = cdivz(2.0 * kap[j] * g(j + 1), za + zb);
      const cx<double> rho = ru * ej * ej, den = mk(1.0, 0.0) + r * rho;
      tau = cdivz(t * ej * tau, den);
      ru = cdivz(r + rho, den);
    }
    // below: layer L-2 over the bottom half-space, then upwards
    cx<double> rd = refl(kap[L - 2] * g(L - 2), kap[L - 1] * g(L - 1));
    for (int j = L - 2; j > c; --j) {
      B[at(j)] = st(rd);
      const cx<double> ej = e(j), r = refl(kap[j - 1] * g(j - 1), kap[j] * g(j));
      const cx<double> rho = rd * ej * ej;
      rd = cdivz(r + rho, mk(1.0, 0.0) + r * rho);
    }
  }
  const cx<double> sp = ld<double>(sigma[q]), sm = ld<double>(sigma[ns + q]);
  const cx<double> g0 = g(0), ec = e(c);
  // source amplitude at the top interface (ys: the source's height above it)
  const cx<double> gs = cexpT<double>(lm.im * xs - g0.re * ys, -lm.re * xs - g0.im * ys);
  cx<double> a = ec * sm + ld<double>(spec[q]), b = sp;
  for (int j = c - 1; j >= 1; --j) {
    const cx<double> tau = ld<double>(A[at(j)]), ru = ld<double>(B[at(j)]);
    const cx<double> s = cdivz(g(j), g(j + 1)) * (a + b), dl = (kap[j + 1] / kap[j]) * (b - a);
    const cx<double> Bj = 0.5 * (s - dl);
    a = Bj * e(j);
    b = ru * a + tau * gs;
    A[at(j)] = st(b);
    B[at(j)] = st(Bj);
  }
  A[at(0)] = make_double2(0.0, 0.0);
  B[at(0)] = st(cdivz(g0, g(1)) * (a + b) - gs);
  cx<double> dn = ec * sp + ld<double>(spec[ns + q]), up = sm;
  for (int j = c + 1; j <= L - 2; ++j) {
    const cx<double> rd = ld<double>(B[at(j)]);
    const cx<double> Aj = 0.5 * (cdivz(g(j), g(j - 1)) * (dn + up) + (kap[j - 1] / kap[j]) * (dn - up));
    dn = Aj * e(j);
    up = rd * dn;
    A[at(j)] = st(Aj);
    B[at(j)] = st(up);
  }
  A[at(L - 1)] = st(cdivz(g(L - 1), g(L - 2)) * (dn + up));
  B[at(L - 1)] = make_double2(0.0, 0.0);
  A[at(c)] = st(sp);
  B[at(c)] = st(sm);
  const cx<double> w = (1.0 / (4.0 * M_PI)) * ld<double>(gw[at(3)]);
  for (int j = 0; j < L; ++j) {
    const cx<double> f = cdivz(w, g(j));
    A[at(j)] = st(f * ld<double>(A[at(j)]));
    B[at(j)] = st(f * ld<double>(B[at(j)]));
  }
}

// Coefficients as the particle sum reads them: per particle b_0, then for each
// order q the pair b_q + (-1)^q b_{-q}, b_q - (-1)^q b_{-q}, so that
// e^{iq phi} b_q + (-1)^q e^{-iq phi} b_{-q} takes four multiply-adds.
__global__ void k_field_coef(const double2 *__restrict__ beta, int n, int p, double2 *__restrict__ D) {
  const int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  const int P = 2 * p + 1;
  if (i >= static_cast<int64_t>(n) * P) return;
  const int64_t m = i / P;
  const int s = static_cast<int>(i - m * P), q = (s + 1) / 2;
  const cx<double> b = ld<double>(beta[m * P + p + q]), a = ld<double>(beta[m * P + p - q]);
  if (s == 0) D[i] = st(b);
  else D[i] = st(((q & 1) != 0) == ((s & 1) != 0) ? b - a : b + a);
}

// H_0(z) and H_1(z), z > 0: from z = kFieldAsym on Hankel's expansion (DLMF
// 10.17.5), nine terms in each of P and Q (the first one left out is below
// 1e-16 there) with one reduced phase for both orders; below, where a wave
// has a lane that close to a particle, the library functions.
constexpr double kFieldAsym = 25.0;
__device__ inline void hankel01(double z, double inv, cx<double> &h0, cx<double> &h1) {
  // a_k(nu) = a_{k-1}(nu) (4 nu^2 - (2k - 1)^2) / (8 k)
  struct Coef {
    double v[2][18];
    constexpr Coef() : v() {
      for (int nu = 0; nu < 2; ++nu) {
        v[nu][0] = 1.0;
        for (int k = 1; k < 18; ++k)
          v[nu][k] = v[nu][k - 1] * (4.0 * nu * nu - (2.0 * k - 1.0) * (2.0 * k - 1.0)) / (8.0 * k);
      }
    }
  };
  constexpr Coef a{};
  const double x = -inv * inv;
  double P[2], Q[2];
#pragma unroll
  for (int nu = 0; nu < 2; ++nu) {
    P[nu] = a.v[nu][16];
    Q[nu] = a.v[nu][17];
#pragma unroll
    for (int k = 7; k >= 0; --k) {
      P[nu] = fma(P[nu], x, a.v[nu][2 * k]);
      Q[nu] = fma(Q[nu], x, a.v[nu][2 * k + 1]);
    }
    Q[nu] *= inv;
  }
  // sqrt(2 / (pi z)) e^{i (z - pi / 4)}
  const cx<double> u = cexpT<double>(0.0, z);
  const double s = sqrt(0.3183098861837907 * inv);  // sqrt(1 / (pi z)): sqrt(1/2) of the rotation included
  const cx<double> f = mk(s * (u.re + u.im), s * (u.im - u.re));
  h0 = f * mk(P[0], Q[0]);
  h1 = mk(f.im, -f.re) * mk(P[1], Q[1]);
  if (z < kFieldAsym) {
    h0 = mk(j0(z), y0(z));
    h1 = mk(j1(z), y1(z));
  }
}

// Partial sums: block (256 receivers, chunk); the first pchunks chunks take
// particles, the others contour nodes.  The loop variable is uniform over the
// block, so coefficients and node data come through the scalar cache.  A
// receiver inside an enclosing disk gets a NaN partial.
__global__ __launch_bounds__(kFieldThreads) void k_field_part(
    const double2 *__restrict__ xy, const double2 *__restrict__ D, int n, int p, const double2 *__restrict__ lam,
    const double2 *__restrict__ gl, const double2 *__restrict__ A, const double2 *__restrict__ B,
    const double *__restrict__ yint, int L, int c, int ns, double kc, double r_enc,
    const int32_t *__restrict__ types, const double *__restrict__ rtype, const double2 *__restrict__ rcv, int64_t nr,
    int pchunks, int plen, int nlen, double2 *__restrict__ part) {
  const int64_t r = blockIdx.x * static_cast<int64_t>(kFieldThreads) + threadIdx.x;
  if (r >= nr) return;
  const double X = rcv[r].x, Y = rcv[r].y;
  // layer of the receiver: interfaces above it; the particle layer keeps y = 0
  int layer = 0;
  for (int i = 0; i < L - 1; ++i) layer += (Y < yint[i]) ? 1 : 0;
  if (Y == yint[c - 1]) layer = c;
  const int ch = blockIdx.y;
  cx<double> acc = mk(0.0, 0.0);
  if (ch >= pchunks) {
    const bool hasA = layer > 0, hasB = layer < L - 1;
    const double ta = hasA ? Y - yint[layer - 1] : 0.0;  // <= 0
    const double tb = hasB ? Y - yint[layer] : 0.0;      // >= 0
    const int64_t o = static_cast<int64_t>(layer) * ns;
    const int q0 = (ch - pchunks) * nlen, q1 = min(ns, q0 + nlen);
    for (int q = q0; q < q1; ++q) {
      const double lr = lam[q].x, li = lam[q].y;
      const cx<double> gq = ld<double>(gl[o + q]);
      if (hasA) cmac(acc, ld<double>(A[o + q]), cexpT<double>(-li * X + gq.re * ta, lr * X + gq.im * ta));
      if (hasB) cmac(acc, ld<double>(B[o + q]), cexpT<double>(-li * X - gq.re * tb, lr * X - gq.im * tb));
    }
  } else if (layer == c) {
    const int P = 2 * p + 1;
    const int m0 = ch * plen, m1 = min(n, m0 + plen);
    bool inside = false;
    for (int m = m0; m < m1; ++m) {
      const double dx = X - xy[m].x, dy = Y - xy[m].y;
      const double d2 = dx * dx + dy * dy;
      // the root rounded as sqrt rounds it (one Newton step from d2 / sqrt(d2)): the
      // phase of a far particle carries the distance's error times kc
      const double ri = rsqrt(d2), r0 = d2 * ri, rr = fma(0.5 * ri, fma(-r0, r0, d2), r0);
      const double rad = types ? rtype[types[m]] : r_enc;
      if (!(rr > (1.0 + 1e-9) * rad) && sqrt(d2) < rad) inside = true;  // decided on the rounded root
      const double z = kc * rr, zi = ri / kc;
      // e^{i phi}, rounded as quotients: its powers multiply its error by the order
      cx<double> t = mk(dx * ri, dy * ri);
      t = mk(fma(fma(-t.re, rr, dx), ri, t.re), fma(fma(-t.im, rr, dy), ri, t.im));
      cx<double> hp, hc;
      hankel01(z, zi, hp, hc);
      const double2 *b = D + static_cast<int64_t>(m) * P;
      cmac(acc, hp, ld<double>(b[0]));
      cx<double> tq = t;
      // 2q / z rounded once per order: 2 / z in two parts (a running sum, or the
      // multiples of a rounded 2 / z, would carry their errors into every order)
      const double tz = 2.0 * zi, tl = fma(-tz, z, 2.0) * zi;
      double qd = 1.0;
#pragma unroll 4
      for (int q = 1; q <= p; ++q) {
        const cx<double> dp = ld<double>(b[2 * q - 1]), dm = ld<double>(b[2 * q]);
        // tq b_q + (-1)^q conj(tq) b_{-q}
        cmac(acc, hc, mk(fma(tq.re, dp.re, -tq.im * dm.im), fma(tq.re, dp.im, tq.im * dm.re)));
        const double f = fma(qd, tz, qd * tl);
        const cx<double> hn = mk(fma(f, hc.re, -hp.re), fma(f, hc.im, -hp.im));  // H_{q+1} = (2q / z) H_q - H_{q-1}
        hp = hc;
        hc = hn;
        qd += 1.0;
        tq = tq * t;
      }
    }
    if (inside) acc = mk<double>(NAN, NAN);
  }
  part[ch * nr + r] = st(acc);
}

// u[r] = sum of the partials, plus the source's free field in the top layer:
// eight lanes per receiver take every eighth slot, added in order.
constexpr int kFieldSumLanes = 8;
__global__ __launch_bounds__(256) void k_field_sum(const double2 *__restrict__ part, int slots, int64_t nr,
                                                   const double2 *__restrict__ rcv, double ytop, int c, double k0,
                                                   double xs, double ys, double2 *__restrict__ u) {
  constexpr int RB = 256 / kFieldSumLanes;
  __shared__ double2 s[kFieldSumLanes][RB];
  const int w = threadIdx.x / RB, i = threadIdx.x % RB;
  const int64_t r = blockIdx.x * static_cast<int64_t>(RB) + i;
  double re = 0.0, im = 0.0;
  if (r < nr) {
#pragma unroll 4
    for (int k = w; k < slots; k += kFieldSumLanes) {
      const double2 v = part[k * nr + r];
      re += v.x;
      im += v.y;
    }
  }
  s[w][i] = make_double2(re, im);
  __syncthreads();
  if (w != 0 || r >= nr) return;
  cx<double> acc = mk(0.0, 0.0);
#pragma unroll
  for (int k = 0; k < kFieldSumLanes; ++k) acc = acc + ld<double>(s[k][i]);
  const double X = rcv[r].x, Y = rcv[r].y;
  if (!(Y < ytop) && !(c == 1 && Y == ytop)) {  // the top layer
    const double dx = X - xs, dy = Y - ys;
    const double z = k0 * sqrt(dx * dx + dy * dy);
    acc = acc + mk(0.0, 0.25) * mk(j0(z), y0(z));
  }
  u[r] = st(acc);
}

}  // namespace

// About 2048 blocks for the particles and a quarter as many for the (cheaper)
// nodes, with chunks of at least 16 particles and 32 nodes: shorter ones spend
// more on writing and adding the partials than the lanes gain.  Receivers go
// in batches, which bounds the partials to 10.5 MB.  With room (entries, at least
// 32768) fewer blocks and smaller batches, so that the partials fit.
FieldShape field_shape(const mpsl_ctx *ctx, int64_t nr, int64_t room) {
  constexpr int64_t kBlocks = 2560;
  const int64_t blocks = room > 0 ? std::min<int64_t>(kBlocks, room / kFieldThreads) : kBlocks;
  const int nb = static_cast<int>(blocks / 5), pb = static_cast<int>(blocks) - nb;
  FieldShape s{1, 1, std::min<int64_t>(nr, 65536)};
  for (int pass = 0; pass < 2; ++pass) {
    const int rb = cdiv(s.batch, kFieldThreads);
    s.pchunks = std::max(1, std::min(pb / rb, cdiv(ctx->n, 16)));
    s.nchunks = std::max(1, std::min(nb / rb, cdiv(ctx->ns, 32)));
    if ((s.pchunks + s.nchunks) * s.batch <= blocks * kFieldThreads) break;
    s.batch = std::min<int64_t>(s.batch, nb * static_cast<int64_t>(kFieldThreads));  // then no chunk count is raised to 1
  }
  return s;
}

size_t field_amp_bytes(const mpsl_ctx *ctx) { return sizeof(double2) * 3 * ctx->ks.size() * ctx->ns; }
size_t field_part_bytes(const FieldShape &s) { return sizeof(double2) * (s.pchunks + s.nchunks) * s.batch; }

double2 *field_idle(const mpsl_ctx *ctx, int64_t *room) {
  const int64_t len = ctx->n * static_cast<int64_t>(2 * ctx->p + 1), stack = 2 * static_cast<int64_t>(ctx->ks.size());
  // (the sizes that the buffers have from the start: what other calls made of them must not change the sums)
  const int64_t a = std::min<int64_t>(ctx->scal.bytes / sizeof(double2), 65536) - stack;
  const int64_t slots = work_slots(ctx) - 1;
  const int64_t b = std::min<int64_t>(slots * len, static_cast<int64_t>(ctx->part.bytes / sizeof(double2)) - len);
  *room = std::max(a, b);
  return a >= b ? static_cast<double2 *>(ctx->scal.p) + stack : static_cast<double2 *>(ctx->part.p) + len;
}

std::vector<double> field_stack(const mpsl_ctx *ctx) {
  const int L = static_cast<int>(ctx->ks.size());
  std::vector<double> h(4 * L, 1.0);  // kappa, thickness, k, interface heights
  for (int j = 0; j < L; ++j) {
    const double k = ctx->ks[j].real();
    if (ctx->pol == MPSL_TE) h[j] = 1.0 / (k * k);
    h[L + j] = ctx->thick[j];
    h[2 * L + j] = k;
    if (j < L - 1) h[3 * L + j] = ctx->yint[j];
  }
  return h;
}

int launch_field(mpsl_ctx *ctx, const FieldShape &s, const std::vector<double> &layers, const void *beta,
                 const void *spec, const void *sigma, const double *src, int64_t nr, const void *rcv, void *u,
                 void *amp, double2 *part) {
  const int L = static_cast<int>(ctx->ks.size()), ns = ctx->ns, n = static_cast<int>(ctx->n), p = ctx->p;
  const int64_t len = static_cast<int64_t>(n) * (2 * p + 1);
  auto *gl = static_cast<double2 *>(amp);
  auto *A = gl + static_cast<size_t>(L) * ns, *B = A + static_cast<size_t>(L) * ns;
  auto *stack = static_cast<double *>(ctx->scal.p);  // the solver's reductions, free here
  auto *D = static_cast<double2 *>(ctx->part.p);  // the matvec's partials, free here, hold n P entries at least
  if (ctx->part.bytes < len * sizeof(double2) || ctx->scal.bytes < layers.size() * sizeof(double))
    return set_err(ctx, MPSL_ESTATE, "work buffers not sized");
  MPSL_HIP_TRY(ctx, hipMemcpyAsync(stack, layers.data(), layers.size() * sizeof(double), hipMemcpyHostToDevice,
                                   ctx->stream));
  const auto *lam = static_cast<const double2 *>(ctx->ct.lam.p);
  const auto *gw = static_cast<const double2 *>(ctx->ct.gw.p);
  hipLaunchKernelGGL(k_field_amp, dim3(cdiv(ns, 64)), dim3(64), 0, ctx->stream, lam, gw,
                     static_cast<const double2 *>(spec), static_cast<const double2 *>(sigma), stack, L, ctx->layer_c,
                     ns, src[0], src[1] - ctx->yint[0], gl, A, B);
  MPSL_HIP_TRY(ctx, hipGetLastError());
  hipLaunchKernelGGL(k_field_coef, dim3(cdiv(len, 256)), dim3(256), 0, ctx->stream,
                     static_cast<const double2 *>(beta), n, p, D);
  MPSL_HIP_TRY(ctx, hipGetLastError());
  for (int64_t r0 = 0; r0 < nr; r0 += s.batch) {
    const int64_t cnt = std::min(s.batch, nr - r0);
    const auto *rc = static_cast<const double2 *>(rcv) + r0;
    hipLaunchKernelGGL(k_field_part, dim3(cdiv(cnt, kFieldThreads), s.pchunks + s.nchunks), dim3(kFieldThreads), 0,
                       ctx->stream, static_cast<const double2 *>(ctx->gt.xy.p), D, n, p, lam, gl, A, B, stack + 3 * L,
                       L, ctx->layer_c, ns, ctx->k2.real(), ctx->r_enc,
                       (ctx->n_types > 1 && !ctx->ptype.empty()) ? static_cast<const int32_t *>(ctx->types_dev.p)
                                                                  : nullptr,
                       static_cast<const double *>(ctx->rtype_dev.p), rc, cnt, s.pchunks, cdiv(n, s.pchunks),
                       cdiv(ns, s.nchunks), part);
    MPSL_HIP_TRY(ctx, hipGetLastError());
    hipLaunchKernelGGL(k_field_sum, dim3(cdiv(cnt, 256 / kFieldSumLanes)), dim3(256), 0, ctx->stream, part,
                       s.pchunks + s.nchunks, cnt, rc, ctx->yint[0], ctx->layer_c, ctx->k1.real(), src[0], src[1],
                       static_cast<double2 *>(u) + r0);
    MPSL_HIP_TRY(ctx, hipGetLastError());
  }
  return MPSL_OK;
}

}  // namespace mpsl
