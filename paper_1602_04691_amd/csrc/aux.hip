// Elementwise and reduction kernels: coefficients of eq. 2.19, the
// right-hand sides, and the COCG vector updates with their bilinear
// reductions.  Reductions are two-stage and deterministic: fixed-order
// per-workgroup partials, then one workgroup per right-hand side
// (k_finalize) in a fixed order.
#include "cx.h"
#include "kernels.h"
#include "launch.h"

namespace ori {
namespace {

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Deterministic workgroup sum of 4 values (kRedThreads threads); thread 0
// writes out[0..3].
template <int NT = kRedThreads>
__device__ __forceinline__ void block_sum4(double (&v)[4], double* out) {
  __shared__ double sh[(NT / 64) * 4];
#pragma unroll
  for (int j = 0; j < 4; ++j) v[j] = wave_sum(v[j]);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) sh[w * 4 + j] = v[j];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      double s = 0.0;
      for (int i = 0; i < NT / 64; ++i) s += sh[i * 4 + j];
      out[j] = s;
    }
  }
}

// Principal square root of a + ib.
__device__ __forceinline__ cxd csqrt(cxd z) {
  if (z.re == 0.0 && z.im == 0.0) return cxd{0.0, 0.0};
  const double r = hypot(z.re, z.im);
  if (z.re >= 0.0) {
    const double t = sqrt(0.5 * (r + z.re));
    return cxd{t, z.im / (2.0 * t)};
  }
  const double t = sqrt(0.5 * (r - z.re));
  return cxd{fabs(z.im) / (2.0 * t), copysign(t, z.im)};
}

__device__ __forceinline__ bool finite_cx(cxd z) { return isfinite(z.re) && isfinite(z.im); }

// grid-stride loop over [0, P) within the right-hand side blockIdx.y
#define ORI_RHS_LOOP(i)                                                                                \
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < P;                 \
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)

// a1, operator part: D = 4 pi h N vol, S = sqrt(D), c = 4 pi N vol.
// Partials per workgroup: {bad-input count, min |S|^2, max |S|^2, 0}.
__global__ void __launch_bounds__(kRedThreads)
    k_coefficients(const cxd* __restrict__ h, const double* __restrict__ N, double vol, int64_t P,
                   cxd* __restrict__ D, cxd* __restrict__ S, cxf* __restrict__ Sf, double* __restrict__ cN,
                   double* __restrict__ partials) {
  constexpr double FOUR_PI = 12.566370614359172954;  // c_S for spheres
  double bad_n = 0.0, mn = INFINITY, mx = 0.0;
  ORI_RHS_LOOP(i) {
    const cxd hv = h[i];
    const double nv = N ? N[i] : 1.0;
    const bool bad = !finite_cx(hv) || !isfinite(nv) || nv < 0.0;
    const double c = bad ? 0.0 : FOUR_PI * nv * vol;
    const cxd d = scale(bad ? cxd{0.0, 0.0} : hv, c);
    const cxd s = csqrt(d);
    D[i] = d;
    S[i] = s;
    if (Sf) Sf[i] = cvt<float>(s);
    cN[i] = c;
    bad_n += bad ? 1.0 : 0.0;
    const double s2 = norm2(s);
    mn = fmin(mn, s2);
    mx = fmax(mx, s2);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    bad_n += __shfl_xor(bad_n, off, 64);
    mn = fmin(mn, __shfl_xor(mn, off, 64));
    mx = fmax(mx, __shfl_xor(mx, off, 64));
  }
  __shared__ double sh[(kRedThreads / 64) * 3];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) {
    sh[3 * w] = bad_n;
    sh[3 * w + 1] = mn;
    sh[3 * w + 2] = mx;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < kRedThreads / 64; ++i) {
      sh[0] += sh[3 * i];
      sh[1] = fmin(sh[1], sh[3 * i + 1]);
      sh[2] = fmax(sh[2], sh[3 * i + 2]);
    }
    double* out = partials + 4 * static_cast<int64_t>(blockIdx.x);
    out[0] = sh[0];
    out[1] = sh[1];
    out[2] = sh[2];
    out[3] = 0.0;
  }
}

// {bad count, min |S|^2, max |S|^2} over nblk partials -> sc[0]; one
// workgroup, strided over the partials, then a fixed-order combine (the
// count is a sum of small integers, so the order does not matter anyway)
__global__ void __launch_bounds__(kRedThreads) k_finalize_coeff(const double* __restrict__ part, int64_t nblk,
                                                                ScalarBlock* sc) {
  double bad = 0.0, mn = INFINITY, mx = 0.0;
  for (int64_t i = threadIdx.x; i < nblk; i += kRedThreads) {
    bad += part[4 * i];
    mn = fmin(mn, part[4 * i + 1]);
    mx = fmax(mx, part[4 * i + 2]);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    bad += __shfl_xor(bad, off, 64);
    mn = fmin(mn, __shfl_xor(mn, off, 64));
    mx = fmax(mx, __shfl_xor(mx, off, 64));
  }
  __shared__ double sh[(kRedThreads / 64) * 3];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) {
    sh[3 * w] = bad;
    sh[3 * w + 1] = mn;
    sh[3 * w + 2] = mx;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  for (int i = 1; i < kRedThreads / 64; ++i) {
    sh[0] += sh[3 * i];
    sh[1] = fmin(sh[1], sh[3 * i + 1]);
    sh[2] = fmax(sh[2], sh[3 * i + 2]);
  }
  sc->flags = sh[0] > 0.0 ? FLAG_BAD_COEFF : 0;
  sc->s2_min = sh[1];
  sc->s2_max = sh[2];
}

// u = w / S, per right-hand side (S shared)
__global__ void __launch_bounds__(256) k_div(const cxd* __restrict__ w, const cxd* __restrict__ s,
                                             cxd* __restrict__ u, int64_t P) {
  const int64_t off = static_cast<int64_t>(blockIdx.y) * P;
  ORI_RHS_LOOP(i) {
    const cxd d = s[i];
    const double inv = 1.0 / norm2(d);
    u[off + i] = scale(w[off + i] * conj(d), inv);
  }
}

// q = (z + r) / S (one right-hand side; S nonzero), the division as in k_div
__global__ void __launch_bounds__(256) k_add_div(const cxd* __restrict__ z, const cxd* __restrict__ r,
                                                 const cxd* __restrict__ s, cxd* __restrict__ q, int64_t P) {
  ORI_RHS_LOOP(i) {
    const cxd d = s[i];
    const double inv = 1.0 / norm2(d);
    q[i] = scale((z[i] + r[i]) * conj(d), inv);
  }
}

// u = w / S as k_div, and the partials {-, -, ||r / S||^2, -} per
// right-hand side (red_grid): with r = b - (I + S G0 S) w and b = S u0,
// r / S = u0 - u - G0 D u, the residual of eq. 2.19 for u = w / S
__global__ void __launch_bounds__(kRedThreads)
    k_div_res(const cxd* __restrict__ w, const cxd* __restrict__ r, const cxd* __restrict__ s, cxd* __restrict__ u,
              int64_t P, double* __restrict__ partials) {
  const int64_t off = static_cast<int64_t>(blockIdx.y) * P;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  ORI_RHS_LOOP(i) {
    const cxd d = s[i];
    const double inv = 1.0 / norm2(d);
    u[off + i] = scale(w[off + i] * conj(d), inv);
    acc[2] += norm2(scale(r[off + i] * conj(d), inv));
  }
  block_sum4(acc, partials + 4 * (static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x));
}

// a1, right-hand sides: b = S u0 (one batch row per blockIdx.y)
__global__ void __launch_bounds__(kRedThreads)
    k_rhs(const cxd* __restrict__ u0, const cxd* __restrict__ S, int64_t P, cxd* __restrict__ b,
          cxd* __restrict__ u0c, double* __restrict__ partials) {
  const int64_t off = static_cast<int64_t>(blockIdx.y) * P;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  ORI_RHS_LOOP(i) {
    const cxd uv = u0[off + i];
    const bool bad = !finite_cx(uv);
    const cxd bv = bad ? cxd{0.0, 0.0} : S[i] * uv;
    b[off + i] = bv;
    u0c[off + i] = bad ? cxd{0.0, 0.0} : uv;
    acc[0] += norm2(bv);
    acc[1] += bad ? 0.0 : norm2(uv);
    acc[2] += bad ? 1.0 : 0.0;
  }
  block_sum4(acc, partials + 4 * (static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x));
}

// FIN_MU: alpha = rho / mu from the sums {mu.re, mu.im, qq, pp}.  A frozen
// right-hand side keeps its alpha for k_x_flush (skip).
struct MuStep {
  bool skip, breakdown;
  double re, im;
};
__device__ __forceinline__ MuStep mu_step(const ScalarBlock& sc, double s0, double s1, double s2, double s3,
                                          double eps) {
  MuStep m{(sc.flags & FLAG_DONE) != 0, false, 0.0, 0.0};
  if (m.skip || s3 == 0.0) return m;  // s3 = 0: r = p = 0, nothing moves
  if (hypot(s0, s1) <= eps * sqrt(s2 * s3)) {
    m.breakdown = true;
    return m;
  }
  const double den = s0 * s0 + s1 * s1;
  m.re = (sc.rho_re * s0 + sc.rho_im * s1) / den;
  m.im = (sc.rho_im * s0 - sc.rho_re * s1) / den;
  return m;
}
__device__ __forceinline__ void store_mu(ScalarBlock* sc, double s0, double s1, double s2, double s3, MuStep m) {
  if (m.skip) return;
  sc->mu_re = s0;
  sc->mu_im = s1;
  sc->pp = s3;
  sc->qq = s2;
  sc->alpha_re = m.re;
  sc->alpha_im = m.im;
}

// The scalars of right-hand side rhs from the sums s0..s3 (one thread).
__device__ __forceinline__ void finalize_scalars(ScalarBlock* sc, int64_t rhs, double s0, double s1, double s2,
                                                 double s3, int32_t mode, double eps, double tol2, int32_t tol2_of_bb,
                                                 const double* __restrict__ tol2_rhs) {
  switch (mode) {
    case FIN_SETUP:
      sc->bb = s0;
      sc->aux = s1;
      // keeps the coefficient check of sc[0] (k_finalize_coeff, earlier on
      // the stream), so that one copy to the host brings both
      sc->flags = (sc->flags & FLAG_BAD_COEFF) | (s2 > 0.0 ? FLAG_BAD_INPUT : 0);
      break;
    case FIN_INIT: {
      sc->rho_re = s0;
      sc->rho_im = s1;
      sc->rr = s2;
      sc->rr0 = s2;
      sc->beta_re = 0.0;
      sc->beta_im = 0.0;
      sc->alpha_re = 0.0;
      sc->alpha_im = 0.0;
      sc->iters = 0;
      sc->mu_broken = 0;
      sc->rr_target = (tol2_rhs ? tol2_rhs[rhs] : tol2) * (tol2_of_bb ? sc->bb : s2);
      int f = 0;
      if (s2 == 0.0) f |= FLAG_ZERO_RESIDUAL;
      else if (s2 <= sc->rr_target) f |= FLAG_CONVERGED;
      else if (hypot(s0, s1) <= eps * s2) f |= FLAG_BREAKDOWN_RHO;
      sc->flags = f;
      break;
    }
    case FIN_MU: {
      const MuStep m = mu_step(*sc, s0, s1, s2, s3, eps);
      store_mu(sc, s0, s1, s2, s3, m);
      if (m.breakdown) sc->flags |= FLAG_BREAKDOWN_MU;
      break;
    }
    case FIN_RHO: {
      int f = sc->flags;
      if (!(f & FLAG_DONE) && sc->mu_broken) sc->flags = f |= FLAG_BREAKDOWN_MU;
      if (f & FLAG_DONE) {  // frozen
        sc->beta_re = 0.0;
        sc->beta_im = 0.0;
        break;
      }
      sc->iters += 1;
      const double ro = sc->rho_re, io = sc->rho_im;
      sc->rr = s2;
      sc->beta_re = 0.0;
      sc->beta_im = 0.0;
      if (s2 == 0.0) {
        f |= FLAG_ZERO_RESIDUAL;
      } else if (s2 <= sc->rr_target) {
        f |= FLAG_CONVERGED;
      } else if (hypot(s0, s1) <= eps * s2) {
        f |= FLAG_BREAKDOWN_RHO;
      } else {
        const double den = ro * ro + io * io;  // beta = rho' / rho
        sc->beta_re = (s0 * ro + s1 * io) / den;
        sc->beta_im = (s1 * ro - s0 * io) / den;
      }
      sc->rho_re = s0;
      sc->rho_im = s1;
      sc->flags = f;
      break;
    }
    case FIN_NORM:
      sc->aux = s2;
      break;
  }
}

// One workgroup per right-hand side: reduce its nblk partial quadruples in a
// fixed order and update its scalars.  1024 threads: after the I1 pass there
// is one quadruple per I1 workgroup (16 384 at n = 256).
constexpr int kFinThreads = 1024;
__device__ __forceinline__ void finalize_body(const double* __restrict__ partials, int64_t nblk, ScalarBlock* scb,
                                              int64_t rhs, int32_t mode, double eps, double tol2, int32_t tol2_of_bb,
                                              const double* __restrict__ tol2_rhs, ScalarBlock* ring) {
  const double* part = partials + 4 * nblk * rhs;
  ScalarBlock* sc = scb + rhs;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int64_t i = threadIdx.x; i < nblk; i += kFinThreads) {
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] += part[4 * i + j];
  }
  __shared__ double tot[4];
  block_sum4<kFinThreads>(acc, tot);
  __syncthreads();
  if (threadIdx.x == 0) finalize_scalars(sc, rhs, tot[0], tot[1], tot[2], tot[3], mode, eps, tol2, tol2_of_bb, tol2_rhs);
  if (mode == FIN_RHO && ring) {
    __syncthreads();
    static_assert(sizeof(ScalarBlock) % sizeof(double) == 0, "scalar blocks are whole doubles");
    constexpr int W = static_cast<int>(sizeof(ScalarBlock) / sizeof(double));
    if (threadIdx.x < W)
      reinterpret_cast<double*>(ring + rhs)[threadIdx.x] = reinterpret_cast<const double*>(sc)[threadIdx.x];
  }
}

__global__ void __launch_bounds__(kFinThreads)
    k_finalize(const double* __restrict__ partials, int64_t nblk, ScalarBlock* scb, int32_t mode, double eps,
               double tol2, int32_t tol2_of_bb, const double* __restrict__ tol2_rhs, ScalarBlock* ring) {
  finalize_body(partials, nblk, scb, blockIdx.x, mode, eps, tol2, tol2_of_bb, tol2_rhs, ring);
}

// FIN_MU inside the update: the sums of nblk <= 1024 quadruples in the order
// of finalize_body on kFinThreads threads (64 quadruples per wave sum, the
// waves' sums added in order, the empty ones being zeros), by kRedThreads
// threads.  Every thread of the workgroup gets them.
__device__ __forceinline__ void mu_sums(const double* __restrict__ part, int64_t nblk, double (&tot)[4]) {
  constexpr int G = kFinThreads / 64, NW = kRedThreads / 64;
  __shared__ double sh[G * 4];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int g = w; g < G; g += NW) {
    const int64_t i = g * 64 + lane;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (g * 64 < nblk) {  // uniform over the wave
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = wave_sum(i < nblk ? 0.0 + part[4 * i + j] : 0.0);
    }
    if (lane < 4) sh[g * 4 + lane] = lane == 0 ? v[0] : lane == 1 ? v[1] : lane == 2 ? v[2] : v[3];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    double s = 0.0;
    for (int g = 0; g < G; ++g) s += sh[g * 4 + j];
    tot[j] = s;
  }
}

// workgroup bid of nb over right-hand side rhs; MU: FIN_MU is part of it (a
// variant of its own, so that the plain update keeps its registers: complex64
// 0.149 vs 0.187 ms at n = 320)
template <typename V, bool MU>
__device__ __forceinline__ void update_body(cx<V>* __restrict__ x, const cx<V>* __restrict__ p, cx<V>* __restrict__ r,
                                            const cx<V>* __restrict__ q, int64_t P, ScalarBlock* scb,
                                            double* __restrict__ partials, int64_t bid, int64_t nb, int64_t rhs,
                                            const double* __restrict__ mu, int64_t mu_nblk, double eps) {
  ScalarBlock* sc = scb + rhs;
  if (sc->flags & FLAG_DONE) return;  // frozen: FIN_RHO reads no partials either
  const int64_t off = rhs * P;
  cxd al;
  if constexpr (MU) {
    // every workgroup takes the same step; the scalars that the first one
    // stores are none of those the others read (a breakdown becomes a flag
    // in FIN_RHO)
    double tot[4];
    mu_sums(mu + 4 * mu_nblk * rhs, mu_nblk, tot);
    const MuStep m = mu_step(*sc, tot[0], tot[1], tot[2], tot[3], eps);
    if (bid == 0 && threadIdx.x == 0) {
      store_mu(sc, tot[0], tot[1], tot[2], tot[3], m);
      sc->mu_broken = m.breakdown ? 1 : 0;
    }
    al = cxd{m.re, m.im};
  } else {
    al = cxd{sc->alpha_re, sc->alpha_im};
  }
  const bool moving = al.re != 0.0 || al.im != 0.0;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int64_t i = bid * blockDim.x + threadIdx.x; i < P; i += nb * blockDim.x) {
    cxd rd;
    if (moving) {
      if (x) x[off + i] = cvt<V>(cfma(al, cvt<double>(p[off + i]), cvt<double>(x[off + i])));
      const cx<V> rs = cvt<V>(cfms(al, cvt<double>(q[off + i]), cvt<double>(r[off + i])));
      r[off + i] = rs;
      rd = cvt<double>(rs);  // reduce what was stored
    } else {
      rd = cvt<double>(r[off + i]);
    }
    const cxd rr = rd * rd;
    acc[0] += rr.re;
    acc[1] += rr.im;
    acc[2] += norm2(rd);
  }
  block_sum4(acc, partials + 4 * (rhs * nb + bid));
}

template <typename V, bool MU>
__global__ void __launch_bounds__(kRedThreads)
    k_update(cx<V>* __restrict__ x, const cx<V>* __restrict__ p, cx<V>* __restrict__ r,
             const cx<V>* __restrict__ q, int64_t P, ScalarBlock* scb, double* __restrict__ partials,
             const double* __restrict__ mu, int64_t mu_nblk, double eps) {
  update_body<V, MU>(x, p, r, q, P, scb, partials, blockIdx.x, gridDim.x, blockIdx.y, mu, mu_nblk, eps);
}

// The finalisation and the update of several problems in one launch
// (MultiFin, MultiUpd): workgroup b belongs to the problem whose range of
// workgroups holds it, and runs that problem's workgroup b - first_block.
template <typename E>
__device__ __forceinline__ int find_problem(const E* __restrict__ tab, int32_t np, int64_t b) {
  int p = 0;
  while (p + 1 < np && tab[p + 1].first_block <= b) ++p;
  return p;
}

__global__ void __launch_bounds__(kFinThreads)
    k_multi_finalize(const MultiFin* __restrict__ tab, int32_t np, int32_t mode, double eps, int64_t ring_at) {
  const MultiFin& m = tab[find_problem(tab, np, blockIdx.x)];
  finalize_body(m.partials, m.nblk, m.sc, blockIdx.x - m.first_block, mode, eps, 0.0, 0, nullptr,
                ring_at >= 0 ? m.ring + ring_at : nullptr);
}

// Every guard band of a workspace block in one launch: workgroup i fills
// band i with 16-byte stores (kGuardBandBytes / 16 = 256 threads).
static_assert(kGuardBandBytes == 256 * 16, "one 16-byte store per thread and band");
__global__ void __launch_bounds__(256) k_fill_guards(GuardBands g) {
  const uint32_t b = g.v & 0xFFu;
  const uint32_t w = b | (b << 8) | (b << 16) | (b << 24);
  uint4* band = reinterpret_cast<uint4*>(static_cast<unsigned char*>(g.base) + g.off[blockIdx.x]);
  band[threadIdx.x] = make_uint4(w, w, w, w);
}

template <typename V, bool MU>
__global__ void __launch_bounds__(kRedThreads) k_multi_update(const MultiUpd* __restrict__ tab, int32_t np, double eps) {
  const MultiUpd& m = tab[find_problem(tab, np, blockIdx.x)];
  update_body<V, MU>(nullptr, static_cast<const cx<V>*>(m.p), static_cast<cx<V>*>(m.r), static_cast<const cx<V>*>(m.q),
                 m.P, m.sc, m.partials, blockIdx.x - m.first_block, m.nblocks, 0, m.mu, m.mu_nblk, eps);
}

template <typename V>
__global__ void __launch_bounds__(256)
    k_x_flush(cx<V>* __restrict__ x, const cx<V>* __restrict__ p, int64_t P, const ScalarBlock* __restrict__ scb) {
  const ScalarBlock* sc = scb + blockIdx.y;
  const int64_t off = static_cast<int64_t>(blockIdx.y) * P;
  const cxd al = {sc->alpha_re, sc->alpha_im};
  if (al.re == 0.0 && al.im == 0.0) return;
  ORI_RHS_LOOP(i) x[off + i] = cvt<V>(cfma(al, cvt<double>(p[off + i]), cvt<double>(x[off + i])));
}

template <typename V>
__global__ void __launch_bounds__(kRedThreads)
    k_init(const cxd* __restrict__ b, const double* __restrict__ m, cx<V>* __restrict__ x, cx<V>* __restrict__ r,
           int64_t P, double* __restrict__ partials) {
  const int64_t off = static_cast<int64_t>(blockIdx.y) * P;
  double sc = 1.0;
  if (m) sc = m[blockIdx.y] > 0.0 ? 1.0 / m[blockIdx.y] : 0.0;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  ORI_RHS_LOOP(i) {
    const cx<V> rs = cvt<V>(scale(b[off + i], sc));
    r[off + i] = rs;
    x[off + i] = cx<V>{};
    const cxd rd = cvt<double>(rs);
    const cxd rr = rd * rd;
    acc[0] += rr.re;
    acc[1] += rr.im;
    acc[2] += norm2(rd);
  }
  block_sum4(acc, partials + 4 * (static_cast<int64_t>(blockIdx.y) * gridDim.x + blockIdx.x));
}

template <typename VI>
__global__ void __launch_bounds__(256)
    k_axpy_batch(const double* __restrict__ m, const cx<VI>* __restrict__ x, cxd* __restrict__ y, int64_t P) {
  const int64_t off = static_cast<int64_t>(blockIdx.y) * P;
  const double a = m[blockIdx.y];
  if (a == 0.0) return;
  ORI_RHS_LOOP(i) y[off + i] = y[off + i] + scale(cvt<double>(x[off + i]), a);
}

__global__ void __launch_bounds__(256) k_mul(const cxd* __restrict__ s, const cxd* __restrict__ x,
                                             cxd* __restrict__ y, int64_t P) {
  const int64_t off = static_cast<int64_t>(blockIdx.y) * P;
  ORI_RHS_LOOP(i) y[off + i] = s[i] * x[off + i];
}

__global__ void __launch_bounds__(kRedThreads)
    k_conj_diff(const cxd* __restrict__ u, const cxd* __restrict__ t, cxd* __restrict__ f, int64_t P,
                double* __restrict__ partials) {
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  ORI_RHS_LOOP(i) {
    const cxd e = u[i] - t[i];
    f[i] = conj(e);
    acc[2] += norm2(e);
  }
  block_sum4(acc, partials + 4 * static_cast<int64_t>(blockIdx.x));
}

__global__ void __launch_bounds__(256) k_gradient(const double* __restrict__ c, const cxd* __restrict__ u,
                                                  const cxd* __restrict__ q, double alpha, cxd* __restrict__ g,
                                                  int64_t P) {
  ORI_RHS_LOOP(i) g[i] = scale(u[i] * q[i], alpha * c[i]);
}

__global__ void __launch_bounds__(256) k_sub_mul(const cxd* __restrict__ f, const cxd* __restrict__ s,
                                                 const cxd* __restrict__ x, cxd* __restrict__ y, int64_t P) {
  ORI_RHS_LOOP(i) y[i] = f[i] - s[i] * x[i];
}

// Twiddles exp(-2 pi i m / L), m < L, in FP64 and FP32, exact at the
// quarter turns (the device counterpart of the host's long double table).
__global__ void __launch_bounds__(256) k_twiddles(int64_t L, cxd* __restrict__ twd, cxf* __restrict__ twf) {
  const int64_t m = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (m >= L) return;
  double cs, sn;
  if ((4 * m) % L == 0) {
    const int64_t q = 4 * m / L;
    cs = q == 0 ? 1.0 : (q == 2 ? -1.0 : 0.0);
    sn = q == 1 ? 1.0 : (q == 3 ? -1.0 : 0.0);
  } else {
    sincospi(2.0 * static_cast<double>(m) / static_cast<double>(L), &sn, &cs);
  }
  twd[m] = cxd{cs, -sn};
  twf[m] = cxf{static_cast<float>(cs), static_cast<float>(-sn)};
}

unsigned grid_for(int64_t P, int threads, int64_t cap) {
  int64_t g = (P + threads - 1) / threads;
  if (g > cap) g = cap;
  if (g < 1) g = 1;
  return static_cast<unsigned>(g);
}

dim3 red_grid(int64_t P, int64_t nrhs, int64_t cap = kRedBlocksMax) {
  return dim3(static_cast<unsigned>(red_blocks(P, cap)), static_cast<unsigned>(nrhs));
}

}  // namespace

hipError_t launch_coefficients(const void* h, const double* N, double vol, int64_t P, void* D, void* S, void* Sf,
                               double* cN, double* partials, hipStream_t st) {
  hipError_t e = hipSuccess;
  e = launch_kernel(k_coefficients, red_grid(P, 1), dim3(kRedThreads), st, static_cast<const cxd*>(h), N, vol, P,
                     static_cast<cxd*>(D), static_cast<cxd*>(S), static_cast<cxf*>(Sf), cN, partials);
  return e;
}

hipError_t launch_finalize_coeff(const double* partials, int64_t nblk, ScalarBlock* sc, hipStream_t st) {
  hipError_t e = hipSuccess;
  e = launch_kernel(k_finalize_coeff, dim3(1), dim3(kRedThreads), st, partials, nblk, sc);
  return e;
}

hipError_t launch_div(const void* w, const void* s, void* u, int64_t P, int64_t nrhs, hipStream_t st) {
  hipError_t e = hipSuccess;
  e = launch_kernel(k_div, dim3(grid_for(P, 256, 8192), static_cast<unsigned>(nrhs)), dim3(256), st,
                     static_cast<const cxd*>(w), static_cast<const cxd*>(s), static_cast<cxd*>(u), P);
  return e;
}

hipError_t launch_add_div(const void* z, const void* r, const void* s, void* q, int64_t P, hipStream_t st) {
  return launch_kernel(k_add_div, dim3(grid_for(P, 256, 8192), 1u), dim3(256), st, static_cast<const cxd*>(z),
                       static_cast<const cxd*>(r), static_cast<const cxd*>(s), static_cast<cxd*>(q), P);
}

hipError_t launch_div_res(const void* w, const void* r, const void* s, void* u, int64_t P, int64_t nrhs,
                          double* partials, hipStream_t st) {
  return launch_kernel(k_div_res, red_grid(P, nrhs), dim3(kRedThreads), st, static_cast<const cxd*>(w),
                       static_cast<const cxd*>(r), static_cast<const cxd*>(s), static_cast<cxd*>(u), P, partials);
}

hipError_t launch_rhs(const void* u0, const void* S, int64_t P, int64_t nrhs, void* b, void* u0c, double* partials,
                      hipStream_t st) {
  hipError_t e = hipSuccess;
  e = launch_kernel(k_rhs, red_grid(P, nrhs), dim3(kRedThreads), st, static_cast<const cxd*>(u0),
                     static_cast<const cxd*>(S), P, static_cast<cxd*>(b), static_cast<cxd*>(u0c), partials);
  return e;
}

hipError_t launch_finalize(const double* partials, int64_t nblk, int64_t nrhs, ScalarBlock* sc, int32_t mode,
                           double eps, double tol2, int32_t tol2_of_bb, const double* tol2_rhs, ScalarBlock* ring,
                           hipStream_t st) {
  return launch_kernel(k_finalize, dim3(static_cast<unsigned>(nrhs)), dim3(kFinThreads), st, partials, nblk, sc, mode,
                       eps, tol2, tol2_of_bb, tol2_rhs, ring);
}

template <typename V>
hipError_t update_t(void* x, const void* p, void* r, const void* q, int64_t P, dim3 grid, ScalarBlock* sc,
                    double* partials, const double* mu, int64_t mu_nblk, double eps, hipStream_t st) {
  return launch_kernel(mu ? k_update<V, true> : k_update<V, false>, grid, dim3(kRedThreads), st, static_cast<cx<V>*>(x),
                       static_cast<const cx<V>*>(p), static_cast<cx<V>*>(r), static_cast<const cx<V>*>(q), P, sc,
                       partials, mu, mu_nblk, eps);
}

hipError_t launch_update(int prec, void* x, const void* p, void* r, const void* q, int64_t P, int64_t nrhs,
                         ScalarBlock* sc, double* partials, const double* mu, int64_t mu_nblk, double eps,
                         hipStream_t st) {
  if (mu && (mu_nblk < 1 || mu_nblk > kFinThreads)) return hipErrorInvalidValue;
  if (prec == PREC_F64) return update_t<double>(x, p, r, q, P, red_grid(P, nrhs), sc, partials, mu, mu_nblk, eps, st);
  return update_t<float>(x, p, r, q, P, red_grid(P, nrhs, kUpdateBlocksMaxF32), sc, partials, mu, mu_nblk, eps, st);
}

hipError_t launch_multi_finalize(const MultiFin* tab, int32_t np, int64_t blocks, int32_t mode, double eps,
                                 int64_t ring_at, hipStream_t st) {
  if (np < 1 || blocks < 1) return hipErrorInvalidValue;
  return launch_kernel(k_multi_finalize, dim3(static_cast<unsigned>(blocks)), dim3(kFinThreads), st, tab, np, mode,
                       eps, ring_at);
}

hipError_t launch_fill_guards(const GuardBands& g, hipStream_t st) {
  if (g.count < 0 || g.count > kMaxGuardBands || !g.base) return hipErrorInvalidValue;
  for (int i = 0; i < g.count; ++i)
    if (g.off[i] < 0 || g.off[i] % 16 != 0) return hipErrorInvalidValue;
  if (g.count == 0) return hipSuccess;
  return launch_kernel(k_fill_guards, dim3(static_cast<unsigned>(g.count)), dim3(256), st, g);
}

hipError_t launch_multi_update(int prec, bool mu, const MultiUpd* tab, int32_t np, int64_t blocks, double eps,
                               hipStream_t st) {
  if (np < 1 || blocks < 1) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(blocks)), block(kRedThreads);
  if (prec == PREC_F64)
    return launch_kernel(mu ? k_multi_update<double, true> : k_multi_update<double, false>, grid, block, st, tab, np,
                         eps);
  return launch_kernel(mu ? k_multi_update<float, true> : k_multi_update<float, false>, grid, block, st, tab, np, eps);
}

hipError_t launch_x_flush(int prec, void* x, const void* p, int64_t P, int64_t nrhs, const ScalarBlock* sc,
                          hipStream_t st) {
  hipError_t e = hipSuccess;
  const dim3 g(static_cast<unsigned>(grid_for(P, 256, 8192)), static_cast<unsigned>(nrhs));
  if (prec == PREC_F64)
    e = launch_kernel(k_x_flush<double>, g, dim3(256), st, static_cast<cxd*>(x), static_cast<const cxd*>(p), P,
                       sc);
  else
    e = launch_kernel(k_x_flush<float>, g, dim3(256), st, static_cast<cxf*>(x), static_cast<const cxf*>(p), P,
                       sc);
  return e;
}

hipError_t launch_init(int prec, const void* b, const double* m, void* x, void* r, int64_t P, int64_t nrhs,
                       double* partials, hipStream_t st) {
  hipError_t e = hipSuccess;
  if (prec == PREC_F64)
    e = launch_kernel(k_init<double>, red_grid(P, nrhs), dim3(kRedThreads), st, static_cast<const cxd*>(b), m,
                       static_cast<cxd*>(x), static_cast<cxd*>(r), P, partials);
  else
    e = launch_kernel(k_init<float>, red_grid(P, nrhs), dim3(kRedThreads), st, static_cast<const cxd*>(b), m,
                       static_cast<cxf*>(x), static_cast<cxf*>(r), P, partials);
  return e;
}

hipError_t launch_axpy_batch(int prec_in, const double* m, const void* x, void* y, int64_t P, int64_t nrhs,
                             hipStream_t st) {
  hipError_t e = hipSuccess;
  const dim3 g(grid_for(P, 256, 8192), static_cast<unsigned>(nrhs));
  if (prec_in == PREC_F64)
    e = launch_kernel(k_axpy_batch<double>, g, dim3(256), st, m, static_cast<const cxd*>(x),
                       static_cast<cxd*>(y), P);
  else
    e = launch_kernel(k_axpy_batch<float>, g, dim3(256), st, m, static_cast<const cxf*>(x), static_cast<cxd*>(y),
                       P);
  return e;
}

hipError_t launch_mul(const void* s, const void* x, void* y, int64_t P, int64_t nrhs, hipStream_t st) {
  hipError_t e = hipSuccess;
  e = launch_kernel(k_mul, dim3(grid_for(P, 256, 8192), static_cast<unsigned>(nrhs)), dim3(256), st,
                     static_cast<const cxd*>(s), static_cast<const cxd*>(x), static_cast<cxd*>(y), P);
  return e;
}

hipError_t launch_conj_diff(const void* u, const void* t, void* f, int64_t P, double* partials, hipStream_t st) {
  hipError_t e = hipSuccess;
  e = launch_kernel(k_conj_diff, red_grid(P, 1), dim3(kRedThreads), st, static_cast<const cxd*>(u),
                     static_cast<const cxd*>(t), static_cast<cxd*>(f), P, partials);
  return e;
}

hipError_t launch_gradient(const double* c, const void* u, const void* q, double alpha, void* g, int64_t P,
                           hipStream_t st) {
  hipError_t e = hipSuccess;
  e = launch_kernel(k_gradient, dim3(grid_for(P, 256, 8192)), dim3(256), st, c, static_cast<const cxd*>(u),
                     static_cast<const cxd*>(q), alpha, static_cast<cxd*>(g), P);
  return e;
}

hipError_t launch_sub_mul(const void* f, const void* s, const void* x, void* lam, int64_t P, hipStream_t st) {
  hipError_t e = hipSuccess;
  e = launch_kernel(k_sub_mul, dim3(grid_for(P, 256, 8192)), dim3(256), st, static_cast<const cxd*>(f),
                     static_cast<const cxd*>(s), static_cast<const cxd*>(x), static_cast<cxd*>(lam), P);
  return e;
}

hipError_t launch_twiddles(int64_t L, void* twd, void* twf, hipStream_t st) {
  hipError_t e = hipSuccess;
  e = launch_kernel(k_twiddles, dim3(static_cast<unsigned>((L + 255) / 256)), dim3(256), st, L, static_cast<cxd*>(twd),
                    static_cast<cxf*>(twf));
  return e;
}

}  // namespace ori
