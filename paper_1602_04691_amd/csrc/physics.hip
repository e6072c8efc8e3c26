// What the solution of eq. 2.19 is used for.
//
//  * Charges (eq. 2.13 summed over the particles of a cell with eq. 2.18):
//    Q_p = -c_S h_p N_p |Delta_p| u_p = -D_p u_p.
//  * The scattered field anywhere (eq. 2.10, the particles of each cell at
//    x_p): v(x) = sum_p G(x, x_p) Q_p, G of eq. 2.6a; a cell point at distance
//    exactly 0 is left out, as the sum of eq. 2.19 leaves out p = q.
//  * Its far-field amplitude: v(r beta) = A(beta) e^{ikr} / r + O(1/r^2) with
//    A(beta) = (1 / 4 pi) sum_p e^{-ik beta.x_p} Q_p.
//  * The refraction recipe (eqs. 2.24-2.26, 4.1-4.2): n = [n0^2 - c_S h N /
//    k^2]^{1/2} with the branch arg in [0, 2 pi), and the h that creates a
//    desired n.
//  * The solution difference of Section 4 (Table 4) between a fine and a
//    coarse grid: the sup over coarse cells of the mean |x_i - y_q| over the
//    fine points x_i inside the cell.
//
// The sums over cells are direct (M points x P cells, FP64): workgroup
// (part of the cells, group of points, right-hand side) writes one partial
// per point; a second kernel adds the partials of each point in a fixed
// order, so results are deterministic.
//
// Both sums are bound by VALU issue, so the kernels are built to issue little
// per point-cell pair: a thread owns columns (i2, i3) of cells and a few
// points, and walks i1.  What depends on the column alone is computed once
// per column, what depends on the cell alone (its charge) once for all the
// points, and what depends on the point and i1 alone is uniform or read from
// LDS.  4 096 points and n = 64 on one MI355X: the field 4.28 -> 1.38 ms
// (120 -> 38 issue slots per pair), the far field 1.44 -> 0.34 ms.
#include "cx.h"
#include "kernels.h"
#include "launch.h"

namespace ori {
namespace {

constexpr int kFieldThreads = 256;
constexpr double kFourPi = 12.566370614359172954;

// s + e = s + v without rounding (Knuth's two-sum), e added to lo
__device__ __forceinline__ void two_sum(double& s, double& lo, double v) {
  const double t = s + v, b = t - s;
  lo += (s - (t - b)) + (v - b);
  s = t;
}

// Sum over the workgroup, thread 0 holds it.  The waves' sums are added with
// their rounding errors kept in *lo if lo is given.
__device__ __forceinline__ cxd block_sum_cx(cxd v, cxd* lo = nullptr) {
  __shared__ double sh[2 * (kFieldThreads / 64)];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    v.re += __shfl_xor(v.re, off, 64);
    v.im += __shfl_xor(v.im, off, 64);
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 0) {
    sh[2 * w] = v.re;
    sh[2 * w + 1] = v.im;
  }
  __syncthreads();
  cxd s{0.0, 0.0};
  if (threadIdx.x == 0)
    for (int i = 0; i < kFieldThreads / 64; ++i) {
      if (lo) {
        two_sum(s.re, lo->re, sh[2 * i]);
        two_sum(s.im, lo->im, sh[2 * i + 1]);
      } else {
        s = s + cxd{sh[2 * i], sh[2 * i + 1]};
      }
    }
  return s;
}

constexpr int kFieldMaxN = 512;

// A workgroup's sum for a point.  It is over neighbouring columns, whose sums
// cancel against those of other workgroups, so the rounding of the last few
// additions would show: their errors are kept.  Error of the field at points
// around a body of n = 64 against long double: 1.0e-16 (k = 5) and 0.8e-16
// (k = 8), 3.6e-16 and 5.8e-16 without, in the same time.
__device__ __forceinline__ void store_part(const FieldArgs& a, int64_t at, cxd v) {
  cxd lo{0.0, 0.0};
  const cxd s = block_sum_cx(v, &lo);
  if (threadIdx.x == 0 && at >= 0) {
    a.part[at] = s;
    a.part_lo[at] = lo;
  }
}

// coordinate of index i along axis d
__device__ __forceinline__ double cell_coord(const FieldArgs& a, int d, int i) {
  return a.origin[d] + a.side * (static_cast<double>(i) + a.offset) / a.dn;
}

// 1 / sqrt(x) for a normal x > 0: the hardware estimate (about 26 bits) and
// one step of Halley's iteration, e = 1 - x y^2, y (1 + e/2 + 3 e^2/8),
// whose error of order e^3 is below the rounding.
__device__ __forceinline__ double fast_rsqrt(double x) {
  const double y = __builtin_amdgcn_rsq(x);
  const double e = fmadd(-(x * y), y, 1.0);
  return fmadd(y * e, fmadd(0.375, e, 0.5), y);
}

// e^{2 pi i t / kTurn} from a table of the kTurn-th roots of unity: t = j +
// d, |d| <= 1/2, e^{2 pi i j / kTurn} read, the small rotation by its Taylor
// series (the angle is at most pi / kTurn = 0.0123: the terms left out are
// below 1e-17).  t is the unevaluated sum th + tl; th below 2^50 in size, so
// that adding 1.5 2^52 rounds it to the integer j and leaves j's low bits in
// the low word.
constexpr int kTurn = 256;
__device__ __forceinline__ cxd turn(double th, double tl, const cxd* __restrict__ tab) {
  constexpr double MAGIC = 6755399441055744.0;  // 1.5 * 2^52
  constexpr double W = 6.28318530717958647693 / kTurn, W2 = W * W;
  const double jm = th + MAGIC;
  const double d = (th - (jm - MAGIC)) + tl;
  const cxd r = tab[static_cast<uint32_t>(__builtin_bit_cast(uint64_t, jm)) & (kTurn - 1)];
  const double z = d * d;
  const double s = d * fmadd(z, fmadd(z, W2 * W2 * W / 120.0, -W2 * W / 6.0), W);
  const double c1 = z * fmadd(z, fmadd(z, -W2 * W2 * W2 / 720.0, W2 * W2 / 24.0), -W2 / 2.0);  // cos - 1
  return {fmadd(r.re, c1, fmadd(-r.im, s, r.re)), fmadd(r.im, c1, fmadd(r.re, s, r.im))};
}

// squared distances from here on take fast_rsqrt
constexpr double kNearSq = 0x1p-900;

// Field: grid (parts, groups of MP points, right-hand sides), part =
// (block of 256 columns, range of i1).  Per pair: the distance (2
// operations: the column's share of r^2 is kept), 1/r (6), r and the phase
// k r in units of 1/kTurn turns as an unevaluated sum of two doubles (4: the
// product's rounding error is kept, so the phase is as good as r itself),
// its e^{i..} (14, above) and the sum (6).  A cell at the point itself is left
// out, whatever its charge: the waves that hold such a column test each
// distance, which changes no other bit.  Points so far away that the phase
// would pass 2^50, or so close to a cell that the short 1/r ends, take the
// library's functions in a loop of their own, so that a point's value does
// not depend on the others of its group.  MP points share a cell's loads and
// charge: 4 where that leaves 1024 workgroups, else 1.
template <int MP>
__global__ void __launch_bounds__(kFieldThreads) k_field_near(FieldArgs a) {
  __shared__ double x1[kFieldMaxN];
  __shared__ cxd tab[kTurn];
  const int n = static_cast<int>(a.n), nn = n * n;
  const int part = blockIdx.x, cb = part / a.nch, ch = part - cb * a.nch;
  const int64_t m0 = static_cast<int64_t>(blockIdx.y) * MP, rhs = blockIdx.z;
  const int lo = static_cast<int>(static_cast<int64_t>(ch) * n / a.nch);
  const int hi = static_cast<int>((static_cast<int64_t>(ch) + 1) * n / a.nch);
  for (int i = lo + threadIdx.x; i < hi; i += kFieldThreads) x1[i] = cell_coord(a, 0, i);
  static_assert(kTurn == kFieldThreads, "one root of unity per thread");
  {
    double s, c;
    sincospi(threadIdx.x * (2.0 / kTurn), &s, &c);
    tab[threadIdx.x] = cxd{c, s};
  }
  const int col = cb * kFieldThreads + threadIdx.x;
  const bool act = col < nn;
  const int cc = act ? col : nn - 1;
  const int i2 = cc / n, i3 = cc - i2 * n;
  const double x2 = cell_coord(a, 1, i2), x3 = cell_coord(a, 2, i3);
  double y0[MP], s23[MP];
  bool lib[MP], any_lib = false, all_lib = true, own = false;
#pragma unroll
  for (int m = 0; m < MP; ++m) {
    const int64_t pm = m0 + m < a.mb ? m0 + m : a.mb - 1;
    const double* y = a.pts + 3 * (a.m0 + pm);
    y0[m] = y[0];
    const double d1 = y[1] - x2, d2 = y[2] - x3;
    s23[m] = d1 * d1 + d2 * d2;
    // the farthest corner of the grid: uniform over the workgroup
    double far2 = 0.0;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const double u = fabs(y[d] - a.corner[d]), v = fabs(y[d] - a.corner[3 + d]);
      far2 += u > v || !(u <= v) ? u * u : v * v;
    }
    // Uniform over the wave.  With |y0| from 2^-390 on, y0 - x1 is 0 or above
    // 2^-443, so r^2 is s23 or from kNearSq on.
    const bool column = __any(s23[m] < kNearSq), close = __any(s23[m] > 0.0 && s23[m] < kNearSq);
    lib[m] = !(far2 * a.kt_hi * a.kt_hi < 0x1p100 && far2 < 0x1p1000) || close ||
             (column && fabs(y0[m]) < 0x1p-390);
    own = own || column;
    any_lib = any_lib || lib[m];
    all_lib = all_lib && lib[m];
  }
  __syncthreads();
  const cxd* __restrict__ u = a.u + rhs * a.P;
  cxd acc[MP] = {};
  // Q_p / (4 pi) of the column's cell at i1; the next cell's values are
  // loaded while the current one is summed
  const cxd* __restrict__ Dc = a.D + cc;
  const cxd* __restrict__ uc = u + cc;
  cxd dn, un;
  auto first_q = [&]() {
    dn = Dc[static_cast<int64_t>(lo) * nn];
    un = uc[static_cast<int64_t>(lo) * nn];
  };
  auto next_q = [&](int i1) -> cxd {
    const cxd q = scale(dn * un, -1.0 / kFourPi);
    const int64_t p = static_cast<int64_t>(i1 + 1 < hi ? i1 + 1 : i1) * nn;
    dn = Dc[p];
    un = uc[p];
    return q;
  };
  auto phase = [&](double r) -> cxd {  // e^{ikr}
    const double th = r * a.kt_hi, tl = fmadd(r, a.kt_lo, fmadd(r, a.kt_hi, -th));
    return turn(th, tl, tab);
  };
  auto sum = [&](auto test_distance) {
    first_q();
    for (int i1 = lo; i1 < hi; ++i1) {
      const cxd q = next_q(i1);
      const double x = x1[i1];
#pragma unroll
      for (int m = 0; m < MP; ++m) {
        const double d0 = y0[m] - x;
        const double rsq = fmadd(d0, d0, s23[m]);
        const bool other = !decltype(test_distance)::value || rsq >= kNearSq;
        const double safe = other ? rsq : 1.0, ir = fast_rsqrt(safe);
        const cxd w = scale(q, ir);
        acc[m] = cfma(phase(safe * ir), other ? w : cxd{0.0, 0.0}, acc[m]);
      }
    }
  };
  if (!all_lib) {
    if (own)
      sum(std::true_type{});
    else
      sum(std::false_type{});
  }
  if (any_lib) {
#pragma unroll
    for (int m = 0; m < MP; ++m)
      if (lib[m]) acc[m] = cxd{0.0, 0.0};
    first_q();
    for (int i1 = lo; i1 < hi; ++i1) {
      const cxd q = next_q(i1);
      const double x = x1[i1];
#pragma unroll
      for (int m = 0; m < MP; ++m) {
        if (!lib[m]) continue;
        const double d0 = y0[m] - x;
        const double rsq = d0 * d0 + s23[m];
        if (rsq > 0.0) {
          const double ir = rsqrt(rsq), r = rsq * ir;
          double s, c;
          sincos(a.k * r, &s, &c);
          acc[m] = acc[m] + cxd{c * ir, s * ir} * q;
        }
      }
    }
  }
  // lanes beyond the last column hold a copy of it
  if (!act) {
#pragma unroll
    for (int m = 0; m < MP; ++m) acc[m] = cxd{0.0, 0.0};
  }
#pragma unroll
  for (int m = 0; m < MP; ++m) {
    if (m > 0) __syncthreads();
    store_part(a, m0 + m < a.mb ? (rhs * a.mb + m0 + m) * a.nparts + part : -1, acc[m]);
  }
}

// Far field: the phase of a cell is the product of three axis phases
// e^{-ik beta_d x_d}, tabulated in LDS per point, so the sum over i1 is one
// complex multiply-add per pair (4 FP64 operations), and the column's two
// phases multiply its sum.  A thread takes COLS columns, which share each
// LDS read of an i1 phase, and MP points, which share a cell's charge.  COLS
// is 4, or 2 or 1 where that holds every column of a smaller grid: the rest
// would be idle lanes (n = 17: 289 columns).
template <int MP, int COLS>
__global__ void __launch_bounds__(kFieldThreads, 4) k_field_far(FieldArgs a) {
  extern __shared__ __align__(16) unsigned char far_smem[];
  cxd* ph = reinterpret_cast<cxd*>(far_smem);  // [3][n][MP]
  const int n = static_cast<int>(a.n), nn = n * n;
  const int part = blockIdx.x, cb = part / a.nch, ch = part - cb * a.nch;
  const int64_t m0 = static_cast<int64_t>(blockIdx.y) * MP, rhs = blockIdx.z;
  const int lo = static_cast<int>(static_cast<int64_t>(ch) * n / a.nch);
  const int hi = static_cast<int>((static_cast<int64_t>(ch) + 1) * n / a.nch);
  for (int t = threadIdx.x; t < 3 * n * MP; t += kFieldThreads) {
    const int m = t % MP, i = t / MP % n, d = t / (MP * n);
    const int64_t pm = m0 + m < a.mb ? m0 + m : a.mb - 1;
    double s, c;
    sincos(-a.k * (a.pts[3 * (a.m0 + pm) + d] * cell_coord(a, d, i)), &s, &c);
    ph[t] = cxd{c, s};
  }
  __syncthreads();
  const cxd* __restrict__ u = a.u + rhs * a.P;
  const int c0 = cb * COLS * kFieldThreads + threadIdx.x;
  int cc[COLS];
#pragma unroll
  for (int j = 0; j < COLS; ++j) cc[j] = c0 + j * kFieldThreads < nn ? c0 + j * kFieldThreads : nn - 1;
  cxd acc[MP][COLS] = {};
  for (int i1 = lo; i1 < hi; ++i1) {
    cxd q[COLS];
#pragma unroll
    for (int j = 0; j < COLS; ++j) {
      const int64_t p = static_cast<int64_t>(i1) * nn + cc[j];
      q[j] = scale(a.D[p] * u[p], -1.0);  // Q_p
    }
#pragma unroll
    for (int m = 0; m < MP; ++m) {
      const cxd e = ph[i1 * MP + m];
#pragma unroll
      for (int j = 0; j < COLS; ++j) acc[m][j] = cfma(e, q[j], acc[m][j]);
    }
  }
#pragma unroll
  for (int m = 0; m < MP; ++m) {
    cxd t{0.0, 0.0};
#pragma unroll
    for (int j = 0; j < COLS; ++j) {
      if (c0 + j * kFieldThreads >= nn) continue;  // a copy of the last column
      const int i2 = cc[j] / n, i3 = cc[j] - i2 * n;
      const cxd e = ph[(n + i2) * MP + m] * ph[(2 * n + i3) * MP + m];
      const cxd s = acc[m][j];
      if (isfinite(s.re) && isfinite(s.im)) {
        t = cfma(e, s, t);
        continue;
      }
      // an infinite or NaN charge, or a sum out of range: cell by cell, since
      // the product of two sums would make infinities NaN
      for (int i1 = lo; i1 < hi; ++i1) {
        const int64_t p = static_cast<int64_t>(i1) * nn + cc[j];
        t = t + (ph[i1 * MP + m] * e) * scale(a.D[p] * u[p], -1.0);
      }
    }
    if (m > 0) __syncthreads();
    store_part(a, m0 + m < a.mb ? (rhs * a.mb + m0 + m) * a.nparts + part : -1, t);
  }
}

// One thread per (point, right-hand side): parts in order, with the rounding
// errors of the sums; a sum that is no number has none.
__global__ void __launch_bounds__(64) k_field_finalize(FieldArgs a, int32_t far) {
  const int64_t m = static_cast<int64_t>(blockIdx.x) * 64 + threadIdx.x, rhs = blockIdx.y;
  if (m >= a.mb) return;
  const int64_t at = (rhs * a.mb + m) * a.nparts;
  const cxd *part = a.part + at, *part_lo = a.part_lo + at;
  cxd s{0.0, 0.0}, lo{0.0, 0.0};
  for (int64_t c = 0; c < a.nparts; ++c) {
    lo = lo + part_lo[c];
    two_sum(s.re, lo.re, part[c].re);
    two_sum(s.im, lo.im, part[c].im);
  }
  if (isfinite(s.re)) s.re += lo.re;
  if (isfinite(s.im)) s.im += lo.im;
  if (far) s = scale(s, 1.0 / kFourPi);
  a.out[rhs * a.M + a.m0 + m] = s;
}

__global__ void __launch_bounds__(256) k_charges(const cxd* __restrict__ D, const cxd* __restrict__ u, int64_t P,
                                                 cxd* __restrict__ q) {
  const int64_t off = static_cast<int64_t>(blockIdx.y) * P;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < P;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    q[off + i] = scale(D[i] * u[off + i], -1.0);
}

// z^{1/2} with arg z in [0, 2 pi) (eq. 4.2): the root with Im >= 0, and the
// positive root on the cut [0, +inf).  The larger component comes from a
// square root, the smaller one from |Im z| / (2 * larger), so neither loses
// digits to cancellation.
__device__ __forceinline__ cxd sqrt_upper(cxd z) {
  if (z.re == 0.0 && z.im == 0.0) return cxd{0.0, 0.0};
  const double r = hypot(z.re, z.im), ay = fabs(z.im);
  double re, im;
  if (z.re >= 0.0) {
    re = sqrt(0.5 * (r + z.re));
    im = ay / (2.0 * re);
  } else {
    im = sqrt(0.5 * (r - z.re));
    re = ay / (2.0 * im);
  }
  if (z.im < 0.0) re = -re;  // arg in (pi, 2 pi): Re < 0
  return cxd{re, im};
}

// partials[block] = number of bad entries (N <= 0 or a non-finite input)
__global__ void __launch_bounds__(256) k_refraction(RefractionArgs a) {
  __shared__ double sh[4];
  double bad = 0.0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < a.P;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const cxd n0 = a.n0[i], x = a.in[i];
    const double N = a.N ? a.N[i] : 1.0;
    const bool ok = isfinite(n0.re) && isfinite(n0.im) && isfinite(x.re) && isfinite(x.im) && isfinite(N) &&
                    (a.design ? N > 0.0 : N >= 0.0);
    cxd out{0.0, 0.0};
    if (ok) {
      if (a.design) {
        // h = k^2 (n0^2 - n^2) / (c_S N)  (eqs. 2.25, 2.26)
        out = scale(n0 * n0 - x * x, a.k * a.k / (a.c_s * N));
      } else {
        // n = [n0^2 - c_S h N / k^2]^{1/2}  (eq. 4.1)
        out = sqrt_upper(n0 * n0 - scale(x, a.c_s * N / (a.k * a.k)));
      }
    }
    a.out[i] = out;
    bad += ok ? 0.0 : 1.0;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) bad += __shfl_xor(bad, off, 64);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = bad;
  __syncthreads();
  if (threadIdx.x == 0) a.bad[blockIdx.x] = sh[0] + sh[1] + sh[2] + sh[3];
}

// One workgroup per coarse cell q: the fine points inside it are those whose
// index i (per axis) has floor((i + off) nc / nf) = q; they lie in a box of
// a few more than nf / nc indices per axis around q nf / nc.
__global__ void __launch_bounds__(kFieldThreads) k_cell_difference(DiffArgs a) {
  const int64_t q = blockIdx.x;
  const int64_t qq[3] = {q / (a.nc * a.nc), (q / a.nc) % a.nc, q % a.nc};
  int64_t lo[3], len[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    const double dn = static_cast<double>(a.nf), dc = static_cast<double>(a.nc);
    int64_t l = static_cast<int64_t>(floor(static_cast<double>(qq[d]) * dn / dc - a.off)) - 1;
    int64_t h = static_cast<int64_t>(ceil(static_cast<double>(qq[d] + 1) * dn / dc - a.off)) + 2;
    l = l < 0 ? 0 : l;
    h = h > a.nf ? a.nf : h;
    lo[d] = l;
    len[d] = h > l ? h - l : 0;
  }
  const cxd yq = a.y[q];
  const int64_t box = len[0] * len[1] * len[2];
  double sum = 0.0, cnt = 0.0;
  for (int64_t t = threadIdx.x; t < box; t += kFieldThreads) {
    const int64_t i[3] = {lo[0] + t / (len[1] * len[2]), lo[1] + (t / len[2]) % len[1], lo[2] + t % len[2]};
    bool in = true;
#pragma unroll
    for (int d = 0; d < 3; ++d)
      in = in && static_cast<int64_t>(floor((static_cast<double>(i[d]) + a.off) * static_cast<double>(a.nc) /
                                            static_cast<double>(a.nf))) == qq[d];
    if (in) {
      const cxd x = a.x[(i[0] * a.nf + i[1]) * a.nf + i[2]];
      sum += hypot(x.re - yq.re, x.im - yq.im);
      cnt += 1.0;
    }
  }
  const cxd t = block_sum_cx(cxd{sum, cnt});
  if (threadIdx.x == 0) a.means[q] = t.im > 0.0 ? t.re / t.im : -1.0;
}

__global__ void __launch_bounds__(256) k_max(const double* __restrict__ v, int64_t P, double* __restrict__ part) {
  __shared__ double sh[4];
  double m = -1.0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < P;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    m = fmax(m, v[i]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = fmax(fmax(sh[0], sh[1]), fmax(sh[2], sh[3]));
}

}  // namespace

static int far_cols(int64_t n) { return n * n > 2 * kFieldThreads ? 4 : n * n > kFieldThreads ? 2 : 1; }

int64_t field_columns(bool far, int64_t n) { return far ? far_cols(n) * kFieldThreads : kFieldThreads; }

hipError_t launch_field(const FieldArgs& a, bool far, hipStream_t st) {
  hipError_t e = hipSuccess;
  if (a.n < 1 || a.n > kFieldMaxN || a.n * a.n * a.n != a.P) return hipErrorInvalidValue;  // the axis tables
  const int64_t cblocks = (a.n * a.n + field_columns(far, a.n) - 1) / field_columns(far, a.n);
  if (a.nch < 1 || a.nch > a.n || a.nparts != cblocks * a.nch || a.mb < 1 || a.nrhs > 65535) return hipErrorInvalidValue;
  auto grid = [&](int mp) {
    return dim3(static_cast<unsigned>(a.nparts), static_cast<unsigned>((a.mb + mp - 1) / mp),
                static_cast<unsigned>(a.nrhs));
  };
  const bool wide = a.nparts * ((a.mb + 3) / 4) * a.nrhs >= 1024;
  const unsigned row = static_cast<unsigned>(3 * a.n * sizeof(cxd));  // far: LDS per point
  if (far && far_cols(a.n) == 1)
    e = launch_kernel_smem(k_field_far<4, 1>, grid(4), dim3(kFieldThreads), 4 * row, st, a);
  else if (far && far_cols(a.n) == 2)
    e = launch_kernel_smem(k_field_far<4, 2>, grid(4), dim3(kFieldThreads), 4 * row, st, a);
  else if (far && a.n <= kFieldMaxN / 2)
    e = launch_kernel_smem(k_field_far<4, 4>, grid(4), dim3(kFieldThreads), 4 * row, st, a);
  else if (far)
    e = launch_kernel_smem(k_field_far<2, 4>, grid(2), dim3(kFieldThreads), 2 * row, st, a);
  else if (wide)
    e = launch_kernel(k_field_near<4>, grid(4), dim3(kFieldThreads), st, a);
  else
    e = launch_kernel(k_field_near<1>, grid(1), dim3(kFieldThreads), st, a);
  if (e != hipSuccess) return e;
  e = launch_kernel(k_field_finalize, dim3(static_cast<unsigned>((a.mb + 63) / 64), static_cast<unsigned>(a.nrhs)),
                     dim3(64), st, a, far ? 1 : 0);
  return e;
}

hipError_t launch_charges(const void* D, const void* u, int64_t P, int64_t nrhs, void* q, hipStream_t st) {
  hipError_t e = hipSuccess;
  int64_t g = (P + 255) / 256;
  if (g > 8192) g = 8192;
  e = launch_kernel(k_charges, dim3(static_cast<unsigned>(g), static_cast<unsigned>(nrhs)), dim3(256), st,
                     static_cast<const cxd*>(D), static_cast<const cxd*>(u), P, static_cast<cxd*>(q));
  return e;
}

int64_t refraction_blocks(int64_t P) {
  const int64_t g = (P + 255) / 256;
  return g < 1 ? 1 : (g > 1024 ? 1024 : g);
}

hipError_t launch_refraction(const RefractionArgs& a, hipStream_t st) {
  hipError_t e = hipSuccess;
  e = launch_kernel(k_refraction, dim3(static_cast<unsigned>(refraction_blocks(a.P))), dim3(256), st, a);
  return e;
}

int64_t max_blocks(int64_t P) {
  const int64_t g = (P + 255) / 256;
  return g < 1 ? 1 : (g > 1024 ? 1024 : g);
}

hipError_t launch_cell_difference(const DiffArgs& a, int64_t P_coarse, double* part, hipStream_t st) {
  hipError_t e = hipSuccess;
  e = launch_kernel(k_cell_difference, dim3(static_cast<unsigned>(P_coarse)), dim3(kFieldThreads), st, a);
  if (e != hipSuccess) return e;
  e = launch_kernel(k_max, dim3(static_cast<unsigned>(max_blocks(P_coarse))), dim3(256), st, a.means, P_coarse,
                     part);
  return e;
}

}  // namespace ori
