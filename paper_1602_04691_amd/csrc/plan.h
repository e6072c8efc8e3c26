// FFT plans for the padded length L = 2n of each axis (Section 3 pads every
// axis before the convolution theorem, eq. 3.3.8).  Shared by host and device
// code: everything here is constexpr.
#pragma once

#include <cstdint>

namespace ori {

// Every supported padded length, one translation unit of FFT kernels each.
#define ORI_FOR_EACH_L(X) \
  X(2) X(4) X(6) X(8) X(10) X(12) X(16) X(20) X(24) X(32) X(40) X(48) X(64) X(72) X(80) X(96) \
  X(100) X(108) X(128) X(144) X(160) X(192) X(200) X(216) X(256) X(288) X(320) X(360) \
  X(384) X(400) X(432) X(512) X(576) X(640) X(720) X(768) X(1024)

// The lengths whose work arrays a context reserves: the shortest of these
// with L >= 2n - 1 sizes its workspace, so that ori_workspace_bytes, which
// callers budget with, does not depend on the plan the passes run.  These
// lengths also have the Z pass's prefetch variant.
#define ORI_FOR_EACH_RESERVED_L(X) \
  X(2) X(4) X(6) X(8) X(10) X(12) X(16) X(20) X(24) X(32) X(40) X(48) X(64) X(80) X(96) \
  X(128) X(192) X(256) X(384) X(512) X(1024)

constexpr bool reserved_length(int L) {
  switch (L) {
#define ORI_RESERVED(Lv) case Lv:
    ORI_FOR_EACH_RESERVED_L(ORI_RESERVED)
#undef ORI_RESERVED
    return true;
    default:
      return false;
  }
}

struct RadixPlan {
  int n;     // number of Stockham stages
  int r[4];  // forward radix order; the inverse runs them in reverse
};

// The first forward radix is even so that the zero upper half of a padded
// input is skipped at compile time.  Radix 8 is the sweet spot on gfx950 in
// complex128: 8 values (32 VGPRs) per butterfly leave room for the spectrum
// and twiddles of the fused Z pass at 4 waves per SIMD, where radix 16 needs
// over 200 VGPRs.  L = 16 is 4 x 4 (four threads per pencil), so that its
// pass bodies fit the register budget of the multi-problem launches.
//
// The lengths between the powers of two (72, 100, 108, 144, ... 768)
// keep an n whose 2n is not planned from paying for the next power of two
// (n = 300 on L = 640 instead of 1024 transforms 2.6 times fewer points).
// They use radices 6, 9, 10 and 12 to stay at two or three stages; the first
// radix is even, and the last is 8 or smaller where the length allows it,
// because the spectrum of the fused Z pass is held in registers in the shape
// of the last stage.  Plans that read the same both ways (8 x 2 x 8) need one
// twiddle table for both directions of the Z pass and begin its inverse with
// the radix 8 butterfly that absorbs the spectrum product: complex64 Z of n =
// 64 with 32 right-hand sides 0.114 -> 0.106 ms against 8 x 4 x 4 on wide
// tiles, complex128 Z of n = 96 36.4 -> 31.8 us against 8 x 8 x 3, of n = 128
// 77.9 -> 71.8 us against 8 x 8 x 4.
constexpr RadixPlan radix_plan(int L) {
  switch (L) {
    case 2: return {1, {2, 0, 0, 0}};
    case 4: return {1, {4, 0, 0, 0}};
    case 6: return {2, {2, 3, 0, 0}};
    case 8: return {1, {8, 0, 0, 0}};
    case 10: return {2, {2, 5, 0, 0}};
    case 12: return {2, {4, 3, 0, 0}};
    case 16: return {2, {4, 4, 0, 0}};
    case 20: return {2, {4, 5, 0, 0}};
    case 24: return {2, {8, 3, 0, 0}};
    case 32: return {2, {8, 4, 0, 0}};
    case 40: return {2, {8, 5, 0, 0}};
    case 48: return {2, {8, 6, 0, 0}};
    case 64: return {2, {8, 8, 0, 0}};
    case 72: return {2, {8, 9, 0, 0}};
    case 80: return {2, {8, 10, 0, 0}};
    case 96: return {2, {8, 12, 0, 0}};
    case 100: return {2, {10, 10, 0, 0}};
    case 108: return {2, {12, 9, 0, 0}};
    case 128: return {3, {8, 2, 8, 0}};
    case 144: return {2, {12, 12, 0, 0}};
    case 160: return {3, {4, 10, 4, 0}};
    case 192: return {3, {8, 3, 8, 0}};
    case 200: return {3, {10, 2, 10, 0}};
    case 216: return {3, {6, 6, 6, 0}};
    case 256: return {3, {8, 4, 8, 0}};
    case 288: return {3, {6, 8, 6, 0}};
    case 320: return {3, {8, 5, 8, 0}};
    case 360: return {3, {6, 10, 6, 0}};
    case 384: return {3, {8, 6, 8, 0}};
    case 400: return {3, {10, 4, 10, 0}};
    case 432: return {3, {8, 9, 6, 0}};
    case 512: return {3, {8, 8, 8, 0}};
    case 576: return {3, {8, 9, 8, 0}};
    case 640: return {3, {8, 10, 8, 0}};
    case 720: return {3, {10, 9, 8, 0}};
    case 768: return {3, {8, 12, 8, 0}};
    case 1024: return {4, {8, 8, 4, 4}};
    default: return {0, {0, 0, 0, 0}};
  }
}

// Alternative plans of the fused Z pass (its radix-plan knob, `zplan`):
// variant 1 factors L into another radix order, or other radices, with the
// same threads per pencil (the smallest butterfly count of a stage), so
// that the Z workgroup shape is unchanged; the first radix stays even.  At
// L = 1024 variant 1 is 16 x 8 x 8: two exchanges per transform instead of
// three with the same 64 threads per pencil (complex128 Z 6.04 vs 6.52 ms
// at n = 512, its default there; 8 x 16 x 8 on 128 threads, whose 122
// registers allow twice the wavefronts, takes 6.60 ms).  Lengths without an
// alternative (L = 64 and most short ones) have variant 1 equal to the
// default.
//
// Variant 2 is not a layout choice: at L = 1024 the complex128 strided passes
// and the complex64 Z pass run 8 x 16 x 8 on 64 threads per pencil, two exchanges per
// transform instead of three (every other length: the default).
constexpr RadixPlan radix_plan(int L, int variant) {
  if (variant == 2 && L == 1024) return {3, {8, 16, 8, 0}};
  if (variant == 1) switch (L) {
      case 32: return {2, {4, 8, 0, 0}};
      case 48: return {3, {8, 2, 3, 0}};
      case 80: return {3, {8, 2, 5, 0}};
      case 96: return {3, {8, 4, 3, 0}};
      case 128: return {3, {8, 4, 4, 0}};
      case 192: return {3, {8, 8, 3, 0}};
      case 256: return {3, {8, 8, 4, 0}};
      case 384: return {4, {8, 3, 4, 4}};
      case 512: return {4, {8, 4, 4, 4}};
      case 1024: return {3, {16, 8, 8, 0}};
      default: break;
    }
  return radix_plan(L);
}

constexpr bool same_plan(const RadixPlan& a, const RadixPlan& b) {
  if (a.n != b.n) return false;
  for (int s = 0; s < a.n; ++s)
    if (a.r[s] != b.r[s]) return false;
  return true;
}

// whether the Z pass has a second plan at L
constexpr bool has_plan_variant(int L) { return !same_plan(radix_plan(L, 1), radix_plan(L)); }

constexpr bool supported_length(int L) { return radix_plan(L).n > 0; }

// Butterflies of one pencil in the stage with the fewest and the most.
constexpr int fewest_butterflies(int L, const RadixPlan& p) {
  int t = L;
  for (int s = 0; s < p.n; ++s)
    if (L / p.r[s] < t) t = L / p.r[s];
  return t;
}
constexpr int most_butterflies(int L, const RadixPlan& p) {
  int t = 0;
  for (int s = 0; s < p.n; ++s)
    if (L / p.r[s] > t) t = L / p.r[s];
  return t;
}

// Threads per pencil: the smallest butterfly count over the stages, so that
// no stage leaves threads idle in its widest configuration, capped at two
// wavefronts (L = 1024: one radix-8 butterfly per thread keeps a complex128
// thread within 128 registers).  The lengths between the reserved ones take
// the largest count where the counts lie close together (L = 640: 80, 64,
// 80): one butterfly per thread and stage holds half the registers of a
// second, mostly empty round, and the threads without a butterfly are whole
// wavefronts of the strided passes, which skip the stage.  Exceptions (one
// product, us; R right-hand sides):
//  - L = 160 (40, 16, 40) takes 20, between 16 and 40: n = 80 complex128 81.9
//    against 77.8 (16) and 82.0 (40), complex64 53.9 against 55.5 and 55.5, n =
//    75 76.4, 76.7, 80.0 and 53.4, 56.1, 54.4, n = 80 with R = 8 401, 393, 454
//    and 201, 205, 223.
//  - L = 80 and 96 take L / 8 and not 8, which keeps the Z tile for both of
//    their plans: n = 40 36.1 against 38.3 and 32.8 against 34.3 (R = 8 70.8
//    against 67.7 and 47.8 against 49.3), n = 48 41.9 against 43.8 and 35.7
//    against 37.0 (R = 8 86.2 against 94.2 and 60.2 against 62.3).
//  - L = 320 (40, 64, 40) takes 40: complex64 is 1 % faster than on 64 (n = 160
//    222 against 225), complex128 7 % slower (442 against 412), and both share
//    the count.
constexpr int threads_per_pencil(int L, int variant = 0) {
  const RadixPlan p = radix_plan(L, variant);
  if (L == 160) return 20;  // 40, 16, 40
  if (L == 80 || L == 96) return L / 8;  // 10, 8 and 12, 8
  const int lo = fewest_butterflies(L, p), hi = most_butterflies(L, p);
  if (!reserved_length(L) && hi <= 2 * lo && hi != 64) return hi;
  return lo > 128 ? 128 : lo;
}

constexpr int pow2_floor(int x) {
  int p = 1;
  while (p * 2 <= x) p *= 2;
  return p;
}

// Pencils per workgroup.  Strided passes need several adjacent pencils per
// row so that each row read/written is a contiguous run (8 x 16 B = 128 B for
// complex128, 16 x 8 B for complex64); contiguous passes only need enough
// threads to fill the workgroup.
// Workgroups are whole wavefronts (64 lanes): the reductions use full-wave
// shuffles.  block_threads rounds NP pencils up to whole wavefronts; the
// lanes beyond NP * TPP own no butterfly (Engine's IDLE).  More pencils are
// taken while more than an eighth of the lanes would idle.
constexpr int block_threads(int threads) { return (threads + 63) / 64 * 64; }
constexpr int whole_waves(int np, int tpp) {
  while ((block_threads(np * tpp) - np * tpp) * 8 > block_threads(np * tpp) && block_threads(2 * np * tpp) <= 1024)
    np *= 2;
  return np;
}

constexpr int pencils_strided(int L, int elem_bytes) {
  int tpp = threads_per_pencil(L);
  int np = pow2_floor(256 / tpp);
  int lo = elem_bytes == 16 ? 8 : 16;
  if (np < lo) np = lo;
  if (np > 64) np = 64;
  while (np > 1 && np * tpp > 1024) np /= 2;  // at most 1024 threads per workgroup
  return whole_waves(np, tpp);
}

// LDS slots of one padded contiguous pencil row
constexpr int padded_row(int L) { return L + L / 8; }

// Contiguous passes of the lengths between the reserved ones take fewer
// pencils and up to a fifth of idle lanes: their rows need no neighbours, and
// half the LDS per workgroup (25 instead of 51 KB at L = 400) keeps twice the
// workgroups resident.
constexpr int pencils_contig(int L) {
  int tpp = threads_per_pencil(L);
  int np = pow2_floor(256 / tpp);
  if (np < 1) np = 1;
  if (reserved_length(L) || (block_threads(np * tpp) - np * tpp) * 5 > block_threads(np * tpp))
    np = whole_waves(np, tpp);
  // complex128 rows within the 64 KB of dynamic LDS of a multi-problem launch
  while (L <= 256 && np * padded_row(L) * 16 > 64 * 1024) np /= 2;
  return np;
}

}  // namespace ori
