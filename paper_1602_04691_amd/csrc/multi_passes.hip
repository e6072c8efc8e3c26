// One FFT pass of several problems of different padded lengths in one
// launch (the uneven batch of independent problems; kernels.h, MultiProblem).
// Every length of multi_length() has its pass bodies compiled here, in a
// namespace of its own, from the same source as its single-problem kernels
// (pass_bodies.inc), with the tile shape of kernels.h; a launch runs each
// problem's workgroups on its own length's body.  Compiled once per precision
// and set of lengths (-DORI_MULTI_PREC=64 or 32, -DORI_MULTI_ALL=0 or 1).
#include "fft_engine.h"
#include "kernels.h"
#include "launch.h"
#include "pass_common.h"

#if !defined(ORI_MULTI_PREC) || (ORI_MULTI_PREC != 64 && ORI_MULTI_PREC != 32) || !defined(ORI_MULTI_ALL)
#error "compile with -DORI_MULTI_PREC=64 and 32, -DORI_MULTI_ALL=0 and 1"
#endif

namespace ori {

namespace ml8 {
constexpr int L = 8;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml8

namespace ml10 {
constexpr int L = 10;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml10

namespace ml12 {
constexpr int L = 12;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml12

namespace ml16 {
constexpr int L = 16;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml16

namespace ml20 {
constexpr int L = 20;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml20

namespace ml24 {
constexpr int L = 24;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml24

namespace ml32 {
constexpr int L = 32;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml32

namespace ml40 {
constexpr int L = 40;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml40

namespace ml48 {
constexpr int L = 48;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml48

namespace ml64 {
constexpr int L = 64;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml64

namespace ml80 {
constexpr int L = 80;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml80

namespace ml96 {
constexpr int L = 96;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml96

namespace ml128 {
constexpr int L = 128;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml128

namespace ml192 {
constexpr int L = 192;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml192

namespace ml256 {
constexpr int L = 256;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml256

#if ORI_MULTI_ALL
namespace ml72 {
constexpr int L = 72;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml72

namespace ml100 {
constexpr int L = 100;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml100

namespace ml108 {
constexpr int L = 108;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml108

namespace ml144 {
constexpr int L = 144;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml144

namespace ml160 {
constexpr int L = 160;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml160

namespace ml200 {
constexpr int L = 200;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml200

namespace ml216 {
constexpr int L = 216;
#include "pass_bodies.inc"
#include "multi_len.inc"
}  // namespace ml216
#endif

// The lengths of this translation unit: every length with multi-problem
// bodies (multi_length in kernels.h), or the reserved ones alone.  The
// lengths between them need more registers (complex128 I1 114 instead of 90,
// I2 116 instead of 78, Z 172 instead of 152), which every workgroup of a
// launch pays for, so a set of problems without such a length runs kernels
// without their bodies (complex128, n = 32, 48, 64, 96: 4.02 vs 4.11 ms, n =
// 48, 96 twice 5.68 vs 5.80 ms).
#define ORI_MULTI_RESERVED(X) X(8) X(10) X(12) X(16) X(20) X(24) X(32) X(40) X(48) X(64) X(80) X(96) X(128) X(192) X(256)
#if ORI_MULTI_ALL
#define ORI_MULTI_LENGTHS(X) ORI_MULTI_RESERVED(X) X(72) X(100) X(108) X(144) X(160) X(200) X(216)
#else
#define ORI_MULTI_LENGTHS(X) ORI_MULTI_RESERVED(X)
#endif

namespace {

#define ORI_MULTI_CHECK(Lv) static_assert(multi_length(Lv), "length without multi-problem bodies");
ORI_MULTI_LENGTHS(ORI_MULTI_CHECK)
#undef ORI_MULTI_CHECK

template <typename T, int PASS>
constexpr int max_threads() {
  int t = 0;
#define ORI_MT(Lv) t = ml##Lv::mp_threads<T, PASS>() > t ? ml##Lv::mp_threads<T, PASS>() : t;
  ORI_MULTI_LENGTHS(ORI_MT)
#undef ORI_MT
  return t;
}

// Waves per SIMD that the complex128 kernels with the lengths between the
// reserved ones keep: Z three, the other passes five.  By themselves they
// take 172 (Z, two waves) and 104 to 116 registers (four); held, they spill 2
// and 40 to 58.  Neither is better for all sets (ms, held and without a
// spill: four n = 72 5.07 and 4.68, n = 33, 50, 70, 100 6.12 and 5.88, n = 100
// twice 6.46 and 6.48, eight n = 36 3.49 and 3.64, n = 54, 80, 108 6.88 and
// 7.28).  The kernels without those lengths keep what they take, F1 116 and
// F2 100 (L = 96 as 8 x 12, four waves): five waves there, by spilling or
// with L = 96 as 8 x 4 x 3, are within 1 % (n = 32, 48, 64, 96 4.02 and 4.01
// to 4.04), and 8 x 4 x 3 is slower alone (n = 48 product 42.3 vs 43.9 us).
template <typename T, int PASS>
constexpr int multi_min_waves() {
  return ORI_MULTI_ALL && sizeof(T) == 8 ? (PASS == MP_Z ? 3 : 5) : 1;
}

// Launch workgroup b runs workgroup b - first_block of the problem whose
// range holds it (problems in ascending first_block), on its length's body.
// The LDS is dynamic: the largest the launch's problems need.
template <typename T, int PASS>
__global__ void __launch_bounds__((max_threads<T, PASS>()), (multi_min_waves<T, PASS>())) k_multi_pass(const MultiProblem* __restrict__ tab,
                                                                       int32_t np) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int64_t b = blockIdx.x;
  int p = 0;
  while (p + 1 < np && tab[p + 1].first_block <= b) ++p;
  const MultiProblem m = tab[p];
  const int64_t bid = b - m.first_block;
  switch (m.L) {
#define ORI_MC(Lv)                                \
  case Lv:                                        \
    ml##Lv::mp_run<T, PASS>(m, bid, smem);        \
    break;
    ORI_MULTI_LENGTHS(ORI_MC)
#undef ORI_MC
    default:
      break;
  }
}

// dynamic LDS of a launch: within the 64 KB a launch gets without asking
constexpr int kMaxDynSmem = 64 * 1024;

template <typename T, int PASS>
hipError_t launch_t(const MultiProblem* tab, int32_t np, int64_t blocks, int threads, int smem, hipStream_t st) {
  if (threads < 64 || threads > max_threads<T, PASS>() || threads % 64 != 0) return hipErrorInvalidValue;
  if (smem < 0 || smem > kMaxDynSmem) return hipErrorInvalidValue;
  return launch_kernel_smem(k_multi_pass<T, PASS>, dim3(static_cast<unsigned>(blocks)), dim3(threads),
                            static_cast<unsigned>(smem), st, tab, np);
}

template <typename T>
hipError_t launch_prec(int pass, const MultiProblem* tab, int32_t np, int64_t blocks, int threads, int smem,
                       hipStream_t st) {
  if (np < 1 || blocks < 1) return hipErrorInvalidValue;
  switch (pass) {
    case MP_F1: return launch_t<T, MP_F1>(tab, np, blocks, threads, smem, st);
    case MP_F2: return launch_t<T, MP_F2>(tab, np, blocks, threads, smem, st);
    case MP_Z: return launch_t<T, MP_Z>(tab, np, blocks, threads, smem, st);
    case MP_I2: return launch_t<T, MP_I2>(tab, np, blocks, threads, smem, st);
    case MP_I1: return launch_t<T, MP_I1>(tab, np, blocks, threads, smem, st);
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
int smem_prec(int L, int pass) {
  switch (L) {
#define ORI_SM(Lv)                                                                \
  case Lv:                                                                        \
    switch (pass) {                                                               \
      case MP_F1: return ml##Lv::mp_smem<T, MP_F1>();                             \
      case MP_F2: return ml##Lv::mp_smem<T, MP_F2>();                             \
      case MP_Z: return ml##Lv::mp_smem<T, MP_Z>();                               \
      case MP_I2: return ml##Lv::mp_smem<T, MP_I2>();                             \
      case MP_I1: return ml##Lv::mp_smem<T, MP_I1>();                             \
      default: return 0;                                                          \
    }
    ORI_MULTI_LENGTHS(ORI_SM)
#undef ORI_SM
    default:
      return 0;
  }
}

#define ORI_SMEM_CHECK(Lv)                                                                              \
  static_assert(ml##Lv::mp_smem<double, MP_F1>() <= kMaxDynSmem && ml##Lv::mp_smem<double, MP_Z>() <= kMaxDynSmem && \
                    ml##Lv::mp_smem<double, MP_F2>() <= kMaxDynSmem,                                     \
                "multi-problem LDS above 64 KB");
ORI_MULTI_LENGTHS(ORI_SMEM_CHECK)
#undef ORI_SMEM_CHECK

template <typename T>
int threads_prec(int L, int pass) {
  switch (L) {
#define ORI_TH(Lv)                                                                \
  case Lv:                                                                        \
    switch (pass) {                                                               \
      case MP_F1: return ml##Lv::mp_threads<T, MP_F1>();                          \
      case MP_F2: return ml##Lv::mp_threads<T, MP_F2>();                          \
      case MP_Z: return ml##Lv::mp_threads<T, MP_Z>();                            \
      case MP_I2: return ml##Lv::mp_threads<T, MP_I2>();                          \
      case MP_I1: return ml##Lv::mp_threads<T, MP_I1>();                          \
      default: return 0;                                                          \
    }
    ORI_MULTI_LENGTHS(ORI_TH)
#undef ORI_TH
    default:
      return 0;
  }
}

}  // namespace

#define ORI_CAT2(a, b, c, d) a##b##c##d
#define ORI_CAT(a, b, c, d) ORI_CAT2(a, b, c, d)
#define ORI_MULTI_TABLE ORI_CAT(multi_kernels_f, ORI_MULTI_PREC, _, ORI_MULTI_ALL)
using MT = std::conditional_t<ORI_MULTI_PREC == 64, double, float>;

const MultiKernels* ORI_MULTI_TABLE() {
  static const MultiKernels k = {threads_prec<MT>, smem_prec<MT>, launch_prec<MT>};
  return &k;
}

}  // namespace ori
