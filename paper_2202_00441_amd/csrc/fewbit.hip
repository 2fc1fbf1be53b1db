// fewbit.hip -- gfx950 kernels and C ABI of the few-bit activation path.
//
// Forward (Listing 1, forward; Eq. (2)): y = f(x) plus, for every element,
// the index of the interval of the piecewise-constant approximation of f'
// it falls in, packed densely at `bits` bits per element.
// Backward (Eq. (1) with f' replaced by the approximation; Listing 1,
// backward): grad_in = grad_out * v[idx].
//
// Both passes are pointwise and bound by HBM bandwidth.  Work is cut into
// wave tiles of 512 consecutive elements, whose codes are exactly 16*b whole
// words, and every 16-byte access instruction of a wave covers 1 KiB of
// contiguous memory.  fp16 / bf16: each lane owns 8 consecutive elements
// (one 16-byte access); their 8 codes make a b-byte field, and the fields
// of 4 neighbouring lanes (one DPP quad) always cover whole words, so lanes
// combine fields with quad permutes instead of atomics or shared memory.
// fp32: a tile is two halves of 256 and each lane owns 4 consecutive
// elements of each half (one 16-byte access per half); the words are then
// gathered from 4b-bit lane fields by cross-lane reads (see fp32 tiles).
// Each packed word has one value, written by its lane (and by lanes that
// store an identical copy, so that full tiles need no masking).
//
// Streams are read and written with 16-byte buffer accesses, read
// non-temporally (nothing is reused).  Most kernels run one wave per tile and
// let the hardware dispatcher balance the compute units; the forward with
// full-range tables is persistent (see the launch-shape knobs below).
//
// fp16 / bf16 forward.  Output pattern and interval index are functions of
// the 16-bit input pattern alone.  bf16 (fwd16_kernel): the few thousand
// patterns on which an activation is neither linear nor constant have one LDS
// word each, from which output and index both follow.  fp16, and bf16 tables
// whose boundaries that range does not hold (fwd16full_kernel): each workgroup
// looks both up in LDS tables over all 65536 patterns, which it builds itself.
// Forwards below a size that depends on type, activation and bit width
// (tab_by_size, kTableMinLog2), and every fp32 forward, evaluate f and search
// the boundaries per element.
//
// The fitted table travels as kernel arguments (scalar registers); the
// backward spreads the values over the lanes of one register and reads
// them with cross-lane permutes.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>

#include "../../include/fewbit.h"
#include "fwd16_out.h"
#include "fwd16_rules.h"

// Launch-shape knobs of the full-range table forward (compile time): threads
// per workgroup, workgroups per CU, and tiles per wave and loop trip.  It holds
// 160 KiB of tables per workgroup (all of a CU's LDS), built at its start, so
// it is persistent with one workgroup per CU, whose waves walk the tiles; it
// ends only when its slowest compute unit has walked its share.  Every other
// kernel launches its waves once, and the dispatcher hands out workgroups as
// earlier ones finish, which balances the load between compute units, whose
// streaming rates differ by a few per cent.
#ifndef FEWBIT_FWD16_THREADS
#define FEWBIT_FWD16_THREADS 512
#endif
#ifndef FEWBIT_FWD16_WG_PER_CU
#define FEWBIT_FWD16_WG_PER_CU 1
#endif
#ifndef FEWBIT_FWD16_UNROLL
#define FEWBIT_FWD16_UNROLL 4
#endif

namespace {

constexpr int kWave = 64;
constexpr int kPerLane = 8;                 // elements per lane per 16-bit tile
constexpr int kTile = kWave * kPerLane;     // 512 elements per wave tile
constexpr uint32_t kLaneBytes = 16;         // one 16-byte access per lane and instruction
constexpr uint32_t kSpanBytes = kWave * kLaneBytes;   // 1 KiB per wave instruction

struct TableArgs {
  float s[15];
  float v[16];
};

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// Stream accesses go through buffer instructions on a wave-uniform span: a
// resource descriptor for `bytes` bytes from a wave-uniform address (scalar
// registers), plus a per-lane byte offset.  The cache policy is explicit in
// every instruction (the non-temporal hint of plain loads and stores can be
// dropped by the compiler when it merges or moves them), and the hardware
// range check turns any access at or past `bytes` into a zero load or a
// dropped store.
//
// Cache-policy bits: 2 = nt (streaming, not kept in cache), 16 = sc1 (device
// scope: a store is written through the L2).  Loads are nt.  Stores are nt
// alone, or through, or both, by the size of the tensor (store_nt); the two
// table forwards store both ways at every size (launch_tab).
constexpr int kNt = 2, kThrough = 16, kThroughNt = 18;

struct Span {
  __amdgpu_buffer_rsrc_t r;
  // 0x00020000: raw (unformatted) 32-bit buffer accesses on gfx9
  __device__ Span(const void* base, uint32_t bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, static_cast<int>(bytes), 0x00020000)) {}
  __device__ u32x4_t ld16(uint32_t off) const { return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, kNt); }
  __device__ uint32_t ld4(uint32_t off) const { return __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, kNt); }
  __device__ uint32_t ld2(uint32_t off) const { return __builtin_amdgcn_raw_buffer_load_b16(r, off, 0, kNt); }
};

// A span that is stored to with the cache policy P.  Code words are never
// kThroughNt: they are what the backward reads, and plain write-through leaves
// them in the memory-side cache while there is room.  (A policy chosen at run
// time, one scalar branch a store, cost every small launch 0.2 us.)
template <int P>
struct OutSpan : Span {
  using Span::Span;
  __device__ void st16(uint32_t off, u32x4_t v) const { __builtin_amdgcn_raw_buffer_store_b128(v, r, off, 0, P); }
  __device__ void st4(uint32_t off, uint32_t v) const {
    __builtin_amdgcn_raw_buffer_store_b32(v, r, off, 0, P == kThroughNt ? kThrough : P);
  }
};

// The partial tile at the end goes element by element through this and Span's
// ld2 / ld4, on a span of the elements that exist: the range check drops the
// others, so there is no branch per element, all of a lane's loads are in
// flight together, and every line is stored with the launch's policy.  (With
// guarded plain accesses the eight loads of a lane followed one another, and
// the tile's lines stayed dirty in the L2 whatever the policy: the launch
// waited for the writing through and for the write-back at its end.  12 layers
// of 2^18 - 1 elements with their backwards in a graph, against this: fp32
// Sigmoid 4 bits 87.2 -> 59.0 us, bf16 GELU 3 bits 77.1 -> 57.0.)
template <int P>
struct OutElements : Span {
  using Span::Span;
  __device__ void st2(uint32_t off, uint32_t v) const {
    __builtin_amdgcn_raw_buffer_store_b16(static_cast<uint16_t>(v), r, off, 0, P);
  }
  __device__ void st4(uint32_t off, uint32_t v) const { __builtin_amdgcn_raw_buffer_store_b32(v, r, off, 0, P); }
};

// ---------------------------------------------------------------- storage
// Half types: two elements per 32-bit word, element 2k in the low half.
template <int DT>
struct Half;

template <>
struct Half<FEWBIT_BF16> {
  // bfloat16 is the upper half of a binary32: widening is a shift
  __device__ static float lo(uint32_t u) { return __uint_as_float(u << 16); }
  __device__ static float hi(uint32_t u) { return __uint_as_float(u & 0xFFFF0000u); }
  __device__ static float widen(uint32_t bits16) { return __uint_as_float(bits16 << 16); }
  // round to nearest even (v_cvt_pk_bf16_f32)
  __device__ static uint32_t pack(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){a, b}, bf16x2_t));
  }
  // magnitudes from here up: exponent all ones (infinity, NaNs)
  static constexpr uint32_t kSpecialFrom = 0x7F80u;
};

template <>
struct Half<FEWBIT_F16> {
  __device__ static float lo(uint32_t u) {
    return static_cast<float>(__builtin_bit_cast(f16x2_t, u).x);
  }
  __device__ static float hi(uint32_t u) {
    return static_cast<float>(__builtin_bit_cast(f16x2_t, u).y);
  }
  __device__ static float widen(uint32_t bits16) {
    return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(bits16)));
  }
  // Round to nearest even from the fp32 value.  The operands pass an empty
  // register barrier first: without it the compiler may fuse the multiply
  // or FMA that produced them into one mixed-precision FMA rounded straight
  // to fp16, which rounds once instead of twice and turns -0 into +0.
  __device__ static uint32_t pack(float a, float b) {
    asm("" : "+v"(a), "+v"(b));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){a, b}, f16x2_t));
  }
  static constexpr uint32_t kSpecialFrom = 0x7C00u;
};

// ---------------------------------------------------------------- activations
// f evaluated in fp32 with hardware exp2 / reciprocal.  x*Phi(x) and
// x*sigmoid(x) are formed as relu(x) - |x| * tail(|x|), tail the upper tail
// probability, which keeps full relative accuracy on the negative side down
// to the subnormals.
//
// The hardware exponential returns no subnormals (results below 2^-126 come
// back as 0), so each exponential is taken of an argument raised by S and
// the factor 2^S is taken back out of the partner operand of the final
// product, which costs nothing: for GELU out of the reciprocal (its
// constants carry 2^S), for SiLU and sigmoid out of the denominator.  S is
// the smallest shift that keeps every product representable in the output
// type (fp16 outputs underflow long before 2^-126, so S = 0 there).
//
// In the product |x| * tail, |x| is clamped to the largest finite float:
// for x = +-inf the other factor is exactly 0 and the product is 0 (not
// inf * 0), so f(x) = relu(x) without a separate branch; NaN still reaches
// the result through the exponential's argument, which is not clamped.
__device__ inline float finite_abs(float x) { return fminf(fabsf(x), 3.4028234663852886e38f); }

// max(x, -0) as one integer op: the unsigned minimum with the bits of -0
// keeps every float with the sign bit clear (+inf, NaN included) and maps
// every negative input to -0.
__device__ inline float relu(float x) {
  return __uint_as_float(min(__float_as_uint(x), 0x80000000u));
}

// 2^e for -1022 <= e <= 1023, from the exponent field
constexpr double pow2(int e) {
  return __builtin_bit_cast(double, static_cast<uint64_t>(1023 + e) << 52);
}

template <int N>
struct Coefs {
  float c[N];
};

// GELU: the normal upper tail Q(t) = P(Z > t) = r exp2(c(r) - t^2/(2 ln 2))
// with r = 1/(1 + p t) and c a polynomial in r (the form of the Chebyshev
// fitted erfc of Numerical Recipes, coefficients fitted here for a minimal
// maximum relative error on t in [0, 15]):
//   degree 3: max rel. error 1.9e-4  (bf16 results: within 1 ulp)
//   degree 4: max rel. error 5.5e-5  (fp16 results: within 1 ulp)
//   degree 6: max rel. error 1.3e-6  (fp32 results: within 1e-5 rel / 2e-6 abs)
template <int DEG>
struct QFit;
template <>
struct QFit<3> {
  static constexpr float p = 0.36950944455033363f;
  static constexpr float c[4] = {-2.7541667327185095f, 1.3469623570975156f,
                                 0.9101290363759839f, -0.5032013588354882f};
};
template <>
struct QFit<4> {
  static constexpr float p = 0.5063964087913556f;
  static constexpr float c[5] = {-2.3043683184461905f, 1.3894173139728148f,
                                 0.6817571899264395f, -1.149862878045882f,
                                 0.38313433006936115f};
};
template <>
struct QFit<6> {
  static constexpr float p = 0.2715552190762726f;
  static constexpr float c[7] = {-3.204975453658058f, 1.4179583422514952f,
                                 0.7853715466157367f, -0.343943261631901f,
                                 1.2761535905064931f, -1.3184075229241483f,
                                 0.3878445554240053f};
};

// Per output type: GELU polynomial degree and the exponent shifts S.
template <int DT>
struct Prec {                       // fp32
  static constexpr int kGeluDeg = 6, kGeluS = 20, kSiluS = 32, kSigmoidS = 24;
};
template <>
struct Prec<FEWBIT_BF16> {
  static constexpr int kGeluDeg = 3, kGeluS = 16, kSiluS = 16, kSigmoidS = 16;
};
template <>
struct Prec<FEWBIT_F16> {
  static constexpr int kGeluDeg = 4, kGeluS = 0, kSiluS = 0, kSigmoidS = 0;
};

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kHalfLog2e = 0.7213475204444817f;   // 1/(2 ln 2)

template <int DT, int ACT>
struct Act;

template <int DT>
struct Act<DT, FEWBIT_GELU> {
  static constexpr int D = Prec<DT>::kGeluDeg, S = Prec<DT>::kGeluS;
  using F = QFit<D>;
  // coefficients of c in r' = 2^-S r: c_i 2^(S i), and c_0 + S (evaluated
  // at compile time: constant-initialised)
  static constexpr Coefs<D + 1> kCoef = [] {
    Coefs<D + 1> a{};
    for (int i = 0; i <= D; ++i)
      a.c[i] = i == 0 ? F::c[0] + static_cast<float>(S)
                      : static_cast<float>(static_cast<double>(F::c[i]) * pow2(S * i));
    return a;
  }();
  static constexpr float kP = static_cast<float>(F::p * pow2(S));
  static constexpr float kScale = static_cast<float>(pow2(S));
  __device__ static float f(float x) {
    const float t = finite_abs(x);
    const float rs = __builtin_amdgcn_rcpf(fmaf(t, kP, kScale));   // 2^-S r
    float c = kCoef.c[D];
#pragma unroll
    for (int i = D - 1; i >= 0; --i) c = fmaf(c, rs, kCoef.c[i]);
    const float e = __builtin_amdgcn_exp2f(fmaf(x * x, -kHalfLog2e, c));    // 2^S Q(t) / r
    return fmaf(-(t * rs), e, relu(x));   // relu(x) - t Q(t); NaN via x*x
  }
};

template <int DT>
struct Act<DT, FEWBIT_SILU> {
  static constexpr int S = Prec<DT>::kSiluS;
  __device__ static float f(float x) {
    const float e = __builtin_amdgcn_exp2f(fmaf(fabsf(x), -kLog2e, static_cast<float>(S)));  // 2^S e^-t
    constexpr float kScale = static_cast<float>(pow2(S));
    const float r = __builtin_amdgcn_rcpf(e + kScale);  // 1/(2^S (1 + e^-t))
    return fmaf(-(finite_abs(x) * e), r, relu(x));    // relu(x) - t sigma(-t); NaN via e
  }
};

// SiLU, fp16 outputs: x sigma(x) = x / (1 + e^-x) directly.  fp16 outputs
// below 2^-25 round to 0, long before e^-x overflows (x < -88), so the
// negative tail needs neither the split above nor a shift; x is raised to
// -FLT_MAX so that -inf gives -FLT_MAX * 0 = -0 (the limit), and a NaN still
// reaches the result through the exponential.  Six instructions instead of
// eight; every fp16 pattern within one unit in the last place.
template <>
struct Act<FEWBIT_F16, FEWBIT_SILU> {
  __device__ static float f(float x) {
    const float r = __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(x * -kLog2e));
    return fmaxf(x, -3.4028234663852886e38f) * r;
  }
};

template <int DT>
struct Act<DT, FEWBIT_SIGMOID> {
  static constexpr int S = Prec<DT>::kSigmoidS;
  __device__ static float f(float x) {
    const float t = fabsf(x);
    const float e = __builtin_amdgcn_exp2f(fmaf(t, -kLog2e, static_cast<float>(S)));  // 2^S e^-t
    constexpr float kScale = static_cast<float>(pow2(S));
    const float r = __builtin_amdgcn_rcpf(e + kScale);  // 1/(2^S (1 + e^-t))
    return ((x >= 0.0f) ? kScale : e) * r;   // NaN: e * r is NaN
  }
};

// tanh, every type: 1 - 2 / (e^(2|x|) + 1) with the hardware exponential and
// reciprocal (absolute error about 2^-22, so relative error below 2^-20 where
// |tanh| >= 0.245), and below |x| = 1/4, where that form loses relative
// accuracy, the odd Taylor series to x^9 (first omitted term below 1e-8
// relative), which keeps it down to the subnormals.  The sign is copied from
// x; NaN and infinities follow from the exponential.
template <int DT>
struct Act<DT, FEWBIT_TANH> {
  __device__ static float f(float x) {
    const float t = fabsf(x);
    const float e = __builtin_amdgcn_exp2f(t * (2.0f * kLog2e));
    const float big = fmaf(-2.0f, __builtin_amdgcn_rcpf(e + 1.0f), 1.0f);
    const float z = x * x;
    const float p = fmaf(z, fmaf(z, fmaf(z, fmaf(z, 62.0f / 2835.0f, -17.0f / 315.0f),
                                         2.0f / 15.0f), -1.0f / 3.0f), 1.0f);
    return copysignf(t < 0.25f ? t * p : big, x);
  }
};

template <int DT>
struct Act<DT, FEWBIT_RELU> {
  // +0 for every x <= 0 (-0 included); a NaN fails the compare and is kept
  __device__ static float f(float x) { return x <= 0.0f ? 0.0f : x; }
};

// Klambauer et al. (2017): lambda and lambda * alpha
constexpr float kSeluLambda = 1.0507009873554805f;
constexpr float kSeluLambdaAlpha = 1.7580993408473766f;

// SELU, 16-bit outputs: lambda x, or lambda alpha (e^x - 1) for x <= 0 with
// e^x - 1 taken from the hardware exponential from x = -1/4 down (there
// |e^x - 1| >= 0.22, so its absolute error of ~2^-23 is a relative one below
// 2^-20) and above -1/4 from the Taylor series to x^6 (first omitted term
// below 6e-8 relative), which keeps relative accuracy down to the
// subnormals.  NaN via the exponential; -inf gives -lambda alpha.
template <int DT>
struct Act<DT, FEWBIT_SELU> {
  __device__ static float f(float x) {
    const float e = __builtin_amdgcn_exp2f(x * kLog2e) - 1.0f;
    const float p = x * fmaf(x, fmaf(x, fmaf(x, fmaf(x, fmaf(x, 1.0f / 720.0f, 1.0f / 120.0f), 1.0f / 24.0f),
                                             1.0f / 6.0f), 0.5f), 1.0f);
    const float m = x > -0.25f ? p : e;
    return x > 0.0f ? kSeluLambda * x : kSeluLambdaAlpha * m;
  }
};
template <>
struct Act<FEWBIT_F32, FEWBIT_SELU> {
  // e^x - 1 from the hardware exponential: near 0 the subtraction cancels,
  // so the error is an absolute one of about 2^-23 (times lambda alpha), not
  // a relative one; the fp32 results stay well inside their tolerance (the
  // 16-bit form above adds the series near 0 that fp16 outputs need).  NaN
  // via the exponential, -inf gives -lambda alpha.
  __device__ static float f(float x) {
    const float e = __builtin_amdgcn_exp2f(x * kLog2e);
    return x > 0.0f ? kSeluLambda * x : kSeluLambdaAlpha * (e - 1.0f);
  }
};

// Softplus, 16-bit outputs: max(x, 0) + log(1 + u), u = e^-|x| in (0, 1]: no
// overflow, and relative accuracy in both tails.  log(1 + u) is ln 2 log2(1 + u)
// with the hardware log2 for u >= 2^-5 (rounding 1 + u costs at most 2^-24
// absolute, below 2^-18 relative there) and the series u (1 - u/2 + u^2/3 -
// u^3/4) below (first omitted term below 2^-22 relative).  The exponential is
// taken of an argument raised by S and the series' leading factor keeps the
// 2^S until the end, so bf16 outputs keep their relative accuracy down to
// the subnormals (u far below 2^-126).  NaN via the exponential; +inf gives
// +inf, -inf gives +0.
template <int DT>
struct Act<DT, FEWBIT_SOFTPLUS> {
  static constexpr int S = Prec<DT>::kSigmoidS;
  __device__ static float f(float x) {
    const float es = __builtin_amdgcn_exp2f(fmaf(fabsf(x), -kLog2e, static_cast<float>(S)));  // 2^S u
    constexpr float kUnscale = static_cast<float>(pow2(-S));
    const float u = es * kUnscale;
    const float series = (es * fmaf(u, fmaf(u, fmaf(u, -0.25f, 1.0f / 3.0f), -0.5f), 1.0f)) * kUnscale;
    const float viaLog = __builtin_amdgcn_logf(1.0f + u) * 0.6931471805599453f;
    return relu(x) + (u < 0x1p-5f ? series : viaLog);
  }
};
template <>
struct Act<FEWBIT_F32, FEWBIT_SOFTPLUS> {
  // The same split with hardware exp2 and log2: log(1 + e) = ln 2 log2(1 + e)
  // for e = e^-|x| in (0, 1].  Rounding 1 + e costs at most 2^-24 of
  // absolute error in log2, so the result is within ~2e-7 absolute of the
  // exact value (tiny outputs, x << 0, come back as absolute errors of that
  // size, not relative ones, which the fp32 tolerance allows; the 16-bit
  // form above keeps relative accuracy there).
  __device__ static float f(float x) {
    const float e = __builtin_amdgcn_exp2f(-fabsf(x) * kLog2e);
    return fmaf(__builtin_amdgcn_logf(1.0f + e), 0.6931471805599453f, relu(x));
  }
};

// ---------------------------------------------------------------- classify
// idx = number of boundaries s[m] <= x: half-open intervals [s[m-1], s[m]).
// IEEE compares: NaN gives 0, -0 == +0, subnormals are not flushed.
//
// Branch-free binary search over the sorted boundaries: level L tests the
// boundary s[idx + step - 1] (step = 2^(BITS-1-L)), chosen among the 2^L
// candidates by the answers of the levels before it (a select tree over
// scalar-register values), so BITS compares replace 2^BITS - 1.  A NaN fails
// every test and lands in interval 0, as with the count.
//
// The boundaries are first copied to scalar registers through an empty asm
// barrier: otherwise the compiler turns the selects into indexed loads from
// the kernel-argument block, a memory load per level and element.
struct Bounds {
  float s[15];
};

__device__ inline Bounds bounds_of(const TableArgs& tab) {
  Bounds b;
#pragma unroll
  for (int m = 0; m < 15; ++m) {
    float t = tab.s[m];
    asm("" : "+s"(t));
    b.s[m] = t;
  }
  return b;
}

template <int BITS, int L, int D, int K>
__device__ inline float pick_boundary(const bool (&c)[BITS], const Bounds& bd) {
  if constexpr (D == L) {
    constexpr int step = 1 << (BITS - 1 - L);
    return bd.s[K * 2 * step + step - 1];
  } else {
    return c[D] ? pick_boundary<BITS, L, D + 1, 2 * K + 1>(c, bd)
                : pick_boundary<BITS, L, D + 1, 2 * K>(c, bd);
  }
}

template <int BITS, int L = 0>
__device__ inline void search_levels(float x, const Bounds& bd, bool (&c)[BITS], uint32_t& idx) {
  if constexpr (L < BITS) {
    c[L] = x >= pick_boundary<BITS, L, 0, 0>(c, bd);
    idx += c[L] ? (1u << (BITS - 1 - L)) : 0u;
    search_levels<BITS, L + 1>(x, bd, c, idx);
  }
}

template <int BITS>
__device__ inline uint32_t classify(float x, const Bounds& bd) {
  bool c[BITS] = {};
  uint32_t idx = 0;
  search_levels<BITS>(x, bd, c, idx);
  return idx;
}

// The classification of the per-element kernels and of the code-table
// build.  Up to 3 bits it is the select tree above.  At 4 bits the tree's
// last level alone takes 7 selects, so there the boundaries are spread over
// the lanes of one register (lane i holds s[i], i < 15): the first level
// compares with the middle boundary, held in a scalar register, and each
// later level reads its boundary from the lane the search has reached with
// one cross-lane permute (ds_bpermute), ~3 VALU operations and one permute
// per level.  All 64 lanes must take part in every call (the permutes read
// other lanes).
template <int BITS>
struct Search {
  static constexpr uint32_t K = 1u << BITS;
  static constexpr bool kPermute = BITS == 4;
  Bounds bd;          // the select tree's boundaries (BITS <= 3)
  float mid;          // s[K/2 - 1]
  int lane_bound;     // s[lane] for lane < 15
  uint32_t keep;      // bits of x that are classified: all, or all but the sign
  __device__ Search(const TableArgs& tab, int lane, int symmetric)
      : bd(bounds_of(tab)), keep(symmetric ? 0x7FFFFFFFu : 0xFFFFFFFFu) {
    float v = 0.0f;
#pragma unroll
    for (int m = 0; m < 15; ++m) {
      v = (lane == m) ? bd.s[m] : v;
      if (m == static_cast<int>(K / 2 - 1)) mid = bd.s[m];
    }
    lane_bound = __float_as_int(v);
  }
  // the index of x, or of |x| for a symmetric table (one AND with the mask:
  // -0 becomes +0 and a NaN stays a NaN, as with fabsf)
  __device__ uint32_t code(float x) const { return (*this)(__uint_as_float(__float_as_uint(x) & keep)); }
  // F = F 2^BITS + index of x (or of |x| when SYM), the bits entering one
  // at a time from the most significant: each level's answer is one
  // add-with-carry (F + F + answer), so a lane that shifts in its elements
  // from last to first ends with element j at bits BITS j.  For SYM the
  // absolute value is a source modifier of the compares.
  template <bool SYM>
  __device__ void shift_in(float x, uint32_t& F) const {
    const float v = SYM ? fabsf(x) : x;
    if constexpr (!kPermute) {
      bool c[BITS] = {};
      shift_levels<0>(v, c, F);
    } else {
      F = (F << BITS) | (*this)(v);
    }
  }
  template <int L>
  __device__ void shift_levels(float v, bool (&c)[BITS], uint32_t& F) const {
    if constexpr (L < BITS) {
      c[L] = v >= pick_boundary<BITS, L, 0, 0>(c, bd);
      F = F + F + (c[L] ? 1u : 0u);
      shift_levels<L + 1>(v, c, F);
    }
  }
  __device__ uint32_t operator()(float x) const {
    if constexpr (!kPermute) {
      return classify<BITS>(x, bd);
    } else {
      // a = 4 idx, the byte address ds_bpermute takes; the constant part of
      // each level's address goes into the instruction's offset field
      uint32_t a = x >= mid ? 4u * (K / 2) : 0u;
#pragma unroll
      for (uint32_t step = K / 4; step >= 1; step /= 2) {
        const float b = __int_as_float(
            __builtin_amdgcn_ds_bpermute(static_cast<int>(a + 4u * (step - 1)), lane_bound));
        a += x >= b ? 4u * step : 0u;
      }
      return a >> 2;
    }
  }
};

// ---------------------------------------------------------------- packing
// quad_perm DPP control: lane k of each quad reads lane sel[k] of the quad.
constexpr int quad_perm(int a, int b, int c, int d) { return a | (b << 2) | (c << 4) | (d << 6); }

template <int CTRL>
__device__ inline uint32_t quad_read(uint32_t v) {
  return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xF, 0xF, false));
}

// word i of a code span
template <int P>
__device__ inline void st_word(const OutSpan<P>& c, int i, uint32_t v) { c.st4(static_cast<uint32_t>(i) * 4u, v); }
__device__ inline uint32_t ld_word(const Span& c, int i) { return c.ld4(static_cast<uint32_t>(i) * 4u); }

// Lane field F holds the 8 codes of the lane (8*BITS bits, code j at bit
// BITS*j).  The tile's stream is the lane fields laid end to end, so lane l's
// field starts at stream bit 8*BITS*l.  Writes the words of the tile whose
// index is below `valid` (the rest belong past the end of the buffer).
// Must be called by all 64 lanes together.
template <int BITS, int P>
__device__ inline void pack_store(const OutSpan<P>& out, uint32_t F, int lane, int64_t valid) {
  if constexpr (BITS == 4) {
    if (lane < valid) st_word(out, lane, F);
  } else if constexpr (BITS == 2) {
    const uint32_t nb = quad_read<quad_perm(1, 1, 3, 3)>(F);
    const uint32_t w = F | (nb << 16);
    const int widx = lane >> 1;
    if (!(lane & 1) && widx < valid) st_word(out, widx, w);
  } else if constexpr (BITS == 1) {
    const uint32_t n1 = quad_read<quad_perm(1, 1, 3, 3)>(F);
    const uint32_t a = F | (n1 << 8);
    const uint32_t n2 = quad_read<quad_perm(2, 2, 2, 2)>(a);
    const uint32_t w = a | (n2 << 16);
    const int widx = lane >> 2;
    if (!(lane & 3) && widx < valid) st_word(out, widx, w);
  } else {  // BITS == 3: a quad's 4 x 24 bits are words 3q, 3q+1, 3q+2
    const uint32_t nx = quad_read<quad_perm(1, 2, 3, 3)>(F);
    const int k = lane & 3;
    const uint32_t w = (F >> (8 * k)) | (nx << (24 - 8 * k));
    const int widx = 3 * (lane >> 2) + k;
    if (k < 3 && widx < valid) st_word(out, widx, w);
  }
}

// Inverse of the layout above: the lane's 8*BITS-bit field.  For 1, 2 and 4
// bits a field lies inside one word (lanes that share a word read the same
// address).  For 3 bits lanes 0..2 of each quad read the quad's 3 words with
// one coalesced load; each lane then takes its own word and the one before
// it from the quad and funnel-shifts its 24 bits out.  Must be called by all
// 64 lanes together.
template <int BITS>
__device__ inline uint32_t load_field(const Span& base, int lane, int64_t valid) {
  if constexpr (BITS == 3) {
    const int k = lane & 3;
    const int widx = 3 * (lane >> 2) + k;
    const uint32_t w = (k < 3 && widx < valid) ? ld_word(base, widx) : 0u;
    const uint32_t prev = quad_read<quad_perm(0, 0, 1, 2)>(w);   // word k-1 (k = 0: word 0)
    const uint32_t own = quad_read<quad_perm(0, 1, 2, 2)>(w);    // word k (k = 3: word 2)
    return __builtin_amdgcn_alignbit(own, prev, (24 * k) & 31);
  } else {
    const int widx = (8 * BITS * lane) >> 5;
    const uint32_t v = (widx < valid) ? ld_word(base, widx) : 0u;
    return v >> ((8 * BITS * lane) & 31);
  }
}

// The same two layouts for a full tile, with every lane active: in the
// loops over full tiles no lane is masked off, so no branch splits the loop
// body and the compiler can keep all of a group's loads in flight.  When
// packing, a lane without a word of its own stores an identical copy of a
// neighbour's word to the same address; when unpacking, lane 3 of each quad
// reloads word 2 of the quad, which the permutes never read.
template <int BITS, int P>
__device__ inline void pack_store_full(const OutSpan<P>& out, uint32_t F, int lane) {
  if constexpr (BITS == 4) {
    st_word(out, lane, F);
  } else if constexpr (BITS == 2) {
    const uint32_t lo = quad_read<quad_perm(0, 0, 2, 2)>(F);
    const uint32_t hi = quad_read<quad_perm(1, 1, 3, 3)>(F);
    st_word(out, lane >> 1, lo | (hi << 16));
  } else if constexpr (BITS == 1) {
    const uint32_t a = quad_read<quad_perm(0, 0, 2, 2)>(F) | (quad_read<quad_perm(1, 1, 3, 3)>(F) << 8);
    const uint32_t w = quad_read<quad_perm(0, 0, 0, 0)>(a) | (quad_read<quad_perm(2, 2, 2, 2)>(a) << 16);
    st_word(out, lane >> 2, w);
  } else {  // BITS == 3: lane k of a quad writes word min(k, 2) of the quad
    const int j = min(lane & 3, 2);
    const uint32_t lo = quad_read<quad_perm(0, 1, 2, 2)>(F);
    const uint32_t hi = quad_read<quad_perm(1, 2, 3, 3)>(F);
    st_word(out, 3 * (lane >> 2) + j, (lo >> (8 * j)) | (hi << (24 - 8 * j)));
  }
}

template <int BITS>
__device__ inline uint32_t load_field_full(const Span& base, int lane) {
  if constexpr (BITS == 3) {
    const int k = lane & 3;
    const uint32_t w = ld_word(base, 3 * (lane >> 2) + min(k, 2));
    const uint32_t prev = quad_read<quad_perm(0, 0, 1, 2)>(w);   // word k-1 (k = 0: word 0)
    const uint32_t own = quad_read<quad_perm(0, 1, 2, 2)>(w);    // word k (k = 3: word 2)
    return __builtin_amdgcn_alignbit(own, prev, (24 * k) & 31);
  } else {
    return ld_word(base, (8 * BITS * lane) >> 5) >> ((8 * BITS * lane) & 31);
  }
}

// packed words of n codes
__host__ __device__ inline int64_t words_of(int64_t n, int bits) { return (n * bits + 31) / 32; }

struct WaveIndex {
  int lane;
  int64_t wave, nwaves;
};
// The waves of every workgroup, numbered across the grid.  The waves per
// workgroup come from the launch's THREADS as a compile-time constant:
// blockDim would be a vector load from the dispatch packet, waited for
// before the first stream load.
template <int THREADS>
__device__ inline WaveIndex wave_index() {
  constexpr int kPerBlock = THREADS / kWave;
  // the wave's number within its workgroup is the same in all its lanes;
  // readfirstlane tells the compiler so, which keeps tile addresses scalar
  const int w = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / kWave));
  return {static_cast<int>(threadIdx.x & (kWave - 1)),
          static_cast<int64_t>(blockIdx.x) * kPerBlock + w,
          static_cast<int64_t>(gridDim.x) * kPerBlock};
}

// ---------------------------------------------------------------- forward, full-range tables
// For 16-bit inputs both results of the forward are functions of the input
// bit pattern alone, so every workgroup holds two tables over all 65536
// patterns in LDS:
//   ylut  the output pattern of f(x), 128 KiB;
//   clut  the interval index, 4 bits per pattern: byte q holds pattern 2q in
//         its low and pattern 2q+1 in its high nibble, 32 KiB.
// A tile then costs two LDS reads and a few integer operations per element
// instead of an evaluation of f and the compares.
//
// ylut depends only on the activation and the storage type, and most of it
// follows a simple rule (fwd16_rules.h, written by gen_fwd16_rules.py: the
// table is 512 blocks of 128 patterns; runs of blocks are the input itself,
// one constant, RNE(x / 2), RNE(lambda x), or need f).  Every workgroup fills
// its ylut from those runs, which travel as kernel arguments, and evaluates f
// (the fp32 f of the per-element path, then one rounding) only in the blocks
// no rule covers: for bf16 GELU 30 blocks of 512.  clut depends on the
// boundaries and is built by every workgroup: the index is monotone in the
// pattern within one sign, so each thread classifies only the two ends of its
// segment of patterns and fills it if they agree; the few segments that hold
// a boundary, infinities or NaNs are then classified pattern by pattern by the
// whole wave.  Neither table outlives the workgroup: the library keeps no
// device memory.
struct OutRuns {
  uint32_t r[fwd16_rules::kMaxRuns];
};

// ylut from the runs, by each wave on its own (no barrier, no scratch):
//   1. wave w fills the 1 KiB chunks w, w + 8, ... of ylut (lane l the 16
//      bytes at 16 l, so one store instruction covers consecutive banks) in
//      the blocks whose rule is integer work on the patterns: IDENTITY,
//      CONST and HALF (one exponent step down).  The chunks' 64 blocks are
//      the wave's: lane l finds the run of block 4 w + 32 (l / 4) + l mod 4
//      and the lanes of each chunk read it with one cross-lane permute.
//      Branch-free: every lane forms both candidates and stores only in
//      those blocks;
//   2. the blocks of the runs that need arithmetic (EVAL: the kernel's f;
//      SCALE), numbered in order, go to the waves in turn; 2 patterns per
//      lane, the rule uniform over the wave.  The two steps store to
//      different blocks.
template <int DT, int ACT>
__device__ void build_output_table(uint16_t* ylut, const OutRuns& runs) {
  using namespace fwd16_rules;
  static_assert(FEWBIT_FWD16_THREADS == 512, "8 waves, 16 chunks each");
  constexpr uint32_t kWaves = FEWBIT_FWD16_THREADS / kWave;
  constexpr uint32_t kChunks = 128u / kWaves;           // 1 KiB chunks per wave
  // x / 2 as one exponent step down (subtracted from both halves of a word)
  constexpr uint32_t kHalfStep = DT == FEWBIT_BF16 ? 0x00800080u : 0x04000400u;
  using H = Half<DT>;
  uint32_t R[kMaxRuns];
#pragma unroll
  for (int j = 0; j < kMaxRuns; ++j) {
    uint32_t t = runs.r[j];
    asm("" : "+s"(t));         // keep the descriptors in scalar registers
    R[j] = t;
  }
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  uint32_t mine = R[0];
  {
    const uint32_t blk = 4u * wave + 32u * (lane >> 2) + (lane & 3u);
#pragma unroll
    for (int j = 1; j < kMaxRuns; ++j) mine = (R[j] & 1023u) <= blk ? R[j] : mine;
  }
  // all permutes first: each waits in LDS order, so issuing one after the
  // previous chunk's store would wait for that store too
  uint32_t descs[kChunks];
#pragma unroll
  for (uint32_t i = 0; i < kChunks; ++i)
    descs[i] = static_cast<uint32_t>(
        __builtin_amdgcn_ds_bpermute(static_cast<int>(4u * (4u * i + (lane >> 4))), static_cast<int>(mine)));
#pragma unroll
  for (uint32_t i = 0; i < kChunks; ++i) {
    const uint32_t p0 = (wave + kWaves * i) * 512u + lane * 8u;   // the lane's first pattern
    const uint32_t desc = descs[i];
    const uint32_t rule = (desc >> 12) & 15u;
    // word e of the lane's 4: base + e step, the pattern pair (one exponent
    // step down for HALF) or the constant
    const uint32_t pair = (p0 | ((p0 + 1u) << 16)) - (rule == HALF ? kHalfStep : 0u);
    // a bit select through a mask in a register: as a ?: the compiler
    // branches around the constant's multiply
    uint32_t is_const = rule == CONST ? ~0u : 0u;
    asm("" : "+v"(is_const));
    const uint32_t base = (((desc >> 16) * 0x10001u) & is_const) | (pair & ~is_const);
    const uint32_t step = 0x00020002u & ~is_const;
    const u32x4_t v = {base, base + step, base + 2u * step, base + 3u * step};
    if (rule == IDENTITY || rule == CONST || rule == HALF) *reinterpret_cast<u32x4_t*>(ylut + p0) = v;
  }
  // the blocks needing arithmetic, numbered across the runs in order: the
  // k-th goes to wave k mod 8
  uint32_t* ylut32 = reinterpret_cast<uint32_t*>(ylut);
  uint32_t before = 0;          // such blocks in the runs before run j
#pragma unroll
  for (int j = 0; j < kMaxRuns; ++j) {
    const uint32_t rule = (R[j] >> 12) & 15u;
    const uint32_t start = R[j] & 1023u;
    const uint32_t end = j + 1 < kMaxRuns ? min(R[j + 1] & 1023u, 512u) : 512u;
    if (start >= 512u || (rule != EVAL && rule != SCALE)) continue;
    const uint32_t first = start + ((wave + 8u - (before & 7u)) & 7u);
    before += end - start;
    for (uint32_t blk = first; blk < end; blk += 8u) {
      const uint32_t p = blk * 128u + 2u * lane;
      const float x0 = H::widen(p), x1 = H::widen(p + 1u);
      ylut32[blk * 64u + lane] = rule == EVAL ? H::pack(Act<DT, ACT>::f(x0), Act<DT, ACT>::f(x1))
                                              : H::pack(x0 * kSeluLambda, x1 * kSeluLambda);
    }
  }
}

template <int DT, int BITS>
__device__ void build_code_table(uint8_t* clut, const TableArgs& tab, int symmetric) {
  // each thread owns one aligned segment of kSeg patterns (kSeg / 2 bytes)
  constexpr uint32_t kSeg = 65536u / FEWBIT_FWD16_THREADS;
  static_assert(kSeg >= 32 && kSeg <= 32768 && 65536u % FEWBIT_FWD16_THREADS == 0,
                "segments of whole 16-byte stores within one sign");
  // every call below is made by all 64 lanes of the wave, as Search's
  // permutes require: the segment loop takes two patterns per lane and kSeg
  // is a multiple of 128, so all lanes run it equally often
  static_assert(kSeg % (2 * kWave) == 0, "whole waves in the segment loop");
  const Search<BITS> cl(tab, static_cast<int>(threadIdx.x & (kWave - 1)), symmetric);
  auto code_of = [&](uint32_t p) { return cl.code(Half<DT>::widen(p)); };
  const uint32_t p0 = threadIdx.x * kSeg;
  const uint32_t last = p0 + kSeg - 1u;
  // the index is monotone in the pattern within one sign, so a segment
  // whose two ends agree is uniform, unless it reaches the infinities and
  // NaNs at the top of its sign (exponent all ones)
  const bool special = (last & 0x7FFFu) >= Half<DT>::kSpecialFrom;
  const uint32_t a = code_of(p0), b = code_of(last);
  const bool uniform = !special && a == b;
  if (uniform) {
    const uint32_t rep = a * 0x11111111u;
#pragma unroll
    for (uint32_t i = 0; i < kSeg / 32u; ++i)
      reinterpret_cast<u32x4_t*>(clut + p0 / 2u)[i] = (u32x4_t){rep, rep, rep, rep};
  }
  // the other segments are classified pattern by pattern by the whole wave
  const uint32_t lane = threadIdx.x & (kWave - 1), first = threadIdx.x - lane;
  uint64_t todo = __ballot(!uniform);
  while (todo) {
    const uint32_t l = static_cast<uint32_t>(__builtin_ctzll(todo));
    todo &= todo - 1u;
    const uint32_t q0 = (first + l) * kSeg;
    for (uint32_t j = 2u * lane; j < kSeg; j += 2u * kWave)
      clut[(q0 + j) / 2u] = static_cast<uint8_t>(code_of(q0 + j) | (code_of(q0 + j + 1u) << 4));
  }
}

__device__ inline uint32_t code_of_pattern(const uint8_t* clut, uint32_t p) {
  return (static_cast<uint32_t>(clut[p >> 1]) >> ((p & 1u) << 2)) & 15u;
}

template <int BITS>
__device__ inline void fwd16_tile(u32x4_t in, const uint16_t* ylut, const uint8_t* clut,
                                  u32x4_t& out, uint32_t& F) {
  F = 0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t w = in[k];
    const uint32_t lo = w & 0xFFFFu, hi = w >> 16;
    out[k] = static_cast<uint32_t>(ylut[lo]) | (static_cast<uint32_t>(ylut[hi]) << 16);
    F |= (code_of_pattern(clut, lo) << (2 * k * BITS)) |
         (code_of_pattern(clut, hi) << ((2 * k + 1) * BITS));
  }
}

template <int DT, int BITS, int ACT>
__global__ __launch_bounds__(FEWBIT_FWD16_THREADS) void fwd16full_kernel(
    const uint16_t* x, uint16_t* y, uint32_t* __restrict__ codes, int64_t n, int64_t nwords,
    TableArgs tab, int symmetric, OutRuns runs) {
  constexpr int U = FEWBIT_FWD16_UNROLL;
  constexpr int kWords = 16 * BITS;
  // clut first: ylut's 32 KiB offset then fits the LDS instruction's
  // immediate offset field
  __shared__ __attribute__((aligned(16))) uint8_t tables[32768 + 2 * 65536];
  uint8_t* clut = tables;
  uint16_t* ylut = reinterpret_cast<uint16_t*>(tables + 32768);
  const WaveIndex wi = wave_index<FEWBIT_FWD16_THREADS>();
  const int64_t full = n / kTile;
  const int64_t groups = full / U;
  const uint32_t lane_b = static_cast<uint32_t>(wi.lane) * kLaneBytes;

  // the wave's first tile group is loaded before the tables are built, so
  // its memory latency passes during the build
  int64_t gi = wi.wave;
  u32x4_t in[U];
  if (gi < groups) {
#pragma unroll
    for (int u = 0; u < U; ++u) in[u] = Span(x + (gi * U + u) * kTile, kSpanBytes).ld16(lane_b);
  }
  build_output_table<DT, ACT>(ylut, runs);
  build_code_table<DT, BITS>(clut, tab, symmetric);
  __syncthreads();

  for (bool loaded = true; gi < groups; gi += wi.nwaves, loaded = false) {
    const int64_t t0 = gi * U;
    u32x4_t out[U];
    uint32_t F[U];
    if (!loaded) {
#pragma unroll
      for (int u = 0; u < U; ++u) in[u] = Span(x + (t0 + u) * kTile, kSpanBytes).ld16(lane_b);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) fwd16_tile<BITS>(in[u], ylut, clut, out[u], F[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      OutSpan<kThroughNt>(y + (t0 + u) * kTile, kSpanBytes).st16(lane_b, out[u]);
      pack_store_full<BITS>(OutSpan<kThroughNt>(codes + (t0 + u) * kWords, kWords * 4), F[u], wi.lane);
    }
  }
  for (int64_t t = groups * U + wi.wave; t < full; t += wi.nwaves) {
    u32x4_t out;
    uint32_t F;
    fwd16_tile<BITS>(Span(x + t * kTile, kSpanBytes).ld16(lane_b), ylut, clut, out, F);
    OutSpan<kThroughNt>(y + t * kTile, kSpanBytes).st16(lane_b, out);
    pack_store_full<BITS>(OutSpan<kThroughNt>(codes + t * kWords, kWords * 4), F, wi.lane);
  }
  // the partial tile at the end, if any, goes to the wave that would own it
  if (n % kTile != 0 && wi.wave == full % wi.nwaves) {
    const int64_t t = full;
    const int rest = static_cast<int>(n - t * kTile);
    uint32_t F = 0, p[kPerLane];
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) p[j] = Span(x + t * kTile, rest * 2u).ld2(lane_b + 2u * j);
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) {
      OutElements<kThroughNt>(y + t * kTile, rest * 2u).st2(lane_b + 2u * j, ylut[p[j]]);
      F |= (wi.lane * kPerLane + j < rest ? code_of_pattern(clut, p[j]) : 0u) << (BITS * j);
    }
    const int64_t wbase = t * kWords;
    pack_store<BITS>(OutSpan<kThroughNt>(codes + wbase, kWords * 4), F, wi.lane, nwords - wbase);
  }
}

// fp16 / bf16 forward by evaluation: f and the compares for every element,
// no tables.  Bound by HBM where f and the compares take up to about 16 VALU
// slots an element (every activation at 1 and most at 2 bits), by VALU beyond.
// Where the full-range table kernel evaluates f (the blocks no rule covers) it
// uses this same f and rounding.
//
// One tile per one-wave workgroup, and nothing between the wave's start and its
// stream load: pointers and size arrive in scalar registers with the wave
// (kernarg preload), there is no loop over the grid, and the boundaries are
// read after the load has gone out.  So the dispatcher alone keeps the memory
// busy: fp16 SiLU 2 bits of 51.4M elements 34.9 -> 32.3 us (84% of 8 TB/s)
// against two tiles per wave in a loop with its boundaries read first, bf16
// SELU 2 bits of 34M 26.5 -> 23.5, fp16 Sigmoid 1 bit of 2^27 86.7 -> 80.5; and
// half the evaluation in series on small tensors (12 fp16 Tanh layers of 2^14,
// 4 bits, with their backwards in a graph: 76 -> 58 us).
//
// A full tile: y from the fp32 f, and the codes shifted into the lane's field
// from its last element to its first (element j of the lane's 8 at bits
// BITS j).  SYM: the table is symmetric, the index is that of |x|.
template <int DT, int BITS, int ACT, bool SYM>
__device__ inline void fwd16v_tile(u32x4_t in, const Search<BITS>& cl, u32x4_t& out, uint32_t& F) {
  using H = Half<DT>;
  F = 0;
#pragma unroll
  for (int k = 3; k >= 0; --k) {
    const float a = H::lo(in[k]), b = H::hi(in[k]);
    cl.template shift_in<SYM>(b, F);
    cl.template shift_in<SYM>(a, F);
    out[k] = H::pack(Act<DT, ACT>::f(a), Act<DT, ACT>::f(b));
  }
}

template <int DT, int BITS, int ACT, bool SYM, int P>
__global__ __launch_bounds__(kWave) void fwd16v_kernel(
    const uint16_t* x, uint16_t* y, uint32_t* __restrict__ codes, int64_t n, TableArgs tab) {
  constexpr int kWords = 16 * BITS;
  const int lane = static_cast<int>(threadIdx.x);
  const uint32_t lane_b = static_cast<uint32_t>(lane) * kLaneBytes;
  const int64_t full = static_cast<int64_t>(static_cast<uint64_t>(n) / kTile);
  const int64_t t = blockIdx.x;
  // of a tile that is not whole nothing is loaded here (0 bytes)
  const u32x4_t in = Span(x + t * kTile, t < full ? kSpanBytes : 0u).ld16(lane_b);
  // the stream load is in flight before the boundaries are put in place
  __builtin_amdgcn_sched_barrier(0);
  const Search<BITS> cl(tab, lane, SYM);
  if (t < full) {
    u32x4_t out;
    uint32_t F;
    fwd16v_tile<DT, BITS, ACT, SYM>(in, cl, out, F);
    OutSpan<P>(y + t * kTile, kSpanBytes).st16(lane_b, out);
    pack_store_full<BITS>(OutSpan<P>(codes + t * kWords, kWords * 4), F, lane);
  } else {                                       // the partial tile at the end
    const int rest = static_cast<int>(n - full * kTile);
    uint32_t F = 0, p[kPerLane];
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) p[j] = Span(x + full * kTile, rest * 2u).ld2(lane_b + 2u * j);
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) {
      const float v = Half<DT>::widen(p[j]);
      const uint32_t c = cl.code(v);                          // all lanes
      OutElements<P>(y + full * kTile, rest * 2u).st2(lane_b + 2u * j, Half<DT>::pack(Act<DT, ACT>::f(v), 0.0f));
      F |= (lane * kPerLane + j < rest ? c : 0u) << (BITS * j);
    }
    const int64_t wbase = full * kWords;
    pack_store<BITS>(OutSpan<P>(codes + wbase, kWords * 4), F, lane, words_of(n, BITS) - wbase);
  }
}

// ---------------------------------------------------------------- forward, bf16, table
// One LDS word per input pattern of the octaves that matter (fwd16_out.h):
// the fp32 output factor, with the interval index in its low 4 bits.  An
// element costs one ds_read_b32 and about eleven VALU operations at every
// activation and bit width, the packing included, and about eight more for its
// share of placing the table (SQ counters, GELU 3 bits: 19.3), where evaluating
// f and the compares takes up to thirty.  Bound by HBM, with VALU busy 83%.
//
// The table is 14-21 KiB, so 32 waves share a CU and the grid needs no
// persistent walk: each wave takes kTabUnroll tiles, whose loads are in flight
// while the table is put in place.  The factors are copied from constant
// memory (they stay in the L2 caches: no HBM traffic), the indices are
// searched for the patterns of each 16-byte chunk by the thread that copies
// it; for most chunks the first and the last pattern's agree and the two
// between need no search.
//
// Measured (GELU, 3 bits, back-to-back launches; the full-range table kernel,
// the per-element kernel, this one): 2^23 elements 12.0, 8.9, 7.5 us; 12.6M
// 14.8, 11.7, 10.8; 2^26 53.4, 52.4, 47.2; 2^28 202, 205, 175 (83.7% of
// 8 TB/s).  Two tiles per wave: one leaves the table's cost on too few elements
// (2^28: 213 us in a probe where two took 191), four leave the last workgroups
// of a CU alone for longer (201).
constexpr int kTabUnroll = 2;

typedef unsigned short u16x2_t __attribute__((ext_vector_type(2)));

// ReLU needs no factors: its words hold the index alone.
template <int ACT>
__device__ constexpr fwd16_out::Table<ACT> kOutTable = fwd16_out::make<ACT>();

template <int ACT>
struct OutForm {
  static constexpr float kMax = fwd16_out::max_of(ACT);
  // At |x| below 2^-126 GELU's and SiLU's x / 2 can be a tie: the index bits
  // are cleared there so that the factor is exactly 1/2.
  static constexpr bool kClear = ACT == FEWBIT_GELU || ACT == FEWBIT_SILU;
  __device__ static float y(float x, uint32_t word) {
    const float t = __uint_as_float(kClear ? word & ~15u : word);
    if constexpr (ACT == FEWBIT_RELU) return Act<FEWBIT_BF16, FEWBIT_RELU>::f(x);
    // maximum / minimum keep a NaN
    if constexpr (ACT == FEWBIT_SOFTPLUS) return __builtin_elementwise_maximum(x, -0.0f) + t;
    if constexpr (ACT == FEWBIT_SIGMOID)
      return __builtin_elementwise_maximum(__builtin_elementwise_minimum(x, t), t);
    if constexpr (ACT == FEWBIT_TANH)
      return __builtin_elementwise_minimum(__builtin_elementwise_maximum(x, -kMax), kMax) * t;
    return __builtin_elementwise_maximum(x, -kMax) * t;
  }
};

// Byte offsets of the table words of the two patterns of w.
template <int ACT>
__device__ inline uint32_t word_offsets(uint32_t w) {
  constexpr uint16_t kBase2 = 2 * fwd16_out::base_of(ACT);
  constexpr uint16_t kCount = fwd16_out::count_of(ACT);
  const u16x2_t p = __builtin_bit_cast(u16x2_t, w);
  // the sign, with -0 on the side of +0 (a boundary may lie at 0); the empty
  // register barrier keeps the packed form (else: two compares and selects)
  u16x2_t neg = __builtin_elementwise_sub_sat(p, (u16x2_t){1, 1});
  asm("" : "+v"(neg));
  neg = neg >> static_cast<uint16_t>(15);
  // twice the magnitude pattern, brought into the range
  u16x2_t m = __builtin_elementwise_sub_sat(static_cast<u16x2_t>(p << static_cast<uint16_t>(1)), (u16x2_t){kBase2, kBase2});
  m = __builtin_elementwise_min(m, (u16x2_t){2 * (kCount - 1), 2 * (kCount - 1)});
  m = neg * (u16x2_t){2 * kCount, 2 * kCount} + m;
  return __builtin_bit_cast(uint32_t, static_cast<u16x2_t>(m << static_cast<uint16_t>(1)));
}

__device__ inline uint32_t table_word(const uint32_t* table, uint32_t offset) {
  return *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(table) + offset);
}

// The tile's outputs and its lanes' code fields.  Each word is rotated into
// the field by its index bits alone (alignbit), element 0 first.  A NaN has
// the output NaN by the arithmetic but shares its word with the infinity of
// its sign: its index is 0, set in a branch that is taken only where a wave
// holds one.
template <int BITS, int ACT>
__device__ inline void tab_tile(u32x4_t in, const uint32_t* table, u32x4_t& out, uint32_t& F) {
  using H = Half<FEWBIT_BF16>;
  uint32_t f = 0;
  u16x2_t top = {0, 0};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const uint32_t w = in[k];
    const uint32_t o = word_offsets<ACT>(w);
    const uint32_t t0 = table_word(table, o & 0xFFFFu), t1 = table_word(table, o >> 16);
    out[k] = H::pack(OutForm<ACT>::y(H::lo(w), t0), OutForm<ACT>::y(H::hi(w), t1));
    f = __builtin_amdgcn_alignbit(t0, f, BITS);
    f = __builtin_amdgcn_alignbit(t1, f, BITS);
    top = __builtin_elementwise_max(top, static_cast<u16x2_t>(__builtin_bit_cast(u16x2_t, w) << static_cast<uint16_t>(1)));
  }
  F = f >> (32 - 8 * BITS);
  constexpr uint16_t kInf2 = 2 * H::kSpecialFrom;
  if (__builtin_bit_cast(uint32_t, __builtin_elementwise_sub_sat(top, (u16x2_t){kInf2, kInf2})) != 0) {
#pragma unroll
    for (int j = 0; j < kPerLane; ++j)
      if (((in[j / 2] >> (16 * (j & 1))) & 0x7FFFu) > H::kSpecialFrom) F &= ~(((1u << BITS) - 1u) << (BITS * j));
  }
}

// Tile of place q in the work of workgroup b.  RUN 0: consecutive tiles.
// Else runs of RUN tiles are dealt to 8 consecutive workgroups, which the
// dispatcher hands to the 8 XCDs, so that the addresses in flight across the
// chip stay close together.
template <int TILES, int RUN>
__device__ inline int64_t tab_tile_at(int64_t b, int q) {
  if constexpr (RUN == 0)
    return b * TILES + q;
  else
    return (b >> 3) * (8 * TILES) + (q / RUN) * (8 * RUN) + static_cast<int>(b & 7) * RUN + q % RUN;
}

template <int DT, int BITS, int ACT, int THREADS, int RUN>
__global__ __launch_bounds__(THREADS, 8) void fwd16_kernel(
    const uint16_t* x, uint16_t* y, uint32_t* __restrict__ codes, int64_t n, int64_t nwords,
    TableArgs tab, int symmetric) {
  static_assert(DT == FEWBIT_BF16, "fp16's octaves hold eight times as many patterns");
  using H = Half<DT>;
  constexpr int kWords = 16 * BITS;
  constexpr int kWaves = THREADS / kWave, kTiles = kWaves * kTabUnroll;
  constexpr uint32_t kBase = fwd16_out::base_of(ACT), kCount = fwd16_out::count_of(ACT);
  constexpr uint32_t kChunks = 2 * kCount / 4;         // 16-byte chunks of the table
  __shared__ __attribute__((aligned(16))) uint32_t table[2 * kCount];
  const int lane = static_cast<int>(threadIdx.x & (kWave - 1));
  const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / kWave));
  const uint32_t lane_b = static_cast<uint32_t>(lane) * kLaneBytes;
  const int64_t full = n / kTile;
  if (tab_tile_at<kTiles, RUN>(blockIdx.x, 0) * kTile >= n) return;      // the whole workgroup

  // tiles past the last full one load nothing and store nothing (a span of 0 bytes)
  int64_t t[kTabUnroll];
  u32x4_t in[kTabUnroll];
#pragma unroll
  for (int u = 0; u < kTabUnroll; ++u) {
    t[u] = tab_tile_at<kTiles, RUN>(blockIdx.x, u * kWaves + wave);
    in[u] = Span(x + t[u] * kTile, t[u] < full ? kSpanBytes : 0u).ld16(lane_b);
  }

  const Search<BITS> cl(tab, lane, symmetric);
#pragma unroll
  for (uint32_t c0 = 0; c0 < kChunks; c0 += THREADS) {
    const uint32_t c = c0 + threadIdx.x;
    if (c0 + THREADS > kChunks && c0 + wave * kWave >= kChunks) break;     // whole waves
    u32x4_t w = {0u, 0u, 0u, 0u};
    if constexpr (ACT != FEWBIT_RELU) w = reinterpret_cast<const u32x4_t*>(kOutTable<ACT>.e)[c];
    const bool neg = 4u * c >= kCount;
    const uint32_t p = kBase + 4u * c - (neg ? kCount : 0u) + (neg ? 0x8000u : 0u);
    uint32_t i[4];
    i[0] = cl.code(H::widen(p));
    i[3] = cl.code(H::widen(p + 3u));
    i[1] = i[2] = i[0];
    if (__any(i[0] != i[3])) {        // by whole waves: the search reads other lanes
      i[1] = cl.code(H::widen(p + 1u));
      i[2] = cl.code(H::widen(p + 2u));
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] |= i[j];
    reinterpret_cast<u32x4_t*>(table)[c] = w;
  }
  __syncthreads();

#pragma unroll
  for (int u = 0; u < kTabUnroll; ++u) {
    u32x4_t out;
    uint32_t F;
    tab_tile<BITS, ACT>(in[u], table, out, F);
    const bool here = t[u] < full;
    OutSpan<kThroughNt>(y + t[u] * kTile, here ? kSpanBytes : 0u).st16(lane_b, out);
    pack_store_full<BITS>(OutSpan<kThroughNt>(codes + t[u] * kWords, here ? kWords * 4 : 0u), F, lane);
  }
  // the partial tile at the end, if any, by the wave whose tile it is
  if (n % kTile != 0) {
#pragma unroll
    for (int u = 0; u < kTabUnroll; ++u) {
      if (t[u] != full) continue;
      const int rest = static_cast<int>(n - full * kTile);
      uint32_t F = 0, p[kPerLane];
#pragma unroll
      for (int j = 0; j < kPerLane; ++j) p[j] = Span(x + full * kTile, rest * 2u).ld2(lane_b + 2u * j);
#pragma unroll
      for (int j = 0; j < kPerLane; ++j) {
        const uint32_t word = table_word(table, word_offsets<ACT>(p[j]) & 0xFFFFu);
        OutElements<kThroughNt>(y + full * kTile, rest * 2u)
            .st2(lane_b + 2u * j, H::pack(OutForm<ACT>::y(H::widen(p[j]), word), 0.0f));
        const bool coded = lane * kPerLane + j < rest && (p[j] & 0x7FFFu) <= H::kSpecialFrom;
        F |= (coded ? word & ((1u << BITS) - 1u) : 0u) << (BITS * j);
      }
      const int64_t wbase = full * kWords;
      pack_store<BITS>(OutSpan<kThroughNt>(codes + wbase, kWords * 4), F, lane, nwords - wbase);
    }
  }
}

// ---------------------------------------------------------------- fp32 tiles
// An fp32 tile is 512 elements in two halves of 256; lane l holds elements
// 4l .. 4l+3 of each half, so each 16-byte access instruction covers 1 KiB
// of contiguous memory.  (Eight consecutive elements per lane would need two
// accesses 32 bytes apart per lane, each instruction touching only every
// other 16 bytes of its span, which streams far below the contiguous rate.)
// In stream order a half's codes are then the lanes' fields of 4*BITS bits
// laid end to end, 8*BITS words per half, 16*BITS per tile.
template <int BITS>
struct Codes32 {
  static constexpr int FB = 4 * BITS;                  // field bits per lane and half
  static constexpr uint32_t kMask = (1u << FB) - 1u;
  static constexpr int kHalfWords = 8 * BITS;
  static constexpr int kWords = 16 * BITS;
  // most lanes whose fields meet one word: 32 / FB when fields tile words,
  // else a partial field at each end (for 12-bit fields: 4 lanes)
  static constexpr int kSources = 32 / FB + ((32 % FB) ? 2 : 0);
};

// Every lane builds word q = lane mod 16*BITS of the tile from the fields
// of the lanes it covers (cross-lane reads of f0 | f1 << 16), and stores it;
// lanes past 16*BITS store identical copies.  FULL: the whole tile exists,
// so no store is masked off; else only words below `valid` are stored.
template <int BITS, bool FULL, int P>
__device__ inline void pack_store32(const OutSpan<P>& out, uint32_t f0, uint32_t f1, int lane,
                                    int64_t valid) {
  using C = Codes32<BITS>;
  const uint32_t both = f0 | (f1 << 16);
  const int q = lane % C::kWords;
  const int v = q / C::kHalfWords, w = q % C::kHalfWords;
  const int a = (32 * w) / C::FB, o = (32 * w) % C::FB;
  uint32_t word = 0;
#pragma unroll
  for (int i = 0; i < C::kSources; ++i) {
    const uint32_t f = (static_cast<uint32_t>(__shfl(static_cast<int>(both), (a + i) & 63)) >>
                        (16 * v)) & C::kMask;
    const int sh = i * C::FB - o;                      // bit position of the field in the word
    word |= (i == 0) ? (f >> o) : (sh < 32 ? f << sh : 0u);
  }
  if (FULL || q < valid) st_word(out, q, word);
}

// The field of lane `lane` in half v: the one or two words it spans,
// funnel-shifted.  FULL: every word of the tile exists; else words from
// `valid` on read as 0.
template <int BITS, bool FULL>
__device__ inline uint32_t load_field32(const Span& base, int v, int lane, int64_t valid) {
  using C = Codes32<BITS>;
  const int b0 = lane * C::FB;
  const int i0 = v * C::kHalfWords + (b0 >> 5);
  const int i1 = min(i0 + 1, C::kWords - 1);           // unused unless the field straddles
  const uint32_t lo = (FULL || i0 < valid) ? ld_word(base, i0) : 0u;
  const uint32_t hi = (FULL || i1 < valid) ? ld_word(base, i1) : 0u;
  return __builtin_amdgcn_alignbit(hi, lo, b0 & 31) & C::kMask;
}

// The lane's i-th element of its 8 in the tile.
__device__ inline int element32(int lane, int i) { return (i / 4) * 256 + lane * 4 + i % 4; }

// One tile per wave, kThreads32 threads per workgroup.
constexpr int kThreads32 = 256;

__device__ inline int64_t tile32() {
  return static_cast<int64_t>(blockIdx.x) * (kThreads32 / kWave) +
         __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / kWave));
}

// ---------------------------------------------------------------- forward, fp32
template <int BITS, int ACT>
__device__ inline void fwd32_half(u32x4_t in, const Search<BITS>& cl, u32x4_t& out, uint32_t& f) {
  f = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float xv = __uint_as_float(in[j]);
    out[j] = __float_as_uint(Act<FEWBIT_F32, ACT>::f(xv));
    f |= cl.code(xv) << (BITS * j);
  }
}

// LATE: the boundaries are put in place after the stream loads have gone out.
template <int BITS, int ACT, int P, bool LATE>
__device__ inline void fwd32_tile(const float* x, float* y, uint32_t* codes, int64_t n, int32_t symmetric,
                                  const TableArgs& tab) {
  constexpr int kWords = Codes32<BITS>::kWords;
  const int lane = static_cast<int>(threadIdx.x & (kWave - 1));
  const int64_t full = static_cast<int64_t>(static_cast<uint64_t>(n) / kTile);
  const int64_t t = tile32();
  const uint32_t lane_b = static_cast<uint32_t>(lane) * kLaneBytes;
  u32x4_t in[2];
  auto load = [&] {
#pragma unroll
    for (int h = 0; h < 2; ++h) in[h] = Span(x + t * kTile + h * 256, t < full ? kSpanBytes : 0u).ld16(lane_b);
  };
  if constexpr (LATE) {
    load();
    __builtin_amdgcn_sched_barrier(0);
  }
  const Search<BITS> cl(tab, lane, symmetric);
  if constexpr (!LATE) load();
  if (t < full) {
    u32x4_t out[2];
    uint32_t f[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) fwd32_half<BITS, ACT>(in[h], cl, out[h], f[h]);
#pragma unroll
    for (int h = 0; h < 2; ++h) OutSpan<P>(y + t * kTile + h * 256, kSpanBytes).st16(lane_b, out[h]);
    pack_store32<BITS, true>(OutSpan<P>(codes + t * kWords, kWords * 4), f[0], f[1], lane, kWords);
  } else if (t == full && n % kTile != 0) {      // the partial tile at the end
    const int rest = static_cast<int>(n - t * kTile);
    uint32_t f[2] = {0u, 0u}, v[kPerLane];
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) v[i] = Span(x + t * kTile, rest * 4u).ld4(element32(lane, i) * 4u);
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) {
      const int e = element32(lane, i);
      const float xv = __uint_as_float(v[i]);
      const uint32_t c = cl.code(xv);                       // all lanes
      OutElements<P>(y + t * kTile, rest * 4u).st4(e * 4u, __float_as_uint(Act<FEWBIT_F32, ACT>::f(xv)));
      f[i / 4] |= (e < rest ? c : 0u) << (BITS * (i % 4));
    }
    const int64_t wbase = t * kWords;
    pack_store32<BITS, false>(OutSpan<P>(codes + wbase, kWords * 4), f[0], f[1], lane, words_of(n, BITS) - wbase);
  }
}

template <int BITS, int ACT, int P>
__global__ __launch_bounds__(kThreads32) void fwd32_kernel(
    const float* x, float* y, uint32_t* __restrict__ codes, int64_t n, int32_t symmetric, TableArgs tab) {
  fwd32_tile<BITS, ACT, P, true>(x, y, codes, n, symmetric, tab);
}

// The shortest launches (small32): the structure comes first, so nothing is
// preloaded (the preload takes the leading pointers and integers only).
template <int BITS, int ACT>
__global__ __launch_bounds__(kThreads32) void fwd32_small_kernel(
    TableArgs tab, const float* x, float* y, uint32_t* __restrict__ codes, int64_t n, int32_t symmetric) {
  fwd32_tile<BITS, ACT, kNt, false>(x, y, codes, n, symmetric, tab);
}

// ---------------------------------------------------------------- backward
// The K values of the table live in one register of each wave, lane i
// holding v[i mod K] (K <= 16 divides 64), and an element's value is read
// from the lane its code names with one cross-lane permute (ds_bpermute).
// No LDS array is filled and no barrier is taken, so a wave issues its
// stream loads as soon as it starts: the backward runs as a grid of
// one-wave workgroups, one tile each, and the hardware dispatcher streams
// them through the device.
template <int BITS>
struct Values {
  int lane_value;
  __device__ explicit Values(const TableArgs& tab) {
    // lane c < K holds v[c] (a chain of selects over scalar registers); the
    // permutes read no other lane.  The values pass an empty asm barrier
    // first, which keeps them in scalar registers: otherwise the compiler
    // may turn the chain into a per-lane load from the kernel-argument
    // block, a vector memory load whose wait would hold back the stream
    // loads.
    const int lane = static_cast<int>(threadIdx.x & (kWave - 1));
    float v = 0.0f;
#pragma unroll
    for (int c = 0; c < (1 << BITS); ++c) {
      float t = tab.v[c];
      asm("" : "+s"(t));
      v = lane == c ? t : v;
    }
    lane_value = __float_as_int(v);
  }
  // v[c] for the code c of this lane; all 64 lanes must take part
  __device__ float operator()(uint32_t c) const {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(static_cast<int>(c << 2), lane_value));
  }
};

template <int DT, int BITS>
__device__ inline u32x4_t grad16_tile(u32x4_t g, uint32_t F, const Values<BITS>& val) {
  using H = Half<DT>;
  constexpr uint32_t kMask = (1u << BITS) - 1u;
  u32x4_t out;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const float v0 = val((F >> (2 * k * BITS)) & kMask);
    const float v1 = val((F >> ((2 * k + 1) * BITS)) & kMask);
    out[k] = H::pack(H::lo(g[k]) * v0, H::hi(g[k]) * v1);   // fp32 products, then RNE
  }
  return out;
}

// The 16-bit backward runs one-wave workgroups, one tile each.  At 1 and 3
// bits a tile's code span (64 or 192 bytes) is not a whole number of 128-byte
// lines: tiles 2p and 2p+1 share one line.  Read by waves on different XCDs,
// whose L2 caches are separate, that line would be fetched from memory twice
// (a third of the code stream again at 3 bits).  So workgroup u takes tile
// tile_of_unit(u): within each run of 16 workgroups, workgroups r and r + 8
// take the two tiles of pair r.  The dispatcher hands workgroups to the 8
// XCDs in turn, so the two land on the same XCD, one after the other, and the
// shared line is fetched once.  The grid is a whole number of such runs;
// units whose tile lies past the end do nothing.
template <int BITS>
struct BwdOrder {
  static constexpr bool kPaired = BITS == 1 || BITS == 3;
  static constexpr int64_t kRun = kPaired ? 16 : 1;
  __host__ __device__ static int64_t tile_of_unit(int64_t u) {
    if constexpr (kPaired) {
      const int64_t r = u & 15;
      return (u - r) + 2 * (r & 7) + (r >> 3);
    } else {
      return u;
    }
  }
  // the inverse: the unit that takes tile t
  __host__ __device__ static int64_t unit_of_tile(int64_t t) {
    if constexpr (kPaired) {
      const int64_t q = t & 15;
      return (t - q) + 8 * (q & 1) + (q >> 1);
    } else {
      return t;
    }
  }
};

template <int DT, int BITS, int P>
__global__ __launch_bounds__(kWave) void bwd_kernel(
    const uint16_t* g, const uint32_t* __restrict__ codes, uint16_t* gin, int64_t n, TableArgs tab) {
  constexpr int kWords = 16 * BITS;
  constexpr uint32_t kMask = (1u << BITS) - 1u;
  const int lane = static_cast<int>(threadIdx.x);
  const int64_t full = static_cast<int64_t>(static_cast<uint64_t>(n) / kTile);
  const int64_t t = BwdOrder<BITS>::tile_of_unit(blockIdx.x);
  if (t < full) {
    const uint32_t lane_b = static_cast<uint32_t>(lane) * kLaneBytes;
    const u32x4_t in = Span(g + t * kTile, kSpanBytes).ld16(lane_b);
    const uint32_t F = load_field_full<BITS>(Span(codes + t * kWords, kWords * 4), lane);
    // the stream loads are in flight before the values are put in place
    __builtin_amdgcn_sched_barrier(0);
    const Values<BITS> val(tab);
    OutSpan<P>(gin + t * kTile, kSpanBytes).st16(lane_b, grad16_tile<DT, BITS>(in, F, val));
  } else if (t == full && n % kTile != 0) {      // the partial tile at the end
    const int rest = static_cast<int>(n - t * kTile);
    uint32_t p[kPerLane];
#pragma unroll
    for (int j = 0; j < kPerLane; ++j)
      p[j] = Span(g + t * kTile, rest * 2u).ld2(static_cast<uint32_t>(lane) * kLaneBytes + 2u * j);
    const Values<BITS> val(tab);
    const int64_t wbase = t * kWords;
    const uint32_t F = load_field<BITS>(Span(codes + wbase, kWords * 4), lane, words_of(n, BITS) - wbase);
    const uint32_t lane_b = static_cast<uint32_t>(lane) * kLaneBytes;
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) {
      const float v = val((F >> (BITS * j)) & kMask);       // all lanes
      OutElements<P>(gin + t * kTile, rest * 2u).st2(lane_b + 2u * j, Half<DT>::pack(Half<DT>::widen(p[j]) * v, 0.0f));
    }
  }
}

// fp32 backward on the fp32 tile layout (see fp32 tiles above).
template <int BITS>
__device__ inline u32x4_t grad32_half(u32x4_t g, uint32_t f, const Values<BITS>& val) {
  constexpr uint32_t kMask = (1u << BITS) - 1u;
  u32x4_t out;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    out[j] = __float_as_uint(__uint_as_float(g[j]) * val((f >> (BITS * j)) & kMask));
  return out;
}

template <int BITS, int P>
__device__ inline void bwd32_tile(const float* g, const uint32_t* codes, float* gin, int64_t n, const TableArgs& tab) {
  constexpr int kWords = Codes32<BITS>::kWords;
  constexpr uint32_t kMask = (1u << BITS) - 1u;
  const int lane = static_cast<int>(threadIdx.x & (kWave - 1));
  const int64_t full = static_cast<int64_t>(static_cast<uint64_t>(n) / kTile);
  const int64_t t = tile32();
  if (t < full) {
    const uint32_t lane_b = static_cast<uint32_t>(lane) * kLaneBytes;
    u32x4_t in[2];
    uint32_t f[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      in[h] = Span(g + t * kTile + h * 256, kSpanBytes).ld16(lane_b);
      f[h] = load_field32<BITS, true>(Span(codes + t * kWords, kWords * 4), h, lane, kWords);
    }
    // the stream loads are in flight before the values are put in place
    __builtin_amdgcn_sched_barrier(0);
    const Values<BITS> val(tab);
#pragma unroll
    for (int h = 0; h < 2; ++h)
      OutSpan<P>(gin + t * kTile + h * 256, kSpanBytes).st16(lane_b, grad32_half<BITS>(in[h], f[h], val));
  } else if (t == full && n % kTile != 0) {      // the partial tile at the end
    const int rest = static_cast<int>(n - t * kTile);
    const int64_t wbase = t * kWords;
    uint32_t p[kPerLane], f[2];
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) p[i] = Span(g + t * kTile, rest * 4u).ld4(element32(lane, i) * 4u);
#pragma unroll
    for (int h = 0; h < 2; ++h)
      f[h] = load_field32<BITS, false>(Span(codes + wbase, kWords * 4), h, lane, words_of(n, BITS) - wbase);
    const Values<BITS> val(tab);
#pragma unroll
    for (int i = 0; i < kPerLane; ++i) {
      const float v = val((f[i / 4] >> (BITS * (i % 4))) & kMask);   // all lanes
      OutElements<P>(gin + t * kTile, rest * 4u).st4(element32(lane, i) * 4u, __float_as_uint(__uint_as_float(p[i]) * v));
    }
  }
}

template <int BITS, int P>
__global__ __launch_bounds__(kThreads32) void bwd32_kernel(
    const float* g, const uint32_t* __restrict__ codes, float* gin, int64_t n, TableArgs tab) {
  bwd32_tile<BITS, P>(g, codes, gin, n, tab);
}

template <int BITS>
__global__ __launch_bounds__(kThreads32) void bwd32_small_kernel(
    TableArgs tab, const float* g, const uint32_t* __restrict__ codes, float* gin, int64_t n) {
  bwd32_tile<BITS, kNt>(g, codes, gin, n, tab);
}

// ---------------------------------------------------------------- host side
int check_table(const fewbit_table* t) {
  if (!t) return FEWBIT_E_NULL;
  if (t->bits < 1 || t->bits > 4) return FEWBIT_E_BITS;
  if (t->act < FEWBIT_GELU || t->act > FEWBIT_SOFTPLUS) return FEWBIT_E_INVALID;
  constexpr int32_t kFlags = FEWBIT_FLAG_SYMMETRIC | FEWBIT_FLAG_TABLE_FWD | FEWBIT_FLAG_ELEMENT_FWD;
  if ((t->flags & ~kFlags) != 0 || t->reserved != 0) return FEWBIT_E_INVALID;
  if ((t->flags & FEWBIT_FLAG_TABLE_FWD) && (t->flags & FEWBIT_FLAG_ELEMENT_FWD)) return FEWBIT_E_INVALID;
  const int K = 1 << t->bits;
  for (int m = 0; m < K - 1; ++m) {
    if (!std::isfinite(t->s[m])) return FEWBIT_E_NUMERIC;
    if (m > 0 && !(t->s[m - 1] < t->s[m])) return FEWBIT_E_NUMERIC;
  }
  for (int m = 0; m < K; ++m)
    if (!std::isfinite(t->v[m])) return FEWBIT_E_NUMERIC;
  return FEWBIT_OK;
}

bool misaligned(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) != 0; }

TableArgs table_args(const fewbit_table* t) {
  TableArgs a;
  const int K = 1 << t->bits;
  for (int m = 0; m < 15; ++m) a.s[m] = (m < K - 1) ? t->s[m] : INFINITY;
  for (int m = 0; m < 16; ++m) a.v[m] = (m < K) ? t->v[m] : 0.0f;
  return a;
}

// Compute units of the current device, read once per device.
int device_cus() {
  static std::atomic<int> cache[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) dev = -1;
  if (dev >= 0 && dev < 64) {
    const int c = cache[dev].load(std::memory_order_relaxed);
    if (c > 0) return c;
  }
  int c = 0;
  if (dev < 0 ||
      hipDeviceGetAttribute(&c, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      c <= 0)
    c = 256;
  if (dev >= 0 && dev < 64) cache[dev].store(c, std::memory_order_relaxed);
  return c;
}

// Workgroups of the full-range table kernel, whose waves walk the tiles in
// groups: one group per wave at most, and at most what the chip holds at once.
dim3 persistent_grid(int64_t n) {
  constexpr int64_t kPerBlock = static_cast<int64_t>(FEWBIT_FWD16_THREADS / kWave) * FEWBIT_FWD16_UNROLL * kTile;
  const int64_t blocks = n / kPerBlock + (n % kPerBlock != 0);
  const int64_t cap = static_cast<int64_t>(device_cus()) * FEWBIT_FWD16_WG_PER_CU;
  return dim3(static_cast<unsigned>(blocks < cap ? blocks : cap));
}

int64_t tiles_of(int64_t n) { return n / kTile + (n % kTile != 0); }

// The grid of a launch with one pass per workgroup over `per` units of its
// work, at most a part's (in_parts).
dim3 grid_of(int64_t units, int per) { return dim3(static_cast<unsigned>((units + per - 1) / per)); }

// A launch holds fewer than 2^32 threads, and the kernels with one pass per
// wave have 64 for 512 elements: longer tensors go in parts of whole tiles, and
// of whole runs of the backward's tile order.  f(at, m) launches the m elements
// from `at` on; their codes start at word at / 32 * bits.  A size that no device
// memory holds (half a terabyte from 2^38 elements on) launches nothing.
template <class F>
hipError_t in_parts(int64_t n, F f) {
  constexpr int64_t kPart = int64_t{1} << 34;
  static_assert(kPart % (16 * kTile) == 0 && kPart / kTile * kWave < int64_t{1} << 32, "whole runs that fit a launch");
  if (n >= int64_t{1} << 38) return hipErrorInvalidConfiguration;
  for (int64_t at = 0; at < n; at += kPart) {
    const hipError_t e = f(at, n - at < kPart ? n - at : kPart);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// The stream must belong to the current device: the grid size, the output
// tables and the launch all refer to the current device.
int check_stream_device(hipStream_t stream) {
  int current = 0;
  hipDevice_t owner = 0;
  if (hipGetDevice(&current) != hipSuccess || hipStreamGetDevice(stream, &owner) != hipSuccess)
    return FEWBIT_E_HIP;
  return owner == current ? FEWBIT_OK : FEWBIT_E_INVALID;
}

// Whether a launch that writes `bytes` of y or grad_in stores with nt alone.
// Its lines then stay dirty in the 32 MB of L2 and are written back when the
// kernel ends, with nothing left to overlap with: writing through is faster on
// small tensors (a graph of 12 bf16 GELU layers of 2^17 elements, 24 kernels:
// 56.7 -> 52.6 us) and on large ones (16-bit backward of 2^28 elements, 3
// bits: 181.4 -> 175.5 us; fp16 SiLU 2-bit pass of 51.4M: 71.1 -> 67.1; fp32
// Tanh 3-bit pass of 2^25: 90.4 -> 84.4).  Between, what decides is not this
// tensor but what is live around it, which a launch does not know: whether a
// stack fits the 256 MB memory-side cache but not the L2.  nt alone stands for
// the stack of many layers.  In a graph, nt and through: 12 fp16 SiLU layers of
// 2^21 elements 82.8 and 89.0 us, 12 fp32 Tanh (3 bits) 107.7 and 112.3; but 4
// layers of 2^19 23.2 and 22.0 and 24.3 and 23.0, 12 of 2^19 54.1 and 51.3 and
// 65.2 and 62.5, 12 SiLU of 6 * 2^20 153 and 147.
//
// y is stored nt as well as through (the passes of 51.4M and 2^25 with y through
// alone: 71.3 and 88.5 us), a short gradient is not (4.97 against 5.08 us at
// 2^22).
constexpr int64_t kNtFrom = int64_t{1} << 20, kNtUpto = int64_t{1} << 24;
bool store_nt(int64_t bytes) { return bytes >= kNtFrom && bytes < kNtUpto; }

// (A forward or a backward repeated alone on the same buffers is another matter:
// fp32 1-bit forward of 22M 26.5 us with nt, 28.1 as it is; fp32 4-bit backward
// of 2^26 87.2 and 88.5.  Over changing buffers the two are level.)
//
// The gradient up to here is left in the memory-side cache for its reader
// (fp32 Tanh 3-bit pass of 2^25 elements 85.1 us, with nt 87.8); a longer one
// does not stay there, and with nt it takes no room from what does (bf16 GELU
// 3-bit pass of 2^28 359.7 us, with nt 344.3; fp32 Sigmoid 4-bit of 2^26 177.2,
// 173.8; the fp32 backward alone of 35M 45.4, 44.6).
constexpr int64_t kGradThroughUpto = int64_t{1} << 27;

// fp32 launches that run the small kernels: nothing preloaded, stores nt, the
// boundaries put in place before the stream loads.  With fewer than four
// workgroups the dispatcher's fetch of the preloaded arguments is on the only
// path there is (12 ReLU layers of 6144 elements, 2 bits, with their backwards
// in a graph: 48.2 us preloaded, 45.9 not; Tanh 4 bits 54.4 and 53.2); from the
// fourth on the waves start sooner for it (8192 elements: 48.0 and 48.9).
bool small32(int64_t n) { return n <= 3 * (kThreads32 / kWave) * kTile; }

struct Launch {
  const fewbit_table* t;
  const void* in;
  void* out;
  uint32_t* codes;
  int64_t n;
  hipStream_t s;
};

// The output-table runs of (ACT, DT) as a kernel argument; unused entries
// start past the last block.
template <int DT, int ACT>
OutRuns out_runs() {
  const fwd16_rules::Runs& src = fwd16_rules::kRuns[ACT][DT == FEWBIT_BF16 ? 1 : 0];
  OutRuns r;
  for (int j = 0; j < fwd16_rules::kMaxRuns; ++j) r.r[j] = j < src.count ? src.r[j] : fwd16_rules::kUnused;
  return r;
}

// log2 of the element count from which an fp16 forward, or a bf16 one whose
// boundaries the compact table does not hold, runs the full-range table
// kernel, by [type: fp16, bf16][activation][bits - 1]; 63: never.  That kernel
// builds its tables in every workgroup (7-10 us of fixed cost for bf16, 12-15
// us for fp16, whose tables need f in far more blocks) and runs as a persistent
// grid, which streams at about 72% of the HBM peak whatever f and the bits are;
// the per-element kernel has no setup and streams at up to 87%, but evaluates f
// and the compares per element.  Measured on MI355X (x ~ N(0, 1), 2^25 .. 2^28
// elements, back-to-back launches; per element, table): fp16 GELU 4 bits, 2^26
// 57.8 and 54.9 us, 2^25 30.1 and 33.2; Tanh 2 bits, 2^27 96.6 and 94.2; SiLU
// 3 bits, 2^28 177 and 189.
constexpr uint8_t kTableMinLog2[2][FEWBIT_SOFTPLUS + 1][4] = {
    {   // fp16
        {63, 63, 26, 26},   // gelu
        {63, 63, 63, 27},   // silu
        {63, 63, 63, 27},   // sigmoid
        {63, 27, 26, 25},   // tanh
        {63, 63, 63, 63},   // relu
        {63, 63, 26, 26},   // selu
        {63, 63, 26, 26},   // softplus
    },
    {   // bf16
        {63, 63, 27, 26},   // gelu
        {63, 63, 63, 63},   // silu
        {63, 63, 63, 63},   // sigmoid
        {63, 63, 26, 26},   // tanh
        {63, 63, 63, 63},   // relu
        {63, 63, 63, 27},   // selu
        {63, 63, 28, 27},   // softplus
    },
};

int64_t table_min_of(int dt, int act, int bits) {
  const int lg = kTableMinLog2[dt == FEWBIT_BF16 ? 1 : 0][act][bits - 1];
  return lg >= 63 ? INT64_MAX : int64_t{1} << lg;
}

// The same for the bf16 kernel with the compact table, wherever the table's
// boundaries allow it (fwd16_out::holds).  Its cost does not depend on the
// activation or the bit width, the per-element kernel's does.  Measured as
// above (per element, table): GELU 3 bits, 2^24 14.8 and 15.0 us, 2^25 27.5 and
// 25.7, 2^28 205 and 175; Sigmoid 3 bits 13.9 and 14.7, 25.3 and 25.7, 190 and
// 177; with 1 or 2 bits the per-element kernel streams at 81-87% of the HBM
// peak and is ahead (GELU 1 bit, 2^28: 160 and 171) or level (2 bits: 171).
constexpr uint8_t kTabMinLog2[FEWBIT_SOFTPLUS + 1][4] = {
    {63, 63, 22, 22},   // gelu
    {63, 63, 25, 22},   // silu
    {63, 63, 26, 26},   // sigmoid
    {63, 63, 22, 22},   // tanh
    {63, 63, 28, 26},   // relu
    {63, 63, 22, 22},   // selu
    {63, 28, 22, 22},   // softplus
};

int64_t tab_min_of(int act, int bits) {
  const int lg = kTabMinLog2[act][bits - 1];
  return lg >= 63 ? INT64_MAX : int64_t{1} << lg;
}

// At 3 and 4 bits it is ahead for every activation while its workgroups of 32
// tiles fill the chip's 512 places about once (Sigmoid 3 bits, the closest, at
// 3, 4, 8 and 10 Mi elements: 5.0, 5.7, 8.4, 9.8 us per element, 4.5, 4.8, 7.8,
// 9.6 by the table; ReLU 3 bits at 8 and 10 Mi 7.9, 9.1 and 7.2, 9.9).
bool tab_by_size(int act, int bits, int64_t n) {
  return n >= tab_min_of(act, bits) || (bits >= 3 && n >= int64_t{3} << 20 && n <= int64_t{8} << 20);
}

// Workgroups of 16 waves that take consecutive tiles below, of 8 waves that
// share runs of 4 tiles with 7 others from here on: GELU 3 bits, 12.6M elements
// 11.5 and 12.9 us, 2^25 27.0 and 26.8, 2^28 191 and 186.
constexpr int64_t kTabLargeFrom = int64_t{1} << 25;

// A launch of it holds fewer than 2^32 threads of 16 elements, so 2^35 elements
// fit with room; the full-range kernel's grid does not grow with the tensor.
constexpr int64_t kTabUpto = int64_t{1} << 35;

// A launch by the runtime's own call, which returns its status: the <<<>>> form
// pushes and pops a launch configuration and leaves the status to two queries
// around it, five runtime calls where this is one (a small forward's host time
// through the C ABI 4.20 -> 4.05 us).
template <class T>
struct Same {
  using type = T;
};
template <class... P>
hipError_t launch(void (*kernel)(P...), dim3 grid, unsigned threads, hipStream_t stream,
                  typename Same<P>::type... args) {
  void* pointers[] = {const_cast<void*>(static_cast<const void*>(&args))...};
  return hipLaunchKernel(reinterpret_cast<const void*>(kernel), grid, dim3(threads), pointers, 0, stream);
}

// It stores nt and through at every size, also where the other kernels store nt
// alone (3 to 8 Mi elements), for the stacks' sake.  Graphs of 12 GELU layers,
// 3 bits, against nt alone: 4 Mi 128.9 and 135.1 us, 8 Mi 180.8 and 182.6; one
// ReLU 4-bit pass of 6 Mi 11.5 and 11.8, of 8 Mi 13.0 and 12.5.  (The full-range
// kernel is chosen only at sizes where the others do the same.)
template <int DT, int BITS, int ACT, int THREADS, int RUN>
hipError_t launch_tab(const Launch& L, int64_t nw, int sym) {
  // elements of a workgroup, or of the 8 that share runs of tiles
  constexpr int64_t kGroups = RUN ? 8 : 1, kSpan = kGroups * (THREADS / kWave) * kTabUnroll * kTile;
  const dim3 grid(static_cast<unsigned>((L.n + kSpan - 1) / kSpan * kGroups));
  return launch(fwd16_kernel<DT, BITS, ACT, THREADS, RUN>, grid, THREADS, L.s,
                static_cast<const uint16_t*>(L.in), static_cast<uint16_t*>(L.out), L.codes, L.n, nw,
                table_args(L.t), sym);
}

template <int DT, int BITS, int ACT>
hipError_t launch_fwd(const Launch& L) {
  const int64_t nw = fewbit_packed_words(L.n, BITS);
  const int sym = (L.t->flags & FEWBIT_FLAG_SYMMETRIC) ? 1 : 0;
  if constexpr (DT == FEWBIT_F32) {
    if (small32(L.n))
      return launch(fwd32_small_kernel<BITS, ACT>, grid_of(tiles_of(L.n), kThreads32 / kWave), kThreads32, L.s,
                    table_args(L.t), static_cast<const float*>(L.in), static_cast<float*>(L.out), L.codes, L.n, sym);
    auto kernel = store_nt(4 * L.n) ? fwd32_kernel<BITS, ACT, kNt> : fwd32_kernel<BITS, ACT, kThroughNt>;
    return in_parts(L.n, [&](int64_t at, int64_t m) {
      return launch(kernel, grid_of(tiles_of(m), kThreads32 / kWave), kThreads32, L.s,
                    static_cast<const float*>(L.in) + at, static_cast<float*>(L.out) + at,
                    L.codes + at / 32 * BITS, m, sym, table_args(L.t));
    });
  } else {
    const bool holds = DT == FEWBIT_BF16 && L.n < kTabUpto && fwd16_out::holds(ACT, sym != 0, L.t->s, (1 << BITS) - 1);
    const bool by_size = holds ? tab_by_size(ACT, BITS, L.n) : L.n >= table_min_of(DT, ACT, BITS);
    const bool table = (L.t->flags & FEWBIT_FLAG_TABLE_FWD) ||
                       (!(L.t->flags & FEWBIT_FLAG_ELEMENT_FWD) && by_size);
    if (!table) {
      const bool nt = store_nt(2 * L.n);
      auto kernel = sym ? (nt ? fwd16v_kernel<DT, BITS, ACT, true, kNt> : fwd16v_kernel<DT, BITS, ACT, true, kThroughNt>)
                        : (nt ? fwd16v_kernel<DT, BITS, ACT, false, kNt> : fwd16v_kernel<DT, BITS, ACT, false, kThroughNt>);
      return in_parts(L.n, [&](int64_t at, int64_t m) {
        return launch(kernel, grid_of(tiles_of(m), 1), kWave, L.s, static_cast<const uint16_t*>(L.in) + at,
                      static_cast<uint16_t*>(L.out) + at, L.codes + at / 32 * BITS, m, table_args(L.t));
      });
    }
    if constexpr (DT == FEWBIT_BF16) {
      if (holds)
        return L.n < kTabLargeFrom ? launch_tab<DT, BITS, ACT, 1024, 0>(L, nw, sym)
                                   : launch_tab<DT, BITS, ACT, 512, 4>(L, nw, sym);
    }
    return launch(fwd16full_kernel<DT, BITS, ACT>, persistent_grid(L.n), FEWBIT_FWD16_THREADS, L.s,
                  static_cast<const uint16_t*>(L.in), static_cast<uint16_t*>(L.out), L.codes, L.n, nw,
                  table_args(L.t), sym, out_runs<DT, ACT>());
  }
}

template <int DT, int BITS>
hipError_t launch_fwd_act(const Launch& L) {
  switch (L.t->act) {
    case FEWBIT_GELU: return launch_fwd<DT, BITS, FEWBIT_GELU>(L);
    case FEWBIT_SILU: return launch_fwd<DT, BITS, FEWBIT_SILU>(L);
    case FEWBIT_SIGMOID: return launch_fwd<DT, BITS, FEWBIT_SIGMOID>(L);
    case FEWBIT_TANH: return launch_fwd<DT, BITS, FEWBIT_TANH>(L);
    case FEWBIT_RELU: return launch_fwd<DT, BITS, FEWBIT_RELU>(L);
    case FEWBIT_SELU: return launch_fwd<DT, BITS, FEWBIT_SELU>(L);
    default: return launch_fwd<DT, BITS, FEWBIT_SOFTPLUS>(L);
  }
}

template <int DT>
hipError_t launch_fwd_bits(const Launch& L) {
  switch (L.t->bits) {
    case 1: return launch_fwd_act<DT, 1>(L);
    case 2: return launch_fwd_act<DT, 2>(L);
    case 3: return launch_fwd_act<DT, 3>(L);
    default: return launch_fwd_act<DT, 4>(L);
  }
}

template <int DT, int BITS>
hipError_t launch_bwd(const Launch& L) {
  if constexpr (DT == FEWBIT_F32) {
    if (small32(L.n))
      return launch(bwd32_small_kernel<BITS>, grid_of(tiles_of(L.n), kThreads32 / kWave), kThreads32, L.s,
                    table_args(L.t), static_cast<const float*>(L.in), L.codes, static_cast<float*>(L.out), L.n);
    auto kernel = store_nt(4 * L.n)             ? bwd32_kernel<BITS, kNt>
                  : 4 * L.n <= kGradThroughUpto ? bwd32_kernel<BITS, kThrough>
                                                : bwd32_kernel<BITS, kThroughNt>;
    return in_parts(L.n, [&](int64_t at, int64_t m) {
      return launch(kernel, grid_of(tiles_of(m), kThreads32 / kWave), kThreads32, L.s,
                    static_cast<const float*>(L.in) + at, L.codes + at / 32 * BITS,
                    static_cast<float*>(L.out) + at, m, table_args(L.t));
    });
  } else {
    auto kernel = store_nt(2 * L.n)             ? bwd_kernel<DT, BITS, kNt>
                  : 2 * L.n <= kGradThroughUpto ? bwd_kernel<DT, BITS, kThrough>
                                                : bwd_kernel<DT, BITS, kThroughNt>;
    return in_parts(L.n, [&](int64_t at, int64_t m) {
      // one-wave workgroups: a whole number of runs of the tile order over the
      // full tiles, and up to the partial tile's unit when that lies past them
      using Order = BwdOrder<BITS>;
      const int64_t full = m / kTile;
      int64_t units = (full + Order::kRun - 1) / Order::kRun * Order::kRun;
      if (m % kTile != 0 && units <= Order::unit_of_tile(full)) units = Order::unit_of_tile(full) + 1;
      return launch(kernel, grid_of(units, 1), kWave, L.s, static_cast<const uint16_t*>(L.in) + at,
                    L.codes + at / 32 * BITS, static_cast<uint16_t*>(L.out) + at, m, table_args(L.t));
    });
  }
}

template <int DT>
hipError_t launch_bwd_bits(const Launch& L) {
  switch (L.t->bits) {
    case 1: return launch_bwd<DT, 1>(L);
    case 2: return launch_bwd<DT, 2>(L);
    case 3: return launch_bwd<DT, 3>(L);
    default: return launch_bwd<DT, 4>(L);
  }
}

// Status of a launch; with FEWBIT_DEBUG set in the environment the HIP error
// behind FEWBIT_E_HIP is printed to stderr.
int launch_status(const char* where, hipError_t e) {
  if (e == hipSuccess) return FEWBIT_OK;
  (void)hipGetLastError();          // not left for the caller's next query
  if (std::getenv("FEWBIT_DEBUG"))
    std::fprintf(stderr, "fewbit: %s launch failed: %s (%s)\n", where, hipGetErrorName(e),
                 hipGetErrorString(e));
  return FEWBIT_E_HIP;
}

}  // namespace

extern "C" int fewbit_fwd(const fewbit_table* t, int32_t dtype, const void* x, void* y,
                          uint32_t* codes, int64_t n, void* stream) {
  int rc = check_table(t);
  if (rc != FEWBIT_OK) return rc;
  if (dtype < FEWBIT_F32 || dtype > FEWBIT_BF16) return FEWBIT_E_DTYPE;
  if (n < 0) return FEWBIT_E_INVALID;
  if (n == 0) return FEWBIT_OK;
  if (!x || !y || !codes) return FEWBIT_E_NULL;
  if (misaligned(x) || misaligned(y) || misaligned(codes)) return FEWBIT_E_ALIGN;
  rc = check_stream_device(static_cast<hipStream_t>(stream));
  if (rc != FEWBIT_OK) return rc;
  const Launch L{t, x, y, codes, n, static_cast<hipStream_t>(stream)};
  const hipError_t e = dtype == FEWBIT_F32   ? launch_fwd_bits<FEWBIT_F32>(L)
                       : dtype == FEWBIT_F16 ? launch_fwd_bits<FEWBIT_F16>(L)
                                             : launch_fwd_bits<FEWBIT_BF16>(L);
  return launch_status("fewbit_fwd", e);
}

extern "C" int64_t fewbit_fwd16_table_min(int32_t act, int32_t bits, int32_t dtype) {
  if (act < FEWBIT_GELU || act > FEWBIT_SOFTPLUS || bits < 1 || bits > 4 ||
      (dtype != FEWBIT_F16 && dtype != FEWBIT_BF16))
    return -1;
  return dtype == FEWBIT_BF16 ? tab_min_of(act, bits) : table_min_of(dtype, act, bits);
}

extern "C" int fewbit_bwd(const fewbit_table* t, int32_t dtype, const void* grad_out,
                          const uint32_t* codes, void* grad_in, int64_t n, void* stream) {
  int rc = check_table(t);
  if (rc != FEWBIT_OK) return rc;
  if (dtype < FEWBIT_F32 || dtype > FEWBIT_BF16) return FEWBIT_E_DTYPE;
  if (n < 0) return FEWBIT_E_INVALID;
  if (n == 0) return FEWBIT_OK;
  if (!grad_out || !codes || !grad_in) return FEWBIT_E_NULL;
  if (misaligned(grad_out) || misaligned(codes) || misaligned(grad_in)) return FEWBIT_E_ALIGN;
  rc = check_stream_device(static_cast<hipStream_t>(stream));
  if (rc != FEWBIT_OK) return rc;
  const Launch L{t, grad_out, grad_in, const_cast<uint32_t*>(codes), n,
                 static_cast<hipStream_t>(stream)};
  const hipError_t e = dtype == FEWBIT_F32   ? launch_bwd_bits<FEWBIT_F32>(L)
                       : dtype == FEWBIT_F16 ? launch_bwd_bits<FEWBIT_F16>(L)
                                             : launch_bwd_bits<FEWBIT_BF16>(L);
  return launch_status("fewbit_bwd", e);
}

extern "C" const char* fewbit_strerror(int32_t status) {
  switch (status) {
    case FEWBIT_OK: return "success";
    case FEWBIT_E_INVALID: return "invalid argument";
    case FEWBIT_E_NULL: return "null pointer";
    case FEWBIT_E_ALIGN: return "pointer not 16-byte aligned";
    case FEWBIT_E_DTYPE: return "unknown storage type";
    case FEWBIT_E_BITS: return "bits must be 1..4";
    case FEWBIT_E_NOMEM: return "host allocation failed";
    case FEWBIT_E_NUMERIC: return "table boundaries not strictly increasing or not finite";
    case FEWBIT_E_HIP: return "HIP launch failed";
  }
  return "unknown status";
}
