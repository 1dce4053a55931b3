// HIP kernels of the DASO synchronisation step for CDNA4 (gfx950).
//
// The step is a pure streaming computation: every output element depends only
// on the same element of each input stream, so the kernels read each stream
// once with 16-byte (fp32) or 8-byte (bf16) coalesced loads, keep everything
// in registers, and write each output once.  It is bound by HBM bandwidth, not
// arithmetic; there is no contraction, so no MFMA.
//
// Arithmetic follows the binary32 operation order stated in daso.h exactly
// (local average: Section 3, Figure 2; optimizer step: Sections 3.1 and 4;
// merge: Eq. (1); bf16 packing: Sections 3 and 4).  Floating-point contraction
// is off for this file and division is the correctly rounded one, so the
// results match a plain IEEE binary32 evaluation bit for bit.
#include "daso_launch.h"

#pragma clang fp contract(off)

namespace daso {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------ memory helpers
// A wavefront's piece of a stream: `p` is the stream's base, `base` the piece's first
// element (the same in every lane) and `off` the lane's first element within it.
// The empty asm keeps the sum of the uniform part in scalar registers, so that
// the access takes it with one 32-bit lane offset that all streams of a type share;
// folded together they would cost each stream a 64-bit address and two
// additions in the vector unit.
#define DASO_GLOBAL __attribute__((address_space(1)))

template <typename V, typename T>
__device__ __forceinline__ V load_vec(const T* __restrict__ p, int64_t base, uint32_t off) {
  auto q = (const DASO_GLOBAL char*)(p + base);
  asm("" : "+s"(q));
  return __builtin_nontemporal_load((const DASO_GLOBAL V*)(q + off * static_cast<uint32_t>(sizeof(T))));
}

// NT: non-temporal.  Every stream is, but for the averaged gradient of a fused step: an extra
// written stream, which the L2 gathers better (resnet50-shaped set, g = 4, P = 0, with statistics
// 151 us, 161 non-temporal; g = 4, P = 4 182 and 194; g = 8, P = 8 without 278 and 283).
template <bool NT, typename V, typename T>
__device__ __forceinline__ void store_vec(T* __restrict__ p, int64_t base, uint32_t off, V v) {
  auto q = (DASO_GLOBAL char*)(p + base);
  asm("" : "+s"(q));
  const auto to = (DASO_GLOBAL V*)(q + off * static_cast<uint32_t>(sizeof(T)));
  if constexpr (NT) __builtin_nontemporal_store(v, to);
  else *to = v;
}

// The elements of a vector that `mask` selects (bit k: element k); the others
// read as 0.
template <typename T>
__device__ __forceinline__ void load_some(const T* __restrict__ p, unsigned mask, T (&r)[kVec]) {
#pragma unroll
  for (int k = 0; k < kVec; ++k) r[k] = (mask & (1u << k)) ? p[k] : T(0);
}

// ------------------------------------------------------------ bf16 helpers
// binary32 -> bfloat16, round to nearest even: add 0x7FFF plus the lowest kept
// bit and drop the low half; a mantissa carry moves to the next binade or to
// infinity.  NaN becomes the quiet NaN 0x7FC0.
__device__ __forceinline__ uint32_t bf16_rne(float f) {
  const uint32_t u = __float_as_uint(f);
  const uint32_t r = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
  return ((u & 0x7FFFFFFFu) > 0x7F800000u) ? 0x7FC0u : r;
}

__device__ __forceinline__ u32x2 pack4(f32x4 v) {
  u32x2 w;
  w.x = bf16_rne(v.x) | (bf16_rne(v.y) << 16);
  w.y = bf16_rne(v.z) | (bf16_rne(v.w) << 16);
  return w;
}

// The same for values of which none is NaN: the conversion instruction rounds
// to nearest even and keeps subnormals; only its NaN patterns are other ones.
__device__ __forceinline__ u32x2 pack4_no_nan(f32x4 v) {
  return __builtin_bit_cast(u32x2, __builtin_convertvector(v, bf16x4));
}

// Whether any lane of the wavefront holds an infinity or a NaN in `v`.
__device__ __forceinline__ bool any_nonfinite(f32x4 v) {
  // x * 0 is 0 for every finite x and NaN otherwise
  const float t = __builtin_fmaf(v.x, 0.0f, __builtin_fmaf(v.y, 0.0f, __builtin_fmaf(v.z, 0.0f, v.w * 0.0f)));
  return __builtin_amdgcn_ballot_w64(t != t) != 0;
}

// Exact bfloat16 -> binary32: the pattern becomes the top half.
__device__ __forceinline__ f32x4 widen(u32x2 h) {
  f32x4 r;
  r.x = __uint_as_float(h.x << 16);
  r.y = __uint_as_float(h.x & 0xFFFF0000u);
  r.z = __uint_as_float(h.y << 16);
  r.w = __uint_as_float(h.y & 0xFFFF0000u);
  return r;
}

// The exchanged copies and the wire are bf16 (XF = false) or fp32 (XF = true,
// the non-blocking exchange of Section 3, which is not cast).
template <bool XF>
struct XType {
  using Elem = uint16_t;
  using Vec = u32x2;
  static __device__ __forceinline__ f32x4 received(Vec v) { return widen(v); }
  static __device__ __forceinline__ Vec sent(f32x4 v) { return pack4(v); }
  static __device__ __forceinline__ Vec sent_finite(f32x4 v) { return pack4_no_nan(v); }
  static __device__ __forceinline__ Vec joined(const Elem (&h)[kVec]) {
    return Vec{h[0] | (static_cast<uint32_t>(h[1]) << 16), h[2] | (static_cast<uint32_t>(h[3]) << 16)};
  }
};
template <>
struct XType<true> {
  using Elem = float;
  using Vec = f32x4;
  static __device__ __forceinline__ f32x4 received(Vec v) { return v; }
  static __device__ __forceinline__ Vec sent(f32x4 v) { return v; }
  static __device__ __forceinline__ Vec sent_finite(f32x4 v) { return v; }
  static __device__ __forceinline__ Vec joined(const Elem (&h)[kVec]) { return Vec{h[0], h[1], h[2], h[3]}; }
};

// Division by a per-bucket or per-call integer d, correctly rounded.  For a power
// of two it is the product with the (exact) reciprocal.  Else q = RN(a * y) with
// y = RN(1 / d) is corrected once by its exact remainder (Markstein 1990): q' =
// RN(q + y * (a - d * q)) is the correctly rounded quotient as long as the
// remainder is representable, which tiny a can violate: they (below 2^-100)
// take the plain division.  Zeros, infinities and NaN are set right by
// v_div_fixup.
struct Divisor {
  float d;
  float inv;
  bool pow2;
};

__device__ __forceinline__ Divisor make_divisor(int k, float inv) {
  return Divisor{static_cast<float>(k), inv, k > 0 && (k & (k - 1)) == 0};
}

__device__ __forceinline__ float quotient(float a, const Divisor& q) {
  const float z = a * q.inv;
  return __builtin_amdgcn_div_fixupf(__builtin_fmaf(__builtin_fmaf(-z, q.d, a), q.inv, z), q.d, a);
}

__device__ __forceinline__ f32x4 divide(f32x4 a, const Divisor& q) {
  if (q.pow2) return a * q.inv;
  // twice the pattern of |a|, less one: zero becomes the largest value
  const auto key = [](float v) { return 2u * __float_as_uint(v) - 1u; };
  const uint32_t least = min(min(key(a.x), key(a.y)), min(key(a.z), key(a.w)));
  constexpr uint32_t kTiny = 2u * ((127u - 100u) << 23) - 1u;  // 2^-100
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(least < kTiny) == 0, 1))
    return f32x4{quotient(a.x, q), quotient(a.y, q), quotient(a.z, q), quotient(a.w, q)};
  return f32x4{a.x / q.d, a.y / q.d, a.z / q.d, a.w / q.d};
}

// --------------------------------------------------------------- statistics
// Sums of a thread (the count fits 32 bits: at most 4 elements per thread and
// partial) or across slices (64-bit count).
template <typename CountT>
struct AccT {
  double gsq;
  double dsq;
  CountT nf;
};
using Acc = AccT<uint32_t>;
using Acc64 = AccT<uint64_t>;

// The square of a binary32 value is exact in binary64, so for the gradients the fused
// multiply-add rounds as a multiplication and an addition would; the difference of two has up
// to 53 bits, and its square is added with one rounding instead of two.
__device__ __forceinline__ void accumulate(Acc& acc, f32x4 gbar, f32x4 xl, f32x4 xn, unsigned mask, bool nonfinite) {
#pragma unroll
  for (int k = 0; k < kVec; ++k) {
    if (mask & (1u << k)) {
      const double gv = static_cast<double>(gbar[k]);
      const double dv = static_cast<double>(xn[k]) - static_cast<double>(xl[k]);
      acc.gsq = __builtin_fma(gv, gv, acc.gsq);
      acc.dsq = __builtin_fma(dv, dv, acc.dsq);
    }
  }
  if (nonfinite) {
#pragma unroll
    for (int k = 0; k < kVec; ++k)
      if ((mask & (1u << k)) && (__float_as_uint(xn[k]) & 0x7F800000u) == 0x7F800000u) ++acc.nf;
  }
}

// One step of a wavefront sum: the value plus that of the lane which the DPP
// control names (0 where it names none).
template <int CTRL, typename T>
__device__ __forceinline__ T dpp_add(T v) {
  if constexpr (sizeof(T) == 4) {
    return v + __builtin_bit_cast(
                   T, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, true));
  } else {
    const u32x2 u = __builtin_bit_cast(u32x2, v);
    u32x2 r;
    r.x = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(u.x), CTRL, 0xF, 0xF, true));
    r.y = static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(u.y), CTRL, 0xF, 0xF, true));
    return v + __builtin_bit_cast(T, r);
  }
}

// Sum over the wavefront in a fixed tree: within rows of 16 lanes, then across
// the rows.  Valid in lane 63.  DPP moves stay in the vector ALU; a shuffle goes
// through LDS and takes several times as long, while the workgroup holds its place
// on the CU with no loads in flight.
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
  v = dpp_add<0x111>(v);  // row_shr:1
  v = dpp_add<0x112>(v);  // row_shr:2
  v = dpp_add<0x114>(v);  // row_shr:4
  v = dpp_add<0x118>(v);  // row_shr:8
  v = dpp_add<0x142>(v);  // row_bcast:15
  v = dpp_add<0x143>(v);  // row_bcast:31
  return v;
}

// Two sums at once: the halves of the wavefront first trade, so that the lower half
// holds a's partial sums and the upper one b's; one tree then serves both.
// The sum of `a` is valid in lane 31, that of `b` in lane 63.
__device__ __forceinline__ double wave_sum2(double a, double b) {
  const u32x2 ua = __builtin_bit_cast(u32x2, a), ub = __builtin_bit_cast(u32x2, b);
  const auto lo = __builtin_amdgcn_permlane32_swap(ua.x, ub.x, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(ua.y, ub.y, false, false);
  double v = __builtin_bit_cast(double, u32x2{lo[0], hi[0]}) + __builtin_bit_cast(double, u32x2{lo[1], hi[1]});
  v = dpp_add<0x111>(v);
  v = dpp_add<0x112>(v);
  v = dpp_add<0x114>(v);
  v = dpp_add<0x118>(v);
  return dpp_add<0x142>(v);  // row_bcast:15: lane 31 and lane 63 hold their half's sum
}

// The sums of a workgroup's wavefronts, in LDS.
template <int kWaves>
struct WaveSums {
  double sq[kWaves][2];  // grad_sq, delta_sq
  uint64_t nf[kWaves];
};

// Deterministic block sum: each wavefront's sum, then those in index order.
// Valid in thread 0.  The caller puts a barrier between two uses of `s`.
template <typename CountT, int kWaves>
__device__ __forceinline__ Acc64 block_sum(const AccT<CountT>& v, WaveSums<kWaves>& s) {
  const double t = wave_sum2(v.gsq, v.dsq);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  CountT n = 0;
  if (__builtin_amdgcn_ballot_w64(v.nf != 0) != 0) n = wave_sum(v.nf);
  if ((lane & 31) == 31) s.sq[wave][lane >> 5] = t;
  if (lane == 63) s.nf[wave] = n;
  __syncthreads();
  Acc64 r = {0.0, 0.0, 0};
  if (threadIdx.x == 0) {
    r = Acc64{s.sq[0][0], s.sq[0][1], s.nf[0]};
#pragma unroll
    for (int w = 1; w < kWaves; ++w) {
      r.gsq += s.sq[w][0];
      r.dsq += s.sq[w][1];
      r.nf += s.nf[w];
    }
  }
  return r;
}

// ---------------------------------------------------- arithmetic of a vector
// The start of Eq. (1)'s sum: the local term 2S * xl.  S = 0 is the blocking
// synchronisation of Section 3, the plain average of the exchanged copies, so
// the local state is left out: the sum starts from -0, the identity of IEEE
// addition (-0 + c == c for every c), and a non-finite xl cannot reach it.
__device__ __forceinline__ f32x4 merge_start(float two_s, f32x4 xl) {
  if (two_s != 0.0f) return two_s * xl;
  return f32x4{-0.0f, -0.0f, -0.0f, -0.0f};
}

// The optimizer step (Section 3.1; PyTorch SGD with momentum, coupled weight
// decay that is skipped when zero): the local state xl; m becomes the new
// momentum.
__device__ __forceinline__ f32x4 sgd_momentum4(const StepArgs& a, f32x4 x, f32x4& m, f32x4 gbar) {
  f32x4 d = gbar;
  if (a.wd != 0.0f) d = gbar + (a.wd * x);
  m = (a.mu * m) + d;
  return x - (a.lr * m);
}

// A result of a wavefront's piece: whole, or (FULL = false) the elements of each
// lane's vector that its `mask` selects.
template <bool FULL, bool NT = true, typename V, typename T>
__device__ __forceinline__ void put(T* __restrict__ p, int64_t base, uint32_t off, unsigned mask, V v) {
  if constexpr (FULL) {
    store_vec<NT>(p, base, off, v);
  } else {
    if (mask == 0xFu) {
      __builtin_nontemporal_store(v, reinterpret_cast<V*>(p + base + off));
    } else {
      T h[kVec];
      __builtin_memcpy(h, &v, sizeof(v));
#pragma unroll
      for (int k = 0; k < kVec; ++k)
        if (mask & (1u << k)) p[base + off + k] = h[k];
    }
  }
}

// The outputs after the merge: params, the wire (of x' or, with
// DASO_PACK_PRE_MERGE, of xl) and the statistics.
template <int MODE, bool STATS, bool XF, bool FULL>
__device__ __forceinline__ void store_results(const StepArgs& a, int64_t base, uint32_t off, unsigned mask,
                                              f32x4 gbar, f32x4 xl, f32x4 xn, Acc& acc) {
  using X = XType<XF>;
  put<FULL>(a.x, base, off, mask, xn);
  bool nonfinite = false;
  if constexpr (STATS || !XF) nonfinite = any_nonfinite(xn);
  if (a.wire) {
    auto* wire = static_cast<typename X::Elem*>(a.wire);
    const bool pre = (MODE == kModeFused) && (a.flags & DASO_PACK_PRE_MERGE);
    const f32x4 y = pre ? xl : xn;
    if (__builtin_expect(!nonfinite && !pre, 1)) put<FULL>(wire, base, off, mask, X::sent_finite(y));
    else put<FULL>(wire, base, off, mask, X::sent(y));
  }
  if constexpr (STATS && MODE == kModeFused) accumulate(acc, gbar, xl, xn, mask, nonfinite);
}

// ------------------------------------------------- a vector of every stream
// All loads of a piece are issued before its first store, so that a wavefront
// keeps every stream in flight at once (the compiler cannot move later loads
// above earlier stores by itself: it cannot prove that the streams do not
// overlap).
// Stream counts: G > 0 and PP >= 0 are exact; G < 0 and PP <= -2 are run-time
// counts bounded by -G and -PP, whose missing streams are skipped; G == 0 and
// PP == -1 are unbounded run-time counts (step_any).
template <int G>
constexpr int g_slots() { return G > 0 ? G : (G < 0 ? -G : 0); }
template <int PP>
constexpr int p_slots() { return PP >= 0 ? PP : (PP <= -2 ? -PP : 0); }

constexpr bool has_grads(int mode) { return mode == kModeAvg || mode == kModeFused; }
constexpr bool has_copies(int mode) { return mode == kModeMerge || mode == kModeMean || mode == kModeFused; }
constexpr bool reads_x(int mode) { return mode == kModeMerge || mode == kModeFused; }

template <int MODE, int G, int PP, bool XF>
struct VecIn {
  static constexpr int kG = has_grads(MODE) ? g_slots<G>() : 0;
  static constexpr int kP = has_copies(MODE) ? p_slots<PP>() : 0;
  f32x4 g[kG > 0 ? kG : 1];
  f32x4 x;  // params (merge, fused) or the source (pack)
  f32x4 m;  // momentum (fused)
  typename XType<XF>::Vec s[kP > 0 ? kP : 1];
};

// A stream pointer that is to be in scalar registers from here on: with run-time
// counts each load sits behind a branch of its own, and reading its pointer there too
// would make every load wait for the one before.
template <bool HOLD, typename T>
__device__ __forceinline__ T* held(T* p) {
  if constexpr (HOLD) asm("" : "+s"(p));
  return p;
}

// Every stream's vector at base + off.
template <int MODE, int G, int PP, bool XF>
__device__ __forceinline__ void load_in(const StepArgs& a, int64_t base, uint32_t off, VecIn<MODE, G, PP, XF>& v) {
  using V = VecIn<MODE, G, PP, XF>;
  using X = XType<XF>;
  if constexpr (MODE == kModePack) v.x = load_vec<f32x4>(a.src, base, off);
  if constexpr (V::kG > 0) {
    const float* p[V::kG];
#pragma unroll
    for (int r = 0; r < V::kG; ++r) p[r] = held<(G < 0)>(a.grads[r]);
#pragma unroll
    for (int r = 0; r < V::kG; ++r)
      if (G > 0 || r < a.g) v.g[r] = load_vec<f32x4>(p[r], base, off);
  }
  if constexpr (reads_x(MODE)) v.x = load_vec<f32x4>(a.x, base, off);
  if constexpr (MODE == kModeFused) v.m = load_vec<f32x4>(a.m, base, off);
  constexpr int kHold = 8;
#pragma unroll
  for (int i = 0; i < V::kP; i += kHold) {
    const void* p[kHold];
#pragma unroll
    for (int j = 0; j < kHold; ++j)
      if (i + j < V::kP) p[j] = held<(PP < 0)>(a.stale[i + j]);
#pragma unroll
    for (int j = 0; j < kHold; ++j)
      if (i + j < V::kP && (PP >= 0 || i + j < a.P))
        v.s[i + j] = load_vec<typename X::Vec>(static_cast<const typename X::Elem*>(p[j]), base, off);
  }
}

// The elements of every stream's vector at element e0 that `mask` selects.
template <int MODE, int G, int PP, bool XF>
__device__ __forceinline__ void load_some_in(const StepArgs& a, int64_t e0, unsigned mask, VecIn<MODE, G, PP, XF>& v) {
  using V = VecIn<MODE, G, PP, XF>;
  using X = XType<XF>;
  const auto f32 = [&](const float* p) {
    float h[kVec];
    load_some(p + e0, mask, h);
    return f32x4{h[0], h[1], h[2], h[3]};
  };
#pragma unroll
  for (int r = 0; r < V::kG; ++r)
    if (G > 0 || r < a.g) v.g[r] = f32(a.grads[r]);
  if constexpr (MODE == kModePack) v.x = f32(a.src);
  if constexpr (reads_x(MODE)) v.x = f32(a.x);
  if constexpr (MODE == kModeFused) v.m = f32(a.m);
#pragma unroll
  for (int i = 0; i < V::kP; ++i)
    if (PP >= 0 || i < a.P) {
      typename X::Elem h[kVec];
      load_some(static_cast<const typename X::Elem*>(a.stale[i]) + e0, mask, h);
      v.s[i] = X::joined(h);
    }
}

template <int MODE, int G, int PP, bool XF, bool STATS, bool FULL>
__device__ __forceinline__ void finish(const StepArgs& a, int64_t base, uint32_t off, unsigned mask,
                                       const VecIn<MODE, G, PP, XF>& v, float two_s, const Divisor& qg,
                                       const Divisor& qm, Acc& acc) {
  using V = VecIn<MODE, G, PP, XF>;
  using X = XType<XF>;
  if constexpr (MODE == kModePack) {
    put<FULL>(static_cast<uint16_t*>(a.wire), base, off, mask, any_nonfinite(v.x) ? pack4(v.x) : pack4_no_nan(v.x));
    return;
  }
  f32x4 gbar = {0.f, 0.f, 0.f, 0.f};
  if constexpr (V::kG > 0) {
    f32x4 s = v.g[0];
#pragma unroll
    for (int r = 1; r < V::kG; ++r)
      if (G > 0 || r < a.g) s = s + v.g[r];
    gbar = divide(s, qg);
    if (MODE == kModeAvg || a.gavg) put<FULL, MODE == kModeAvg>(a.gavg, base, off, mask, gbar);
    if constexpr (MODE == kModeAvg) return;
  }
  f32x4 xl = {0.f, 0.f, 0.f, 0.f};  // (mean) not used: 2S is 0
  if constexpr (reads_x(MODE)) xl = v.x;
  if constexpr (MODE == kModeFused) {
    f32x4 m = v.m;
    xl = sgd_momentum4(a, v.x, m, gbar);
    put<FULL>(a.m, base, off, mask, m);
  }
  f32x4 xn = xl;
  if constexpr (V::kP > 0) {
    if (PP >= 0 || a.P > 0) {
      f32x4 sum = merge_start(two_s, xl);
#pragma unroll
      for (int i = 0; i < V::kP; ++i)
        if (PP >= 0 || i < a.P) sum = sum + X::received(v.s[i]);
      xn = divide(sum, qm);
    }
  }
  store_results<MODE, STATS, XF, FULL>(a, base, off, mask, gbar, xl, xn, acc);
}

// Whether an instance has compile-time stream counts or bounds, and so takes
// every stream's vector before the first addition.
template <int MODE, int G, int PP>
constexpr bool batched() {
  if constexpr (MODE == kModePack) return true;
  if constexpr (MODE == kModeAvg) return G != 0;
  if constexpr (MODE == kModeMerge || MODE == kModeMean) return PP != -1;
  return G != 0 && PP != -1;
}

template <int MODE, int G, int PP>
constexpr Counts counts_of() {
  if (!batched<MODE, G, PP>()) return Counts::kUnbounded;
  return (has_grads(MODE) && G < 0) || (has_copies(MODE) && PP < 0) ? Counts::kBounded : Counts::kExact;
}

// Wavefronts per workgroup.  With statistics 4, which share one partial (one
// wavefront each took the resnet50-shaped step from 206.7 to 207.4 us and the
// GPT-shaped one from 6960 to 7120: four times the partials to write and to sum), or 8 for exact
// counts that take 88 to 128 bytes per element (GPT-shaped 6903 against 7005 us, g = 8
// with 16 fp32 copies 498 against 504; the resnet50-shaped step would lose, 219 against 213).
// Without them one, so that a place on a CU is free again as soon as its own loads and
// stores are done (resnet50-shaped 196 against 204 us, the average of 8 gradients
// 140 against 145, g = 8 with 12 fp32 copies 406 against 437), except for exact
// counts that take 88 bytes per element or more, or merges of 32 bf16 copies: there 4
// wavefronts on one CU run 1 to 9% faster than 4 spread over the chip (g = 8, P = 32: 473
// against 486 us; the merge 289 against 300 at best, the mean 263 against 282).
template <int MODE, int G, int PP, bool XF>
constexpr bool heavy() {
  using V = VecIn<MODE, G, PP, XF>;
  constexpr int bytes = 4 * V::kG + (XF ? 4 : 2) * V::kP + (MODE == kModeFused ? 8 : reads_x(MODE) ? 4 : 0);
  constexpr bool merge32 = MODE != kModeFused && !XF && V::kP >= 32;
  return counts_of<MODE, G, PP>() == Counts::kExact && (bytes >= 88 || merge32);
}

template <int MODE, int G, int PP, bool STATS, bool XF>
constexpr int waves_of() {
  constexpr bool is_heavy = heavy<MODE, G, PP, XF>();
  if (STATS) return is_heavy && 4 * G + (XF ? 4 : 2) * PP + 8 <= 128 ? 8 : 4;
  return is_heavy ? 4 : 1;
}

// A short call has few workgroups of eight for the CUs there are: it takes fours (g = 8,
// P = 32, 131,072 parameters 7.0 us against 7.8, 1M 20.4 and 21.5, 3M 61.7 and 63.7, but 25.6M
// 497 and 479).  `f` is called with the number of wavefronts per workgroup, a compile-time constant.
template <int MODE, int G, int PP, bool STATS, bool XF, typename F>
auto with_waves(const StepArgs& a, const F& f) {
  constexpr int kWaves = waves_of<MODE, G, PP, STATS, XF>();
  if constexpr (kWaves == 8)
    if (a.n <= kShortCall) return f(std::integral_constant<int, 4>{});
  return f(std::integral_constant<int, kWaves>{});
}

// ------------------------------------------------- unbounded run-time counts
// How the lanes of a wavefront take the vectors of which `mask` selects elements: kWhole, all are
// selected; kCut, one by one; kRead, one by one from params and momentum, whose other elements
// another wavefront may be writing, and whole from the gradients and copies (see whole_reads).
enum class Lanes { kWhole, kRead, kCut };

template <bool FULL, typename V, typename T>
__device__ __forceinline__ V get(const T* p, int64_t base, uint32_t off, unsigned mask) {
  if constexpr (FULL) {
    return load_vec<V>(p, base, off);
  } else {
    T h[kVec];
    load_some(p + base + off, mask, h);
    V v;
    __builtin_memcpy(&v, h, sizeof(v));
    return v;
  }
}

// Whether a piece's gradients and copies may be read as whole vectors whatever elements are
// selected: none of the vectors reaches past the buffers' n elements, and no gradient is
// being overwritten with the average.  Four loads in place of one for every stream of a cut
// piece are the longest chain of a short call (g = 9, P = 40, 30,000 parameters in two buckets
// without statistics 18.6 us, with whole vectors 10.7; 25.6M parameters 581 and 577).
__device__ __forceinline__ bool whole_reads(const StepArgs& a, int64_t base) {
  return a.in_place_avg == 0 && (base + kPiece <= a.n || (a.n & (kVec - 1)) == 0);
}

// sum + p[0] + p[1] + ...  Streams come in batches, the loads of a batch all
// issued before its additions, which run in stream order.  Batches of 8 leave room
// for enough wavefronts to cover their latency (g = 4, P = 64 and g = 3, P = 40, 25.6M
// parameters: 690 and 459 us; batches of 16 712 and 472, with the next batch loaded before
// this one's additions 714 and 473).
template <bool XF, bool FULL>
__device__ __forceinline__ f32x4 add_streams(f32x4 sum, const void* const* p, int count, int64_t base, uint32_t off,
                                             unsigned mask) {
  using X = XType<XF>;
  constexpr int kBatch = 8;
  static_assert(DASO_MAX_G % kBatch == 0 && DASO_MAX_P % kBatch == 0, "a batch's pointers lie within StepArgs' arrays");
  for (int i = 0; i < count; i += kBatch) {
    const void* q[kBatch];
    typename X::Vec t[kBatch];
#pragma unroll
    for (int j = 0; j < kBatch; ++j) q[j] = held<FULL>(p[i + j]);
#pragma unroll
    for (int j = 0; j < kBatch; ++j)
      if (i + j < count) t[j] = get<FULL, typename X::Vec>(static_cast<const typename X::Elem*>(q[j]), base, off, mask);
#pragma unroll
    for (int j = 0; j < kBatch; ++j)
      if (i + j < count) sum = sum + X::received(t[j]);
  }
  return sum;
}

template <int MODE, bool STATS, bool XF, Lanes L>
__device__ __forceinline__ void step_any(const StepArgs& a, int64_t base, uint32_t off, unsigned mask, float two_s,
                                         const Divisor& qg, const Divisor& qm, Acc& acc) {
  constexpr bool FULL = L == Lanes::kWhole, READ = L != Lanes::kCut;
  f32x4 xl = {0.f, 0.f, 0.f, 0.f};  // (mean) not used: 2S is 0
  f32x4 m = {0.f, 0.f, 0.f, 0.f};
  if constexpr (reads_x(MODE)) xl = get<FULL, f32x4>(a.x, base, off, mask);
  if constexpr (MODE == kModeFused) m = get<FULL, f32x4>(a.m, base, off, mask);
  f32x4 gbar = {0.f, 0.f, 0.f, 0.f};
  if constexpr (has_grads(MODE)) {
    // -0 + G_0 == G_0 for every G_0
    gbar = divide(add_streams<true, READ>(f32x4{-0.0f, -0.0f, -0.0f, -0.0f},
                                          reinterpret_cast<const void* const*>(a.grads), a.g, base, off, mask), qg);
    if (MODE == kModeAvg || a.gavg) put<FULL, MODE == kModeAvg>(a.gavg, base, off, mask, gbar);
    if constexpr (MODE == kModeAvg) return;
  }
  if constexpr (MODE == kModeFused) {
    xl = sgd_momentum4(a, xl, m, gbar);
    put<FULL>(a.m, base, off, mask, m);
  }
  f32x4 xn = xl;
  if (a.P > 0) xn = divide(add_streams<XF, READ>(merge_start(two_s, xl), a.stale, a.P, base, off, mask), qm);
  store_results<MODE, STATS, XF, FULL>(a, base, off, mask, gbar, xl, xn, acc);
}

// ------------------------------------------------------------------ buckets
// The bucket of the launch that holds element e: the last whose start is not
// past it (buckets are sorted by start; of several at one start all but the last
// are empty).
__device__ __forceinline__ int bucket_of(const StepArgs& a, int64_t e) {
  int lo = 0, hi = a.nb - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.start[mid] <= e) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// The statistics of one bucket: the whole workgroup sums the partials [t0, t1)
// in a fixed assignment and reduction tree (thread k adds partials t0 + k,
// t0 + k + kBlock, ... in that order), so the result does not depend on timing,
// on which kernel runs it or on kLoads.  Valid in thread 0.
// The sum is latency-bound: each thread issues the loads of up to kLoads
// partials before it adds them in order.  Missing ones count as zeros, which
// leaves every sum unchanged (sums of squares are never -0).
template <bool SHARED, typename T>
__device__ __forceinline__ T partial_word(const T& p) {
  if constexpr (SHARED) return __hip_atomic_load(&p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else return p;
}

template <int kLoads, bool SHARED, int kWaves>
__device__ __forceinline__ Acc64 bucket_stats(const SlicePartial* partials, int64_t t0, int64_t t1,
                                              WaveSums<kWaves>& s) {
  constexpr int kThreads = 64 * kWaves;
  Acc64 v = {0.0, 0.0, 0};
  for (int64_t base = t0 + static_cast<int64_t>(threadIdx.x); base < t1; base += kThreads * kLoads) {
    SlicePartial p[kLoads];
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      const int64_t j = base + u * kThreads;
      p[u] = SlicePartial{0.0, 0.0, 0};
      if (j < t1)
        p[u] = SlicePartial{partial_word<SHARED>(partials[j].grad_sq), partial_word<SHARED>(partials[j].delta_sq),
                            partial_word<SHARED>(partials[j].nonfinite)};
    }
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
      v.gsq += p[u].grad_sq;
      v.dsq += p[u].delta_sq;
      v.nf += p[u].nonfinite;
    }
  }
  __syncthreads();  // s may still be read from the call before
  return block_sum(v, s);
}

__device__ __forceinline__ void put_stats(daso_bucket_stats* stats, const BucketSlots& t, Acc64 r) {
  daso_bucket_stats* out = stats + t.out;
  if (t.add) r = Acc64{out->grad_sq + r.gsq, out->delta_sq + r.dsq, out->nonfinite + r.nf};
  out->grad_sq = r.gsq;
  out->delta_sq = r.dsq;
  out->nonfinite = r.nf;
}

// The partials of bucket i of a launch.
template <int SHIFT>
__device__ __forceinline__ BucketSlots slots_of(const StepArgs& a, int i) {
  const int64_t bs = a.start[i], be = a.start[i + 1];
  const int64_t first = a.slot0 + slot_of((bs >> SHIFT) - a.sb0, i);
  return BucketSlots{first, be > bs ? a.slot0 + slot_of(((be - 1) >> SHIFT) - a.sb0, i) + 8 : first, a.out[i],
                     i == 0 ? a.cont : 0};
}

// A launch of few workgroups sums its statistics in its own last workgroup instead
// of a second launch.  The partials are agent-scope atomic stores, which the
// hardware completes at the point that all XCDs share; a workgroup waits for its own to
// complete and then counts itself done, and the one that counts last reads them with
// agent-scope atomic loads.  So no workgroup needs the release fence, whose write-back of
// its XCD's L2 (about 0.1 us each, one after the other) is for ordinary stores.
// The last workgroup sums every bucket in the order of stats_kernel (no thread has more
// than one partial to add, so that the smaller workgroup changes nothing) and sets the
// counter back to zero for the next launch.
template <int SHIFT, int kWaves>
__device__ __forceinline__ void finish_stats_if_last(const StepArgs& a, WaveSums<kWaves>& s) {
  __shared__ bool last;
  if (threadIdx.x == 0) {  // which stored this workgroup's partials
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    // such a launch has one row of workgroups
    last = __hip_atomic_fetch_add(a.done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gridDim.x - 1;
  }
  __syncthreads();
  if (!last) return;
  for (int i = 0; i < a.nb; ++i) {
    const BucketSlots t = slots_of<SHIFT>(a, i);
    const Acc64 r = bucket_stats<1, true>(a.partials, t.first, t.end, s);
    if (threadIdx.x == 0) put_stats(a.stats, t, r);
  }
  if (threadIdx.x == 0) __hip_atomic_store(a.done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ------------------------------------------------------------------- kernel
// The elements of the vector at e0 that lie in [lo, hi), as a mask.
__device__ __forceinline__ unsigned vec_mask(int64_t e0, int64_t lo, int64_t hi) {
  unsigned mask = 0;
#pragma unroll
  for (int k = 0; k < kVec; ++k)
    if (e0 + k >= lo && e0 + k < hi) mask |= 1u << k;
  return mask;
}

// One workgroup per slice (see the work decomposition in daso_plan.h).
//
// The step is bound by HBM: while a wavefront's loads are not in flight, its place
// on the CU is idle, so everything else is kept off the way to them.  The loads depend
// on nothing but the workgroup's index; the bucket (the staleness S, the
// place of its statistics) is looked up while they are in flight.  Against the
// tiles that came before (2048 or 1024 elements of one bucket each, in runs per XCD,
// looked up first), same buffers in turn: ragged step 82.7 to 78.0 us, many small
// buckets 712 to 680, resnet50-shaped 216 to 206 (without statistics 213.5 to 196),
// the average of 8 gradients 444 to 399, merges 5 to 9% faster; boxes differ by a few percent.
template <int MODE, int G, int PP, bool STATS, bool XF, int kWaves>
__global__ __launch_bounds__(64 * kWaves) void step_kernel(const StepArgs a) {
  constexpr bool kBatched = batched<MODE, G, PP>();
  constexpr bool kStats = STATS && MODE == kModeFused;
  constexpr int kShift = super_shift(kWaves);
  const int64_t w = (int64_t(blockIdx.y) << kRowShift) + blockIdx.x;
  const int wave = kWaves == 1 ? 0 : __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const uint32_t off = (threadIdx.x & 63u) * kVec;  // of the lane's elements in its piece
  const int64_t sbase = (a.sb0 + (w >> 3)) << kShift;
  const int64_t base = sbase + (wave * 8 + static_cast<int>(w & 7)) * kPiece;
  const bool whole = base >= a.lo && base + kPiece <= a.hi;
  // the buckets that overlap the superblock (with statistics: the workgroup
  // writes a partial for each) or the piece
  const int64_t from = kStats ? sbase : base, to = kStats ? sbase + (int64_t(1) << kShift) : base + kPiece;
  const Divisor qg = (G > 0) ? make_divisor(G, 1.0f / (G > 0 ? G : 1)) : make_divisor(a.g, a.g_inv);
  const int P = (PP >= 0) ? PP : a.P;
  __shared__ WaveSums<kWaves> s_sum;
  const auto put_partial = [&](int b, const Acc& acc) {
    const Acc64 t = block_sum(acc, s_sum);
    if (threadIdx.x == 0) {
      const int64_t slot = a.slot0 + slot_of((sbase >> kShift) - a.sb0, b) + (w & 7);
      SlicePartial* p = a.partials + slot;
      if (a.done != nullptr) {
        __hip_atomic_store(&p->grad_sq, t.gsq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&p->delta_sq, t.dsq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&p->nonfinite, t.nf, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else {
        *p = SlicePartial{t.gsq, t.dsq, t.nf};
      }
    }
  };
  VecIn<MODE, G, PP, XF> v;
  int b = 0;
  bool done = false;
  if (__builtin_expect(whole, 1)) {
    if constexpr (kBatched) load_in<MODE, G, PP, XF>(a, base, off, v);
    b = bucket_of(a, from > a.lo ? from : a.lo);
    if (__builtin_expect(from >= a.start[b] && to <= a.start[b + 1], 1)) {  // all in one bucket
      const Divisor qm = make_divisor(2 * a.S[b] + P, a.inv[b]);
      const float two_s = static_cast<float>(2 * a.S[b]);
      Acc acc = {0.0, 0.0, 0u};
      if constexpr (kBatched) finish<MODE, G, PP, XF, STATS, true>(a, base, off, 0xFu, v, two_s, qg, qm, acc);
      else step_any<MODE, STATS, XF, Lanes::kWhole>(a, base, off, 0xFu, two_s, qg, qm, acc);
      if constexpr (kStats) put_partial(b, acc);
      done = true;
    }
  } else {
    done = w >= a.nslices;
    if (!done) {
      b = bucket_of(a, from > a.lo ? from : a.lo);
      if constexpr (kBatched) {
        const unsigned mask = vec_mask(base + off, a.lo, a.hi);
        // The vectors of a call that ends at multiples of 4 are whole or not touched.  Where a vector
        // has many loads, four for each are the longest chain of a short call (g = 8, P = 32, 30,000
        // parameters 7.7 us, without statistics 5.8; 6.5 and 4.5 with whole ones).
        if (heavy<MODE, G, PP, XF>() && ((a.lo | a.hi) & (kVec - 1)) == 0) {
          if (mask) load_in<MODE, G, PP, XF>(a, base, off, v);
        } else if (mask) {
          load_some_in<MODE, G, PP, XF>(a, base + off, mask, v);
        }
      }
    }
  }
  if (!done) {
    // With unbounded counts a lane's streams are read batch after batch, the longest chain of a
    // short call, so a piece whose vectors each lie in one bucket takes all its buckets in one pass,
    // before the workgroup meets for the first one's partial (g = 9, P = 40, two buckets in
    // 30,000 parameters 10.9 us against 14.7, without statistics 7.4 and 10.7; in 500,000 14.8 and 20.9).
    bool once = false;
    int own = -1;  // the lane's bucket
    Acc of_own = {0.0, 0.0, 0u};
    if constexpr (!kBatched) {
      const int64_t e = base + off;
      Divisor qm = make_divisor(1, 1.0f);
      float two_s = 0.0f;
      for (int k = bucket_of(a, base > a.lo ? base : a.lo);; ++k) {
        if (e >= a.start[k] && e + kVec <= a.start[k + 1]) {
          own = k;
          qm = make_divisor(2 * a.S[k] + P, a.inv[k]);
          two_s = static_cast<float>(2 * a.S[k]);
        }
        if (k + 1 >= a.nb || a.start[k + 1] >= base + kPiece) break;
      }
      once = __ballot(own < 0 && vec_mask(e, a.lo, a.hi) != 0) == 0;
      if (once && own >= 0) step_any<MODE, STATS, XF, Lanes::kWhole>(a, base, off, 0xFu, two_s, qg, qm, of_own);
      if (once && !kStats) return;
    }
    // one bucket after the other; each lane stores the elements of its vector that lie in it
    for (;; ++b) {
      const Divisor qm = make_divisor(2 * a.S[b] + P, a.inv[b]);
      const float two_s = static_cast<float>(2 * a.S[b]);
      Acc acc = {0.0, 0.0, 0u};
      if (once && b == own) acc = of_own;
      const unsigned mask = once ? 0u : vec_mask(base + off, a.start[b], a.start[b + 1]);
      if (mask) {
        if constexpr (kBatched) finish<MODE, G, PP, XF, STATS, false>(a, base, off, mask, v, two_s, qg, qm, acc);
        else if (whole_reads(a, base)) step_any<MODE, STATS, XF, Lanes::kRead>(a, base, off, mask, two_s, qg, qm, acc);
        else step_any<MODE, STATS, XF, Lanes::kCut>(a, base, off, mask, two_s, qg, qm, acc);
      }
      if constexpr (kStats) {
        put_partial(b, acc);
        __syncthreads();  // before s_sum is written again
      }
      if (b + 1 >= a.nb || a.start[b + 1] >= to) break;
    }
  }
  if constexpr (kStats) {
    static_assert(64 * kWaves >= kLaunchBuckets, "one thread per bucket writes the table");
    // for stats_kernel (the grid has at least one workgroup)
    if (w == 0 && threadIdx.x < a.nb) a.table[threadIdx.x] = slots_of<kShift>(a, static_cast<int>(threadIdx.x));
    if (a.done != nullptr) finish_stats_if_last<kShift>(a, s_sum);
  }
}

// A launch of small buckets only: with statistics a workgroup of 4 wavefronts for each, which
// writes the bucket's statistics itself and leaves the statistics pass of the call's other launches an
// empty entry to add; without, a wavefront for every 256 elements of the largest bucket.
// step_kernel takes the buckets of a piece (without statistics) or of a superblock one after the
// other, at 0.4 us each and more with many streams, and a launch of 128 small ones has
// few of either.
constexpr int bucket_waves(bool stats) { return stats ? 4 : 1; }

template <int MODE, bool STATS, bool XF>
__global__ __launch_bounds__(64 * bucket_waves(STATS)) void bucket_kernel(const StepArgs a) {
  constexpr int kWaves = bucket_waves(STATS);
  const int i = static_cast<int>(blockIdx.x);
  const int wave = kWaves == 1 ? static_cast<int>(blockIdx.y) : __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
  const int waves = kWaves == 1 ? static_cast<int>(gridDim.y) : kWaves;
  const int64_t bs = a.start[i], be = a.start[i + 1];
  const Divisor qg = make_divisor(a.g, a.g_inv), qm = make_divisor(2 * a.S[i] + a.P, a.inv[i]);
  const float two_s = static_cast<float>(2 * a.S[i]);
  const uint32_t off = (threadIdx.x & 63u) * kVec;
  Acc acc = {0.0, 0.0, 0u};
  for (int64_t base = (bs & -int64_t(kVec)) + wave * kPiece; base < be; base += waves * kPiece) {
    const unsigned mask = vec_mask(base + off, bs, be);
    if (whole_reads(a, base)) {
      if (mask) step_any<MODE, STATS, XF, Lanes::kRead>(a, base, off, mask, two_s, qg, qm, acc);
    } else if (mask) {
      step_any<MODE, STATS, XF, Lanes::kCut>(a, base, off, mask, two_s, qg, qm, acc);
    }
  }
  if constexpr (STATS) {
    __shared__ WaveSums<kWaves> s_sum;
    const Acc64 r = block_sum(acc, s_sum);
    if (threadIdx.x == 0) {
      put_stats(a.stats, BucketSlots{0, 0, a.out[i], i == 0 ? a.cont : 0}, r);
      a.table[i] = BucketSlots{0, 0, a.out[i], 1};
    }
  }
}

// Sets the counter of StepArgs::done at the start of a new statistics buffer
// to zero (a kernel rather than a memset, so that it may also sit in a graph).
__global__ void clear_counter_kernel(uint32_t* counter) {
  if (threadIdx.x == 0) *counter = 0u;
}

// Statistics of one launch: workgroup i sums the partials of bucket i.
// Runs after step_kernel on the same stream, which makes every partial, and the
// table, visible without any fence inside step_kernel.
__global__ __launch_bounds__(kStatsBlock) void stats_kernel(const StatsArgs a) {
  __shared__ WaveSums<kStatsBlock / 64> s_sum;
  const BucketSlots t = a.table[blockIdx.x];
  // 8 loads per thread in flight: a 25 MiB bucket has about 6 partials for each
  const Acc64 r = bucket_stats<8, false>(a.partials, t.first, t.end, s_sum);
  if (threadIdx.x == 0) put_stats(a.stats, t, r);
}

// Fused instances: compile-time stream counts for the node shapes, g = 4 or 8
// replicas (the GPUs of a node) with P in {2, 4, 8, 16, 32, 64} exchanged copies (the
// nodes of a group), and for the local step (P = 0); counts bounded by 4 or 8
// replicas and 8, 16 or 32 copies for the rest, whose missing streams are
// skipped; unbounded run-time counts beyond 8 replicas or 32 copies.  A bound of 64
// copies does not fit the registers of two wavefronts per SIMD (g = 3, P = 40: 574
// us against 497 with unbounded counts); for a few streams less than its bound an instance
// loses nothing (g = 5, P = 20 with a bound of 32: 332 us against 456 unbounded).
template <bool STATS, bool XF, int GB, typename F>
auto dispatch_bounded(const StepArgs& a, const F& f) {
  if (a.P <= 8) return f.template run<kModeFused, GB, -8, STATS, XF>();
  if (a.P <= 16) return f.template run<kModeFused, GB, -16, STATS, XF>();
  if (a.P <= 32) return f.template run<kModeFused, GB, -32, STATS, XF>();
  return f.template run<kModeFused, 0, -1, STATS, XF>();
}

template <bool STATS, bool XF, int G, typename F>
auto dispatch_node(const StepArgs& a, const F& f) {
  switch (a.P) {
    case 0: return f.template run<kModeFused, G, 0, STATS, XF>();
    case 2: return f.template run<kModeFused, G, 2, STATS, XF>();
    case 4: return f.template run<kModeFused, G, 4, STATS, XF>();
    case 8: return f.template run<kModeFused, G, 8, STATS, XF>();
    case 16: return f.template run<kModeFused, G, 16, STATS, XF>();
    case 32: return f.template run<kModeFused, G, 32, STATS, XF>();
    default: break;
  }
  if constexpr (!XF)
    if (a.P == 64) return f.template run<kModeFused, G, 64, STATS, false>();
  return dispatch_bounded<STATS, XF, -G>(a, f);
}

template <bool STATS, bool XF, typename F>
auto dispatch_fused(const StepArgs& a, const F& f) {
  if (a.g > 8) return f.template run<kModeFused, 0, -1, STATS, XF>();
  if (a.g == 4) return dispatch_node<STATS, XF, 4>(a, f);
  if (a.g == 8) return dispatch_node<STATS, XF, 8>(a, f);
  if (!XF && a.P == 0) {
    if (a.g == 1) return f.template run<kModeFused, 1, 0, STATS, false>();
    if (a.g == 2) return f.template run<kModeFused, 2, 0, STATS, false>();
  }
  if (a.g < 4) return dispatch_bounded<STATS, XF, -4>(a, f);
  return dispatch_bounded<STATS, XF, -8>(a, f);
}

template <int MODE, bool XF, typename F>
auto dispatch_merge(const StepArgs& a, const F& f) {
  switch (a.P) {
    case 0: return f.template run<kModeMerge, 0, 0, false, XF>();  // never the mean of nothing
    case 2: return f.template run<MODE, 0, 2, false, XF>();
    case 4: return f.template run<MODE, 0, 4, false, XF>();
    case 8: return f.template run<MODE, 0, 8, false, XF>();
    case 16: return f.template run<MODE, 0, 16, false, XF>();
    case 32: return f.template run<MODE, 0, 32, false, XF>();
    default: break;
  }
  if (a.P <= 8) return f.template run<MODE, 0, -8, false, XF>();
  if (a.P <= 16) return f.template run<MODE, 0, -16, false, XF>();
  if (a.P <= 32) return f.template run<MODE, 0, -32, false, XF>();
  return f.template run<MODE, 0, -1, false, XF>();
}

// The instance for a call, chosen in one place: `f.template run<MODE, G, PP,
// STATS, XF>()` is called for it.  Fully unrolled instances exist for common stream counts;
// any other count takes the runtime-count instance, which computes the same bits.
template <typename F>
auto dispatch(Mode mode, bool with_stats, const StepArgs& a, const F& f) {
  switch (mode) {
    case kModeAvg:
      switch (a.g) {
        case 1: return f.template run<kModeAvg, 1, -1, false, false>();
        case 2: return f.template run<kModeAvg, 2, -1, false, false>();
        case 4: return f.template run<kModeAvg, 4, -1, false, false>();
        case 8: return f.template run<kModeAvg, 8, -1, false, false>();
        default:
          if (a.g <= 8) return f.template run<kModeAvg, -8, -1, false, false>();
          return f.template run<kModeAvg, 0, -1, false, false>();
      }
    case kModePack:
      return f.template run<kModePack, 0, -1, false, false>();
    case kModeMerge: return a.xf32 ? dispatch_merge<kModeMerge, true>(a, f) : dispatch_merge<kModeMerge, false>(a, f);
    case kModeMean: return a.xf32 ? dispatch_merge<kModeMean, true>(a, f) : dispatch_merge<kModeMean, false>(a, f);
    case kModeFused:
    default:
      if (a.xf32) return with_stats ? dispatch_fused<true, true>(a, f) : dispatch_fused<false, true>(a, f);
      return with_stats ? dispatch_fused<true, false>(a, f) : dispatch_fused<false, false>(a, f);
  }
}

// Launches report their own status (hipLaunchKernel's return value), so an
// error left behind by an earlier, unrelated HIP call is neither blamed on
// this call nor consumed by it.
struct Launcher {
  const StepArgs& a;
  dim3 grid;
  uint32_t lds;  // LDS held per workgroup (unused by the kernel; caps workgroups per CU)
  hipStream_t stream;
  template <int MODE, int G, int PP, bool STATS, bool XF>
  hipError_t run() const {
    void* args[] = {const_cast<StepArgs*>(&a)};
    return with_waves<MODE, G, PP, STATS, XF>(a, [&](auto waves) {
      return hipLaunchKernel(reinterpret_cast<const void*>(&step_kernel<MODE, G, PP, STATS, XF, waves()>), grid,
                             dim3(64 * waves()), args, lds, stream);
    });
  }
};

struct ShapeOf {
  const StepArgs& a;
  template <int MODE, int G, int PP, bool STATS, bool XF>
  Shape run() const {
    return with_waves<MODE, G, PP, STATS, XF>(
        a, [](auto waves) { return Shape{waves(), counts_of<MODE, G, PP>()}; });
  }
};

}  // namespace

Shape launch_shape(Mode mode, bool with_stats, const StepArgs& a) { return dispatch(mode, with_stats, a, ShapeOf{a}); }

hipError_t launch_step(Mode mode, bool with_stats, const StepArgs& a, dim3 grid, uint32_t lds, hipStream_t stream) {
  return dispatch(mode, with_stats, a, Launcher{a, grid, lds, stream});
}

hipError_t launch_buckets(Mode mode, bool with_stats, const StepArgs& a, int32_t waves, hipStream_t stream) {
  const void* k = nullptr;
  if (mode == kModeFused && with_stats)
    k = a.xf32 ? reinterpret_cast<const void*>(&bucket_kernel<kModeFused, true, true>)
               : reinterpret_cast<const void*>(&bucket_kernel<kModeFused, true, false>);
  else if (mode == kModeFused)
    k = a.xf32 ? reinterpret_cast<const void*>(&bucket_kernel<kModeFused, false, true>)
               : reinterpret_cast<const void*>(&bucket_kernel<kModeFused, false, false>);
  else
    k = a.xf32 ? reinterpret_cast<const void*>(&bucket_kernel<kModeMerge, false, true>)
               : reinterpret_cast<const void*>(&bucket_kernel<kModeMerge, false, false>);
  void* args[] = {const_cast<StepArgs*>(&a)};
  const dim3 grid(static_cast<uint32_t>(a.nb), static_cast<uint32_t>(with_stats ? 1 : waves));
  return hipLaunchKernel(k, grid, dim3(64 * bucket_waves(with_stats)), args, 0, stream);
}

hipError_t launch_stats(const SlicePartial* partials, const BucketSlots* table, daso_bucket_stats* stats, int32_t nb,
                        hipStream_t stream) {
  StatsArgs a = {partials, table, stats};
  void* args[] = {&a};
  return hipLaunchKernel(reinterpret_cast<const void*>(&stats_kernel), dim3(static_cast<uint32_t>(nb)),
                         dim3(kStatsBlock), args, 0, stream);
}

hipError_t clear_stats_counter(void* buffer, hipStream_t stream) {
  void* args[] = {&buffer};
  return hipLaunchKernel(reinterpret_cast<const void*>(&clear_counter_kernel), dim3(1), dim3(64), args, 0, stream);
}

}  // namespace daso
