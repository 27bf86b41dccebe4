// kc_compare.hip -- gfx950 typed compare of candidate / golden buffer pairs.
//
// One launch walks a tile list that covers every pair (uneven sizes, mixed
// element types).  A workgroup takes a run of consecutive tiles and streams
// each pair's part of it in rounds of kUnroll 16-byte loads per thread and
// side.  A round whose bytes are equal and hold no NaN ends there.  In any other, each
// lane marks its elements that differ (or are NaN) in a bit mask, the round's
// bytes are staged in LDS (so that the next round's loads can go to the same
// registers while this one is worked on), and the lanes then take their marked
// elements one per step through the exact path (ULP distance, fp64 abs / rel
// error, NaN classes): a round costs as many steps as the lane with the most
// marked elements has, not one per element.
//
// What bounds it: memory while few elements differ, the exact path's
// instructions when many do.  So that path holds no division unless the
// relative error is about to grow (see rel_may_grow), keeps the running maxima
// and the first mismatch per workgroup in LDS (a wave writes at most once a
// round, when it exceeds them), and counts into a ULP histogram of kHistCopies copies, one
// per LDS bank, so that lanes with the same distance do not queue on one bin.
//
// Measured (16 pairs of f16, bf16, f32 and fp8, 768 MiB a side, 11.3 % of the
// elements off): 0.38 ms a call, 1.95 ms when every element of a run that
// differed took the exact path with its division; 10,000 uneven pairs of 8 GiB
// a side with 1e-4 off: 2.50 ms (6.9 TB/s) against 3.16.  The loads of the next
// round are issued run by run, as each run has been looked at: issued together
// after the last, those 10,000 pairs took 2 % longer.
//
// A workgroup's totals of a pair go to per-pair accumulators with integer
// atomics (max of non-negative doubles via their bit patterns, first mismatch
// via max of its complement), nothing if its elements were all equal, and a
// second small kernel writes the reports once the pass has finished.  When every
// pair is one tile neither is needed: its workgroup writes the report, and the
// call is one launch (16 pairs of 64 KiB: see kCompareWideTile).
#include "kc_device.h"
#include "kc_internal.h"

namespace kc {
namespace {

constexpr uint32_t kThreads = 256, kWideThreads = 1024;
constexpr uint32_t kUnroll = 4;
constexpr uint32_t kBins = 48;

// Element formats.  B holds one element's encoding; kind 0 = floating point
// in sign-magnitude order, 1 = two's complement integer, 2 = raw bytes.
template <uint32_t DT> struct Fmt;
template <> struct Fmt<KC_F32> {
  using B = uint32_t;
  static constexpr uint32_t size = 4, kind = 0;
  static constexpr B mag = 0x7FFFFFFFu;
  __device__ static bool nan(B b) { return (b & mag) > 0x7F800000u; }
  __device__ static bool inf(B b) { return (b & mag) == 0x7F800000u; }
  __device__ static double value(B b) { return (double)__uint_as_float(b); }
};
template <> struct Fmt<KC_F64> {
  using B = uint64_t;
  static constexpr uint32_t size = 8, kind = 0;
  static constexpr B mag = 0x7FFFFFFFFFFFFFFFull;
  __device__ static bool nan(B b) { return (b & mag) > 0x7FF0000000000000ull; }
  __device__ static bool inf(B b) { return (b & mag) == 0x7FF0000000000000ull; }
  __device__ static double value(B b) { return __longlong_as_double((long long)b); }
};
template <> struct Fmt<KC_BF16> {
  using B = uint32_t;
  static constexpr uint32_t size = 2, kind = 0;
  static constexpr B mag = 0x7FFFu;
  __device__ static bool nan(B b) { return (b & mag) > 0x7F80u; }
  __device__ static bool inf(B b) { return (b & mag) == 0x7F80u; }
  __device__ static double value(B b) { return (double)__uint_as_float(b << 16); }
};
// An 8-bit float's magnitude bits moved to the exponent and mantissa fields of
// a binary32 and scaled by the difference of the biases: exact, subnormals
// included (binary32 subnormal inputs are not flushed).
__device__ __forceinline__ double small_value(uint32_t b, uint32_t mbits, float scale) {
  const float v = __uint_as_float((b & 0x7Fu) << (23u - mbits)) * scale;
  return (double)((b & 0x80u) ? -v : v);
}
template <> struct Fmt<KC_F16> {
  using B = uint32_t;
  static constexpr uint32_t size = 2, kind = 0;
  static constexpr B mag = 0x7FFFu;
  __device__ static bool nan(B b) { return (b & mag) > 0x7C00u; }
  __device__ static bool inf(B b) { return (b & mag) == 0x7C00u; }
  __device__ static double value(B b) { return (double)(float)__builtin_bit_cast(_Float16, (uint16_t)b); }
};
template <> struct Fmt<KC_FP8_E4M3FN> {
  using B = uint32_t;
  static constexpr uint32_t size = 1, kind = 0;
  static constexpr B mag = 0x7Fu;
  __device__ static bool nan(B b) { return (b & mag) == 0x7Fu; }
  __device__ static bool inf(B) { return false; }
  __device__ static double value(B b) { return small_value(b, 3, 0x1p120f); }  // bias 127 - 7
};
template <> struct Fmt<KC_FP8_E4M3FNUZ> {
  using B = uint32_t;
  static constexpr uint32_t size = 1, kind = 0;
  static constexpr B mag = 0x7Fu;
  __device__ static bool nan(B b) { return b == 0x80u; }
  __device__ static bool inf(B) { return false; }
  __device__ static double value(B b) { return small_value(b, 3, 0x1p119f); }
};
template <> struct Fmt<KC_FP8_E5M2> {
  using B = uint32_t;
  static constexpr uint32_t size = 1, kind = 0;
  static constexpr B mag = 0x7Fu;
  __device__ static bool nan(B b) { return (b & mag) > 0x7Cu; }
  __device__ static bool inf(B b) { return (b & mag) == 0x7Cu; }
  __device__ static double value(B b) {
    const double inf = (b & 0x80u) ? -__builtin_inf() : __builtin_inf();
    return (b & mag) == 0x7Cu ? inf : small_value(b, 2, 0x1p112f);
  }
};
template <> struct Fmt<KC_FP8_E5M2FNUZ> {
  using B = uint32_t;
  static constexpr uint32_t size = 1, kind = 0;
  static constexpr B mag = 0x7Fu;
  __device__ static bool nan(B b) { return b == 0x80u; }
  __device__ static bool inf(B) { return false; }
  __device__ static double value(B b) { return small_value(b, 2, 0x1p111f); }
};
template <uint32_t SIZE, typename BT> struct IntFmt {
  using B = BT;
  static constexpr uint32_t size = SIZE, kind = 1;
  static constexpr B mag = 0;
  __device__ static bool nan(B) { return false; }
  __device__ static bool inf(B) { return false; }
  __device__ static int64_t sext(B b) {
    if (SIZE == 1) return (int64_t)(int8_t)(uint8_t)b;
    if (SIZE == 2) return (int64_t)(int16_t)(uint16_t)b;
    if (SIZE == 4) return (int64_t)(int32_t)(uint32_t)b;
    return (int64_t)b;
  }
  __device__ static double value(B b) { return (double)sext(b); }
};
template <> struct Fmt<KC_I8> : IntFmt<1, uint32_t> {};
template <> struct Fmt<KC_I16> : IntFmt<2, uint32_t> {};
template <> struct Fmt<KC_I32> : IntFmt<4, uint32_t> {};
template <> struct Fmt<KC_I64> : IntFmt<8, uint64_t> {};
template <> struct Fmt<KC_U8> {
  using B = uint32_t;
  static constexpr uint32_t size = 1, kind = 2;
  __device__ static bool nan(B) { return false; }
  __device__ static bool inf(B) { return false; }
  __device__ static double value(B) { return 0.0; }
};

// Top bit of every element lane (byte, half-word, word) of a 32-bit word.
template <uint32_t SIZE> constexpr uint32_t kTops = SIZE == 1 ? 0x80808080u : (SIZE == 2 ? 0x80008000u : 0x80000000u);

// Top bits of the element lanes of x that are not zero.
template <uint32_t SIZE> __device__ __forceinline__ uint32_t nonzero_tops(uint32_t x) {
  constexpr uint32_t rest = ~kTops<SIZE>;
  return (((x & rest) + rest) | x) & kTops<SIZE>;
}

// Top bits of the element lanes of golden word i of a 16-byte run that hold a
// NaN (binary64: the odd word's top bit, from both words).  Adding the
// distance from the largest non-NaN magnitude to the lane's top bit carries
// into it for NaN magnitudes only.
template <uint32_t DT> __device__ __forceinline__ uint32_t nan_tops(const uint32_t (&g)[4], int i) {
  const uint32_t x = g[i];
  if (DT == KC_F32) return ((x & 0x7FFFFFFFu) + 0x007FFFFFu) & 0x80000000u;              // above 0x7F800000
  if (DT == KC_BF16) return ((x & 0x7FFF7FFFu) + 0x007F007Fu) & 0x80008000u;             // above 0x7F80
  if (DT == KC_F16) return ((x & 0x7FFF7FFFu) + 0x03FF03FFu) & 0x80008000u;              // above 0x7C00
  if (DT == KC_FP8_E4M3FN) return ((x & 0x7F7F7F7Fu) + 0x01010101u) & 0x80808080u;       // magnitude 0x7F
  if (DT == KC_FP8_E5M2) return ((x & 0x7F7F7F7Fu) + 0x03030303u) & 0x80808080u;         // above 0x7C
  if (DT == KC_FP8_E4M3FNUZ || DT == KC_FP8_E5M2FNUZ) return nonzero_tops<1>(x ^ 0x80808080u) ^ 0x80808080u;  // 0x80
  if (DT == KC_F64 && (i & 1))  // above 0x7FF00000'00000000: a non-zero low word counts as bit 0 of the high one
    return (((x & 0x7FFFFFFFu) | (g[i - 1] != 0u ? 1u : 0u)) + 0x000FFFFFu) & 0x80000000u;
  return 0u;
}

constexpr uint32_t kHistCopies = 32;
// After the ULP bins, one for each NaN class: in both sides, in the candidate only, in the golden only.
constexpr uint32_t kNanBins = kBins, kAllBins = kBins + 3u;

// What a workgroup shares of the pair it is on.  The maxima and the first
// mismatch live here rather than in registers: a lane compares with its own
// copy of them, taken once per round, and writes only what exceeds it.
struct TileLds {
  uint32_t hist[kAllBins * kHistCopies];  // bin b, copy c at b * kHistCopies + c; lane l counts into copy l mod 32
  unsigned long long max_abs, max_rel;  // bits of non-negative doubles
  unsigned long long first;             // lowest differing element
  uint32_t any[2];                      // some thread saw an element that differs or is NaN; pairs take turns
  uint32_t cnt[4];                      // kCntMis .. kCntNotClose below
  uint32_t bins[kAllBins];              // the histogram's totals, once a pair is done
};
enum : uint32_t { kCntMis = 0, kCntBytes, kCntOver, kCntNotClose };

struct Partial {
  uint32_t mis_elems, mis_bytes, over, not_close;  // of this thread
  bool any;                                        // this thread saw an element that differs or is NaN
  double max_abs, max_rel, half_ulp;               // of this thread and, as of the round's start, of all; half_ulp:
                                                   // half the distance from max_rel to the next double
};

struct Tol {
  uint32_t ulp;
  double atol, rtol;
};

__device__ __forceinline__ uint64_t dbl_bits(double x) { return (uint64_t)__double_as_longlong(x); }
__device__ __forceinline__ double bits_dbl(uint64_t x) { return __longlong_as_double((long long)x); }
// The larger of a non-negative double and one given by its bits.
__device__ __forceinline__ double fmax_pos(double x, unsigned long long bits) {
  const double y = __longlong_as_double((long long)bits);
  return y > x ? y : x;
}

// Half the gap above a non-negative finite double, or less (zero for tiny ones).
__device__ __forceinline__ double half_gap(double x) {
  const uint32_t e = (uint32_t)(dbl_bits(x) >> 52);
  return e > 53u ? __longlong_as_double((long long)((uint64_t)(e - 53u) << 52)) : 0.0;
}

// Whether the rounded quotient a / g may exceed m (a >= 0, g > 0; half is
// half_gap(m)).  a - m g is formed with one rounding, so it is at least half g
// whenever the exact a / g is at least m + half; below that the quotient rounds
// to m or less.  Ties with the running maximum, common in narrow formats, are
// so settled by one fused multiply-add instead of a division.  An infinite g
// gives false (the sum is -inf or a NaN): it has no relative error.
__device__ __forceinline__ bool rel_may_grow(double a, double g, double m, double half) {
  return __builtin_fma(-m, g, a) >= half * g;
}

template <typename D> __device__ __forceinline__ uint32_t ulp_bin(D d) {
  if (d <= 16u) return (uint32_t)d;
  const uint32_t top = sizeof(D) == 8 ? 64u - (uint32_t)__clzll((uint64_t)d - 1ull) : 32u - (uint32_t)__clz((uint32_t)d - 1u);
  return min(12u + top, kBins - 1u);  // 12 + ceil(log2 d)
}

// Bytes of x (not zero) that are not zero.
template <typename B, uint32_t SIZE> __device__ __forceinline__ uint32_t byte_count(B x) {
  if (SIZE == 1) return 1u;
  uint32_t n = (uint32_t)__popc(nonzero_tops<1>((uint32_t)x));
  if (SIZE == 8) n += (uint32_t)__popc(nonzero_tops<1>((uint32_t)((uint64_t)x >> 32)));
  return n;
}

__device__ __forceinline__ void count_nans(TileLds& lds, uint32_t which, uint32_t n) {
  if (n != 0u) atomicAdd(&lds.hist[(kNanBins + which) * kHistCopies + threadIdx.x % kHistCopies], n);
}

// One element that is a NaN on some side; true if the two differ.
template <uint32_t DT>
__device__ __forceinline__ bool nan_element(typename Fmt<DT>::B c, typename Fmt<DT>::B g, Partial& p, TileLds& lds) {
  const bool nc = Fmt<DT>::nan(c), ng = Fmt<DT>::nan(g);
  count_nans(lds, nc && ng ? 0u : nc ? 1u : 2u, 1u);
  if (c == g) return false;
  ++p.mis_elems;
  p.mis_bytes += byte_count<typename Fmt<DT>::B, Fmt<DT>::size>(c ^ g);
  return true;
}

// Exact path of one element that differs, neither side a NaN.  Straight-line
// but for new maxima of the relative error.
template <uint32_t DT>
__device__ __forceinline__ void element(typename Fmt<DT>::B c, typename Fmt<DT>::B g, const Tol& tol, Partial& p,
                                        TileLds& lds) {
  using F = Fmt<DT>;
  using B = typename F::B;
  using D = B;  // distances of elements up to 32 bits fit in 32 bits
  ++p.mis_elems;
  p.mis_bytes += byte_count<B, F::size>(c ^ g);
  if constexpr (F::kind != 2) {
    D d;
    if constexpr (F::kind == 1) {
      const int64_t ci = F::sext(c), gi = F::sext(g);
      d = (D)(ci >= gi ? (uint64_t)ci - (uint64_t)gi : (uint64_t)gi - (uint64_t)ci);  // exact below 2^64
    } else {
      constexpr B sb = (B)1 << (8u * F::size - 1u);
      const D mc = (D)(c & F::mag), mg = (D)(g & F::mag);
      const D same = max(mc, mg) - min(mc, mg), across = mc + mg;  // across zero: the two magnitudes
      d = ((c ^ g) & sb) == 0 ? same : across;
    }
    p.over += d > tol.ulp ? 1u : 0u;
    // distance 0 (+0 and -0) lands in bin 0, which the report does not read
    atomicAdd(&lds.hist[ulp_bin<D>(d) * kHistCopies + threadIdx.x % kHistCopies], 1u);
    const double vc = F::value(c), vg = F::value(g), ag = __builtin_fabs(vg);
    const double a = F::kind == 1 ? (double)d : __builtin_fabs(vc - vg);
    p.max_abs = a > p.max_abs ? a : p.max_abs;
    if (vg != 0.0 && rel_may_grow(a, ag, p.max_rel, p.half_ulp)) {
      const double r = a / ag;
      if (r > p.max_rel) {
        p.max_rel = r;
        p.half_ulp = half_gap(r);
      }
    }
    // tolerance test: an infinity is close only to an equal value, and these two differ
    const double bound = tol.atol + tol.rtol * ag;
    p.not_close += (a > bound || F::inf(c) || F::inf(g)) ? 1u : 0u;
  }
}

// Ends a round: the maxima that grew in it (from max_abs and max_rel) and the
// lowest differing element (from round0; ~0: none) go to the shared ones: from
// each lane that has some if they are few, else once per wave.  All lanes take
// part.  (With an atomic per lane whatever their number, the first rounds' lanes
// queued on these addresses: 1076 pairs of 920 bytes, 60 % off, 46 us, so 22; 214
// pairs of 260 KB, 11.3 % off, 61 -> 45.  With a reduction whatever their number,
// 16 pairs of 64 KiB, 0.1 % off, took 10.0 us a call, so 8.7.)
constexpr int kFewLanes = 8;
__device__ __forceinline__ void share_found(Partial& p, double max_abs, double max_rel, uint64_t round0, uint32_t low,
                                            TileLds& lds) {
  const bool grew = p.max_abs > max_abs || p.max_rel > max_rel;
  unsigned long long a = dbl_bits(p.max_abs), r = dbl_bits(p.max_rel);  // not negative: ordered as their bits
  const uint64_t growing = __ballot(grew);
  bool tell = grew;
  if (__popcll(growing) > kFewLanes) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
      a = max(a, __shfl_xor(a, d, 64));
      r = max(r, __shfl_xor(r, d, 64));
    }
    tell = threadIdx.x % kWave == 0u;
  }
  if (tell) {
    atomicMax(&lds.max_abs, a);
    atomicMax(&lds.max_rel, r);
  }
  if (__ballot(round0 < lds.first) == 0ull) return;  // not one of the first rounds that differ
  tell = low != ~0u;
  if (__popcll(__ballot(tell)) > kFewLanes) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) low = min(low, (uint32_t)__shfl_xor(low, d, 64));
    tell = threadIdx.x % kWave == 0u;
  }
  if (tell) atomicMin(&lds.first, (unsigned long long)(round0 + low));
}

// One element of `es` bytes at a naturally aligned address, zero-extended.
template <typename B, uint32_t ES>
__device__ __forceinline__ B load_elem(const uint8_t* base, uint64_t e) {
  const uint64_t a = (uint64_t)base + e * ES;
  if (ES == 1) return (B)*(const KC_GLOBAL uint8_t*)a;
  if (ES == 2) return (B)*(const KC_GLOBAL uint16_t*)a;
  if (ES == 4) return (B)*(const KC_GLOBAL uint32_t*)a;
  return (B)*(const KC_GLOBAL uint64_t*)a;
}

// 16 bytes at an address aligned to the element only (a view at an odd element
// offset): still one 16-byte load, which gfx950 serves at any byte address.
template <uint32_t ES> struct Run16;
template <> struct Run16<1> { typedef unsigned int T __attribute__((ext_vector_type(4), aligned(1))); };
template <> struct Run16<2> { typedef unsigned int T __attribute__((ext_vector_type(4), aligned(2))); };
template <> struct Run16<4> { typedef unsigned int T __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct Run16<8> { typedef unsigned int T __attribute__((ext_vector_type(4), aligned(8))); };
template <uint32_t ES> __device__ __forceinline__ uint4 ld_run(uint64_t addr) {
  using T = typename Run16<ES>::T;
  const T v = __builtin_nontemporal_load((const KC_GLOBAL T*)addr);
  return make_uint4(v[0], v[1], v[2], v[3]);
}

// Bits for the marked elements of a round: 64 of 8 bits, at most 32 of others.
template <uint32_t ES> struct Mask { typedef uint32_t T; };
template <> struct Mask<1> { typedef uint64_t T; };

// Marks elements of word j = 4 u + i of a lane's runs from their top bits: 8-bit
// elements: byte k of word j is bit 8k + 7 - (j & 7) of half j >> 3; 16-bit:
// half-word k of word j is bit 16k + 15 - j; 32-bit: bit j; 64-bit: element e
// (its odd word's top bit) is bit e.
template <uint32_t ES> __device__ __forceinline__ void add_marks(uint32_t (&m)[2], uint32_t j, uint32_t tops) {
  if (ES == 8) m[0] |= tops >> (31u - (j >> 1));
  else if (ES == 4) m[0] |= tops >> (31u - j);
  else if (ES == 2) m[0] |= tops >> j;
  else m[j >> 3] |= tops >> (j & 7u);
}

// Marks of one lane that may be NaNs from which its wave counts a round's NaNs
// together (round_nans); with fewer each lane takes its own one by one.  Together
// costs the same however many there are, about 14 of them one by one.  256 MiB with
// 11.3 % off, one by one / together: as bf16 with 0.1, 1 and 10 % NaNs 118 / 158, 123 /
// 163 and 145 / 160 us, as fp8 with 0.1 and 3 % 157 / 198 and 180 / 196; half of each
// 256 bytes NaN, as fp8, 310 / 102.  Binary64 has 8 elements a lane: always one by one.
constexpr uint32_t kManyNans = 12;

// From marks of the first words of runs: of all their words.
template <uint32_t ES> __device__ __forceinline__ uint32_t any_word(uint32_t m) {
  return ES == 8 ? m * 3u : ES == 4 ? m * 15u : (m >> 3) * 15u;
}

// The NaNs of a round, from its staged runs (bit u of `runs`: run u is staged;
// v: this lane's first run, of nvec): counted by class, and where the two sides
// differ the element, its bytes and the lowest of them; taken out of the marks m.
// (Taken through the exact path one by one, 256 MiB of NaN in both sides took
// 0.27 ms as f32 and 1.03 ms as fp8; so 0.13 for either.)
template <uint32_t DT, uint32_t T>
__device__ __forceinline__ void round_nans(const uint4* cs, const uint4* gs, uint32_t runs, uint32_t v, uint32_t nvec,
                                           uint32_t (&m)[2], uint32_t& low, Partial& p, TileLds& lds) {
  constexpr uint32_t es = Fmt<DT>::size;
  static_assert(es < 8u, "one word holds whole elements");
  uint32_t both = 0u, cand = 0u, gold = 0u, nans[2] = {0u, 0u};
#pragma unroll
  for (uint32_t u = 0; u < kUnroll; ++u) {
    if (((runs >> u) & 1u) == 0u) continue;
    const uint4 c = cs[u * T], g = gs[u * T];
    const uint32_t cw[4] = {c.x, c.y, c.z, c.w}, gw[4] = {g.x, g.y, g.z, g.w};
    const uint32_t in = v + u * T < nvec ? ~0u : 0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t nc = nan_tops<DT>(cw, i) & in, ng = nan_tops<DT>(gw, i) & in, n = nc | ng;
      both += (uint32_t)__popc(nc & ng);
      cand += (uint32_t)__popc(nc & ~ng);
      gold += (uint32_t)__popc(~nc & ng);
      add_marks<es>(nans, 4u * u + (uint32_t)i, n);
      // all bits of their lanes
      const uint32_t lanes = es == 1u ? (n >> 7) * 0xFFu : es == 2u ? (n >> 15) * 0xFFFFu : 0u - (n >> 31);
      const uint32_t x = (cw[i] ^ gw[i]) & lanes, d = nonzero_tops<es>(x);
      p.mis_elems += (uint32_t)__popc(d);
      p.mis_bytes += (uint32_t)(es == 1u ? __popc(d) : __popc(nonzero_tops<1>(x)));
      if (d != 0u)
        low = min(low, (u * T + threadIdx.x) * (16u / es) + ((uint32_t)i * 4u + ((uint32_t)__builtin_ctz(d) >> 3)) / es);
    }
  }
  m[0] &= ~nans[0];
  m[1] &= ~nans[1];
  count_nans(lds, 0u, both);
  count_nans(lds, 1u, cand);
  count_nans(lds, 2u, gold);
}

// The bytes [b0, b1) of a pair.  stage: kUnroll runs of each side per thread.
template <uint32_t DT, uint32_t T>
__device__ __forceinline__ void tile_body(const CmpPairDev& pr, uint64_t b0, uint64_t b1, Partial& p, TileLds& lds,
                                          uint4* stage) {
  using F = Fmt<DT>;
  using B = typename F::B;
  constexpr uint32_t es = F::size;
  constexpr uint32_t epv = 16u / es;  // elements per run
  const uint32_t tid = threadIdx.x;
  const uint32_t n_el = (uint32_t)((b1 - b0) / es), per_round = T * kUnroll;
  // whole runs; none when every element can have a thread of its own, which spares one wave a chain of exact paths
  // (230 pairs of 870 bytes with 60 % off: 15 us, 27 with runs)
  const uint32_t nvec = n_el <= T ? 0u : (uint32_t)((b1 - b0) / 16u);
  const Tol tol{pr.tol, pr.atol, pr.rtol};
  const uint64_t ca = (uint64_t)pr.cand + b0, ga = (uint64_t)pr.gold + b0, e0 = b0 / es;
  uint4* const cs = stage + tid;                 // run u of this thread at cs[u * T]
  uint4* const gs = stage + per_round + tid;
  uint4 c[kUnroll], g[kUnroll];
  auto load = [&](uint32_t u, uint32_t v0) {  // runs past the end are read as the last one and not looked at
    const uint32_t o = min(v0 + u * T + tid, nvec - 1u) * 16u;
    c[u] = ld_run<es>(ca + o);
    g[u] = ld_run<es>(ga + o);
  };
  if (nvec != 0u) {
#pragma unroll
    for (uint32_t u = 0; u < kUnroll; ++u) load(u, 0u);
  }
  for (uint32_t v0 = 0; v0 < nvec; v0 += per_round) {
    // Marked elements: those that differ or are NaN (add_marks).
    uint32_t m[2] = {0u, 0u};
    uint32_t runs = 0u;          // of the wave: runs that hold one, as bits
    uint32_t nan[2] = {0u, 0u};  // NaNs in any word of a run, marked as if in its first
#pragma unroll
    for (uint32_t u = 0; u < kUnroll; ++u) {
      const uint32_t cw[4] = {c[u].x, c[u].y, c[u].z, c[u].w}, gw[4] = {g[u].x, g[u].y, g[u].z, g[u].w};
      uint32_t any = 0u;
#pragma unroll
      for (int i = 0; i < 4; ++i) any |= (cw[i] ^ gw[i]) | nan_tops<DT>(gw, i);
      if (__ballot(any != 0u) != 0ull) {  // some lane's run holds one
        runs |= 1u << u;
        const uint32_t in = v0 + u * T + tid < nvec ? ~0u : 0u;
        uint32_t run_nan = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (es == 8u && !(i & 1)) continue;  // with the odd word
          const uint32_t x = es == 8u ? (cw[i] ^ gw[i]) | (cw[i & 2] ^ gw[i & 2]) : cw[i] ^ gw[i];
          const uint32_t ng = nan_tops<DT>(gw, i);
          add_marks<es>(m, 4u * u + (uint32_t)i, (nonzero_tops<es>(x) | ng) & in);
          run_nan |= nan_tops<DT>(cw, i) | ng;
        }
        add_marks<es>(nan, 4u * u, run_nan);
        cs[u * T] = c[u];
        gs[u * T] = g[u];
      }
      load(u, v0 + per_round);  // the next round's, run by run (after the last round: its last run again)
    }
    asm volatile("" ::: "memory");  // the runs are read back as elements of another type
    if (runs == 0u) continue;
    p.any = p.any || (m[0] | m[1]) != 0u;
    uint32_t low = ~0u;  // lowest differing element of this lane, from the round's first
    if constexpr (F::kind == 0) {  // nan: the marks that may be NaNs
      nan[0] = any_word<es>(nan[0]) & m[0];
      nan[1] = es == 1u ? any_word<es>(nan[1]) & m[1] : 0u;
      if constexpr (epv * kUnroll >= kManyNans) {
        if (__ballot((uint32_t)(__popc(nan[0]) + __popc(nan[1])) >= kManyNans) != 0ull) {
          round_nans<DT, T>(cs, gs, runs, v0 + tid, nvec, m, low, p, lds);
          nan[0] = nan[1] = 0u;
        }
      }
    }
    using M = typename Mask<es>::T;
    M mask = es == 1 ? (M)(((uint64_t)m[1] << 32) | m[0]) : (M)m[0];
    p.max_abs = fmax_pos(p.max_abs, lds.max_abs);
    p.max_rel = fmax_pos(p.max_rel, lds.max_rel);
    p.half_ulp = half_gap(p.max_rel);
    const uint64_t round0 = e0 + (uint64_t)v0 * epv;
    // the place (byte offset in cs and gs, element from round0) of the lowest marked bit
    auto place = [&](M m, uint32_t& at) -> uint32_t {
      const uint32_t b = sizeof(M) == 8 ? (uint32_t)__builtin_ctzll(m) : (uint32_t)__builtin_ctz((uint32_t)m);
      uint32_t j, k;  // word and lane inside it
      if (es == 1) {
        j = ((b >> 5) << 3) + (7u - (b & 7u));
        k = (b >> 3) & 3u;
      } else if (es == 2) {
        j = 15u - (b & 15u);
        k = b >> 4;
      } else {
        j = es == 8 ? 2u * b : b;
        k = 0u;
      }
      const uint32_t byte = (j & 3u) * 4u + k * es;
      at = ((j >> 2) * T + tid) * epv + byte / es;
      return (j >> 2) * (T * 16u) + byte;
    };
    auto get = [&](const uint4* side, uint32_t o) -> B {
      const uint8_t* const x = reinterpret_cast<const uint8_t*>(side) + o;
      if (es == 1) return (B)*x;
      if (es == 2) return (B)*reinterpret_cast<const uint16_t*>(x);
      return *reinterpret_cast<const B*>(x);
    };
    const double max_abs = p.max_abs, max_rel = p.max_rel;
    if constexpr (F::kind == 2) {  // raw bytes: the marks are all there is to know (256 MiB all off: 203 us one by one, so 117)
      const uint32_t n = (uint32_t)(__popc(m[0]) + __popc(m[1]));
      p.mis_elems += n;
      p.mis_bytes += n;
      if (n != 0u) {
        const uint32_t half = m[0] == 0u ? 1u : 0u, x = half ? m[1] : m[0], word = x | (x >> 16);
        const uint32_t top = 31u - (uint32_t)__clz((word | (word >> 8)) & 0xFFu);  // the half's lowest word: highest bit
        const uint32_t j = half * 8u + 7u - top, k = (uint32_t)__builtin_ctz((x >> top) & 0x01010101u) >> 3;
        low = ((j >> 2) * T + tid) * epv + (j & 3u) * 4u + k;
      }
    } else {
      if (F::kind == 0) {  // few NaNs: one by one, taken out of the marks
        for (M left = es == 1 ? (M)(((uint64_t)nan[1] << 32) | nan[0]) : (M)nan[0]; left != 0; left &= left - 1) {
          uint32_t at;
          const uint32_t o = place(left, at);
          const B cv = get(cs, o), gv = get(gs, o);
          if (!F::nan(cv) && !F::nan(gv)) continue;
          if (nan_element<DT>(cv, gv, p, lds)) low = min(low, at);
          mask &= ~(left & (~left + 1));
        }
      }
      for (; mask != 0; mask &= mask - 1) {
        uint32_t at;
        const uint32_t o = place(mask, at);
        low = min(low, at);
        element<DT>(get(cs, o), get(gs, o), tol, p, lds);
      }
    }
    share_found(p, max_abs, max_rel, round0, low, lds);
    asm volatile("" ::: "memory");
  }
  // elements past the last whole run (fewer than a run's, or all), one per thread
  if (nvec * epv == n_el) return;
  const double max_abs = p.max_abs, max_rel = p.max_rel;
  const uint32_t at = nvec * epv + tid;
  uint32_t low = ~0u;
  if (at < n_el) {
    const B cv = load_elem<B, es>((const uint8_t*)ca, at), gv = load_elem<B, es>((const uint8_t*)ga, at);
    const bool nc = F::nan(cv), ng = F::nan(gv);
    p.any = p.any || cv != gv || ng;
    if (cv != gv) low = at;
    if (nc || ng) {
      count_nans(lds, nc && ng ? 0u : nc ? 1u : 2u, 1u);
      p.mis_elems += cv != gv ? 1u : 0u;
      p.mis_bytes += cv != gv ? byte_count<B, es>(cv ^ gv) : 0u;
    } else if (cv != gv) {
      element<DT>(cv, gv, tol, p, lds);
    }
  }
  share_found(p, max_abs, max_rel, e0, low, lds);
}


// A value for what is done where a pair ends, as the thread's index: lanes,
// addresses and constants made from it there are not kept from the kernel's start
// on, in registers that the rounds need (seven to thirteen of them were spilled).
template <typename V> __device__ __forceinline__ V made_here(V x) {
  asm volatile("" : "+v"(x));
  return x;
}

__device__ __forceinline__ void clear_tile_lds(TileLds& lds) {
  const uint32_t tid = made_here(threadIdx.x);
  for (uint32_t i = tid; i < kAllBins * kHistCopies; i += blockDim.x) lds.hist[i] = 0u;
  if (tid < 4u) lds.cnt[tid] = 0u;
  if (tid < 2u) lds.any[tid] = 0u;
  if (tid == 0u) {
    const unsigned long long none = made_here(0ull);
    lds.max_abs = lds.max_rel = none;
    lds.first = ~none;
  }
}

// The bytes [b0, b1) of a pair, added to what the workgroup has found of it.
// No barrier: its waves share only counters.
template <uint32_t T>
__device__ __forceinline__ void compare_bytes(const CmpPairDev& pr, uint64_t b0, uint64_t b1, Partial& p, TileLds& lds,
                                              uint4* stage) {
  switch (pr.dtype) {
    case KC_F32: tile_body<KC_F32, T>(pr, b0, b1, p, lds, stage); break;
    case KC_BF16: tile_body<KC_BF16, T>(pr, b0, b1, p, lds, stage); break;
    case KC_F16: tile_body<KC_F16, T>(pr, b0, b1, p, lds, stage); break;
    case KC_FP8_E4M3FN: tile_body<KC_FP8_E4M3FN, T>(pr, b0, b1, p, lds, stage); break;
    case KC_F64: tile_body<KC_F64, T>(pr, b0, b1, p, lds, stage); break;
    case KC_FP8_E4M3FNUZ: tile_body<KC_FP8_E4M3FNUZ, T>(pr, b0, b1, p, lds, stage); break;
    case KC_FP8_E5M2: tile_body<KC_FP8_E5M2, T>(pr, b0, b1, p, lds, stage); break;
    case KC_FP8_E5M2FNUZ: tile_body<KC_FP8_E5M2FNUZ, T>(pr, b0, b1, p, lds, stage); break;
    case KC_I8: tile_body<KC_I8, T>(pr, b0, b1, p, lds, stage); break;
    case KC_I16: tile_body<KC_I16, T>(pr, b0, b1, p, lds, stage); break;
    case KC_I32: tile_body<KC_I32, T>(pr, b0, b1, p, lds, stage); break;
    case KC_I64: tile_body<KC_I64, T>(pr, b0, b1, p, lds, stage); break;
    default: tile_body<KC_U8, T>(pr, b0, b1, p, lds, stage); break;
  }
}

// Word w of a report (61 of 8 bytes, one per lane) comes from this word of the
// pair's accumulators; -1: from none of them.
__device__ __forceinline__ int acc_of_word(uint32_t w) {
  if (w >= 10u && w < 10u + kBins) return (int)(w - 10u + kAccHist);
  switch (w) {
    case 1: return kAccMisElems;
    case 2: return kAccMisBytes;
    case 3: return kAccFirstInv;
    case 4: return kAccNanBoth;
    case 5: return kAccNanCand;
    case 6: return kAccNanGold;
    case 7: return kAccOverTol;
    case 8: return kAccMaxAbs;
    case 9: return kAccMaxRel;
    case 59: return kAccNotClose;
    default: return -1;
  }
}
static_assert(sizeof(kc_cmp_result) == 61 * 8, "report layout");

// One wave writes a pair's report; x: the accumulator word acc_of_word(lane).
__device__ __forceinline__ void write_report(uint64_t n_elems, uint32_t dtype, uint64_t x, kc_cmp_result* r) {
  const uint32_t lane = made_here(threadIdx.x) % kWave;
  const uint64_t rest = wave_sum_u64(lane > 10u && lane < 10u + kBins ? x : 0ull);  // counted at a distance above 0
  const uint64_t mis = __shfl(x, 1, 64), nb = __shfl(x, 4, 64), nc = __shfl(x, 5, 64), ng = __shfl(x, 6, 64);
  const uint64_t over = __shfl(x, 7, 64), not_close = __shfl(x, 59, 64);
  const bool raw = dtype == KC_U8, no_nan = (nc | ng) == 0ull;
  if (lane == 0u) x = n_elems;
  if (lane == 3u) x = ~x;  // the accumulator holds the complement
  if (lane == 10u) x = raw ? 0ull : n_elems - nb - nc - ng - rest;
  if (lane == 58u) x = (raw ? mis == 0ull : over == 0ull && no_nan) ? 1u : 0u;  // pass, and status 0 above it
  if (lane == 60u) x = (raw ? mis == 0ull : not_close == 0ull && no_nan) ? 1u : 0u;
  if (lane < 61u) reinterpret_cast<uint64_t*>(r)[lane] = x;
}

// The accumulator words of a pair as the workgroup found them (totals summed).
__device__ __forceinline__ uint64_t found_word(const TileLds& lds, int i) {
  if (i < 0) return 0ull;
  if (i >= (int)kAccHist) return lds.bins[i - (int)kAccHist];
  if (i == kAccMaxAbs) return lds.max_abs;
  if (i == kAccMaxRel) return lds.max_rel;
  if (i == kAccFirstInv) return ~lds.first;
  if (i >= (int)kAccNanBoth && i <= (int)kAccNanGold) return lds.bins[kNanBins + (uint32_t)i - kAccNanBoth];
  return lds.cnt[i == kAccMisElems ? kCntMis : i == kAccMisBytes ? kCntBytes : i == kAccOverTol ? kCntOver : kCntNotClose];
}

// Ends a workgroup's work on a pair; leaves lds clear.  DIRECT: it was the
// whole pair, and the workgroup writes the report.  Else what it found goes to
// the pair's accumulators (nothing if every element was equal): once per run of
// tiles of one pair, not per tile, since the atomics of all workgroups on one
// pair meet at the same addresses and cost about 0.1 us each there (a 250 MiB
// pair with one element in 10,000 off, flushed per 64 KiB tile: 0.70 ms for a
// 0.31 ms pass).
template <bool DIRECT>
__device__ __forceinline__ void end_pair(const CmpPairDev& pr, const Partial& p, unsigned long long* acc,
                                         kc_cmp_result* res, TileLds& lds, uint32_t& turn) {
  const uint32_t tid = made_here(threadIdx.x), lane = tid & 63u;
  // A wave past this barrier may reach the next pair's before another has read this flag: hence the turns.
  uint32_t& any = lds.any[turn & 1u];
  ++turn;
  if (__ballot(p.any) != 0ull && lane == 0) any = 1u;
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(any) == 0u) {  // nothing but equal elements, none NaN
    if (DIRECT && tid < kWave) write_report(pr.n_elems, pr.dtype, 0ull, res);
    return;
  }
  const uint32_t v0 = wave_sum_u32(p.mis_elems), v1 = wave_sum_u32(p.mis_bytes);
  const uint32_t v2 = wave_sum_u32(p.over), v3 = wave_sum_u32(p.not_close);
  if (lane == 0) {
    atomicAdd(&lds.cnt[kCntMis], v0);
    atomicAdd(&lds.cnt[kCntBytes], v1);
    atomicAdd(&lds.cnt[kCntOver], v2);
    atomicAdd(&lds.cnt[kCntNotClose], v3);
  }
  // four threads per bin sum its copies (eight words each)
  for (uint32_t i = tid; i < kAllBins * 4u; i += blockDim.x) {
    const uint4* h = reinterpret_cast<const uint4*>(lds.hist + i * 8u);
    const uint4 x = h[0], y = h[1];
    uint32_t n = x.x + x.y + x.z + x.w + y.x + y.y + y.z + y.w;
    n += __shfl_xor(n, 1, 64);
    n += __shfl_xor(n, 2, 64);
    if ((i & 3u) == 0u) lds.bins[i / 4u] = n;
  }
  __syncthreads();
  if (DIRECT) {
    if (tid < kWave) write_report(pr.n_elems, pr.dtype, found_word(lds, acc_of_word(lane)), res);
  } else if (tid < kAccHist + kBins) {  // thread i flushes accumulator word i
    const unsigned long long x = tid <= kAccNotClose || tid >= kAccHist ? found_word(lds, (int)tid) : 0ull;
    if (x != 0ull) {
      if (tid >= kAccMaxAbs && tid <= kAccFirstInv) atomicMax(&acc[tid], x);
      else atomicAdd(&acc[tid], x);
    }
  }
  __syncthreads();
  clear_tile_lds(lds);
  __syncthreads();
}
// n consecutive tiles of a pair from tile `idx`, as one run of bytes (so that
// the loads of one tile's first round are in flight while the last one's is
// worked on), in pieces whose offsets fit 32 bits.
constexpr uint64_t kMaxRun = 1ull << 30;
template <uint32_t T, bool DIRECT>
__device__ __forceinline__ void compare_tiles(const CmpPairDev& pr, uint64_t idx, uint64_t n, uint32_t tile_bytes,
                                              unsigned long long* acc, kc_cmp_result* res, TileLds& lds,
                                              uint4* stage, uint32_t& turn) {
  // The pair's maxima so far are thresholds below which nothing needs to be recorded (they only grow).
  Partial p{0, 0, 0, 0, false, 0.0, 0.0, 0.0};
  if (!DIRECT) {
    p.max_abs = bits_dbl(acc[kAccMaxAbs]);
    p.max_rel = bits_dbl(acc[kAccMaxRel]);
  }
  const uint64_t end = min((idx + n) * tile_bytes, pr.n_elems * pr.esize);
  for (uint64_t b0 = idx * tile_bytes; b0 < end; b0 += kMaxRun)
    compare_bytes<T>(pr, b0, min(b0 + kMaxRun, end), p, lds, stage);
  end_pair<DIRECT>(pr, p, acc, res, lds, turn);
}

// The tiles [t, end) of this workgroup of a launch over n: consecutive ones, so
// that a workgroup meets few pairs and reads on where it was.
__device__ __forceinline__ void my_tiles(const CmpWalk& w, uint32_t n, uint32_t& t, uint32_t& end) {
  const uint32_t b = blockIdx.x;
  if (w.run == 0u) {
    const uint32_t each = n / w.grid, more = n % w.grid;
    t = b * each + min(b, more);
    end = t + each + (b < more ? 1u : 0u);
  } else if (b < w.whole) {
    t = b * w.run;
    end = min(t + w.run, n);
  } else {  // kTaperRuns runs of each half of the last length, then single tiles
    const uint32_t i = b - w.whole, k = i >> kTaperShift, phases = 31u - (uint32_t)__clz(w.run);
    const bool single = k >= phases;
    const uint32_t len = single ? 1u : w.run >> (k + 1u);
    const uint32_t before = single ? phases : k;  // phases before this one
    t = w.whole * w.run + ((w.run - (w.run >> before)) << kTaperShift) + (i - (before << kTaperShift)) * len;
    end = min(t + len, n);
  }
}

// The accumulators of a pair that this workgroup adds to.
__device__ __forceinline__ unsigned long long* my_acc(unsigned long long* acc_all, uint32_t pair, const CmpWalk& w) {
  return acc_all + ((uint64_t)pair * w.copies + (blockIdx.x & (w.copies - 1u))) * kAccWords;
}

static_assert((kAccCopies & (kAccCopies - 1u)) == 0u, "a power of two");
static_assert(kAccNanCand == kAccNanBoth + 1 && kAccNanGold == kAccNanBoth + 2, "order of the NaN classes");

// T threads per workgroup: kThreads, or kWideThreads when the tiles are no more
// than the CUs (a tile of 64 KiB is then one round).  DIRECT: every pair of the
// launch is one tile.  (Decided per launch: with the choice made per pair, the
// pass over 10,000 pairs of one to a thousand tiles took 2.59 ms, not 2.53.)
template <uint32_t T, bool DIRECT>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(4))) void k_compare(
    const CmpPairDev* pairs, const CmpTileDev* tiles, uint32_t n_tiles, uint32_t tile_bytes,
    unsigned long long* acc_all, kc_cmp_result* res, CmpWalk walk) {
  __shared__ uint4 stage[2 * kUnroll * T];
  __shared__ __attribute__((aligned(16))) TileLds lds;
  clear_tile_lds(lds);
  __syncthreads();
  uint32_t turn = 0;
  uint32_t t, end;
  my_tiles(walk, n_tiles, t, end);
  while (t < end) {
    const CmpTileDev tl = const_load(tiles + t);
    const CmpPairDev pr = const_load(pairs + tl.pair);
    const uint32_t n = min(end - t, pr.n_tiles - tl.idx);
    compare_tiles<T, DIRECT>(pr, tl.idx, n, tile_bytes, my_acc(acc_all, tl.pair, walk), res + tl.pair, lds, stage, turn);
    t += n;
  }
}

// The same pass over the pairs carried in the kernel arguments: tile t
// belongs to the first pair whose inclusive tile prefix exceeds t.
template <uint32_t T, bool DIRECT>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(4))) void k_compare_args(
    CmpArgPairs a, uint32_t tile_bytes, unsigned long long* acc_all, kc_cmp_result* res, CmpWalk walk) {
  __shared__ uint4 stage[2 * kUnroll * T];
  __shared__ __attribute__((aligned(16))) TileLds lds;
  clear_tile_lds(lds);
  __syncthreads();
  uint32_t turn = 0;
  uint32_t t, end;
  my_tiles(walk, a.n_tiles, t, end);
  while (t < end) {
    uint32_t lo = 0, hi = a.n - 1u;
    while (lo < hi) {
      const uint32_t mid = (lo + hi) >> 1;
      if (a.tile_end[mid] > t) hi = mid; else lo = mid + 1u;
    }
    const uint32_t start = lo == 0u ? 0u : a.tile_end[lo - 1u], n = min(end, a.tile_end[lo]) - t;
    compare_tiles<T, DIRECT>(a.pair[lo], t - start, n, tile_bytes, my_acc(acc_all, lo, walk), res + lo, lds, stage, turn);
    t += n;
  }
}

// One wave per pair turns its accumulators (all copies of them) into the report
// and zeroes them for the next call.
__device__ __forceinline__ void finalize_pair(uint64_t n_elems, uint32_t dtype, unsigned long long* acc_all,
                                              uint64_t pair, uint32_t copies, kc_cmp_result* r) {
  const uint32_t lane = threadIdx.x % kWave;
  const int i = acc_of_word(lane);
  unsigned long long* const acc = acc_all + pair * copies * kAccWords;
  uint64_t x = 0ull;
  for (uint32_t c = 0; c < copies; ++c) {
    const uint64_t y = i >= 0 ? acc[c * kAccWords + (uint32_t)i] : 0ull;
    x = i >= (int)kAccMaxAbs && i <= (int)kAccFirstInv ? max(x, y) : x + y;
  }
  write_report(n_elems, dtype, x, r);
  asm volatile("" ::: "memory");  // the lanes clear words that other lanes have read above
  for (uint32_t c = 0; c < copies; ++c) acc[c * kAccWords + lane] = 0ull;
}
static_assert(kAccWords == kWave, "one accumulator word per lane");

__global__ __launch_bounds__(256) void k_compare_finalize(const CmpPairDev* pairs, uint32_t n_pairs,
                                                          unsigned long long* acc_all, uint32_t copies,
                                                          kc_cmp_result* res) {
  const uint32_t i = __builtin_amdgcn_readfirstlane(blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave);
  if (i >= n_pairs) return;
  const CmpPairDev pr = const_load(pairs + i);
  finalize_pair(pr.n_elems, pr.dtype, acc_all, i, copies, res + i);
}

__global__ __launch_bounds__(64) void k_compare_args_finalize(CmpArgPairs a, unsigned long long* acc_all,
                                                              uint32_t copies, kc_cmp_result* res) {
  const uint32_t i = blockIdx.x;
  finalize_pair(a.pair[i].n_elems, a.pair[i].dtype, acc_all, i, copies, res + i);
}

}  // namespace

// The instantiation for a launch shape, called with T and DIRECT.
#define KC_COMPARE_CASE(KERNEL, W, D, ...)                                                                      \
  if (wide == W && direct == D) {                                                                               \
    constexpr uint32_t kT = W ? kWideThreads : kThreads;                                                        \
    hipLaunchKernelGGL((KERNEL<kT, D>), dim3(walk.grid), dim3(kT), 0, s, __VA_ARGS__);                               \
  }
#define KC_COMPARE_LAUNCH(KERNEL, ...)              \
  KC_COMPARE_CASE(KERNEL, true, true, __VA_ARGS__)  \
  KC_COMPARE_CASE(KERNEL, false, true, __VA_ARGS__) \
  KC_COMPARE_CASE(KERNEL, false, false, __VA_ARGS__)

hipError_t launch_compare(const CmpPairDev* pairs, const CmpTileDev* tiles, uint32_t n_tiles, uint32_t tile_bytes,
                          unsigned long long* acc, kc_cmp_result* res, CmpWalk walk, bool wide, bool direct,
                          hipStream_t s) {
  if (n_tiles == 0) return hipSuccess;
  KC_COMPARE_LAUNCH(k_compare, pairs, tiles, n_tiles, tile_bytes, acc, res, walk)
  return hipGetLastError();
}

hipError_t launch_compare_finalize(const CmpPairDev* pairs, uint32_t n_pairs, unsigned long long* acc, uint32_t copies,
                                   kc_cmp_result* res, hipStream_t s) {
  if (n_pairs == 0) return hipSuccess;
  hipLaunchKernelGGL(k_compare_finalize, dim3((n_pairs + 3) / 4), dim3(256), 0, s, pairs, n_pairs, acc, copies, res);
  return hipGetLastError();
}

hipError_t launch_compare_args(const CmpArgPairs& a, uint32_t tile_bytes, unsigned long long* acc,
                               kc_cmp_result* res, CmpWalk walk, bool wide, hipStream_t s) {
  if (a.n == 0) return hipSuccess;
  const bool direct = a.n_tiles == a.n;  // every pair one tile: the pass writes the reports
  KC_COMPARE_LAUNCH(k_compare_args, a, tile_bytes, acc, res, walk)
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || direct) return e;
  hipLaunchKernelGGL(k_compare_args_finalize, dim3(a.n), dim3(64), 0, s, a, acc, walk.copies, res);
  return hipGetLastError();
}
#undef KC_COMPARE_LAUNCH
#undef KC_COMPARE_CASE

}  // namespace kc
