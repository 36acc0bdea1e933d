// hcao_kernels.hip -- gfx950 kernels of the HCAO DSMC collision step.
//
// A workgroup owns a run of consecutive reservoir cells for several steps
// (persistent): it keeps the tables and the cells' headers in LDS, forms NTC
// candidate pairs from a keyed permutation, tests them with the VHS
// acceptance, runs the reaction decision / Larsen-Borgnakke relaxation /
// isotropic scattering of each accepted pair in one lane, and places products
// and removes recombined particles with wavefront ballots. Cells never
// exchange particles, so a launch needs no inter-workgroup communication and
// the result does not depend on the launch shape.
//
// Arithmetic is IEEE fp64 without contraction (built with -ffp-contract=off);
// log/exp are the library's own fixed-sequence versions, so that every
// decision is reproducible bit for bit. The mixed form (MIX) keeps fp32
// velocities, kinematics and sampler arithmetic and fp64 energies.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "hcao_tables.h"

namespace hcao {
namespace {

constexpr double kBoltz = 1.380649e-23;
constexpr uint32_t kDead = 255;  // species of a particle removed by recombination

// Instrumented builds (HCAO_PHASE_CLOCKS) let thread 0 of every step
// workgroup sum the shader clock spent between the barriers that end each
// phase; the default build compiles the marks away.
#ifdef HCAO_PHASE_CLOCKS
#define HCAO_PHASE_MARK(k)               \
  do {                                   \
    if (tid == 0) {                      \
      const uint64_t t_ = clock64();     \
      clk_acc[k] += t_ - clk_t;          \
      clk_t = t_;                        \
    }                                    \
  } while (0)
// per-wave marks inside the collision phase: every active lane reads the
// (wave-uniform) clock, the leading active lane of the wave keeps the sums
#define HCAO_WAVE_MARK(acc, k)           \
  do {                                   \
    const uint64_t t_ = clock64();       \
    (acc)[(k) - kPhaseCollideGather] += t_ - (acc##_t); \
    acc##_t = t_;                        \
  } while (0)
#else
#define HCAO_PHASE_MARK(k) \
  do {                     \
  } while (0)
#define HCAO_WAVE_MARK(acc, k) \
  do {                         \
  } while (0)
#endif

// ---------------------------------------------------------------------------
// Philox4x32-10 counter-based generator (Salmon et al., SC'11)
// ---------------------------------------------------------------------------
__device__ __forceinline__ void philox10(uint32_t k0, uint32_t k1, uint32_t &x0, uint32_t &x1, uint32_t &x2,
                                         uint32_t &x3) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    const uint64_t p0 = (uint64_t)0xD2511F53u * x0, p1 = (uint64_t)0xCD9E8D57u * x2;
    const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
    const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
    const uint32_t y0 = hi1 ^ x1 ^ k0;
    const uint32_t y2 = hi0 ^ x3 ^ k1;
    x0 = y0;
    x1 = lo1;
    x2 = y2;
    x3 = lo0;
  }
}

// A stream (seed; pair, cell, step). The fp64 form takes one 64-bit draw
// (two words, low first) per uniform, (u >> 11) 2^-53; the mixed form takes
// one 32-bit word per uniform, (w >> 8) 2^-24 (exact in either type).
template <bool MIX>
struct RngT {
  uint32_t k0, k1, pair, cell, step, block;
  uint32_t w0, w1, w2, w3;
  uint32_t used;  // words consumed from the current block

  __device__ __forceinline__ void open(uint64_t seed, uint32_t p, uint32_t c, uint32_t s) {
    k0 = (uint32_t)seed;
    k1 = (uint32_t)(seed >> 32);
    pair = p;
    cell = c;
    step = s;
    block = 0;
    used = 4;
  }
  __device__ __forceinline__ void refill() {
    uint32_t x0 = block, x1 = pair, x2 = cell, x3 = step;
    philox10(k0, k1, x0, x1, x2, x3);
    w0 = x0;
    w1 = x1;
    w2 = x2;
    w3 = x3;
    block += 1;
    used = 0;
  }
  // word i of the current block, selected by value: a conditional over the
  // members themselves becomes a choice of addresses, which put the whole
  // generator into scratch memory (every draw of the mixed form then waited
  // for memory: 0.52 against 0.43 ms per step of 65,536 cells)
  __device__ __forceinline__ uint32_t word(uint32_t i) const {
    const uint32_t x0 = w0, x1 = w1, x2 = w2, x3 = w3;
    const uint32_t lo = (i & 1u) ? x1 : x0, hi = (i & 1u) ? x3 : x2;
    return (i & 2u) ? hi : lo;
  }
  __device__ __forceinline__ uint64_t next64() {
    if (used >= 4) refill();
    uint64_t r = (used == 0) ? (((uint64_t)w1 << 32) | w0) : (((uint64_t)w3 << 32) | w2);
    used += 2;
    return r;
  }
  __device__ __forceinline__ uint32_t next32() {
    if (used >= 4) refill();
    const uint32_t r = word(used);
    used += 1;
    return r;
  }
  __device__ __forceinline__ double uniform() {
    if (MIX) return (double)((float)(next32() >> 8) * 0x1p-24f);
    return (double)(next64() >> 11) * 0x1p-53;
  }
  __device__ __forceinline__ float uniform_f() { return (float)(next32() >> 8) * 0x1p-24f; }
  // The next two uniforms of this form as raw words (64-bit in the fp64 form,
  // low word first; 32-bit in the mixed form), with one block computation for
  // both. The fp64 form's pair always needs exactly one new block (two words
  // are left or none), so its lanes never diverge here.
  __device__ __forceinline__ void next_two(uint64_t &a, uint64_t &b) {
    if constexpr (MIX) {
      if (used >= 3) {
        const bool one = used == 3;
        const uint32_t last = w3;
        refill();
        const uint32_t first = w0, second = w1;
        a = one ? last : first;
        b = one ? first : second;
        used = one ? 1u : 2u;
      } else {
        a = word(used);
        b = word(used + 1);
        used += 2;
      }
    } else {
      const bool left = used == 2;
      const uint64_t last = ((uint64_t)w3 << 32) | w2;
      refill();
      const uint64_t lo = ((uint64_t)w1 << 32) | w0, hi = ((uint64_t)w3 << 32) | w2;
      a = left ? last : lo;
      b = left ? lo : hi;
      used = left ? 2u : 4u;
    }
  }
  // a word of next_two as the uniform itself, and in single precision (the
  // fp64 form's estimate: within 2^-32 + 2^-24 u of it)
  static __device__ __forceinline__ double exact_of(uint64_t w) {
    if constexpr (MIX)
      return (double)((float)((uint32_t)w >> 8) * 0x1p-24f);
    else
      return (double)(w >> 11) * 0x1p-53;
  }
  static __device__ __forceinline__ float single_of(uint64_t w) {
    if constexpr (MIX)
      return (float)((uint32_t)w >> 8) * 0x1p-24f;
    else
      return (float)(uint32_t)(w >> 32) * 0x1p-32f;
  }
  // the next uniform's word
  __device__ __forceinline__ uint64_t next_word() {
    if constexpr (MIX)
      return next32();
    else
      return next64();
  }
  // passes over the next n uniforms of this form without using them (blocks
  // wholly passed over are not computed)
  __device__ __forceinline__ void skip(uint32_t n) {
    if (n == 0) return;
    const uint32_t words = MIX ? n : 2 * n;
    // word index within the stream of the next word to be used
    const uint32_t at = (used >= 4 ? 4 * block : 4 * (block - 1) + used) + words;
    const uint32_t b = at / 4, w = at % 4;
    if (w == 0) {
      block = b;
      used = 4;  // the next draw computes block b
    } else if (b != block - 1 || used >= 4) {
      block = b;
      refill();  // computes block b, block = b + 1
      used = w;
    } else {
      used = w;
    }
  }
  // a 53-bit uniform in either form: the next two words (low first); the
  // fp64 form's uniform() takes the same two words
  __device__ __forceinline__ double uniform53() {
    if (!MIX) return uniform();
    const uint64_t lo = next32();
    const uint64_t hi = next32();
    return (double)(((hi << 32) | lo) >> 11) * 0x1p-53;
  }
};
using Rng = RngT<false>;

// Arithmetic type of the velocities, kinematics and sampler draws: fp64 in
// the fp64 form, fp32 in the mixed form.
template <bool MIX>
struct RealOf {
  using type = double;
};
template <>
struct RealOf<true> {
  using type = float;
};
template <bool MIX>
using Real = typename RealOf<MIX>::type;

template <bool MIX>
__device__ __forceinline__ Real<MIX> draw(RngT<MIX> &rng) {
  if constexpr (MIX)
    return rng.uniform_f();
  else
    return rng.uniform();
}

template <typename R>
struct V3 {
  R x, y, z;
};
using Vec3 = V3<double>;

// velocity of slot i in the state's own precision
#ifdef HCAO_CHECKED
// Bounds-checked builds: an index outside [0, n) raises kErrBounds and is
// replaced by 0, so that no access leaves its array (the call then reports
// HCAO_EBOUNDS and its results are void).
__device__ __forceinline__ uint64_t checked_index(uint64_t i, uint64_t n, uint32_t *err) {
  if (i < n) return i;
  atomicOr(err, kErrBounds);
  return 0;
}
#define HCAO_IDX(i, n, err) checked_index((i), (n), (err))
#define HCAO_ERR_PARAM , uint32_t *err
#define HCAO_ERR_ARG(e) , e
#else
#define HCAO_IDX(i, n, err) (i)
#define HCAO_ERR_PARAM
#define HCAO_ERR_ARG(e)
#endif

// a particle's velocity and species
template <typename R>
struct BodyOf {
  V3<R> v;
  uint32_t sp;
};
template <bool MIX>
__device__ __forceinline__ BodyOf<Real<MIX>> ldb(const State &s, uint64_t i) {
  if constexpr (MIX) {
    const Body32 b = s.b32[i];
    return {{b.x, b.y, b.z}, b.sp};
  } else {
    const Body64 b = s.b64[i];
    return {{b.x, b.y, b.z}, (uint32_t)b.sp};
  }
}
template <bool MIX>
__device__ __forceinline__ void stb(const State &s, uint64_t i, V3<Real<MIX>> v, uint32_t sp) {
  if constexpr (MIX)
    s.b32[i] = Body32{v.x, v.y, v.z, sp};
  else
    s.b64[i] = Body64{v.x, v.y, v.z, sp};
}
template <bool MIX>
__device__ __forceinline__ void stv(const State &s, uint64_t i, V3<Real<MIX>> v) {
  if constexpr (MIX) {
    s.b32[i].x = v.x;
    s.b32[i].y = v.y;
    s.b32[i].z = v.z;
  } else {
    s.b64[i].x = v.x;
    s.b64[i].y = v.y;
    s.b64[i].z = v.z;
  }
}
// the same for kernels that serve both forms (the set that is not null)
__device__ __forceinline__ BodyOf<double> load_body(const State &s, uint64_t i) {
  if (s.b32) {
    const Body32 b = s.b32[i];
    return {{(double)b.x, (double)b.y, (double)b.z}, b.sp};
  }
  const Body64 b = s.b64[i];
  return {{b.x, b.y, b.z}, (uint32_t)b.sp};
}
__device__ __forceinline__ void store_body(const State &s, uint64_t i, double x, double y, double z, uint32_t sp) {
  if (s.b32)
    s.b32[i] = Body32{(float)x, (float)y, (float)z, sp};
  else
    s.b64[i] = Body64{x, y, z, sp};
}

// ---------------------------------------------------------------------------
// Fixed-sequence exp / log / pow (Cody-Waite reduction + fixed series)
// ---------------------------------------------------------------------------
__device__ __forceinline__ double dexp(double x) {
  const double kLn2Hi = 0x1.62e42feep-1;
  const double kLn2Lo = 0x1.a39ef35793c76p-33;
  const double kInvLn2 = 0x1.71547652b82fep+0;
  if (x != x) return x;
  if (x > 708.0) return __longlong_as_double(0x7ff0000000000000LL);
  if (x < -707.0) return 0.0;
  const double kd = floor(x * kInvLn2 + 0.5);
  const double r = (x - kd * kLn2Hi) - kd * kLn2Lo;
  double p = 1.0 / 355687428096000.0;  // 1/17!
  p = p * r + 1.0 / 20922789888000.0;
  p = p * r + 1.0 / 1307674368000.0;
  p = p * r + 1.0 / 87178291200.0;
  p = p * r + 1.0 / 6227020800.0;
  p = p * r + 1.0 / 479001600.0;
  p = p * r + 1.0 / 39916800.0;
  p = p * r + 1.0 / 3628800.0;
  p = p * r + 1.0 / 362880.0;
  p = p * r + 1.0 / 40320.0;
  p = p * r + 1.0 / 5040.0;
  p = p * r + 1.0 / 720.0;
  p = p * r + 1.0 / 120.0;
  p = p * r + 1.0 / 24.0;
  p = p * r + 1.0 / 6.0;
  p = p * r + 0.5;
  p = p * r + 1.0;
  p = p * r + 1.0;
  const long long k = (long long)kd;
  return p * __longlong_as_double((k + 1023) << 52);
}

__device__ __forceinline__ double dlog(double x) {
  const double kLn2Hi = 0x1.62e42feep-1;
  const double kLn2Lo = 0x1.a39ef35793c76p-33;
  const double kSqrt2 = 0x1.6a09e667f3bcdp+0;
  if (x != x) return x;
  if (x < 0.0) return __longlong_as_double(0x7ff8000000000000LL);
  if (x == 0.0) return __longlong_as_double((long long)0xfff0000000000000ULL);
  if (x == __longlong_as_double(0x7ff0000000000000LL)) return x;
  int e = 0;
  unsigned long long b = (unsigned long long)__double_as_longlong(x);
  if ((b >> 52) == 0) {
    x = x * 0x1p54;
    b = (unsigned long long)__double_as_longlong(x);
    e = -54;
  }
  e += (int)((b >> 52) & 0x7ff) - 1023;
  double m = __longlong_as_double((long long)((b & 0x000fffffffffffffULL) | 0x3ff0000000000000ULL));
  if (m > kSqrt2) {
    m = m * 0.5;
    e += 1;
  }
  const double s = (m - 1.0) / (m + 1.0);
  const double z = s * s;
  double q = 1.0 / 23.0;
  q = q * z + 1.0 / 21.0;
  q = q * z + 1.0 / 19.0;
  q = q * z + 1.0 / 17.0;
  q = q * z + 1.0 / 15.0;
  q = q * z + 1.0 / 13.0;
  q = q * z + 1.0 / 11.0;
  q = q * z + 1.0 / 9.0;
  q = q * z + 1.0 / 7.0;
  q = q * z + 1.0 / 5.0;
  q = q * z + 1.0 / 3.0;
  q = q * z + 1.0;
  const double t = s * q;
  const double lm = t + t;
  const double ed = (double)e;
  return (ed * kLn2Lo + lm) + ed * kLn2Hi;
}

__device__ __forceinline__ double dpow(double x, double y) {
  if (x == 0.0) return (y > 0.0) ? 0.0 : ((y == 0.0) ? 1.0 : __longlong_as_double(0x7ff0000000000000LL));
  return dexp(y * dlog(x));
}

// Quantum numbers of slot i, a row of s.lrow uint16 read and written as
// dwords (two modes each). load_levels unpacks the first n modes to
// dst[m * ds]; store_levels packs src[m * ss] for m < n and zeros for
// n <= m < top (top >= n: modes only the old species had), in whole dwords
// (a mode past top in the last dword is 0 in the state and stays 0).
__device__ __forceinline__ void load_levels(const State &s, uint64_t i, uint32_t n, uint16_t *dst, uint32_t ds) {
  const uint32_t *row = reinterpret_cast<const uint32_t *>(s.lvl + i * s.lrow);
  for (uint32_t w = 0; 2 * w < n; ++w) {
    const uint32_t x = row[w];
    dst[2 * w * ds] = (uint16_t)(x & 0xFFFFu);
    if (2 * w + 1 < n) dst[(2 * w + 1) * ds] = (uint16_t)(x >> 16);
  }
}
__device__ __forceinline__ void store_levels(const State &s, uint64_t i, uint32_t n, uint32_t top, const uint16_t *src,
                                             uint32_t ss) {
  uint32_t *row = reinterpret_cast<uint32_t *>(s.lvl + i * s.lrow);
  for (uint32_t w = 0; 2 * w < top; ++w) {
    const uint32_t lo = 2 * w < n ? src[2 * w * ss] : 0u;
    const uint32_t hi = 2 * w + 1 < n ? src[(2 * w + 1) * ss] : 0u;
    row[w] = lo | (hi << 16);
  }
}
// the whole row of slot from to slot to (dwords)
__device__ __forceinline__ void copy_levels(const State &src, uint64_t from, const State &dst, uint64_t to) {
  const uint32_t *a = reinterpret_cast<const uint32_t *>(src.lvl + from * src.lrow);
  uint32_t *b = reinterpret_cast<uint32_t *>(dst.lvl + to * dst.lrow);
  for (uint32_t w = 0; w < src.lrow / 2; ++w) b[w] = a[w];
}

// orders the LDS accesses of a wave's lanes before and after it (a wave's LDS
// instructions complete in order; this keeps the compiler from moving them)
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The value lane + S holds, delivered to the lanes that a halving tree
// reads at level S (lane < S); other lanes receive arbitrary values. VALU
// cross-lane moves of gfx950 instead of LDS-routed shuffles: the 32- and
// 16-lane swaps for S = 32 and 16, DPP row shifts for S = 8 .. 1.
template <int S>
__device__ __forceinline__ uint32_t lane_down(uint32_t v) {
  if constexpr (S == 32)
    return __builtin_amdgcn_permlane32_swap(v, v, false, false)[1];
  else if constexpr (S == 16)
    return __builtin_amdgcn_permlane16_swap(v, v, false, false)[1];
  else
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x100 + S, 0xF, 0xF, false);
}
template <int S>
__device__ __forceinline__ double tree_down(double v) {
  const uint32_t lo = lane_down<S>((uint32_t)__double2loint(v));
  const uint32_t hi = lane_down<S>((uint32_t)__double2hiint(v));
  return __hiloint2double((int)hi, (int)lo);
}
// Halving tree over the 64 lanes of a wave (lane t adds lane t + s, s = 32
// .. 1): lane 0 ends with the sum, in that order; every lane must be active.
template <int N>
__device__ __forceinline__ void tree_sum(double (&y)[N]) {
#pragma unroll
  for (int x = 0; x < N; ++x) y[x] = y[x] + tree_down<32>(y[x]);
#pragma unroll
  for (int x = 0; x < N; ++x) y[x] = y[x] + tree_down<16>(y[x]);
#pragma unroll
  for (int x = 0; x < N; ++x) y[x] = y[x] + tree_down<8>(y[x]);
#pragma unroll
  for (int x = 0; x < N; ++x) y[x] = y[x] + tree_down<4>(y[x]);
#pragma unroll
  for (int x = 0; x < N; ++x) y[x] = y[x] + tree_down<2>(y[x]);
#pragma unroll
  for (int x = 0; x < N; ++x) y[x] = y[x] + tree_down<1>(y[x]);
}

// The same tree over six values at once, packed as it shrinks: the 32- and
// 16-lane swaps take two registers each and leave the two values' halves side
// by side, so that one addition serves both, and the 8-lane level puts the
// last register into the upper halves of the rows. Every addition is the one
// tree_sum makes (lane t's partial sum plus lane t + s's), 10 of them instead
// of 36. tree6_value(lane) tells where each value ends;
// what the other lanes hold is of no use.
__device__ __forceinline__ double swap_add32(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)__double2loint(a), (uint32_t)__double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)__double2hiint(a), (uint32_t)__double2hiint(b), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double swap_add16(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)__double2loint(a), (uint32_t)__double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)__double2hiint(a), (uint32_t)__double2hiint(b), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
// lanes 0-7 of each row: a; lanes 8-15: b of the lane eight below
__device__ __forceinline__ uint32_t upper_half(uint32_t a, uint32_t b) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)a, (int)b, 0x118, 0xF, 0xC, false);
}
__device__ __forceinline__ double tree_sum6(double y0, double y1, double y2, double y3, double y4, double y5) {
  const double s01 = swap_add32(y0, y1), s23 = swap_add32(y2, y3), s45 = swap_add32(y4, y5);
  double a = swap_add16(s01, s23);  // rows: y0 y2 y1 y3
  double b = swap_add16(s45, s45);  // rows: y4 y4 y5 y5
  a = a + tree_down<8>(a);
  b = b + tree_down<8>(b);
  double c = __hiloint2double((int)upper_half((uint32_t)__double2hiint(a), (uint32_t)__double2hiint(b)),
                              (int)upper_half((uint32_t)__double2loint(a), (uint32_t)__double2loint(b)));
  c = c + tree_down<4>(c);
  c = c + tree_down<2>(c);
  return c + tree_down<1>(c);
}
// which value a lane holds after tree_sum6 (6: none)
__device__ __forceinline__ uint32_t tree6_value(uint32_t lane) {
  return lane == 0 ? 0u : lane == 32 ? 1u : lane == 16 ? 2u : lane == 48 ? 3u : lane == 8 ? 4u : lane == 40 ? 5u : 6u;
}

// Exact comparisons against a power through a single-precision filter.
// est = 2^(y log2 x) from the hardware log2/exp2 (v_log_f32, v_exp_f32) is
// within 5e-6 of x^y for x in [2^-53, 2^64] and y in (0, 1] (measured over
// 1.7e7 operands); a decision further than kFilter from est is the one the
// fp64 power gives, and only the band in between evaluates dpow. The
// result of every comparison is therefore that of the fp64 expression.
constexpr double kFilter = 1e-4;

__device__ __forceinline__ double pow_estimate(double x, double y) {
  return (double)__builtin_amdgcn_exp2f((float)y * __builtin_amdgcn_logf((float)x));
}

// u < x^y (as dpow computes it), for x in (0, 1] and y in (0, 1]
__device__ __forceinline__ bool below_pow(double u, double x, double y) {
  const double est = pow_estimate(x, y);
  if (u < est * (1.0 - kFilter)) return true;
  if (u > est * (1.0 + kFilter)) return false;
  return u < dpow(x, y);
}

// x^y in single precision (mixed form)
__device__ __forceinline__ float pow_f(float x, float y) {
  return __builtin_amdgcn_exp2f(y * __builtin_amdgcn_logf(x));
}

// Larsen-Borgnakke acceptance u < (num / den)^q for num, den > 0: the fp64
// form divides in fp64 and decides as the fp64 power does; the mixed form
// takes the ratio and the power in fp32 (u is then an fp32 draw)
template <bool MIX>
__device__ __forceinline__ bool lb_accept(double u, double num, double den, double q) {
  if constexpr (MIX)
    return (float)u < pow_f((float)num / (float)den, (float)q);
  else
    return below_pow(u, num / den, q);
}

// ---------------------------------------------------------------------------
// keyed permutation of [0, n): Feistel network on Z_m x Z_m, m = ceil(sqrt n),
// with addition modulo m (generalised Feistel cipher, Black-Rogaway), 16
// rounds for m <= 8 and 10 above, cycle walking into [0, n) (m^2 / n < 1.2
// for n >= 25, so walks are short). The round function multiplies 24-bit
// factors (full-rate v_mul_u32_u24) and scales the hash to [0, m) by its
// high product with m.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t feistel_f(uint32_t r, uint32_t key, uint32_t m) {
  uint32_t h = __umul24(r ^ key, 0x9E3779u);
  h ^= h >> 15;
  h = __umul24(h, 0x85EBCBu);
  h ^= h >> 13;
  return __umulhi(h, m);
}

struct Perm {
  uint32_t n, m, pad, rounds;
  uint32_t k[16];
};

// the permutation evaluated with its keys in registers
struct PermReg {
  uint32_t n, m, rounds;
  uint32_t k[16];
  __device__ __forceinline__ void load(const Perm &P) {
    n = P.n;
    m = P.m;
    rounds = P.rounds;
#pragma unroll
    for (int i = 0; i < 16; ++i) k[i] = P.k[i];
  }
  template <int R>
  __device__ __forceinline__ void once_r(uint32_t &l, uint32_t &r) const {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      uint32_t s = l + feistel_f(r, k[i], m);
      s = s >= m ? s - m : s;
      l = r;
      r = s;
    }
  }
  __device__ __forceinline__ void once(uint32_t &l, uint32_t &r) const {
    if (rounds == 10)
      once_r<10>(l, r);
    else
      once_r<16>(l, r);
  }
  // i = l m + r. Below 2^24 the quotient comes from a single-precision
  // estimate, off by at most one and put right by its remainder (an integer
  // division takes three times the instructions).
  __device__ __forceinline__ void divide(uint32_t i, uint32_t &l, uint32_t &r) const {
    if (n <= (1u << 24)) {
      l = (uint32_t)((float)i * __builtin_amdgcn_rcpf((float)m));
      r = i - l * m;
      if ((int32_t)r < 0) {
        l -= 1u;
        r += m;
      } else if (r >= m) {
        l += 1u;
        r -= m;
      }
    } else {
      l = i / m;
      r = i - l * m;
    }
  }
  __device__ __forceinline__ uint32_t operator()(uint32_t i) const {
    uint32_t l, r;
    divide(i, l, r);
    once(l, r);
    while (l * m + r >= n) once(l, r);
    return l * m + r;
  }
  // the images a, b of 2k and 2k + 1. The two first evaluations run side by
  // side; then one walk serves both: a lane steps whichever of its two
  // values still lies outside [0, n). Two walks after one another each
  // lasted until the slowest lane of the wave was inside (at 300 particles
  // per cell about 2.6 evaluations each, 5.2 per 64 pairs; now 3.8).
  __device__ __forceinline__ void pair(uint32_t k, uint32_t &a, uint32_t &b) const {
    uint32_t l0, r0;
    divide(2 * k, l0, r0);
    uint32_t l1 = l0, r1 = r0 + 1u;
    if (r1 == m) {
      l1 += 1u;
      r1 = 0;
    }
    once(l0, r0);
    once(l1, r1);
    a = l0 * m + r0;
    b = l1 * m + r1;
    while (a >= n || b >= n) {
      const bool first = a >= n;
      uint32_t l = first ? l0 : l1, r = first ? r0 : r1;
      once(l, r);
      const uint32_t x = l * m + r;
      if (first) {
        l0 = l;
        r0 = r;
        a = x;
      } else {
        l1 = l;
        r1 = r;
        b = x;
      }
    }
  }
};

__device__ __forceinline__ void make_perm(Perm &P, uint32_t n, uint64_t seed, uint32_t cell, uint32_t step) {
  P.n = n;
  uint32_t m = (uint32_t)sqrtf((float)n);
  while (m * m < n) ++m;
  while (m > 1 && (m - 1) * (m - 1) >= n) --m;
  P.m = m;
  P.pad = 0;
  P.rounds = m <= 8 ? 16u : 10u;
  const uint32_t k0 = (uint32_t)seed, k1 = (uint32_t)(seed >> 32);
#pragma unroll
  for (uint32_t blk = 0; blk < 4; ++blk) {
    uint32_t x0 = blk, x1 = 0xFFFFFFFFu, x2 = cell, x3 = step;
    philox10(k0, k1, x0, x1, x2, x3);
    P.k[4 * blk] = x0;
    P.k[4 * blk + 1] = x1;
    P.k[4 * blk + 2] = x2;
    P.k[4 * blk + 3] = x3;
  }
}

// ---------------------------------------------------------------------------
// tables in LDS
// ---------------------------------------------------------------------------
// species / pair / reaction tables and stretch levels, staged in LDS
struct Tab {
  const SpeciesTab *sp;
  const PairTab *pr;  // [a * ns + b]
  const ReactionTab *rx;
  const double *lev;
  const double *beta;  // exact sampler's beta tables (global memory)
  uint32_t ns, nr, mm, rec_nt;
  __device__ __forceinline__ const PairTab &pair(uint32_t a, uint32_t b) const { return pr[a * ns + b]; }
};

struct Ctx {
  Tab T;
  unsigned long long *ctr;  // LDS counters of the pair's cell
  uint16_t *scr;            // per-lane scratch, [2 * max_modes][block]
  uint32_t lane, block;
};

__device__ __forceinline__ double mode_energy(const SpeciesTab &S, const double *lev, uint32_t m, uint32_t i) {
  if (m < S.n_bend) return ((double)i + 0.5) * S.kt[m];
  return lev[S.lev_off[m] + i];
}

__device__ __forceinline__ double vib_energy(const SpeciesTab &S, const double *lev, const uint16_t *lv,
                                             uint32_t stride) {
  // bends, then stretches: two plain loops whose table reads do not wait for
  // the running sum
  double e = 0.0;
  const uint32_t nb = S.n_bend, nm = S.n_modes;
#pragma unroll 2
  for (uint32_t m = 0; m < nb; ++m) e = e + ((double)lv[m * stride] + 0.5) * S.kt[m];
#pragma unroll 2
  for (uint32_t m = nb; m < nm; ++m) e = e + lev[S.lev_off[m] + lv[m * stride]];
  return e;
}

// top quantum number of a bend of energy quantum kt that may hold energy e:
// floor(e / kt - 1/2) clamped to 0..65535. The quotient's single-precision
// estimate is within 3e-7 (x + 1); only one within 1e-6 (x + 1) of an
// integer evaluates the fp64 division, so the level is the fp64
// expression's.
__device__ __forceinline__ uint32_t bend_top(double kt, float inv_kt, double e) {
  const float x = (float)e * inv_kt - 0.5f;
  if (fabsf(x - rintf(x)) > 1e-6f * (fabsf(x) + 1.0f)) {
    const float f = floorf(x);
    return f < 0.0f ? 0u : (f > 65535.0f ? 65535u : (uint32_t)f);
  }
  double fi = floor(e / kt - 0.5);
  fi = fi < 0.0 ? 0.0 : fi;
  fi = fi > 65535.0 ? 65535.0 : fi;
  return (uint32_t)fi;
}

// highest level of stretch m strictly below e (the ladder increases
// strictly), at least 0, and its energy. A Morse ladder is inverted in
// single precision, v = 2 t / (1 + sqrt(1 - 4 x_e t)) with t = e / (h c w_e)
// (SpeciesTab::guess: the host has checked v against every level of the
// ladder), and three levels around the guess, read together, settle it;
// other ladders are bisected (five dependent reads for 22 levels).
__device__ __forceinline__ uint32_t stretch_top(const SpeciesTab &S, const double *lev, uint32_t m, double e,
                                                double &e_top) {
  const double *L = lev + S.lev_off[m];
  const uint32_t d = S.idiss[m];
  if ((S.guess >> m) & 1u) {
    const float t = (float)e * S.inv[m];
    const float v = (t + t) * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_sqrtf(fmaxf(1.0f - S.anharm4[m] * t, 0.0f)));
    const float f = fminf(fmaxf(v - 0.5f, 0.0f), (float)d);
    const uint32_t g = (uint32_t)f;
    const uint32_t up = g < d ? g + 1u : d, dn = g ? g - 1u : 0u;
    const double eg = L[g], eu = L[up], ed = L[dn];
    if (g < d && eu < e) {
      e_top = eu;
      return up;
    }
    if (g && !(eg < e)) {
      e_top = ed;
      return dn;
    }
    e_top = eg;
    return g;
  }
  uint32_t lo = 0, hi = d;
  while (lo < hi) {
    const uint32_t mid = (lo + hi + 1) >> 1;
    if (L[mid] < e)
      lo = mid;
    else
      hi = mid - 1;
  }
  e_top = L[lo];
  return lo;
}

// top quantum number a mode may be proposed at, given the energy e it may hold
__device__ __forceinline__ uint32_t mode_top(const SpeciesTab &S, const double *lev, uint32_t m, double e) {
  if (m < S.n_bend) return bend_top(S.kt[m], S.inv[m], e);
  double unused;
  return stretch_top(S, lev, m, e, unused);
}

// uniform level on 0..top from one draw: min(floor(u (top + 1)), top)
template <bool MIX>
__device__ __forceinline__ uint32_t pick_level(uint32_t top, RngT<MIX> &rng) {
  uint32_t i;
  if constexpr (MIX)
    i = (uint32_t)(rng.uniform_f() * (float)(top + 1));
  else
    i = (uint32_t)floor(rng.uniform() * ((double)top + 1.0));
  return i > top ? top : i;
}

// u < exp(-a) for a >= 0, decided as the fp64 dexp decides (fp32 filter)
__device__ __forceinline__ bool below_exp_neg(double u, double a) {
  const double est = (double)__builtin_amdgcn_exp2f(-(float)a * 1.44269504f);
  if (u < est * (1.0 - kFilter)) return true;
  if (u > est * (1.0 + kFilter)) return false;
  return u < dexp(-a);
}

// Exact sampler, level proposal of one mode in the form's own arithmetic: the
// geometric level floor(-ln(1 - u) / c) with c = beta * slope. Returns false
// when it lies above top (the caller draws again).
template <bool MIX>
__device__ __forceinline__ bool geometric_exact(double u, double c, uint32_t top, uint32_t &i) {
  if constexpr (MIX) {
    const float x = -__builtin_amdgcn_logf(1.0f - (float)u) * (0.69314718f / (float)c);
    if (!(x < (float)top + 1.0f)) return false;
    i = (uint32_t)floorf(x);
    return true;
  } else {
    const double x = -dlog(1.0 - u) / c;
    if (!(x < (double)top + 1.0)) return false;
    i = (uint32_t)floor(x);
    return true;
  }
}
// The same from a single-precision estimate with k = ln 2 / c (to 1e-6): clear
// is set when it settles the level, which is then the one geometric_exact
// gives; ok tells whether the level is at most top.
template <bool MIX>
__device__ __forceinline__ bool geometric_estimate(uint64_t w, float k, uint32_t top, uint32_t &i, bool &clear) {
  float v;
  bool fine = true;
  if constexpr (MIX) {
    v = 1.0f - RngT<MIX>::single_of(w);
  } else {
    const uint32_t h = ~(uint32_t)(w >> 32);
    fine = h >= (1u << 21);  // 1 - u to 5e-7
    v = (float)h * 0x1p-32f;
  }
  const float ftop1 = (float)top + 1.0f;
  const float x = -__builtin_amdgcn_logf(v) * k;
  const float band = 1e-5f * (x + 1.0f) + 2e-6f * k;
  const float fl = floorf(x);
  i = (uint32_t)fminf(fl, (float)top);
  const bool above = x >= ftop1 + band;
  clear = fine && (above || (x - fl > band && (fl + 1.0f) - x > band && x < ftop1 - band));
  return !above;
}

// Exact sampler, slope of the geometric proposal of mode m on 0..top: the
// harmonic spacing of a bend; for a stretch the chord (E_top - E_0) / top,
// a lower bound of (E_i - E_0) / i when the spacings never grow, else the
// smallest (E_i - E_0) / i
__device__ __forceinline__ double exact_slope(const SpeciesTab &S, const double *lev, uint32_t m, uint32_t top) {
  if (m < S.n_bend) return S.kt[m];
  const double *L = lev + S.lev_off[m];
  if ((S.concave >> m) & 1u) return (L[top] - L[0]) / (double)top;
  double sl = L[1] - L[0];
  for (uint32_t i = 2; i <= top; ++i) {
    const double v = (L[i] - L[0]) / (double)i;
    if (v < sl) sl = v;
  }
  return sl;
}

// a value the compiler has to take as new: what depends on it is read or
// computed again where it is used, instead of being held in registers from an
// earlier use or hoisted out of the branch that needs it
__device__ __forceinline__ void renew(uint32_t &x) { asm volatile("" : "+v"(x)); }

// Gibbs proposal and acceptance in the form's own arithmetic. de_top = E_top
// - E_0, den = E_c - E_0; slope tells whether the linear envelope applies.
__device__ __forceinline__ double gibbs_slope(bool slope, double q, double de_top, uint32_t top, double den) {
  return slope ? (q * de_top) / ((double)top * den) : 0.0;
}
template <bool MIX>
__device__ __forceinline__ uint32_t gibbs_level(double u, bool slope, double q, double de_top, uint32_t top,
                                                double den) {
  const double c = gibbs_slope(slope, q, de_top, top, den);
  const double z = ((double)top + 1.0) * (1.0 - (0.5 * c) * (double)top);
  const double h = 1.0 + 0.5 * c;
  const double hh = h * h, c2 = 2.0 * c;
  if constexpr (MIX) {
    const float sv = (float)u * (float)z;
    const float k = (2.0f * sv) / ((float)h + sqrtf((float)hh - (float)c2 * sv));
    const float fi = floorf(k);
    return fi > (float)top ? top : (uint32_t)fi;
  } else {
    const double sv = u * z;
    const double k = (2.0 * sv) / (h + sqrt(hh - c2 * sv));
    const double fi = floor(k);
    return fi > (double)top ? top : (uint32_t)fi;
  }
}
template <bool MIX>
__device__ __forceinline__ bool gibbs_accept(double ua, bool slope, double q, double de_top, uint32_t top, double den,
                                             uint32_t i, double ec, double ei) {
  const double c = gibbs_slope(slope, q, de_top, top, den);
  if (!(ei < ec)) return false;
  if constexpr (MIX) {
    const float w = 1.0f - (float)c * (float)i;
    return lb_accept<MIX>((double)((float)ua * w), ec - ei, den, q);
  } else {
    return lb_accept<MIX>(ua * (1.0 - c * (double)i), ec - ei, den, q);
  }
}
// When a single-precision Gibbs trial is clear of a boundary. The estimates
// of c, z and h carry a few 1e-7 each, and the inverse's square root turns
// the error d of its argument into d / (2 sqrt(arg)): above kGibbsDisc the
// inverse k is within 6e-6 (k + 1) of the exact one, the product u w within
// 1e-6, the power within 2e-6 of itself.
constexpr float kGibbsTol = 3e-5f;
constexpr float kGibbsDisc = 0.05f;
constexpr float kGibbsBand = 5e-5f;

// Larsen-Borgnakke relaxation of one molecule (levels at lv[m * stride]);
// e_tr is the pair's translational energy on entry and exit; btab is the
// molecule's beta table (exact sampler only). The exact sampler is compiled
// only into the instantiations with EX set, which run when some species
// uses it, so that it does not weigh on the register allocation of the
// others.
template <bool MIX, bool EX>
__device__ uint32_t relax(const Ctx &C, const SpeciesTab &S, uint16_t *lv, uint32_t stride, double &e_tr,
                          double q, const double *btab, RngT<MIX> &rng, bool &capped) {
  uint32_t trials = 0;
  capped = false;
  const uint32_t nm = S.n_modes;
  if (EX && S.sampler == HCAO_SAMPLER_EXACT) {
    // Independent draw from the joint target (E' - S)^q on S < E' (S: sum of
    // the modes' energies above their ground levels, E' = E_coll - ZPE) by
    // rejection from per-mode Boltzmann proposals at inverse temperature
    // beta: bends geometric, stretches geometric on the chord slope thinned
    // by exp(-beta (E_i - E_0 - slope i)); target / proposal over its
    // maximum is exp(q (ln y + 1 - y)), y = beta (E' - S) / q.
    const double e_coll = e_tr + vib_energy(S, C.T.lev, lv, stride);
    const double ep = e_coll - S.zpe;
    if (!(ep > 0.0)) return 0;
    uint32_t bin = (uint32_t)((unsigned long long)__double_as_longlong(ep) >> 48);
    bin = bin < kExactBinLo ? kExactBinLo : (bin > kExactBinHi ? kExactBinHi : bin);
    double beta = btab[bin - kExactBinLo];
    if (beta * ep < q) beta = q / ep;
    uint16_t *tops = C.scr + C.lane;
    uint16_t *cand = C.scr + (size_t)nm * C.block + C.lane;
    const double *lev = C.T.lev;
    for (uint32_t m = 0; m < nm; ++m)
      tops[m * C.block] = (uint16_t)mode_top(S, lev, m, ep + mode_energy(S, lev, m, 0));
    // Levels, thinning and acceptance are decided from single-precision
    // estimates; only a decision near its boundary evaluates the form's own
    // expressions (each mode's draw took three fp64 divisions before).
    const float bf = (float)beta, kb = 0.69314718f * __builtin_amdgcn_rcpf(bf);
    const float rq = __builtin_amdgcn_rcpf((float)q), qf = (float)q;
    for (;;) {
      double sum = 0.0;
      for (uint32_t m = 0; m < nm && !capped; ++m) {
        const uint32_t top = tops[m * C.block];
        const bool bend = m < S.n_bend;
        const double kt = S.kt[m];
        const double *L = lev + S.lev_off[m];  // a bend reads level 0 of the array and ignores it
        const double l0 = L[0];
        const double e0 = bend ? 0.5 * kt : l0;
        uint32_t i = 0;
        double de = 0.0;  // E_i - E_0
        if (top > 0) {
          // the slope to 1e-6: 1 / slope of a bend is tabulated, a stretch's
          // chord is divided in single precision
          const bool chord = !bend && ((S.concave >> m) & 1u);
          float slf = 0.0f, inv = S.inv[m];
          if (!bend) {
            slf = chord ? (float)(L[top] - l0) * __builtin_amdgcn_rcpf((float)top) : (float)exact_slope(S, lev, m, top);
            inv = __builtin_amdgcn_rcpf(slf);
          }
          const float k = kb * inv;
          for (;;) {
            ++trials;
            if (trials >= kMaxTrials) {
              capped = true;
              break;
            }
            const uint64_t w = rng.next_word();
            bool clear;
            bool ok = geometric_estimate<MIX>(w, k, top, i, clear);
            if (!clear) {
              uint32_t t = top;  // (taken as new: the slope's division would be hoisted to every mode)
              renew(t);
              ok = geometric_exact<MIX>(RngT<MIX>::exact_of(w), beta * exact_slope(S, lev, m, t), t, i);
            }
            if (!ok) continue;
            const double li = L[bend ? 0u : i];
            de = (bend ? ((double)i + 0.5) * kt : li) - e0;
            if (!bend && i > 0) {
              const float def = (float)de;
              float df = def - slf * (float)i;
              const bool sure = fabsf(df) > 1e-5f * def;
              double d = 0.0;
              if (!sure) {
                uint32_t t = top;
                renew(t);
                d = de - exact_slope(S, lev, m, t) * (double)i;
                df = d > 0.0 ? 1.0f : -1.0f;
              }
              if (df > 0.0f) {
                const uint64_t w2 = rng.next_word();
                const float est = __builtin_amdgcn_exp2f(-(bf * df) * 1.44269504f);
                const float u2 = RngT<MIX>::single_of(w2);
                bool keep = u2 < est;
                if (!sure || fabsf(u2 - est) <= 1e-4f * est + 1e-6f) {
                  uint32_t t = top;
                  renew(t);
                  d = de - exact_slope(S, lev, m, t) * (double)i;
                  if constexpr (MIX)
                    keep = u2 < __builtin_amdgcn_exp2f(-(float)(beta * d) * 1.44269504f);
                  else
                    keep = below_exp_neg(RngT<MIX>::exact_of(w2), beta * d);
                }
                if (!keep) continue;
              }
            }
            break;
          }
        }
        cand[m * C.block] = (uint16_t)i;
        sum = sum + (capped ? mode_energy(S, lev, m, i) - e0 : de);
      }
      if (capped) break;
      ++trials;
      if (sum < ep) {
        const uint64_t w = rng.next_word();
        const float yf = (bf * (float)(ep - sum)) * rq;
        const float ex = qf * ((__builtin_amdgcn_logf(yf) * 0.69314718f + 1.0f) - yf);
        const float est = __builtin_amdgcn_exp2f(ex * 1.44269504f);
        const float ua = RngT<MIX>::single_of(w);
        bool ok = ua < est;
        // (the estimate of ex is within 2e-6 (1 + |ex|) of the exact one)
        if (!(fabsf(ua - est) > (1e-5f + 4e-6f * fabsf(ex)) * est + 1e-6f)) {
          const double y = (beta * (ep - sum)) / q;
          const float y2 = (float)y;
          const float ex2 = qf * ((__builtin_amdgcn_logf(y2) * 0.69314718f + 1.0f) - y2);
          if constexpr (MIX) {
            ok = ua < __builtin_amdgcn_exp2f(ex2 * 1.44269504f);
          } else {
            const double u = RngT<MIX>::exact_of(w);
            const double est2 = (double)__builtin_amdgcn_exp2f(ex2 * 1.44269504f);
            if (u < est2 * (1.0 - kFilter))
              ok = true;
            else if (u > est2 * (1.0 + kFilter))
              ok = false;
            else
              ok = u < dexp(q * ((dlog(y) + 1.0) - y));
          }
        }
        if (ok) {
          double ev = 0.0;
          for (uint32_t m = 0; m < nm; ++m) {
            const uint16_t l = cand[m * C.block];
            lv[m * stride] = l;
            ev = ev + mode_energy(S, C.T.lev, m, l);
          }
          e_tr = e_coll - ev;
          break;
        }
      }
      if (trials >= kMaxTrials) {
        capped = true;
        break;
      }
    }
    return trials;
  }
  // Gibbs sweep: the level of mode m is proposed from the linear envelope
  // w_i = 1 - c i of the target ((E_c - E_i) / (E_c - E_0))^q on 0..top
  // (valid for q <= 1 and levels whose spacings never grow; c = 0 gives the
  // uniform proposal) by inverting its discrete CDF, and accepted with
  // probability target / w_i.
  //
  // The proposed level and the acceptance are decided from single-precision
  // estimates of c, the CDF's inverse and the power; a proposal too near a
  // boundary (an integer of the inverse, a square root near 0, or u near the
  // target) is decided by the form's own expressions (gibbs_level and
  // gibbs_accept), so every decision is theirs. A wave waits here for its
  // slowest lane at each mode, so the length of this chain sets the time of the
  // collision phase: in the form's own arithmetic it held two fp64 divisions and
  // a bisection per mode, and two divisions and a square root per trial.
  double et = e_tr;
  const double *lev = C.T.lev;
  const float qf = (float)q;
  for (uint32_t m = 0; m < nm; ++m) {
    const bool bend = m < S.n_bend;
    const double kt = S.kt[m];
    const double *L = lev + S.lev_off[m];  // a bend reads level 0 of the array and ignores it
    const uint32_t cur = lv[m * stride];
    const double l0 = L[0], lc = L[bend ? 0u : cur];
    const double e0 = bend ? 0.5 * kt : l0;
    const double ec = et + (bend ? ((double)cur + 0.5) * kt : lc);
    const double den = ec - e0;
    if (!(den > 0.0)) continue;
    uint32_t top;
    double e_top;
    if (bend) {
      top = bend_top(kt, S.inv[m], ec);
      e_top = ((double)top + 0.5) * kt;
    } else {
      top = stretch_top(S, lev, m, ec, e_top);
    }
    const bool slope = top > 0 && ((S.concave >> m) & 1u);
    const float tf = (float)top;
    const float rden = __builtin_amdgcn_rcpf((float)den);
    const float cf = slope ? (qf * (float)(e_top - e0)) * (rden * __builtin_amdgcn_rcpf(tf)) : 0.0f;
    const float zf = (tf + 1.0f) * (1.0f - (0.5f * cf) * tf);
    const float hf = 1.0f + 0.5f * cf;
    const float hhf = hf * hf, c2f = 2.0f * cf;
    for (;;) {
      ++trials;
      uint64_t w1, w2;
      rng.next_two(w1, w2);
      const float sv = RngT<MIX>::single_of(w1) * zf;
      const float disc = hhf - c2f * sv;
      const float k = (sv + sv) * __builtin_amdgcn_rcpf(hf + __builtin_amdgcn_sqrtf(disc));
      const float fl = floorf(k), fr = k - fl;
      const float tol = kGibbsTol * (k + 1.0f);
      bool clear = (disc > kGibbsDisc) & (fr > tol) & (fr < 1.0f - tol);
      uint32_t i = (uint32_t)fminf(fl, tf);
      const double li = L[bend ? 0u : i];
      double ei = bend ? ((double)i + 0.5) * kt : li;
      const float a = RngT<MIX>::single_of(w2) * (1.0f - cf * (float)i);
      const float est = __builtin_amdgcn_exp2f(qf * __builtin_amdgcn_logf((float)(ec - ei) * rden));
      const bool below = ei < ec;
      bool ok = below & (a < est);
      clear = clear & (!below | (fabsf(a - est) > kGibbsBand * est + 1e-6f));
      if (!clear) {
        // (top taken as new: its divisions would be hoisted to every mode)
        uint32_t t = top;
        renew(t);
        i = gibbs_level<MIX>(RngT<MIX>::exact_of(w1), slope, q, e_top - e0, t, den);
        ei = mode_energy(S, lev, m, i);
        ok = gibbs_accept<MIX>(RngT<MIX>::exact_of(w2), slope, q, e_top - e0, t, den, i, ec, ei);
      }
      if (ok) {
        lv[m * stride] = (uint16_t)i;
        et = ec - ei;
        break;
      }
      if (trials >= kMaxTrials) {
        capped = true;
        break;
      }
    }
    if (capped) break;
  }
  e_tr = et;
  return trials;
}

// The joint sampler's molecules of a wave, one slot per lane (LDS)
struct JointJob {
  double e_coll;
  uint32_t pos, pair, cell;  // first word of the next trial, the stream
  uint8_t sp, pr;            // the molecule's species, the pair table entry of its exponent
  uint16_t owner;            // slot i of a wave's lanes names its i-th unaccepted molecule's lane
};
static_assert(sizeof(JointJob) == 24 && kMaxSpecies * kMaxSpecies <= 256, "the joint sampler's LDS slots");

// Joint sampler (uniform proposals over the box of levels, one acceptance of
// the whole vector) for the lanes of a wave with job set; every lane of the
// wave takes part. Trial t of a molecule always takes the same n_modes + 1
// uniforms of its stream, so trials are independent work: the lanes of a wave
// share out the next trials of the molecules still unaccepted (G = 2^sh lanes
// each), and the first accepted trial in stream order wins, which is the one a
// serial loop stops at. One lane per molecule keeps the whole wave until its
// slowest molecule is accepted (a mean of 16 trials for the triatomic, about
// 75 for the slowest of 64); shared out, 64 of them take about 25 rounds.
//
// A molecule's tops are rows 0 .. n_modes - 1 of its owner's column of the
// scratch; a trial's proposals are rows max_modes on of the column of the lane
// that tests it. A lane may test a molecule with fewer modes than the one it
// owns, whose tops must outlast the test.
template <bool MIX>
__device__ __forceinline__ uint32_t relax_joint(const Ctx &C, JointJob *J, bool job, uint32_t sp, uint32_t partner,
                                                uint16_t *lv, uint32_t stride, double &e_tr, RngT<MIX> &rng,
                                                bool &capped) {
  const double *lev = C.T.lev;
  // (the proposals' first row taken as new: computed outside, it holds registers
  // of every step, 1.5% of the fp64 chemistry)
  uint32_t mm = C.T.mm;
  renew(mm);
  const uint32_t lane = C.lane & 63u, first_lane = C.lane - lane;
  const unsigned long long lt = lane ? ((1ull << lane) - 1ull) : 0ull;
  double e_coll = 0.0;
  uint32_t trials = 0, nm = 0;
  capped = false;
  if (job) {
    const SpeciesTab &S = C.T.sp[sp];
    nm = S.n_modes;
    e_coll = e_tr + vib_energy(S, lev, lv, stride);
    const double denom = e_coll - S.zpe;
    job = denom > 0.0;
    if (job) {
      for (uint32_t m = 0; m < nm; ++m) C.scr[m * C.block + C.lane] = (uint16_t)mode_top(S, lev, m, e_coll);
      J[C.lane].e_coll = e_coll;
      J[C.lane].pos = rng.used >= 4 ? 4 * rng.block : 4 * (rng.block - 1) + rng.used;  // next word of the stream
      J[C.lane].pair = rng.pair;
      J[C.lane].cell = rng.cell;
      J[C.lane].sp = (uint8_t)sp;
      J[C.lane].pr = (uint8_t)(sp * C.T.ns + partner);
    }
  }
  unsigned long long pend = __ballot(job);
  while (pend) {
    const uint32_t np = (uint32_t)__popcll(pend);
    const uint32_t sh = 6u - (np > 1 ? 32u - (uint32_t)__builtin_clz(np - 1u) : 0u), G = 1u << sh;
    const uint32_t rank = (uint32_t)__popcll(pend & lt);
    if (job) {
      J[first_lane + rank].owner = (uint16_t)lane;
    }
    wave_sync();
    bool ok = false;
    double sum = 0.0;
    if ((lane >> sh) < np) {
      const uint32_t o = first_lane + J[first_lane + (lane >> sh)].owner;
      const SpeciesTab &S = C.T.sp[J[o].sp];
      const uint32_t n = S.n_modes;
      const uint32_t at = J[o].pos + (lane & (G - 1u)) * (n + 1u) * (MIX ? 1u : 2u);
      RngT<MIX> r = rng;
      r.pair = J[o].pair;
      r.cell = J[o].cell;
      r.block = at / 4u;
      r.used = 4;
      if (at % 4u) {
        r.refill();
        r.used = at % 4u;
      }
      uint16_t *cand = C.scr + mm * C.block + C.lane;
      for (uint32_t m = 0; m < n; ++m) {
        const uint32_t i = pick_level<MIX>(C.scr[m * C.block + o], r);
        cand[m * C.block] = (uint16_t)i;
        sum = sum + mode_energy(S, lev, m, i);
      }
      const double ua = (double)draw<MIX>(r);
      const double e = J[o].e_coll;
      ok = sum < e && lb_accept<MIX>(ua, e - sum, e - S.zpe, C.T.pr[J[o].pr].q);
    }
    const unsigned long long won = __ballot(ok);
    const unsigned long long mine = (won >> (rank << sh)) & (G < 64u ? (1ull << G) - 1ull : ~0ull);
    const uint32_t hit = mine ? (uint32_t)__ffsll((long long)mine) - 1u : G;
    const uint32_t from = ((rank << sh) + hit) & 63u;
    const double won_sum = __shfl(sum, (int)from);
    wave_sync();
    if (job) {
      if (trials + hit >= kMaxTrials) {
        // (the serial loop stops after trial kMaxTrials unless that one is accepted)
        trials = (uint32_t)kMaxTrials;
        capped = true;
        job = false;
      } else if (hit < G) {
        trials += hit + 1u;
        const uint16_t *cand = C.scr + mm * C.block + first_lane + from;
        for (uint32_t m = 0; m < nm; ++m) lv[m * stride] = cand[m * C.block];
        e_tr = e_coll - won_sum;
        job = false;
      } else {
        trials += G;
        J[C.lane].pos += G * (nm + 1u) * (MIX ? 1u : 2u);
        if (trials >= kMaxTrials) {
          capped = true;
          job = false;
        }
      }
      if (!job) rng.skip(trials * (nm + 1u));
    }
    wave_sync();
    pend = __ballot(job);
  }
  return trials;
}

// isotropic unit vector (Marsaglia 1972)
template <bool MIX>
__device__ __forceinline__ V3<Real<MIX>> unit_vector(RngT<MIX> &rng) {
  using R = Real<MIX>;
  R x, y, s;
  for (;;) {
    uint64_t w1, w2;
    rng.next_two(w1, w2);
    x = R(2) * (R)RngT<MIX>::exact_of(w1) - R(1);
    y = R(2) * (R)RngT<MIX>::exact_of(w2) - R(1);
    s = x * x + y * y;
    if (s < R(1)) break;
  }
  const R f = R(2) * sqrt(R(1) - s);
  return V3<R>{x * f, y * f, R(1) - R(2) * s};
}

// centre-of-mass velocity of a pair (the mixed form weighs with the mass
// fractions in fp32)
template <bool MIX>
__device__ __forceinline__ V3<Real<MIX>> com(const PairTab &P, V3<Real<MIX>> a, V3<Real<MIX>> b) {
  if constexpr (MIX) {
    const float fa = (float)P.wb, fb = (float)P.wa;  // m_a / M, m_b / M
    return V3<float>{fa * a.x + fb * b.x, fa * a.y + fb * b.y, fa * a.z + fb * b.z};
  } else {
    return Vec3{(P.m_a * a.x + P.m_b * b.x) / P.msum, (P.m_a * a.y + P.m_b * b.y) / P.msum,
                (P.m_a * a.z + P.m_b * b.z) / P.msum};
  }
}

// two bodies about the centre-of-mass velocity with relative energy e
template <bool MIX>
__device__ __forceinline__ void split(const PairTab &P, V3<Real<MIX>> vcm, double e, RngT<MIX> &rng,
                                      V3<Real<MIX>> &va, V3<Real<MIX>> &vb) {
  using R = Real<MIX>;
  R g;
  if constexpr (MIX)
    g = sqrtf((float)(2.0 * e) / (float)P.mr);
  else
    g = sqrt((2.0 * e) / P.mr);
  const V3<R> n = unit_vector<MIX>(rng);
  const R ga = (R)P.wa * g, gb = (R)P.wb * g;
  va = V3<R>{vcm.x + ga * n.x, vcm.y + ga * n.y, vcm.z + ga * n.z};
  vb = V3<R>{vcm.x - gb * n.x, vcm.y - gb * n.y, vcm.z - gb * n.z};
}

// kinetic energy 1/2 m |v|^2 in fp64
template <typename R>
__device__ __forceinline__ double kinetic(double m, V3<R> v) {
  const double x = v.x, y = v.y, z = v.z;
  return 0.5 * m * ((x * x + y * y) + z * z);
}

__device__ __forceinline__ void zero_levels(uint16_t *lv, uint32_t stride, uint32_t mm) {
  for (uint32_t m = 0; m < mm; ++m) lv[m * stride] = 0;
}

// One colliding pair held on chip: velocities and species in registers,
// quantum numbers in per-lane LDS slots (mode m of side x at lv_x[m * ls]).
// Rotational Larsen-Borgnakke share: the fraction f of E_tr + E_rot that the
// rotor keeps has density proportional to f^(zeta/2 - 1) (1 - f)^q:
// zeta = 2 by inversion, f = 1 - (1 - u)^(1/(q+1)); zeta = 3 by rejection
// from the uniform against the density over its value at the mode
// f* = 1/(1 + 2q).
template <bool MIX>
__device__ double rot_fraction(uint32_t zeta, double q, RngT<MIX> &rng) {
  if constexpr (MIX) {
    const float qf = (float)q;
    if (zeta == 2) return (double)(1.0f - pow_f(1.0f - rng.uniform_f(), 1.0f / (qf + 1.0f)));
    const float fs = 1.0f / (1.0f + 2.0f * qf);
    for (;;) {
      const float f = rng.uniform_f(), u2 = rng.uniform_f();
      if (u2 < pow_f(f / fs, 0.5f) * pow_f((1.0f - f) / (1.0f - fs), qf)) return (double)f;
    }
  } else {
    if (zeta == 2) return 1.0 - dpow(1.0 - rng.uniform(), 1.0 / (q + 1.0));
    const double fs = 1.0 / (1.0 + 2.0 * q);
    for (;;) {
      const double f = rng.uniform(), u2 = rng.uniform();
      if (u2 < dpow(f / fs, 0.5) * dpow((1.0 - f) / (1.0 - fs), q)) return f;
    }
  }
}

template <bool MIX>
struct PairLocal {
  uint32_t sp0, sp1;
  uint16_t *lv0, *lv1, *lvn;  // quantum numbers of p, q and the product
  uint32_t ls;
  double r0, r1, rn;  // rotational energies of p, q and the product (rotors only)
};

// What the collision decided for a pair: 0 scattering only, 1 dissociation,
// 2 exchange, 3 recombination; the reaction, its side (A of a dissociation
// or exchange, B of a recombination), the third body of a recombination (slot
// in its cell, species) and the translational energy left to the scattering.
struct Outcome {
  int kind, rx;
  uint32_t side, m, sp_m;
  double et;
};

__device__ __forceinline__ double vib_local(const Tab &T, uint32_t sp, const uint16_t *lv, uint32_t ls) {
  return vib_energy(T.sp[sp], T.lev, lv, ls);
}

struct Channel {
  int32_t rx, side, mode;
};

// Channel enumeration of one pair (dissociation channels of p then q, then
// exchange channels of p then q, registration order). Pass 0 draws the
// steric numbers, counts the open channels and sums their excess energy;
// pass 1 repeats the same arithmetic to find the channel that holds target.
struct ChannelScan {
  uint32_t nch;
  double total;
  Channel first, last, pick;
  bool found;
};

template <bool MIX, bool EX>
__device__ __forceinline__ void scan_channels(const Tab &T, uint32_t sp0, uint32_t sp1, double ev0, double ev1,
                                              const uint16_t *lv0, const uint16_t *lv1, uint32_t ls, double e_tr,
                                              double rot0, double rot1, RngT<MIX> &rng, uint64_t &steric_ok,
                                              int pass, double target, ChannelScan &S) {
  double cum = 0.0;
  uint32_t seen = 0, ex_i = 0;
  for (uint32_t kind = 0; kind < 2; ++kind) {
    for (uint32_t side = 0; side < 2; ++side) {
      const uint32_t A = side ? sp1 : sp0, B = side ? sp0 : sp1;
      const double evA = side ? ev1 : ev0, evB = side ? ev0 : ev1;
      const uint16_t *lA = side ? lv1 : lv0;
      const SpeciesTab &SA = T.sp[A];
      for (uint32_t r = 0; r < T.nr; ++r) {
        const ReactionTab &R = T.rx[r];
        if (kind == 0) {
          if (R.kind != HCAO_RX_DISSOCIATION || (uint32_t)R.a != A) continue;
          const uint32_t nst = SA.n_modes - SA.n_bend;
          for (uint32_t j = 0; j < nst; ++j) {
            if (!((R.mask >> j) & 1ull)) continue;
            const uint32_t m = SA.n_bend + j;
            // Eq. Ecoll-diss: E_tr (+ gamma E_rot,A) + E_vib,A - sum ZPE(A, B, C) + E_A,j(0)
            const double etg = EX ? e_tr + R.gamma_rot * (side ? rot1 : rot0) : e_tr;
            const double ecoll = ((etg + evA) - R.zsum) + T.lev[SA.lev_off[m]];
            const double eex = ecoll - SA.kt[m];
            const double pool = (etg + evA) - R.dh;
            const double left = (pool - T.sp[R.c].zpe) - T.sp[R.d].zpe;
            if (eex > 0.0 && left > 0.0 && seen < (uint32_t)kMaxChannels) {
              const Channel ch{(int32_t)r, (int32_t)side, (int32_t)m};
              ++seen;
              if (pass == 0) {
                if (seen == 1) S.first = ch;
                S.last = ch;
                S.total = S.total + eex;
              } else if (!S.found) {
                cum = cum + eex;
                if (target < cum) {
                  S.pick = ch;
                  S.found = true;
                }
              }
            }
          }
        } else {
          if (R.kind != HCAO_RX_EXCHANGE || (uint32_t)R.a != A || (uint32_t)R.b != B) continue;
          bool st_ok;
          if (pass == 0) {
            st_ok = (double)draw<MIX>(rng) < R.steric;
            if (st_ok && ex_i < 64) steric_ok |= (1ull << ex_i);
          } else {
            st_ok = ex_i < 64 ? ((steric_ok >> ex_i) & 1ull) != 0 : false;
          }
          ++ex_i;
          // Eq. Ecoll-exch: E_tr (+ gamma E_rot,A) + sum_j alpha_j E_vib,A,j
          const double etg = EX ? e_tr + R.gamma_rot * (side ? rot1 : rot0) : e_tr;
          double ecoll = etg;
          for (uint32_t m = 0; m < SA.n_modes; ++m)
            ecoll = ecoll + R.alpha[m] * mode_energy(SA, T.lev, m, lA[m * ls]);
          const double eex = ecoll - R.ea;
          const double pool = ((etg + evA) + evB) - R.dh;
          const double left = (pool - T.sp[R.c].zpe) - T.sp[R.d].zpe;
          if (st_ok && eex > 0.0 && left > 0.0 && seen < (uint32_t)kMaxChannels) {
            const Channel ch{(int32_t)r, (int32_t)side, -1};
            ++seen;
            if (pass == 0) {
              if (seen == 1) S.first = ch;
              S.last = ch;
              S.total = S.total + eex;
            } else if (!S.found) {
              cum = cum + eex;
              if (target < cum) {
                S.pick = ch;
                S.found = true;
              }
            }
          }
        }
      }
    }
  }
  if (pass == 0) S.nch = seen;
}

// Sums of m, m v_x, m v_y, m v_z and m |v|^2 over a cell's particles by one
// wave: lane t sums particles t, t + 64, t + 128, ... in slot order (loads
// of four blocks issued together), then a halving tree (lane t takes lane
// t + s for s = 32, ..., 1) combines the 64 partial sums; lane 0 returns
// them (every lane of the wave takes part). The running sums of the cell
// temperature start from these.
template <bool MIX>
__device__ void cell_sums(const State &st, const SpeciesTab *spt, uint64_t base, uint32_t n, uint32_t lane,
                          double out[5]) {
  constexpr int U = 4;
  double x0 = 0.0, x1 = 0.0, x2 = 0.0, x3 = 0.0, x4 = 0.0;
  for (uint32_t b0 = 0; b0 < n; b0 += 64 * U) {
    double m[U], vx[U], vy[U], vz[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t i = b0 + 64 * u + lane;
      m[u] = 0.0;
      vx[u] = vy[u] = vz[u] = 0.0;
      if (i < n) {
        const uint64_t g = base + i;
        const BodyOf<Real<MIX>> b = ldb<MIX>(st, g);
        m[u] = spt[b.sp].mass;
        vx[u] = b.v.x;
        vy[u] = b.v.y;
        vz[u] = b.v.z;
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (b0 + 64 * u + lane < n) {
        x0 = x0 + m[u];
        x1 = x1 + m[u] * vx[u];
        x2 = x2 + m[u] * vy[u];
        x3 = x3 + m[u] * vz[u];
        x4 = x4 + m[u] * ((vx[u] * vx[u] + vy[u] * vy[u]) + vz[u] * vz[u]);
      }
    }
  }
  double x[5] = {x0, x1, x2, x3, x4};
  tree_sum(x);
  for (int q = 0; q < 5; ++q) out[q] = x[q];
}

// adds one particle's terms m, m v, m |v|^2 to acc (in that order)
template <typename R>
__device__ __forceinline__ void add_terms(double acc[5], double m, V3<R> v) {
  const double x = v.x, y = v.y, z = v.z;
  acc[0] = acc[0] + m;
  acc[1] = acc[1] + m * x;
  acc[2] = acc[2] + m * y;
  acc[3] = acc[3] + m * z;
  acc[4] = acc[4] + m * ((x * x + y * y) + z * z);
}

// ---------------------------------------------------------------------------
// the collision step: one workgroup per group of consecutive cells
// ---------------------------------------------------------------------------
// Per-cell state kept in LDS across the steps of a launch (base .. weight)
// and per-step quantities (ncand .. perm).
struct CellHdr {
  uint64_t base;
  uint32_t cell, n, cap, ncand, cstart, pad;
  double sgmax, rem, volume, weight;
  double rem_new, n_cell, rec_f;
  double defect;  // mixed form: energy the cell's particles lack
  double tsum[5];  // recombination: running sums m, m v, m |v|^2 of the cell's particles
  int32_t rec_i, pad2;
  unsigned long long sgbits, excess;
  Perm perm;
};

// Reaction decision of one accepted pair (velocities v0, v1; H its cell, k its
// index there, e_tr its translational energy). The molecules to relax are then
// taken in draw order (at most two) through one sampler loop. Velocities are
// not changed here: scatter() reads them again, so that none is held in
// registers while the samplers run (held, they and what depends on them were
// spilled and reloaded around every sampler).
template <bool MIX, bool EX>
__device__ __forceinline__ Outcome decide(const Ctx &C, PairLocal<MIX> &P, const CellHdr &H, uint32_t k, const State &st,
                                          V3<Real<MIX>> v0, V3<Real<MIX>> v1, double e_tr0, RngT<MIX> &rng,
                                          const double *rec HCAO_ERR_PARAM) {
  using Rl = Real<MIX>;
  const Tab &T = C.T;
  const uint32_t ls = P.ls;
  const uint32_t sp0 = P.sp0, sp1 = P.sp1;
  const PairTab &PP = T.pair(sp0, sp1);
  Outcome O;
  O.kind = 0;
  O.rx = -1;
  O.side = 0;
  O.m = 0;
  O.sp_m = 0;
  double et = e_tr0;

  // (pairs that no reaction lists skip the decision; it would draw nothing)
  if (PP.react) {
    const double ev0 = vib_local(T, sp0, P.lv0, ls), ev1 = vib_local(T, sp1, P.lv1, ls);
    // --- recombination first: B + C (+M) -> A (+M) ---
    for (uint32_t r = 0; (PP.react & kReactRecomb) && r < T.nr && O.kind == 0; ++r) {
      const ReactionTab &R = T.rx[r];
      if (R.kind != HCAO_RX_RECOMBINATION) continue;
      uint32_t sb;
      if (sp0 == (uint32_t)R.a && sp1 == (uint32_t)R.b)
        sb = 0;
      else if (sp1 == (uint32_t)R.a && sp0 == (uint32_t)R.b)
        sb = 1;
      else
        continue;
      // 53 bits in both forms: the per-collision probability can be far below
      // the 2^-24 steps of the mixed form's single-word uniforms
      const double u = rng.uniform53();
      // third body of pair k: the particle at permutation index 2 N_cand + k
      if (!(2 * H.ncand + k < H.n)) {
        atomicAdd(&C.ctr[HCAO_CTR_SUPPRESSED], 1ull);
        continue;
      }
      PermReg perm;
      perm.load(H.perm);
      const uint32_t im = perm(2 * H.ncand + k);
      const uint64_t gm = HCAO_IDX(H.base + im, st.n_slots, err);
      const BodyOf<Rl> third = ldb<MIX>(st, gm);
      const uint32_t sp_m = third.sp;
      const double *tab = rec + R.rec_off + (size_t)sp_m * T.rec_nt;
      double prob;
      if (H.rec_i == -1)
        prob = tab[0];
      else if (H.rec_i == -2)
        prob = tab[T.rec_nt - 1];
      else
        prob = tab[H.rec_i] + H.rec_f * (tab[H.rec_i + 1] - tab[H.rec_i]);
      prob = prob * H.n_cell;
      if (prob > 1.0) prob = 1.0;
      if (!(u < prob)) continue;
      const V3<Rl> c3 = com<MIX>(T.pair(R.a, R.b), sb ? v1 : v0, sb ? v0 : v1);
      const V3<Rl> vm = third.v;
      const double gx = (double)c3.x - (double)vm.x, gy = (double)c3.y - (double)vm.y,
                   gz = (double)c3.z - (double)vm.z;
      const double e_am = T.pair(R.c, sp_m).hm * ((gx * gx + gy * gy) + gz * gz);
      double pool = (((e_am + e_tr0) + (sb ? ev1 : ev0)) + (sb ? ev0 : ev1)) - R.dh;
      double rsum = 0.0;
      if constexpr (EX) {
        // B's and C's rotation: kept by A's rotor, else pooled
        rsum = (sb ? P.r1 : P.r0) + (sb ? P.r0 : P.r1);
        if (T.sp[R.c].zeta_rot == 0) pool = pool + rsum;
      }
      const double e_left = pool - T.sp[R.c].zpe;
      if (!(e_left > 0.0)) {
        atomicAdd(&C.ctr[HCAO_CTR_SUPPRESSED], 1ull);
        continue;
      }
      O.kind = 3;
      O.rx = (int)r;
      O.side = sb;
      O.m = im;
      O.sp_m = sp_m;
      et = e_left;
      if constexpr (EX) {
        const double ra = T.sp[R.c].zeta_rot > 0 ? rsum : 0.0;
        P.r0 = sb ? 0.0 : ra;
        P.r1 = sb ? ra : 0.0;
      }
    }

    // --- dissociation and exchange channels, competition by excess energy ---
    // A pair none of whose channels can open skips the scan (its steric draws
    // are passed over): the bounds are tested with a margin far above the
    // rounding of the scan's own sums, so only pairs that certainly stay shut
    // skip it and the result is the scan's.
    bool may_open = false;
    if (O.kind == 0) {
      const PairBound &B = PP.bound;
      for (uint32_t sd = 0; sd < 2; ++sd) {
        const double ev = sd ? ev1 : ev0;
        const double eb = EX ? e_tr0 + (sd ? P.r1 : P.r0) : e_tr0;
        const double scale = 1e-9 * ((fabs(eb) + ev) + fabs(B.dis_c[sd] < 0.0 ? 0.0 : B.dis_c[sd]) + 1e-30);
        if ((eb + ev) + B.dis_c[sd] > -scale - 1e-9 * fabs(B.dis_c[sd])) may_open = true;
        if (B.ex_a[sd] >= 0.0 && (eb + B.ex_a[sd] * ev) - B.ex_e[sd] > -scale - 1e-9 * B.ex_e[sd]) may_open = true;
      }
      if (!may_open) rng.skip(B.n_steric);
    }
    if (may_open) {
      uint64_t steric_ok = 0;
      ChannelScan S;
      S.nch = 0;
      S.total = 0.0;
      S.found = false;
      S.first = S.last = S.pick = Channel{-1, 0, 0};
      scan_channels<MIX, EX>(T, sp0, sp1, ev0, ev1, P.lv0, P.lv1, ls, e_tr0, P.r0, P.r1, rng, steric_ok, 0, 0.0, S);
      if (S.nch > 0) {
        Channel pick = S.first;
        if (S.nch > 1) {
          const double target = (double)draw<MIX>(rng) * S.total;
          scan_channels<MIX, EX>(T, sp0, sp1, ev0, ev1, P.lv0, P.lv1, ls, e_tr0, P.r0, P.r1, rng, steric_ok, 1,
                                 target, S);
          pick = S.found ? S.pick : S.last;
        }
        const ReactionTab &R = T.rx[pick.rx];
        O.rx = pick.rx;
        O.side = (uint32_t)pick.side;
        const uint32_t side = O.side;
        const double eva = side ? ev1 : ev0, evb = side ? ev0 : ev1;
        const double ra = side ? P.r1 : P.r0, rb = side ? P.r0 : P.r1;
        const double grot = EX ? R.gamma_rot * ra : 0.0;
        const double etg = EX ? e_tr0 + grot : e_tr0;
        if (R.kind == HCAO_RX_DISSOCIATION) {
          O.kind = 1;
          et = (((etg + eva) - R.dh) - T.sp[R.c].zpe) - T.sp[R.d].zpe;
          if constexpr (EX) {
            // the uncoupled rotation stays with B's rotor, else is pooled
            double keep = ra - grot;
            if (T.sp[R.c].zeta_rot == 0) {
              et = et + keep;
              keep = 0.0;
            }
            if (side)
              P.r1 = keep;
            else
              P.r0 = keep;
            P.rn = 0.0;
          }
        } else {
          O.kind = 2;
          et = ((((etg + eva) + evb) - R.dh) - T.sp[R.c].zpe) - T.sp[R.d].zpe;
          if constexpr (EX) {
            // A's uncoupled rotation goes to C's rotor, B's to D's; else pooled
            double keep_c = ra - grot, keep_d = rb;
            if (T.sp[R.c].zeta_rot == 0) {
              et = et + keep_c;
              keep_c = 0.0;
            }
            if (T.sp[R.d].zeta_rot == 0) {
              et = et + keep_d;
              keep_d = 0.0;
            }
            P.r0 = side ? keep_d : keep_c;
            P.r1 = side ? keep_c : keep_d;
          }
        }
      }
    }
  }

  O.et = et;
  return O;
}

// Molecule j (0, 1) to relax after the decision, in draw order: its species,
// the partner that sets the exponent, its levels. A reaction's products start
// in the ground state: B takes A's slot in a dissociation and C is new, C and
// D take A's and B's in an exchange, A takes B's in a recombination (one
// molecule only).
template <bool MIX>
__device__ __forceinline__ void relax_job(const Tab &T, const PairLocal<MIX> &P, const Outcome &O, uint32_t j,
                                          uint32_t &sp, uint32_t &partner, uint16_t *&lv) {
  // (by value: a choice among members would put the whole struct into scratch)
  const uint32_t sp0 = P.sp0, sp1 = P.sp1;
  uint16_t *const lv0 = P.lv0, *const lv1 = P.lv1, *const lvn = P.lvn;
  if (O.kind == 0) {
    sp = j ? sp1 : sp0;
    partner = j ? sp0 : sp1;
    lv = j ? lv1 : lv0;
    return;
  }
  const ReactionTab &RX = T.rx[O.rx];
  const uint32_t c = (uint32_t)RX.c, d = (uint32_t)RX.d, sp_m = O.sp_m;
  const bool b = (O.side != 0) != (j != 0);
  lv = O.kind == 1 && j ? lvn : (b ? lv1 : lv0);
  sp = j ? d : c;
  partner = O.kind == 1 ? (O.side ? sp0 : sp1) : (O.kind == 2 ? (j ? c : d) : sp_m);
  zero_levels(lv, P.ls, T.mm);
}

// rotational relaxation of each rotor of a non-reactive pair in turn
template <bool MIX>
__device__ __forceinline__ void relax_rotors(const Tab &T, PairLocal<MIX> &P, double &et, RngT<MIX> &rng) {
  const double q = T.pair(P.sp0, P.sp1).q;
  for (uint32_t x = 0; x < 2; ++x) {
    const uint32_t sp0 = P.sp0, sp1 = P.sp1;
    const double r0 = P.r0, r1 = P.r1;
    const SpeciesTab &S = T.sp[x ? sp1 : sp0];
    if (S.zeta_rot == 0) continue;
    const double u = (double)draw<MIX>(rng);
    if (!(u < S.p_rot)) continue;
    const double ec = et + (x ? r1 : r0);
    const double er = rot_fraction<MIX>(S.zeta_rot, q, rng) * ec;
    if (x)
      P.r1 = er;
    else
      P.r0 = er;
    et = ec - er;
  }
}

// Scattering and reaction application: the outgoing velocities and species
// of the pair, the third body and the product. v0, v1 (and vm) are the
// velocities before the collision.
template <bool MIX>
struct Scattered {
  V3<Real<MIX>> v0, v1, vm, vn;
  uint32_t sp0, sp1;
  bool dead0, dead1;
};
template <bool MIX, bool EX>
__device__ __forceinline__ Scattered<MIX> scatter(const Ctx &C, const Outcome &O, uint32_t sp0, uint32_t sp1,
                                                  V3<Real<MIX>> v0, V3<Real<MIX>> v1, V3<Real<MIX>> vm,
                                                  RngT<MIX> &rng) {
  using Rl = Real<MIX>;
  const Tab &T = C.T;
  Scattered<MIX> F;
  F.sp0 = sp0;
  F.sp1 = sp1;
  F.dead0 = F.dead1 = false;
  F.vm = vm;
  F.vn = V3<Rl>{Rl(0), Rl(0), Rl(0)};
  const PairTab *t1 = &T.pair(sp0, sp1);
  V3<Rl> cm;
  double e1 = O.et, e2 = 0.0;
  if (O.kind == 0) {
    cm = com<MIX>(*t1, v0, v1);
  } else {
    const ReactionTab &RX = T.rx[O.rx];
    const uint32_t side = O.side;
    if (O.kind == 1) {
      // share of the translational energy in the B-C motion: density
      // proportional to sqrt(beta (1 - beta)), by rejection
      Rl beta;
      for (;;) {
        const Rl u1 = draw<MIX>(rng), u2 = draw<MIX>(rng);
        if (u2 * Rl(0.5) < sqrt(u1 * (Rl(1) - u1))) {
          beta = u1;
          break;
        }
      }
      e2 = (double)beta * O.et;
      e1 = O.et - e2;
    }
    const V3<Rl> va0 = side ? v1 : v0, vb0 = side ? v0 : v1;
    const uint32_t spA = side ? sp1 : sp0, spB = side ? sp0 : sp1;
    if (O.kind == 3) {
      t1 = &T.pair(RX.c, O.sp_m);
      cm = com<MIX>(*t1, com<MIX>(T.pair(RX.a, RX.b), va0, vb0), vm);
    } else {
      cm = com<MIX>(T.pair(spA, spB), va0, vb0);
      t1 = O.kind == 1 ? &T.pair(spA, spB) : &T.pair(RX.c, RX.d);
    }
  }
  V3<Rl> x1, y1;
  split<MIX>(*t1, cm, e1, rng, x1, y1);
  F.v0 = x1;
  F.v1 = y1;
  if (O.kind != 0) {
    const ReactionTab &RX = T.rx[O.rx];
    const uint32_t side = O.side;
    if (O.kind == 1) {
      V3<Rl> x2, y2;
      split<MIX>(T.pair(RX.c, RX.d), x1, e2, rng, x2, y2);
      x1 = x2;
      F.vn = y2;
      atomicAdd(&C.ctr[HCAO_CTR_BIRTHS], 1ull);
    }
    if (O.kind == 3) {
      F.vm = y1;
      y1 = side ? v0 : v1;  // C's velocity is not kept
      atomicAdd(&C.ctr[HCAO_CTR_DEATHS], 1ull);
    }
    const uint32_t new_b = O.kind == 2 ? (uint32_t)RX.d : (side ? sp0 : sp1);
    F.v0 = side ? y1 : x1;
    F.v1 = side ? x1 : y1;
    F.sp0 = side ? new_b : (uint32_t)RX.c;
    F.sp1 = side ? (uint32_t)RX.c : new_b;
    F.dead0 = O.kind == 3 && side;
    F.dead1 = O.kind == 3 && !side;
    atomicAdd(&C.ctr[HCAO_CTR_REACTION0 + O.rx], 1ull);
  }
  return F;
}

// the cell of flattened candidate j: the last cell whose range starts at or before j
__device__ __forceinline__ uint32_t group_cell(const CellHdr *hdr, uint32_t ncell, uint32_t j) {
  uint32_t lo = 0, hi = ncell;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (hdr[mid].cstart <= j)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

// a candidate's per-pair records: the changes of its cell's running sums and
// the mixed form's energy defect (all 0 if it was not accepted)
struct Records {
  double y0, y1, y2, y3, y4, y5;
};

// Phase C lists the step's products (candidate of each) in LDS while they are
// few; with more of them it looks at every candidate's flag instead.
constexpr uint32_t kBornList = 128;
// A cell with more candidates than this has its per-pair records reduced by
// all waves of the workgroup, chunk by chunk, before one wave adds up the
// chunks (a wave takes a microsecond per chunk: a cell of 100,000 particles
// has 600, which kept the other waves waiting for half of the step; at 512
// candidates the extra barrier costs what eight chunks do).
constexpr uint32_t kBigCell = 512;

// an accepted pair's velocities, handed from phase A to phase B
template <typename R>
struct PairVel {
  V3<R> p, q;
};

// Phase 0 stages the tables in LDS and computes each cell's NTC candidate
// count and permutation keys (and, with recombination, the cell
// temperature). Phase A tests every candidate pair of the group (lane per
// candidate) and appends the accepted ones to a work list. Phase B gives
// every lane one accepted pair: the pair's state is gathered once into
// registers and per-lane LDS, the reaction / relaxation / scattering runs
// on chip, and the result is written back. Phase C removes recombined
// particles, places the products of each cell in pair order and writes the
// per-cell state. Pairs are disjoint and every draw is keyed by (cell,
// pair), so the order in which lanes take work does not change the result.
//
// The mixed form (MIX) keeps fp32 velocities, tests VHS acceptance and
// samples levels in fp32, and keeps energies, thresholds and accumulators in
// fp64. Each pair records the fp64 energy its fp32 velocities lost or gained
// (the audit of its particles before and after); the cell's sum, reduced in
// pair order, is owed to the cell and joins the translational energy of the
// cell's pair 0 in the next step in which that pair collides.
//
// What bounds it: vector arithmetic, where there are cells enough to fill the
// chip (the pairs' samplers, then the permutation and the generator: about
// 19,000 vector instructions per seven cells of 256 particles and step; in the
// mixed form the issue slots are 93% busy). It was bound by cache lines before: 262,144 cells
// of 256, 50 steps, 93 ms mixed and 101 fp64, now 63 and 73. Velocity and
// species are therefore one record; an accepted pair's velocities go from
// phase A to B, and from B's decision to its scattering, through a dense list
// that stays in cache; per-pair records are dense by entry. Four waves per SIMD
// (128 registers; three with the exact sampler, which needs 136) came with
// that: alone they gained nothing. Few cells: bound by the chain of a step's
// phases, so groups get smaller and workgroups wider (choose_shape). Large
// cells (4,096 reservoirs of 1,000 to 100,000 particles, 25 steps: 101 to 45
// ms): the candidates' gathers land on scattered lines.
template <int BLOCK, bool MIX, int EX>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(EX >= 2 ? 3 : 4))) void k_step(StepArgs A) {
  using R = Real<MIX>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ uint32_t s_nwork, s_total, s_next;
  __shared__ uint32_t s_bin[256];
  __shared__ WorkRound s_rounds[kLdsRounds];
  __shared__ uint32_t s_nborn, s_born[kBornList];
  __shared__ uint32_t s_big;
  const uint32_t tid = threadIdx.x;
  // the wave index is the same on every lane of a wave: held in a scalar
  // register, so that per-wave loops (one wave per cell) and what they
  // address stay scalar
  const uint32_t lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const unsigned long long lt = lane ? ((1ull << lane) - 1ull) : 0ull;
  const Tables *GT = A.tab;
  const uint32_t ns = GT->n_species, nr = GT->n_reactions, mm = GT->max_modes, nl = GT->n_levels;
  const uint32_t nctr = 8 + nr;
  const uint32_t c0 = A.grp[2 * blockIdx.x], c1 = A.grp[2 * blockIdx.x + 1];
  const uint32_t ncell = c1 - c0;
  const uint64_t wbase = A.grp_work[3 * blockIdx.x];
#ifdef HCAO_PHASE_CLOCKS
  uint64_t clk_acc[kPhases] = {};
  uint64_t clk_t = clock64();
  __shared__ unsigned long long s_wclk[5];  // collision sub-phases, summed over the workgroup's waves
  if (tid < 5) s_wclk[tid] = 0ull;
#endif

  // ---- LDS carve-up ----
  unsigned char *q = smem;
  SpeciesTab *l_sp = reinterpret_cast<SpeciesTab *>(q);
  q += sizeof(SpeciesTab) * ns;
  PairTab *l_pr = reinterpret_cast<PairTab *>(q);
  q += sizeof(PairTab) * ns * ns;
  ReactionTab *l_rx = reinterpret_cast<ReactionTab *>(q);
  q += sizeof(ReactionTab) * nr;
  double *l_lev = reinterpret_cast<double *>(q);
  q += sizeof(double) * (nl ? nl : 1);  // bends read level 0 without using it
  CellHdr *hdr = reinterpret_cast<CellHdr *>(q);
  q += sizeof(CellHdr) * ncell;
  unsigned long long *l_ctr = reinterpret_cast<unsigned long long *>(q);
  q += sizeof(unsigned long long) * nctr * ncell * 2;  // per-step counters, then totals
  uint16_t *scr = reinterpret_cast<uint16_t *>(q);  // [2 mm][BLOCK] sampler scratch (joint and exact samplers)
  uint16_t *plv = scr + (GT->sampler_scratch ? (size_t)2 * mm * BLOCK : 0);  // [3 mm][BLOCK] pair levels

  unsigned long long *l_tot = l_ctr + (size_t)nctr * ncell;  // counters summed over the launch's steps

  // ---- once per launch: tables and the persistent cell state ----
  {
    const uint64_t *src = reinterpret_cast<const uint64_t *>(GT->sp);
    uint64_t *dst = reinterpret_cast<uint64_t *>(l_sp);
    for (uint32_t i = tid; i < ns * sizeof(SpeciesTab) / 8; i += BLOCK) dst[i] = src[i];
    for (uint32_t i = tid; i < ns * ns; i += BLOCK) l_pr[i] = GT->pr[i / ns][i % ns];
    src = reinterpret_cast<const uint64_t *>(GT->rx);
    dst = reinterpret_cast<uint64_t *>(l_rx);
    for (uint32_t i = tid; i < nr * sizeof(ReactionTab) / 8; i += BLOCK) dst[i] = src[i];
    for (uint32_t i = tid; i < nl; i += BLOCK) l_lev[i] = A.lev[i];
    for (uint32_t i = tid; i < nctr * ncell; i += BLOCK) l_tot[i] = 0ull;
  }
  for (uint32_t g = tid; g < ncell; g += BLOCK) {
    CellHdr &H = hdr[g];
    const uint32_t c = c0 + g;
    H.base = A.cells.off[c];
    H.cell = c;
    H.n = A.cells.cnt[c];
    H.cap = A.cells.cap[c];
    H.sgmax = A.cells.sgmax[c];
    H.rem = A.cells.rem[c];
    H.volume = A.cells.volume[c];
    H.weight = A.cells.weight[c];
    H.defect = MIX ? A.cells.defect[c] : 0.0;
    if (A.cells.tsum)
      for (int q = 0; q < 5; ++q) H.tsum[q] = A.cells.tsum[(size_t)q * A.cells.n_cells + c];
  }
  if constexpr (EX >= 1) {
    // spatial mode: the particles were re-binned since the last step, so the
    // running sums start afresh from them (one wave per cell; masses from
    // the species table in LDS)
    if (A.cells.tsum && A.st.px) {
      __syncthreads();
      for (uint32_t g = wave; g < ncell; g += BLOCK / 64) {
        double sums[5];
        cell_sums<MIX>(A.st, l_sp, hdr[g].base, hdr[g].n, lane, sums);
        if (lane == 0)
          for (int q = 0; q < 5; ++q) hdr[g].tsum[q] = sums[q];
      }
    }
  }
  const Tab T{l_sp, l_pr, l_rx, l_lev, A.beta, ns, nr, mm, GT->rec_nt};
  const uint32_t wcap = (uint32_t)(A.grp_work[3 * blockIdx.x + 1] - wbase);
  uint32_t *work_in = A.work + (size_t)kWorkWords * wbase;  // accepted pairs as found
  uint32_t *work = work_in + (size_t)kWorkFound * wcap;       // their indices sorted by key
  uint8_t *bflag = A.bflag + wbase;
  PairVel<R> *pv = reinterpret_cast<PairVel<R> *>(A.pv) + wbase;
  // the rounds stay in LDS where they fit (a group of up to 4,096 candidates)
  WorkRound *rounds = wcap <= 64 * kLdsRounds ? s_rounds : A.rounds + A.grp_work[3 * blockIdx.x + 2];
  double *wdef = MIX ? A.wdef + wbase : nullptr;
  __syncthreads();
  HCAO_PHASE_MARK(kPhaseLoad);

  // the joint sampler's slots lie after the pair levels
  const bool any_joint = (GT->sampler_scratch & 2u) != 0;
  JointJob *jobs = reinterpret_cast<JointJob *>(reinterpret_cast<unsigned char *>(plv) +
                                                (((size_t)6 * mm * BLOCK + 7) & ~(size_t)7));
  const uint32_t step0 = A.step_dev ? *A.step_dev + A.step : A.step;
  for (uint32_t si = 0; si < A.n_steps; ++si) {
  const uint32_t step = step0 + si;

  // ---- phase 0: candidate counts and permutation keys of the step ----
  for (uint32_t i = tid; i < nctr * ncell; i += BLOCK) l_ctr[i] = 0ull;
  for (uint32_t i = tid; i < 256; i += BLOCK) s_bin[i] = 0;  // the work-list sort's bins, counted in phase A
  for (uint32_t g = tid; g < ncell; g += BLOCK) {
    CellHdr &H = hdr[g];
    const uint32_t n = H.n;
    // NTC candidate count: floor(1/2 N (N-1) F_N (sigma g)_max dt / V + remainder)
    const double x = 0.5 * (double)n * (double)(n - (n > 0 ? 1u : 0u)) * H.weight * H.sgmax * A.dt / H.volume + H.rem;
    const double fl = floor(x);
    uint64_t ncand = (uint64_t)fl;
    uint64_t excess = 0;
    if (ncand > n / 2) {
      excess = ncand - n / 2;
      ncand = n / 2;
    }
    H.ncand = (uint32_t)ncand;
    H.rem_new = x - fl;
    H.n_cell = (double)n * H.weight / H.volume;
    H.rec_i = -1;
    H.rec_f = 0.0;
    H.sgbits = 0ull;
    H.excess = excess;
    if (ncand > 0) make_perm(H.perm, n, A.seed, H.cell, step);
    if (GT->has_recomb && n >= 2) {
      // cell temperature from the running sums and its recombination-table coordinate
      const double p2 = (H.tsum[1] * H.tsum[1] + H.tsum[2] * H.tsum[2]) + H.tsum[3] * H.tsum[3];
      const double t = (H.tsum[4] - p2 / H.tsum[0]) / (3.0 * kBoltz * (double)n);
      if (t > 0.0) {
        const double u = (dlog(t) - GT->rec_l0) * GT->rec_inv_step;
        if (!(u > 0.0)) {
          H.rec_i = -1;
        } else if (!(u < (double)(GT->rec_nt - 1))) {
          H.rec_i = -2;
        } else {
          const double fi = floor(u);
          H.rec_i = (int32_t)fi;
          H.rec_f = u - fi;
        }
      }
    }
  }
  __syncthreads();
  HCAO_PHASE_MARK(kPhaseNtc);
  if (tid == 0) {
    uint32_t acc = 0, most = 0;
    for (uint32_t g = 0; g < ncell; ++g) {
      const uint32_t n = hdr[g].ncand;
      hdr[g].cstart = acc;
      acc += n;
      most = n > most ? n : most;
    }
    s_total = acc;
    s_nborn = 0;
    s_big = most > kBigCell ? 1u : 0u;
    s_nwork = 0;
    s_next = 0;
  }
  __syncthreads();
  HCAO_PHASE_MARK(kPhaseTemperature);
  const uint32_t total = s_total;

  // ---- phase A: candidate pairs, VHS acceptance ----
  // Accepted pairs are appended to a work list (one LDS atomic per wave)
  // with a key that orders them by the sampler work they carry: the mode
  // counts of p and of q. A counting sort by that key (largest first) then
  // gives each wave of phase B pairs whose relaxations have the same shape.
  for (uint32_t j0 = 0; j0 < total; j0 += BLOCK) {
    const uint32_t j = j0 + tid;
    bool acc = false;
    uint32_t pj = 0, qj = 0, packed = 0, rw1 = 0, rw2 = 0, rw3 = 0;
    PairVel<R> vel{};
    if (j < total) {
      const uint32_t g = group_cell(hdr, ncell, j);
      const CellHdr &H = hdr[g];
      const uint32_t k = j - H.cstart;
      PermReg perm;
      perm.load(H.perm);
      uint32_t p, qq;
      perm.pair(k, p, qq);
      pj = p;
      qj = qq;
      const uint64_t gp = HCAO_IDX(H.base + p, A.st.n_slots, A.err), gq = HCAO_IDX(H.base + qq, A.st.n_slots, A.err);
      const BodyOf<R> bp = ldb<MIX>(A.st, gp), bq = ldb<MIX>(A.st, gq);
      const V3<R> vp = bp.v, vq = bq.v;
      vel = PairVel<R>{vp, vq};
      const R dx = vp.x - vq.x, dy = vp.y - vq.y, dz = vp.z - vq.z;
      const R g2 = (dx * dx + dy * dy) + dz * dz;
      const uint32_t a = bp.sp, b = bq.sp;
      const PairTab &PP = T.pair(a, b);
      RngT<MIX> rng;
      rng.open(A.seed, k, H.cell, step);
      const R ua = draw<MIX>(rng);
      // the rest of the pair stream's first block, handed to the collision pass
      rw1 = rng.w1;
      rw2 = rng.w2;
      rw3 = rng.w3;
      // VHS acceptance ua < sigma g / (sigma g)_max with sigma g = C (g^2)^(1-w).
      if constexpr (MIX) {
        const float sg = (g2 > 0.0f) ? (float)PP.csg * pow_f(g2, (float)PP.esg) : 0.0f;
        const unsigned long long sb = (unsigned long long)__double_as_longlong((double)sg);
        if ((double)sg > H.sgmax && sb > hdr[g].sgbits) atomicMax(&hdr[g].sgbits, sb);
        acc = ua < sg / (float)H.sgmax;
      } else {
        // The exact sigma g is needed for the decision only near the filter
        // band, and for the (sigma g)_max update only when it may exceed the
        // cell's current value (the update keeps the larger of the two).
        const double est = (g2 > 0.0) ? PP.csg * pow_estimate(g2, PP.esg) : 0.0;
        const double ratio = est / H.sgmax;
        const bool need_max = est >= H.sgmax * (1.0 - 2.0 * kFilter);
        if (ua < ratio * (1.0 - kFilter) && !need_max) {
          acc = true;
        } else if (ua > ratio * (1.0 + kFilter) && !need_max) {
          acc = false;
        } else {
          const double sg = (g2 > 0.0) ? PP.csg * dpow(g2, PP.esg) : 0.0;
          const unsigned long long sb = (unsigned long long)__double_as_longlong(sg);
          if (sb > hdr[g].sgbits) atomicMax(&hdr[g].sgbits, sb);
          acc = ua < sg / H.sgmax;
        }
      }
      const uint32_t na = T.sp[a].n_modes < 15 ? T.sp[a].n_modes : 15;
      const uint32_t nb = T.sp[b].n_modes < 15 ? T.sp[b].n_modes : 15;
      const uint32_t key = 255u - (na * 16u + nb);
      packed = key | (g << kWorkCell) | (a << kWorkSp0) | (b << kWorkSp1);
      if (acc) atomicAdd(&s_bin[key], 1u);
    }
    const unsigned long long ma = __ballot(acc);
    uint32_t wb = 0;
    if (lane == 0 && ma) wb = atomicAdd(&s_nwork, (uint32_t)__popcll(ma));
    wb = __builtin_amdgcn_readfirstlane(wb);  // every lane is active here: lane 0's value
    const uint32_t jr = j0 + 64 * wave;  // the wave's first candidate
    if (lane == 0 && jr < total) rounds[HCAO_IDX(jr / 64, (wcap + 63) / 64, A.err)] = WorkRound{ma, wb, 0};
    if (acc) {
      const uint32_t f = (uint32_t)HCAO_IDX(wb + (uint32_t)__popcll(ma & lt), wcap, A.err);
      uint32_t *w = work_in + (size_t)kWorkFound * f;
      w[0] = j;
      w[1] = pj;
      w[2] = qj;
      w[3] = packed;
      w[4] = rw1;
      w[5] = rw2;
      w[6] = rw3;
      pv[f] = vel;
    }
  }
  __syncthreads();
  HCAO_PHASE_MARK(kPhaseAccept);

  // ---- counting sort of the work list by key ----
  // (the bins were counted as phase A appended the pairs)
  const uint32_t nwork = s_nwork;
  if (tid < 64) {
    // exclusive scan of the 256 bins, four per lane
    const uint32_t b0 = s_bin[4 * lane], b1 = s_bin[4 * lane + 1], b2 = s_bin[4 * lane + 2], b3 = s_bin[4 * lane + 3];
    const uint32_t sum = ((b0 + b1) + b2) + b3;
    uint32_t inc = sum;
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t o = __shfl_up(inc, d);
      if ((int)lane >= d) inc += o;
    }
    const uint32_t ex = inc - sum;
    s_bin[4 * lane] = ex;
    s_bin[4 * lane + 1] = ex + b0;
    s_bin[4 * lane + 2] = ex + b0 + b1;
    s_bin[4 * lane + 3] = ex + b0 + b1 + b2;
  }
  __syncthreads();
  for (uint32_t i = tid; i < nwork; i += BLOCK) {
    const uint32_t *f = work_in + (size_t)kWorkFound * i;
    work[HCAO_IDX(atomicAdd(&s_bin[f[3] & 0xFFu], 1u), wcap, A.err)] = i;  // the entry itself stays where it was found
  }
  __syncthreads();
  HCAO_PHASE_MARK(kPhaseSort);

  // ---- phase B: one accepted pair per lane ----
  // Waves take 64 consecutive pairs of the sorted list at a time from a
  // shared counter, so that a wave that drew light pairs takes the next
  // block instead of waiting at the barrier for one that drew heavy ones.
  // (With the joint sampler, whose lanes share the work of fewer pairs, the
  // blocks are as even as the waves can take them.)
  uint32_t take = 64;
  if (any_joint) {
    const uint32_t per = (nwork + BLOCK / 64 - 1) / (BLOCK / 64), rounds_b = (per + 63) / 64;
    if (rounds_b) take = (per + rounds_b - 1) / rounds_b;
  }
  for (;;) {
    uint32_t c0 = 0;
    if (lane == 0) c0 = atomicAdd(&s_next, take);
    c0 = __builtin_amdgcn_readfirstlane(c0);  // every lane is active here: lane 0's value
    if (c0 >= nwork) break;
    const uint32_t i = c0 + lane;
    const bool act = lane < take && i < nwork;
#ifdef HCAO_PHASE_CLOCKS
    uint64_t wclk[5] = {0, 0, 0, 0, 0}, wclk_t = clock64();  // collision sub-phase clocks
    const bool lead = lane == (uint32_t)(__ffsll((long long)__ballot(1)) - 1);
#endif
    uint32_t at = 0;
    unsigned long long *ctr = l_ctr;
    PairLocal<MIX> P;
    P.ls = BLOCK;
    P.lv0 = plv + tid;
    P.lv1 = plv + (size_t)mm * BLOCK + tid;
    P.lvn = plv + (size_t)2 * mm * BLOCK + tid;
    P.sp0 = P.sp1 = 0;
    P.r0 = P.r1 = P.rn = 0.0;
    RngT<MIX> rng;
    rng.open(A.seed, 0, 0, step);
    Outcome O{0, -1, 0, 0, 0, 0.0};
    if (act) {
      at = (uint32_t)HCAO_IDX(work[i], wcap, A.err);
      const uint32_t *wi = work_in + (size_t)kWorkFound * at;
      const PairVel<R> vel = pv[at];
      const V3<R> v0 = vel.p, v1 = vel.q;
      const uint32_t packed = wi[3], g = (packed >> kWorkCell) & 63u;
      const CellHdr &H = hdr[g];
      const uint32_t k = wi[0] - H.cstart;
      const uint64_t gp = HCAO_IDX(H.base + wi[1], A.st.n_slots, A.err),
                     gq = HCAO_IDX(H.base + wi[2], A.st.n_slots, A.err);
      P.sp0 = (packed >> kWorkSp0) & 15u;
      P.sp1 = (packed >> kWorkSp1) & 15u;
      // quantum numbers of the species' own modes (the others are 0 in the state
      // and nothing reads them here)
      load_levels(A.st, gp, T.sp[P.sp0].n_modes, P.lv0, BLOCK);
      load_levels(A.st, gq, T.sp[P.sp1].n_modes, P.lv1, BLOCK);
      if constexpr (EX >= 2) {
        if (A.st.rot) {
          P.r0 = A.st.rot[gp];
          P.r1 = A.st.rot[gq];
        }
      }
      rng.open(A.seed, k, H.cell, step);
      // resume after the acceptance draw of phase A: its block's other words
      rng.block = 1;
      rng.w1 = wi[4];
      rng.w2 = wi[5];
      rng.w3 = wi[6];
      rng.used = MIX ? 1u : 2u;
      // |v_p - v_q|^2 in fp64 (exact differences of fp32 velocities in the mixed form)
      const double dx = (double)v0.x - (double)v1.x, dy = (double)v0.y - (double)v1.y,
                   dz = (double)v0.z - (double)v1.z;
      double e_tr = T.pair(P.sp0, P.sp1).hm * ((dx * dx + dy * dy) + dz * dz);
      // energy owed to the cell's particles by earlier rounding joins the
      // cell's pair 0 when the sum stays positive
      if constexpr (MIX)
        if (k == 0 && H.defect != 0.0 && e_tr + H.defect > 0.0) e_tr = e_tr + H.defect;
      ctr = l_ctr + (size_t)g * nctr;
      atomicAdd(&ctr[HCAO_CTR_COLLISIONS], 1ull);
      const Ctx C{T, ctr, scr, tid, BLOCK};
      HCAO_WAVE_MARK(wclk, kPhaseCollideGather);
      O = decide<MIX, (EX >= 2)>(C, P, H, k, A.st, v0, v1, e_tr, rng, A.rec HCAO_ERR_ARG(A.err));
    }
    HCAO_WAVE_MARK(wclk, kPhaseCollideDecide);
    // the molecules to relax: the joint sampler's together, each other one in
    // its own lane
    {
      const Ctx C{T, ctr, scr, tid, BLOCK};
      uint32_t tr = 0, nrel = 0, ncap = 0;
      for (uint32_t j = 0; j < 2; ++j) {
        bool job = act && (j == 0 || O.kind != 3), joint = false;
        uint32_t sj = 0, partner = 0;
        uint16_t *lv = P.lv0;
        if (job) {
          relax_job<MIX>(T, P, O, j, sj, partner, lv);
          const SpeciesTab &S = T.sp[sj];
          job = S.n_modes > 0;
          if (job && O.kind == 0) {
            const double u = (double)draw<MIX>(rng);
            job = u < S.p_vib;
            nrel += job ? 1u : 0u;
          }
          if (job) {
            joint = S.sampler == HCAO_SAMPLER_JOINT;
            if (!joint) {
              bool capped = false;
              const PairTab &PJ = T.pair(sj, partner);
              const uint32_t bo = PJ.beta_off;
              tr += relax<MIX, (EX >= 2)>(C, S, lv, BLOCK, O.et, PJ.q, T.beta + (bo == 0xFFFFFFFFu ? 0u : bo), rng,
                                          capped);
              ncap += capped ? 1u : 0u;
            }
          }
        }
        if (any_joint && __ballot(joint)) {
          bool capped;
          const uint32_t t = relax_joint<MIX>(C, jobs, joint, sj, partner, lv, BLOCK, O.et, rng, capped);
          tr += t;
          ncap += capped ? 1u : 0u;
        }
      }
      if (tr) atomicAdd(&ctr[HCAO_CTR_TRIALS], (unsigned long long)tr);
      if (nrel) atomicAdd(&ctr[HCAO_CTR_RELAX], (unsigned long long)nrel);
      if (ncap) atomicAdd(&ctr[HCAO_CTR_CAPPED], (unsigned long long)ncap);
    }
    HCAO_WAVE_MARK(wclk, kPhaseCollideRelax);
    if (act) {
    if constexpr (EX >= 2)
      if (O.kind == 0) relax_rotors<MIX>(T, P, O.et, rng);
    // the pair's entry and velocities are read again (the dense lists of the
    // step, still in cache) rather than kept in registers through the samplers
    renew(at);
    {
      const uint32_t *wi = work_in + (size_t)kWorkFound * at;
      const PairVel<R> vel = pv[at];
      const V3<R> v0 = vel.p, v1 = vel.q;
      const uint32_t j = wi[0], g = (wi[3] >> kWorkCell) & 63u;
      const CellHdr &H = hdr[g];
      const uint64_t gp = HCAO_IDX(H.base + wi[1], A.st.n_slots, A.err),
                     gq = HCAO_IDX(H.base + wi[2], A.st.n_slots, A.err),
                     gm = HCAO_IDX(H.base + O.m, A.st.n_slots, A.err);
      const bool recoil = O.kind == 3, born = O.kind == 1;
      V3<R> vm{R(0), R(0), R(0)};
      if (recoil) vm = ldb<MIX>(A.st, gm).v;
      const Ctx C{T, l_ctr + (size_t)g * nctr, scr, tid, BLOCK};
      const Scattered<MIX> F = scatter<MIX, (EX >= 2)>(C, O, P.sp0, P.sp1, v0, v1, vm, rng);
      HCAO_WAVE_MARK(wclk, kPhaseCollideScatter);
      const uint32_t nb_sp = born ? (uint32_t)T.rx[O.rx].d : 0u;
      const double m0 = T.sp[P.sp0].mass, m1 = T.sp[P.sp1].mass;
      if constexpr (MIX) {
        // Energy audit of the fp32 kinematics: the scattering intends the
        // kinetic energy of the total centre-of-mass motion plus the
        // translational energy handed to it (vibrational and formation energy
        // are bookkept in fp64 and cancel); the defect is the intended minus
        // the stored fp32 kinetic energy, less energy owed that joined here.
        double mt = m0 + m1;
        double px = m0 * (double)v0.x + m1 * (double)v1.x;
        double py = m0 * (double)v0.y + m1 * (double)v1.y;
        double pz = m0 * (double)v0.z + m1 * (double)v1.z;
        if (recoil) {
          const double mm3 = T.sp[O.sp_m].mass;
          mt = mt + mm3;
          px = px + mm3 * (double)vm.x;
          py = py + mm3 * (double)vm.y;
          pz = pz + mm3 * (double)vm.z;
        }
        const double ke_int = (0.5 * ((px * px + py * py) + pz * pz)) / mt + O.et;
        double ke_out = 0.0;
        if (!F.dead0) ke_out = ke_out + kinetic(T.sp[F.sp0].mass, F.v0);
        if (!F.dead1) ke_out = ke_out + kinetic(T.sp[F.sp1].mass, F.v1);
        if (born) ke_out = ke_out + kinetic(T.sp[nb_sp].mass, F.vn);
        if (recoil) ke_out = ke_out + kinetic(T.sp[O.sp_m].mass, F.vm);
        double fold_used = 0.0;
        if (j == H.cstart && H.defect != 0.0) {
          const double dx = (double)v0.x - (double)v1.x, dy = (double)v0.y - (double)v1.y,
                       dz = (double)v0.z - (double)v1.z;
          const double e_tr = T.pair(P.sp0, P.sp1).hm * ((dx * dx + dy * dy) + dz * dz);
          if (e_tr + H.defect > 0.0) fold_used = H.defect;
        }
        wdef[at] = (ke_int - ke_out) - fold_used;
      }
      if (A.tdelta) {
        // the pair's change of its cell's running sums: its particles after
        // (p, q, the recoiling third body, the product) minus before (p, q,
        // the third body if it took part)
        double before[5] = {0.0, 0.0, 0.0, 0.0, 0.0}, after[5] = {0.0, 0.0, 0.0, 0.0, 0.0};
        add_terms(before, m0, v0);
        add_terms(before, m1, v1);
        if (recoil) add_terms(before, T.sp[O.sp_m].mass, vm);
        if (!F.dead0) add_terms(after, T.sp[F.sp0].mass, F.v0);
        if (!F.dead1) add_terms(after, T.sp[F.sp1].mass, F.v1);
        if (recoil) add_terms(after, T.sp[O.sp_m].mass, F.vm);
        if (born) add_terms(after, T.sp[nb_sp].mass, F.vn);
        const uint64_t e = HCAO_IDX(wbase + at, A.tdelta_stride, A.err);
        for (int x = 0; x < 5; ++x) A.tdelta[(size_t)x * A.tdelta_stride + e] = after[x] - before[x];
      }
      stb<MIX>(A.st, gp, F.v0, F.dead0 ? kDead : F.sp0);
      stb<MIX>(A.st, gq, F.v1, F.dead1 ? kDead : F.sp1);
      // the new species' modes, and zeros over the modes only the old species had
      // (a removed particle's levels are not kept)
      const uint32_t nm0 = T.sp[P.sp0].n_modes, nm1 = T.sp[P.sp1].n_modes;
      if (!F.dead0) {
        const uint32_t nn = T.sp[F.sp0].n_modes;
        store_levels(A.st, gp, nn, nn > nm0 ? nn : nm0, P.lv0, BLOCK);
      }
      if (!F.dead1) {
        const uint32_t nn = T.sp[F.sp1].n_modes;
        store_levels(A.st, gq, nn, nn > nm1 ? nn : nm1, P.lv1, BLOCK);
      }
      if constexpr (EX >= 2) {
        if (A.st.rot) {
          A.st.rot[gp] = F.dead0 ? 0.0 : P.r0;
          A.st.rot[gq] = F.dead1 ? 0.0 : P.r1;
        }
      }
      if (recoil) stv<MIX>(A.st, gm, F.vm);
      if (born) {
        const uint64_t gb = HCAO_IDX(wbase + j, A.born.n_slots, A.err);
        stb<MIX>(A.born, gb, F.vn, nb_sp);
        store_levels(A.born, gb, mm, A.born.lrow, P.lvn, BLOCK);
        if constexpr (EX >= 1) {
          if (A.born.rot) A.born.rot[gb] = P.rn;
          if (A.st.px) {
            const uint64_t gs = O.side ? gq : gp;
            A.born.px[gb] = A.st.px[gs];
            A.born.py[gb] = A.st.py[gs];
            A.born.pz[gb] = A.st.pz[gs];
          }
        }
      }
      bflag[at] = born ? 1 : 0;
      if (born) {
        const uint32_t b = atomicAdd(&s_nborn, 1u);
        if (b < kBornList) s_born[b] = j;
      }
    }
    HCAO_WAVE_MARK(wclk, kPhaseCollideWrite);
#ifdef HCAO_PHASE_CLOCKS
    if (lead)
      for (int x = 0; x < 5; ++x) atomicAdd(&s_wclk[x], (unsigned long long)wclk[x]);
#endif
    }
  }
  __syncthreads();
  HCAO_PHASE_MARK(kPhaseCollide);

  // ---- phase C: deaths, products in pair order, per-cell state ----
  // one wave per cell: ballots give each survivor its new slot and each
  // product its rank in pair order. In the mixed form the per-pair records
  // of a cell's first 64 candidates are loaded while the wave still works
  // on its previous cell, so that their latency overlaps it (the fp64 form
  // has no registers to spare for it).
  const bool records = MIX || A.tdelta != nullptr;
  constexpr bool kPrefetch = MIX;
  // entry of the group's candidate j, ~0u if it was not accepted
  auto entry_of = [&](uint32_t j) {
    const WorkRound r = rounds[HCAO_IDX(j / 64, (wcap + 63) / 64, A.err)];
    const uint32_t i = j & 63u;
    return (r.mask >> i) & 1ull ? r.first + (uint32_t)__popcll(r.mask & ((1ull << i) - 1ull)) : ~0u;
  };
  auto chunk_load = [&](uint32_t g, uint32_t k0) {
    const CellHdr &H = hdr[g];
    const uint32_t k = k0 + lane;
    Records r{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    const uint32_t f = k < H.ncand ? entry_of(H.cstart + k) : ~0u;
    if (f != ~0u) {
      const uint32_t i = (uint32_t)HCAO_IDX(f, wcap, A.err);
      if (A.tdelta) {
        const uint64_t e = wbase + i;
        r.y0 = A.tdelta[e];
        r.y1 = A.tdelta[A.tdelta_stride + e];
        r.y2 = A.tdelta[2 * A.tdelta_stride + e];
        r.y3 = A.tdelta[3 * A.tdelta_stride + e];
        r.y4 = A.tdelta[4 * A.tdelta_stride + e];
      }
      if (MIX) r.y5 = wdef[i];
    }
    return r;
  };
  // the product of candidate j to slot `slot`
  auto place_born = [&](uint32_t j, uint64_t slot) {
    const uint64_t from = HCAO_IDX(wbase + j, A.born.n_slots, A.err), to = HCAO_IDX(slot, A.st.n_slots, A.err);
    const BodyOf<R> b = ldb<MIX>(A.born, from);
    stb<MIX>(A.st, to, b.v, b.sp);
    copy_levels(A.born, from, A.st, to);
    if constexpr (EX >= 1) {
      if (A.st.rot) A.st.rot[to] = A.born.rot[from];
      if (A.st.px) {
        A.st.px[to] = A.born.px[from];
        A.st.py[to] = A.born.py[from];
        A.st.pz[to] = A.born.pz[from];
      }
    }
  };
  // one chunk's sums: value tree6_value(lane) (the defect alone: lane 0)
  auto chunk_sum = [&](const Records &r) {
    if (A.tdelta) return tree_sum6(r.y0, r.y1, r.y2, r.y3, r.y4, r.y5);
    double z[1] = {r.y5};
    tree_sum(z);
    return z[0];
  };
  const uint32_t vx = A.tdelta ? tree6_value(lane) : (lane == 0 ? 5u : 6u);
  // chunk sums of big cells, in the memory of the pairs' velocities (free
  // from here to the next step): six numbers per chunk
  double *chunks = reinterpret_cast<double *>(pv);
  const bool big = records && s_big != 0;
  if (big) {
    for (uint32_t g = 0; g < ncell; ++g) {
      const uint32_t nc = hdr[g].ncand;
      if (nc <= kBigCell) continue;
      double *to = chunks + 6 * (size_t)(hdr[g].cstart / 64 + g);
      for (uint32_t h = wave; h * 64 < nc; h += BLOCK / 64) {
        const double d = chunk_sum(chunk_load(g, h * 64));
        if (vx < 6u) to[6 * (size_t)h + vx] = d;
      }
    }
    __syncthreads();
  }
  Records next{0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  if (kPrefetch && records && wave < ncell) next = chunk_load(wave, 0);
  for (uint32_t g = wave; g < ncell; g += BLOCK / 64) {
    const CellHdr &H = hdr[g];
    const unsigned long long *in = l_ctr + (size_t)g * nctr;
    const Records first = next;
    if (kPrefetch && records && g + BLOCK / 64 < ncell) next = chunk_load(g + BLOCK / 64, 0);
    uint32_t alive = H.n;
    if (in[HCAO_CTR_DEATHS] != 0ull) {
      // stable in-place compaction: a chunk's survivors move to lower slots
      // after the whole chunk has been read
      uint32_t kept = 0;
      for (uint32_t i0 = 0; i0 < H.n; i0 += 64) {
        const uint32_t i = i0 + lane;
        const uint64_t src = HCAO_IDX(H.base + i, A.st.n_slots, A.err);
        BodyOf<R> b{{R(0), R(0), R(0)}, kDead};
        if (i < H.n) b = ldb<MIX>(A.st, src);
        const bool live = b.sp != kDead;
        const unsigned long long m = __ballot(live);
        const uint64_t dst = HCAO_IDX(H.base + kept + (uint32_t)__popcll(m & lt), A.st.n_slots, A.err);
        if (live) stb<MIX>(A.st, dst, b.v, b.sp);
        if (live) copy_levels(A.st, src, A.st, dst);
        if constexpr (EX >= 1) {
          if (A.st.rot) {
            double rv = 0.0;
            if (live) rv = A.st.rot[src];
            if (live) A.st.rot[dst] = rv;
          }
          if (A.st.px) {
            double x = 0.0, y = 0.0, z = 0.0;
            if (live) {
              x = A.st.px[src];
              y = A.st.py[src];
              z = A.st.pz[src];
            }
            if (live) {
              A.st.px[dst] = x;
              A.st.py[dst] = y;
              A.st.pz[dst] = z;
            }
          }
        }
        kept += (uint32_t)__popcll(m);
      }
      alive = kept;
    }
    const uint32_t births = (uint32_t)in[HCAO_CTR_BIRTHS];
    const bool overflow = alive + births > H.cap;
    if (births && !overflow && s_nborn <= kBornList) {
      const uint32_t nb = s_nborn;
      for (uint32_t e = lane; e < nb; e += 64) {
        const uint32_t j = s_born[e];
        if (j < H.cstart || j - H.cstart >= H.ncand) continue;
        uint32_t rank = 0;  // products of the cell from earlier pairs
        for (uint32_t t = 0; t < nb; ++t) rank += s_born[t] >= H.cstart && s_born[t] < j ? 1u : 0u;
        place_born(j, H.base + alive + rank);
      }
    } else if (births && !overflow) {
      uint32_t done = 0;
      for (uint32_t k0 = 0; k0 < H.ncand; k0 += 64) {
        const uint32_t k = k0 + lane;
        const uint32_t e = k < H.ncand ? entry_of(H.cstart + k) : ~0u;
        const bool f = e != ~0u && bflag[HCAO_IDX(e, wcap, A.err)] != 0;
        const unsigned long long m = __ballot(f);
        if (f) {
          place_born(H.cstart + k, H.base + alive + done + (uint32_t)__popcll(m & lt));
        }
        done += (uint32_t)__popcll(m);
      }
    }
    // Per-pair records of the cell, over chunks of 64 consecutive candidates
    // (left to right), each chunk reduced by a halving tree: the mixed
    // form's energy defects, and the changes of the running sums (a
    // candidate that did not collide contributes 0). A chunk's loads are all
    // issued before any is used.
    if (records) {
      double d = 0.0;  // sum of the lane's value
      if (big && H.ncand > kBigCell) {
        const double *from = chunks + 6 * (size_t)(H.cstart / 64 + g) + (vx < 6u ? vx : 0u);
        const uint32_t nch = (H.ncand + 63) / 64;
        uint32_t h = 0;
        for (; h + 16 <= nch; h += 16) {  // sixteen loads in flight, added in order
          double y[16];
#pragma unroll
          for (int x = 0; x < 16; ++x) y[x] = from[6 * (size_t)(h + x)];
#pragma unroll
          for (int x = 0; x < 16; ++x) d = d + y[x];
        }
        for (; h < nch; ++h) d = d + from[6 * (size_t)h];
      } else {
        for (uint32_t k0 = 0; k0 < H.ncand; k0 += 64) {
          Records r = first;
          if (!kPrefetch || k0) r = chunk_load(g, k0);
          d = d + chunk_sum(r);
        }
      }
      if (vx < 5u && A.tdelta) hdr[g].tsum[vx] = H.tsum[vx] + d;
      if (MIX && vx == 5u) hdr[g].defect = H.defect + d;
    }
    unsigned long long *tot = l_tot + (size_t)g * nctr;
    for (uint32_t i = lane; i < nctr; i += 64) {
      unsigned long long v = in[i];
      if (i == HCAO_CTR_CANDIDATES) v = H.ncand;
      if (i == HCAO_CTR_SUPPRESSED) v += H.excess;
      tot[i] += v;
    }
    if (lane == 0) {
      if (overflow) atomicOr(A.err, kErrCapacity);
      CellHdr &Hm = hdr[g];
      Hm.n = overflow ? alive : alive + births;
      const double seen = __longlong_as_double((long long)H.sgbits);
      Hm.sgmax = seen > H.sgmax ? seen : H.sgmax;
      Hm.rem = H.rem_new;
    }
  }
  __syncthreads();
  HCAO_PHASE_MARK(kPhasePlace);
  }  // steps

  // ---- persistent cell state back to HBM ----
  for (uint32_t g = wave; g < ncell; g += BLOCK / 64) {
    const CellHdr &H = hdr[g];
    const uint32_t c = H.cell;
    unsigned long long *out = A.cells.ctr + (size_t)c * kNumCtr;
    const unsigned long long *tot = l_tot + (size_t)g * nctr;
    for (uint32_t i = lane; i < nctr; i += 64)
      if (tot[i]) atomicAdd(&out[i], tot[i]);  // no return value: the wave does not wait
    if (lane == 0) {
      A.cells.cnt[c] = H.n;
      A.cells.sgmax[c] = H.sgmax;
      A.cells.rem[c] = H.rem;
      if (MIX) A.cells.defect[c] = H.defect;
      if (A.cells.tsum)
        for (int q = 0; q < 5; ++q) A.cells.tsum[(size_t)q * A.cells.n_cells + c] = H.tsum[q];
    }
  }
#ifdef HCAO_PHASE_CLOCKS
  HCAO_PHASE_MARK(kPhaseStore);
  if (tid == 0 && A.clk)
    for (int k = 0; k < kPhases; ++k)
      atomicAdd(&A.clk[k], k >= kPhaseCollideGather ? s_wclk[k - kPhaseCollideGather] : (unsigned long long)clk_acc[k]);
#endif
}

// ---------------------------------------------------------------------------
// thermal initial state
// ---------------------------------------------------------------------------
__device__ __forceinline__ void polar_normals(Rng &rng, double &n1, double &n2) {
  double x, y, s;
  for (;;) {
    x = 2.0 * rng.uniform() - 1.0;
    y = 2.0 * rng.uniform() - 1.0;
    s = x * x + y * y;
    if (s < 1.0 && s > 0.0) break;
  }
  const double f = sqrt((-2.0 * dlog(s)) / s);
  n1 = x * f;
  n2 = y * f;
}

// Internal state of a new molecule at T_vib (levels) and T_rot (rotational
// energy): bends by the floor form, stretches by the uniform proposal with
// the Boltzmann acceptance, then (rotors only) Gamma(zeta/2, k T_rot):
// -ln(1 - u) plus, for zeta = 3, half the square of one polar normal. Writes
// the level row and the rotational energy of
// slot g. The thermal initial state and admission through open faces draw
// the same way.
//
// LANES (a power of two) consecutive lanes may share one molecule, all with
// its state: lane i of them then tests the stretch trial that lies i further
// in the stream (a trial is two uniforms, one block), and the first accepted
// one is the sampler's, as is the stream position after it.
template <uint32_t LANES>
__device__ __forceinline__ void sample_internal(const SpeciesTab &S, const double *theta, const double *lev, Rng &rng, double tv,
                                                double trot, const State &st, uint64_t g, uint32_t mm) {
  const uint32_t sub = threadIdx.x & (LANES - 1u), lane0 = (threadIdx.x & 63u) - sub;
  const bool writer = sub == 0;
  for (uint32_t m = 0; m < mm; ++m) {
    uint32_t l = 0;
    if (m < S.n_modes) {
      if (m < S.n_bend) {
        // floor(-ln(1 - u) T / Theta): a single-precision estimate settles it
        // unless it lies near an integer
        const double r = 1.0 - rng.uniform();
        const double ratio = tv / theta[m];
        const float k = (float)(ratio * 0.6931471805599453), x = -__builtin_amdgcn_logf((float)r) * k;
        const float fl = floorf(x), band = 1e-5f * (x + 1.0f) + 1e-6f * k;
        if (x - fl > band && (fl + 1.0f) - x > band && fl < 65000.0f) {
          l = (uint32_t)fl;
        } else {
          const double lg = -dlog(r);
          double fi = floor(lg * ratio);
          fi = fi > 65535.0 ? 65535.0 : fi;
          l = (uint32_t)fi;
        }
      } else {
        const uint32_t top = S.idiss[m];
        const double *L = lev + S.lev_off[m];
        const double kt = kBoltz * tv;
        for (;;) {
          Rng r = rng;
          if (LANES > 1 && sub > 0) {
            // trial sub: as many blocks further on, with the words that the
            // trial before it left
            r.block += sub;
            if (r.used == 2) {
              r.block -= 1;
              r.refill();
              r.used = 2;
            }
          }
          const double u = r.uniform();
          uint32_t j = (uint32_t)floor(u * (double)(top + 1));
          j = j > top ? top : j;
          const double u2 = r.uniform();
          const double xx = (L[j] - L[0]) / kt;
          const bool ok = below_exp_neg(u2, xx);
          if constexpr (LANES == 1) {
            rng = r;
            if (ok) {
              l = j;
              break;
            }
          } else {
            const uint32_t hit = (uint32_t)(__ballot(ok) >> lane0) & ((1u << LANES) - 1u);
            const int src = (int)lane0 + (hit ? __ffs((int)hit) - 1 : (int)LANES - 1);
            rng.block = __shfl(r.block, src);
            rng.used = __shfl(r.used, src);
            rng.w0 = __shfl(r.w0, src);
            rng.w1 = __shfl(r.w1, src);
            rng.w2 = __shfl(r.w2, src);
            rng.w3 = __shfl(r.w3, src);
            l = __shfl(j, src);
            if (hit) break;
          }
        }
      }
    }
    if (writer) st.lvl[g * st.lrow + m] = (uint16_t)l;
  }
  if (writer)
    for (uint32_t m = mm; m < st.lrow; ++m) st.lvl[g * st.lrow + m] = 0;
  if (st.rot) {
    double e = 0.0;
    if (S.zeta_rot > 0) {
      double gm = -dlog(1.0 - rng.uniform());
      if (S.zeta_rot == 3) {
        double z1, z2;
        polar_normals(rng, z1, z2);
        gm = gm + 0.5 * (z1 * z1);
      }
      e = (kBoltz * trot) * gm;
    }
    if (writer) st.rot[g] = e;
  }
}

struct InitArgs {
  const Tables *tab;
  const double *lev;
  State st;
  const uint64_t *off;
  const uint32_t *counts;  // [n_cells][n_species]
  const double *t_trans, *t_vib;
  uint64_t seed;
  uint32_t n_cells;
  uint32_t nx, ny, nz;  // spatial mode grid (positions drawn when st.px is set)
  double len[3];
};

__global__ __launch_bounds__(256) void k_init(InitArgs A) {
  const uint32_t c = blockIdx.x;
  const Tables &T = *A.tab;
  const uint32_t ns = T.n_species, mm = T.max_modes;
  const uint32_t *cnt = A.counts + (size_t)c * ns;
  uint32_t n = 0;
  for (uint32_t s = 0; s < ns; ++s) n += cnt[s];
  const double tt = A.t_trans[c], tv = A.t_vib[c];
  for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
    uint32_t s = 0, acc = cnt[0];
    while (i >= acc) acc += cnt[++s];
    const SpeciesTab &S = T.sp[s];
    Rng rng;
    rng.open(A.seed, i, c, 0xFFFFFFFEu);
    double n1, n2, n3, n4;
    polar_normals(rng, n1, n2);
    polar_normals(rng, n3, n4);
    const double sigma = sqrt((kBoltz * tt) / S.mass);
    const uint64_t g = A.off[c] + i;
    store_body(A.st, g, sigma * n1, sigma * n2, sigma * n3, s);
    sample_internal<1>(S, T.theta[s], A.lev, rng, tv, tt, A.st, g, mm);
    if (A.st.px) {
      // spatial mode: uniform in the cell, one draw per axis
      const uint32_t ix = c % A.nx, iy = (c / A.nx) % A.ny, iz = c / (A.nx * A.ny);
      A.st.px[g] = ((double)ix + rng.uniform()) * (A.len[0] / (double)A.nx);
      A.st.py[g] = ((double)iy + rng.uniform()) * (A.len[1] / (double)A.ny);
      A.st.pz[g] = ((double)iz + rng.uniform()) * (A.len[2] / (double)A.nz);
    }
  }
}

// ---------------------------------------------------------------------------
// initial (sigma g)_max bound per cell: max over present species pairs of
// C (4 max|v|^2)^(1-w); remainder reset
// ---------------------------------------------------------------------------
struct CellInitArgs {
  const Tables *tab;
  State st;
  CellArrays cells;
};

__global__ __launch_bounds__(256) void k_cell_init(CellInitArgs A) {
  __shared__ unsigned long long s_v;
  __shared__ uint32_t s_mask;
  const uint32_t c = blockIdx.x;
  const uint64_t base = A.cells.off[c];
  const uint32_t n = A.cells.cnt[c];
  if (threadIdx.x == 0) {
    s_v = 0ull;
    s_mask = 0u;
  }
  __syncthreads();
  double vmax2 = 0.0;
  uint32_t mask = 0;
  for (uint32_t i = threadIdx.x; i < n; i += blockDim.x) {
    const BodyOf<double> b = load_body(A.st, base + i);
    const double v2 = (b.v.x * b.v.x + b.v.y * b.v.y) + b.v.z * b.v.z;
    vmax2 = v2 > vmax2 ? v2 : vmax2;
    mask |= 1u << b.sp;
  }
  atomicMax(&s_v, (unsigned long long)__double_as_longlong(vmax2));
  atomicOr(&s_mask, mask);
  if (A.cells.tsum && threadIdx.x < 64) {
    // the running sums of the cell temperature start from the particles
    double sums[5];
    if (A.st.b32)
      cell_sums<true>(A.st, A.tab->sp, base, n, threadIdx.x, sums);
    else
      cell_sums<false>(A.st, A.tab->sp, base, n, threadIdx.x, sums);
    if (threadIdx.x == 0)
      for (int q = 0; q < 5; ++q) A.cells.tsum[(size_t)q * A.cells.n_cells + c] = sums[q];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const Tables &T = *A.tab;
    const double g2 = 4.0 * __longlong_as_double((long long)s_v);
    double best = 0.0;
    if (g2 > 0.0) {
      for (uint32_t a = 0; a < T.n_species; ++a) {
        if (!((s_mask >> a) & 1u)) continue;
        for (uint32_t b = 0; b < T.n_species; ++b) {
          if (!((s_mask >> b) & 1u)) continue;
          const double sg = T.pr[a][b].csg * dpow(g2, T.pr[a][b].esg);
          best = sg > best ? sg : best;
        }
      }
    }
    A.cells.sgmax[c] = best;
    A.cells.rem[c] = 0.0;
    unsigned long long *ctr = A.cells.ctr + (size_t)c * kNumCtr;
    for (int i = 0; i < kNumCtr; ++i) ctr[i] = 0ull;
  }
}

// ---------------------------------------------------------------------------
// moments per cell: [0..2] sum m v, [3] sum m |v|^2, [4] sum m, [5] sum h_s,
// [6 + s] count_s, [6 + S + s] sum (E_vib - ZPE)_s, [6 + 2 S + s] sum E_rot_s.
// Lane partials are combined by a fixed halving tree.
// ---------------------------------------------------------------------------
struct MomentArgs {
  const Tables *tab;
  const double *lev;
  State st;
  const uint64_t *off;
  const uint32_t *cnt;
  double *out;  // [n_cells][6 + 3 S]: sums, counts, E_vib above ZPE, E_rot per species
  uint32_t n_cells;
  const uint32_t *cap, *list;  // list: the cells with more than kMomentsLarge slots, if some have so many
};

// WAVES waves per cell: one for cells of a few hundred particles (four cells
// per workgroup), eight for large ones. NS: a bound of the species count, so
// that the per-species sums stay in registers. One workgroup of 256 threads
// per cell, each sum reduced through LDS with nine barriers, took 7.0 ms for
// 262,144 cells of 256 particles; with a wave per cell the whole read of the
// moments takes 1.1, most of it the pass over the state. Large cells among
// small ones have a launch of their own (list): one of a million particles beside
// 999 of 100 keeps one wave for 20.8 ms, eight for 3.1.
template <int NS, int WAVES>
__global__ __launch_bounds__(WAVES == 1 ? 256 : 64 * WAVES) void k_moments(MomentArgs A) {
  constexpr int kW = 6 + 2 * NS;  // per-lane sums: the common ones, E_vib and E_rot per species
  constexpr int kCells = WAVES == 1 ? 4 : 1;
  __shared__ double s_part[WAVES][6 + 3 * NS];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t c = blockIdx.x * kCells + (WAVES == 1 ? wave : 0u);
  if (WAVES == 1) {
    if (c >= A.n_cells || (A.list && A.cap[c] > kMomentsLarge)) return;
  } else if (A.list) {
    c = A.list[c];
  }
  const Tables &T = *A.tab;
  const uint32_t ns = T.n_species;
  const uint64_t base = A.off[c];
  const uint32_t n = A.cnt[c];
  double acc[kW];
  uint32_t count[NS];
#pragma unroll
  for (int j = 0; j < kW; ++j) acc[j] = 0.0;
#pragma unroll
  for (int j = 0; j < NS; ++j) count[j] = 0;
  for (uint32_t i0 = WAVES == 1 ? 0u : 64u * wave; i0 < n; i0 += 64u * WAVES) {
    const uint32_t i = i0 + lane;
    const bool in = i < n;
    const uint64_t g = base + (in ? i : 0u);
    BodyOf<double> b{{0.0, 0.0, 0.0}, ~0u};
    if (in) b = load_body(A.st, g);
    const uint32_t s = b.sp;
    double ev = 0.0, er = 0.0;
    if (in) {
      const SpeciesTab &S = T.sp[s];
      const double m = S.mass;
      const Vec3 v = b.v;
      acc[0] += m * v.x;
      acc[1] += m * v.y;
      acc[2] += m * v.z;
      acc[3] += m * ((v.x * v.x + v.y * v.y) + v.z * v.z);
      acc[4] += m;
      acc[5] += S.formation;
      const uint32_t *row = reinterpret_cast<const uint32_t *>(A.st.lvl + g * A.st.lrow);
      const uint32_t nb = S.n_bend, nm = S.n_modes;
      for (uint32_t q = 0; q < nm; q += 2) {
        const uint32_t x = row[q / 2];
        const uint32_t l0 = x & 0xFFFFu, l1 = x >> 16;
        ev = ev + (q < nb ? ((double)l0 + 0.5) * S.kt[q] : A.lev[S.lev_off[q] + l0]);
        if (q + 1 < nm) ev = ev + (q + 1 < nb ? ((double)l1 + 0.5) * S.kt[q + 1] : A.lev[S.lev_off[q + 1] + l1]);
      }
      ev = ev - S.zpe;
      if (A.st.rot) er = A.st.rot[g];
    }
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      const bool is = s == (uint32_t)j;
      count[j] += (uint32_t)__popcll(__ballot(is));
      acc[6 + j] += is ? ev : 0.0;
      if (A.st.rot) acc[6 + NS + j] += is ? er : 0.0;
    }
  }
#pragma unroll
  for (int j = 0; j < kW; ++j) {
    double y[1] = {acc[j]};
    if (j < 6 + NS || A.st.rot) tree_sum(y);
    acc[j] = y[0];
  }
  double *out = A.out + (size_t)c * (6 + 3 * ns);
  double *to = WAVES == 1 ? out : s_part[wave];
  if (lane == 0) {
#pragma unroll
    for (int j = 0; j < 6; ++j) to[j] = acc[j];
#pragma unroll
    for (int j = 0; j < NS; ++j) {
      if ((uint32_t)j < ns) {
        to[6 + j] = (double)count[j];
        to[6 + ns + j] = acc[6 + j];
        to[6 + 2 * ns + j] = A.st.rot ? acc[6 + NS + j] : 0.0;
      }
    }
  }
  if (WAVES > 1) {
    __syncthreads();
    for (uint32_t j = tid; j < 6 + 3 * ns; j += 64 * WAVES) {
      double y = s_part[0][j];
      for (int w = 1; w < WAVES; ++w) y = y + s_part[w][j];
      out[j] = y;
    }
  }
}

// Sums of the cells' moments, their weighted counts (w columns, then S) and
// their energy defects (one more): workgroup b takes the b-th of gridDim.x
// equal runs of cells, one wave per column; lanes take cells in turn and a
// halving tree combines them.
struct MomentSumArgs {
  const double *in, *weight, *defect;
  double *out;  // [gridDim.x][w + S + 1]
  uint32_t n_cells, w, ns;
};
__global__ __launch_bounds__(256) void k_moments_sum(MomentSumArgs A) {
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6, cols = A.w + A.ns + 1;
  const uint32_t per = (A.n_cells + gridDim.x - 1) / gridDim.x;
  const uint32_t c0 = blockIdx.x * per, c1 = c0 + per < A.n_cells ? c0 + per : A.n_cells;
  for (uint32_t k = wave; k < cols; k += 4) {
    double y[1] = {0.0};
    for (uint32_t c = c0 + lane; c < c1; c += 64) {
      if (k < A.w)
        y[0] = y[0] + A.in[(size_t)c * A.w + k];
      else if (k < A.w + A.ns)
        y[0] = y[0] + A.in[(size_t)c * A.w + 6 + (k - A.w)] * A.weight[c];
      else
        y[0] = y[0] + A.defect[c];
    }
    tree_sum(y);
    if (lane == 0) A.out[(size_t)blockIdx.x * cols + k] = y[0];
  }
}

// Vibrational temperature of every (cell, species): the temperature whose
// Boltzmann mean energy above the ground levels equals the species' mean, by
// the Illinois form of regula falsi in log T between two nodes of a table of
// means (512 nodes over 1 .. 1e6 K, equally spaced in log T). One thread
// each; on the host the same took 2.4 us per cell and species (the moments of
// 12,345 cells: 28.6 ms, now 1.9).
struct ThermoArgs {
  const Tables *tab;
  const double *lev;
  const double *mean;  // [S][kThermoNodes]
  const double *in;    // [n_cells][w]
  double *t;           // [n_cells][S]
  uint32_t n_cells, w, ns;
  uint32_t same[kMaxSpecies];  // bit m: stretch m has stretch m - 1's ladder
};
__device__ __forceinline__ double thermo_mean(const ThermoArgs &A, uint32_t s, double t) {
  const SpeciesTab &S = A.tab->sp[s];
  double e = 0.0, last = 0.0;
  for (uint32_t m = 0; m < S.n_bend; ++m) {
    const double th = A.tab->theta[s][m];
    e = e + kBoltz * th / expm1(th / t);
  }
  const double kt = kBoltz * t;
  for (uint32_t m = S.n_bend; m < S.n_modes; ++m) {
    if (!((A.same[s] >> m) & 1u)) {
      const double *L = A.lev + S.lev_off[m];
      double top = 0.0, bottom = 0.0;
      for (uint32_t i = 0; i <= S.idiss[m]; ++i) {
        const double d = L[i] - L[0], w = exp(-d / kt);
        top = top + d * w;
        bottom = bottom + w;
      }
      last = top / bottom;
    }
    e = e + last;
  }
  return e;
}
__global__ __launch_bounds__(64) void k_thermometer(ThermoArgs A) {
  const uint64_t i = (uint64_t)blockIdx.x * 64 + threadIdx.x;
  if (i >= (uint64_t)A.n_cells * A.ns) return;
  // a wave takes one species of 64 cells
  const uint32_t c = (uint32_t)(i % A.n_cells), s = (uint32_t)(i / A.n_cells);
  const double *r = A.in + (size_t)c * A.w;
  const double n = r[6 + s];
  double t = 0.0;
  const double e = n > 0.0 ? r[6 + A.ns + s] / n : 0.0;
  if (A.tab->sp[s].n_modes > 0 && e > 0.0) {
    const double *M = A.mean + (size_t)s * kThermoNodes;
    const double top = log(1.0e6);
    if (!(e < M[kThermoNodes - 1])) {
      t = exp(top);
    } else {
      uint32_t lo = 0, hi = kThermoNodes - 1;  // first node whose mean reaches e
      while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (M[mid] < e)
          lo = mid + 1;
        else
          hi = mid;
      }
      hi = hi ? hi : 1u;
      double a = top * (double)(hi - 1) / (double)(kThermoNodes - 1), b = top * (double)hi / (double)(kThermoNodes - 1);
      double fa = M[hi - 1] - e, fb = M[hi] - e;
      int side = 0;
      bool found = fb == 0.0;
      if (found) t = exp(b);
      for (int it = 0; !found && it < 100 && b - a > 1e-15 * (1.0 + fabs(b)); ++it) {
        const double x = (a * fb - b * fa) / (fb - fa);
        const double fx = thermo_mean(A, s, exp(x)) - e;
        if (fx == 0.0) {
          t = exp(x);
          found = true;
          break;
        }
        if ((fx < 0.0) == (fa < 0.0)) {
          a = x;
          fa = fx;
          if (side == -1) fb *= 0.5;
          side = -1;
        } else {
          b = x;
          fb = fx;
          if (side == 1) fa *= 0.5;
          side = 1;
        }
        if (x == a && x == b) break;
      }
      if (!found) t = exp(fabs(fa) < fabs(fb) ? a : b);
    }
  }
  A.t[(size_t)c * A.ns + s] = t;
}

// reactions performed, summed over cells: out[r] (cleared before the launch)
__global__ __launch_bounds__(256) void k_reaction_sum(const unsigned long long *ctr, uint32_t n_cells, uint32_t nr,
                                                      unsigned long long *out) {
  const uint32_t lane = threadIdx.x & 63u;
  for (uint32_t r = 0; r < nr; ++r) {
    unsigned long long s = 0;
    for (uint32_t c = blockIdx.x * 256 + threadIdx.x; c < n_cells; c += gridDim.x * 256)
      s += ctr[(size_t)c * kNumCtr + HCAO_CTR_REACTION0 + r];
    for (int d = 32; d > 0; d >>= 1) s += __shfl_down(s, d);
    if (lane == 0 && s) atomicAdd(&out[r], s);
  }
}

// ---------------------------------------------------------------------------
// stable counting sort of particles by cell (LSD radix, passes of equal digit
// width up to 9 bits): per-tile digit histograms, one exclusive scan in digit-major order, and a
// stable scatter that ranks equal digits inside a wavefront with ballots.
// ---------------------------------------------------------------------------
constexpr int kSortBlock = 256;
constexpr int kSortItems = 16;
constexpr int kSortTile = kSortBlock * kSortItems;
constexpr uint32_t kSortMaxBits = 9;  // digit width of a pass: up to 9 bits (512 bins)
constexpr uint32_t kSortMaxBins = 1u << kSortMaxBits;

__global__ __launch_bounds__(kSortBlock) void k_sort_hist(const uint32_t *keys, uint64_t n, uint32_t shift,
                                                          uint32_t bits, uint32_t *hist, uint32_t n_tiles) {
  __shared__ uint32_t s_h[kSortMaxBins];
  const uint32_t bins = 1u << bits, mask = bins - 1u;
  for (uint32_t b = threadIdx.x; b < bins; b += kSortBlock) s_h[b] = 0;
  __syncthreads();
  const uint64_t t0 = (uint64_t)blockIdx.x * kSortTile;
  for (int it = 0; it < kSortItems; ++it) {
    const uint64_t i = t0 + (uint64_t)it * kSortBlock + threadIdx.x;
    if (i < n) atomicAdd(&s_h[(keys[i] >> shift) & mask], 1u);
  }
  __syncthreads();
  for (uint32_t b = threadIdx.x; b < bins; b += kSortBlock) hist[(uint64_t)b * n_tiles + blockIdx.x] = s_h[b];
}

// Multi-block exclusive scan of u32 into u64: each 256-thread block scans a
// chunk of kScanChunk entries (four neighbours per thread and round, scanned by
// wave shuffles) and leaves its total in bsum; a second pass adds the totals of
// the chunks before. Integer sums, so the result does not depend on the split.
// (A block of 1,024 threads with 16 neighbours each, two barriers per doubling
// and a launch of its own for the totals took 26 us for the smallest scan.)
constexpr int kScanRounds = 4;
constexpr uint64_t kScanChunk = 256 * 4 * kScanRounds;

__device__ __forceinline__ uint64_t wave_inclusive(uint64_t v, uint32_t lane) {
  for (uint32_t d = 1; d < 64; d <<= 1) {
    const uint64_t o = __shfl_up(v, d);
    if (lane >= d) v += o;
  }
  return v;
}

__global__ __launch_bounds__(256) void k_scan_chunk(const uint32_t *in, uint64_t *out, uint64_t n, uint64_t *bsum) {
  __shared__ uint64_t s_wave[kScanRounds][4];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint64_t b0 = (uint64_t)blockIdx.x * kScanChunk + 4 * tid;
  uint32_t x[kScanRounds][4];
  uint64_t sum[kScanRounds], inc[kScanRounds];
#pragma unroll
  for (int r = 0; r < kScanRounds; ++r) {
    const uint64_t i = b0 + 1024u * r;
#pragma unroll
    for (int k = 0; k < 4; ++k) x[r][k] = i + k < n ? in[i + k] : 0u;
    sum[r] = ((uint64_t)x[r][0] + x[r][1]) + ((uint64_t)x[r][2] + x[r][3]);
  }
#pragma unroll
  for (int r = 0; r < kScanRounds; ++r) {
    inc[r] = wave_inclusive(sum[r], lane);
    if (lane == 63) s_wave[r][wave] = inc[r];
  }
  __syncthreads();
  uint64_t run = 0;
#pragma unroll
  for (int r = 0; r < kScanRounds; ++r) {
    uint64_t acc = run;
#pragma unroll
    for (uint32_t w = 0; w < 4; ++w) {
      const uint64_t t = s_wave[r][w];
      if (w < wave) acc += t;
      run += t;
    }
    acc += inc[r] - sum[r];
    const uint64_t i = b0 + 1024u * r;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      if (i + k < n) out[i + k] = acc;
      acc += x[r][k];
    }
  }
  if (tid == 0) bsum[blockIdx.x] = run;
}

// adds the totals of the earlier chunks to every chunk but the first
__global__ __launch_bounds__(256) void k_scan_add(uint64_t *out, uint64_t n, const uint64_t *bsum) {
  __shared__ uint64_t s_wave[4];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, chunk = blockIdx.x + 1;
  uint64_t v = 0;
  for (uint32_t b = tid; b < chunk; b += 256) v += bsum[b];
  for (int d = 32; d > 0; d >>= 1) v += __shfl_down(v, d);
  if (lane == 0) s_wave[tid >> 6] = v;
  __syncthreads();
  v = (s_wave[0] + s_wave[1]) + (s_wave[2] + s_wave[3]);
  const uint64_t b0 = (uint64_t)chunk * kScanChunk;
  for (uint64_t i = b0 + tid; i < b0 + kScanChunk && i < n; i += 256) out[i] += v;
}

__global__ __launch_bounds__(kSortBlock) void k_sort_scatter(const uint32_t *keys_in, const uint32_t *idx_in,
                                                             uint32_t *keys_out, uint32_t *idx_out, uint64_t n,
                                                             uint32_t shift, uint32_t bits, const uint64_t *offs,
                                                             uint32_t n_tiles) {
  constexpr int kWaves = kSortBlock / 64;
  __shared__ uint32_t s_run[kSortMaxBins];
  __shared__ uint32_t s_wave[kWaves][kSortMaxBins];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t bins = 1u << bits, mask = bins - 1u;
  for (uint32_t b = tid; b < bins; b += kSortBlock) s_run[b] = 0;
  __syncthreads();
  const uint64_t t0 = (uint64_t)blockIdx.x * kSortTile;
  const unsigned long long lt = lane ? ((1ull << lane) - 1ull) : 0ull;
  // the tile's keys and indices are loaded at once, before the ranking
  // rounds (whose barriers would otherwise wait on each round's loads)
  uint32_t kr[kSortItems], ir[kSortItems];
#pragma unroll
  for (int it = 0; it < kSortItems; ++it) {
    const uint64_t i = t0 + (uint64_t)it * kSortBlock + tid;
    kr[it] = i < n ? keys_in[i] : 0u;
    ir[it] = idx_in ? (i < n ? idx_in[i] : 0u) : (uint32_t)i;  // the first pass: entry i is entry i
  }
#pragma unroll
  for (int it = 0; it < kSortItems; ++it) {
    for (int w = 0; w < kWaves; ++w)
      for (uint32_t b = tid; b < bins; b += kSortBlock) s_wave[w][b] = 0;
    __syncthreads();
    const uint64_t i = t0 + (uint64_t)it * kSortBlock + tid;
    const bool valid = i < n;
    const uint32_t key = kr[it];
    const uint32_t d = (key >> shift) & mask;
    unsigned long long same = __ballot(valid);
#pragma unroll
    for (uint32_t bit = 0; bit < kSortMaxBits; ++bit) {
      if (bit < bits) {  // the same on every lane
        const unsigned long long bb = __ballot(((d >> bit) & 1u) != 0u);
        same &= ((d >> bit) & 1u) ? bb : ~bb;
      }
    }
    const uint32_t rank = (uint32_t)__popcll(same & lt);
    if (valid && rank == 0) s_wave[wave][d] = (uint32_t)__popcll(same);
    __syncthreads();
    uint32_t before = s_run[d];
    for (uint32_t w = 0; w < wave; ++w) before += s_wave[w][d];
    if (valid) {
      const uint64_t pos = offs[(uint64_t)d * n_tiles + blockIdx.x] + before + rank;
      keys_out[pos] = key;
      idx_out[pos] = ir[it];
    }
    __syncthreads();
    for (uint32_t b = tid; b < bins; b += kSortBlock) {
      uint32_t add = 0;
      for (int w = 0; w < kWaves; ++w) add += s_wave[w][b];
      s_run[b] += add;
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// load: validate host particles, count per cell, place in sorted order
// ---------------------------------------------------------------------------
struct LoadArgs {
  const Tables *tab;
  const uint32_t *cell;
  const uint8_t *sp;
  const double *vel;   // 3n
  const uint16_t *lvl; // n x mm
  uint64_t n;
  uint32_t n_cells;
  uint32_t *count;     // [n_cells]
  uint32_t *err;
};

__global__ __launch_bounds__(256) void k_load_check(LoadArgs A) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= A.n) return;
  const Tables &T = *A.tab;
  const uint32_t mm = T.max_modes;
  uint32_t err = 0;
  const uint32_t c = A.cell[i], s = A.sp[i];
  if (c >= A.n_cells || s >= T.n_species) {
    err |= kErrInvalid;
  } else {
    const double vx = A.vel[3 * i], vy = A.vel[3 * i + 1], vz = A.vel[3 * i + 2];
    if (!isfinite(vx) || !isfinite(vy) || !isfinite(vz)) err |= kErrNonFinite;
    const SpeciesTab &S = T.sp[s];
    for (uint32_t m = 0; m < mm; ++m) {
      const uint32_t l = A.lvl[i * mm + m];
      if (m >= S.n_modes) {
        if (l != 0) err |= kErrLevel;
      } else if (m >= S.n_bend && l > S.idiss[m]) {
        err |= kErrLevel;
      }
    }
    atomicAdd(&A.count[c], 1u);
  }
  if (err) atomicOr(A.err, err);
}

struct PlaceArgs {
  const Tables *tab;
  const uint32_t *sorted_cell, *sorted_idx;
  const uint64_t *packed_start;  // exclusive scan of counts
  const uint64_t *off;           // slot offsets
  const uint8_t *sp;
  const double *vel;
  const uint16_t *lvl;
  const double *rot;  // may be null
  const double *pos;  // 3n, spatial mode
  State st;
  uint64_t n;
};

__global__ __launch_bounds__(256) void k_load_place(PlaceArgs A) {
  const uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= A.n) return;
  const uint32_t c = A.sorted_cell[j];
  const uint64_t src = A.sorted_idx[j];
  const uint64_t g = A.off[c] + (j - A.packed_start[c]);
  const uint32_t mm = A.tab->max_modes;
  store_body(A.st, g, A.vel[3 * src], A.vel[3 * src + 1], A.vel[3 * src + 2], A.sp[src]);
  for (uint32_t m = 0; m < A.st.lrow; ++m) A.st.lvl[g * A.st.lrow + m] = m < mm ? A.lvl[src * mm + m] : (uint16_t)0;
  if (A.st.rot) A.st.rot[g] = A.rot ? A.rot[src] : 0.0;
  if (A.st.px) {
    A.st.px[g] = A.pos[3 * src];
    A.st.py[g] = A.pos[3 * src + 1];
    A.st.pz[g] = A.pos[3 * src + 2];
  }
}

// Particles [p0, p1) of the canonical order into dense arrays (what a reader
// wants of a cell-padded state): workgroup b packs cell c0 + b, whose first
// particle has index start[c]. Levels in rows of mm.
struct PackArgs {
  State st;
  const uint64_t *off, *start;
  const uint32_t *cnt;
  uint8_t *sp;
  double *vel;
  uint16_t *lvl;
  uint64_t p0, p1;
  uint32_t c0, mm;
};
__global__ __launch_bounds__(256) void k_pack(PackArgs A) {
  const uint32_t c = A.c0 + blockIdx.x, n = A.cnt[c], mm = A.mm;
  const uint64_t base = A.off[c], first = A.start[c];
  if (first >= A.p1 || first + n <= A.p0) return;
  const uint32_t i0 = first < A.p0 ? (uint32_t)(A.p0 - first) : 0u;
  const uint32_t i1 = first + n > A.p1 ? (uint32_t)(A.p1 - first) : n;
  const uint64_t to = first + i0 - A.p0;  // of particle i0
  for (uint32_t i = i0 + threadIdx.x; i < i1; i += 256) {
    const uint64_t j = to + (i - i0);
    const BodyOf<double> b = load_body(A.st, base + i);
    A.vel[3 * j] = b.v.x;
    A.vel[3 * j + 1] = b.v.y;
    A.vel[3 * j + 2] = b.v.z;
    A.sp[j] = (uint8_t)b.sp;
  }
  // levels number by number, so that a wave's stores are consecutive
  const uint64_t nl = (uint64_t)(i1 - i0) * mm;
  for (uint64_t f = threadIdx.x; f < nl; f += 256) {
    const uint64_t i = f / mm;
    A.lvl[to * mm + f] = A.st.lvl[(base + i0 + i) * A.st.lrow + (f - i * mm)];
  }
}

// The records of n slots from slot `first` on as arrays of fp64 velocities,
// species and level rows of mm (a checkpoint's form), and back. On the host the
// same took a third of a save or restore.
__global__ __launch_bounds__(256) void k_slots_out(State st, uint64_t first, uint64_t n, uint32_t mm, double *vel,
                                                   uint8_t *sp, uint16_t *lvl) {
  const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const BodyOf<double> b = load_body(st, first + i);
  vel[i] = b.v.x;
  vel[n + i] = b.v.y;
  vel[2 * n + i] = b.v.z;
  sp[i] = (uint8_t)b.sp;
  for (uint32_t m = 0; m < mm; ++m) lvl[i * mm + m] = st.lvl[(first + i) * st.lrow + m];
}
__global__ __launch_bounds__(256) void k_slots_in(State st, uint64_t first, uint64_t n, uint32_t mm, const double *vel,
                                                  const uint8_t *sp, const uint16_t *lvl) {
  const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  store_body(st, first + i, vel[i], vel[n + i], vel[2 * n + i], sp[i]);
  for (uint32_t m = 0; m < st.lrow; ++m) st.lvl[(first + i) * st.lrow + m] = m < mm ? lvl[i * mm + m] : (uint16_t)0;
}

// advances the device step index after the launches of a graph replay
__global__ void k_advance(uint32_t *step, uint32_t n) {
  if (threadIdx.x == 0) step[0] = step[0] + n;
}

__global__ void k_iota(uint32_t *x, uint64_t n) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) x[i] = (uint32_t)i;
}


// ---------------------------------------------------------------------------
// spatial mode: ballistic move with periodic or specular walls, then a
// stable re-bin by (new cell, old slot) that sorts only the particles that
// left their cell
// ---------------------------------------------------------------------------
// one coordinate over dt: periodic axes wrap into [0, L); a specular face
// reflects (x < 0: -x, x > L: 2L - x, velocity reversed; flip set) until
// inside [0, L]; crossing an open face sets left and ends the move
__device__ __forceinline__ double move_axis(double x, double &v, double dt, double len, bool periodic, bool open_lo,
                                           bool open_hi, bool &left, bool &flip) {
  double y = x + v * dt;
  if (periodic) {
    while (y < 0.0) y = y + len;
    while (y >= len) y = y - len;
  } else {
    for (;;) {
      if (y < 0.0) {
        if (open_lo) {
          left = true;
          break;
        }
        y = -y;
        v = -v;
        flip = true;
      } else if (y > len) {
        if (open_hi) {
          left = true;
          break;
        }
        y = (len + len) - y;
        v = -v;
        flip = true;
      } else {
        break;
      }
    }
  }
  return y;
}

// a particle over dt on x, then y, then z; true if it leaves through an open
// face (its coordinates are then of no use); flip tells whether a specular
// face reversed a velocity component
__device__ __forceinline__ bool move_particle(double &x, double &y, double &z, double &vx, double &vy, double &vz,
                                              double dt, const double len[3], uint32_t periodic, uint32_t open,
                                              bool &flip) {
  bool left = false;
  x = move_axis(x, vx, dt, len[0], (periodic & 1u) != 0, (open & 1u) != 0, (open & 2u) != 0, left, flip);
  if (left) return true;
  y = move_axis(y, vy, dt, len[1], (periodic & 2u) != 0, (open & 4u) != 0, (open & 8u) != 0, left, flip);
  if (left) return true;
  z = move_axis(z, vz, dt, len[2], (periodic & 4u) != 0, (open & 16u) != 0, (open & 32u) != 0, left, flip);
  return left;
}

__device__ __forceinline__ uint32_t axis_index(double x, double len, uint32_t n) {
  const double f = floor(x / (len / (double)n));
  if (!(f >= 0.0)) return 0;
  if (f >= (double)n) return n - 1;
  return (uint32_t)f;
}

// a moved particle's new cell; false if it left through an open face. The moved
// state is not stored: the place pass moves the particle again as it copies it
// (the same arithmetic, so the same bits)
__device__ __forceinline__ bool moved_cell(const MoveArgs &A, double x, double y, double z, Vec3 v, uint32_t &key) {
  bool flip = false;
  if (move_particle(x, y, z, v.x, v.y, v.z, A.dt, A.len, A.periodic, A.open, flip)) return false;
  key = axis_index(x, A.len[0], A.nx) + A.nx * (axis_index(y, A.len[1], A.ny) + A.ny * axis_index(z, A.len[2], A.nz));
  return true;
}

// stayer ranks count up from the cell's first slot, mover ranks down from its
// last: together they never pass n <= cap entries
__device__ __forceinline__ void list_particle(const MoveArgs &A, uint64_t base, uint32_t top, uint32_t i, uint32_t key,
                                              bool mover, bool stayer, uint32_t rank_m, uint32_t rank_s) {
  if (mover) {
    const uint64_t at = base + top - rank_m;
    A.list[at] = i;
    A.key[at] = key;
  }
  if (stayer) A.list[base + rank_s] = i;
}

__device__ __forceinline__ void finish_cell(const MoveArgs &A, uint32_t c, uint32_t n, uint32_t stay, uint32_t move) {
  A.n_stay[c] = stay;
  A.n_move[c] = move;
  const uint32_t gone = n - stay - move;
  if (gone && A.flux) atomicAdd(&A.flux[1], (unsigned long long)gone);
}

// The move of one cell by a wave, two slots per lane loaded together; ranks in
// slot order come from ballots.
__device__ __forceinline__ void move_cell_wave(const MoveArgs &A, uint32_t c, uint32_t n, uint32_t lane) {
  constexpr uint32_t kPer = 2;
  const uint64_t base = A.off[c];
  const uint32_t top = A.cap[c] - 1u;
  const uint64_t below_lane = (1ull << lane) - 1ull;
  uint32_t run_s = 0, run_m = 0;
  for (uint32_t i0 = 0; i0 < n; i0 += 64 * kPer) {
    Vec3 v[kPer];
    double x[kPer], y[kPer], z[kPer];
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
      const uint32_t i = i0 + 64 * q + lane;
      if (i < n) {
        const uint64_t g = base + i;
        v[q] = load_body(A.st, g).v;
        x[q] = A.st.px[g];
        y[q] = A.st.py[g];
        z[q] = A.st.pz[g];
      }
    }
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
      const uint32_t i = i0 + 64 * q + lane;
      uint32_t key = 0;
      const bool here = i < n && moved_cell(A, x[q], y[q], z[q], v[q], key);
      const bool mover = here && key != c, stayer = here && key == c;
      const uint64_t bm = __ballot(mover), bs = __ballot(stayer);
      list_particle(A, base, top, i, key, mover, stayer, run_m + (uint32_t)__popcll(bm & below_lane),
                    run_s + (uint32_t)__popcll(bs & below_lane));
      run_s += (uint32_t)__popcll(bs);
      run_m += (uint32_t)__popcll(bm);
    }
  }
  if (lane == 0) finish_cell(A, c, n, run_s, run_m);
}

// The same by the four waves of a workgroup, one slot per lane; the waves' totals
// of a chunk meet in LDS (s_cnt, used in turn so that one barrier per chunk does).
__device__ __forceinline__ void move_cell_group(const MoveArgs &A, uint32_t c, uint32_t n, uint32_t w, uint32_t lane,
                                                uint32_t (*s_cnt)[2][4], uint32_t &turn) {
  const uint64_t base = A.off[c];
  const uint32_t top = A.cap[c] - 1u;
  const uint64_t below_lane = (1ull << lane) - 1ull;
  uint32_t run_s = 0, run_m = 0;
  for (uint32_t i0 = 0; i0 < n; i0 += 256) {
    const uint32_t i = i0 + 64 * w + lane;
    const uint64_t g = base + i;
    uint32_t key = 0;
    const bool here = i < n && moved_cell(A, A.st.px[g], A.st.py[g], A.st.pz[g], load_body(A.st, g).v, key);
    const bool mover = here && key != c, stayer = here && key == c;
    const uint64_t bm = __ballot(mover), bs = __ballot(stayer);
    uint32_t(*t)[4] = s_cnt[turn & 1u];
    ++turn;
    if (lane == 0) {
      t[0][w] = (uint32_t)__popcll(bs);
      t[1][w] = (uint32_t)__popcll(bm);
    }
    __syncthreads();
    uint32_t pre_s = run_s, pre_m = run_m;
#pragma unroll
    for (uint32_t u = 0; u < 4; ++u) {
      if (u < w) {
        pre_s += t[0][u];
        pre_m += t[1][u];
      }
      run_s += t[0][u];
      run_m += t[1][u];
    }
    list_particle(A, base, top, i, key, mover, stayer, pre_m + (uint32_t)__popcll(bm & below_lane),
                  pre_s + (uint32_t)__popcll(bs & below_lane));
  }
  if (lane == 0 && w == 0) finish_cell(A, c, n, run_s, run_m);
}

// Bandwidth bound. CELLS 1: four waves per cell. CELLS 4: one wave per cell, for
// many small cells; with BIG, a cell of more than kMoveBig particles still takes
// the workgroup's four waves (boxes without such a cell do without the test: 98
// and 102 us for the channel of 40,095 cells of 200).
// us with CELLS 1 and 4: fp64, 262,144 cells of 100: 559, 350; of 256: 827, 892;
// 40,095 of 200: 110, 115; 32,768 of 600: 242, 276. Mixed, 262,144 of 256: 886,
// 679; 40,095 of 200: 107, 91; 32,768 of 400: 131, 142; of 600: 188, 210. Few
// cells leave the chip idle in fours: 4,096 of 100 10.9, 9.3; 1,728 of 200 7.9,
// 9.5; 512 of 600 7.5, 18; 64 of 100,000 600, 2,800.
constexpr uint32_t kMoveBig = 1024;      // particles
constexpr uint32_t kMoveManyCells = 4096;
constexpr uint32_t kMoveSmall64 = 160, kMoveSmall32 = 300;  // mean particles per cell, fp64 and mixed form
template <uint32_t CELLS, bool BIG>
__global__ __launch_bounds__(256) void k_move(MoveArgs A) {
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63u;
  const uint32_t c0 = blockIdx.x * CELLS, own = c0 + wave;
  if constexpr (CELLS > 1) {
    if (own < A.n_cells) {
      const uint32_t n = A.cnt[own];
      if (!BIG || n <= kMoveBig) move_cell_wave(A, own, n, lane);
    }
  }
  if constexpr (BIG) {
    __shared__ uint32_t s_cnt[2][2][4];
    uint32_t turn = 0;
    for (uint32_t q = 0; q < CELLS && c0 + q < A.n_cells; ++q) {
      const uint32_t n = A.cnt[c0 + q];
      if (CELLS == 1 || n > kMoveBig) move_cell_group(A, c0 + q, n, wave, lane, s_cnt, turn);
    }
  }
}

// geometry of face cell t / n_species: face f, its axis k and side, the two
// tangential axes a < b, the face cell's indices and the cell behind it
struct FaceCell {
  uint32_t f, k, side, a, b, ia, ib, cell;
  double da, db;
};
__device__ __forceinline__ FaceCell face_cell(const InflowArgs &A, uint32_t gfc) {
  FaceCell F;
  F.f = 0;
  while (gfc >= A.face_base[F.f + 1]) ++F.f;
  F.k = F.f >> 1;
  F.side = F.f & 1u;
  F.a = F.k == 0 ? 1u : 0u;
  F.b = F.k == 2 ? 1u : 2u;
  const uint32_t n3[3] = {A.nx, A.ny, A.nz};
  const uint32_t na = n3[F.a], nb = n3[F.b];
  const uint32_t j = gfc - A.face_base[F.f];
  F.ia = j % na;
  F.ib = j / na;
  uint32_t idx[3];
  idx[F.k] = F.side ? n3[F.k] - 1u : 0u;
  idx[F.a] = F.ia;
  idx[F.b] = F.ib;
  F.cell = idx[0] + A.nx * (idx[1] + A.ny * idx[2]);
  F.da = A.len[F.a] / (double)na;
  F.db = A.len[F.b] / (double)nb;
  return F;
}

__global__ __launch_bounds__(256) void k_inflow_count(InflowArgs A) {
  const uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint32_t ns = A.n_species;
  if (t >= (uint64_t)A.face_base[6] * ns) return;
  const uint32_t gfc = (uint32_t)(t / ns), s = (uint32_t)(t % ns);
  const FaceCell F = face_cell(A, gfc);
  uint32_t cnt = 0;
  if ((A.open >> F.f) & 1u) {
    const double area = F.da * F.db;
    const double x = ((A.flux_s[s] * area) * A.dt) / A.weight[F.cell] + A.rem[t];
    const double fl = floor(x);
    if (fl < 16777216.0) {
      cnt = (uint32_t)fl;
      A.rem[t] = x - fl;
    } else {
      atomicOr(A.err, kErrCapacity);
    }
  }
  A.count[t] = cnt;
}

// admission j of the step: its (face cell, species) t is the last with
// ibase[t] <= j (entries without admissions share the next one's base), i =
// j - ibase[t]. Normal speed from the flux-weighted Maxwellian, sigma
// sqrt(-2 ln(1 - u)); tangential speeds, a polar normal pair times sigma;
// the flight fraction tau; the place on the face cell, uniform per
// tangential axis; levels and rotation as the thermal initial state draws
// them; then a move over tau dt.
//
// A step may admit too few molecules to fill the chip, and each is one long
// chain of draws, mostly rejected stretch proposals: LANES lanes share a
// molecule and its trials, and the tables come from LDS. 20,000 admissions of a
// step of the 45 x 33 x 27 channel: 150 us with a lane each and the tables in
// memory, 134 with the tables in LDS, 61 with four lanes. Lanes are shared
// while the chip has room for them; with 1, 4 and 8 lanes, 7,600 admissions
// take 106, 48 and 34 us, 108,500 take 165, 142 and 206, 244,000 take 240, 247
// and 400, 549,000 take 357, 492 and 760.
constexpr uint64_t kInflowEight = 16384, kInflowFour = 196608;  // the most admissions that take so many lanes
constexpr uint32_t kInflowLevels = 4096;  // levels staged in LDS at most (32 KB); larger ladders are read from memory
template <uint32_t LANES>
__global__ __launch_bounds__(64) void k_inflow_make(InflowArgs A) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  SpeciesTab *l_sp = reinterpret_cast<SpeciesTab *>(smem);
  double *l_theta = reinterpret_cast<double *>(l_sp + A.n_species), *l_lev = l_theta + A.n_species * kMaxModes;
  {
    const uint64_t *src = reinterpret_cast<const uint64_t *>(A.tab->sp);
    uint64_t *dst = reinterpret_cast<uint64_t *>(l_sp);
    for (uint32_t i = threadIdx.x; i < A.n_species * sizeof(SpeciesTab) / 8; i += blockDim.x) dst[i] = src[i];
    for (uint32_t i = threadIdx.x; i < A.n_species * kMaxModes; i += blockDim.x)
      l_theta[i] = A.tab->theta[i / kMaxModes][i % kMaxModes];
    for (uint32_t i = threadIdx.x; i < A.n_levels; i += blockDim.x) l_lev[i] = A.lev[i];
  }
  __syncthreads();
  const double *lev = A.n_levels ? l_lev : A.lev;
  const uint64_t j = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) / LANES;
  const bool writer = (threadIdx.x & (LANES - 1u)) == 0;
  if (j >= A.n_ins) return;
  if (j >= A.cap_ins) {
    atomicOr(A.err, kErrCapacity);
    return;
  }
  const uint32_t ns = A.n_species;
  uint64_t lo = 0, hi = (uint64_t)A.face_base[6] * ns - 1;
  while (lo < hi) {
    const uint64_t mid = (lo + hi + 1) >> 1;
    if (A.ibase[mid] <= j)
      lo = mid;
    else
      hi = mid - 1;
  }
  const uint64_t t = lo;
  const uint32_t i = (uint32_t)(j - A.ibase[t]);
  const uint32_t gfc = (uint32_t)(t / ns), s = (uint32_t)(t % ns);
  const FaceCell F = face_cell(A, gfc);
  const SpeciesTab &S = l_sp[s];
  const uint32_t mm = A.tab->max_modes;
  const double sigma = sqrt((kBoltz * A.t_trans) / S.mass);
  Rng rng;
  rng.open(A.seed, (s << 24) | i, A.n_cells + gfc, A.step);
  const double vn = sigma * sqrt(-2.0 * dlog(1.0 - rng.uniform()));
  double n1, n2;
  polar_normals(rng, n1, n2);
  const double tau = rng.uniform();
  const double ua = rng.uniform();
  const double ub = rng.uniform();
  double p[3], v[3];
  p[F.k] = F.side ? A.len[F.k] : 0.0;
  v[F.k] = F.side ? -vn : vn;
  p[F.a] = ((double)F.ia + ua) * F.da;
  p[F.b] = ((double)F.ib + ub) * F.db;
  v[F.a] = sigma * n1;
  v[F.b] = sigma * n2;
  sample_internal<LANES>(S, l_theta + s * kMaxModes, lev, rng, A.t_vib, A.t_trans, A.ins, j, mm);
  bool flip = false;
  const bool left =
      move_particle(p[0], p[1], p[2], v[0], v[1], v[2], tau * A.dt, A.len, A.periodic, A.open, flip);
  if (!writer) return;
  store_body(A.ins, j, v[0], v[1], v[2], s);
  A.ins.px[j] = p[0];
  A.ins.py[j] = p[1];
  A.ins.pz[j] = p[2];
  const uint64_t m_real = A.mbase[A.n_cells];
  A.mkey[m_real + j] = left ? A.n_cells
                            : axis_index(p[0], A.len[0], A.nx) +
                                  A.nx * (axis_index(p[1], A.len[1], A.ny) + A.ny * axis_index(p[2], A.len[2], A.nz));
  A.mslot[m_real + j] = (uint32_t)(A.tot + j);
  if (i == 0) atomicAdd(&A.flux[0], (unsigned long long)A.count[t]);
  if (left) atomicAdd(&A.flux[1], 1ull);
}

// movers of cell c into the list, in slot order
// (one wave per cell, four cells per workgroup)
__global__ __launch_bounds__(256) void k_list_movers(RebinArgs A) {
  const uint32_t c = blockIdx.x * 4u + (threadIdx.x >> 6);
  if (c >= A.n_cells) return;
  const uint32_t nm = A.n_move[c];
  const uint64_t base = A.off[c], mb = A.mbase[c];
  const uint64_t top = base + A.cap[c] - 1u;
  for (uint32_t r = threadIdx.x & 63u; r < nm; r += 64u) {
    A.mkey[mb + r] = A.key[top - r];
    A.mslot[mb + r] = (uint32_t)(base + A.list[top - r]);
  }
}

// start of every key's run in the sorted keys: packed[c] = first j with
// key[j] >= c, for c = 0..n_cells (packed[n_cells] = n); each run boundary
// fills the starts of the keys it skips
__global__ __launch_bounds__(256) void k_run_starts(const uint32_t *key, uint64_t n, uint32_t n_cells,
                                                    uint64_t *packed) {
  const uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= n) return;
  const uint32_t k = key[j] < n_cells ? key[j] : n_cells;
  const uint32_t prev = j ? (key[j - 1] < n_cells ? key[j - 1] : n_cells) : 0u;
  const uint32_t from = j ? prev + 1 : 0u;
  if (j == 0 || k != prev)
    for (uint32_t c = from; c <= k; ++c) packed[c] = j;
  if (j == n - 1)
    for (uint32_t c = k + 1; c <= n_cells; ++c) packed[c] = n;
}

__device__ __forceinline__ void copy_particle(const State &s, const State &d, uint64_t from, uint64_t to, uint32_t mm) {
  if (s.b32)
    d.b32[to] = s.b32[from];
  else
    d.b64[to] = s.b64[from];
  copy_levels(s, from, d, to);
  if (s.rot) d.rot[to] = s.rot[from];
  d.px[to] = s.px[from];
  d.py[to] = s.py[from];
  d.pz[to] = s.pz[from];
}

// per new cell k: the split of its run of sorted list entries at the first
// entry from a slot above off[k] (by bisection: the run is in slot order),
// its count (capped at its capacity, which raises the capacity error; the
// place pass stores it) and where its particles go (RebinDest). One thread
// per cell.
__global__ __launch_bounds__(256) void k_rebin_cells(RebinArgs A) {
  const uint64_t k = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k >= A.n_cells) return;
  const uint64_t base = A.off[k];
  uint64_t lo = 0, hi = 0;
  if (A.m) {
    lo = A.packed[k];
    hi = A.packed[k + 1];
  }
  uint64_t a = lo, b = hi;
  while (a < b) {
    const uint64_t mid = (a + b) >> 1;
    if (A.mslot[A.sidx[mid]] < base)
      a = mid + 1;
    else
      b = mid;
  }
  const uint32_t ns = A.n_stay[k], cap = A.cap[k];
  const uint64_t want = (hi - lo) + ns;
  const uint32_t total = (uint32_t)(want > cap ? cap : want);
  if (want > cap) atomicOr(A.err, kErrCapacity);
  RebinDest d;
  d.first = base - lo;
  d.split = a;
  d.end = base + total;
  d.below = (uint32_t)(a - lo);
  d.ns = ns;
  A.dest[k] = d;
}

// Cells of up to kStageSlots old slots are staged through LDS by the place
// pass; an output entry of kNoSlot is dropped (capacity overflow).
constexpr uint32_t kStageSlots = 384;
constexpr uint64_t kNoSlot = ~0ull;

// New slot of every list entry (by its sorted position j: its new cell's
// destination record gives it), ~0u when the entry is dropped (an
// admission that left again, or a slot past its new cell's capacity).
// Slots of the spatial mode fit 32 bits below ~0u. One thread per sorted
// entry; the writes scatter by list index, so that the place pass reads
// its movers' slots in list order.
constexpr uint32_t kNoSlot32 = 0xFFFFFFFFu;
__global__ __launch_bounds__(256) void k_rebin_slots(RebinArgs A) {
  const uint64_t j = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (j >= A.m) return;
  const uint32_t k = A.skey[j];
  uint32_t slot = kNoSlot32;
  if (k < A.n_cells) {
    const RebinDest d = A.dest[k];
    const uint64_t to = d.first + j + (j >= d.split ? d.ns : 0u);
    if (to < d.end) slot = (uint32_t)to;
  }
  A.slot[HCAO_IDX(A.sidx[j], A.m, A.err)] = slot;
}

__device__ __forceinline__ uint64_t entry_slot(const RebinArgs &A, uint64_t m) {
  const uint32_t v = A.slot[m];
  return v == kNoSlot32 ? kNoSlot : (uint64_t)v;
}

// one particle to its new slot with the step's move applied (the same
// arithmetic as the move pass)
__device__ __forceinline__ void copy_moved(const RebinArgs &A, uint64_t from, uint64_t to) {
  const State &s = A.src, &d = A.dst;
  const BodyOf<double> b = load_body(s, from);
  double vx = b.v.x, vy = b.v.y, vz = b.v.z;
  double x = s.px[from], y = s.py[from], z = s.pz[from];
  bool flip = false;
  move_particle(x, y, z, vx, vy, vz, A.dt, A.len, A.periodic, A.open, flip);
  store_body(d, to, vx, vy, vz, b.sp);
  copy_levels(s, from, d, to);
  if (s.rot) d.rot[to] = s.rot[from];
  d.px[to] = x;
  d.py[to] = y;
  d.pz[to] = z;
}

// The place pass, pushed from the old cells: one workgroup per old cell j
// writes each of its particles, moved over the step, to its slot in the
// new cell. The order in
// every new cell is that of a stable sort of all particles by new cell:
// movers from slots below off[k], k's stayers, the other movers, the
// admissions (k_rebin_admit). The movers from j into one new cell hold
// consecutive sorted positions, hence consecutive new slots; the workgroup
// ranks its movers by new slot, so that its writes form runs. A cell of up
// to kStageSlots old slots is read whole, in slot order, into registers
// (issued first, so that the loads overlap the ranking) and then LDS, and
// written from there in output order; its level rows (4 to 32 bytes each)
// follow as one run of dwords, read in order and written dword by dword in
// output order. Larger cells copy each particle directly. The old count is
// read before the new one is written (only this workgroup touches cnt[j]).
// Workgroups go to the eight XCDs in turn; each XCD takes kPushRun
// consecutive cells at a time, since movers go to neighbouring cells, whose
// lines are then in the same L2, and so that the XCDs together work through
// one region of the grid (67.1 M particles in fp64: 3.10 ms with an eighth
// of the grid per XCD, 2.98 with runs of 256 cells). A grid's last, incomplete
// round of runs is shared out evenly.
constexpr uint32_t kPushRun = 256;
__global__ __launch_bounds__(256) void k_rebin_push(RebinArgs A) {
  constexpr uint32_t kPer = (kStageSlots + 255u) / 256u;  // staged slots per thread
  constexpr uint32_t kPerL = (kStageSlots * (kMaxModes / 2) + 255u) / 256u;  // staged level dwords per thread
  // positions (rows 0-2) and velocities (rows 3-5: bits of a double, or of
  // a float); mover new slots while ranking, level rows after the fields
  __shared__ uint64_t s_pv[6][kStageSlots];
  static_assert(kStageSlots * (kMaxModes / 2) * 4 <= sizeof(s_pv), "level rows must fit the staging rows");
  uint64_t(*s_pos)[kStageSlots] = s_pv;
  uint64_t(*s_vel)[kStageSlots] = s_pv + 3;
  __shared__ uint64_t s_rot[kStageSlots];
  __shared__ uint64_t s_to[kStageSlots];
  __shared__ uint16_t s_src[kStageSlots], s_msrc[kStageSlots];
  __shared__ uint8_t s_sp[kStageSlots];
  const uint32_t per_xcd = gridDim.x >> 3;
  const uint32_t xcd = blockIdx.x & 7u, turn = blockIdx.x >> 3, whole = per_xcd / kPushRun * kPushRun;
  const uint32_t j = turn < whole ? (turn / kPushRun * 8u + xcd) * kPushRun + turn % kPushRun
                                  : whole * 8u + xcd * (per_xcd - whole) + (turn - whole);
  if (j >= A.n_cells) return;
  const uint32_t tid = threadIdx.x;
  const uint64_t base = A.off[j], mb = A.mbase[j];
  const uint32_t ns = A.n_stay[j], nm = (uint32_t)(A.mbase[j + 1] - mb), n_old = A.cnt[j];
  const RebinDest own = A.dest[j];
  const uint32_t n_out = ns + nm;
  const State &S = A.src, &D = A.dst;
  if (n_old > kStageSlots) {
    for (uint32_t t = tid; t < n_out; t += blockDim.x) {
      uint64_t from, to;
      if (t < ns) {
        from = base + A.list[base + t];
        to = base + own.below + t;
        if (to >= own.end) continue;
      } else {
        const uint64_t m = HCAO_IDX(mb + (t - ns), A.m, A.err);
        from = A.mslot[m];
        to = entry_slot(A, m);
        if (to == kNoSlot) continue;
      }
      copy_moved(A, HCAO_IDX(from, S.n_slots, A.err), HCAO_IDX(to, D.n_slots, A.err));
    }
  } else {
    const bool f32 = S.b32 != nullptr, rot = S.rot != nullptr;
    uint64_t rp[kPer][3], rv[kPer][3], rr[kPer];
    uint8_t rs[kPer];
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
      const uint32_t i = tid + 256u * q;
      if (i < n_old) {
        const uint64_t g = base + i;
        rp[q][0] = reinterpret_cast<const uint64_t *>(S.px)[g];
        rp[q][1] = reinterpret_cast<const uint64_t *>(S.py)[g];
        rp[q][2] = reinterpret_cast<const uint64_t *>(S.pz)[g];
        if (f32) {
          const uint4 b = reinterpret_cast<const uint4 *>(S.b32)[g];
          rv[q][0] = b.x;
          rv[q][1] = b.y;
          rv[q][2] = b.z;
          rs[q] = (uint8_t)b.w;
        } else {
          const Body64 b = S.b64[g];
          rv[q][0] = (uint64_t)__double_as_longlong(b.x);
          rv[q][1] = (uint64_t)__double_as_longlong(b.y);
          rv[q][2] = (uint64_t)__double_as_longlong(b.z);
          rs[q] = (uint8_t)b.sp;
        }
        rr[q] = rot ? reinterpret_cast<const uint64_t *>(S.rot)[g] : 0u;
      }
    }
    // the step's move (positions, and velocities a specular face reversed);
    // a particle that left through an open face is in no list
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
      if (tid + 256u * q < n_old) {
        double x = __longlong_as_double((long long)rp[q][0]), y = __longlong_as_double((long long)rp[q][1]),
               z = __longlong_as_double((long long)rp[q][2]);
        double vx, vy, vz;
        if (f32) {
          vx = (double)__uint_as_float((uint32_t)rv[q][0]);
          vy = (double)__uint_as_float((uint32_t)rv[q][1]);
          vz = (double)__uint_as_float((uint32_t)rv[q][2]);
        } else {
          vx = __longlong_as_double((long long)rv[q][0]);
          vy = __longlong_as_double((long long)rv[q][1]);
          vz = __longlong_as_double((long long)rv[q][2]);
        }
        bool flip = false;
        move_particle(x, y, z, vx, vy, vz, A.dt, A.len, A.periodic, A.open, flip);
        rp[q][0] = (uint64_t)__double_as_longlong(x);
        rp[q][1] = (uint64_t)__double_as_longlong(y);
        rp[q][2] = (uint64_t)__double_as_longlong(z);
        if (flip) {
          if (f32) {
            rv[q][0] = __float_as_uint((float)vx);
            rv[q][1] = __float_as_uint((float)vy);
            rv[q][2] = __float_as_uint((float)vz);
          } else {
            rv[q][0] = (uint64_t)__double_as_longlong(vx);
            rv[q][1] = (uint64_t)__double_as_longlong(vy);
            rv[q][2] = (uint64_t)__double_as_longlong(vz);
          }
        }
      }
    }
    // the cell's level rows as one run of n_old * L dwords, loaded in order
    // (lane t takes dwords t, t + 256, ...)
    const uint32_t L = S.lrow / 2u, n_lv = n_old * L;
    const uint32_t *lsrc = reinterpret_cast<const uint32_t *>(S.lvl) + base * L;
    uint32_t rl[kPerL];
#pragma unroll
    for (uint32_t q = 0; q < kPerL; ++q) {
      const uint32_t f = tid + 256u * q;
      rl[q] = f < n_lv ? lsrc[f] : 0u;
    }
    // output entries: the stayers in slot order, then the movers ranked by
    // new slot (dropped movers, kNoSlot, last)
    for (uint32_t t = tid; t < ns; t += blockDim.x) {
      const uint64_t to = base + own.below + t;
      s_src[t] = (uint16_t)A.list[base + t];
      s_to[t] = to < own.end ? HCAO_IDX(to, D.n_slots, A.err) : kNoSlot;
    }
    uint64_t *s_mto = s_pos[0];
    for (uint32_t r = tid; r < nm; r += blockDim.x) {
      const uint64_t m = HCAO_IDX(mb + r, A.m, A.err);
      const uint64_t to = entry_slot(A, m);
      s_mto[r] = to == kNoSlot ? kNoSlot : HCAO_IDX(to, D.n_slots, A.err);
      s_msrc[r] = (uint16_t)(A.mslot[m] - base);
    }
    __syncthreads();
    for (uint32_t r = tid; r < nm; r += blockDim.x) {
      const uint64_t me = s_mto[r];
      uint32_t rank = 0;
      for (uint32_t u = 0; u < nm; ++u) {
        const uint64_t o = s_mto[u];
        rank += (o < me || (o == me && u < r)) ? 1u : 0u;
      }
      s_src[ns + rank] = s_msrc[r];
      s_to[ns + rank] = me;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < kPer; ++q) {
      const uint32_t i = tid + 256u * q;
      if (i < n_old) {
        for (int a = 0; a < 3; ++a) {
          s_pos[a][i] = rp[q][a];
          s_vel[a][i] = rv[q][a];
        }
        s_rot[i] = rr[q];
        s_sp[i] = rs[q];
      }
    }
    __syncthreads();
    for (uint32_t w = tid; w < n_out; w += blockDim.x) {
      const uint64_t to = s_to[w];
      if (to == kNoSlot) continue;
      const uint32_t i = s_src[w];
      reinterpret_cast<uint64_t *>(D.px)[to] = s_pos[0][i];
      reinterpret_cast<uint64_t *>(D.py)[to] = s_pos[1][i];
      reinterpret_cast<uint64_t *>(D.pz)[to] = s_pos[2][i];
      if (f32)
        reinterpret_cast<uint4 *>(D.b32)[to] =
            make_uint4((uint32_t)s_vel[0][i], (uint32_t)s_vel[1][i], (uint32_t)s_vel[2][i], s_sp[i]);
      else
        D.b64[to] = Body64{__longlong_as_double((long long)s_vel[0][i]), __longlong_as_double((long long)s_vel[1][i]),
                           __longlong_as_double((long long)s_vel[2][i]), s_sp[i]};
      if (rot) reinterpret_cast<uint64_t *>(D.rot)[to] = s_rot[i];
    }
    // level rows through LDS (over the staged positions and velocities, read
    // for the last time above), written dword by dword in output order, so
    // that reads and writes of a wave are runs of consecutive dwords:
    // output dword f is dword f mod L of entry f / L (exact as f * ceil(2^16
    // / L) >> 16 for f <= 3072, L <= 8)
    __syncthreads();
    uint32_t *s_lv = reinterpret_cast<uint32_t *>(&s_pv[0][0]);
#pragma unroll
    for (uint32_t q = 0; q < kPerL; ++q) {
      const uint32_t f = tid + 256u * q;
      if (f < n_lv) s_lv[f] = rl[q];
    }
    __syncthreads();
    uint32_t *ldst = reinterpret_cast<uint32_t *>(D.lvl);
    const uint32_t inv = (65536u + L - 1u) / L;
    for (uint32_t f = tid; f < n_out * L; f += blockDim.x) {
      const uint32_t w = (f * inv) >> 16, d = f - w * L;
      const uint64_t to = s_to[w];
      if (to != kNoSlot) ldst[to * L + d] = s_lv[(uint32_t)s_src[w] * L + d];
    }
  }
  __syncthreads();  // every wave has read the old count
  if (tid == 0) A.cnt[j] = (uint32_t)(own.end - base);
}

// the admissions of the step (list entries m_real .. m - 1, staged in ins in
// the order made): one thread each; one that left again (key n_cells) is
// dropped
__global__ __launch_bounds__(256) void k_rebin_admit(RebinArgs A) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const uint64_t m = A.m_real + i;
  if (m >= A.m) return;
  const uint64_t to = entry_slot(A, m);
  if (to == kNoSlot) return;
  copy_particle(A.ins, A.dst, HCAO_IDX(A.mslot[m] - A.tot, A.ins.n_slots, A.err), HCAO_IDX(to, A.dst.n_slots, A.err),
                A.mm);
}

}  // namespace

// ---------------------------------------------------------------------------
// launch wrappers (host side)
// ---------------------------------------------------------------------------
// the joint sampler's part of step_lds_bytes
size_t step_joint_lds_bytes(const Tables &T, int block) {
  return T.sampler_scratch & 2u ? sizeof(JointJob) * (size_t)block : 0;
}

size_t step_lds_bytes(const Tables &T, uint32_t max_cells, int block) {
  const uint32_t ns = T.n_species, nr = T.n_reactions;
  size_t b = sizeof(SpeciesTab) * ns + sizeof(PairTab) * ns * ns + sizeof(ReactionTab) * nr + 8 * (size_t)(T.n_levels ? T.n_levels : 1);
  b += sizeof(CellHdr) * max_cells + 2 * 8 * (size_t)(8 + nr) * max_cells;
  b += (size_t)2 * ((T.sampler_scratch ? 2 : 0) + 3) * (T.max_modes ? T.max_modes : 1) * block;
  b = ((b + 7) & ~(size_t)7) + step_joint_lds_bytes(T, block);
  return (b + 15) & ~(size_t)15;
}

template <bool MIX, int EX>
static const void *step_kernel(int block) {
  switch (block) {
    case 64: return (const void *)k_step<64, MIX, EX>;
    case 128: return (const void *)k_step<128, MIX, EX>;
    case 256: return (const void *)k_step<256, MIX, EX>;
    case 512: return (const void *)k_step<512, MIX, EX>;
    case 1024:
      if constexpr (EX == 0) return (const void *)k_step<1024, MIX, EX>;
      return nullptr;
    default: return nullptr;
  }
}

// Step workgroups of this size that a CU holds at once (0: not launchable).
// LDS is given out in pieces of 1,280 bytes (160 KB / 128), which the
// occupancy query does not count.
int step_blocks_per_cu(size_t lds, int block, bool mixed, int level) {
  const void *f = level >= 2 ? (mixed ? step_kernel<true, 2>(block) : step_kernel<false, 2>(block))
                  : level == 1 ? (mixed ? step_kernel<true, 1>(block) : step_kernel<false, 1>(block))
                               : (mixed ? step_kernel<true, 0>(block) : step_kernel<false, 0>(block));
  int n = 0;
  hipFuncAttributes at{};
  if (!f || hipFuncGetAttributes(&at, f) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, block, lds) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  constexpr size_t kPiece = 1280, kPieces = 128;
  return std::min(n, (int)(kPieces / ((at.sharedSizeBytes + lds + kPiece - 1) / kPiece)));
}

template <bool MIX, int EX>
static hipError_t launch_step_t(const StepArgs &a, size_t lds, int block, uint32_t n_groups, hipStream_t s) {
  switch (block) {
    case 64: hipLaunchKernelGGL((k_step<64, MIX, EX>), dim3(n_groups), dim3(64), lds, s, a); break;
    case 128: hipLaunchKernelGGL((k_step<128, MIX, EX>), dim3(n_groups), dim3(128), lds, s, a); break;
    case 256: hipLaunchKernelGGL((k_step<256, MIX, EX>), dim3(n_groups), dim3(256), lds, s, a); break;
    case 512: hipLaunchKernelGGL((k_step<512, MIX, EX>), dim3(n_groups), dim3(512), lds, s, a); break;
    case 1024:
      if constexpr (EX == 0) {
        hipLaunchKernelGGL((k_step<1024, MIX, EX>), dim3(n_groups), dim3(1024), lds, s, a);
        break;
      }
      return hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// level 0: the collision step; 1: and positions (spatial mode); 2: and the
// exact sampler and rotors (positions included)
hipError_t launch_step(const StepArgs &a, size_t lds, int block, bool mixed, int level, uint32_t n_groups,
                       hipStream_t s) {
  if (n_groups == 0) return hipSuccess;
  if (level >= 2)
    return mixed ? launch_step_t<true, 2>(a, lds, block, n_groups, s)
                 : launch_step_t<false, 2>(a, lds, block, n_groups, s);
  if (level == 1)
    return mixed ? launch_step_t<true, 1>(a, lds, block, n_groups, s)
                 : launch_step_t<false, 1>(a, lds, block, n_groups, s);
  return mixed ? launch_step_t<true, 0>(a, lds, block, n_groups, s)
               : launch_step_t<false, 0>(a, lds, block, n_groups, s);
}

// Fixed device array for the allocation-free step (hcao_step_static): the
// work lists, pair flags, pair energy defects and products staging of one
// step call. Host code never passes the array's name to a kernel: it uses
// the device address that static_scratch_address() returns for the current
// device.
static __device__ __align__(256) unsigned char scratch[kStaticArrayBytes];

hipError_t static_scratch_address(void **ptr) { return hipGetSymbolAddress(ptr, HIP_SYMBOL(scratch)); }

hipError_t launch_advance(uint32_t *step, uint32_t n, hipStream_t s) {
  hipLaunchKernelGGL(k_advance, dim3(1), dim3(64), 0, s, step, n);
  return hipGetLastError();
}

// the dynamic LDS limit of every k_step instantiation the launcher can pick
// (block sizes 64..512, both precisions, levels 0..2, and 1,024 at level 0)
template <bool MIX, int EX>
static hipError_t set_lds_limit_level(int bytes) {
  hipError_t e = hipSuccess;
  for (int block = 64; block <= 1024; block *= 2) {
    const void *f = step_kernel<MIX, EX>(block);
    const hipError_t r =
        f ? hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, bytes) : hipSuccess;
    if (r != hipSuccess) e = r;
  }
  return e;
}

hipError_t set_step_lds_limit(size_t bytes) {
  const int b = (int)bytes;
  const hipError_t r[] = {set_lds_limit_level<false, 0>(b), set_lds_limit_level<true, 0>(b),
                          set_lds_limit_level<false, 1>(b), set_lds_limit_level<true, 1>(b),
                          set_lds_limit_level<false, 2>(b), set_lds_limit_level<true, 2>(b)};
  for (hipError_t e : r)
    if (e != hipSuccess) return e;
  return hipSuccess;
}

hipError_t launch_init(const Tables *tab, const double *lev, const State &st, const uint64_t *off,
                       const uint32_t *counts, const double *tt, const double *tv, uint64_t seed, uint32_t n_cells,
                       const uint32_t grid[3], const double len[3], hipStream_t s) {
  InitArgs a{tab, lev, st, off, counts, tt, tv, seed, n_cells, grid[0], grid[1], grid[2], {len[0], len[1], len[2]}};
  hipLaunchKernelGGL(k_init, dim3(n_cells), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_cell_init(const Tables *tab, const State &st, const CellArrays &cells, uint32_t n_cells,
                            hipStream_t s) {
  CellInitArgs a{tab, st, cells};
  hipLaunchKernelGGL(k_cell_init, dim3(n_cells), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_moments(const Tables *tab, const double *lev, const State &st, const uint64_t *off,
                          const uint32_t *cnt, const uint32_t *cap, double *out, uint32_t n_cells, uint32_t ns,
                          bool large, const uint32_t *list, uint32_t n_list, hipStream_t s) {
  MomentArgs a{tab, lev, st, off, cnt, out, n_cells, cap, large ? nullptr : list};
  if (n_cells == 0) return hipSuccess;
  const dim3 waves((n_cells + 3u) / 4u);
  const uint32_t groups = large ? n_cells : (list ? n_list : 0u);
  if (ns <= 6) {
    if (!large) hipLaunchKernelGGL((k_moments<6, 1>), waves, dim3(256), 0, s, a);
    if (groups) hipLaunchKernelGGL((k_moments<6, 8>), dim3(groups), dim3(512), 0, s, a);
  } else {
    if (!large) hipLaunchKernelGGL((k_moments<kMaxSpecies, 1>), waves, dim3(256), 0, s, a);
    if (groups) hipLaunchKernelGGL((k_moments<kMaxSpecies, 8>), dim3(groups), dim3(512), 0, s, a);
  }
  return hipGetLastError();
}

hipError_t launch_moments_sum(const double *in, const double *weight, const double *defect, double *out,
                              uint32_t n_cells, uint32_t w, uint32_t ns, uint32_t blocks, hipStream_t s) {
  MomentSumArgs a{in, weight, defect, out, n_cells, w, ns};
  hipLaunchKernelGGL(k_moments_sum, dim3(blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_thermometer(const Tables *tab, const double *lev, const double *mean, const double *in, double *t,
                              uint32_t n_cells, uint32_t w, uint32_t ns, const uint32_t *same, hipStream_t s) {
  ThermoArgs a{tab, lev, mean, in, t, n_cells, w, ns, {}};
  for (uint32_t k = 0; k < ns; ++k) a.same[k] = same[k];
  const uint64_t n = (uint64_t)n_cells * ns;
  hipLaunchKernelGGL(k_thermometer, dim3((unsigned)((n + 63) / 64)), dim3(64), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_reaction_sum(const unsigned long long *ctr, uint32_t n_cells, uint32_t nr, unsigned long long *out,
                               hipStream_t s) {
  const uint32_t blocks = (n_cells + 255u) / 256u;
  hipLaunchKernelGGL(k_reaction_sum, dim3(blocks < 256u ? blocks : 256u), dim3(256), 0, s, ctr, n_cells, nr, out);
  return hipGetLastError();
}

hipError_t launch_pack(const State &st, const uint64_t *off, const uint64_t *start, const uint32_t *cnt, uint8_t *sp,
                       double *vel, uint16_t *lvl, uint64_t p0, uint64_t p1, uint32_t c0, uint32_t c1, uint32_t mm,
                       hipStream_t s) {
  if (c1 <= c0 || p1 <= p0) return hipSuccess;
  PackArgs a{st, off, start, cnt, sp, vel, lvl, p0, p1, c0, mm};
  hipLaunchKernelGGL(k_pack, dim3(c1 - c0), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_slots_out(const State &st, uint64_t first, uint64_t n, uint32_t mm, double *vel, uint8_t *sp,
                            uint16_t *lvl, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_slots_out, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, st, first, n, mm, vel, sp, lvl);
  return hipGetLastError();
}

hipError_t launch_slots_in(const State &st, uint64_t first, uint64_t n, uint32_t mm, const double *vel,
                           const uint8_t *sp, const uint16_t *lvl, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_slots_in, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, st, first, n, mm, vel, sp, lvl);
  return hipGetLastError();
}

uint64_t scan_tmp_entries(uint64_t n) { return (n + kScanChunk - 1) / kScanChunk + 1; }

// exclusive scan; tmp holds scan_tmp_entries(n) entries
hipError_t launch_scan_u32(const uint32_t *in, uint64_t *out, uint64_t n, uint64_t *tmp, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const uint64_t nb = (n + kScanChunk - 1) / kScanChunk;
  if (nb > 0x7FFFFFFFull) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_scan_chunk, dim3((unsigned)nb), dim3(256), 0, s, in, out, n, tmp);
  if (nb > 1) hipLaunchKernelGGL(k_scan_add, dim3((unsigned)(nb - 1)), dim3(256), 0, s, out, n, tmp);
  return hipGetLastError();
}

hipError_t launch_load_check(const Tables *tab, const uint32_t *cell, const uint8_t *sp, const double *vel,
                             const uint16_t *lvl, uint64_t n, uint32_t n_cells, uint32_t *count, uint32_t *err,
                             hipStream_t s) {
  LoadArgs a{tab, cell, sp, vel, lvl, n, n_cells, count, err};
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_load_check, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

// Stable sort of (key, index) by the low key_bits bits of the key; buffers
// of n entries each, hist and offs of sort_hist_entries(n) entries (u32,
// u64). The passes take digits of equal width up to 9 bits: one pass up to
// 9 bits, two up to 18, three up to 27 (19 bits: three of 7; two of 10 cost
// more in their larger histogram scans). Result in
// keys/idx or the tmp buffers (ping-pong handled here; returns which buffer
// holds the result).
hipError_t launch_sort(uint32_t *keys, uint32_t *idx, uint32_t *keys_tmp, uint32_t *idx_tmp, uint32_t *hist,
                       uint64_t *offs, uint64_t *scan_tmp, uint64_t n, uint32_t key_bits, hipStream_t s,
                       bool &result_in_tmp) {
  result_in_tmp = false;
  if (n == 0) return hipSuccess;
  const uint32_t tiles = (uint32_t)((n + kSortTile - 1) / kSortTile);
  if (key_bits == 0) {  // one key: nothing to sort
    hipLaunchKernelGGL(k_iota, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, idx, n);
    return hipGetLastError();
  }
  uint32_t *kin = keys, *iin = idx, *kout = keys_tmp, *iout = idx_tmp;
  if (key_bits > 32) return hipErrorInvalidValue;
  const uint32_t passes = (key_bits + kSortMaxBits - 1) / kSortMaxBits;
  const uint32_t bits = passes ? (key_bits + passes - 1) / passes : 0;
  for (uint32_t shift = 0; shift < key_bits; shift += bits) {
    hipLaunchKernelGGL(k_sort_hist, dim3(tiles), dim3(kSortBlock), 0, s, kin, n, shift, bits, hist, tiles);
    const hipError_t e = launch_scan_u32(hist, offs, (uint64_t)(1u << bits) * tiles, scan_tmp, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_sort_scatter, dim3(tiles), dim3(kSortBlock), 0, s, kin, shift ? iin : nullptr, kout, iout, n,
                       shift, bits, offs, tiles);
    uint32_t *tk = kin, *ti = iin;
    kin = kout;
    iin = iout;
    kout = tk;
    iout = ti;
    result_in_tmp = !result_in_tmp;
  }
  return hipGetLastError();
}

uint64_t sort_tiles(uint64_t n) { return (n + kSortTile - 1) / kSortTile; }
uint64_t sort_hist_entries(uint64_t n) { return (uint64_t)kSortMaxBins * sort_tiles(n); }

hipError_t launch_move(const MoveArgs &a, hipStream_t s) {
  if (a.n_cells == 0) return hipSuccess;
  if (!a.off || !a.cnt || !a.cap || !a.key || !a.list || !a.n_stay || !a.n_move || !a.st.px || !a.st.py || !a.st.pz)
    return hipErrorInvalidValue;
  const uint64_t small = a.st.b32 ? kMoveSmall32 : kMoveSmall64;
  const dim3 fours((a.n_cells + 3u) / 4u);
  if (a.n_cells < kMoveManyCells || a.particles > small * a.n_cells)
    hipLaunchKernelGGL((k_move<1, true>), dim3(a.n_cells), dim3(256), 0, s, a);
  else if (a.largest > kMoveBig)
    hipLaunchKernelGGL((k_move<4, true>), fours, dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((k_move<4, false>), fours, dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_list_movers(const RebinArgs &a, hipStream_t s) {
  if (a.n_cells == 0 || a.m == 0) return hipSuccess;
  if (!a.off || !a.cap || !a.key || !a.list || !a.n_move || !a.mbase || !a.mkey || !a.mslot)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_list_movers, dim3((a.n_cells + 3u) / 4u), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_inflow_count(const InflowArgs &a, hipStream_t s) {
  const uint64_t n = (uint64_t)a.face_base[6] * a.n_species;
  if (n == 0) return hipSuccess;
  if (!a.tab || !a.weight || !a.rem || !a.count || !a.err) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_inflow_count, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_inflow_make(const InflowArgs &a, hipStream_t s) {
  const uint64_t n = a.n_ins;
  if (n == 0 || a.face_base[6] == 0 || a.n_species == 0) return hipSuccess;
  if (!a.tab || !a.lev || !a.count || !a.ibase || !a.mbase || !a.mkey || !a.mslot || !a.flux || !a.err ||
      !a.ins.lvl || !a.ins.px || !a.ins.py || !a.ins.pz || (!a.ins.b64 && !a.ins.b32))
    return hipErrorInvalidValue;
  InflowArgs b = a;
  if (b.n_levels > kInflowLevels) b.n_levels = 0;
  const size_t lds = b.n_species * (sizeof(SpeciesTab) + kMaxModes * 8) + (size_t)b.n_levels * 8;
  const uint32_t lanes = n <= kInflowEight ? 8u : n <= kInflowFour ? 4u : 1u;
  const dim3 grid((unsigned)((n * lanes + 63) / 64));
  if (lanes == 8)
    hipLaunchKernelGGL(k_inflow_make<8>, grid, dim3(64), lds, s, b);
  else if (lanes == 4)
    hipLaunchKernelGGL(k_inflow_make<4>, grid, dim3(64), lds, s, b);
  else
    hipLaunchKernelGGL(k_inflow_make<1>, grid, dim3(64), lds, s, b);
  return hipGetLastError();
}

// run starts of the sorted list, the new cells' counts and destinations,
// every list entry's new slot, then the place pass from the old cells and
// the admissions
hipError_t launch_rebin_place(const RebinArgs &a, hipStream_t s) {
  if (a.n_cells == 0) return hipSuccess;
  if (!a.off || !a.cap || !a.list || !a.n_stay || !a.mbase || !a.packed || !a.dest || !a.cnt || !a.err ||
      a.m_real > a.m || (a.m && (!a.skey || !a.sidx || !a.mslot || !a.slot)))
    return hipErrorInvalidValue;
  if (a.m)
    hipLaunchKernelGGL(k_run_starts, dim3((unsigned)((a.m + 255) / 256)), dim3(256), 0, s, a.skey, a.m, a.n_cells,
                       a.packed);
  hipLaunchKernelGGL(k_rebin_cells, dim3((a.n_cells + 255u) / 256u), dim3(256), 0, s, a);
  if (a.m) hipLaunchKernelGGL(k_rebin_slots, dim3((unsigned)((a.m + 255) / 256)), dim3(256), 0, s, a);
  hipLaunchKernelGGL(k_rebin_push, dim3(((a.n_cells + 7u) / 8u) * 8u), dim3(256), 0, s, a);
  if (a.m > a.m_real)
    hipLaunchKernelGGL(k_rebin_admit, dim3((unsigned)((a.m - a.m_real + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_place(const Tables *tab, const uint32_t *sorted_cell, const uint32_t *sorted_idx,
                        const uint64_t *packed_start, const uint64_t *off, const uint8_t *sp, const double *vel,
                        const uint16_t *lvl, const double *rot, const double *pos, const State &st, uint64_t n,
                        hipStream_t s) {
  PlaceArgs a{tab, sorted_cell, sorted_idx, packed_start, off, sp, vel, lvl, rot, pos, st, n};
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(k_load_place, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace hcao
