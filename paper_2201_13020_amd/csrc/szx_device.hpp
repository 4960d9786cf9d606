// szx_device.hpp -- device-side building blocks of the SZx kernels for gfx950.
//
// Element traits, IEEE-754 totalOrder keys, the exact "a - c <= e" decision,
// the bit budget of eq. (4) with the byte shift of eq. (5), wave/group scans,
// the workgroup-wide scan, and the decoupled look-back that chains tiles of a
// single-pass device-wide prefix sum (Sec. V-B: the output offset of each
// block is the prefix sum of the bytes of the blocks before it).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "szx_layout.hpp"

namespace szx {

// A pointer read from a field descriptor in memory is typed generic, so every
// access through it would compile to flat instructions (which wait on both
// the vector-memory and the LDS counters). Descriptors only hold device
// memory: re-read the pointer's bits as a global-memory pointer, so that the
// compiler infers global accesses through it.
template <typename P>
__device__ __forceinline__ P as_global(const P& member) {
  const uint64_t raw = *reinterpret_cast<const uint64_t*>(&member);
  return (P)(__attribute__((address_space(1))) char*)raw;
}

// A pointer to memory that nothing writes while the kernel runs, re-read as a
// constant-memory pointer: a read at a wave-uniform address through it is a
// scalar load (no vector register, no wait on vector loads), also in a kernel
// that stores.
template <typename V>
__device__ __forceinline__ const V* as_constant(const V* p) {
  return (const V*)(__attribute__((address_space(4))) const char*)(uintptr_t)p;
}

constexpr int kWave = 64;
constexpr int kWG = 256;
constexpr int kWavesPerWG = kWG / kWave;
constexpr uint32_t kHeaderBytes = 96;
constexpr uint32_t kMagic = 0x4D585A53u;  // "SZXM" little-endian
constexpr uint8_t kVersion = 1;
constexpr uint8_t kRawK = 0xFF;

template <typename T>
struct Traits;

template <>
struct Traits<float> {
  using U = uint32_t;
  static constexpr int W = 32;     // bits per value
  static constexpr int E = 8;      // exponent bits
  static constexpr int BIAS = 127;
  static constexpr int BYTES = 4;
  static constexpr int KMIN = 1 + E;
};

template <>
struct Traits<double> {
  using U = uint64_t;
  static constexpr int W = 64;
  static constexpr int E = 11;
  static constexpr int BIAS = 1023;
  static constexpr int BYTES = 8;
  static constexpr int KMIN = 1 + E;
};

// Geometry of the extrema pass, by the block size b: each lane owns EPL
// consecutive values, LPB lanes share one block, a row of a 256-thread
// workgroup holds TB whole blocks. It changes no output byte.
template <typename T, int B>
struct Geo {
  static constexpr int EPL = B >= 512 ? B / 64 : 8;
  static constexpr int LPB = B / EPL;  // 1..64, divides 64
  static constexpr int TB = kWG / LPB;
  static constexpr int TILE = TB * B;  // values per row
  static_assert(LPB >= 1 && LPB <= 64 && (64 % LPB) == 0, "group must fit a wave");
};

__device__ __forceinline__ uint32_t bits_of(float v) { return __float_as_uint(v); }
__device__ __forceinline__ uint64_t bits_of(double v) { return (uint64_t)__double_as_longlong(v); }
__device__ __forceinline__ float float_from(uint32_t u) { return __uint_as_float(u); }
__device__ __forceinline__ double double_from(uint64_t u) { return __longlong_as_double((long long)u); }

template <typename T>
__device__ __forceinline__ T from_bits(typename Traits<T>::U u);
template <>
__device__ __forceinline__ float from_bits<float>(uint32_t u) { return float_from(u); }
template <>
__device__ __forceinline__ double from_bits<double>(uint64_t u) { return double_from(u); }

// Unsigned key whose order is IEEE-754 totalOrder (-0 < +0): flip all bits of
// negatives, set the sign bit of non-negatives.
template <typename U>
__device__ __forceinline__ U order_key(U u) {
  constexpr U sign = (U)1 << (sizeof(U) * 8 - 1);
  return (u & sign) ? (U)~u : (U)(u | sign);
}
template <typename U>
__device__ __forceinline__ U key_to_bits(U k) {
  constexpr U sign = (U)1 << (sizeof(U) * 8 - 1);
  return (k & sign) ? (U)(k & ~sign) : (U)~k;
}

// Keys of -max finite and +max finite: a block is all-finite iff its key range
// lies inside [kLo, kHi].
template <typename T>
struct FiniteKeys {
  using U = typename Traits<T>::U;
  static constexpr U EXPMASK = (((U)1 << Traits<T>::E) - 1) << (Traits<T>::W - 1 - Traits<T>::E);
  static constexpr U SIGN = (U)1 << (Traits<T>::W - 1);
  static constexpr U MAXF = EXPMASK - 1;          // largest finite magnitude pattern
  static constexpr U HI = MAXF | SIGN;            // key of +max
  static constexpr U LO = (U)~(MAXF | SIGN);      // key of -max
};

template <typename T>
__device__ __forceinline__ bool is_finite_bits(typename Traits<T>::U u) {
  return (u & FiniteKeys<T>::EXPMASK) != FiniteKeys<T>::EXPMASK;
}

// Exact decision of (a - c) <= e for finite a, c, e whose difference does not
// overflow. s = fl(a - c) lies on the same side of e as the exact difference
// whenever s != e (rounding is monotone); when s == e the rounding error,
// recovered exactly by Knuth's TwoSum, decides.
template <typename T>
__device__ __forceinline__ bool exact_le(T a, T c, T e) {
  const T nb = -c;
  const T s = a + nb;
  const T bv = s - a;
  const T av = s - bv;
  const T t = (a - av) + (nb - bv);
  // bitwise on purpose: no branch (branches here nest in every value of the
  // encoder's verification and cost it its scalar registers)
  return (bool)((int)(s < e) | ((int)(s == e) & (int)(t <= (T)0)));
}

// p(y) of eq. (4): unbiased exponent of |y|, with zero and subnormals at the
// smallest normal exponent.
template <typename T>
__device__ __forceinline__ int exp_of(T y) {
  using U = typename Traits<T>::U;
  const U u = bits_of(y);
  int f = (int)((u >> (Traits<T>::W - 1 - Traits<T>::E)) & ((1u << Traits<T>::E) - 1));
  f = f < 1 ? 1 : f;
  return f - Traits<T>::BIAS;
}

// Largest T value <= ed, for ed >= 0 (possibly +inf).
template <typename T>
__device__ __forceinline__ T round_down_to(double ed);
template <>
__device__ __forceinline__ float round_down_to<float>(double ed) {
  if (!(ed > 0.0)) return 0.0f;
  if (__builtin_isinf(ed)) return 3.40282346638528859812e+38f;
  float f = __double2float_rn(ed);
  if (__builtin_isinf(f)) return 3.40282346638528859812e+38f;
  while ((double)f > ed) f = __uint_as_float(__float_as_uint(f) - 1u);
  return f;
}
template <>
__device__ __forceinline__ double round_down_to<double>(double ed) {
  if (!(ed > 0.0)) return 0.0;
  if (__builtin_isinf(ed)) return 1.79769313486231570815e+308;
  return ed;
}

// Bound e from the parameters and, for REL, the global finite range (keys;
// lo > hi means no finite value was seen).
template <typename T>
__device__ __forceinline__ T bound_from(int rel, double eb, uint64_t klo, uint64_t khi) {
  using U = typename Traits<T>::U;
  double ed;
  if (!rel) {
    ed = eb;
  } else if (klo > khi || eb == 0.0) {
    ed = 0.0;
  } else {
    const T gmin = from_bits<T>(key_to_bits<U>((U)klo));
    const T gmax = from_bits<T>(key_to_bits<U>((U)khi));
    const double range = (double)gmax - (double)gmin;
    ed = eb * range;
  }
  return round_down_to<T>(ed);
}

// Kept leading bits K = min(W, 1 + E + m) (eq. (4) read as a count of kept
// bits: sign, exponent and m mantissa bits), its right shift s (eq. (5)) and
// the number of whole bytes nb = (K + s) / 8.
__device__ __forceinline__ int shift_of(int K) { return (8 - (K & 7)) & 7; }
__device__ __forceinline__ int bytes_of(int K) { return (K + shift_of(K)) >> 3; }

template <typename T>
__device__ __forceinline__ int kept_bits(int m) {
  const int k = 1 + Traits<T>::E + m;
  return k > Traits<T>::W ? Traits<T>::W : k;
}

// Mid-range and constant test of one block from its totalOrder extrema.
// Returns true for a constant block. m0 receives the mantissa budget of eq. (4)
// for a non-constant one.
template <typename T>
__device__ __forceinline__ bool classify_block(T mn, T mx, T e, T& mu, int& m0) {
  mu = (T)0.5 * mn + (T)0.5 * mx;
  if (exact_le<T>(mx, mu, e) && exact_le<T>(mu, mn, e)) {
    m0 = 0;
    return true;
  }
  T r1 = mx - mu;
  T r2 = mn - mu;
  r1 = r1 < (T)0 ? -r1 : r1;
  r2 = r2 < (T)0 ? -r2 : r2;
  const T r = r1 > r2 ? r1 : r2;
  const int m = exp_of<T>(r) - exp_of<T>(e);
  m0 = m < 0 ? 0 : m;
  return false;
}

// Mask of the top nb bytes of a word.
template <typename U>
__device__ __forceinline__ U top_bytes_mask(int nb) {
  constexpr int W = sizeof(U) * 8;
  return nb >= W / 8 ? (U)~(U)0 : (nb <= 0 ? (U)0 : (U) ~(((U)1 << (W - 8 * nb)) - 1));
}


// Leading zero bits of z; any value >= the width for z = 0 (callers cap it).
__device__ __forceinline__ uint32_t lead_zero_bits(uint32_t z) { return (uint32_t)__clz((int)z); }

__device__ __forceinline__ uint32_t byte_swap(uint32_t v) { return __builtin_bswap32(v); }
__device__ __forceinline__ uint64_t byte_swap(uint64_t v) { return __builtin_bswap64(v); }

// ---------------------------------------------------------------- scans ----

__device__ __forceinline__ int lane_id() { return (int)__lane_id(); }

// Orders a wave's LDS accesses: what its lanes stored before is there for its
// other lanes' loads after (the LDS serves a wave in order, so this only holds
// the compiler).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Inclusive sum of 32-bit values over the 64 lanes of a wave with DPP: row
// shifts by 1, 2, 4, 8 within each row of 16 lanes, then the last lane of
// rows 0 and 2 added to rows 1 and 3 (row_bcast:15) and the last lane of row 1
// to rows 2 and 3 (row_bcast:31). Lanes without a source add 0. No LDS.
__device__ __forceinline__ uint32_t wave_incl_sum_u32(uint32_t v) {
  // (unsigned: the sums wrap where they overflow)
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);  // row_shr:1
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);  // row_shr:2
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);  // row_shr:4
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);  // row_shr:8
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);  // row_bcast:15
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return v;
}

// Lane i - d within each row of 16 lanes (row_shr:d, d in {1, 2, 4, 8});
// the first d lanes of a row get 0.
__device__ __forceinline__ uint32_t dpp_shr(int d, uint32_t v) {
  switch (d) {
    case 1: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);
    case 2: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
    case 4: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
    default: return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
  }
}

// A wave-uniform value held in scalar registers.
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)v); }
__device__ __forceinline__ uint64_t uniform(uint64_t v) {
  return ((uint64_t)uniform((uint32_t)(v >> 32)) << 32) | uniform((uint32_t)v);
}

// Lanes that begin a group of LPB.
template <int LPB>
__device__ __forceinline__ constexpr uint64_t first_lanes() {
  return LPB == 64   ? 1ull
         : LPB == 32 ? 0x0000000100000001ull
         : LPB == 16 ? 0x0001000100010001ull
         : LPB == 8  ? 0x0101010101010101ull
         : LPB == 4  ? 0x1111111111111111ull
         : LPB == 2  ? 0x5555555555555555ull
                     : ~0ull;
}

// A buffer resource over bytes bytes at p: reads past them return zeros and
// stores past them do nothing, without touching memory.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
template <typename T>
__device__ __forceinline__ T buffer_value(__amdgpu_buffer_rsrc_t rs, uint32_t off);
template <>
__device__ __forceinline__ float buffer_value<float>(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, 0, 0));
}
template <>
__device__ __forceinline__ double buffer_value<double>(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  using v2u = unsigned int __attribute__((ext_vector_type(2)));
  const v2u u = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)off, 0, 0);
  return __longlong_as_double((long long)(((uint64_t)u.y << 32) | u.x));
}

// The 16 bytes that start 4 k + sh bytes into the 32 of q0 and q1 (k, sh < 4,
// k the same for every lane: a uniform branch picks the words).
__device__ __forceinline__ uint4 realign16(const uint4& q0, const uint4& q1, uint32_t k, uint32_t sh) {
  const uint32_t w[8] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w};
  switch (k) {
    case 0:
      return make_uint4(__builtin_amdgcn_alignbyte(w[1], w[0], sh), __builtin_amdgcn_alignbyte(w[2], w[1], sh),
                        __builtin_amdgcn_alignbyte(w[3], w[2], sh), __builtin_amdgcn_alignbyte(w[4], w[3], sh));
    case 1:
      return make_uint4(__builtin_amdgcn_alignbyte(w[2], w[1], sh), __builtin_amdgcn_alignbyte(w[3], w[2], sh),
                        __builtin_amdgcn_alignbyte(w[4], w[3], sh), __builtin_amdgcn_alignbyte(w[5], w[4], sh));
    case 2:
      return make_uint4(__builtin_amdgcn_alignbyte(w[3], w[2], sh), __builtin_amdgcn_alignbyte(w[4], w[3], sh),
                        __builtin_amdgcn_alignbyte(w[5], w[4], sh), __builtin_amdgcn_alignbyte(w[6], w[5], sh));
    default:
      return make_uint4(__builtin_amdgcn_alignbyte(w[4], w[3], sh), __builtin_amdgcn_alignbyte(w[5], w[4], sh),
                        __builtin_amdgcn_alignbyte(w[6], w[5], sh), __builtin_amdgcn_alignbyte(w[7], w[6], sh));
  }
}

// Inclusive sum over groups of G consecutive lanes (G a power of two <= 64).
template <int G, typename V>
__device__ __forceinline__ V group_incl_sum(V v) {
  if constexpr (G == 64 && sizeof(V) == 4) return (V)wave_incl_sum_u32((uint32_t)v);
  const int lg = lane_id() & (G - 1);
#pragma unroll
  for (int d = 1; d < G; d <<= 1) {
    const V t = __shfl_up(v, d, G);
    if (lg >= d) v += t;
  }
  return v;
}

// Minimum and maximum over groups of G consecutive lanes (all lanes of a
// group end with the group's value).
template <int G, typename U>
__device__ __forceinline__ U group_min(U v) {
#pragma unroll
  for (int d = 1; d < G; d <<= 1) {
    const U o = __shfl_xor(v, d, G);
    v = o < v ? o : v;
  }
  return v;
}
template <int G, typename U>
__device__ __forceinline__ U group_max(U v) {
#pragma unroll
  for (int d = 1; d < G; d <<= 1) {
    const U o = __shfl_xor(v, d, G);
    v = o > v ? o : v;
  }
  return v;
}

template <int G>
__device__ __forceinline__ bool group_all(bool p) {
  const uint64_t m = __ballot(p);
  if (G == 64) return m == ~0ull;
  const int base = lane_id() & ~(G - 1);
  const uint64_t gm = ((G == 64) ? ~0ull : ((1ull << G) - 1)) << base;
  return (m & gm) == gm;
}

// Exclusive prefix sum over the 256 threads of a workgroup (thread order).
// `scratch` holds kWavesPerWG entries. Returns the exclusive prefix; `total`
// receives the workgroup total. Contains barriers: call from all threads.
template <typename V>
__device__ __forceinline__ V wg_excl_sum(V v, V* scratch, V& total) {
  const V inc = group_incl_sum<kWave, V>(v);
  const int w = threadIdx.x / kWave;
  if (lane_id() == kWave - 1) scratch[w] = inc;
  __syncthreads();
  V before = 0, all = 0;
#pragma unroll
  for (int i = 0; i < kWavesPerWG; ++i) {
    const V s = scratch[i];
    before += (i < w) ? s : (V)0;
    all += s;
  }
  __syncthreads();
  total = all;
  return before + inc - v;
}

// S exclusive prefix sums over the 256 threads at once, laid end to end: the
// prefix of value s of a thread counts all values s' < s of every thread, then
// value s of the threads before it. tot[s] receives the total of value s.
// `scratch` holds S * kWavesPerWG entries. Contains barriers.
template <int S>
__device__ __forceinline__ void wg_excl_scan_multi(const uint32_t (&v)[S], uint32_t (&excl)[S],
                                                   uint32_t (&tot)[S], uint32_t* scratch) {
  uint32_t inc[S];
#pragma unroll
  for (int s = 0; s < S; ++s) inc[s] = group_incl_sum<kWave, uint32_t>(v[s]);
  const int w = threadIdx.x / kWave;
  if (lane_id() == kWave - 1) {
#pragma unroll
    for (int s = 0; s < S; ++s) scratch[s * kWavesPerWG + w] = inc[s];
  }
  __syncthreads();
  uint32_t running = 0;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < kWavesPerWG; ++i) {
      const uint32_t x = scratch[s * kWavesPerWG + i];
      before += (i < w) ? x : 0u;
      all += x;
    }
    excl[s] = running + before + inc[s] - v[s];
    tot[s] = all;
    running += all;
  }
  __syncthreads();
}

// ------------------------------------------------------ decoupled look-back -

// A tile's status word: flag in the top two bits (0 = not yet published,
// 1 = aggregate of the tile alone, 2 = inclusive prefix), value below. An
// aggregate takes at most 24 bits (the 2^23 bytes of 1024 blocks of 1024
// doubles), so a window of 256 of them adds up in 32 bits, with DPP and no LDS (sums of 64-bit
// words by lane shuffles cost 12 LDS permutes a window, one after another).
constexpr uint64_t kFlagAgg = 1ull << 62;
constexpr uint64_t kFlagIncl = 2ull << 62;
constexpr uint64_t kValueMask = (1ull << 62) - 1;

// The flag and the value share one 64-bit word, so a reader never needs any
// other memory of the writer: relaxed device-scope atomics are enough. (An
// acquire/release pair would add a write-back or an invalidation of the L2 of
// the XCD at every publish and every poll.)
// Status words live in device memory: the accesses are typed global, so that
// a look-back compiled out of line (its pointer generic) does not poll with
// flat instructions.
typedef __attribute__((address_space(1))) uint64_t global_u64;
__device__ __forceinline__ void status_store(uint64_t* p, uint64_t v) {
  __hip_atomic_store((global_u64*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t status_load(const uint64_t* p) {
  return __hip_atomic_load((global_u64*)const_cast<uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Two counts in one word, summed together: an aggregate holds the first in
// its low 17 bits (at most 1024 a tile, 64 tiles a window) and the second
// above (at most 256 a tile), an inclusive prefix the first in its low 32
// bits and the second above.
__device__ __forceinline__ uint64_t pair_aggregate(uint32_t a, uint32_t c) { return a | (c << 17); }
__device__ __forceinline__ uint64_t pair_sum(uint32_t s) { return (uint64_t)(s & 0x1FFFFu) | ((uint64_t)(s >> 17) << 32); }

// Device-wide exclusive prefix sums over tiles (decoupled look-back). A tile
// first publishes its own aggregate, then resolves its exclusive prefix from
// its predecessors' words and publishes its inclusive prefix. A tile waits
// only on lower-numbered tiles; every tile is taken by a running workgroup
// in increasing order within its ticket class and publishes its aggregate
// before it waits on anything, so every wait ends. Waits are bounded all the
// same: on exhaustion err is raised to err_code and the partial prefix is
// returned.
template <bool PAIR = false>
__device__ __forceinline__ void lookback_publish(uint64_t* status, uint32_t t, uint64_t agg) {
  if (PAIR && t == 0)
    status_store(status, kFlagIncl | pair_sum((uint32_t)agg));
  else
    status_store(status + t, (t == 0 ? kFlagIncl : kFlagAgg) | (agg & kValueMask));
}

// The 64-bit word of lane i (i wave-uniform).
__device__ __forceinline__ uint64_t lane_word(uint64_t w, int i) {
  return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(w >> 32), i) << 32) |
         (uint32_t)__builtin_amdgcn_readlane((int)w, i);
}
__device__ __forceinline__ uint32_t wave_total_u32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_sum_u32(v), 63);
}

// Called by all 64 lanes of one wave after lookback_publish; returns the same
// exclusive prefix in every lane.
template <int R = 4, bool PAIR = false>  // R: status words per lane per round (a window of 64 R tiles)
__device__ __noinline__ uint64_t lookback_resolve(uint64_t* status, uint32_t t, uint64_t agg,
                                                  uint32_t* err, uint32_t err_code) {
  const int lane = lane_id();
  if (t == 0) return 0;
  uint64_t excl = 0;
  int64_t base = (int64_t)t - 1;
  uint32_t spins = 0;
  for (;;) {
    uint64_t w[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
      // every lane loads (word 0 before the first tile, replaced below): a load
      // in a branch would wait for the one before it
      const int64_t j = base - (k * kWave + lane);
      w[k] = status_load(status + (j >= 0 ? j : 0));
    }
#pragma unroll
    for (int k = 0; k < R; ++k) w[k] = base - (k * kWave + lane) >= 0 ? w[k] : kFlagIncl;
    bool done = false, retry = false;
    int consumed = 0;
#pragma unroll
    for (int k = 0; k < R; ++k) {
      if (done || retry) continue;
      const uint64_t flag = w[k] >> 62;
      const uint64_t incl = __ballot(flag == 2);
      const uint64_t inval = __ballot(flag == 0);
      const int first = incl ? (int)__ffsll((long long)incl) - 1 : 64;
      const uint64_t need = first >= 63 ? ~0ull : ((2ull << first) - 1);
      if (inval & need) {
        retry = true;
        continue;
      }
      // the aggregates ahead of the inclusive word, then that word itself
      const uint32_t sum = wave_total_u32(lane < first ? (uint32_t)w[k] : 0u);
      excl += PAIR ? pair_sum(sum) : sum;
      if (first < 64) {
        excl += lane_word(w[k], first) & kValueMask;
        done = true;
      } else {
        ++consumed;
      }
    }
    if (done) break;
    base -= (int64_t)consumed * kWave;
    if (retry) {
      if (++spins > kSpinLimit) {
        if (lane == 0) atomicMax(err, err_code);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
  if (lane == 0) status_store(status + t, kFlagIncl | ((excl + (PAIR ? pair_sum((uint32_t)agg) : agg)) & kValueMask));
  return excl;
}

// Prefix sums over tiles kept by one scan workgroup, for a pass whose tiles
// are many and in flight all at once: the tiles only publish their
// aggregates; the scan workgroup reads them in tile order, 1024 words a round
// (256 a wave), and publishes every tile's inclusive prefix as soon as all
// earlier tiles have published, so a tile's own wait is one status word. (A
// decoupled look-back walks back through every tile still in flight, one
// window per round and per tile.) The tile that it waits for may be one that no
// running workgroup holds yet (the launch's later workgroups start as earlier
// ones, or another launch's, end), so its wait is bounded by far more rounds
// than a tile's: on exhaustion err is raised and it stops, and the tiles still
// waiting give up on their own bounds. Returns the sum over all tiles. A round
// is one trip to the device's coherence point: the loads go out together (none
// in a branch, where it would wait for the one before it; past the last tile
// they read the word behind it, which stays unpublished) and the sums take
// 32-bit DPP steps. (One wave that read 16 words a lane, each
// load behind a branch and spilled, and summed 64-bit words by lane shuffles
// took 6.5 us a round of 1024: the encoder of a 2 GiB float64 field, 65536
// tiles, ran 421 us and waited on it; with this 331 us.)
struct ScanShared {
  uint32_t count[2][kWavesPerWG], sum[2][kWavesPerWG];
};
__device__ __forceinline__ uint64_t scan_workgroup(uint64_t* status, uint64_t ntiles, uint32_t* err, uint32_t err_code,
                                               ScanShared& sh) {
  constexpr int R = 4;
  const int lane = lane_id();
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  uint64_t first = 0, run = 0;
  uint32_t spins = 0;
  for (uint32_t par = 0; first < ntiles; par ^= 1) {
    uint64_t* const base = status + first;
    const uint32_t left = (uint32_t)(ntiles - first < 4096u ? ntiles - first : 4096u);
    const uint32_t j0 = wave * (R * kWave) + (uint32_t)lane;
    uint64_t w[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint32_t j = j0 + (uint32_t)(k * kWave);
      w[k] = status_load(base + (j < left ? j : left));
    }
    // the wave's published words from its window's start, consecutively, and
    // their prefix sums
    uint32_t count = 0, sum = 0, incl[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
      const uint64_t pub = __ballot((w[k] >> 62) != 0);
      const uint32_t c = pub == ~0ull ? 64u : (uint32_t)__ffsll((long long)~pub) - 1u;
      incl[k] = sum + wave_incl_sum_u32((uint32_t)w[k]);
      if (count == (uint32_t)(k * kWave) && c > 0) {
        sum = (uint32_t)__builtin_amdgcn_readlane((int)incl[k], (int)c - 1);
        count += c;
      }
    }
    if (lane == 0) {
      sh.count[par][wave] = count;
      sh.sum[par][wave] = sum;
    }
    __syncthreads();  // one a round: the next round writes the other half
    uint32_t adv = 0, before = 0, total = 0;
    bool open = true, mine = true;
#pragma unroll
    for (uint32_t i = 0; i < (uint32_t)kWavesPerWG; ++i) {
      const uint32_t c = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.count[par][i]);
      const uint32_t v = (uint32_t)__builtin_amdgcn_readfirstlane((int)sh.sum[par][i]);
      if (i == wave) {
        mine = open;
        before = total;
      }
      adv += open ? c : 0u;
      total += open ? v : 0u;
      open = open && c == R * kWave;
    }
    if (mine) {
#pragma unroll
      for (int k = 0; k < R; ++k)
        if ((uint32_t)(k * kWave + lane) < count)
          status_store(base + (j0 + (uint32_t)(k * kWave)), kFlagIncl | ((run + before + incl[k]) & kValueMask));
    }
    run += total;
    first += adv;
    if (adv == 0) {
      if (++spins > kScanSpinLimit) {
        if (threadIdx.x == 0) atomicMax(err, err_code);
        break;
      }
      __builtin_amdgcn_s_sleep(2);
    } else {
      spins = 0;
    }
  }
  return run;
}

// A tile's exclusive prefix once the scan workgroup has published its inclusive
// one (the inclusive prefix less the tile's own aggregate). Bounded: on
// exhaustion ok becomes false and 0 is returned.
__device__ __forceinline__ uint64_t scan_wait(const uint64_t* status, uint32_t t, uint64_t agg, bool& ok,
                                              uint64_t first = 0) {
  // `first`: the word as read earlier by the caller (0: not read)
  if ((first >> 62) == 2) return ((first & kValueMask) - agg) & kValueMask;
  uint32_t spins = 0;
  for (;;) {
    const uint64_t w = status_load(status + t);
    if ((w >> 62) == 2) return ((w & kValueMask) - agg) & kValueMask;
    if (++spins > kSpinLimit) {
      ok = false;
      return 0;
    }
    __builtin_amdgcn_s_sleep(1);
  }
}

// The look-back with its window sized to the tiles of the scan: every status
// load is a transaction at the device's coherence point, so where many tiles
// are in flight a window of 64 (one word per lane) costs less than fewer,
// wider rounds; where few are, a window of 256 covers them in one round.
template <bool PAIR = false>
__device__ __forceinline__ uint64_t lookback_resolve_n(uint64_t* status, uint32_t t, uint64_t agg, uint32_t* err,
                                                       uint32_t err_code, uint64_t ntiles) {
  return ntiles > 512 ? lookback_resolve<1, PAIR>(status, t, agg, err, err_code)
                      : lookback_resolve<4, PAIR>(status, t, agg, err, err_code);
}

}  // namespace szx
