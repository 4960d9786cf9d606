// szx_compress.hip -- compression kernels of the SZx method for gfx950.
//
// Pipeline of one large sz_compress call, or of one batch of fields (all on the
// caller's stream; every pass is one launch over all fields of the batch, or one a
// type where that is faster; a large single call is a batch of one, with its own
// list of tiles):
//   k_stats     clears the counters, tickets and tile status words the later
//               passes use; per-block totalOrder min/max (Alg. 1 needs both
//               for mu_k); each workgroup folds its finite value range into
//               one of the field's range slots (two 64-bit atomic maxima)
//   k_classify  the absolute bound e (for the relative bound: eb times the
//               field's finite range, Sec. III footnote -- every wave folds
//               the range slots itself), then mid-range mu and constant test
//               of every block (Alg. 1), the state bits and the mu section; a
//               light single-pass prefix count of non-constant blocks gives
//               each encode tile its first rank and a single call its list of
//               tiles to encode. The field's last tile writes
//               the header (all but the mid-byte total) and the section
//               padding, and leaves the range slots zero for the next call.
//   k_encode    per non-constant block: normalise, keep K bits (eq. (4)), shift
//               (eq. (5)), verify the bound where it is not proved a priori,
//               2-bit leading-byte codes and mid bytes. Persistent workgroups
//               take tiles from interleaved ticket counters (float32 tiles of
//               all fields, then float64 tiles); each tile's output offset comes
//               from a single-pass prefix sum over the tiles (Sec. V-B) by
//               a scan workgroup, and while a tile waits for it the next tile is
//               encoded. Bytes are packed in LDS and leave in aligned 16-byte
//               stores. The stream ends there too (mid-byte total, stream
//               size): by the scan workgroup in a single call, with its field's last
//               tile in a batch.
//   Short single calls take fewer launches: one of one workgroup (k_small), or
//   k_stats and one more launch that classifies and encodes (k_mid).
//   k_finalize  the header of fields without values (only where there are any)
#include <algorithm>

#include "szx_device.hpp"
#include "szx_launch.hpp"

namespace szx {

// The stream size while a compression runs (the classification pass sets
// it, the end of the encode pass replaces it; the launch that does both, too).
constexpr uint64_t kSizePending = ~0ull;

// Field of a call, or of a batch entry, as the kernels see it (a copy with
// its pointers typed as global memory).
// BATCH: false for a single call (the descriptor is the kernel argument
// itself), true for a table in memory, else decided at run time.
enum : int { kAnyCall = -1, kSingle = 0, kBatch = 1 };
template <int BATCH = kAnyCall>
__device__ __forceinline__ FieldC field_at(const CBatch& b, uint32_t fi) {
  // (the table is only read while a batch runs: read as constant memory, it
  // comes with scalar loads also where the kernel stores in between)
  FieldC f;
  if constexpr (BATCH == kSingle)
    f = b.one;
  else if (BATCH == kBatch || b.fields)
    f = *as_constant(b.fields + fi);
  else
    f = b.one;
  f.in = as_global(f.in);
  f.out = as_global(f.out);
  f.out_size = as_global(f.out_size);
  f.ctr = as_global(f.ctr);
  f.clean = as_global(f.clean);
  f.range = as_global(f.range);
  f.ext_range = as_global(f.ext_range);
  f.parts = as_global(f.parts);
  f.stats = as_global(f.stats);
  f.plan = as_global(f.plan);
  f.enc_r0 = as_global(f.enc_r0);
  f.cls_status = as_global(f.cls_status);
  f.enc_mid = as_global(f.enc_mid);
  return f;
}
template <int BATCH = kAnyCall>
__device__ __forceinline__ uint32_t field_of(const uint32_t* map, uint64_t t) {
  if (BATCH == kSingle || (BATCH == kAnyCall && !map)) return 0u;
  return *as_constant(map + t);
}

// Load EPL consecutive values starting at element i0 (aligned to EPL); values
// at or beyond n are zero. Returns the number of valid values.
template <typename T, int EPL>
__device__ __forceinline__ int load_run(const T* __restrict__ x, uint64_t i0, uint64_t n, T (&v)[EPL]) {
  constexpr int PER16 = 16 / sizeof(T);
  if (i0 + EPL <= n) {
    const uint4* p = reinterpret_cast<const uint4*>(x + i0);
#pragma unroll
    for (int c = 0; c < EPL / PER16; ++c) {
      const uint4 u = p[c];
      if constexpr (sizeof(T) == 4) {
        v[c * 4 + 0] = __uint_as_float(u.x);
        v[c * 4 + 1] = __uint_as_float(u.y);
        v[c * 4 + 2] = __uint_as_float(u.z);
        v[c * 4 + 3] = __uint_as_float(u.w);
      } else {
        v[c * 2 + 0] = __longlong_as_double((long long)(((uint64_t)u.y << 32) | u.x));
        v[c * 2 + 1] = __longlong_as_double((long long)(((uint64_t)u.w << 32) | u.z));
      }
    }
    return EPL;
  }
  int cnt = 0;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const bool ok = i0 + i < n;
    v[i] = ok ? x[i0 + i] : (T)0;
    cnt += ok ? 1 : 0;
  }
  return cnt;
}

// Inclusive running min (MAX = false) or max over groups of G consecutive
// lanes: the group's last lane ends with the group's extremum. DPP row shifts
// for G <= 16 (no LDS), lane shuffles otherwise.
template <int G, typename U, bool MAX>
__device__ __forceinline__ U group_scan_last(U v) {
  if constexpr (G == 1) {
    return v;
  } else if constexpr (G <= 16) {
    const int lg = lane_id() & (G - 1);
#pragma unroll
    for (int d = 1; d < G; d <<= 1) {
      U o;
      if constexpr (sizeof(U) == 4) {
        o = (U)dpp_shr(d, (uint32_t)v);
      } else {
        const uint32_t lo = dpp_shr(d, (uint32_t)v), hi = dpp_shr(d, (uint32_t)(v >> 32));
        o = ((U)hi << 32) | lo;
      }
      const U m = MAX ? (o > v ? o : v) : (o < v ? o : v);
      v = lg >= d ? m : v;
    }
    return v;
  } else {
    return MAX ? group_max<G, U>(v) : group_min<G, U>(v);
  }
}

// Geometry of the encode pass: a workgroup's tile is about 32 KiB of values,
// each of its four waves a contiguous quarter of it, in SUB rows of EPL
// consecutive values a lane (whole blocks a row). Sixteen float32 values a
// lane share the per-row work (ranks, prefix sums, K and code writes) among
// twice the values of eight; sixteen doubles would not fit the registers.
template <typename T, int B>
struct EncGeo {
  static constexpr int EPL = (int)lane_values(B, sizeof(T));
  static constexpr int LPB = B / EPL;       // lanes per block
  static constexpr int GPW = kWave / LPB;   // blocks per row
  static constexpr int ROW = kWave * EPL;   // values per row
  static constexpr int TBLK = (int)enc_blocks(B, sizeof(T));
  static constexpr int WBLK = TBLK / kWavesPerWG;  // blocks per wave
  static constexpr int SUB = WBLK / GPW;    // rows per wave
  static constexpr int ROWS = SUB * kWavesPerWG;
  // the wave's LDS ring holds its worst case (every value stored whole); the
  // slack behind it, the run of the lane that crosses the ring's end
  static constexpr uint32_t RING = (uint32_t)(ROW * SUB * (int)sizeof(T));
  static constexpr uint32_t SLACK = (uint32_t)(EPL * (int)sizeof(T)) + 16u;
  static_assert(LPB >= 1 && LPB <= 64 && GPW * LPB == kWave && SUB * GPW * kWavesPerWG == TBLK, "whole rows");
  static_assert((RING & (RING - 1)) == 0, "the ring wraps by masking");
  // waves per SIMD, as the rings fit the 160 KiB of LDS: four workgroups of 32
  // KiB, or two of the 64 KiB of 1024-double blocks
  static constexpr int WAVES = RING > 8192u ? 2 : 4;
  static_assert(WAVES == (int)enc_resident(B, sizeof(T)), "as the default number of workgroups counts them");
};

// ----------------------------------------------------------------- stats ---

// Per-block totalOrder extrema (as keys) of all values over a chunk of
// kStatsChunk tiles of one field (two tiles per iteration keep more loads in
// flight), and the chunk's finite range folded into one of the field's range
// slots.
template <typename T, int B>
__device__ __forceinline__ void stats_tile(const T (&v)[Geo<T, B>::EPL], int cnt, uint64_t i0, uint64_t nblk,
                                           typename Traits<T>::U* __restrict__ stats,
                                           typename Traits<T>::U& flo, typename Traits<T>::U& fhi) {
  using U = typename Traits<T>::U;
  constexpr int EPL = Geo<T, B>::EPL, LPB = Geo<T, B>::LPB;
  U kmin = (U)~(U)0, kmax = 0;
  if (cnt == EPL) {  // every lane but the field's last partial one
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const U k = order_key<U>(bits_of(v[i]));
      kmin = k < kmin ? k : kmin;
      kmax = k > kmax ? k : kmax;
    }
  } else {
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const U k = order_key<U>(bits_of(v[i]));
      kmin = (i < cnt && k < kmin) ? k : kmin;
      kmax = (i < cnt && k > kmax) ? k : kmax;
    }
  }
  // the block's extrema gather in the group's last lane
  kmin = group_scan_last<LPB, U, false>(kmin);
  kmax = group_scan_last<LPB, U, true>(kmax);
  const uint64_t blk = i0 / B;
  const bool last = (threadIdx.x % LPB) == LPB - 1;
  if (last && blk < nblk) {
    // one store for the pair (8- or 16-byte aligned: the array starts 256-byte aligned)
    if constexpr (sizeof(U) == 4) {
      *reinterpret_cast<uint2*>(stats + 2 * blk) = make_uint2(kmin, kmax);
    } else {
      *reinterpret_cast<ulonglong2*>(stats + 2 * blk) = make_ulonglong2(kmin, kmax);
    }
  }
  // finite range: a block whose extrema are finite is finite throughout and
  // adds [kmin, kmax]; a block holding a NaN or an infinity (rare) adds its
  // finite values one by one, in every lane of its group
  const bool finite = kmin >= FiniteKeys<T>::LO && kmax <= FiniteKeys<T>::HI;
  if (last && finite && blk < nblk) {
    flo = kmin < flo ? kmin : flo;
    fhi = kmax > fhi ? kmax : fhi;
  }
  const uint64_t odd = __ballot(last && !finite && blk < nblk);
  const int gl = (lane_id() & ~(LPB - 1)) + LPB - 1;  // the group's last lane
  if ((odd >> gl) & 1ull) {
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const U u = bits_of(v[i]);
      const U k = order_key<U>(u);
      const bool fin = i < cnt && is_finite_bits<T>(u);
      flo = (fin && k < flo) ? k : flo;
      fhi = (fin && k > fhi) ? k : fhi;
    }
  }
}

// Per-block totalOrder extrema (as keys) of all values over a chunk of
// kStatsChunk tiles of one field (two tiles per iteration keep more loads in
// flight), and the chunk's finite range folded into one of the field's range
// slots -- or, on the field's first use of the workspace, stored as the
// chunk's partial.
template <typename T, int B>
__device__ __forceinline__ void stats_chunk(const FieldC& f, uint64_t c, uint64_t* s_lo, uint64_t* s_hi) {
  using U = typename Traits<T>::U;
  using G = Geo<T, B>;
  constexpr int EPL = G::EPL;
  const T* x = reinterpret_cast<const T*>(f.in);
  U* stats = reinterpret_cast<U*>(f.stats);
  U flo = (U)~(U)0, fhi = 0;
  const uint64_t ntile = cdiv(f.n, (uint64_t)G::TILE);
  const uint64_t t0 = c * kStatsChunk;
  const uint64_t t1 = std::min<uint64_t>(ntile, t0 + kStatsChunk);
  for (uint64_t t = t0; t < t1; t += 2) {
    const uint64_t i0 = t * G::TILE + (uint64_t)threadIdx.x * EPL;
    const uint64_t i1 = i0 + G::TILE;
    const bool second = t + 1 < t1;
    T v0[EPL], v1[EPL];
    const int c0 = load_run<T, EPL>(x, i0, f.n, v0);
    const int c1 = second ? load_run<T, EPL>(x, i1, f.n, v1) : 0;
    stats_tile<T, B>(v0, c0, i0, f.nblk, stats, flo, fhi);
    if (second) stats_tile<T, B>(v1, c1, i1, f.nblk, stats, flo, fhi);
  }
  flo = group_min<kWave, U>(flo);
  fhi = group_max<kWave, U>(fhi);
  const int w = threadIdx.x / kWave;
  if (lane_id() == 0) {
    s_lo[w] = flo;
    s_hi[w] = fhi;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint64_t lo = s_lo[0], hi = s_hi[0];
    for (int i = 1; i < kWavesPerWG; ++i) {
      lo = s_lo[i] < lo ? s_lo[i] : lo;
      hi = s_hi[i] > hi ? s_hi[i] : hi;
    }
    if (*f.clean != kCleanWord) {
      // lo > hi: no finite value
      *reinterpret_cast<ulonglong2*>(f.parts + 2 * c) = make_ulonglong2(lo, hi);
    } else if (lo <= hi) {  // the chunk saw a finite value
      uint64_t* slot = f.range + (c % f.nslots) * (kRangeStride / 8);
      atomicMax((unsigned long long*)slot, ~(unsigned long long)lo);
      atomicMax((unsigned long long*)slot + 1, (unsigned long long)hi);
    }
  }
}

// Every extrema workgroup (of both element types) also clears its slice of
// the words that the later passes count, publish and wait on: they run after
// this pass, and nothing in it reads them. A single call and a batch take
// separate (uniform) paths, so that each reads its descriptor with scalar
// loads: one expression choosing between the kernel argument and the table
// would read it through a generic pointer.
template <typename T, int B>
__global__ __launch_bounds__(256) void k_stats(CBatch b) {
  __shared__ uint64_t s_lo[kWavesPerWG], s_hi[kWavesPerWG];
  constexpr int DT = sizeof(T) == 4 ? 0 : 1;
  const uint64_t g = blockIdx.x;
  const uint64_t all = b.tiles_stats[0] + b.tiles_stats[1];
  for (uint64_t i = ((DT ? b.tiles_stats[0] : 0) + g) * kWG + threadIdx.x; i < b.zero_words; i += all * kWG)
    b.zero_begin[i] = 0;
  if (b.fields) {
    const FieldC f = field_at<kBatch>(b, field_of<kBatch>(b.field_stats[DT], g));
    stats_chunk<T, B>(f, g - f.base_stats, s_lo, s_hi);
  } else {
    const FieldC f = field_at<kSingle>(b, 0);
    stats_chunk<T, B>(f, g, s_lo, s_hi);
  }
}

// A batch of both element types runs each pass as one launch, the float32
// fields' workgroups first, where the two types' kernels need alike registers
// and LDS (below b = 1024): a launch for each type has its own start and its
// own nearly empty end. b = 128, in a launch a type, and so: 8 fields of a median of
// 1 MiB 40.6 -> 28.2 us a call (graph replays), 32 of 256 KiB 49.1 -> 33.4. (5 us of
// each is the pass that ended the batch's streams, which the encode pass does now.)
template <int B>
constexpr bool kOneLaunch = B < 1024;
// The encode pass up to 4608 tiles in all (144 MiB), and up to 16384 (512 MiB) where
// at most 2048 of them are float64: a float64 tile costs 2-3 ns more in the kernel of
// both types, a launch and its end 6 us, and beyond 512 MiB that is nothing. Fields of 1
// MiB, a launch a type and one, us a call at b = 128 (and 512): 96 MiB, four tenths of
// it float64, 79.0 and 77.5 (78.9 and 79.4), three quarters 73.4 and 76.7 (73.9 and 76.6),
// nine tenths 72.5 and 64.6 (73.3 and 65.3); 144 MiB 99.7 and 99.4 (100.4 and 101.2),
// 96.0 and 97.8 (95.2 and 99.5), 91.9 and 90.5 (91.3 and 91.3); 192 MiB, a tenth 122.5 and
// 116.9 (125.5 and 119.7), a fifth 124.4 and 123.5 (126.6 and 125.9), nine tenths 112.6
// and 116.1 (114.0 and 117.0); 512 MiB, a tenth 290.7 and 288.4 (292.5 and 296.6; b = 32
// 326.9 and 318.7), half 279.0 and 296.6 (280.9 and 301.2).
inline bool one_encode_launch(uint64_t f32_tiles, uint64_t f64_tiles) {
  const uint64_t all = f32_tiles + f64_tiles;
  return all <= 4608 || (all <= 16384 && f64_tiles <= 2048);
}

template <int B>
__global__ __launch_bounds__(256) void k_stats_both(CBatch b) {
  __shared__ uint64_t s_lo[kWavesPerWG], s_hi[kWavesPerWG];
  uint64_t g = blockIdx.x;
  for (uint64_t i = g * kWG + threadIdx.x; i < b.zero_words; i += (uint64_t)gridDim.x * kWG) b.zero_begin[i] = 0;
  if (g < b.tiles_stats[0]) {
    const FieldC f = field_at<kBatch>(b, field_of<kBatch>(b.field_stats[0], g));
    stats_chunk<float, B>(f, g - f.base_stats, s_lo, s_hi);
  } else {
    g -= b.tiles_stats[0];
    const FieldC f = field_at<kBatch>(b, field_of<kBatch>(b.field_stats[1], g));
    stats_chunk<double, B>(f, g - f.base_stats, s_lo, s_hi);
  }
}

// ----------------------------------------------------------------- range ---

__device__ __forceinline__ uint64_t bound_of(const FieldC& f, uint64_t lo, uint64_t hi) {
  const int rel = f.eb_mode == 1;
  return f.dtype == 0 ? (uint64_t)bits_of(bound_from<float>(rel, f.eb, lo, hi))
                      : (uint64_t)bits_of(bound_from<double>(rel, f.eb, lo, hi));
}

// The bound of a field from its range slots, folded by each wave, one per lane.
__device__ __forceinline__ uint64_t slots_bound(const FieldC& f) {
  const uint32_t l = lane_id();
  uint64_t lo_inv = 0, hi = 0;
  if (l < f.nslots) {
    lo_inv = f.range[l * (kRangeStride / 8)];
    hi = f.range[l * (kRangeStride / 8) + 1];
  }
  lo_inv = group_max<kWave, uint64_t>(lo_inv);
  hi = group_max<kWave, uint64_t>(hi);
  return bound_of(f, ~lo_inv, hi);
}

// The bound e of a field (as the bits of a T) from its parameters and, for
// the relative bound, the field's finite range (no finite value: the range
// is empty and e = 0). Every thread of classification tile t calls it.
// Range slots in use (clean): each wave folds them by itself, one per lane.
// First use: tile t = 0 folds the chunks' partials and publishes the bound
// in the counters; the other tiles wait for it (tile 0 waits on nothing, and
// a workgroup runs only once every lower-numbered one has been dispatched).
// Contains a barrier on the first-use path of tile 0.
__device__ __forceinline__ uint64_t field_bound(const FieldC& f, uint32_t t, bool clean, uint64_t nchunks,
                                               uint64_t* s_red) {
  if (f.eb_mode != 1) return bound_of(f, ~0ull, 0ull);  // absolute bound: no range needed
  const uint32_t l = lane_id();
  if (f.next_range) {
    // a shard of a larger field: the range of the whole field from the
    // shards' ranges (pairs of doubles, which hold the element values exactly)
    double lo = __builtin_inf(), hi = -__builtin_inf();
    for (uint32_t i = l; i < f.next_range; i += kWave) {
      const double a = f.ext_range[2 * i], c = f.ext_range[2 * i + 1];
      lo = a < lo ? a : lo;
      hi = c > hi ? c : hi;
    }
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
      const double a = __shfl_xor(lo, d), c = __shfl_xor(hi, d);
      lo = a < lo ? a : lo;
      hi = c > hi ? c : hi;
    }
    if (!(lo <= hi) || f.eb == 0.0) return bound_of(f, ~0ull, 0ull);  // no finite value
    return f.dtype == 0 ? (uint64_t)bits_of(round_down_to<float>(f.eb * (hi - lo)))
                        : (uint64_t)bits_of(round_down_to<double>(f.eb * (hi - lo)));
  }
  if (clean) return slots_bound(f);
  if (t == 0) {
    uint64_t lo = ~0ull, hi = 0;
    // eight partials in flight per thread
    constexpr int U = 8;
    const ulonglong2* parts = reinterpret_cast<const ulonglong2*>(f.parts);
    for (uint64_t i0 = 0; i0 < nchunks; i0 += (uint64_t)U * kWG) {
      ulonglong2 p[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint64_t i = i0 + (uint64_t)u * kWG + threadIdx.x;
        p[u] = i < nchunks ? parts[i] : make_ulonglong2(~0ull, 0ull);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        lo = p[u].x < lo ? p[u].x : lo;
        hi = p[u].y > hi ? p[u].y : hi;
      }
    }
    lo = group_min<kWave, uint64_t>(lo);
    hi = group_max<kWave, uint64_t>(hi);
    const int w = threadIdx.x / kWave;
    if (l == 0) {
      s_red[2 * w] = lo;
      s_red[2 * w + 1] = hi;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kWavesPerWG; ++i) {
      lo = s_red[2 * i] < lo ? s_red[2 * i] : lo;
      hi = s_red[2 * i + 1] > hi ? s_red[2 * i + 1] : hi;
    }
    const uint64_t e_bits = bound_of(f, lo, hi);
    if (threadIdx.x == 0) {
      f.ctr->e_bits = e_bits;
      __hip_atomic_store(&f.ctr->e_ready, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    }
    return e_bits;
  }
  // relaxed polls (an acquiring load would invalidate caches at every poll),
  // one acquire fence once the flag is up
  uint32_t spins = 0;
  while (__hip_atomic_load(&f.ctr->e_ready, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) {
    if (++spins > kSpinLimit) {
      if (l == 0) atomicMax(&f.ctr->err, 1u);
      return 0;
    }
    __builtin_amdgcn_s_sleep(8);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  return __hip_atomic_load(&f.ctr->e_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Parameters of one block from its totalOrder extrema (keys): K = -1 for a
// block with a non-finite value (stored raw), 0 for a constant block, else the
// kept bits of eq. (4). verify is false where the bound is proved a priori.
template <typename T>
struct BlockPlan {
  T mu;
  int K;
  bool verify;
};

template <typename T>
__device__ __forceinline__ BlockPlan<T> plan_block(typename Traits<T>::U kmin, typename Traits<T>::U kmax, T e) {
  using U = typename Traits<T>::U;
  BlockPlan<T> p;
  p.mu = (T)0;
  p.K = -1;
  p.verify = true;
  if (kmin < FiniteKeys<T>::LO || kmax > FiniteKeys<T>::HI) return p;
  const T mn = from_bits<T>(key_to_bits<U>(kmin));
  const T mx = from_bits<T>(key_to_bits<U>(kmax));
  int m0;
  if (classify_block<T>(mn, mx, e, p.mu, m0)) {
    p.K = 0;
    return p;
  }
  p.K = kept_bits<T>(m0);
  // A priori bound: truncation errs by < 2^p(e); the two roundings (of x - mu
  // and of mu + v') by at most 2^(p(M) - (mantissa bits - 2)) together, with
  // M = max(|mn|, |mx|). If e - 2^p(e) covers that, every value passes.
  constexpr int MANT = Traits<T>::W - 1 - Traits<T>::E;
  const U emask = FiniteKeys<T>::EXPMASK;
  const U ebits = bits_of(e);
  const U pow2_bits = (ebits & emask) ? (ebits & emask) : ((U)1 << MANT);
  const T slack = e - from_bits<T>(pow2_bits);  // exact: same binade
  const T amn = mn < (T)0 ? -mn : mn, amx = mx < (T)0 ? -mx : mx;
  const T M = amn > amx ? amn : amx;
  const bool slack_normal = slack > (T)0 && (bits_of(slack) & emask) != 0;
  p.verify = !(slack_normal && exp_of<T>(slack) >= exp_of<T>(M) - (MANT - 2));
  return p;
}

// The lanes whose block is not constant: plan_block's K != 0 for the whole
// wave. The rounded half ranges decide (rounding is monotone) unless one equals
// e, which sends the wave through the exact test.
template <typename T>
__device__ __forceinline__ uint64_t stored_blocks(typename Traits<T>::U kmin, typename Traits<T>::U kmax, T e,
                                                 bool present) {
  using U = typename Traits<T>::U;
  const bool finite = kmin >= FiniteKeys<T>::LO && kmax <= FiniteKeys<T>::HI;
  const T mn = from_bits<T>(key_to_bits<U>(kmin)), mx = from_bits<T>(key_to_bits<U>(kmax));
  const T mu = (T)0.5 * mn + (T)0.5 * mx;
  const T up = mx - mu, down = mu - mn;
  const T d = up > down ? up : down;
  uint64_t stored = __ballot(present && !(finite && d < e));
  if (__ballot(present && finite && d == e) != 0)
    stored = __ballot(present && !(finite && exact_le<T>(mx, mu, e) && exact_le<T>(mu, mn, e)));
  return stored;
}

// A block's plan in one byte: 0 constant, 0xFF raw, else K with bit 7 set
// when the values must be verified.
template <typename T>
__device__ __forceinline__ uint32_t plan_byte(const BlockPlan<T>& p) {
  return p.K < 0 ? 0xFFu : p.K == 0 ? 0u : (uint32_t)p.K | (p.verify ? 0x80u : 0u);
}

// ---------------------------------------------------------------- header ---

// Header and the zero padding after the state bits, mu, K and codes sections
// of a field's stream, by the threads of one workgroup. Returns the stream
// size.
__device__ __forceinline__ uint64_t write_stream_header(const FieldC& f, uint64_t e_bits, uint64_t n_nc,
                                                        uint64_t mid_total) {
  const uint32_t w = f.dtype == 0 ? 4 : 8;
  const Sections s = sections(f.nblk, n_nc, w, f.b, mid_total);
  uint8_t* out = f.out;
  if (threadIdx.x == 0) {
    uint32_t* o32 = reinterpret_cast<uint32_t*>(out);
    uint64_t* o64 = reinterpret_cast<uint64_t*>(out);
    o32[0] = kMagic;
    o32[1] = (uint32_t)kVersion | (f.dtype << 8) | (f.eb_mode << 16) | (f.ndims << 24);
    o32[2] = f.b;
    o32[3] = 0;
    for (int d = 0; d < 4; ++d) o64[2 + d] = f.dims[d];
    o64[6] = f.n;
    o64[7] = (uint64_t)__double_as_longlong(f.eb);
    o64[8] = e_bits;
    o64[9] = f.nblk;
    o64[10] = n_nc;
    o64[11] = mid_total;
  }
  const uint64_t pads[4][2] = {{96 + cdiv(f.nblk, 8), s.mu},
                               {s.mu + f.nblk * w, s.kbytes},
                               {s.kbytes + n_nc, s.codes},
                               {s.codes + n_nc * (f.b / 4), s.mid}};
  for (int p = 0; p < 4; ++p)
    for (uint64_t i = pads[p][0] + threadIdx.x; i < pads[p][1]; i += blockDim.x) out[i] = 0;
  return s.total;
}

// The end of a field's stream, once every tile of it has published its size:
// the mid-byte total (the header's last field) and the stream size, or 0
// there if a bounded wait of this compression gave up. (A wait that gives up
// meanwhile raises the error first and then clears the size itself; the error
// is read once more after the size has been stored, so one of the two sees the
// other. Both words are device-scope atomics, so the wait for the store orders
// them; a fence would drop the XCD's L2, once a field: 256 batched fields 357
// us a call, so 344.)
__device__ __forceinline__ void finish_stream(const FieldC& f, uint64_t mid_total) {
  const uint64_t mid_off = sections(f.nblk, f.ctr->n_nc, f.dtype == 0 ? 4 : 8, f.b, 0).mid;
  reinterpret_cast<uint64_t*>(f.out)[11] = mid_total;
  const uint64_t size = mid_off + mid_total;
  if (__hip_atomic_load(&f.ctr->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) {
    __hip_atomic_store(f.out_size, size, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (__hip_atomic_load(&f.ctr->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0) return;
  }
  __hip_atomic_store(f.out_size, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// -------------------------------------------------------------- classify ---

// A single call's list of tiles to encode, behind the first ranks of its tiles.
template <typename T, int B>
__device__ __forceinline__ uint32_t* tile_list(const FieldC& f) {
  return f.enc_r0 + cdiv(f.nblk, (uint64_t)EncGeo<T, B>::TBLK) + 1;
}

// mu and the constant test of every block, the state bits, and the rank of the
// first non-constant block of every encode tile (a prefix count over tiles of
// CLS blocks, four per thread at most). The last tile writes n_nc. listed: a
// single call, whose encode pass takes its tiles from a list.
template <typename T, int B>
__device__ __forceinline__ void classify_tile(const FieldC& f, uint32_t t, bool listed, uint32_t* s_scan,
                                              uint32_t* s_state, uint64_t* s_base, uint64_t* s_red) {
  using U = typename Traits<T>::U;
  constexpr int TBLK = EncGeo<T, B>::TBLK;
  constexpr int CLS = (int)kClsBlocks;
  constexpr int BPT = CLS / kWG;  // blocks per thread
  const U* stats = reinterpret_cast<const U*>(f.stats);
  const uint64_t nblk = f.nblk;
  const uint64_t k0 = (uint64_t)t * CLS + (uint64_t)threadIdx.x * BPT;
  static_assert(BPT == 4 && TBLK % BPT == 0 && CLS % TBLK == 0, "a thread's four blocks lie in one encode tile");
  // a thread's blocks are consecutive and start 16-byte aligned in the
  // extrema, mu and plan arrays, so a full group moves as 16-byte words. The
  // extrema come through a buffer resource over the tile's blocks (reads
  // past the field's last block return zeros): one load form for every lane,
  // so the range slots' loads below go out before any of them is waited for
  const bool full = k0 + BPT <= nblk;
  U kmin[BPT], kmax[BPT];
  {
    const uint64_t kt = (uint64_t)t * CLS;
    const uint32_t nb_t = (uint32_t)std::min<uint64_t>(nblk - kt, (uint64_t)CLS);
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<U*>(stats + 2 * kt), (short)0, (int)(nb_t * 2u * (uint32_t)sizeof(U)), 0x00020000);
    using v4u = unsigned int __attribute__((ext_vector_type(4)));
    U w[2 * BPT];
    constexpr int NQ = 2 * BPT * (int)sizeof(U) / 16;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const v4u u = __builtin_amdgcn_raw_buffer_load_b128(
          rs, (int)((uint32_t)threadIdx.x * (uint32_t)(2 * BPT * sizeof(U)) + 16u * (uint32_t)q), 0, 0);
      reinterpret_cast<v4u*>(w)[q] = u;
    }
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      kmin[i] = w[2 * i];
      kmax[i] = w[2 * i + 1];
    }
  }
  const bool clean = *f.clean == kCleanWord;
  for (int i = threadIdx.x; i < CLS / 32; i += kWG) s_state[i] = 0;
  const uint64_t nchunks = cdiv(cdiv(f.n, (uint64_t)Geo<T, B>::TILE), (uint64_t)kStatsChunk);
  const uint64_t e_bits = field_bound(f, t, clean, nchunks, s_red);
  __syncthreads();
  const T e = from_bits<T>((U)e_bits);
  if (t == 0 && threadIdx.x == 0) {
    f.ctr->e_bits = e_bits;  // read by the encode pass
    *f.out_size = kSizePending;
  }
  const uint32_t ntiles = (uint32_t)cdiv(nblk, CLS);
  T* mus = reinterpret_cast<T*>(f.out + f.mu_off);
  uint32_t cnt = 0, bits = 0;
  T mv[BPT];
  uint32_t pv = 0;  // plan bytes, block i in byte i
#pragma unroll
  for (int i = 0; i < BPT; ++i) {
    const uint64_t k = k0 + i;
    mv[i] = (T)0;
    if (k < nblk) {
      const BlockPlan<T> p = plan_block<T>(kmin[i], kmax[i], e);
      mv[i] = p.mu;
      pv |= plan_byte(p) << (8 * i);
      const bool nc = p.K != 0;
      cnt += nc ? 1u : 0u;
      bits |= (nc ? 1u : 0u) << i;
    }
  }
  if (full) {
    constexpr int NQ = BPT * (int)sizeof(T) / 16;
#pragma unroll
    for (int q = 0; q < NQ; ++q) reinterpret_cast<uint4*>(mus + k0)[q] = reinterpret_cast<const uint4*>(mv)[q];
    *reinterpret_cast<uint32_t*>(f.plan + k0) = pv;
  } else {
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      if (k0 + i < nblk) {
        mus[k0 + i] = mv[i];
        f.plan[k0 + i] = (uint8_t)(pv >> (8 * i));
      }
    }
  }
  if (bits) atomicOr(&s_state[(threadIdx.x * BPT) / 32], bits << ((threadIdx.x * BPT) % 32));
  __syncthreads();
  // whether an encode tile that starts in this thread's blocks has a
  // non-constant one
  const bool starts = (k0 % TBLK) == 0 && k0 < nblk;
  uint32_t used = 0;
  if (starts) {
    const uint32_t b0 = threadIdx.x * BPT;
    if constexpr (TBLK >= 32) {
#pragma unroll
      for (int i = 0; i < TBLK / 32; ++i) used |= s_state[b0 / 32 + i];
    } else {
      used = (s_state[b0 / 32] >> (b0 % 32)) & ((1u << (TBLK % 32)) - 1u);
    }
    used = used ? 1u : 0u;
  }
  const uint32_t v2[2] = {cnt, used};
  uint32_t ex2[2], tot2[2];
  wg_excl_scan_multi<2>(v2, ex2, tot2, s_scan);  // has barriers
  const uint32_t total = tot2[0], ex = ex2[0];
  if (threadIdx.x < kWave) {
    const uint64_t agg = pair_aggregate(total, tot2[1]);
    if (threadIdx.x == 0) lookback_publish<true>(f.cls_status, t, agg);
    const uint64_t p = lookback_resolve_n<true>(f.cls_status, t, agg, &f.ctr->err, 1u, ntiles);
    if (threadIdx.x == 0) *s_base = p;
  }
  // state bytes of this tile, never past the state section
  const uint64_t state_bytes = (nblk + 7) / 8;
  for (int i = threadIdx.x; i < CLS / 8; i += kWG) {
    const uint64_t byte = (uint64_t)t * (CLS / 8) + i;
    if (byte < state_bytes) f.out[96 + byte] = (uint8_t)(s_state[i / 4] >> (8 * (i % 4)));
  }
  __syncthreads();
  const uint32_t base = (uint32_t)*s_base, tbase = (uint32_t)(*s_base >> 32);
  // first rank of every encode tile that starts in this thread's blocks, and
  // (a single call) its place in the list of tiles to encode, or its size, 0
  if (starts) {
    const uint32_t et = (uint32_t)(k0 / TBLK);
    f.enc_r0[et] = base + ex;
    if (listed) {
      if (used)
        tile_list<T, B>(f)[tbase + (ex2[1] - total)] = et;
      else
        status_store(f.enc_mid + et, et == 0 ? kFlagIncl : kFlagAgg);
    }
  }
  if (t == ntiles - 1) {
    // Every tile has published, so every tile has read the range slots: the
    // last one clears them for the next call and marks them clean; it also
    // writes the header (the encode pass adds the mid-byte total) and the
    // padding between the sections.
    const uint64_t n_nc = (uint64_t)base + total;
    if (threadIdx.x == 0) {
      f.ctr->n_nc = n_nc;
      f.ctr->n_tiles = tbase + tot2[1];
    }
    if (threadIdx.x < kRangeSlots)
      *reinterpret_cast<ulonglong2*>(f.range + threadIdx.x * (kRangeStride / 8)) = make_ulonglong2(0, 0);
    if (threadIdx.x == 0) *f.clean = kCleanWord;
    write_stream_header(f, e_bits, n_nc, 0);
  }
}

template <typename T, int B>
__global__ __launch_bounds__(256) void k_classify(CBatch b) {
  __shared__ uint32_t s_scan[2 * kWavesPerWG];
  __shared__ uint32_t s_state[kClsBlocks / 32];
  __shared__ uint64_t s_base;
  __shared__ uint64_t s_red[2 * kWavesPerWG];
  const uint64_t g = blockIdx.x;
  const FieldC f = field_at(b, field_of(b.field_cls[Traits<T>::BYTES / 8], g));
  classify_tile<T, B>(f, (uint32_t)(g - f.base_cls), !b.fields, s_scan, s_state, &s_base, s_red);
}

template <int B>
__global__ __launch_bounds__(256) void k_classify_both(CBatch b) {
  __shared__ uint32_t s_scan[2 * kWavesPerWG];
  __shared__ uint32_t s_state[kClsBlocks / 32];
  __shared__ uint64_t s_base;
  __shared__ uint64_t s_red[2 * kWavesPerWG];
  uint64_t g = blockIdx.x;
  if (g < b.tiles_cls[0]) {
    const FieldC f = field_at<kBatch>(b, field_of<kBatch>(b.field_cls[0], g));
    classify_tile<float, B>(f, (uint32_t)(g - f.base_cls), false, s_scan, s_state, &s_base, s_red);
  } else {
    g -= b.tiles_cls[0];
    const FieldC f = field_at<kBatch>(b, field_of<kBatch>(b.field_cls[1], g));
    classify_tile<double, B>(f, (uint32_t)(g - f.base_cls), false, s_scan, s_state, &s_base, s_red);
  }
}

// ---------------------------------------------------------------- encode ---

// Whether every valid value of a lane's run reconstructs within e exactly
// when K leading bits of x - mu are kept.
template <typename T, int EPL>
__device__ __forceinline__ bool run_within(const T (&x)[EPL], int cnt, T mu, T e, int K) {
  using U = typename Traits<T>::U;
  const int s = shift_of(K);
  const U keep = (U)(top_bytes_mask<U>(bytes_of(K)) << s);
  bool ok = true;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const T xr = mu + from_bits<T>((U)(bits_of(x[i] - mu) & keep));
    // bitwise on purpose: both checks, no short-circuit branch
    const bool good = (bool)((int)exact_le<T>(x[i], xr, e) & (int)exact_le<T>(xr, x[i], e));
    ok = (bool)((int)ok & ((int)good | (int)(i >= cnt)));
    // one value at a time: interleaving all of them costs registers, and
    // this path is rare
    __builtin_amdgcn_sched_barrier(0);
  }
  return ok;
}

// The high 32 bits of a value's shifted word (the bytes that leading-byte
// codes look at), and its low 32 bits (float64 only).
__device__ __forceinline__ uint32_t high_word(uint32_t q) { return q; }
__device__ __forceinline__ uint32_t high_word(uint64_t q) { return (uint32_t)(q >> 32); }
__device__ __forceinline__ uint32_t low_word(uint32_t) { return 0; }
__device__ __forceinline__ uint32_t low_word(uint64_t q) { return (uint32_t)q; }

// Byte selectors of the packer for words of which the top nb bytes (nb <= 4)
// may be stored. Shifted right by c bytes (a value that drops its c leading
// bytes, c <= min(3, nb)) they give
//   w: the word's stored bytes, most significant first (v_perm_b32 indices
//      0-3 of the word), then the bytes of the string behind it (indices 4-7);
//   x: the bytes 4 - L and on of the eight bytes behind it (L = nb - c).
// Byte j of both is 4 + j - nb, but for the first nb bytes of w.
struct PackSel {
  uint32_t w, x, hi;
  __device__ __forceinline__ explicit PackSel(uint32_t nb) {
    const uint32_t nb4 = __builtin_amdgcn_perm(0u, nb, 0u);  // nb in every byte
    x = 0x07060504u - nb4;
    hi = 0x0B0A0908u - nb4;
    const uint32_t rest = (uint32_t)(~0ull << (8u * nb));  // 64-bit: nb = 4 leaves none
    w = (x & rest) | (0x00010203u & ~rest);
  }
  __device__ __forceinline__ uint32_t w_at(uint32_t c) const { return __builtin_amdgcn_alignbyte(hi, w, c); }
  __device__ __forceinline__ uint32_t x_at(uint32_t c) const { return __builtin_amdgcn_alignbyte(hi, x, c); }
};

// The dword at LDS address a (positions in the packer are LDS addresses, so
// that no base is added per string).
typedef __attribute__((address_space(3))) uint32_t lds_u32;
__device__ __forceinline__ lds_u32* lds_at(uint32_t a) { return (lds_u32*)a; }
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)p;
}

// Packs a lane's byte strings, last one first, into its run of an LDS byte
// stream. w holds the four stream bytes from the current string's start on
// and x the four after them (zero past the run's end). Putting a string in
// front is two byte permutes, and the aligned dword at or after its start
// (its bytes all lie in w and x) is stored as it is then: every dword that
// starts inside the run is written with its run bytes, most of them more
// than once and always the same. A dword that starts at or past the run's
// end may be overwritten with zeros, but only before the last of the run's
// strings is put (put_first, which does not write there): it is the first
// aligned dword of a later lane, which that lane's own put_first, the same
// instruction, restores. What remains are the bytes before the run's first
// aligned dword, OR-ed into the dword that the lanes before left zero there
// (or_head). No per-string branch, no dword to clear beforehand, one LDS
// store a string.
struct RunPacker {
  uint32_t m;  // ~(position + 3): its low two bits are the bytes up to the next aligned dword
  uint32_t w, x;
  __device__ __forceinline__ explicit RunPacker(uint32_t end) : m(~(end + 3u)), w(0), x(0) {}
  // L = nb - c <= 4 bytes of the word v
  __device__ __forceinline__ void prepend(uint32_t v, uint32_t nb, uint32_t c, const PackSel& sel) {
    m = __builtin_amdgcn_sad_u8(nb, c, m);  // m + nb - c
    const uint32_t nx = __builtin_amdgcn_perm(x, w, sel.x_at(c));
    w = __builtin_amdgcn_perm(w, v, sel.w_at(c));
    x = nx;
  }
  __device__ __forceinline__ uint32_t dword_at() const { return ~(m | 3u); }
  __device__ __forceinline__ void store() { *lds_at(dword_at()) = __builtin_amdgcn_alignbyte(x, w, m); }
  __device__ __forceinline__ void store_first(uint32_t end) {
    if (dword_at() < end) store();
  }
  __device__ __forceinline__ void or_head(uint32_t start) {
    __hip_atomic_fetch_or(lds_at(start & ~3u), w << (8u * (start & 3u)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
};

// Copy the wave's total staged bytes to out + [dst, dst + total). They start
// at the 16-byte word at16 of its LDS ring of mask16 + 1 such words (a power
// of two) and may wrap around its end. Whole aligned 16-byte chunks of the
// destination go out as single stores: a chunk starts h bytes into a staged
// word (h the bytes before the first whole chunk, the same for every chunk),
// so every lane reads two consecutive 16-byte words (a wave reads a
// contiguous range: no LDS bank conflicts) and realigns them with byte funnel
// shifts by the same amount. The bytes before the first whole chunk and after
// the last go out one a lane.
__device__ __forceinline__ void copy_out(uint8_t* __restrict__ out, uint64_t dst, const uint8_t* stage, uint32_t at16,
                                         uint32_t mask16, uint32_t total) {
  const uint4* ring = reinterpret_cast<const uint4*>(stage);
  const uint32_t bmask = mask16 * 16u + 15u;
  const uint32_t l = (uint32_t)lane_id();
  uint8_t* base = out + dst;
  uint32_t h = (16u - (uint32_t)(dst & 15u)) & 15u;
  h = h < total ? h : total;
  const uint32_t nfull = (total - h) / 16u;
  {
    const uint32_t tail0 = h + nfull * 16u;
    const uint32_t i = l < 16u ? l : tail0 + (l - 16u);
    const bool on = l < 16u ? l < h : (l < 32u && i < total);
    if (on) base[i] = stage[(at16 * 16u + i) & bmask];
  }
  const uint32_t k = h >> 2, sh = h & 3u;
  for (uint32_t c = l; c < nfull; c += kWave) {
    const uint4 q0 = ring[(at16 + c) & mask16];
    const uint4 q1 = ring[(at16 + c + 1) & mask16];
    *reinterpret_cast<uint4*>(base + h + c * 16u) = realign16(q0, q1, k, sh);
  }
}

// The previous lane's value over the whole wave (wave_shr:1; lane 0 gets 0).
__device__ __forceinline__ uint32_t wave_before(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xF, 0xF, false);
}

// Plan of a wave's blocks: each row's mu and plan byte (both left by the
// classification pass), what the rank of the wave's first block is counted
// from (the tile's plan bytes, or its state bits where the tile has more
// blocks than a wave lanes), and the rank of the tile's first block.
template <typename T, int B>
struct WavePlan {
  T mu[EncGeo<T, B>::SUB];
  uint32_t pb[EncGeo<T, B>::SUB];
  uint32_t ahead;
  uint32_t r0;
};

// Through buffer resources over the tile's entries: reads past the field's
// last block return zeros (a constant block, which stores nothing), so no
// load sits in a branch and the compiler can count the loads in flight.
// on = false loads nothing (every plan byte 0).
template <typename T, int B>
__device__ __forceinline__ void plan_load(WavePlan<T, B>& p, const FieldC* f, uint32_t t, uint32_t wave, bool on) {
  using G = EncGeo<T, B>;
  constexpr int SUB = G::SUB, TBLK = G::TBLK;
  const uint32_t lane = (uint32_t)lane_id(), g = lane / G::LPB;
  // the tile's first block (wave-uniform) and its block count
  const uint64_t kb = on ? (uint64_t)t * TBLK : 0;
  const uint32_t nblk_t = on ? (uint32_t)std::min<uint64_t>(f->nblk - kb, (uint64_t)TBLK) : 0u;
  const __amdgpu_buffer_rsrc_t rm =
      buffer_of(reinterpret_cast<const T*>(f->out + f->mu_off) + kb, nblk_t * (uint32_t)sizeof(T));
  const __amdgpu_buffer_rsrc_t rp = buffer_of(f->plan + kb, nblk_t);
#pragma unroll
  for (int s = 0; s < SUB; ++s)
    p.pb[s] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b8(rp, (int)(wave * G::WBLK + (uint32_t)(s * G::GPW) + g), 0, 0);
  if constexpr (TBLK <= kWave) {
    p.ahead = (uint32_t)__builtin_amdgcn_raw_buffer_load_b8(rp, (int)lane, 0, 0);
  } else {
    // whole words of state bits: bits past the field's last block are never
    // counted (a word past the section's end reads its padding or mu)
    static_assert(TBLK <= 32 * kWave && TBLK % 32 == 0, "a wave covers the tile's state words");
    const __amdgpu_buffer_rsrc_t rb = buffer_of(f->out + 96 + kb / 8, (nblk_t + 31) / 32 * 4);
    p.ahead = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rb, (int)(lane * 4u), 0, 0);
  }
#pragma unroll
  for (int s = 0; s < SUB; ++s)
    p.mu[s] = buffer_value<T>(rm, (wave * G::WBLK + (uint32_t)(s * G::GPW) + g) * (uint32_t)sizeof(T));
  p.r0 = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(buffer_of(f->enc_r0 + (on ? t : 0u), 4u), 0, 0, 0);
}

// Non-constant blocks of the tile before the wave's first one.
template <typename T, int B>
__device__ __forceinline__ uint32_t rank_ahead(uint32_t ahead, uint32_t wave) {
  using G = EncGeo<T, B>;
  if constexpr (G::TBLK <= kWave) {
    return (uint32_t)__popcll(__ballot(ahead != 0) & ((1ull << (wave * G::WBLK)) - 1ull));
  } else {
    const int left = (int)(wave * G::WBLK) - lane_id() * 32;
    const uint32_t mask = left >= 32 ? ~0u : left <= 0 ? 0u : (1u << left) - 1u;
    return wave_total_u32((uint32_t)__popc(ahead & mask));
  }
}

// The descriptor of a field as constant memory behind an address that the
// compiler cannot see through, so that each use reads the members it needs
// again with scalar loads: kept in scalar registers over the tile loop they
// spill to vector lanes, a vector instruction each way.
template <int BATCH>
__device__ __forceinline__ const FieldC* field_ref(const CBatch& b, uint32_t fi) {
  uint64_t p = BATCH == kSingle
                   ? (uint64_t)(uintptr_t)__builtin_amdgcn_kernarg_segment_ptr() + __builtin_offsetof(CBatch, one)
                   : (uint64_t)(uintptr_t)(b.fields + fi);
  p = uniform(p);
  asm volatile("" : "+s"(p));
  return as_constant(reinterpret_cast<const FieldC*>((uintptr_t)p));
}

// Row s of the wave's values (left in flight), through a buffer resource over
// the tile's values (to the field's end): reads past its range return zeros
// without touching memory, so lanes of constant blocks (sent far past it) and
// a short block's run past the field's end need no branch.
template <typename T, int B, int EPL>
__device__ __forceinline__ void row_load(T (&x)[EPL], __amdgpu_buffer_rsrc_t rs, uint32_t wave, int s, uint32_t pb) {
  using G = EncGeo<T, B>;
  constexpr int PER16 = 16 / (int)sizeof(T);
  const uint32_t lane = (uint32_t)lane_id();
  const uint32_t lk = wave * G::WBLK + (uint32_t)(s * G::GPW) + lane / G::LPB;
  const uint32_t off = pb != 0 ? (lk * B + (lane % G::LPB) * EPL) * (uint32_t)sizeof(T) : 0x40000000u;
  using v4u = unsigned int __attribute__((ext_vector_type(4)));
#pragma unroll
  for (int c = 0; c < EPL / PER16; ++c) {
    const v4u u = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(off + 16u * (uint32_t)c), 0, 0);
    if constexpr (sizeof(T) == 4) {
      x[4 * c + 0] = __uint_as_float(u.x);
      x[4 * c + 1] = __uint_as_float(u.y);
      x[4 * c + 2] = __uint_as_float(u.z);
      x[4 * c + 3] = __uint_as_float(u.w);
    } else {
      x[2 * c + 0] = __longlong_as_double((long long)(((uint64_t)u.y << 32) | u.x));
      x[2 * c + 1] = __longlong_as_double((long long)(((uint64_t)u.w << 32) | u.z));
    }
  }
}

// Buffer resource over the values of tile t of a field.
template <typename T, int B>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t values_of(const FieldC* f, uint32_t t) {
  const uint64_t i0 = (uint64_t)t * EncGeo<T, B>::TBLK * B;
  return buffer_of(reinterpret_cast<const T*>(f->in) + i0,
                   (uint32_t)std::min<uint64_t>(f->n - i0, (uint64_t)EncGeo<T, B>::TBLK * B) * (uint32_t)sizeof(T));
}

// A row's words as a lane encodes them: its EPL values of one block.
template <typename T, int B>
struct RowWords {
  using U = typename Traits<T>::U;
  static constexpr int EPL = EncGeo<T, B>::EPL, LPB = EncGeo<T, B>::LPB, BYTES = Traits<T>::BYTES;
  // a value's word: its top nb bytes are stored (less the leading ones its
  // code names); a raw value's bytes in storage order
  U q[EPL];
  uint32_t c[EPL], codes;  // the values' codes, and all of them (first value in the top bits)
  uint32_t nb, lb;         // whole bytes kept of a value; stored bytes of the lane

  // From K kept bits (-1 raw, 0 constant or absent: nothing is stored). Error
  // control where the bound is not proved (check): K, then one more mantissa
  // bit, then raw; every lane of a block votes, and K becomes the outcome.
  // special: some lane of the wave is raw or checks.
  __device__ __forceinline__ void code(const T (&x)[EPL], T mu, int& K, bool check, bool special, T e, int cnt,
                                       bool tail, uint32_t lig) {
    if (special) {
      const bool ok = !check || run_within<T, EPL>(x, cnt, mu, e, K);
      if (!group_all<LPB>(ok)) {
        const int K1 = kept_bits<T>(K - Traits<T>::KMIN + 1);
        const bool ok1 = K1 != K && run_within<T, EPL>(x, cnt, mu, e, K1);
        K = group_all<LPB>(ok1) ? K1 : -1;
      }
    }
    nb = ((uint32_t)K + 7u) >> 3;
    const uint32_t sft = 8u * nb - (uint32_t)K;
    // Codes: leading identical bytes capped at min(3, nb) (0 for raw blocks),
    // at most 24 bits, so a 64-bit word's high half decides: a bit set at the
    // cap ends the count there.
    uint32_t cap = 0x80000000u >> (8u * (nb < 3u ? nb : 3u));
#pragma unroll
    for (int i = 0; i < EPL; ++i) q[i] = (U)(bits_of(x[i] - mu) >> sft);
    if (special) {
      if (K < 0) {
        nb = (uint32_t)BYTES;
        cap = 0x80000000u;
#pragma unroll
        for (int i = 0; i < EPL; ++i) q[i] = byte_swap(bits_of(x[i]));
      }
    }
    uint32_t prev = wave_before(high_word(q[EPL - 1]));
    prev = lig == 0 ? 0u : prev;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const uint32_t hw = high_word(q[i]);
      c[i] = lead_zero_bits((hw ^ prev) | cap) >> 3;
      prev = hw;
    }
    uint32_t live = nb * EPL;
    if (tail) {
      int cv = cnt;
      asm volatile("" : "+v"(cv));  // keeps this branch's tests inside it
#pragma unroll
      for (int i = 0; i < EPL; ++i) c[i] = i < cv ? c[i] : 0u;
      live = nb * (uint32_t)cnt;
    }
    codes = 0;
#pragma unroll
    for (int i = 0; i < EPL; ++i) codes = (codes << 2) | c[i];
    // stored bytes of the lane: nb per valid value less the identical ones
    lb = live - ((uint32_t)__popc(codes) + (uint32_t)__popc(codes & 0xAAAAAAAAu));
  }

  // The strings into the lane's run, which ends at LDS address end.
  __device__ __forceinline__ void pack(RunPacker& pk, int cnt, bool tail, uint32_t end) const {
    const uint32_t nbh = nb < 4u ? nb : 4u, nbl = nb - nbh;
    const PackSel sel(nbh);
    if (tail) {
      int cv = cnt;
      asm volatile("" : "+v"(cv));
      const PackSel sell(nbl);
#pragma unroll
      for (int i = EPL - 1; i >= 0; --i) {
        if (sizeof(T) == 8) {
          if (i < cv) pk.prepend(low_word(q[i]), nbl, 0u, sell);
          pk.store();
        }
        if (i < cv) pk.prepend(high_word(q[i]), nbh, c[i], sel);
        if (i > 0) pk.store();
      }
    } else if (sizeof(T) == 8 && __ballot(nb > 4u) != 0) {
      const PackSel sell(nbl);
#pragma unroll
      for (int i = EPL - 1; i >= 0; --i) {
        pk.prepend(low_word(q[i]), nbl, 0u, sell);
        pk.store();
        pk.prepend(high_word(q[i]), nbh, c[i], sel);
        if (i > 0) pk.store();
      }
    } else {
#pragma unroll
      for (int i = EPL - 1; i >= 0; --i) {
        pk.prepend(high_word(q[i]), nbh, c[i], sel);
        if (i > 0) pk.store();
      }
    }
    pk.store_first(end);
  }
};

// What the workgroup's waves share.
struct EncShared {
  uint32_t tot[2][kWavesPerWG];  // a tile's bytes by wave, by the tile's parity
  uint32_t next[2];              // the tile after the next one
};

// The encode pass for the tiles of element type T: persistent workgroups take
// tickets from the kTicketClasses counters of this type; ticket i of class c
// is global tile kTicketClasses * i + c, global tiles running over the fields
// of this type in order. A single call's tickets run over the list of tiles
// with a non-constant block that the classification pass made (it published
// the other tiles' sizes, zero). A launch with a workgroup for every tile
// takes no tickets: workgroups are dispatched in order, so a tile waits only
// on running or finished ones all the same.
//
// Each wave encodes a contiguous quarter of its workgroup's tile by itself:
// its rows' prefix sums, ranks and packing stay in the wave, and its mid bytes
// go to an LDS ring of its own. The waves meet at one barrier a tile, where
// their byte counts add up and the next ticket is handed out; then thread 0
// publishes the tile's count. A wave leaves a tile's bytes in its ring,
// pending, while it encodes its quarter of the next tile behind them; only
// then does it take the pending tile's offset in the mid section, which the
// scan workgroup has published by then, and copy its bytes out. When a row
// would reach the pending bytes, they are written out first (incompressible
// tiles: no overlap).
//
// Bound: the values' reads and the stream's writes (100x500x500 float32 at
// REL 1e-3, 100 MB in and 41 MB out, take 27 us at the copy rate of 5.2 TB/s)
// and, about as long, 18 vector instructions a value plus 250 a tile. Measured
// there 36 us a launch, and 233 us on 2^28 float64 values at REL 1e-3 (43 and
// 421 us with a barrier for every row's sums, LDS atomics for every packed
// dword and tickets for constant tiles); 256 fields of a median of 1 MiB (599 MiB), 185
// us for the float32 ones and 31 for the float64 ones (239 and 35). Smaller
// workgroups without the pending tile, eight a compute unit, took 51 us: every
// tile then waits 4-5 us for its offset.
//
// wid is the workgroup's number among wgs.
template <typename T, int B, int BATCH>
__device__ __forceinline__ void encode_pass(const CBatch& b, EncShared& sh, uint8_t* s_ring, uint32_t wid, uint32_t wgs) {
  using U = typename Traits<T>::U;
  using G = EncGeo<T, B>;
  constexpr int EPL = G::EPL, LPB = G::LPB, SUB = G::SUB;
  constexpr int BYTES = Traits<T>::BYTES;
  constexpr uint32_t RING = G::RING;
  constexpr uint32_t MASK16 = RING / 16 - 1;
  constexpr int DT = sizeof(T) == 4 ? 0 : 1;
  const uint32_t cls = wid % kTicketClasses;
  const bool direct = wgs >= b.tiles_enc[DT];  // a workgroup for every tile
  const FieldC* const one = BATCH == kSingle ? field_ref<BATCH>(b, 0) : nullptr;
  const uint64_t ntiles = BATCH == kSingle ? listed_tiles(as_constant(one->ctr)->err, as_constant(one->ctr)->n_tiles)
                                           : b.tiles_enc[DT];
  const uint32_t* const list = BATCH == kSingle ? as_global(tile_list<T, B>(*one)) : nullptr;
  uint32_t* ticket = b.tickets + (DT * kTicketClasses + cls) * 64;
  const uint32_t wave = uniform(threadIdx.x / kWave);
  const uint32_t lane = (uint32_t)lane_id(), lig = lane % LPB;
  uint8_t* const stage = s_ring + wave * (RING + G::SLACK);
  const uint32_t ring0 = uniform(lds_address(stage));

  // A claimed tile travels as its global number (a single call's, as the list
  // has it), or ntiles (past every tile) when there is none left.
  auto number = [&](uint32_t tk) -> uint64_t { return (uint64_t)tk * kTicketClasses + cls; };
  auto listed = [&](uint64_t g) -> uint32_t {
    if (g >= ntiles) return ~0u;
    return BATCH == kSingle ? list[g] : (uint32_t)g;
  };
  auto tile_in = [&](uint32_t gt, uint32_t& fi) -> uint32_t {
    fi = field_of<BATCH>(b.field_enc[DT], gt);
    return BATCH == kSingle ? gt : gt - (uint32_t)field_ref<BATCH>(b, fi)->base_enc;
  };

  // The first tile and its plan; then the ticket of the second, taken only
  // now, so that the workgroups' first tiles come before all second ones.
  uint32_t gt;
  if (direct) {
    if (wid >= ntiles) return;
    gt = uniform(listed(wid));
  } else {
    if (threadIdx.x == 0) sh.next[0] = listed(number(atomicAdd(ticket, 1u)));
    __syncthreads();
    gt = uniform(sh.next[0]);
    if (gt == ~0u) return;
  }
  T x[SUB][EPL];
  WavePlan<T, B> cur, nxt;
  uint32_t fi;
  uint32_t t = tile_in(gt, fi);
  uint32_t fi_n = fi, t_n = t;
  uint32_t tk = 0, tn = ~0u;
  bool more = false;
  {
    const FieldC* f = field_ref<BATCH>(b, fi);
    const __amdgpu_buffer_rsrc_t rs = values_of<T, B>(f, t);
    plan_load<T, B>(cur, f, t, wave, true);
    if (!direct && threadIdx.x == 0) tk = atomicAdd(ticket, 1u);
    // the first tile's values without regard to its plan, a memory latency
    // earlier (constant blocks' are not used)
#pragma unroll
    for (int s = 0; s < SUB; ++s) row_load<T, B, EPL>(x[s], rs, wave, s, 1u);
  }
  // the next tile (from slot `slot`) and its plan's loads, and the ticket of
  // the tile after it
  auto next = [&](uint32_t slot) {
    if (!direct) {
      const uint32_t g = uniform(sh.next[slot]);
      more = g != ~0u;
      if (more) t_n = tile_in(g, fi_n);
    }
    plan_load<T, B>(nxt, field_ref<BATCH>(b, fi_n), t_n, wave, more);
    if (more && threadIdx.x == 0) tk = atomicAdd(ticket, 1u);
  };
  if (!direct) {
    if (threadIdx.x == 0) sh.next[1] = listed(number(tk));
    __syncthreads();
  }
  next(1);

  // the pending tile (wave-uniform): its bytes in the wave's ring from byte
  // p_at (16-byte aligned) on, its offset not yet taken
  bool pend = false;
  uint32_t p_tile = 0, p_field = 0, p_bytes = 0, p_at = 0, p_total = 0, p_before = 0;
  uint32_t at = 0;  // ring byte of the current tile's start (16-byte aligned)
  // Take the pending tile's offset and copy the wave's share of it out. The
  // scan workgroup's sums run over all fields of the type: a batch's tile
  // takes off the sum up to its field's first tile.
  auto flush = [&](uint64_t first_poll) {
    const FieldC* fp = field_ref<BATCH>(b, p_field);
    Counters* const ctr = as_global(fp->ctr);
    uint64_t* const st = as_global(fp->enc_mid);
    bool ok = true;
    uint64_t base = uniform(scan_wait(st, p_tile, p_total, ok, first_poll));
    if constexpr (BATCH == kBatch) {
      if (fp->base_enc > 0) base -= uniform(scan_wait(st - 1, 0, 0, ok));
    }
    if (!ok) {  // a bounded wait gave up: the field has no stream (finish_stream)
      atomicMax(&ctr->err, 1u);
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "agent");
      __hip_atomic_store(as_global(fp->out_size), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const uint64_t nblk = fp->nblk;
    const uint64_t mid = sections(nblk, *as_constant(&ctr->n_nc), BYTES, B, 0).mid;
    // the output holds the worst case (every block raw; the caller's capacity
    // is checked against it)
    if (ok && mid + base + p_total <= sections(nblk, nblk, BYTES, B, fp->n * BYTES).total)
      copy_out(as_global(fp->out), mid + base + p_before, stage, p_at / 16, MASK16, p_bytes);
    // a batch's field ends with its last tile
    if constexpr (BATCH == kBatch) {
      if (ok && p_tile == (uint32_t)cdiv(nblk, (uint64_t)G::TBLK) - 1 && threadIdx.x == 0)
        finish_stream(field_at<kBatch>(b, p_field), base + p_total);
    }
    pend = false;
  };

  for (uint32_t par = 0;; par ^= 1) {
    const FieldC* f = field_ref<BATCH>(b, fi);
    uint8_t* const out = as_global(f->out);
    const uint64_t kb = (uint64_t)t * G::TBLK;
    const uint32_t nval_t = (uint32_t)std::min<uint64_t>(f->n - kb * B, (uint64_t)G::TBLK * B);
    const bool tail = nval_t != (uint32_t)(G::TBLK * B);  // the field's last tile may hold a short block
    const __amdgpu_buffer_rsrc_t rx = values_of<T, B>(field_ref<BATCH>(b, fi_n), t_n);
    // the wave's K bytes and codes from their first; rows index them with
    // 32-bit offsets (lanes without one store far past the range: nothing)
    const uint64_t r0 = uniform(cur.r0) + rank_ahead<T, B>(cur.ahead, wave);
    const Sections sec = sections(f->nblk, as_constant(f->ctr)->n_nc, BYTES, B, 0);
    const __amdgpu_buffer_rsrc_t rk = buffer_of(out + sec.kbytes + r0, G::WBLK);
    const __amdgpu_buffer_rsrc_t rc = buffer_of(out + sec.codes + r0 * (B / 4), G::WBLK * (B / 4));
    const T e = from_bits<T>((U)as_constant(f->ctr)->e_bits);
    uint32_t wbytes = 0, wrank = 0;
#pragma unroll
    for (int s = 0; s < SUB; ++s) {
      const uint32_t pb = cur.pb[s];
      const uint64_t has = __ballot(pb != 0);
      if (has != 0) {  // a row of constant blocks stores nothing (wave-uniform)
        int K = pb == 0xFFu ? -1 : (int)(pb & 0x7Fu);
        const T mu = cur.mu[s];
        const uint32_t lk = wave * G::WBLK + (uint32_t)(s * G::GPW) + lane / LPB;  // block of the tile
        int cnt = EPL;
        if (tail) {
          const int rem = (int)nval_t - (int)(lk * B + lig * EPL);
          cnt = rem < 0 ? 0 : (rem > EPL ? EPL : rem);
        }
        const bool special = __ballot((pb & 0x80u) != 0) != 0;
        RowWords<T, B> w;
        w.code(x[s], mu, K, K > 0 && (pb & 0x80u), special, e, cnt, tail, lig);
        if (special && K < 0 && pb != 0xFFu && lig == 0) reinterpret_cast<T*>(out + f->mu_off)[kb + lk] = (T)0;
        const bool raw = K < 0;
        const uint32_t lb = w.lb, codes = w.codes;
        const uint32_t inc = wave_incl_sum_u32(lb);
        const uint32_t rtot = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
        // K bytes and codes. The group's first lane does not count its own
        // block; the others see it counted.
        const uint64_t firsts = has & first_lanes<LPB>();
        const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
            (uint32_t)(firsts >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)firsts, wrank - (lig != 0 ? 1u : 0u)));
        wrank += (uint32_t)__popcll(firsts);
        __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(raw ? kRawK : (uint8_t)K), rk,
                                             (int)(pb != 0 && lig == 0 ? rank : 0x40000000u), 0, 0);
        const uint32_t coff = pb != 0 ? rank * (uint32_t)(B / 4) + lig * (EPL / 4) : 0x40000000u;
        if constexpr (EPL == 8) {
          __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(((codes >> 8) & 0xFFu) | ((codes & 0xFFu) << 8)), rc,
                                                (int)coff, 0, 0);
        } else {
          static_assert(EPL == 16, "a lane's codes are one or two half words");
          __builtin_amdgcn_raw_buffer_store_b32(__builtin_bswap32(codes), rc, (int)coff, 0, 0);
        }
        // the ring from this tile's start up to the pending tile's must hold
        // the row and the dword that may be zeroed behind it
        if (pend && wbytes + rtot + 8u > RING - ((p_bytes + 15u) & ~15u)) flush(0);
        if (!pend && wbytes == 0) at = 0;
        // a tile that fills the ring: the dword zeroed behind the row may be
        // the tile's first one (never where the tile starts at 0: behind it
        // is the slack)
        const bool tight = wbytes + rtot + 8u > RING;
        uint32_t kept = 0;
        if (tight) kept = *lds_at(ring0 + at);
        // stage the kept bytes. A lane's run starts inside the ring and may
        // end in the slack behind it.
        const uint32_t start = ring0 + ((at + wbytes + inc - lb) & (RING - 1u));
        const uint32_t end = start + lb;
        RunPacker pk(end);
        w.pack(pk, cnt, tail, end);
        // the run of the lane that crosses the ring's end: its dwords behind
        // the end move to the ring's start
        const uint64_t over = __ballot(end > ring0 + RING);
        if (over != 0) {
          const uint32_t ov =
              (uint32_t)__builtin_amdgcn_readlane((int)end, (int)__ffsll((long long)over) - 1) - ring0 - RING;
          if (lane * 4u < ov) *lds_at(ring0 + lane * 4u) = *lds_at(ring0 + RING + lane * 4u);
        }
        pk.or_head(start);
        if (tight && wbytes > 0) *lds_at(ring0 + at) = kept;
        wbytes += rtot;
      }
      // the row's registers are free: the next tile's row goes out
      row_load<T, B, EPL>(x[s], rx, wave, s, nxt.pb[s]);
      // the ticket has arrived: its tile's number, needed at the barrier
      if (s == 0 && more && threadIdx.x == 0) tn = listed(number(tk));
    }
    if (lane == 0) sh.tot[par][wave] = wbytes;
    if (threadIdx.x == 0) sh.next[par] = tn;
    __syncthreads();
    uint32_t total = 0, before = 0;
#pragma unroll
    for (uint32_t i = 0; i < (uint32_t)kWavesPerWG; ++i) {
      const uint32_t v = uniform(sh.tot[par][i]);
      before += i < wave ? v : 0u;
      total += v;
    }
    // (the first tile's sum is its own)
    if (threadIdx.x == 0)
      status_store(as_global(f->enc_mid) + t, (t == 0 && (BATCH == kSingle || f->base_enc == 0) ? kFlagIncl : kFlagAgg) | total);
    uint64_t first_poll = 0;
    if (pend) first_poll = status_load(as_global(field_ref<BATCH>(b, p_field)->enc_mid) + p_tile);
    const bool last = !more;
    const uint32_t t_c = t, fi_c = fi;
    t = t_n;
    fi = fi_n;
    cur = nxt;
    if (!last) next(par);
    if (pend) flush(first_poll);
    pend = true;
    p_tile = t_c;
    p_field = fi_c;
    p_bytes = wbytes;
    p_total = total;
    p_before = before;
    p_at = at;
    at = (at + ((wbytes + 15u) & ~15u)) & (RING - 1u);
    if (last) break;
  }
  flush(0);
}

// Workgroup 0 is the scan workgroup of the tiles' mid-byte offsets (every
// other waits on one status word a tile).
template <typename T, int B, int BATCH>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(EncGeo<T, B>::WAVES))) void k_encode(CBatch b) {
  using G = EncGeo<T, B>;
  constexpr int DT = sizeof(T) == 4 ? 0 : 1;
  __shared__ union {
    EncShared enc;
    ScanShared scan;
  } s_sh;
  __shared__ __align__(16) uint8_t s_ring[kWavesPerWG * (G::RING + G::SLACK)];
  if (blockIdx.x == 0) {
    // the type's status words lie in one array, its first field's first
    const FieldC* f = field_ref<BATCH>(b, BATCH == kSingle ? 0u : *as_constant(b.field_enc[DT]));
    // (where a single call's classification gave up, no tile is encoded and none is waited for)
    const uint64_t ntiles = BATCH == kSingle ? listed_tiles(as_constant(f->ctr)->err, b.tiles_enc[DT]) : b.tiles_enc[DT];
    const uint64_t total = scan_workgroup(as_global(f->enc_mid), ntiles, &as_global(f->ctr)->err, 1u, s_sh.scan);
    if constexpr (BATCH == kSingle) {
      if (threadIdx.x == 0) finish_stream(field_at<BATCH>(b, 0), total);
    }
    return;
  }
  encode_pass<T, B, BATCH>(b, s_sh.enc, s_ring, blockIdx.x - 1, gridDim.x - 1);
}

// Both types of a batch: the float32 tiles and then the float64 tiles.
// Workgroup 0 scans the float32 tiles, workgroup 1 the float64 ones. (One that
// scanned both in turn would hold the float64 offsets until the last float32
// tile is encoded: where that tile's workgroup is not dispatched yet, those
// that wait for a float64 offset never make room for it.)
template <int B>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(EncGeo<float, B>::WAVES))) void k_encode_both(
    CBatch b) {
  using G4 = EncGeo<float, B>;
  using G8 = EncGeo<double, B>;
  static_assert(G4::WAVES == G8::WAVES, "the two types need alike registers and LDS");
  __shared__ union {
    EncShared enc;
    ScanShared scan;
  } s_sh;
  __shared__ __align__(16) uint8_t s_ring[kWavesPerWG * std::max(G4::RING + G4::SLACK, G8::RING + G8::SLACK)];
  if (blockIdx.x < 2) {
    const uint32_t dt = blockIdx.x;
    const FieldC* f = field_ref<kBatch>(b, *as_constant(b.field_enc[dt]));
    scan_workgroup(as_global(f->enc_mid), b.tiles_enc[dt], &as_global(f->ctr)->err, 1u, s_sh.scan);
    return;
  }
  const uint32_t wid = blockIdx.x - 2, wgs = gridDim.x - 2;
  encode_pass<float, B, kBatch>(b, s_sh.enc, s_ring, wid, wgs);
  __syncthreads();
  encode_pass<double, B, kBatch>(b, s_sh.enc, s_ring, wid, wgs);
}

// ------------------------------------------------------------------ small ---

// The largest field that one workgroup compresses (its rings take as much LDS),
// and the workgroup's waves for a field of at most `bytes` bytes.
constexpr uint32_t kSmallestBytes = 32u << 10;
template <typename T>
constexpr uint32_t kSmallBytes = sizeof(T) == 4 ? 64u << 10 : 96u << 10;
template <typename T, int B>
constexpr uint32_t small_waves(uint32_t bytes) {
  return bytes / EncGeo<T, B>::RING;
}

// A single field of at most 64 KiB (float64: 96) in one launch of one workgroup: each wave
// reads its blocks once and keeps them in registers through their extrema, the
// bound, the plan, the codes and the packing; the waves meet at three
// barriers (finite range, ranks, byte counts), and no word of the workspace is
// used. Three launches spend a small call in their latencies and in look-backs:
// 4099 float32 values took 15.6 us a call in three, 7.3 in one.
template <typename T, int B, uint32_t NW>
__global__ __launch_bounds__(64 * NW) void k_small(CBatch b) {
  using U = typename Traits<T>::U;
  using G = EncGeo<T, B>;
  constexpr int EPL = G::EPL, LPB = G::LPB, SUB = G::SUB;
  constexpr int BYTES = Traits<T>::BYTES;
  __shared__ uint64_t s_lo[NW], s_hi[NW];
  __shared__ uint32_t s_nc[NW], s_tot[NW];
  __shared__ uint32_t s_state[NW * G::WBLK / 32 + 1];
  __shared__ __align__(16) uint8_t s_ring[NW * (G::RING + G::SLACK)];
  const FieldC f = field_at<kSingle>(b, 0);
  const uint32_t n = (uint32_t)f.n, nblk = (uint32_t)f.nblk;
  const uint32_t wave = uniform(threadIdx.x / kWave), nw = blockDim.x / kWave;
  const uint32_t lane = (uint32_t)lane_id(), lig = lane % LPB;
  uint8_t* const stage = s_ring + wave * (G::RING + G::SLACK);
  for (uint32_t i = threadIdx.x; i < NW * G::WBLK / 32 + 1; i += blockDim.x) s_state[i] = 0;

  T x[SUB][EPL];
  const __amdgpu_buffer_rsrc_t rs = buffer_of(f.in, n * (uint32_t)sizeof(T));
#pragma unroll
  for (int s = 0; s < SUB; ++s) row_load<T, B, EPL>(x[s], rs, wave, s, 1u);
  // every block's extrema (in all its lanes) and the field's finite range
  auto count = [&](int s) -> int {
    const int rem = (int)n - (int)((wave * G::WBLK + (uint32_t)(s * G::GPW) + lane / LPB) * B + lig * EPL);
    return rem < 0 ? 0 : (rem > EPL ? EPL : rem);
  };
  U kmin[SUB], kmax[SUB], flo = (U)~(U)0, fhi = 0;
#pragma unroll
  for (int s = 0; s < SUB; ++s) {
    const int cnt = count(s);
    U lo = (U)~(U)0, hi = 0;
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const U k = order_key<U>(bits_of(x[s][i]));
      lo = (i < cnt && k < lo) ? k : lo;
      hi = (i < cnt && k > hi) ? k : hi;
    }
    lo = group_min<LPB, U>(lo);
    hi = group_max<LPB, U>(hi);
    kmin[s] = lo;
    kmax[s] = hi;
    if (lo >= FiniteKeys<T>::LO && hi <= FiniteKeys<T>::HI) {  // an absent block leaves the range as it is
      flo = lo < flo ? lo : flo;
      fhi = hi > fhi ? hi : fhi;
    } else {
#pragma unroll
      for (int i = 0; i < EPL; ++i) {
        const U u = bits_of(x[s][i]);
        const U k = order_key<U>(u);
        const bool fin = i < cnt && is_finite_bits<T>(u);
        flo = (fin && k < flo) ? k : flo;
        fhi = (fin && k > fhi) ? k : fhi;
      }
    }
  }
  flo = group_min<kWave, U>(flo);
  fhi = group_max<kWave, U>(fhi);
  if (lane == 0) {
    s_lo[wave] = flo == (U)~(U)0 ? ~0ull : (uint64_t)flo;
    s_hi[wave] = fhi;
  }
  __syncthreads();
  uint64_t glo = ~0ull, ghi = 0;
  for (uint32_t i = 0; i < nw; ++i) {
    glo = s_lo[i] < glo ? s_lo[i] : glo;
    ghi = s_hi[i] > ghi ? s_hi[i] : ghi;
  }
  const uint64_t e_bits = f.eb_mode == 1 ? bound_of(f, glo, ghi) : bound_of(f, ~0ull, 0ull);
  const T e = from_bits<T>((U)e_bits);

  // plans, state bits and ranks
  BlockPlan<T> plan[SUB];
  uint32_t wnc = 0;
#pragma unroll
  for (int s = 0; s < SUB; ++s) {
    const uint32_t lk = wave * G::WBLK + (uint32_t)(s * G::GPW) + lane / LPB;
    plan[s] = plan_block<T>(kmin[s], kmax[s], e);
    if (lk >= nblk) plan[s].K = 0;
    const bool nc = plan[s].K != 0;
    if (nc && lig == 0) atomicOr(&s_state[lk / 32], 1u << (lk % 32));
    wnc += (uint32_t)__popcll(__ballot(nc) & first_lanes<LPB>());
  }
  if (lane == 0) s_nc[wave] = wnc;
  __syncthreads();
  uint32_t n_nc = 0, wrank = 0;
  for (uint32_t i = 0; i < nw; ++i) {
    wrank += i < wave ? s_nc[i] : 0u;
    n_nc += s_nc[i];
  }
  for (uint32_t i = threadIdx.x; i < (nblk + 7) / 8; i += blockDim.x)
    f.out[96 + i] = (uint8_t)(s_state[i / 4] >> (8 * (i % 4)));
  const Sections sec = sections(nblk, n_nc, BYTES, B, 0);
  T* const mus = reinterpret_cast<T*>(f.out + sec.mu);

  uint32_t wbytes = 0;
#pragma unroll
  for (int s = 0; s < SUB; ++s) {
    const uint32_t lk = wave * G::WBLK + (uint32_t)(s * G::GPW) + lane / LPB;
    int K = plan[s].K;
    const bool stored = K != 0;
    T mu = plan[s].mu;
    const uint64_t has = __ballot(stored);
    if (has != 0) {
      const int cnt = count(s);
      const bool tail = __ballot(stored && cnt != EPL) != 0;
      RowWords<T, B> w;
      w.code(x[s], mu, K, K > 0 && plan[s].verify, __ballot(K < 0 || (K > 0 && plan[s].verify)) != 0, e, cnt, tail, lig);
      if (K < 0) mu = (T)0;
      const uint32_t inc = wave_incl_sum_u32(w.lb);
      const uint64_t firsts = has & first_lanes<LPB>();
      const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
          (uint32_t)(firsts >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)firsts, wrank - (lig != 0 ? 1u : 0u)));
      wrank += (uint32_t)__popcll(firsts);
      if (stored) {
        if (lig == 0) f.out[sec.kbytes + rank] = K < 0 ? kRawK : (uint8_t)K;
        uint8_t* const cdst = f.out + sec.codes + (rank * (uint32_t)(B / 4) + lig * (EPL / 4));
        if constexpr (EPL == 8)
          *reinterpret_cast<uint16_t*>(cdst) = (uint16_t)(((w.codes >> 8) & 0xFFu) | ((w.codes & 0xFFu) << 8));
        else
          *reinterpret_cast<uint32_t*>(cdst) = __builtin_bswap32(w.codes);
      }
      const uint32_t start = uniform(lds_address(stage)) + wbytes + inc - w.lb, end = start + w.lb;
      RunPacker pk(end);
      w.pack(pk, cnt, tail, end);
      pk.or_head(start);
      wbytes += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    }
    if (lig == 0 && lk < nblk) mus[lk] = mu;
  }
  if (lane == 0) s_tot[wave] = wbytes;
  __syncthreads();
  uint32_t mid_total = 0, before = 0;
  for (uint32_t i = 0; i < nw; ++i) {
    before += i < wave ? s_tot[i] : 0u;
    mid_total += s_tot[i];
  }
  copy_out(f.out, sec.mid + before, stage, 0, G::RING / 16 - 1, wbytes);
  const uint64_t total = write_stream_header(f, e_bits, n_nc, mid_total);
  if (threadIdx.x == 0) *f.out_size = total;
}

// -------------------------------------------------------------------- mid ---

constexpr uint32_t kMidBlocks = 8192, kMidTiles = 256;  // (at most 2^24 mid bytes)

// Classification and encoding of a single field of a few hundred tiles in one
// launch: a workgroup a tile, one row a wave. Every workgroup counts the
// field's non-constant blocks by itself, from the extrema and the bound (a
// wave tests 64 blocks at a time, so the counts are scalar ones), which takes
// the place of the classification pass and its scan; each tile's own plans
// stay in registers. Tiles are few enough for a wave to read every earlier
// tile's byte count at once, four a lane, so the offset is one trip to the
// device's coherence point after the last of them is published. (A tile waits
// only on lower-numbered ones, which publish before they wait.) The last tile
// ends the stream; it has seen every tile's count, so every tile has read the
// range, and it clears the slots for the next call.
//
// Bound: latencies (a launch, the extrema, the earlier tiles' counts) and the
// count, 22 vector instructions for 64 blocks: 365x731 float64 values, b = 128,
// absolute bound, 17.9 us a call in three launches, 12.4 in two; 2^20 float32
// values 18.4 and 15.2. With a scan workgroup, an offset takes two trips: 196608
// float32 values 12.9 us, so 11.3.
template <typename T, int B>
__global__ __launch_bounds__((64 * EncGeo<T, B>::ROWS)) void k_mid(CBatch b) {
  using U = typename Traits<T>::U;
  using G = EncGeo<T, B>;
  constexpr int EPL = G::EPL, LPB = G::LPB, BYTES = Traits<T>::BYTES;
  constexpr uint32_t NW = G::ROWS, RING = G::RING / G::SUB;
  constexpr int U4 = 4;  // words of 64 blocks in flight
  __shared__ uint32_t s_all[NW], s_ahead[NW], s_row[NW], s_tot[NW], s_base, s_ok;
  __shared__ __align__(16) uint8_t s_ring[NW * (RING + G::SLACK)];
  const FieldC f = field_at<kSingle>(b, 0);
  const uint32_t nblk = (uint32_t)f.nblk, t = blockIdx.x, kb = t * G::TBLK;
  const bool last = t + 1 == gridDim.x;
  const uint32_t wave = uniform(threadIdx.x / kWave);
  const uint32_t lane = (uint32_t)lane_id(), lig = lane % LPB;
  const uint32_t lk = wave * G::GPW + lane / LPB;  // the lane's block of the tile

  // the extrema of a block, and of the field's blocks 64 at a time
  using v2u = unsigned int __attribute__((ext_vector_type(2)));
  using v4u = unsigned int __attribute__((ext_vector_type(4)));
  const __amdgpu_buffer_rsrc_t re = buffer_of(f.stats, nblk * 2u * (uint32_t)sizeof(U));
  auto extrema = [&](uint32_t k, U& lo, U& hi) {
    if constexpr (sizeof(U) == 4) {
      const v2u u = __builtin_amdgcn_raw_buffer_load_b64(re, (int)(k * 8u), 0, 0);
      lo = u.x;
      hi = u.y;
    } else {
      const v4u u = __builtin_amdgcn_raw_buffer_load_b128(re, (int)(k * 16u), 0, 0);
      lo = ((uint64_t)u.y << 32) | u.x;
      hi = ((uint64_t)u.w << 32) | u.z;
    }
  };
  const uint32_t words = (nblk + 63) / 64;
  U lo[U4], hi[U4], kmin, kmax;
#pragma unroll
  for (int u = 0; u < U4; ++u) extrema((wave + (uint32_t)u * NW) * 64u + lane, lo[u], hi[u]);
  extrema(kb + lk, kmin, kmax);
  T x[EPL];
  {
    const uint64_t i0 = (uint64_t)kb * B;
    const __amdgpu_buffer_rsrc_t rs =
        buffer_of(reinterpret_cast<const T*>(f.in) + i0,
                  (uint32_t)std::min<uint64_t>(f.n - i0, (uint64_t)G::TBLK * B) * (uint32_t)sizeof(T));
    row_load<T, B, EPL>(x, rs, 0, (int)wave, 1u);
  }
  uint64_t e_bits;
  if (f.eb_mode != 1) {
    e_bits = bound_of(f, ~0ull, 0ull);
  } else {
    const bool clean = *f.clean == kCleanWord;
    e_bits = slots_bound(f);  // (of any words where they are not clean)
    if (!clean) {  // first use of the workspace: the chunks' partials
      const uint64_t nchunks = cdiv(cdiv(f.n, (uint64_t)Geo<T, B>::TILE), (uint64_t)kStatsChunk);
      uint64_t plo = ~0ull, phi = 0;
      for (uint64_t i = lane; i < nchunks; i += kWave) {
        const ulonglong2 p = reinterpret_cast<const ulonglong2*>(f.parts)[i];
        plo = p.x < plo ? p.x : plo;
        phi = p.y > phi ? p.y : phi;
      }
      e_bits = bound_of(f, group_min<kWave, uint64_t>(plo), group_max<kWave, uint64_t>(phi));
    }
  }
  const T e = from_bits<T>((U)e_bits);

  uint32_t all = 0, ahead = 0;
  for (uint32_t w0 = wave; w0 < words; w0 += U4 * NW) {
    U nlo[U4], nhi[U4];
#pragma unroll
    for (int u = 0; u < U4; ++u) extrema((w0 + (uint32_t)(U4 + u) * NW) * 64u + lane, nlo[u], nhi[u]);
#pragma unroll
    for (int u = 0; u < U4; ++u) {
      const uint32_t k0 = (w0 + (uint32_t)u * NW) * 64u;
      if (u > 0 && k0 >= nblk) break;
      const uint64_t m = stored_blocks<T>(lo[u], hi[u], e, k0 + lane < nblk);
      const uint64_t below = k0 + 64u <= kb ? ~0ull : k0 >= kb ? 0ull : (1ull << (kb - k0)) - 1ull;
      all += (uint32_t)__popcll(m);
      ahead += (uint32_t)__popcll(m & below);
      // state bits leave with the tile of their first block
      if (k0 - kb < (uint32_t)G::TBLK && lane == 0) {
        uint8_t* const to = f.out + 96 + k0 / 8;
        if (k0 + 64u <= nblk) {
          *reinterpret_cast<uint64_t*>(to) = m;
        } else {
          for (uint32_t i = 0; i < (nblk - k0 + 7) / 8; ++i) to[i] = (uint8_t)(m >> (8 * i));
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U4; ++u) {
      lo[u] = nlo[u];
      hi[u] = nhi[u];
    }
  }
  BlockPlan<T> plan = plan_block<T>(kmin, kmax, e);
  const bool present = kb + lk < nblk;
  if (!present) plan.K = 0;
  int K = plan.K;
  T mu = plan.mu;
  const uint64_t has = __ballot(K != 0);
  if (lane == 0) {
    s_all[wave] = all;
    s_ahead[wave] = ahead;
    s_row[wave] = (uint32_t)__popcll(has & first_lanes<LPB>());
  }
  __syncthreads();
  uint32_t n_nc = 0, rank0 = 0;
#pragma unroll
  for (uint32_t i = 0; i < NW; ++i) {
    n_nc += s_all[i];
    rank0 += s_ahead[i] + (i < wave ? s_row[i] : 0u);
  }
  n_nc = uniform(n_nc);
  rank0 = uniform(rank0);

  const Sections sec = sections(nblk, n_nc, BYTES, B, 0);
  const uint32_t ring0 = uniform(lds_address(s_ring + wave * (RING + G::SLACK)));
  uint32_t wbytes = 0;
  if (has != 0) {
    const int rem = (int)(uint32_t)std::min<uint64_t>(f.n - (uint64_t)kb * B, (uint64_t)G::TBLK * B) -
                    (int)(lk * B + lig * EPL);
    const int cnt = rem < 0 ? 0 : (rem > EPL ? EPL : rem);
    const bool stored = K != 0;
    const bool tail = __ballot(stored && cnt != EPL) != 0;
    RowWords<T, B> w;
    w.code(x, mu, K, K > 0 && plan.verify, __ballot(K < 0 || (K > 0 && plan.verify)) != 0, e, cnt, tail, lig);
    if (K < 0) mu = (T)0;
    const uint32_t inc = wave_incl_sum_u32(w.lb);
    const uint64_t firsts = has & first_lanes<LPB>();
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
        (uint32_t)(firsts >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)firsts, rank0 - (lig != 0 ? 1u : 0u)));
    wbytes = (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);
    const uint32_t start = ring0 + inc - w.lb, end = start + w.lb;
    RunPacker pk(end);
    w.pack(pk, cnt, tail, end);
    pk.or_head(start);
    if (stored) {
      if (lig == 0) f.out[sec.kbytes + rank] = K < 0 ? kRawK : (uint8_t)K;
      uint8_t* const cdst = f.out + sec.codes + ((uint64_t)rank * (uint32_t)(B / 4) + lig * (EPL / 4));
      if constexpr (EPL == 8)
        *reinterpret_cast<uint16_t*>(cdst) = (uint16_t)(((w.codes >> 8) & 0xFFu) | ((w.codes & 0xFFu) << 8));
      else
        *reinterpret_cast<uint32_t*>(cdst) = __builtin_bswap32(w.codes);
    }
  }
  if (lig == 0 && present) reinterpret_cast<T*>(f.out + sec.mu)[kb + lk] = mu;
  if (lane == 0) s_tot[wave] = wbytes;
  __syncthreads();
  uint32_t total = 0, before = 0;
#pragma unroll
  for (uint32_t i = 0; i < NW; ++i) {
    const uint32_t v = uniform(s_tot[i]);
    before += i < wave ? v : 0u;
    total += v;
  }
  if (threadIdx.x == 0) status_store(f.enc_mid + t, kFlagAgg | total);
  if (last) {
    write_stream_header(f, e_bits, n_nc, 0);
    if (threadIdx.x == 0) {
      f.ctr->n_nc = n_nc;
      *f.out_size = kSizePending;
    }
  }
  if (wave == 0) {
    constexpr int R = (int)kMidTiles / kWave;
    uint32_t sum = 0, spins = 0;
    bool ok = true;
    for (;;) {
      bool missing = false;
      sum = 0;
#pragma unroll
      for (int r = 0; r < R; ++r) {
        // (lanes past the tile read word 0, as its wait may need it anyway)
        const uint32_t j = (uint32_t)(r * kWave) + lane;
        const uint64_t w = status_load(f.enc_mid + (j < t ? j : 0u));
        missing |= j < t && (w >> 62) == 0;
        sum += j < t ? (uint32_t)w : 0u;
      }
      if (__ballot(missing) == 0) break;
      if (++spins > kSpinLimit) {
        ok = false;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    sum = wave_total_u32(sum);
    if (lane == 0) {
      s_base = sum;
      s_ok = ok;
    }
  }
  __syncthreads();
  const uint32_t base = uniform(s_base);
  if (s_ok == 0) {  // a bounded wait gave up: the field has no stream (finish_stream)
    if (threadIdx.x == 0) {
      atomicMax(&f.ctr->err, 1u);
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "agent");
      __hip_atomic_store(f.out_size, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (last) *f.clean = 0;  // the slots keep this call's range
    }
    return;
  }
  copy_out(f.out, sec.mid + base + before, s_ring + wave * (RING + G::SLACK), 0, RING / 16 - 1, wbytes);
  if (last) {
    if (threadIdx.x < kRangeSlots)
      *reinterpret_cast<ulonglong2*>(f.range + threadIdx.x * (kRangeStride / 8)) = make_ulonglong2(0, 0);
    if (threadIdx.x == 0) {
      *f.clean = kCleanWord;
      finish_stream(f, (uint64_t)base + total);
    }
  }
}

// --------------------------------------------------------------- finalize ---

// Fields without values, one workgroup a field of the call: they have no
// extrema, classification or encode tiles and get their whole header here (the
// bound from an empty range) and their size.
__global__ void k_finalize(CBatch b) {
  const FieldC f = field_at(b, blockIdx.x);
  if (f.nblk != 0) return;
  const int rel = f.eb_mode == 1;
  const uint64_t e_bits = f.dtype == 0 ? (uint64_t)bits_of(bound_from<float>(rel, f.eb, ~0ull, 0ull))
                                       : (uint64_t)bits_of(bound_from<double>(rel, f.eb, ~0ull, 0ull));
  const uint64_t total = write_stream_header(f, e_bits, 0, 0);
  if (threadIdx.x == 0) *f.out_size = total;
}

// ---------------------------------------------------------------- launch ---

// (The smallest fields ask for a half or a third of the LDS, so that a busy compute unit
// takes them too.)
template <typename T, int B>
void launch_small(const CBatch& b, hipStream_t stream) {
  constexpr uint32_t few = small_waves<T, B>(kSmallestBytes), all = small_waves<T, B>(kSmallBytes<T>);
  const uint32_t waves = (uint32_t)cdiv(b.one.nblk, EncGeo<T, B>::WBLK);
  if (waves <= few)
    k_small<T, B, few><<<1, 64 * waves, 0, stream>>>(b);
  else
    k_small<T, B, all><<<1, 64 * waves, 0, stream>>>(b);
}

template <int B>
hipError_t launch_compress_b(const CBatch& b, const CLaunchGeom& g, hipStream_t stream, TimerHook hook) {
  auto run = [&](const char* name, auto&& fn) {
    if (hook) hook(name, stream, 1);
    fn();
    if (hook) hook(name, stream, 0);
  };
  // The lines lie where the ways meet (b = 128, us a call): one launch of one
  // workgroup takes 8.5 at 64 KiB of float32 values, 10.9 at 96 KiB, two launches
  // 10.1 and 10.3; float64 8.3 at 64 KiB, 10.5 at 96, 12.1 at 128 and 11.4, 10.6,
  // 11.3. Other block sizes meet there too: 64 KiB of float32 take 10.4, 8.5, 8.9, 9.0
  // and 9.0 in one and 12.2, 10.9, 11.0, 11.0 and 11.3 in two at b = 8, 32, 256, 512 and
  // 1024; 96 KiB of float64 10.4, 10.2, 10.8, 10.9 and 12.0, and 12.4, 11.3, 12.3, 12.3 and
  // 15.1. (Fields of raw blocks alone would meet at 32 and 64 KiB: b = 128, 64 KiB of float32
  // 13.6 and 12.4, 96 KiB of float64 17.0 and 12.8; three launches took 20. A shard's
  // bound comes from elsewhere.)
  const bool single = !b.fields && !b.any_empty && b.one.next_range == 0;
  if (single && b.one.n * (b.one.dtype == 0 ? 4 : 8) <= (b.one.dtype == 0 ? kSmallBytes<float> : kSmallBytes<double>)) {
    if (b.one.dtype == 0)
      run("k_small", [&] { launch_small<float, B>(b, stream); });
    else
      run("k_small", [&] { launch_small<double, B>(b, stream); });
    return hipGetLastError();
  }
  // Two launches or three: beyond one tile a compute unit the persistent
  // encoder overlaps its tiles, and every workgroup's count grows with the
  // blocks. float32, b = 128: 8192 blocks in 128 tiles 15.2 us in two, 18.4 in
  // three; 16384 blocks 19.4 and 18.9; b = 256, 256 tiles 16.7 and 19.2, 320
  // tiles 21.6 and 21.0. float64, b = 128: 8192 blocks in 256 tiles 17.5 and
  // 18.9, 10240 in 320 22.1 and 20.3. Within the lines two are faster at every block
  // size, for raw blocks too: 8192 blocks or 256 tiles at b = 8, 32, 512 and 1024 take 13.7,
  // 14.8, 15.8 and 15.2 in two, 19.1, 18.2, 19.1 and 19.7 in three (float64 15.3, 16.4, 15.3 and
  // 18.8, and 18.4, 18.6, 19.5 and 25.0).
  if (single && b.one.nblk <= kMidBlocks && b.tiles_enc[0] + b.tiles_enc[1] <= kMidTiles) {
    const uint32_t gs = (uint32_t)(b.tiles_stats[0] + b.tiles_stats[1]);
    const uint32_t ge = (uint32_t)(b.tiles_enc[0] + b.tiles_enc[1]);
    if (b.one.dtype == 0) {
      run("k_stats", [&] { k_stats<float, B><<<gs, 256, 0, stream>>>(b); });
      run("k_mid", [&] { k_mid<float, B><<<ge, 64 * EncGeo<float, B>::ROWS, 0, stream>>>(b); });
    } else {
      run("k_stats", [&] { k_stats<double, B><<<gs, 256, 0, stream>>>(b); });
      run("k_mid", [&] { k_mid<double, B><<<ge, 64 * EncGeo<double, B>::ROWS, 0, stream>>>(b); });
    }
    return hipGetLastError();
  }
  // at least one workgroup per ticket class: tiles of a class without one
  // would never be encoded (and every later tile would wait for them)
  auto encoders = [&](int dt) {
    return (uint32_t)std::min<uint64_t>(b.tiles_enc[dt], std::max<uint64_t>(g.encode_wgs[dt], kTicketClasses));
  };
  bool done = b.tiles_stats[0] + b.tiles_stats[1] == 0, encoded = false;
  if constexpr (kOneLaunch<B>) {
    if (b.fields && b.tiles_stats[0] && b.tiles_stats[1]) {
      const uint32_t gs = (uint32_t)(b.tiles_stats[0] + b.tiles_stats[1]);
      const uint32_t gc = (uint32_t)(b.tiles_cls[0] + b.tiles_cls[1]);
      const uint32_t ge = std::max(encoders(0), encoders(1)) + 2;  // two scan workgroups
      run("k_stats", [&] { k_stats_both<B><<<gs, 256, 0, stream>>>(b); });
      run("k_classify", [&] { k_classify_both<B><<<gc, 256, 0, stream>>>(b); });
      encoded = one_encode_launch(b.tiles_enc[0], b.tiles_enc[1]);
      if (encoded) run("k_encode", [&] { k_encode_both<B><<<ge, 256, 0, stream>>>(b); });
      done = true;
    }
  }
  if (!done) {
    if (b.tiles_stats[0]) run("k_stats", [&] { k_stats<float, B><<<(uint32_t)b.tiles_stats[0], 256, 0, stream>>>(b); });
    if (b.tiles_stats[1]) run("k_stats", [&] { k_stats<double, B><<<(uint32_t)b.tiles_stats[1], 256, 0, stream>>>(b); });
    if (b.tiles_cls[0]) run("k_classify", [&] { k_classify<float, B><<<(uint32_t)b.tiles_cls[0], 256, 0, stream>>>(b); });
    if (b.tiles_cls[1]) run("k_classify", [&] { k_classify<double, B><<<(uint32_t)b.tiles_cls[1], 256, 0, stream>>>(b); });
  }
  if (!encoded) {
    for (int dt = 0; dt < 2; ++dt) {
      if (!b.tiles_enc[dt]) continue;
      const uint32_t genc = encoders(dt);
      const bool batch = b.fields != nullptr;
      // workgroup 0 is the scan workgroup
      if (dt == 0 && !batch)
        run("k_encode", [&] { k_encode<float, B, kSingle><<<genc + 1, 256, 0, stream>>>(b); });
      else if (dt == 0)
        run("k_encode", [&] { k_encode<float, B, kBatch><<<genc + 1, 256, 0, stream>>>(b); });
      else if (!batch)
        run("k_encode", [&] { k_encode<double, B, kSingle><<<genc + 1, 256, 0, stream>>>(b); });
      else
        run("k_encode", [&] { k_encode<double, B, kBatch><<<genc + 1, 256, 0, stream>>>(b); });
    }
  }
  if (b.any_empty) run("k_finalize", [&] { k_finalize<<<b.nfields, 64, 0, stream>>>(b); });
  return hipGetLastError();
}

hipError_t launch_compress(const CBatch& b, uint32_t block, const CLaunchGeom& g, hipStream_t stream,
                           TimerHook hook) {
  switch (block) {
    case 8: return launch_compress_b<8>(b, g, stream, hook);
    case 16: return launch_compress_b<16>(b, g, stream, hook);
    case 32: return launch_compress_b<32>(b, g, stream, hook);
    case 64: return launch_compress_b<64>(b, g, stream, hook);
    case 128: return launch_compress_b<128>(b, g, stream, hook);
    case 256: return launch_compress_b<256>(b, g, stream, hook);
    case 512: return launch_compress_b<512>(b, g, stream, hook);
    case 1024: return launch_compress_b<1024>(b, g, stream, hook);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace szx
