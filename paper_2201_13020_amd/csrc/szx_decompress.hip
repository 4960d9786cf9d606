// szx_decompress.hip -- decompression kernels of the SZx method for gfx950.
//
// Two kernels per call:
//   k_dindex  over tiles of consecutive blocks: state bits give each tile's
//             non-constant blocks and their ranks (hence their K byte and
//             codes) -- the population count of the state bits before the
//             tile for the first 256 tiles, a light single-pass prefix count
//             after them; per value the number of stored mid bytes is the kept
//             bytes minus the leading bytes its 2-bit code shares, and their
//             prefix sum gives the first mid byte of every wave of a decode
//             tile (Sec. V-B locates the mid bytes by a prefix sum of these
//             counts before they are read). Where every field has at most 256
//             index tiles the tiles wait on nothing: each leaves its total,
//             which the decode tiles add up. Else a second light prefix sum
//             chains them, and workgroup 0 first clears the status words of
//             both (a gate holds the others).
//   k_decode  every wave of a decode tile on its own, no waiting: it stages its
//             mid bytes in LDS with aligned 16-byte loads, resolves leading
//             bytes -- byte j of value i is the stored byte j of the nearest
//             value i' <= i whose code stores byte j (Sec. V-B, index
//             propagation) -- lane by lane, then across the lanes of a block
//             with one inclusive scan over (code, top bytes) pairs under the
//             associative operator (c_a, S_a) . (c_b, S_b) = (min(c_a, c_b),
//             (S_a & top(c_b)) | S_b), and writes x' = mu + (q' << s);
//             constant blocks get mu, raw blocks their stored bytes.
// Every read of the stream is bounded by in_bytes; a malformed stream sets
// *status = SZ_ECORRUPT and no access leaves the given buffers.
#include <algorithm>

#include "szx_device.hpp"
#include "szx_launch.hpp"

namespace szx {

constexpr uint32_t kStatusCorrupt = 3;  // SZ_ECORRUPT
constexpr uint32_t kStatusDevice = 4;   // SZ_EDEVICE: a bounded wait gave up

// Field of a call, or of a batch entry (a copy with its pointers typed as
// global memory).
__device__ __forceinline__ FieldD field_at(const DBatch& b, uint32_t fi) {
  FieldD f;
  if (b.fields)
    f = *as_constant(b.fields + fi);
  else
    f = b.one;
  f.in = as_global(f.in);
  f.out = as_global(f.out);
  f.status = as_global(f.status);
  f.index = as_global(f.index);
  f.rank_st = as_global(f.rank_st);
  f.mid_st = as_global(f.mid_st);
  return f;
}
__device__ __forceinline__ uint32_t dfield_of(const uint32_t* map, uint64_t t) { return map ? *as_constant(map + t) : 0u; }

// Only for calls without index tiles (every field empty): their status words.
__global__ __launch_bounds__(256) void k_dinit(DBatch b) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t nf = b.fields ? b.nfields : 1;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nf; i += stride) *field_at(b, (uint32_t)i).status = 0;
}

// ---------------------------------------------------------------- gate ---
// (Only the chained index has one.) The index pass's status words and every field's status word must be zero
// before any index tile publishes or reports an error, and no launch of its
// own clears them. Workgroup 0 of the call's first index launch (dispatched
// first) clears them and then stores the call's token in the go word; every
// other workgroup waits for the token before its first publish or report
// (its stream loads are already out). A second index launch (b = 1024, both
// types) finds the token there and clears nothing. The token changes with
// every call: the last decode launch advances the epoch it comes from, when
// no index tile reads it any more.
__device__ __forceinline__ uint64_t gate_token(const DBatch& b) {
  return status_load(as_global(b.gate) + kGateEpochWord) ^ kGateKey;
}

__device__ __forceinline__ void gate_open(const DBatch& b, int* s_flag) {
  uint64_t* gate = as_global(b.gate);
  if (threadIdx.x == 0) *s_flag = status_load(gate + kGateGoWord) != gate_token(b);
  __syncthreads();
  if (!*s_flag) return;  // the same in every thread
  for (uint64_t i = threadIdx.x; i < b.zero_words; i += kWG) status_store(as_global(b.zero_begin) + i, 0);
  const uint32_t nf = b.fields ? b.nfields : 1u;
  for (uint32_t i = threadIdx.x; i < nf; i += kWG)
    __hip_atomic_store((__attribute__((address_space(1))) uint32_t*)field_at(b, i).status, 0u, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  // every wave's stores are performed before the barrier (a release only: an
  // acquire would also drop this XCD's L2)
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __syncthreads();
  if (threadIdx.x == 0) status_store(gate + kGateGoWord, gate_token(b));
}

// Every workgroup but 0 waits for the token before its first publish or
// error report. Its later reads of the cleared words are device-scope atomic
// loads issued after the token is seen, so they need no fence (a fence here
// would drop the XCD's L2 for every tile). Workgroup 0 opens the gate right
// after its descriptor and header loads (a store ahead of them would keep the
// compiler from making them scalar loads), while the others load their state
// bits.
__device__ __forceinline__ void gate_wait(const DBatch& b, uint32_t* status) {
  if (blockIdx.x == 0) return;
  if (threadIdx.x == 0) {
    const uint64_t* go = as_global(b.gate) + kGateGoWord;
    const uint64_t tok = gate_token(b);
    uint32_t spins = 0;
    while (status_load(go) != tok) {
      if (++spins > kSpinLimit) {
        atomicMax(status, kStatusDevice);
        break;
      }
      __builtin_amdgcn_s_sleep(2);
    }
  }
  __syncthreads();
}

__device__ __forceinline__ void gate_advance(const DBatch& b) {
  __hip_atomic_fetch_add((__attribute__((address_space(1))) uint64_t*)(as_global(b.gate) + kGateEpochWord), 1ull,
                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Header words (nothing writes a stream that is being decoded: scalar loads).
__device__ __forceinline__ uint64_t rd64(const uint8_t* p) { return *as_constant(reinterpret_cast<const uint64_t*>(p)); }
__device__ __forceinline__ uint32_t rd32(const uint8_t* p) { return *as_constant(reinterpret_cast<const uint32_t*>(p)); }

// Mask of the top c bytes (c in [0, 3]) of the 24-bit leading field kept in
// bits 31..8, branch-free: the field's mask shifted left by 8 (3 - c).
__device__ __forceinline__ uint32_t lead_mask(uint32_t c) { return 0xFFFFFF00u << (8u * (3u - c)); }

// Composition of two leading-byte transforms packed as (S in bits 31..8, c in
// bits 1..0): first `a`, then `b`.
__device__ __forceinline__ uint32_t lead_compose(uint32_t a, uint32_t b) {
  const uint32_t ca = a & 3u, cb = b & 3u;
  const uint32_t s = ((a & 0xFFFFFF00u) & lead_mask(cb)) | (b & 0xFFFFFF00u);
  return s | (ca < cb ? ca : cb);
}

// Geometry of the decode pass: a workgroup's tile is about 16 KiB of values (at
// least 8 blocks, so that it owns whole state bytes), each of its four waves a
// contiguous quarter of it, in SUB rows (mostly one) of EPL consecutive values
// a lane. Sixteen float32 values a lane share the per-row work among twice the
// values of eight (with eight, and tiles of 8 KiB: 42 us where sixteen take 35).
constexpr uint32_t kStageHead = 16;
template <typename T, int B>
struct DecGeo {
  static constexpr int EPL = (int)lane_values(B, sizeof(T));
  static constexpr int LPB = B / EPL;       // lanes per block
  static constexpr int GPW = kWave / LPB;   // blocks per row
  static constexpr int ROW = kWave * EPL;   // values per row
  static constexpr int TBLK = (int)dec_blocks(B, sizeof(T));
  static constexpr int WBLK = TBLK / kWavesPerWG;  // blocks per wave
  static constexpr int SUB = WBLK / GPW;    // rows per wave
  static constexpr uint32_t MOST = (uint32_t)(ROW * SUB * (int)sizeof(T));  // mid bytes of a wave
  // the wave's LDS stage: kStageHead bytes that reads before the first mid
  // byte may touch, its mid bytes at most, the 15-byte misalignment of
  // their start and the round-up to whole 16-byte chunks, then room for the
  // unguarded reads of a lane: it starts at most at the end of all stored
  // bytes, advances at most a word per value before its last read, and a read
  // takes up to 12 bytes
  static constexpr uint32_t STAGE = kStageHead + MOST + 32u + (uint32_t)(EPL * (int)sizeof(T)) + 16u;
  static_assert(LPB >= 1 && LPB <= 64 && SUB * GPW * kWavesPerWG == TBLK, "whole rows");
  static_assert(STAGE % 16 == 0, "stages start 16-byte aligned");
  // Waves per SIMD, as the LDS allows; sixteen float32 values a lane take 76
  // registers, so six (held to eight waves they spill: 35 -> 50 us for the
  // decompression of the 100x500x500 float32 field at REL 1e-3).
  static constexpr int WAVES = STAGE > 17000u ? 2 : STAGE > 5000u ? 4 : sizeof(T) == 4 && EPL == 16 ? 6 : 8;
};

// Four bytes at LDS byte offset off of the staged stream, the first in the low
// byte: two aligned dwords and a byte funnel shift (an unaligned LDS read takes
// a clock a lane, 64 against 9).
__device__ __forceinline__ uint32_t stage_get(const uint8_t* stage, uint32_t off) {
  const uint32_t* p = reinterpret_cast<const uint32_t*>(stage + (off & ~3u));
  return __builtin_amdgcn_alignbyte(p[1], p[0], off);
}

// The lane's codes with those of values past cn cleared (first value in the
// top bits).
template <int EPL>
__device__ __forceinline__ uint32_t valid_codes(uint32_t c, int cn) {
  return c & (uint32_t)(((1ull << (2 * cn)) - 1) << (2 * (EPL - cn)));
}

// Smallest of a lane's EPL two-bit codes.
template <int EPL>
__device__ __forceinline__ uint32_t min_code(uint32_t c) {
  constexpr uint32_t LO = EPL == 16 ? 0x55555555u : 0x5555u;
  const uint32_t hi = (c >> 1) & LO, lo = c & LO;
  return hi == LO ? (lo == LO ? 3u : 2u) : ((hi | lo) == LO ? 1u : 0u);
}

// D lanes before, within groups of G lanes (lanes with lig < D get garbage,
// which callers discard): DPP row shifts for G <= 16.
template <int G, int D>
__device__ __forceinline__ uint32_t lane_up(uint32_t v) {
  if constexpr (G <= 16) {
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x110 + D, 0xF, 0xF, false);  // row_shr:D
  } else {
    return __shfl_up(v, D, G);
  }
}

// Header of the stream, checked against the caller's expectations; identical
// in every workgroup.
struct StreamInfo {
  bool ok;
  uint64_t n_nc, mid_total;
  Sections sec;
};

template <int BYTES, int B>
__device__ __forceinline__ StreamInfo read_header(const FieldD& a) {
  StreamInfo h;
  const uint8_t* in = a.in;
  h.ok = a.in_bytes >= kHeaderBytes;
  h.n_nc = 0;
  h.mid_total = 0;
  h.sec = sections(a.nblk, 0, BYTES, B, 0);
  if (h.ok) {
    const uint32_t w1 = rd32(in + 4);
    h.ok = rd32(in) == kMagic && (w1 & 0xFFu) == kVersion && ((w1 >> 8) & 0xFFu) == a.dtype &&
           ((w1 >> 16) & 0xFFu) <= 1 && ((w1 >> 24) & 0xFFu) == a.ndims && rd32(in + 8) == (uint32_t)B &&
           rd64(in + 48) == a.n && rd64(in + 72) == a.nblk;
    for (int d = 0; d < 4; ++d) h.ok = h.ok && rd64(in + 16 + 8 * d) == a.dims[d];
    h.n_nc = rd64(in + 80);
    h.mid_total = rd64(in + 88);
    h.ok = h.ok && h.n_nc <= a.nblk && h.mid_total <= a.n * BYTES;
    if (h.ok) {
      h.sec = sections(a.nblk, h.n_nc, BYTES, B, h.mid_total);
      h.ok = h.sec.total <= a.in_bytes;
    }
  }
  return h;
}

// A block's code bytes as words of 16 codes (b = 8: one half word in the
// low 16 bits), read through a buffer resource at byte offset off (reads past
// its range return zeros). A block's codes start 16-byte aligned (the codes
// section is, and each block holds b / 4 bytes), so from b = 64 on they load
// as 16-byte words.
template <int B>
struct BlockCodes {
  static constexpr uint32_t NW = B >= 16 ? B / 16 : 1;
  uint32_t raw[NW];
};
template <int B>
__device__ __forceinline__ void load_codes(__amdgpu_buffer_rsrc_t rs, uint32_t off, BlockCodes<B>& c) {
  using v4u = unsigned int __attribute__((ext_vector_type(4)));
  if constexpr (B >= 64) {
#pragma unroll
    for (uint32_t q = 0; q < BlockCodes<B>::NW / 4; ++q) {
      const v4u u = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(off + 16u * q), 0, 0);
      c.raw[4 * q + 0] = u.x;
      c.raw[4 * q + 1] = u.y;
      c.raw[4 * q + 2] = u.z;
      c.raw[4 * q + 3] = u.w;
    }
  } else if constexpr (B >= 16) {
#pragma unroll
    for (uint32_t j = 0; j < BlockCodes<B>::NW; ++j)
      c.raw[j] = __builtin_amdgcn_raw_buffer_load_b32(rs, (int)(off + 4u * j), 0, 0);
  } else {
    c.raw[0] = __builtin_amdgcn_raw_buffer_load_b16(rs, (int)off, 0, 0);
  }
}

// Mid bytes of one non-constant block of nk values with K byte Kb and codes
// c; raises bad for a K outside [1 + E, W] or a code above the kept bytes.
template <typename T, int B>
__device__ __forceinline__ uint32_t block_mid_bytes(const BlockCodes<B>& c, uint32_t Kb, uint32_t nk, bool& bad) {
  constexpr int BYTES = Traits<T>::BYTES;
  if (Kb == kRawK) return nk * BYTES;
  if ((int)Kb < Traits<T>::KMIN || (int)Kb > Traits<T>::W) {
    bad = true;
    return 0;
  }
  const uint32_t nb = (uint32_t)bytes_of((int)Kb);
  uint32_t sum = 0, over = 0;
  // b/4 code bytes, 4 codes per byte, first value in the top bits (a code's two
  // bits lie in one byte, so only the short last block needs their order)
  const bool brief = __ballot(nk < (uint32_t)B) != 0;
#pragma unroll
  for (uint32_t j = 0; j < BlockCodes<B>::NW; ++j) {
    uint32_t w = c.raw[j];
    if constexpr (B < 16) w &= 0xFFFFu;
    if (brief) {
      const uint32_t first = 16 * j;  // value index of the word's first code
      if (first >= nk) w = 0;
      else if (nk - first < 16) w &= __builtin_bswap32(~0u << (2 * (16 - (nk - first))));  // codes past the block end
    }
    sum += (uint32_t)__popc(w) + (uint32_t)__popc(w & 0xAAAAAAAAu);
    over |= w & (w >> 1) & 0x55555555u;  // a code of 3
  }
  if (nb == 2 && over) bad = true;
  return nk * nb - sum;
}

// An entry of the decode tiles' index: the tile's first mid byte (48 bits) and
// first rank (32), and the mid bytes before its waves 1, 2 and 3 (16 bits
// each: a tile holds at most 64 KiB).
__device__ __forceinline__ void index_store(uint64_t* e, uint64_t mid, uint64_t rank, uint32_t w1, uint32_t w2,
                                            uint32_t w3) {
  *reinterpret_cast<ulonglong2*>(e) =
      make_ulonglong2(mid | ((uint64_t)w1 << 48), rank | ((uint64_t)w2 << 32) | ((uint64_t)w3 << 48));
}
constexpr uint64_t kIndexMid = (1ull << 48) - 1;
// In a direct index the first mid byte counts from its index tile's start (24
// bits) and the tile's mid bytes follow it (17 bits).
__device__ __forceinline__ uint64_t index_direct(uint32_t mid, uint32_t bytes) { return mid | ((uint64_t)bytes << 24); }
constexpr uint32_t kTotalBad = 0x80000000u;  // in an index tile's total: the stream failed validation there
// A direct index's totals: each index tile's mid bytes, in place of status words.
__device__ __forceinline__ uint32_t* direct_totals(const FieldD& a) { return reinterpret_cast<uint32_t*>(a.mid_st); }

// How the index pass finds what lies before a tile: kChained by single-pass
// prefix sums, kDirect by counting it, kOne where the field is one index tile
// that every workgroup of the decode pass indexes for itself.
enum : int { kChained = 0, kDirect = 1, kOne = 2 };

// Per tile of CLS blocks (four per thread): ranks of the non-constant blocks
// and mid bytes, each through a light single-pass prefix sum; writes the index
// entry of every decode tile in it.
// kOne: the entry of decode tile dt goes to `entry` instead, and decode tile
// 0 sets the field's status; returns whether the tile may be decoded.
template <typename T, int B, int MODE>
__device__ __forceinline__ bool dindex_tile(const DBatch& b, const FieldD& a, uint32_t t, uint32_t* s_scan,
                                            uint64_t* s_r0p, uint64_t* s_m0p, uint32_t* s_wave, int* s_flag,
                                            uint32_t dt = 0, uint64_t* entry = nullptr) {
  constexpr bool DIRECT = MODE != kChained;
  constexpr int BYTES = Traits<T>::BYTES;
  constexpr int CLS = (int)kClsBlocks;
  constexpr int BPT = CLS / kWG;
  using D = DecGeo<T, B>;
  static_assert(D::TBLK % BPT == 0 && CLS % D::TBLK == 0, "every decode tile starts at some thread's first block");
  uint64_t& s_r0 = *s_r0p;
  uint64_t& s_m0 = *s_m0p;
  const StreamInfo h = read_header<BYTES, B>(a);
  if constexpr (DIRECT) {
    // tile 0 sets the field's status (the decode pass raises it), and the
    // launch's first workgroup those of fields without values
    if (t == 0 && dt == 0 && threadIdx.x == 0 && (MODE == kDirect || !h.ok)) *a.status = h.ok ? 0u : kStatusCorrupt;
    if (MODE == kDirect && blockIdx.x == 0 && b.any_empty && b.fields) {
      for (uint32_t i = threadIdx.x; i < b.nfields; i += kWG)
        if (b.fields[i].nblk == 0) *as_global(b.fields[i].status) = 0;
    }
    if (!h.ok) return false;
  } else {
    if (blockIdx.x == 0) gate_open(b, s_flag);
    if (!h.ok) {
      gate_wait(b, a.status);
      if (t == 0 && threadIdx.x == 0) atomicMax(a.status, kStatusCorrupt);
      return false;
    }
  }
  const uint32_t ntiles = (uint32_t)cdiv(a.nblk, CLS);
  const uint8_t* in = a.in;
  const uint64_t k0 = (uint64_t)t * CLS + (uint64_t)threadIdx.x * BPT;
  bool bad = false;
  // a thread's blocks share one state byte (BPT divides 8): one load
  static_assert(8 % BPT == 0, "a thread's state bits lie in one byte");
  const uint32_t sbyte = k0 < a.nblk ? (uint32_t)in[h.sec.state + (k0 >> 3)] : 0u;
  uint32_t ncb = 0, cnt = 0;
#pragma unroll
  for (int i = 0; i < BPT; ++i) {
    const uint64_t k = k0 + i;
    const bool nc = k < a.nblk && ((sbyte >> ((uint32_t)(k0 & 7) + i)) & 1u);
    ncb |= (nc ? 1u : 0u) << i;
    cnt += nc ? 1u : 0u;
  }
  // A tile whose preceding state bits are few (the first kDirectTiles
  // tiles: at most 32 KiB of them) counts its first rank directly, as the
  // population count of those bits (16-byte words from a 16-byte aligned
  // section, all loads issued at once), and publishes it as inclusive; later
  // tiles chain by look-back and stop at those words.
  const bool direct = MODE == kDirect || (MODE == kChained && t < kDirectTiles);
  uint32_t pop = 0;
  if (direct) {
    constexpr uint32_t W16 = kDirectTiles * (CLS / 8) / 16 / kWG;  // words per thread, at most
    const uint32_t n16 = t * (CLS / 8) / 16;
    // a buffer resource over exactly those bytes: words past it read zero, so
    // every lane issues the same loads (no branch but a wave-uniform one, no
    // waits between them)
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(in + h.sec.state), (short)0, (int)(n16 * 16u), 0x00020000);
    using v4u = unsigned int __attribute__((ext_vector_type(4)));
    v4u u[W16];
#pragma unroll
    for (uint32_t j = 0; j < W16; ++j) {
      u[j] = v4u{0, 0, 0, 0};
      if (j * kWG < n16) u[j] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)((threadIdx.x + j * kWG) * 16u), 0, 0);
    }
#pragma unroll
    for (uint32_t j = 0; j < W16; ++j) pop += __popc(u[j].x) + __popc(u[j].y) + __popc(u[j].z) + __popc(u[j].w);
  }
  const uint32_t v2[2] = {cnt, pop};
  uint32_t ex2[2], tot2[2];
  wg_excl_scan_multi<2>(v2, ex2, tot2, s_scan);
  const uint32_t rex = ex2[0], tnc = tot2[0];
  uint64_t R0 = tot2[1];
  if constexpr (!DIRECT) {
    gate_wait(b, a.status);
    if (direct) {
      if (threadIdx.x == 0) status_store(a.rank_st + t, kFlagIncl | (((uint64_t)tot2[1] + tnc) & kValueMask));
      if (threadIdx.x == 0) s_r0 = tot2[1];
    } else if (threadIdx.x < kWave) {
      if (threadIdx.x == 0) lookback_publish(a.rank_st, t, tnc);
      const uint64_t p = lookback_resolve_n(a.rank_st, t, tnc, a.status, kStatusDevice, ntiles);
      if (threadIdx.x == 0) s_r0 = p;
    }
    __syncthreads();
    R0 = s_r0;
  }
  // The K bytes and codes of the tile's ranks [R0, R0 + tnc) that the
  // stream holds, through buffer resources over just those bytes (32-bit
  // offsets from the tile's first rank; reads past them return zeros): every
  // load of the thread goes out before any of them is used.
  // Blocks whose codes a thread has in flight: all, or two of b = 1024 (64
  // registers a block). A load as each block is counted, in its branch, adds a
  // memory latency a block: 32768 float32 values of b = 256, 512 and 1024 took
  // 10.2, 15.1 and 25.2 us a call so, 8.2, 10.8 and 17.0 this way (with the count
  // in memory order, of it 0.7 us at b = 128: 7.7 and 7.0).
  constexpr int AHEAD = B < 1024 ? BPT : 2;
  const uint64_t have_nc = h.n_nc > R0 ? std::min<uint64_t>(h.n_nc - R0, (uint64_t)tnc) : 0;
  const __amdgpu_buffer_rsrc_t rk_ = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(in + h.sec.kbytes + R0), (short)0, (int)have_nc, 0x00020000);
  const __amdgpu_buffer_rsrc_t rc_ = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(in + h.sec.codes + R0 * (B / 4)), (short)0, (int)(have_nc * (B / 4)), 0x00020000);
  uint32_t mid = 0, midb[BPT] = {};
  // A wave of constant blocks has none to look at: their loads, though of
  // nothing, cost a constant field of 2^18 float32 values 11.6 us a call at
  // b = 1024 (9.7 without) and 9.2 at b = 512 (8.1).
  if (__ballot(ncb != 0) != 0) {
    uint32_t kbv[BPT];
    BlockCodes<B> cv[AHEAD];
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      // this block's rank from the tile's first: rex plus the thread's
      // non-constant blocks before it (constant blocks read far past the range)
      const uint32_t rl = rex + (uint32_t)__popc(ncb & ((1u << i) - 1u));
      const bool live = (ncb >> i) & 1u;
      kbv[i] = __builtin_amdgcn_raw_buffer_load_b8(rk_, live ? (int)rl : 0x40000000, 0, 0);
      if (i < AHEAD) load_codes<B>(rc_, live ? rl * (uint32_t)(B / 4) : 0x40000000u, cv[i]);
    }
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      const uint64_t k = k0 + i;
      midb[i] = mid;  // the thread's mid bytes before its block i
      if ((ncb >> i) & 1u) {
        const uint32_t rl = rex + (uint32_t)__popc(ncb & ((1u << i) - 1u));
        if ((uint64_t)rl < have_nc) {
          const uint32_t nk = (uint32_t)std::min<uint64_t>((uint64_t)B, a.n - k * B);
          mid += block_mid_bytes<T, B>(cv[i % AHEAD], kbv[i], nk, bad);
        } else {
          bad = true;
        }
      }
      if (i + AHEAD < BPT) {
        const uint32_t rl = rex + (uint32_t)__popc(ncb & ((1u << (i + AHEAD)) - 1u));
        load_codes<B>(rc_, (ncb >> (i + AHEAD)) & 1u ? rl * (uint32_t)(B / 4) : 0x40000000u, cv[i % AHEAD]);
      }
    }
  }
  uint32_t tmid;
  const uint32_t mex = wg_excl_sum<uint32_t>(mid, s_scan, tmid);
  if constexpr (!DIRECT) {
    if (threadIdx.x < kWave) {
      if (threadIdx.x == 0) lookback_publish(a.mid_st, t, tmid);
      const uint64_t p = lookback_resolve_n(a.mid_st, t, tmid, a.status, kStatusDevice, ntiles);
      if (threadIdx.x == 0) s_m0 = p;
    }
  }
  // mid bytes before every wave of a decode tile, within this tile
#pragma unroll
  for (int i = 0; i < BPT; ++i)
    if ((threadIdx.x * BPT + i) % D::WBLK == 0) s_wave[(threadIdx.x * BPT + i) / D::WBLK] = mex + midb[i];
  if (DIRECT) {
    if (threadIdx.x == 0) s_wave[CLS / D::WBLK] = tmid;
    if (t == ntiles - 1 && R0 + tnc != h.n_nc) bad = true;
    if (MODE == kOne && tmid != h.mid_total) bad = true;
    const uint64_t any = __ballot(bad);
    if (lane_id() == 0) s_scan[kWavesPerWG + threadIdx.x / kWave] = any != 0 ? 1u : 0u;  // past the sums' words
  }
  __syncthreads();
  if ((k0 % D::TBLK) == 0 && k0 < a.nblk && (MODE != kOne || k0 / D::TBLK == dt)) {
    const uint32_t w = threadIdx.x * BPT / D::WBLK;
    const uint32_t m = s_wave[w];
    const uint64_t m0 = DIRECT ? index_direct(m, s_wave[w + 4] - m) : s_m0 + m;
    index_store(MODE == kOne ? entry : a.index + 2 * (k0 / D::TBLK), m0, R0 + rex, s_wave[w + 1] - m, s_wave[w + 2] - m, s_wave[w + 3] - m);
  }
  if constexpr (DIRECT) {
    if (threadIdx.x == 0) {
      uint32_t any = 0;
#pragma unroll
      for (int i = 0; i < kWavesPerWG; ++i) any |= s_scan[kWavesPerWG + i];
      if constexpr (MODE == kDirect)
        direct_totals(a)[t] = tmid | (any ? kTotalBad : 0u);
      else if (dt == 0)
        *a.status = any ? kStatusCorrupt : 0u;
    }
  } else {
    if (t == ntiles - 1 && threadIdx.x == 0) {
      if (R0 + tnc != h.n_nc || s_m0 + tmid != h.mid_total) bad = true;
      // the end of the last decode tile
      index_store(a.index + 2 * cdiv(a.nblk, D::TBLK), h.mid_total, h.n_nc, 0, 0, 0);
    }
    if (__ballot(bad) != 0 && lane_id() == 0) atomicMax(a.status, kStatusCorrupt);
  }
  return true;
}

template <typename T, int B, int MODE>
__global__ __launch_bounds__(256) void k_dindex(DBatch b) {
  __shared__ uint32_t s_scan[2 * kWavesPerWG];
  __shared__ uint64_t s_r0, s_m0;
  __shared__ uint32_t s_wave[kClsBlocks / DecGeo<T, B>::WBLK + 1];
  __shared__ int s_flag;
  const uint64_t g = blockIdx.x;
  const FieldD f = field_at(b, dfield_of(b.field_idx[Traits<T>::BYTES / 8], g));
  dindex_tile<T, B, MODE>(b, f, (uint32_t)(g - f.base_idx), s_scan, &s_r0, &s_m0, s_wave, &s_flag);
}

// A batch of both element types runs each pass as one launch, the float32
// fields' workgroups first, where the two types' kernels need alike registers
// and LDS (below b = 1024): a launch for each type has its own start and its
// own nearly empty end. Fields of a median of 1 MiB, b = 128, in a launch a type,
// and so: 8 of them 23.6 -> 13.5 us a call (graph replays), 256 of them 165 ->
// 159; 32 of 256 KiB 24.2 -> 14.7, at b = 512 40.3 -> 22.9.
template <int B>
constexpr bool kOneLaunch = B < 1024;
// The decode pass only where few tiles are of the type that loses by it: the
// kernel of both types has the float32 kernel's registers, which cost the
// float64 tiles waves, but at b = 512 the float64 kernel's LDS, which costs the
// float32 tiles theirs. Fields of 1 MiB, a launch a type and one, us a call:
// b = 128, 96 MiB, nine tenths of it float64, 36.7 and 34.1; 176 MiB, three quarters
// (8448 tiles) 61.0 and 59.9, nine tenths (10048) 59.0 and 59.1; 192 MiB, nine tenths
// 62.0 and 63.3; 384 MiB, half (12288) 112.6 and 114.7; 512 MiB, nine tenths 129.7 and
// 140.5 (b = 32 134.3 and 144.9). b = 512, 160 MiB, four tenths (6144 float32 tiles) 75.1
// and 75.8, nine tenths 82.2 and 77.2; 192 MiB, a tenth 81.5 and 88.1, half (6144) 88.5
// and 88.5; 512 MiB, a tenth 172.4 and 196.2, nine tenths 234.4 and 234.7.
template <int B>
bool one_decode_launch(const DBatch& b) {
  return B < 512 ? b.tiles_dec[1] <= 8192 : b.tiles_dec[0] <= 6144;
}

template <int B, int MODE>
__global__ __launch_bounds__(256) void k_dindex_both(DBatch b) {
  constexpr int W4 = DecGeo<float, B>::WBLK, W8 = DecGeo<double, B>::WBLK;
  __shared__ uint32_t s_scan[2 * kWavesPerWG];
  __shared__ uint64_t s_r0, s_m0;
  __shared__ uint32_t s_wave[kClsBlocks / (W4 < W8 ? W4 : W8) + 1];
  __shared__ int s_flag;
  uint64_t g = blockIdx.x;
  if (g < b.tiles_idx[0]) {
    const FieldD f = field_at(b, dfield_of(b.field_idx[0], g));
    dindex_tile<float, B, MODE>(b, f, (uint32_t)(g - f.base_idx), s_scan, &s_r0, &s_m0, s_wave, &s_flag);
  } else {
    g -= b.tiles_idx[0];
    const FieldD f = field_at(b, dfield_of(b.field_idx[1], g));
    dindex_tile<double, B, MODE>(b, f, (uint32_t)(g - f.base_idx), s_scan, &s_r0, &s_m0, s_wave, &s_flag);
  }
}

// A direct index's totals of the first n <= kDirectTiles index tiles, four a
// lane; their sum (every lane the same), and whether one of the tiles found the
// stream corrupt.
static_assert(kDirectTiles == 4 * kWave, "four totals a lane");
struct Totals {
  uint32_t v[4];
};
__device__ __forceinline__ Totals totals_load(const uint32_t* totals, uint32_t n) {
  using v4u = unsigned int __attribute__((ext_vector_type(4)));
  const v4u u = __builtin_amdgcn_raw_buffer_load_b128(buffer_of(totals, (n + 3u) / 4u * 16u), lane_id() * 16, 0, 0);
  Totals t;
#pragma unroll
  for (uint32_t k = 0; k < 4; ++k) t.v[k] = (uint32_t)lane_id() * 4u + k < n ? u[k] : 0u;
  return t;
}
__device__ __forceinline__ uint32_t totals_sum(const Totals& t) {
  uint32_t sum = 0;
#pragma unroll
  for (uint32_t k = 0; k < 4; ++k) sum += t.v[k] & ~kTotalBad;
  return wave_total_u32(sum);
}
__device__ __forceinline__ bool totals_bad(const Totals& t) {
  return __ballot(((t.v[0] | t.v[1] | t.v[2] | t.v[3]) & kTotalBad) != 0) != 0;
}

// One decode tile, each wave its quarter by itself: no barrier, nothing shared.
//
// Bound: the stream's reads and the values' writes (100x500x500 float32 at REL
// 1e-3: 41 MB in and 100 MB out, 27 us at the copy rate of 5.2 TB/s; measured
// 24 us, part of the stream coming from the last-level cache; 31.5 us with four
// barriers a tile, byte masks a value and gaps in every store). 2^28 float64
// values at REL 1e-5: 443 us a call with the index pass (552), the copy rate as
// well.
// `entry`: the tile's entry of the index where the workgroup made it itself
// (kOne), else null.
template <typename T, int B, bool ONE>
__device__ __forceinline__ void decode_tile(const FieldD& a, uint32_t t, bool direct, uint8_t* s_stage,
                                            const uint64_t* entry) {
  using U = typename Traits<T>::U;
  using G = DecGeo<T, B>;
  constexpr int EPL = G::EPL, LPB = G::LPB, SUB = G::SUB, TBLK = G::TBLK;
  constexpr int BYTES = Traits<T>::BYTES;
  using v4u = unsigned int __attribute__((ext_vector_type(4)));

  // the index first: its loads go out beside the header's
  const uint32_t it = t / (uint32_t)(kClsBlocks / TBLK);  // the index tile
  Totals sums;
  uint64_t e0, e1, e2 = 0;
  if constexpr (ONE) {
    e0 = uniform(entry[0]);
    e1 = uniform(entry[1]);
  } else {
    sums = totals_load(direct_totals(a), direct ? it : 0u);
    const uint64_t* e = as_constant(a.index + 2 * (uint64_t)t);
    e0 = e[0];
    e1 = e[1];
    e2 = e[2];
  }
  const StreamInfo h = read_header<BYTES, B>(a);
  if (!h.ok) return;  // k_dindex reported it
  const uint8_t* in = a.in;
  const uint32_t wave = uniform(threadIdx.x / kWave);
  const uint32_t lane = (uint32_t)lane_id(), lig = lane % LPB;
  uint8_t* const stage = s_stage + wave * G::STAGE;
  bool bad = false;

  // the tile's first block, its block and value counts (wave-uniform); lanes
  // index from them with 32-bit offsets
  const uint64_t kb = (uint64_t)t * TBLK;
  const uint32_t nblk_t = (uint32_t)std::min<uint64_t>(a.nblk - kb, (uint64_t)TBLK);
  const uint32_t nval_t = (uint32_t)std::min<uint64_t>(a.n - kb * B, (uint64_t)TBLK * B);
  const bool tail = nval_t != (uint32_t)(TBLK * B);

  // State bits: of the lane's block in every row, and of the tile's blocks
  // before the wave (one block a lane where the tile has no more blocks than
  // a wave lanes, else words of 32). mu. All before anything waits.
  const __amdgpu_buffer_rsrc_t rst = buffer_of(in + h.sec.state + (kb >> 3), (nblk_t + 7) / 8);
  const __amdgpu_buffer_rsrc_t rmu =
      buffer_of(reinterpret_cast<const T*>(in + h.sec.mu) + kb, nblk_t * (uint32_t)sizeof(T));
  uint32_t ahead, sbyte[SUB];
  if constexpr (TBLK <= kWave) {
    ahead = (uint32_t)__builtin_amdgcn_raw_buffer_load_b8(rst, (int)(lane >> 3), 0, 0);
  } else {
    ahead = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(
        buffer_of(in + h.sec.state + (kb >> 3), (nblk_t + 31) / 32 * 4), (int)(lane * 4u), 0, 0);
#pragma unroll
    for (int s = 0; s < SUB; ++s)
      sbyte[s] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b8(
          rst, (int)((wave * G::WBLK + (uint32_t)(s * G::GPW) + lane / LPB) >> 3), 0, 0);
  }
  T mu[SUB];
#pragma unroll
  for (int s = 0; s < SUB; ++s)
    mu[s] = buffer_value<T>(rmu, (wave * G::WBLK + (uint32_t)(s * G::GPW) + lane / LPB) * (uint32_t)sizeof(T));

  // the wave's mid bytes: [m0, m1) of the mid section, from the tile's entry
  // of the index and the next one's
  const uint64_t r0_t = e1 & 0xFFFFFFFFull;
  uint64_t m0_t = e0 & kIndexMid, m1_t = e2 & kIndexMid;
  if (ONE || direct) {
    const uint32_t base = ONE ? 0u : totals_sum(sums);
    const uint32_t rel = (uint32_t)m0_t & 0xFFFFFFu;
    m1_t = (uint64_t)base + rel + ((uint32_t)(m0_t >> 24) & 0x1FFFFu);
    m0_t = (uint64_t)base + rel;
    // once a field: the index tiles' own findings, and the sum of all
    if (!ONE && kb + nblk_t == a.nblk) {
      const Totals all = totals_load(direct_totals(a), it + 1);
      if (totals_sum(all) != h.mid_total || totals_bad(all)) bad = true;
    }
  }
  const uint32_t w1 = (uint32_t)(e0 >> 48), w2 = (uint32_t)(e1 >> 32) & 0xFFFFu, w3 = (uint32_t)(e1 >> 48);
  const uint64_t m0 = m0_t + (wave == 0 ? 0u : wave == 1 ? w1 : wave == 2 ? w2 : w3);
  uint64_t m1 = wave == 3 ? m1_t : m0_t + (wave == 0 ? w1 : wave == 1 ? w2 : w3);
  if (m1 < m0 || m1 - m0 > (uint64_t)G::MOST || h.sec.mid + m1 > a.in_bytes) {
    bad = true;
    m1 = m0;
  }
  const uint32_t wbytes = (uint32_t)(m1 - m0);
  const uint64_t src = h.sec.mid + m0;
  const uint32_t st = (uint32_t)(src & 15u);
  // Staged with 16-byte loads, all of them before the stores to LDS (loads
  // return in order). The chunk that holds the stream's end goes byte by byte:
  // nothing is read past in_bytes.
  constexpr uint32_t NCH = ((15u + G::MOST + 15u) / 16u + kWave - 1u) / kWave;
  v4u u[NCH];
  {
    const uint8_t* base = in + (src - st);
    const uint32_t nchunk = wbytes ? (st + wbytes + 15u) / 16u : 0u;
    const uint64_t room = a.in_bytes - (src - st);
    const uint32_t nwhole = (uint32_t)std::min<uint64_t>(room / 16u, (uint64_t)nchunk);
    const __amdgpu_buffer_rsrc_t rs = buffer_of(base, nwhole * 16u);
#pragma unroll
    for (uint32_t j = 0; j < NCH; ++j) {
      if (j * kWave < nwhole)  // wave-uniform
        u[j] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)((lane + j * kWave) * 16u), 0, 0);
    }
    if (nwhole < nchunk && lane < (uint32_t)(room - nwhole * 16u)) stage[kStageHead + nwhole * 16u + lane] = base[nwhole * 16u + lane];
#pragma unroll
    for (uint32_t j = 0; j < NCH; ++j) {
      if (lane + j * kWave < nwhole) reinterpret_cast<v4u*>(stage + kStageHead)[lane + j * kWave] = u[j];
    }
  }

  wave_sync();

  // ranks of the wave's non-constant blocks, their K bytes and codes
  uint64_t tile_nc = 0;  // the tile's blocks, one bit each (TBLK <= 64)
  uint32_t wrank;        // rank of the wave's first block, within the tile
  if constexpr (TBLK <= kWave) {
    tile_nc = __ballot(lane < nblk_t && ((ahead >> (lane & 7u)) & 1u));
    wrank = (uint32_t)__popcll(tile_nc & ((1ull << (wave * G::WBLK)) - 1ull));
  } else {
    const int left = (int)(wave * G::WBLK) - (int)lane * 32;
    const uint32_t mask = left >= 32 ? ~0u : left <= 0 ? 0u : (1u << left) - 1u;
    wrank = wave_total_u32((uint32_t)__popc(ahead & mask));
  }
  // what the stream holds of the tile's ranks
  const uint32_t nnc_t = (uint32_t)std::min<uint64_t>(h.n_nc > r0_t ? h.n_nc - r0_t : 0, (uint64_t)TBLK);
  const __amdgpu_buffer_rsrc_t rk = buffer_of(in + h.sec.kbytes + r0_t, nnc_t);
  const __amdgpu_buffer_rsrc_t rc = buffer_of(in + h.sec.codes + r0_t * (B / 4), nnc_t * (uint32_t)(B / 4));
  bool nc[SUB];
  uint32_t kraw[SUB], craw[SUB];
#pragma unroll
  for (int s = 0; s < SUB; ++s) {
    const uint32_t lk = wave * G::WBLK + (uint32_t)(s * G::GPW) + lane / LPB;
    if constexpr (TBLK <= kWave)
      nc[s] = (tile_nc >> lk) & 1u;
    else
      nc[s] = lk < nblk_t && ((sbyte[s] >> (lk & 7u)) & 1u);
    const uint64_t firsts = __ballot(nc[s]) & first_lanes<LPB>();
    // the group's first lane does not count its own block; the others see it
    // counted
    const uint32_t rank = __builtin_amdgcn_mbcnt_hi(
        (uint32_t)(firsts >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)firsts, wrank - (lig != 0 ? 1u : 0u)));
    wrank += (uint32_t)__popcll(firsts);
    bad = bad || (nc[s] && rank >= nnc_t);
    kraw[s] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b8(rk, (int)(nc[s] ? rank : 0x40000000u), 0, 0);
    const uint32_t coff = nc[s] ? rank * (uint32_t)(B / 4) + lig * (EPL / 4) : 0x40000000u;
    if constexpr (EPL == 8)
      craw[s] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(rc, (int)coff, 0, 0);
    else
      craw[s] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(rc, (int)coff, 0, 0);
  }

  uint32_t done = kStageHead + st;  // stage offset of the row's first mid byte
#pragma unroll
  for (int s = 0; s < SUB; ++s) {
    const uint32_t lk = wave * G::WBLK + (uint32_t)(s * G::GPW) + lane / LPB;
    int cnt = EPL;
    if (tail) {
      const int rem = (int)nval_t - (int)(lk * B + lig * EPL);  // values from this lane's first one to the tile's end
      cnt = rem < 0 ? 0 : (rem > EPL ? EPL : rem);
    }
    T* const y = reinterpret_cast<T*>(a.out) + kb * B;  // of the tile
    const uint32_t i0 = (wave * G::WBLK + (uint32_t)(s * G::GPW)) * (uint32_t)B;  // the row's first value
    constexpr uint32_t CH = (uint32_t)(EPL * BYTES) / 16u;  // 16-byte chunks a lane
    // chunk d of the row, as far as the field goes; streamed past the caches
    // (the values are not read again here)
    auto put = [&](uint32_t d, const v4u& w) {
      const uint32_t first = i0 + d * (16u / BYTES);  // its first value
      if (!tail || first + 16u / BYTES <= nval_t) {
        __builtin_nontemporal_store(w, reinterpret_cast<v4u*>(y + first));
      } else {
        uint32_t* const yw = reinterpret_cast<uint32_t*>(y + first);
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j)
          if (first + j * 4u / BYTES < nval_t) yw[j] = w[j];
      }
    };
    // A float64 row of constant blocks has nothing to decode: 2^28 values, two
    // thirds of the blocks constant, 476 -> 418 us a call. (float32 rows, of
    // twice the blocks, rarely are: the branch cost them 2-5 %.)
    T v[EPL];
    if (sizeof(T) == 8 && __ballot(nc[s]) == 0) {
#pragma unroll
      for (int i = 0; i < EPL; ++i) v[i] = mu[s];
    } else {
      // kept bits K (0: constant, absent or unusable), stored bytes a value
      uint32_t K = kraw[s];
      const bool raw = K == kRawK;
      if (nc[s] && !raw && ((int)K < Traits<T>::KMIN || (int)K > Traits<T>::W)) {
        bad = true;
        K = 0;
      }
      if (raw) K = 0;
      const uint32_t nb = (K + 7u) >> 3;
      const uint32_t sh = 8u * nb - K;
      uint32_t c;  // the lane's codes, first value in the top bits
      if constexpr (EPL == 8)
        c = ((craw[s] & 0xFFu) << 8) | (craw[s] >> 8);
      else
        c = __builtin_bswap32(craw[s]);
      // Codes of values past the end are cleared; a code above nb marks the
      // stream bad and its lane is then read as if all codes were 0, which
      // keeps every offset within the stage.
      if (tail) c = valid_codes<EPL>(c, cnt);
      c = K ? c : 0u;
      uint32_t per = nb;  // stored bytes of a value whose code is 0
      bool some_raw = false;
      if (__ballot(nc[s] && nb < 3u) != 0) {  // few kept bytes, or raw
        const uint32_t hi = c & 0xAAAAAAAAu, lo = c & 0x55555555u;
        const bool over = K && ((nb == 1u && hi != 0) || (nb == 2u && (lo & (hi >> 1)) != 0));
        bad = bad || over;
        c = over ? 0u : c;
        per = raw ? (uint32_t)BYTES : nb;
        some_raw = __ballot(raw) != 0;
        // A row of raw blocks alone is its stored bytes, realigned. (Lane by lane, as
        // below, their runs of 64 or 128 bytes all start in the same four or two LDS
        // banks. 160 MB of raw blocks, us a call with the general reads of raw lanes
        // there too, without, and this way: float32, b = 128, 178, 92 and 80; float64
        // 171, 79 and 72, b = 1024 329, 147 and 94. Smaller blocks do without: there the
        // path's code costs coded rows 1 %, the 100x500x500 float32 field at REL 1e-3
        // 32.2 us for 31.8.)
        if (B >= 512 && __builtin_expect(some_raw, 0) && __ballot(raw || cnt == 0) == ~0ull) {
          const uint32_t at = uniform(done);
          const uint4* const q = reinterpret_cast<const uint4*>(stage + (at & ~15u));
#pragma unroll 1
          for (uint32_t k = 0; k < CH; ++k) {
            const uint32_t d = k * kWave + lane;
            const uint4 u = realign16(q[d], q[d + 1], (at >> 2) & 3u, at & 3u);
            put(d, v4u{u.x, u.y, u.z, u.w});
          }
          done += (tail ? std::min<uint32_t>(nval_t > i0 ? nval_t - i0 : 0u, (uint32_t)G::ROW) : (uint32_t)G::ROW) *
                  (uint32_t)BYTES;
          continue;
        }
      }
      // stored bytes of the lane, and its first one's place in the stage
      const uint32_t lb = (uint32_t)__umul24(per, (uint32_t)cnt) -
                          ((uint32_t)__popc(c) + (uint32_t)__popc(c & 0xAAAAAAAAu));
      const uint32_t inc = wave_incl_sum_u32(lb);
      uint32_t o = done + inc - lb;
      done += (uint32_t)__builtin_amdgcn_readlane((int)inc, 63);

      // Values. Reads of the stage go unguarded: a lane starts at most at the end
      // of the wave's stored bytes and advances at most a word per value, which
      // the stage's size allows for. Values past the end of a short block read
      // whatever lies there and are not stored; being last in their lane and
      // block, they only reach other such values. (Lanes of constant blocks run
      // along with nb = 0, and so do those of raw blocks, all at one address.)
      const uint32_t nbh = nb < 4u ? nb : 4u;
      const bool longer = sizeof(T) == 8 && __ballot(nb > 4u) != 0;  // some value stores bytes of its low word
      uint32_t got[EPL], gotl[sizeof(T) == 8 ? EPL : 1], own[EPL];
      uint32_t run = 0;
      const uint32_t o0 = o;
      o = raw ? kStageHead : o;
#pragma unroll
      for (int i = 0; i < EPL; ++i) {
        // o: where the value's word would start if its leading bytes were stored
        // too, so that its stored bytes lie in place; shared bytes come from the
        // word before, whatever follows the stored ones is cleared by `keep`
        const uint32_t ci = (c >> (2 * (EPL - 1 - i))) & 3u;
        o = i == 0 ? o - ci : __builtin_amdgcn_sad_u8(nb, ci, o);  // o + nb - ci
        got[i] = __builtin_bswap32(stage_get(stage, o));
        if constexpr (sizeof(T) == 8) {
          if (longer) gotl[i] = stage_get(stage, o + 4u);
        }
        own[i] = __builtin_amdgcn_alignbyte(~0u, 0u, ci);  // the top ci bytes: the shared ones
        run = (run & own[i]) | (got[i] & ~own[i]);
      }
      // Leading bytes from the lanes before this one in the block: the lanes'
      // (smallest code, top three bytes) pairs scanned under lead_compose.
      // Bytes below the kept ones never reach a kept byte (a code keeps at most
      // the top min(3, nb) bytes of a live value).
      uint32_t carry = 0;
      if constexpr (LPB > 1) {
        uint32_t pk = (run & 0xFFFFFF00u) | min_code<EPL>(c);
        uint32_t o2 = lane_up<LPB, 1>(pk);
        pk = lig >= 1 ? lead_compose(o2, pk) : pk;
        if constexpr (LPB > 2) {
          o2 = lane_up<LPB, 2>(pk);
          pk = lig >= 2 ? lead_compose(o2, pk) : pk;
        }
        if constexpr (LPB > 4) {
          o2 = lane_up<LPB, 4>(pk);
          pk = lig >= 4 ? lead_compose(o2, pk) : pk;
        }
        if constexpr (LPB > 8) {
          o2 = lane_up<LPB, 8>(pk);
          pk = lig >= 8 ? lead_compose(o2, pk) : pk;
        }
        if constexpr (LPB > 16) {
          o2 = __shfl_up(pk, 16, LPB);
          pk = lig >= 16 ? lead_compose(o2, pk) : pk;
        }
        if constexpr (LPB > 32) {
          o2 = __shfl_up(pk, 32, LPB);
          pk = lig >= 32 ? lead_compose(o2, pk) : pk;
        }
        carry = lane_up<LPB, 1>(pk) & 0xFFFFFF00u;
        carry = lig == 0 ? 0u : carry;
      }
      // x' = mu + (q' << s), the words once more with the carried bytes in front
      run = carry;
      if constexpr (sizeof(T) == 4) {
        const uint32_t keep = top_bytes_mask<uint32_t>((int)nbh) << sh;
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
          run = (run & own[i]) | (got[i] & ~own[i]);
          v[i] = mu[s] + from_bits<T>((run << sh) & keep);
        }
      } else if (!longer) {
        const uint32_t keep = top_bytes_mask<uint32_t>((int)nbh) << sh;
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
          run = (run & own[i]) | (got[i] & ~own[i]);
          v[i] = mu[s] + from_bits<T>((U)((run << sh) & keep) << (sizeof(U) * 8 - 32));
        }
      } else {
        const U keep = (U)(top_bytes_mask<U>((int)nb) << sh);
#pragma unroll
        for (int i = 0; i < EPL; ++i) {
          run = (run & own[i]) | (got[i] & ~own[i]);
          const U q = ((U)run << (sizeof(U) * 8 - 32)) | (U)__builtin_bswap32(gotl[i]);
          v[i] = mu[s] + from_bits<T>((U)(q << sh) & keep);
        }
      }
      if (__ballot(K == 0) != 0) {
        if (K == 0) {  // constant: mu itself (mu + 0 would lose a zero's sign)
#pragma unroll
          for (int i = 0; i < EPL; ++i) v[i] = mu[s];
        }
        if (__builtin_expect(some_raw, 0) && raw) {  // the stored words
          const uint32_t* p = reinterpret_cast<const uint32_t*>(stage + (o0 & ~3u));
          uint32_t at = *p;
          auto word = [&]() {
            const uint32_t next = *++p, w = __builtin_amdgcn_alignbyte(next, at, o0);
            at = next;
            return w;
          };
#pragma unroll
          for (int i = 0; i < EPL; ++i) {
            const uint32_t lo = word();
            if constexpr (sizeof(T) == 4)
              v[i] = from_bits<T>(lo);
            else
              v[i] = from_bits<T>((U)lo | ((U)word() << (sizeof(U) * 8 - 32)));
          }
        }
      }
    }

    if constexpr (SUB == 1) {
      // The row passes through the stage (its mid bytes are used up), so that
      // every store of the wave covers 1 KiB without gaps. Chunk c of lane L
      // sits at slot L CH + (c ^ (L / (16 / CH)) mod CH): 16 lanes writing one
      // chunk each, or reading 16 consecutive ones, touch all 64 banks.
      v4u* const slots = reinterpret_cast<v4u*>(stage);
      constexpr uint32_t PER = 16u / CH;
      wave_sync();
#pragma unroll
      for (uint32_t k = 0; k < CH; ++k) {
        v4u w;
        if constexpr (sizeof(T) == 4) {
          w = v4u{(uint32_t)bits_of(v[4 * k]), (uint32_t)bits_of(v[4 * k + 1]), (uint32_t)bits_of(v[4 * k + 2]),
                  (uint32_t)bits_of(v[4 * k + 3])};
        } else {
          const U p = bits_of(v[2 * k]), q = bits_of(v[2 * k + 1]);
          w = v4u{(uint32_t)p, (uint32_t)(p >> (sizeof(U) * 8 - 32)), (uint32_t)q, (uint32_t)(q >> (sizeof(U) * 8 - 32))};
        }
        slots[lane * CH + (k ^ ((lane / PER) % CH))] = w;
      }
      wave_sync();
#pragma unroll
      for (uint32_t k = 0; k < CH; ++k) {
        const uint32_t d = k * kWave + lane;  // chunk of the row
        const uint32_t L = d / CH;
        put(d, slots[L * CH + ((d % CH) ^ ((L / PER) % CH))]);
      }
    } else {
      T* const yl = y + (i0 + lane * EPL);
      if (cnt == EPL) {
#pragma unroll
        for (uint32_t k = 0; k < CH; ++k) {
          v4u w;
          if constexpr (sizeof(T) == 4) {
            w = v4u{(uint32_t)bits_of(v[4 * k]), (uint32_t)bits_of(v[4 * k + 1]), (uint32_t)bits_of(v[4 * k + 2]),
                    (uint32_t)bits_of(v[4 * k + 3])};
          } else {
            const U p = bits_of(v[2 * k]), q = bits_of(v[2 * k + 1]);
            w = v4u{(uint32_t)p, (uint32_t)(p >> (sizeof(U) * 8 - 32)), (uint32_t)q,
                    (uint32_t)(q >> (sizeof(U) * 8 - 32))};
          }
          reinterpret_cast<v4u*>(yl)[k] = w;
        }
      } else {
#pragma unroll
        for (int i = 0; i < EPL; ++i)
          if (i < cnt) yl[i] = v[i];
      }
    }
  }
  if (done - kStageHead - st != wbytes) bad = true;
  // (kOne: the index has looked at every K byte, code and sum of the field,
  // and decode tile 0 has stored what it found)
  if (!ONE && __ballot(bad) != 0 && lane == 0) atomicMax(a.status, kStatusCorrupt);
}

template <typename T, int B>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(DecGeo<T, B>::WAVES))) void k_decode(DBatch b) {
  using G = DecGeo<T, B>;
  __shared__ __align__(16) uint8_t s_stage[kWavesPerWG * G::STAGE];
  const uint64_t g = blockIdx.x;
  const FieldD f = field_at(b, dfield_of(b.field_dec[Traits<T>::BYTES / 8], g));
  decode_tile<T, B, false>(f, (uint32_t)(g - f.base_dec), b.direct != 0, s_stage, nullptr);
  // the call's last decode launch advances the gate's epoch (no index tile
  // reads it any more); at the end, so that no load comes after the atomic
  if (g == 0 && threadIdx.x == 0 && !b.direct && (sizeof(T) == 8 || b.tiles_dec[1] == 0)) gate_advance(b);
}

template <int B>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(
    DecGeo<float, B>::WAVES < DecGeo<double, B>::WAVES ? DecGeo<float, B>::WAVES : DecGeo<double, B>::WAVES))) void
k_decode_both(DBatch b) {
  __shared__ __align__(16) uint8_t s_stage[kWavesPerWG * std::max(DecGeo<float, B>::STAGE, DecGeo<double, B>::STAGE)];
  uint64_t g = blockIdx.x;
  if (g < b.tiles_dec[0]) {
    const FieldD f = field_at(b, dfield_of(b.field_dec[0], g));
    decode_tile<float, B, false>(f, (uint32_t)(g - f.base_dec), b.direct != 0, s_stage, nullptr);
  } else {
    g -= b.tiles_dec[0];
    const FieldD f = field_at(b, dfield_of(b.field_dec[1], g));
    decode_tile<double, B, false>(f, (uint32_t)(g - f.base_dec), b.direct != 0, s_stage, nullptr);
  }
  if (blockIdx.x == 0 && threadIdx.x == 0 && !b.direct) gate_advance(b);
}

// A small field's decompression in one launch: every workgroup indexes the whole
// field (one index tile, kept in LDS) and decodes its own tile. Two launches
// spend most of a small call in their latencies: 4099 float32 values take 10.3
// us a call in two, 8.0 in one (7.3 with the shorter count).
template <typename T, int B>
__global__ __launch_bounds__(256) void k_dsmall(DBatch b) {
  using G = DecGeo<T, B>;
  __shared__ uint32_t s_scan[2 * kWavesPerWG];
  __shared__ uint32_t s_wave[kClsBlocks / G::WBLK + 1];
  __shared__ __align__(16) uint64_t s_entry[2];
  __shared__ __align__(16) uint8_t s_stage[kWavesPerWG * G::STAGE];
  FieldD f = b.one;
  f.in = as_global(f.in);
  f.out = as_global(f.out);
  f.status = as_global(f.status);
  if (!dindex_tile<T, B, kOne>(b, f, 0, s_scan, s_entry, s_entry, s_wave, nullptr, blockIdx.x, s_entry)) return;
  __syncthreads();
  decode_tile<T, B, true>(f, blockIdx.x, true, s_stage, s_entry);
}

// ---------------------------------------------------------------- launch ---

template <int B>
hipError_t launch_decompress_b(const DBatch& b, hipStream_t stream, TimerHook hook) {
  auto run = [&](const char* name, auto&& fn) {
    if (hook) hook(name, stream, 1);
    fn();
    if (hook) hook(name, stream, 0);
  };
  // the index pass clears what it needs itself (its gate); a call without
  // index tiles only has status words to set
  if (b.tiles_idx[0] + b.tiles_idx[1] == 0) {
    const uint64_t nf = b.fields ? b.nfields : 1;
    const uint32_t gi = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(cdiv(nf, 256), 1024));
    run("k_dinit", [&] { k_dinit<<<gi, 256, 0, stream>>>(b); });
  }
  // The line: one index tile, and codes that every workgroup can look through
  // (131072 values: 32 KiB of them). At 131072 float32 values, b = 128, 32
  // workgroups: one launch 8.3 us, two 10.3 (7.5 in one with the shorter count); at b = 512
  // 11.0 and 13.2, at b = 1024 18.0 and 19.6; float64 12.4 and 14.6, 20.0 and 21.4.
  if (!b.fields && b.tiles_idx[0] + b.tiles_idx[1] == 1 && b.one.n <= 131072) {
    if (b.tiles_idx[0])
      run("k_dsmall", [&] { k_dsmall<float, B><<<(uint32_t)b.tiles_dec[0], 256, 0, stream>>>(b); });
    else
      run("k_dsmall", [&] { k_dsmall<double, B><<<(uint32_t)b.tiles_dec[1], 256, 0, stream>>>(b); });
    return hipGetLastError();
  }
  bool indexed = false;
  if constexpr (kOneLaunch<B>) {
    if (b.fields && b.tiles_idx[0] && b.tiles_idx[1]) {
      const uint32_t gi = (uint32_t)(b.tiles_idx[0] + b.tiles_idx[1]);
      if (b.direct)
        run("k_dindex", [&] { k_dindex_both<B, kDirect><<<gi, 256, 0, stream>>>(b); });
      else
        run("k_dindex", [&] { k_dindex_both<B, kChained><<<gi, 256, 0, stream>>>(b); });
      indexed = true;
      if (one_decode_launch<B>(b)) {
        run("k_decode", [&] { k_decode_both<B><<<(uint32_t)(b.tiles_dec[0] + b.tiles_dec[1]), 256, 0, stream>>>(b); });
        return hipGetLastError();
      }
    }
  }
  for (int dt = 0; dt < 2 && !indexed; ++dt) {
    const uint32_t n = (uint32_t)b.tiles_idx[dt];
    if (!n) continue;
    if (dt == 0 && b.direct)
      run("k_dindex", [&] { k_dindex<float, B, kDirect><<<n, 256, 0, stream>>>(b); });
    else if (dt == 0)
      run("k_dindex", [&] { k_dindex<float, B, kChained><<<n, 256, 0, stream>>>(b); });
    else if (b.direct)
      run("k_dindex", [&] { k_dindex<double, B, kDirect><<<n, 256, 0, stream>>>(b); });
    else
      run("k_dindex", [&] { k_dindex<double, B, kChained><<<n, 256, 0, stream>>>(b); });
  }
  if (b.tiles_dec[0]) run("k_decode", [&] { k_decode<float, B><<<(uint32_t)b.tiles_dec[0], 256, 0, stream>>>(b); });
  if (b.tiles_dec[1]) run("k_decode", [&] { k_decode<double, B><<<(uint32_t)b.tiles_dec[1], 256, 0, stream>>>(b); });
  return hipGetLastError();
}

hipError_t launch_decompress(const DBatch& b, uint32_t block, hipStream_t stream, TimerHook hook) {
  switch (block) {
    case 8: return launch_decompress_b<8>(b, stream, hook);
    case 16: return launch_decompress_b<16>(b, stream, hook);
    case 32: return launch_decompress_b<32>(b, stream, hook);
    case 64: return launch_decompress_b<64>(b, stream, hook);
    case 128: return launch_decompress_b<128>(b, stream, hook);
    case 256: return launch_decompress_b<256>(b, stream, hook);
    case 512: return launch_decompress_b<512>(b, stream, hook);
    case 1024: return launch_decompress_b<1024>(b, stream, hook);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace szx
