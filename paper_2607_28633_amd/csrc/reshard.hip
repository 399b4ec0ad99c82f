// reshard.hip - one layer moved between cache layouts on gfx950: head-sliced
// pack and unpack (a tensor-parallel shard's heads), pool-to-pool
// re-blocking between page sizes without a staging buffer, and pools whose
// pages are head-major.  The layouts and the entry points are specified in
// include/topkv.h (per-layer unit: Section 5.2; K-then-V token-major wire
// order: Section 3.5; paged pools: Section 6; KV heads per layer: Sections
// 2.2 and 5.3).
//
// Design.  Every move copies, per request, kept token and plane, the moved
// heads' values.  The unit of contiguity is a granule: one head's head_dim
// values, or all moved heads at once when both sides keep heads adjacent (a
// packed buffer and a slot-major pool do, a head-major pool does not).  The
// work is flattened in the packed order (request, plane, token, granule,
// 16-byte piece), so
//   * a packed side's address is simply piece index * piece bytes, and both
//     sides walk consecutive bytes across consecutive lanes wherever their
//     layout allows (a head-major side still gets whole granules);
//   * the request comes from a binary search over per-request prefix sums
//     held in LDS (built with a wave64 shuffle scan from the device lengths),
//     every other index from multiply-high divisions by launch constants;
//   * when a token's pieces fill whole wave spans (every 70B-class shape),
//     request, plane, token and page are wave-uniform: they are computed once
//     per wave in scalar registers and the block-table entries come through
//     scalar loads, the last one reused while the page does not change.
// Granules are at least one head's values (256 bytes for head_dim 128 in
// bf16), so both sides touch whole cache lines: no LDS staging of the data is
// needed even where the layout transposes (slot-major <-> head-major).
// Each lane issues all of its loads before its stores.  Moves of up to 1024
// requests run a direct grid (kv_reshard_direct_kernel: one workgroup per
// tile, no prefix scan, any row size) while that is short, and past that the
// same tiles in a grid that follows the lengths (kv_reshard_live_kernel);
// larger batches, and runs of fewer than 16 bytes, the general persistent one
// (kv_reshard_kernel).  Table entries and lengths are bounds-checked on the
// device before any access.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <atomic>
#include <cstdint>

#include "internal.h"
#include "topkv.h"

namespace topkv_reshard {

#ifndef TOPKV_RS_VPT
#define TOPKV_RS_VPT 8            // pieces per lane per tile
#endif
#ifndef TOPKV_RS_FILL
#define TOPKV_RS_FILL 512         // direct grids: smaller tiles until there are this many workgroups
#endif
#ifndef TOPKV_RS_SLOTS
#define TOPKV_RS_SLOTS 8192       // direct grids of device lengths: most workgroups; more run the live grid
#endif
#ifndef TOPKV_RS_WG_PER_CU
#define TOPKV_RS_WG_PER_CU 16     // grid cap = CUs * this
#endif

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kVpt = TOPKV_RS_VPT;
constexpr int kWgPerCu = TOPKV_RS_WG_PER_CU;
constexpr int kLiveVpt = 4;       // live grid: chunks per lane (large moves between pools: twice that)

template <int B> struct Vec;
template <> struct Vec<16> { typedef unsigned int type __attribute__((ext_vector_type(4))); };
template <> struct Vec<8> { typedef unsigned int type __attribute__((ext_vector_type(2))); };
template <> struct Vec<4> { typedef unsigned int type; };
template <> struct Vec<2> { typedef unsigned short type; };
template <> struct Vec<1> { typedef unsigned char type; };

// n / d for 0 <= n < 2^31 by a multiply-high (Granlund and Montgomery, 1994):
// with s = ceil(log2 d) and m = floor(2^32 (2^s - d) / d) + 1, the quotient is
// (mulhi(n, m) + n) >> s; the sum cannot overflow because mulhi(n, m) <= n.
struct FastDiv {
  uint32_t d, m, s;
};

FastDiv make_div(uint32_t d) {
  uint32_t s = 0;
  while ((1ull << s) < d) ++s;
  const uint64_t m = (((1ull << 32) * ((1ull << s) - d)) / d) + 1;
  return FastDiv{d, (uint32_t)m, s};
}

__device__ __forceinline__ uint32_t quot(uint32_t n, uint32_t m, uint32_t s) { return (__umulhi(n, m) + n) >> s; }

__device__ __forceinline__ uint32_t fdiv(uint32_t n, const FastDiv& f) { return quot(n, f.m, f.s); }

// One side of a move (kernel argument, by value).
struct Side {
  char* base;               // pool: the layer slab; packed: the buffer
  int64_t layer_stride;     // several layers on grid z: bytes from one layer's base to the next
  const int32_t* tables;    // pool: [num_reqs][bt_stride]
  int64_t page_bytes;
  int64_t plane_bytes;
  int64_t head0_bytes;      // offset of the first moved head within a slot
  int64_t num_pages;        // valid page indices are [0, num_pages)
  int32_t slot_bytes;       // stride between slots of a page plane
  int32_t gran_stride;      // stride between consecutive granules of a slot
  int32_t bt_stride;
  int32_t packed;           // 1: packed buffer (shard regions of Params::packed_cap bytes)
  FastDiv page;             // tokens per page
  FastDiv upp;              // direct grids: units per page
};

struct Params {
  Side src, dst;
  int64_t packed_cap;       // bytes of each shard region of the packed side (one region unsharded)
  FastDiv vpg;              // pieces per granule
  FastDiv gpt;              // granules per (token, plane)
  FastDiv ktp;              // pieces per (token, plane) = gpt * vpg
  FastDiv gps;              // granules per shard (= gpt when unsharded)
  int32_t num_reqs;
  int32_t planes;
  int32_t window;
  int32_t max_tok;          // lengths are clamped to [0, max_tok]
  int32_t n_host;           // one request with a host-side length: its tokens (else unused)
  // direct and live grids:
  FastDiv unit;             // tokens per unit
  FastDiv cpu;              // 16-byte chunks per unit of one plane
  FastDiv cpg;              // 16-byte chunks per granule (kHeads)
  FastDiv reqs;             // requests (grid z is layer * requests + request)
  int64_t total_cap;        // packed bytes from the first layer's region to the end of the last one's
  int32_t gran;             // bytes of one granule of one token
  int32_t region_gran;      // bytes of one token in a packed region (all its granules)
  int32_t grain;            // a run cut short by the packed capacity is a multiple of this (a power of two)
  int32_t strict;           // 1: a request whose packed block would end past the capacity is not moved at all
};

// Per-request kept-token counts and first kept tokens, and the exclusive
// prefix of planes * count (token-planes before request r), into LDS.
__device__ void request_prefix(const Params& p, const int32_t* __restrict__ seq_lens, int32_t* tp,
                               int32_t* st, int32_t* cnt, int32_t* wsum) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  int32_t carry = 0;
  for (int base = 0; base < p.num_reqs; base += kThreads) {
    const int r = base + threadIdx.x;
    int32_t v = 0;
    if (r < p.num_reqs) {
      int32_t n = seq_lens[r];
      n = n < 0 ? 0 : (n > p.max_tok ? p.max_tok : n);
      const int32_t start = (p.window > 0 && n > p.window) ? n - p.window : 0;
      st[r] = start;
      cnt[r] = n - start;
      v = (n - start) * p.planes;
    }
    int32_t x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int32_t y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    int32_t before = carry, chunk = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      if (w < wave) before += wsum[w];
      chunk += wsum[w];
    }
    if (r < p.num_reqs) tp[r] = before + x - v;
    carry += chunk;
    __syncthreads();
  }
  if (threadIdx.x == 0) tp[p.num_reqs] = carry;
  __syncthreads();
}

// Byte offset of piece (r, c, t, k, e) on a pool side; false if the table
// entry is out of range.
__device__ __forceinline__ bool pool_offset(const Side& s, int32_t r, uint32_t c, uint32_t t, uint32_t k,
                                            uint32_t e_bytes, int64_t* off) {
  const uint32_t i = fdiv(t, s.page);
  const uint32_t slot = t - i * s.page.d;
  const int32_t page = s.tables[(int64_t)r * s.bt_stride + i];
  if (page < 0 || (int64_t)page >= s.num_pages) return false;
  *off = (int64_t)page * s.page_bytes + (int64_t)c * s.plane_bytes + (int64_t)slot * s.slot_bytes +
         s.head0_bytes + (int64_t)k * s.gran_stride + e_bytes;
  return true;
}

// Byte offset of piece (q2, k, e) on the packed side: granule k belongs to
// shard k / gps, which holds its own (request, plane, token)-ordered granules
// at shard * packed_cap.  Unsharded (gps = gpt) this is the piece index * VB.
// False past the shard's capacity.
template <int VB>
__device__ __forceinline__ bool packed_offset(const Params& p, uint32_t q2, uint32_t k, uint32_t e,
                                              int64_t* off) {
  const uint32_t sh = fdiv(k, p.gps);
  const uint32_t pos = k - sh * p.gps.d;
  const int64_t in_shard = ((int64_t)q2 * p.gps.d + pos) * ((int64_t)p.vpg.d * VB) + (int64_t)e * VB;
  *off = (int64_t)sh * p.packed_cap + in_shard;
  return in_shard + VB <= p.packed_cap;
}

struct Loc {
  int32_t r;                // request
  uint32_t c, t;            // plane, token
};

// Request, plane and token of global (request, plane, token) index q2: the
// largest r with tp[r] <= q2 owns it (its count is then > 0), and the plane
// is the number of whole token runs below q2 within the request.
__device__ __forceinline__ Loc locate(uint32_t q2, const int32_t* tp, const int32_t* st, const int32_t* cnt,
                                      int32_t num_reqs) {
  int lo = 0, hi = num_reqs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if ((uint32_t)tp[mid] <= q2) lo = mid; else hi = mid - 1;
  }
  uint32_t local = q2 - (uint32_t)tp[lo];
  const uint32_t n_r = (uint32_t)cnt[lo];
  uint32_t c = 0;
  while (local >= n_r) { local -= n_r; ++c; }
  return Loc{lo, c, (uint32_t)st[lo] + local};
}

// Page lookups of one side for wave-uniform tokens.  Block tables are never
// written while a move runs, so they are read through the constant address
// space (scalar loads and the scalar cache); consecutive wave spans of a tile
// usually sit on the same page, so the last entry is kept.
struct PageCache {
  int32_t r = -1;
  uint32_t i = ~0u;
  int32_t page = -1;
};

typedef __attribute__((address_space(4))) const int32_t ConstInt;

// pool_offset for a wave-uniform (request, plane, token): the page lookup and
// everything but the piece's place inside the token's granules are uniform.
__device__ __forceinline__ bool pool_offset_wave(const Side& s, const Loc& at, uint32_t k, uint32_t e_bytes,
                                                 PageCache& pc, int64_t* off) {
  const uint32_t i = fdiv(at.t, s.page);
  const uint32_t slot = at.t - i * s.page.d;
  if (at.r != pc.r || i != pc.i) {
    const ConstInt* tab = (const ConstInt*)s.tables;
    pc.page = __builtin_amdgcn_readfirstlane(tab[(int64_t)at.r * s.bt_stride + i]);
    pc.r = at.r;
    pc.i = i;
  }
  const int32_t page = pc.page;
  if (page < 0 || (int64_t)page >= s.num_pages) return false;
  const int64_t base = (int64_t)page * s.page_bytes + (int64_t)at.c * s.plane_bytes +
                       (int64_t)slot * s.slot_bytes + s.head0_bytes;
  *off = base + (int64_t)k * s.gran_stride + e_bytes;
  return true;
}

// kWave: the pieces of one (request, plane, token) fill whole 64-piece wave
// spans (pieces per token-plane divisible by 64), so every wave instruction
// has one request, plane, token and page per side: those are found once per
// wave, with uniform (scalar) arithmetic and loads, and only the piece's
// place inside the token's granules varies across lanes.  Otherwise every
// lane locates its own piece.
template <int VB, bool kWave>
__global__ __launch_bounds__(kThreads) void kv_reshard_kernel(Params p, const int32_t* __restrict__ seq_lens) {
  typedef typename Vec<VB>::type V;
  extern __shared__ int32_t lds_i32[];
  int32_t* wsum = lds_i32;                     // [kWaves]
  int32_t* tp = wsum + kWaves;                 // [num_reqs + 1]
  int32_t* st = tp + (p.num_reqs + 1);         // [num_reqs]
  int32_t* cnt = st + p.num_reqs;              // [num_reqs]
  request_prefix(p, seq_lens, tp, st, cnt, wsum);

  const uint32_t per_tp = p.ktp.d;                            // pieces per (token, plane)
  const uint32_t total = (uint32_t)tp[p.num_reqs] * per_tp;   // the host keeps this below 2^31
  constexpr uint32_t kTile = (uint32_t)kThreads * kVpt;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave_first = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);

  PageCache src_pc, dst_pc;
  for (uint32_t base = blockIdx.x * kTile; base < total; base += gridDim.x * kTile) {
    // Three phases: every piece's addresses (searches, divisions, table
    // lookups), then every load, then every store.  No loop or branch sits
    // between the loads, so all kVpt of them are in flight at once; a skipped
    // piece loads from the source base (always valid) and is not stored.
    int64_t soff[kVpt], doff[kVpt];
    bool ok[kVpt];
#pragma unroll
    for (int j = 0; j < kVpt; ++j) {
      soff[j] = doff[j] = 0;
      ok[j] = false;
      if (kWave) {
        const uint32_t wbase = base + j * kThreads + wave_first;   // uniform
        if (wbase < total) {
          const uint32_t q2 = fdiv(wbase, p.ktp);
          const uint32_t m = wbase - q2 * per_tp + lane;            // < per_tp
          const uint32_t k = fdiv(m, p.vpg);
          const uint32_t e = m - k * p.vpg.d;
          Loc at = locate(q2, tp, st, cnt, p.num_reqs);
          at.r = __builtin_amdgcn_readfirstlane(at.r);
          at.c = __builtin_amdgcn_readfirstlane(at.c);
          at.t = __builtin_amdgcn_readfirstlane(at.t);
          int64_t so = 0, o = 0;
          // both sides' table entries are in-bounds reads whatever the other
          // side holds, so both lookups issue before either is tested
          const bool s_ok = p.src.packed ? packed_offset<VB>(p, q2, k, e, &so)
                                         : pool_offset_wave(p.src, at, k, e * VB, src_pc, &so);
          const bool d_ok = p.dst.packed ? packed_offset<VB>(p, q2, k, e, &o)
                                         : pool_offset_wave(p.dst, at, k, e * VB, dst_pc, &o);
          ok[j] = s_ok & d_ok;
          soff[j] = ok[j] ? so : 0;
          doff[j] = o;
        }
      } else {
        const uint32_t idx = base + j * kThreads + threadIdx.x;
        if (idx < total) {
          const uint32_t q = fdiv(idx, p.vpg);
          const uint32_t e = idx - q * p.vpg.d;
          const uint32_t q2 = fdiv(q, p.gpt);
          const uint32_t k = q - q2 * p.gpt.d;
          const Loc at = locate(q2, tp, st, cnt, p.num_reqs);
          int64_t so = 0, o = 0;
          const bool s_ok = p.src.packed ? packed_offset<VB>(p, q2, k, e, &so)
                                         : pool_offset(p.src, at.r, at.c, at.t, k, e * VB, &so);
          const bool d_ok = p.dst.packed ? packed_offset<VB>(p, q2, k, e, &o)
                                         : pool_offset(p.dst, at.r, at.c, at.t, k, e * VB, &o);
          ok[j] = s_ok & d_ok;
          soff[j] = ok[j] ? so : 0;
          doff[j] = o;
        }
      }
    }
    V v[kVpt];
#pragma unroll
    for (int j = 0; j < kVpt; ++j) v[j] = __builtin_nontemporal_load(reinterpret_cast<const V*>(p.src.base + soff[j]));
#pragma unroll
    for (int j = 0; j < kVpt; ++j)
      if (ok[j]) __builtin_nontemporal_store(v[j], reinterpret_cast<V*>(p.dst.base + doff[j]));
  }
}

// Kept tokens of requests [0, r): the (plane, token) offset of request r in
// the packed order is planes times this.  Each wave sums the lengths on its own
// (lanes stride over them, then a butterfly), so no LDS and no barrier are
// involved.
// `mine` is seq_lens[lane] for lanes below r, already loaded by the caller.
__device__ __forceinline__ int32_t kept_before(const int32_t* __restrict__ seq_lens, int32_t r, int32_t max_tok,
                                               int32_t window, int32_t mine) {
  const int lane = threadIdx.x & 63;
  int32_t s = 0;
  for (int j = lane; j < r; j += 64) {
    int32_t n = j == lane ? mine : seq_lens[j];
    n = n < 0 ? 0 : (n > max_tok ? max_tok : n);
    s += (window > 0 && n > window) ? window : n;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
  return __builtin_amdgcn_readfirstlane(s);
}

// A 16-byte vector at any byte address: gfx950's vector memory instructions
// take unaligned addresses, so a chunk needs no alignment of its run.
typedef unsigned int Chunk16 __attribute__((ext_vector_type(4), aligned(1)));

// Entry i of a table row, i wave-uniform, through the scalar cache, the last entry kept.
__device__ __forceinline__ int32_t page_of_wave(const int32_t* row, uint32_t i, PageCache& pc) {
  if (i != pc.i) {
    pc.page = __builtin_amdgcn_readfirstlane(((const ConstInt*)row)[i]);
    pc.i = i;
  }
  return pc.page;
}

__device__ __forceinline__ bool page_ok(const Side& s, int32_t page) {
  return page >= 0 && (int64_t)page < s.num_pages;
}

// Byte of token t (in table entry i of a unit) of plane c, granule k, on a pool side.
__device__ __forceinline__ int64_t pool_byte(const Side& s, uint32_t c, uint32_t t, uint32_t k, uint32_t i,
                                             int32_t page) {
  return (int64_t)page * s.page_bytes + (int64_t)c * s.plane_bytes + (int64_t)(t - i * s.page.d) * s.slot_bytes +
         s.head0_bytes + (int64_t)k * s.gran_stride;
}

// The same with the page looked up, for the byte-by-byte chunks; false for a
// page outside the pool.
template <bool kPool>
__device__ __forceinline__ bool slow_page(const Side& s, const int32_t* row, uint32_t c, uint32_t unit, uint32_t t,
                                          uint32_t k, int64_t* off) {
  *off = 0;
  if (!kPool) return true;
  const uint32_t i = fdiv(unit, s.upp);
  const int32_t page = row[i];
  *off = pool_byte(s, c, t, k, i, page);
  return page_ok(s, page);
}

__device__ __forceinline__ void copy_bytes(char* dst, const char* src, int32_t n) {
  for (int32_t x = 0; x < n; ++x) dst[x] = src[x];
}

// Direct grid: workgroup (x, y, z) copies tile x of plane y of request z (of
// layer z / num_reqs when several layers go out in one grid), in packed order.
// With a window x and z change places: the first tiles of every request come
// first.  A window's grid is as long as the window for each request, and where
// requests are shorter than it only their first tiles have tokens; with a
// request's tiles side by side those recur every so many workgroups, and the
// round-robin dispatch gives them to few CUs (16 requests of 200 tokens of 1 KiB
// in windows of 1000: 7.5 -> 4.3 us a launch).
// A request's plane is cut into units: the most tokens that are one
// contiguous run on both sides (the smaller side's page, or what divides both
// page sizes, when whole rows move; one token when heads are sliced or laid
// out head-major), and a unit into 16-byte chunks (of its granules when it
// has several).  So a tile is full whatever the page size; the last unit or a
// window's first one is simply shorter.  A run's last chunk is moved back to
// end with the run: it repeats bytes of the chunk before it, with the same
// values, and no chunk needs any alignment.
//   kDir: pool -> packed, packed -> pool, or pool -> pool.
//   kWave: a unit's chunks fill whole 64-chunk wave spans, so every wave
//     instruction has one unit and page per side: scalar arithmetic and loads.
//     Otherwise every lane finds its own unit, and the lanes' table entries
//     are gathered (they share cache lines) before the data.
//   kHeads: several granules per unit (head-major sides, shard regions).
//   kHostLen: one request with the launch constant n_host; otherwise device
//     lengths, requests on grid z, each at the offset of the lengths before it.
// A unit's page depends on the length only through a window's start, so
// without a window the first lookups go out together with the length load.
// Tiles past a request's tokens exit at once.  Runs of fewer than 16 bytes
// (the last token or two of narrow rows) and runs that the packed capacity
// cuts short go byte by byte after the rest.
// Bound: HBM, below about 30 MB a launch the launch and one chain of table
// entry, data, store.  Measured against the persistent grid (its length scan,
// a request search and two dependent divisions per piece) on launches that
// only it took: 8 requests of 1-8k tokens in slices of two of eight 256-byte
// heads (68 MB read and written) 20.7 -> 16.7 us a launch, 16 MLA requests
// re-blocked 64 -> 16 (184 MB) 46.3 -> 36.5 us; and, with sides and lengths
// as template parameters and the store addresses kept out of the load phase,
// against the one-request grid before it, one 70B request's layer (33.5 MB)
// 7.8 -> 7.5 us.  With the first table entries and the length loaded together
// from preloaded arguments, and tiles sized as at max_vpt: 7.5 -> 7.25 us, the
// head slices 16.9 -> 14.8, the re-block 36.7 -> 35.7, 16 requests into
// one-token pages of 512 bytes (42 MB) 10.8 -> 9.6 (pack and unpack).
enum { kPack = 0, kUnpack = 1, kPools = 2 };

// What the table entries and the length are found with comes before Params as
// 14 dwords of plain arguments, which the hardware preloads into scalar
// registers: those loads go out next to a wave's loads of Params instead of
// behind them.  `shifts` holds the shift counts of the
// divisions by cpu, src.upp, dst.upp and the requests, a byte each.
constexpr uint32_t kWindowedBit = 1u << 31;                   // in `shifts`: the move has a window

// A tile of the live grid, found from the lengths.
struct LiveTile {
  uint32_t lz, c, base, n, before;   // layer, plane, first chunk, request's length, tokens of the requests before it
  int32_t r;
};

// One workgroup's tile in either grid: the direct one finds it from blockIdx
// and its length, the live one brings it.  (By value, as a kernel has them: a
// reference to Params makes the compiler order its loads differently.)
template <int kDir, bool kWave, bool kHeads, bool kHostLen, bool kLive, int VPT>
__device__ __forceinline__ void move_tile(const int32_t* src_tables, const int32_t* dst_tables, const int32_t* seq_lens,
                                          uint32_t shifts, uint32_t cpu_m, uint32_t src_upp_m, uint32_t dst_upp_m,
                                          uint32_t src_stride, uint32_t dst_stride, uint32_t num_reqs, uint32_t reqs_m,
                                          Params p, const LiveTile& live) {
  constexpr uint32_t kTile = (uint32_t)kThreads * VPT;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t wave_first = __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
  const uint32_t c = kLive ? live.c : blockIdx.y;
  const bool windowed = !kHostLen && (shifts & kWindowedBit);
  const bool lookup = kLive || windowed;                      // the table entries wait for the length
  const uint32_t block_z = windowed ? blockIdx.x : blockIdx.z, block_x = windowed ? blockIdx.z : blockIdx.x;
  const uint32_t cpu_s = shifts & 31u, src_upp_s = shifts >> 8 & 31u, dst_upp_s = shifts >> 16 & 31u;
  const uint32_t lz = kLive ? live.lz : kHostLen ? block_z : quot(block_z, reqs_m, shifts >> 24 & 31u);
  const int32_t r = kLive ? live.r : kHostLen ? 0 : (int32_t)(block_z - lz * num_reqs);
  const uint32_t base = kLive ? live.base : block_x * kTile;
  const int32_t* const src_row = kDir != kUnpack ? src_tables + (int64_t)r * src_stride : nullptr;
  const int32_t* const dst_row = kDir != kPack ? dst_tables + (int64_t)r * dst_stride : nullptr;
  // Without a window the units are known before the length, so their table
  // entries load next to it: this wave's first unit, or every lane's (kept
  // inside the row, whatever the tile; with a window, entries not used).
  constexpr int kEarly = kWave ? 1 : VPT;
  uint32_t is[kEarly], id[kEarly];
#pragma unroll
  for (int j = 0; j < kEarly; ++j) {
    const uint32_t u = quot(base + (kWave ? wave_first : j * kThreads + threadIdx.x), cpu_m, cpu_s);
    is[j] = quot(u, src_upp_m, src_upp_s);
    id[j] = quot(u, dst_upp_m, dst_upp_s);
    is[j] = is[j] < src_stride ? is[j] : src_stride - 1;
    id[j] = id[j] < dst_stride ? id[j] : dst_stride - 1;
  }
  const int32_t* const own_len = kHostLen || kLive ? nullptr : seq_lens + r;
  PageCache src_pc, dst_pc;
  int32_t spage[VPT], dpage[VPT];
  if (kLive) {
  } else if (kWave) {
    src_pc.i = is[0];
    dst_pc.i = id[0];
    if (kDir != kUnpack) src_pc.page = __builtin_amdgcn_readfirstlane(((const ConstInt*)src_row)[is[0]]);
    if (kDir != kPack) dst_pc.page = __builtin_amdgcn_readfirstlane(((const ConstInt*)dst_row)[id[0]]);
  } else {
#pragma unroll
    for (int j = 0; j < kEarly; ++j) {
      if (kDir != kUnpack) spage[j] = src_row[is[j]];
      if (kDir != kPack) dpage[j] = dst_row[id[j]];
    }
  }
  // with a batch, each lane below r also loads one earlier request's length
  // (for the request's packed offset) next to this request's own, so the
  // offset costs no memory latency of its own
  int32_t mine = 0;
  if (!kLive && !kHostLen && kDir != kPools) mine = __builtin_nontemporal_load(seq_lens + ((int32_t)lane < r ? (int32_t)lane : r));
  int32_t len = kLive ? (int32_t)live.n : kHostLen ? 0 : __builtin_amdgcn_readfirstlane(*(const ConstInt*)own_len);
  if (!kLive) __builtin_amdgcn_sched_barrier(0);                          // these loads go out before more index arithmetic
  if (kHostLen) len = p.n_host;
  if (!kLive && !kHostLen && kDir != kPools) asm volatile("" ::"v"(mine));   // keep the load here: not sunk past the exit test
  // Every cache line of Params is on its way with the length, not first
  // touched after the exit test.
  if (!kLive)
    asm volatile("" ::"s"(p.src.plane_bytes), "s"(p.src.upp.m), "s"(p.dst.page_bytes), "s"(p.packed_cap), "s"(p.gps.m),
                 "s"(p.cpu.m), "s"(p.strict));
  len = len < 0 ? 0 : (len > p.max_tok ? p.max_tok : len);
  const uint32_t n = (uint32_t)len;
  const uint32_t start = (p.window > 0 && len > p.window) ? (uint32_t)(len - p.window) : 0u;
  const uint32_t unit0 = p.window > 0 ? fdiv(start, p.unit) : 0u;                        // first unit with a moved token
  const uint32_t end = n > 0 ? (fdiv(n - 1, p.unit) + 1 - unit0) * p.cpu.d : 0u;         // chunks of this plane
  if (base >= end) return;                                                               // past this request's tokens
  const char* const src_base = p.src.base + (int64_t)lz * p.src.layer_stride;
  char* const dst_base = p.dst.base + (int64_t)lz * p.dst.layer_stride;

  // The packed side: the (plane, token) index of the plane's first moved
  // token and the bytes of each region of this layer.  False when the request
  // does not fit and moves whole or not at all; `cut` when its plane does not
  // fit and moves as far as it does.
  uint32_t q = 0;
  int64_t cap = INT64_MAX;
  bool cut = false;
  auto packed_side = [&]() -> bool {
    const uint32_t before = kLive ? live.before
                            : (!kHostLen && r > 0) ? (uint32_t)kept_before(seq_lens, r, p.max_tok, p.window, mine)
                                                   : 0u;
    q = (uint32_t)p.planes * before + c * (n - start);
    const int64_t left = p.total_cap - (int64_t)lz * (kDir == kPack ? p.dst.layer_stride : p.src.layer_stride);
    cap = left < p.packed_cap ? left : p.packed_cap;
    cut = (int64_t)(q + (n - start)) * p.region_gran > cap;
    return !(p.strict && (int64_t)((uint32_t)p.planes * (before + (n - start))) * p.region_gran > cap);
  };
  // Chunk j of this lane: its unit, first moved token and granule, the run it
  // belongs to and its place in that run.
  struct Piece {
    uint32_t unit, t, k;
    int32_t at, run;
    bool live;
  };
  auto piece = [&](uint32_t tile, int j) -> Piece {
    const uint32_t first = tile + j * kThreads + (kWave ? wave_first : threadIdx.x);
    Piece a;
    a.live = first < end;                                     // (kWave: whole spans)
    const uint32_t rel = a.live ? fdiv(first, p.cpu) : 0u;
    const uint32_t m = (a.live ? first - rel * p.cpu.d : 0u) + (kWave ? lane : 0u);
    a.unit = unit0 + rel;
    const uint32_t f = a.unit * p.unit.d;
    const uint32_t l = f + p.unit.d < n ? f + p.unit.d : n;
    a.t = f > start ? f : start;
    a.k = kHeads ? fdiv(m, p.cpg) : 0u;
    a.at = (int32_t)((kHeads ? m - a.k * p.cpg.d : m) * 16u);
    a.run = kHeads ? p.gran : (int32_t)(l - a.t) * p.gran;
    return a;
  };
  // Its run's offset on the packed side, and inside its region.
  auto packed_byte = [&](const Piece& a, int64_t* in_region) -> int64_t {
    const int64_t tok = (int64_t)(q + (a.t - start));
    if (!kHeads) return *in_region = tok * p.gran;
    const uint32_t sh = fdiv(a.k, p.gps);
    *in_region = (tok * p.gps.d + (a.k - sh * p.gps.d)) * p.gran;
    return *in_region + (int64_t)sh * p.packed_cap;
  };
  // Per lane, entries not loaded yet: all in flight together, ahead of the data
  // (a chunk past the end looks up the first unit).
  if (!kWave && lookup) {
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
      const uint32_t idx = base + j * kThreads + threadIdx.x;
      const uint32_t u = unit0 + (idx < end ? fdiv(idx, p.cpu) : 0u);
      if (kDir != kUnpack) spage[j] = src_row[fdiv(u, p.src.upp)];
      if (kDir != kPack) dpage[j] = dst_row[fdiv(u, p.dst.upp)];
    }
  }
  // The run's byte of each side; false when its page lies outside the pool.
  auto source = [&](const Piece& a, int j, int64_t* off) -> bool {
    if (kDir == kUnpack) {
      int64_t in_region;
      *off = packed_byte(a, &in_region);
      return true;
    }
    const uint32_t i = fdiv(a.unit, p.src.upp);
    const int32_t page = kWave ? page_of_wave(src_row, i, src_pc) : spage[j];
    *off = pool_byte(p.src, c, a.t, a.k, i, page);
    return page_ok(p.src, page);
  };
  auto target = [&](const Piece& a, int j, int64_t* off) -> bool {
    if (kDir == kPack) {
      int64_t in_region;
      *off = packed_byte(a, &in_region);
      return true;
    }
    const uint32_t i = fdiv(a.unit, p.dst.upp);
    const int32_t page = kWave ? page_of_wave(dst_row, i, dst_pc) : dpage[j];
    *off = pool_byte(p.dst, c, a.t, a.k, i, page);
    return page_ok(p.dst, page);
  };

  if (kDir == kUnpack && !packed_side()) return;
  // Every load, then every store.  No loop or branch sits between the loads:
  // a lane past its run's end loads the run's last chunk, and a chunk that
  // does not move that way (past the tokens, an outside page, a short or cut
  // run) the source's first bytes.  The stores' addresses are worked out
  // while the loads are in flight, not carried past them: their scalars would
  // not fit the registers.
  Chunk16 v[VPT];
  uint32_t voff[VPT];                                         // the chunk's place in its run
  uint32_t ok = 0;                                            // bit j: chunk j is a whole vector to store
#pragma unroll
  for (int j = 0; j < VPT; ++j) {
    const Piece a = piece(base, j);
    int64_t so;
    const bool in_pool = source(a, j, &so);
    const bool usable = a.live & in_pool & (a.run >= 16) & !cut;
    voff[j] = a.run >= 16 ? (uint32_t)(a.at < a.run - 16 ? a.at : a.run - 16) : 0u;
    ok |= ((usable & (a.at < a.run)) ? 1u : 0u) << j;
    v[j] = __builtin_nontemporal_load(
        reinterpret_cast<const Chunk16*>((usable ? src_base + so : p.src.base) + (usable || kDir != kUnpack ? voff[j] : 0u)));
  }
  if (kDir == kPack && !packed_side()) return;
  uint32_t tile = base;
  asm volatile("" : "+s"(tile));
  if (!cut) {
#pragma unroll
    for (int j = 0; j < VPT; ++j) {
      const Piece a = piece(tile, j);
      int64_t o;
      const bool in_pool = target(a, j, &o);
      if (in_pool & (ok >> j & 1)) __builtin_nontemporal_store(v[j], reinterpret_cast<Chunk16*>(dst_base + o + voff[j]));
    }
  }
  if (cut | (p.gran < 16 && !kHeads)) {
#pragma unroll 1
    for (int j = 0; j < VPT; ++j) {
      const Piece a = piece(tile, j);
      int64_t so, o, in_region = 0;
      const bool s_ok = slow_page<kDir != kUnpack>(p.src, src_row, c, a.unit, a.t, a.k, &so);
      const bool d_ok = slow_page<kDir != kPack>(p.dst, dst_row, c, a.unit, a.t, a.k, &o);
      int32_t run = a.run;
      if (kDir != kPools) {
        (kDir == kPack ? o : so) = packed_byte(a, &in_region);
        if (in_region + run > cap) run = in_region < cap ? (int32_t)(cap - in_region) & -p.grain : 0;
      }
      if (a.live && s_ok && d_ok && (cut || a.run < 16) && a.at < run)
        copy_bytes(dst_base + o + a.at, src_base + so + a.at, run - a.at < 16 ? run - a.at : 16);
    }
  }
}

template <int kDir, bool kWave, bool kHeads, bool kHostLen, int VPT>
__global__ __launch_bounds__(kThreads) void kv_reshard_direct_kernel(
    const int32_t* __restrict__ src_tables, const int32_t* __restrict__ dst_tables,
    const int32_t* __restrict__ seq_lens, uint32_t shifts, uint32_t cpu_m, uint32_t src_upp_m, uint32_t dst_upp_m,
    uint32_t src_stride, uint32_t dst_stride, uint32_t num_reqs, uint32_t reqs_m, Params p) {
  move_tile<kDir, kWave, kHeads, kHostLen, false, VPT>(src_tables, dst_tables, seq_lens, shifts, cpu_m, src_upp_m, dst_upp_m,
                                                       src_stride, dst_stride, num_reqs, reqs_m, p, LiveTile{});
}

// The live grid: the same tiles in a grid that follows the lengths instead of
// the table's width.  Workgroups stride over the tiles that have tokens; each
// scans the lengths once into the requests' live tiles and kept tokens
// (exclusive prefix sums in LDS) and finds a tile's request with two ballots.
// It takes the moves whose direct grid would have more than TOPKV_RS_SLOTS
// workgroups.
// A slot past its request's tokens costs the direct grid 0.41 ns, so tables
// wider than their requests, and batches of uneven ones, would cost more than
// the data.  us a launch, direct grid -> live grid: slices of two of eight
// heads, 64 requests of 1000 tokens in tables of 32768 113 -> 25, of 131072
// 419 -> 25, 64 x 100 in 32768 106 -> 5.8; 128 requests around 512 tokens (sigma
// 1) in a table that fits the longest 56 -> 35; MLA re-block, 64 x 1000 in 32768
// 99 -> 30; head-major, the same, 262 -> 90.  Where the requests fill their
// tables the two are even (slices 256 x 1000 89.7 and 89.4, head-major 355 and
// 356, 8 layers into one-token pages 184 and 188) but for the scan of a shorter
// launch (slices 64 x 1000, 8064 workgroups, 22.7 and 25.2): at the line a launch
// of dead slots costs the direct grid 3.4 us.
// One tile a workgroup, as far as the host can tell how many there are
// (live_workgroups): a workgroup that goes on to another tile is slower
// (2056-byte rows, 256 x 1000, 1 GB: 385 us in 24 workgroups per CU, 371 in 64,
// 362 in 128, one tile each), one too many costs 0.65 ns.
// 4 chunks per lane: slices 64 x 1000 25.0 us with 2, 24.3 with 4, 24.8 with 8;
// two TP2 shards, 64 x 4096, one tile a workgroup 372 with 4, 376 with 8.  8 only
// for wave spans between pools that must go on to further tiles: half as many
// (re-block 16 -> 64, 64 x 4096, 1 GB: 432 -> 424; four layers of 16 x 4096 215 -> 208).
__device__ void live_prefix(const Params& p, const int32_t* __restrict__ seq_lens, uint32_t tile, int32_t* first,
                            int32_t* kept, int32_t* lens, uint64_t* wsum) {
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  uint64_t carry = 0;                                         // kept tokens in the high half, tiles in the low one
  for (int32_t at = 0; at < p.num_reqs; at += kThreads) {
    const int32_t r = at + (int32_t)threadIdx.x;
    uint64_t v = 0;
    if (r < p.num_reqs) {
      int32_t len = seq_lens[r];
      len = len < 0 ? 0 : (len > p.max_tok ? p.max_tok : len);
      lens[r] = len;
      if (len > 0) {
        const uint32_t start = (p.window > 0 && len > p.window) ? (uint32_t)(len - p.window) : 0u;
        const uint32_t units = fdiv((uint32_t)len - 1, p.unit) + 1 - fdiv(start, p.unit);
        const uint32_t tiles = (units * p.cpu.d + tile - 1) / tile;
        v = (uint64_t)((uint32_t)len - start) << 32 | (uint32_t)p.planes * tiles;
      }
    }
    uint64_t x = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint64_t y = __shfl_up(x, d, 64);
      if (lane >= d) x += y;
    }
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    uint64_t before = carry, all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      if (w < wave) before += wsum[w];
      all += wsum[w];
    }
    if (r < p.num_reqs) {
      first[r] = (int32_t)(uint32_t)(before + x - v);
      kept[r] = (int32_t)((before + x - v) >> 32);
    }
    carry += all;
    __syncthreads();
  }
  if (threadIdx.x == 0) first[p.num_reqs] = (int32_t)(uint32_t)carry;
  __syncthreads();
}

// The request that tile t < first[num_reqs] belongs to: the last one with
// first[r] <= t.  A wave tests one request in `step` and then that step's; at
// most 64 x 64 requests.
__device__ __forceinline__ int32_t tile_owner(const int32_t* first, int32_t num_reqs, int32_t t) {
  const int32_t lane = threadIdx.x & 63;
  const int32_t step = (num_reqs + 63) >> 6;
  const int32_t a = lane * step;
  const int32_t group = (__popcll(__ballot(a < num_reqs && first[a < num_reqs ? a : 0] <= t)) - 1) * step;
  if (step == 1) return group;
  const int32_t b = group + lane;
  const bool in = lane < step && b < num_reqs;
  return group + __popcll(__ballot(in && first[in ? b : 0] <= t)) - 1;
}

template <int kDir, bool kWave, bool kHeads, int VPT>
__global__ __launch_bounds__(kThreads) void kv_reshard_live_kernel(const int32_t* __restrict__ src_tables,
                                                                   const int32_t* __restrict__ dst_tables,
                                                                   const int32_t* __restrict__ seq_lens, uint32_t layers,
                                                                   Params p) {
  constexpr uint32_t kTile = (uint32_t)kThreads * VPT;
  extern __shared__ uint64_t lds_u64[];
  int32_t* const first = reinterpret_cast<int32_t*>(lds_u64 + kWaves);   // [num_reqs + 1]
  int32_t* const kept = first + p.num_reqs + 1;                          // [num_reqs]
  int32_t* const lens = kept + p.num_reqs;                               // [num_reqs]
  live_prefix(p, seq_lens, kTile, first, kept, lens, lds_u64);
  const uint32_t per_layer = (uint32_t)__builtin_amdgcn_readfirstlane(first[p.num_reqs]);
  const uint32_t all = per_layer * layers;                               // the host keeps this below 2^31
  for (uint32_t w = blockIdx.x; w < all; w += gridDim.x) {
    const uint32_t lz = w / per_layer;
    const uint32_t t = w - lz * per_layer;
    const int32_t r = __builtin_amdgcn_readfirstlane(tile_owner(first, p.num_reqs, (int32_t)t));
    const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane(lens[r]);
    const uint32_t before = (uint32_t)__builtin_amdgcn_readfirstlane(kept[r]);
    const uint32_t local = t - (uint32_t)__builtin_amdgcn_readfirstlane(first[r]);
    const uint32_t tiles = (uint32_t)__builtin_amdgcn_readfirstlane(first[r + 1] - first[r]) / (uint32_t)p.planes;
    const uint32_t c = local / tiles;
    move_tile<kDir, kWave, kHeads, false, true, VPT>(src_tables, dst_tables, seq_lens, 0, 0, 0, 0,
                                                     (uint32_t)p.src.bt_stride, (uint32_t)p.dst.bt_stride, 0, 0, p,
                                                     LiveTile{lz, c, (local - c * tiles) * kTile, n, before, r});
  }
}

// One request's plain layer: the direct grid's case of whole rows between a
// pool and a packed buffer, no window, a row a multiple of 16 bytes and a page
// plane whole wave spans.  The plane is then one run of 16-byte chunks on the
// packed side, a span lies in one page, and nothing is left but the page's
// place.  Lane j of a wave loads the table entry of span j next to the length,
// one load for all.  The short code lets a lane take up to 16 chunks, so the
// grid fills the chip in one round of workgroups, or in two.
// A request that does not fit the packed bytes is not moved; a page outside
// the pool is not moved (its loads go to page 0, its stores nowhere).
// Bound: the launch and the chain of entry, data, store below about 8 MB a
// launch, HBM above.  Against the general direct grid (a unit, a run and a
// page of its own for each chunk), one 70B layer, us a launch: 1000 tokens
// (8 MB read and written) 4.0 -> 3.3, 2048 5.0 -> 4.4, 4096 7.2 -> 6.6 (5.1
// TB/s), 8192 13.9 -> 12.6, 32000 49.0 -> 48.6; one head, 16384 tokens 5.0 -> 4.5.
struct RowsParams {
  int64_t page_bytes, plane_bytes;
  uint32_t num_pages, max_total;   // max_total: chunks of a plane that fit the packed bytes
  int32_t max_tok;
};

template <bool kPack, bool kHostLen, int VPT>
__global__ __launch_bounds__(kThreads) void kv_rows_kernel(char* __restrict__ pool, char* __restrict__ packed,
                                                           const int32_t* __restrict__ table,
                                                           const int32_t* __restrict__ seq_lens, int32_t n_host,
                                                           uint32_t bt_stride, uint32_t per_page, uint32_t per_page_m,
                                                           uint32_t per_page_s, uint32_t per_token, RowsParams p) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t base = blockIdx.x * (kThreads * VPT) + __builtin_amdgcn_readfirstlane(threadIdx.x & ~63u);
  const uint32_t i = quot(base + (lane < VPT ? lane : VPT - 1) * kThreads, per_page_m, per_page_s);
  const int32_t entries = table[i < bt_stride ? i : bt_stride - 1];
  int32_t len = kHostLen ? n_host : __builtin_amdgcn_readfirstlane(*(const ConstInt*)seq_lens);
  asm volatile("" ::"v"(entries), "s"(p.page_bytes), "s"(p.max_total));      // loads of their own are on their way by now
  len = len < 0 ? 0 : (len > p.max_tok ? p.max_tok : len);
  const uint32_t total = (uint32_t)len * per_token;                          // chunks of a plane
  if (base >= total || total > p.max_total) return;
  char* const pool_plane = pool + (int64_t)blockIdx.y * p.plane_bytes;
  char* const packed_plane = packed + (int64_t)blockIdx.y * total * 16;
  // Every load, then every store.  A chunk past the tokens loads the pool's
  // first ones or the plane's last one, one of a page outside the pool the
  // pool's first ones.
  Chunk16 v[VPT];
  uint32_t ok = 0;
#pragma unroll
  for (int j = 0; j < VPT; ++j) {
    const uint32_t first = base + j * kThreads;
    const uint32_t entry = (uint32_t)__builtin_amdgcn_readlane(entries, j);
    const bool usable = (first < total) & (entry < p.num_pages);
    ok |= (usable ? 1u : 0u) << j;
    const char* from;
    if (kPack) {
      const uint32_t m = first - quot(first, per_page_m, per_page_s) * per_page;
      from = pool_plane + (usable ? (int64_t)entry * p.page_bytes + (int64_t)m * 16 : 0) + lane * 16u;
    } else {
      from = packed_plane + (int64_t)(first + lane < total ? first + lane : total - 1) * 16;
    }
    v[j] = __builtin_nontemporal_load(reinterpret_cast<const Chunk16*>(from));
  }
#pragma unroll
  for (int j = 0; j < VPT; ++j) {
    const uint32_t first = base + j * kThreads;
    char* to;
    if (kPack) {
      to = packed_plane + (int64_t)first * 16 + lane * 16u;
    } else {
      const uint32_t m = first - quot(first, per_page_m, per_page_s) * per_page;
      to = pool_plane + (int64_t)(uint32_t)__builtin_amdgcn_readlane(entries, j) * p.page_bytes + (int64_t)m * 16 + lane * 16u;
    }
    if ((ok >> j & 1) && first + lane < total) __builtin_nontemporal_store(v[j], reinterpret_cast<Chunk16*>(to));
  }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

constexpr int kMaxDevices = 64;
std::atomic<int> g_cus[kMaxDevices];

topkv_status_t cu_count(int* out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return TOPKV_ERR_DEVICE;
  const int cached = dev < kMaxDevices ? g_cus[dev].load(std::memory_order_relaxed) : 0;
  if (cached > 0) { *out = cached; return TOPKV_OK; }
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0)
    return TOPKV_ERR_DEVICE;
  if (dev < kMaxDevices) g_cus[dev].store(cus, std::memory_order_relaxed);
  *out = cus;
  return TOPKV_OK;
}

struct PoolInfo {
  int64_t head_bytes, slot_bytes, plane_bytes, page_bytes, layer_bytes;
};

// Strides of a pool view in its layout, after validating the descriptor.
topkv_status_t pool_info(const topkv_view_t* v, int32_t head_count, PoolInfo* g) {
  const topkv_pool_t& pl = v->pool;
  if (!pl.base || pl.num_pages <= 0 || pl.num_layers <= 0 || pl.page_size <= 0 || pl.planes <= 0 ||
      pl.num_heads <= 0 || pl.head_dim <= 0)
    return TOPKV_ERR_INVALID_ARG;
  if (pl.elem_bytes != 1 && pl.elem_bytes != 2 && pl.elem_bytes != 4 && pl.elem_bytes != 8)
    return TOPKV_ERR_INVALID_ARG;
  if (v->layer < 0 || v->layer >= pl.num_layers || v->bt_stride <= 0 || v->head_begin < 0 ||
      head_count > pl.num_heads - v->head_begin)
    return TOPKV_ERR_INVALID_ARG;
  int64_t head, row, plane, page, layer, all;
  if (__builtin_mul_overflow((int64_t)pl.head_dim, (int64_t)pl.elem_bytes, &head) ||
      __builtin_mul_overflow(head, (int64_t)pl.num_heads, &row) ||
      __builtin_mul_overflow(row, (int64_t)pl.page_size, &plane) ||
      __builtin_mul_overflow(plane, (int64_t)pl.planes, &page) ||
      __builtin_mul_overflow(page, pl.num_pages, &layer) ||
      __builtin_mul_overflow(layer, (int64_t)pl.num_layers, &all))
    return TOPKV_ERR_UNSUPPORTED;
  if (plane > INT32_MAX || pl.num_pages > INT32_MAX) return TOPKV_ERR_UNSUPPORTED;
  const bool head_major = v->layout == TOPKV_LAYOUT_POOL_HEAD_MAJOR;
  g->head_bytes = head_major ? head * pl.page_size : head;
  g->slot_bytes = head_major ? head : row;
  g->plane_bytes = plane;
  g->page_bytes = page;
  g->layer_bytes = layer;
  return TOPKV_OK;
}

bool valid_layout(int32_t l) {
  return l == TOPKV_LAYOUT_PACKED || l == TOPKV_LAYOUT_POOL || l == TOPKV_LAYOUT_POOL_HEAD_MAJOR;
}

typedef void (*KernelFn)(Params, const int32_t*);
typedef void (*DirectFn)(const int32_t*, const int32_t*, const int32_t*, uint32_t, uint32_t, uint32_t, uint32_t,
                         uint32_t, uint32_t, uint32_t, uint32_t, Params);

template <bool kWave>
KernelFn kernel_for_mode(int vb) {
  switch (vb) {
    case 16: return kv_reshard_kernel<16, kWave>;
    case 8: return kv_reshard_kernel<8, kWave>;
    case 4: return kv_reshard_kernel<4, kWave>;
    case 2: return kv_reshard_kernel<2, kWave>;
    default: return kv_reshard_kernel<1, kWave>;
  }
}

KernelFn kernel_for(int vb, bool wave) { return wave ? kernel_for_mode<true>(vb) : kernel_for_mode<false>(vb); }

// Chunks per lane of a direct grid, at most.  Lanes that find their own units
// take 2: with 8 each lane's table entries and addresses pile up ahead of its
// first load (8 requests in slices of two of eight heads, 68 MB a launch:
// 16.9 us with 8, 15.8 with 4, 14.8 with 2, 18.3 with 1; 350-byte rows, 26 MB:
// 8.9, 8.1, 7.8 and 9.4).  Whole wave spans take 4 where a span's sides lie
// scattered over heads or two pools (MLA re-block, 184 MB: 36.4 us with 8,
// 35.7 with 4, 41.3 with 2; head-major, 270 MB: 102 us, 98.7, 98.8), and 8 (32
// KiB tiles, as the page grids use) between a pool and a packed buffer.
constexpr int max_vpt(bool wave, bool scattered) { return !wave ? 2 : scattered ? 4 : 8; }

template <int kDir, bool kWave, bool kHeads, bool kHostLen>
DirectFn direct_kernel_vpt(int vpt) {
  constexpr int kMax = max_vpt(kWave, kHeads || kDir == kPools);
  switch (vpt) {
    case 8: return kv_reshard_direct_kernel<kDir, kWave, kHeads, kHostLen, (kMax >= 8) ? 8 : kMax>;
    case 4: return kv_reshard_direct_kernel<kDir, kWave, kHeads, kHostLen, (kMax >= 4) ? 4 : kMax>;
    case 2: return kv_reshard_direct_kernel<kDir, kWave, kHeads, kHostLen, 2>;
    default: return kv_reshard_direct_kernel<kDir, kWave, kHeads, kHostLen, 1>;
  }
}

template <int kDir>
DirectFn direct_kernel_dir(bool wave, bool heads, int vpt) {
  if (heads) return wave ? direct_kernel_vpt<kDir, true, true, false>(vpt) : direct_kernel_vpt<kDir, false, true, false>(vpt);
  return wave ? direct_kernel_vpt<kDir, true, false, false>(vpt) : direct_kernel_vpt<kDir, false, false, false>(vpt);
}

// A host length comes from a plain pack or unpack only: whole rows, one packed side.
template <int kDir>
DirectFn direct_kernel_host(bool wave, int vpt) {
  return wave ? direct_kernel_vpt<kDir, true, false, true>(vpt) : direct_kernel_vpt<kDir, false, false, true>(vpt);
}

DirectFn direct_kernel_for(int dir, bool wave, bool heads, bool host_len, int vpt) {
  if (host_len) return dir == kPack ? direct_kernel_host<kPack>(wave, vpt) : direct_kernel_host<kUnpack>(wave, vpt);
  switch (dir) {
    case kPack: return direct_kernel_dir<kPack>(wave, heads, vpt);
    case kUnpack: return direct_kernel_dir<kUnpack>(wave, heads, vpt);
    default: return direct_kernel_dir<kPools>(wave, heads, vpt);
  }
}

typedef void (*LiveFn)(const int32_t*, const int32_t*, const int32_t*, uint32_t, Params);

template <int kDir>
LiveFn live_kernel_dir(bool wave, bool heads) {
  if (heads)
    return wave ? kv_reshard_live_kernel<kDir, true, true, kLiveVpt> : kv_reshard_live_kernel<kDir, false, true, kLiveVpt>;
  return wave ? kv_reshard_live_kernel<kDir, true, false, kLiveVpt> : kv_reshard_live_kernel<kDir, false, false, kLiveVpt>;
}

// vpt: kLiveVpt, or twice that (wave spans between pools)
LiveFn live_kernel_for(int dir, bool wave, bool heads, int vpt) {
  if (vpt > kLiveVpt)
    return heads ? kv_reshard_live_kernel<kPools, true, true, 2 * kLiveVpt>
                 : kv_reshard_live_kernel<kPools, true, false, 2 * kLiveVpt>;
  switch (dir) {
    case kPack: return live_kernel_dir<kPack>(wave, heads);
    case kUnpack: return live_kernel_dir<kUnpack>(wave, heads);
    default: return live_kernel_dir<kPools>(wave, heads);
  }
}

typedef void (*RowsFn)(char*, char*, const int32_t*, const int32_t*, int32_t, uint32_t, uint32_t, uint32_t, uint32_t,
                       uint32_t, RowsParams);

template <bool kPack, bool kHostLen>
RowsFn rows_kernel_vpt(int vpt) {
  switch (vpt) {
    case 16: return kv_rows_kernel<kPack, kHostLen, 16>;
    case 12: return kv_rows_kernel<kPack, kHostLen, 12>;
    case 8: return kv_rows_kernel<kPack, kHostLen, 8>;
    case 6: return kv_rows_kernel<kPack, kHostLen, 6>;
    case 4: return kv_rows_kernel<kPack, kHostLen, 4>;
    case 3: return kv_rows_kernel<kPack, kHostLen, 3>;
    case 2: return kv_rows_kernel<kPack, kHostLen, 2>;
    default: return kv_rows_kernel<kPack, kHostLen, 1>;
  }
}

RowsFn rows_kernel_for(bool pack, bool host_len, int vpt) {
  if (host_len) return pack ? rows_kernel_vpt<true, true>(vpt) : rows_kernel_vpt<false, true>(vpt);
  return pack ? rows_kernel_vpt<true, false>(vpt) : rows_kernel_vpt<false, false>(vpt);
}

// The most workgroups of a live grid that are still one for each tile.  With a
// packed side, whose size follows the batch, 256 per CU (lanes that find their
// own units, which gain less: 128), or 32 and a layer.  Between pools, whose size
// doesn't (a big pool and a few short requests would be all dead workgroups), 32
// per CU and layer: the dead ones take 5 us at most, which the general grid takes
// for its smallest launch.  us a launch at 128, 256 and 512 per CU: two TP2
// shards, 64 x 4096 (1 GB) 390, 372, 372; head-major 100 uneven requests (2.6 GB)
// 917, 878, 854.
int64_t live_most(int64_t layers, int64_t cus, bool pools, bool wave) {
  const int64_t most = pools ? 32 * layers : wave ? 256 : 128;
  return cus * (most > 32 * layers ? most : 32 * layers);
}

int64_t gcd(int64_t a, int64_t b) {
  while (b) {
    const int64_t r = a % b;
    a = b;
    b = r;
  }
  return a;
}

// direct_only: launch only a grid of up to 1024 requests (rows, direct or live;
// *launched reports whether it did), for a plain pack or unpack whose caller
// has its own kernels; otherwise whichever grid applies.  layers > 1: the
// views' layers and the next layers - 1 in one direct or live grid (a pool
// side's layer slabs follow each other; a packed side's layer z starts at data
// + z * packed_layer_stride), launched only when one of them applies: *launched
// stays false otherwise, with nothing queued.  The caller has checked the
// layer ranges and the stride.  total_cap >= 0: packed bytes of all layers
// together; strict: requests that do not fit their layer's packed bytes are
// not moved (else their pieces that do fit are).
topkv_status_t move_layer_impl(const topkv_view_t* src, const topkv_view_t* dst, int32_t num_reqs,
                               const int32_t* seq_lens, int32_t head_count, int32_t window,
                               const topkv_launch_t& launch, bool direct_only, bool* launched,
                               int32_t n_host = -1, int32_t layers = 1, int64_t packed_layer_stride = 0,
                               int64_t total_cap = -1, bool strict = false) {
  *launched = false;
  if (!src || !dst || !valid_layout(src->layout) || !valid_layout(dst->layout)) return TOPKV_ERR_INVALID_ARG;
  if (src->layout == TOPKV_LAYOUT_PACKED && dst->layout == TOPKV_LAYOUT_PACKED) return TOPKV_ERR_INVALID_ARG;
  // a host-side length (n_host >= 0) stands for seq_lens: one request of a plain pack or unpack
  const bool host_len = n_host >= 0;
  if (host_len && (num_reqs != 1 || !direct_only || seq_lens)) return TOPKV_ERR_INVALID_ARG;
  if (num_reqs < 0 || head_count <= 0 || window < 0 || (num_reqs > 0 && !seq_lens && !host_len))
    return TOPKV_ERR_INVALID_ARG;
  if (num_reqs > TOPKV_MAX_BATCH_REQS) return TOPKV_ERR_UNSUPPORTED;

  const topkv_view_t* sides[2] = {src, dst};
  const topkv_pool_t* geo = nullptr;     // geometry both pool sides share
  PoolInfo info[2] = {};
  int64_t packed_cap = 0;
  int64_t shards = 1;
  int64_t max_tok = INT32_MAX;
  for (int i = 0; i < 2; ++i) {
    const topkv_view_t* v = sides[i];
    if (v->layout == TOPKV_LAYOUT_PACKED) {
      if (v->bytes < 0 || (v->bytes > 0 && !v->data) || v->shards < 0) return TOPKV_ERR_INVALID_ARG;
      packed_cap = v->bytes;
      shards = v->shards > 1 ? v->shards : 1;
      if (head_count % shards != 0) return TOPKV_ERR_INVALID_ARG;
      continue;
    }
    const topkv_status_t st = pool_info(v, head_count, &info[i]);
    if (st != TOPKV_OK) return st;
    if (num_reqs > 0 && !v->block_tables) return TOPKV_ERR_INVALID_ARG;
    if (geo && (geo->planes != v->pool.planes || geo->head_dim != v->pool.head_dim ||
                geo->elem_bytes != v->pool.elem_bytes))
      return TOPKV_ERR_INVALID_ARG;
    geo = &v->pool;
    const int64_t cap = (int64_t)v->bt_stride * v->pool.page_size;
    if (cap < max_tok) max_tok = cap;
  }
  if (num_reqs == 0) return TOPKV_OK;

  // Checked mode: validate each pool side's tables (an unpack destination for
  // pages named twice), and the packed side's room for every kept token.  The
  // one-request route from a pack/unpack call was checked by its caller.
  if (!direct_only && topkv_internal::checked_mode()) {
    const bool has_packed = src->layout == TOPKV_LAYOUT_PACKED || dst->layout == TOPKV_LAYOUT_PACKED;
    const int64_t per_token = (int64_t)geo->planes * (head_count / shards) * geo->head_dim * geo->elem_bytes;
    bool cap_checked = false;
    for (int i = 0; i < 2; ++i) {
      const topkv_view_t* v = sides[i];
      if (v->layout == TOPKV_LAYOUT_PACKED) continue;
      const bool with_cap = has_packed && !cap_checked;
      const topkv_status_t cs = topkv_internal::checked_tables(
          &v->pool, num_reqs, v->block_tables, v->bt_stride, seq_lens, 0, window, i == 1, with_cap ? per_token : 0,
          0, with_cap ? packed_cap : INT64_MAX, launch.stream);
      if (cs != TOPKV_OK) return cs;
      cap_checked = cap_checked || with_cap;
    }
  }

  // Heads ride together in one granule when both sides keep them adjacent.
  const int64_t head = (int64_t)geo->head_dim * geo->elem_bytes;
  bool adjacent = true;
  for (int i = 0; i < 2; ++i)
    if (sides[i]->layout == TOPKV_LAYOUT_POOL_HEAD_MAJOR) adjacent = false;
  const int64_t heads_per_gran = adjacent ? head_count / shards : 1;
  const int64_t gran = heads_per_gran * head;
  // Piece width: every stride and base the pieces are addressed with.
  int vb = 16;
  for (; vb > 1; vb >>= 1) {
    bool fits = gran % vb == 0;
    for (int i = 0; i < 2 && fits; ++i) {
      const topkv_view_t* v = sides[i];
      if (v->layout == TOPKV_LAYOUT_PACKED) {
        fits = reinterpret_cast<uintptr_t>(v->data) % vb == 0 && (shards == 1 || packed_cap % vb == 0) &&
               packed_layer_stride % vb == 0;
      } else {
        const uintptr_t b = reinterpret_cast<uintptr_t>(v->pool.base);
        fits = b % vb == 0 && info[i].layer_bytes % vb == 0 && info[i].page_bytes % vb == 0 &&
               info[i].plane_bytes % vb == 0 && info[i].slot_bytes % vb == 0 && info[i].head_bytes % vb == 0;
      }
    }
    if (fits) break;
  }
  const int64_t vpg = gran / vb;
  const int64_t gpt = head_count / heads_per_gran;
  // Upper bound of pieces in the launch; indices are 32-bit in the kernel.
  if (max_tok <= 0) return TOPKV_OK;
  int64_t bound;
  if (__builtin_mul_overflow((int64_t)num_reqs * max_tok, (int64_t)geo->planes, &bound) ||
      __builtin_mul_overflow(bound, gpt * vpg, &bound) || bound >= ((int64_t)1 << 31) || vpg >= ((int64_t)1 << 31))
    return TOPKV_ERR_UNSUPPORTED;
  // Skipped pieces load from the source's base, so it must hold one piece; a
  // packed source smaller than that holds nothing to move.
  if (src->layout == TOPKV_LAYOUT_PACKED && packed_cap < vb) return TOPKV_OK;

  Params p = {};
  for (int i = 0; i < 2; ++i) {
    const topkv_view_t* v = sides[i];
    Side& s = i == 0 ? p.src : p.dst;
    if (v->layout == TOPKV_LAYOUT_PACKED) {
      s.base = static_cast<char*>(v->data);
      s.layer_stride = packed_layer_stride;
      s.packed = 1;
      s.page = make_div(1);
      continue;
    }
    s.base = static_cast<char*>(v->pool.base) + (int64_t)v->layer * info[i].layer_bytes;
    s.layer_stride = info[i].layer_bytes;
    s.tables = v->block_tables;
    s.page_bytes = info[i].page_bytes;
    s.plane_bytes = info[i].plane_bytes;
    s.head0_bytes = (int64_t)v->head_begin * info[i].head_bytes;
    s.num_pages = v->pool.num_pages;
    s.slot_bytes = (int32_t)info[i].slot_bytes;
    s.gran_stride = (int32_t)(heads_per_gran * info[i].head_bytes);
    s.bt_stride = v->bt_stride;
    s.page = make_div((uint32_t)v->pool.page_size);
  }
  p.packed_cap = src->layout == TOPKV_LAYOUT_PACKED || dst->layout == TOPKV_LAYOUT_PACKED ? packed_cap : INT64_MAX;
  p.vpg = make_div((uint32_t)vpg);
  p.gpt = make_div((uint32_t)gpt);
  p.ktp = make_div((uint32_t)(gpt * vpg));
  p.gps = make_div((uint32_t)(gpt / shards));
  p.num_reqs = num_reqs;
  p.planes = geo->planes;
  p.window = window;
  p.max_tok = (int32_t)max_tok;
  p.n_host = host_len ? (n_host < max_tok ? n_host : (int32_t)max_tok) : 0;

  // Direct grid: units of the most tokens that are one run on both sides.
  // Whole rows of a slot-major pool are adjacent over a page's slots, and a
  // packed side's over all tokens.
  const bool heads = gpt > 1;
  int64_t unit = 0;
  for (int i = 0; i < 2; ++i) {
    const topkv_view_t* v = sides[i];
    if (v->layout == TOPKV_LAYOUT_PACKED) continue;
    const bool rows = !heads && head_count == v->pool.num_heads;
    unit = rows ? gcd(unit, v->pool.page_size) : 1;
    if (!rows) break;
  }
  const int64_t cpg = (gran + 15) / 16;
  const int64_t cpu = heads ? gpt * cpg : (unit * gran + 15) / 16;
  const int64_t max_units = (max_tok + unit - 1) / unit;
  int64_t grid_units = max_units;
  if (host_len) grid_units = ((int64_t)p.n_host + unit - 1) / unit;
  else if (window > 0 && ((int64_t)window + unit - 2) / unit + 1 < max_units)
    grid_units = ((int64_t)window + unit - 2) / unit + 1;   // units that `window` consecutive tokens can touch
  // Chunks are 16 bytes, so a unit's run (a granule's, when it has several)
  // holds at least one; indices stay below 2^31.
  const int64_t span = grid_units * cpu;
  bool direct = !(host_len && (heads || window > 0)) && (heads ? gran : unit * gran) >= 16 && unit * gran <= INT32_MAX - 16 &&
                span < ((int64_t)1 << 31) - 16 * kThreads && geo->planes <= 65535 && layers <= 65535 &&
                (src->layout != TOPKV_LAYOUT_PACKED || (packed_cap >= 16 && (total_cap < 0 || total_cap >= 16)));
  // Up to 1024 requests: each workgroup of the direct grid sums the lengths
  // before its request, each of the live grid holds all of them in LDS.
  direct = direct && num_reqs <= 1024 && (int64_t)num_reqs * layers <= 65535;
  if (direct && grid_units == 0) return TOPKV_OK;             // a host-side length of 0: nothing to move
  if (!direct && (direct_only || layers > 1)) return TOPKV_OK;

  const dim3 threads(kThreads);
  dim3 grid;
  size_t lds = 0;
  const bool to_packed = dst->layout == TOPKV_LAYOUT_PACKED;
  if (direct && strict && num_reqs == 1 && layers == 1 && window == 0 && !heads && gran % 16 == 0 && cpu % 64 == 0 &&
      (to_packed || src->layout == TOPKV_LAYOUT_PACKED)) {
    int cus = 0;
    const topkv_status_t st = cu_count(&cus);
    if (st != TOPKV_OK) return st;
    auto workgroups = [&](int v) { return (span + v * kThreads - 1) / (v * kThreads) * geo->planes; };
    // The smallest tiles that leave at most one workgroup per CU, or fill most
    // of two rounds; past that 32 KiB tiles (24 KiB ones while they make three
    // rounds, where 32 KiB make a little more than two), and 4 KiB ones when the
    // host knows the length (a table wider than its request costs a workgroup per
    // tile that is not there).  One 70B layer, us a launch: 4096 tokens 6.5 in
    // 256 workgroups, 7.6-8.2 in more; 4200 tokens 8.2 in 32 KiB tiles, 7.5 in 24
    // KiB ones; 8192 tokens 12.6 in 512 workgroups, 13.6-14.2 in more; 32000
    // tokens 46.4 in 4 KiB tiles, 48.6 in 32 KiB ones; 500 tokens in a table of
    // 32768 4.3 in 32 KiB tiles, 12.0 in 4 KiB ones.
    int vpt = host_len ? 1 : workgroups(6) <= 3 * (int64_t)cus ? 6 : 8;
    for (const int v : {1, 2, 3, 4, 6, 8, 12, 16}) {
      const int64_t w = workgroups(v);
      if (w > cus && !(v >= 12 && w <= 2 * cus && w * 10 >= cus * 16)) continue;
      vpt = v;
      break;
    }
    const Side& ps = to_packed ? p.src : p.dst;
    char *pool_base = ps.base, *packed_base = to_packed ? p.dst.base : p.src.base;
    const int32_t* table = ps.tables;
    FastDiv per_page = make_div((uint32_t)cpu);
    uint32_t stride = (uint32_t)ps.bt_stride, per_token = (uint32_t)(gran / 16);
    const int64_t fit = (total_cap >= 0 && total_cap < packed_cap ? total_cap : packed_cap) / 16 / geo->planes;
    RowsParams q = {ps.page_bytes, ps.plane_bytes, (uint32_t)ps.num_pages, fit < UINT32_MAX ? (uint32_t)fit : UINT32_MAX,
                    p.max_tok};
    void* args[] = {&pool_base, &packed_base, &table, &seq_lens, &p.n_host, &stride, &per_page.d, &per_page.m, &per_page.s,
                    &per_token, &q};
    const void* f = reinterpret_cast<const void*>(rows_kernel_for(to_packed, host_len, vpt));
    grid = dim3((unsigned)((span + vpt * kThreads - 1) / (vpt * kThreads)), (unsigned)geo->planes);
    const hipError_t e = launch.start || launch.stop
                             ? hipExtLaunchKernel(f, grid, threads, args, 0, launch.stream, launch.start, launch.stop, 0)
                             : hipLaunchKernel(f, grid, threads, args, 0, launch.stream);
    if (e != hipSuccess) return TOPKV_ERR_LAUNCH;
    *launched = true;
    return TOPKV_OK;
  }
  KernelFn fn;
  if (direct) {
    p.unit = make_div((uint32_t)unit);
    p.cpu = make_div((uint32_t)cpu);
    p.cpg = make_div((uint32_t)cpg);
    p.total_cap = total_cap < 0 ? INT64_MAX : total_cap;
    p.gran = (int32_t)gran;
    p.region_gran = (int32_t)(gpt / shards * gran);
    p.reqs = make_div((uint32_t)num_reqs);
    p.grain = vb;
    p.strict = strict ? 1 : 0;
    for (int i = 0; i < 2; ++i) {
      Side& s = i == 0 ? p.src : p.dst;
      s.upp = make_div(s.packed ? 1u : (uint32_t)(sides[i]->pool.page_size / unit));
    }
    const int dir = dst->layout == TOPKV_LAYOUT_PACKED ? kPack : src->layout == TOPKV_LAYOUT_PACKED ? kUnpack : kPools;
    const bool wave = cpu % 64 == 0, scattered = heads || dir == kPools;
    auto workgroups = [&](int v) {
      return (span + v * kThreads - 1) / (v * kThreads) * geo->planes * num_reqs * layers;
    };
    // The most chunks per lane there may be while they give the chip two
    // workgroups per CU; below that, smaller tiles.
    int vpt = max_vpt(wave, scattered);
    while (vpt > 1 && workgroups(vpt) < TOPKV_RS_FILL) vpt >>= 1;
    if (!host_len && workgroups(vpt) > TOPKV_RS_SLOTS) {
      if (layers > 1 && workgroups(kLiveVpt) > INT32_MAX) return TOPKV_OK;   // the caller moves one layer per launch
      int cus = 0;
      const topkv_status_t st = cu_count(&cus);
      if (st != TOPKV_OK) return st;
      // Tokens that can move: those of the tables, of the packed bytes, and of
      // the destination pool, whose pages are named once.
      int64_t tokens = (int64_t)num_reqs * max_tok;
      if (dir != kPools && packed_cap / (geo->planes * (gpt / shards) * gran) < tokens)
        tokens = packed_cap / (geo->planes * (gpt / shards) * gran);
      if (dir != kPack && dst->pool.num_pages * (int64_t)dst->pool.page_size < tokens)
        tokens = dst->pool.num_pages * (int64_t)dst->pool.page_size;
      auto tiles = [&](int v) {
        const int64_t t = ((tokens / unit + num_reqs) * cpu / (v * kThreads) + num_reqs) * geo->planes * layers;
        return t < workgroups(v) ? t : workgroups(v);
      };
      const int64_t most = live_most(layers, cus, dir == kPools, wave);
      vpt = dir == kPools && wave && tiles(kLiveVpt) > most ? 2 * kLiveVpt : kLiveVpt;
      // tiles past `most`: the workgroups go on to further ones, between pools in one round of them
      grid = dim3((unsigned)(tiles(vpt) <= most ? tiles(vpt) : dir == kPools ? 24 * (int64_t)cus : most));
      lds = sizeof(uint64_t) * kWaves + sizeof(int32_t) * (3 * (size_t)num_reqs + 1);
      uint32_t count = (uint32_t)layers;
      void* args[] = {&p.src.tables, &p.dst.tables, &seq_lens, &count, &p};
      const void* f = reinterpret_cast<const void*>(live_kernel_for(dir, wave, heads, vpt));
      const hipError_t e = launch.start || launch.stop
                               ? hipExtLaunchKernel(f, grid, threads, args, lds, launch.stream, launch.start, launch.stop, 0)
                               : hipLaunchKernel(f, grid, threads, args, lds, launch.stream);
      if (e != hipSuccess) return TOPKV_ERR_LAUNCH;
      *launched = true;
      return TOPKV_OK;
    }
    const int64_t tiles = (span + vpt * kThreads - 1) / (vpt * kThreads);
    grid = dim3((unsigned)tiles, (unsigned)geo->planes, (unsigned)(num_reqs * layers));
    if (window > 0) grid = dim3(grid.z, grid.y, grid.x);      // at most TOPKV_RS_SLOTS tiles: no host length here
    const DirectFn direct_fn = direct_kernel_for(dir, wave, heads, host_len, vpt);
    const uint32_t shifts = p.cpu.s | p.src.upp.s << 8 | p.dst.upp.s << 16 | p.reqs.s << 24 | (window > 0 ? kWindowedBit : 0u);
    const int32_t* tables[2] = {p.src.tables, p.dst.tables};
    uint32_t strides[2] = {(uint32_t)p.src.bt_stride, (uint32_t)p.dst.bt_stride}, requests = (uint32_t)num_reqs;
    void* args[] = {&tables[0], &tables[1], &seq_lens, const_cast<uint32_t*>(&shifts), &p.cpu.m, &p.src.upp.m, &p.dst.upp.m,
                    &strides[0], &strides[1], &requests, &p.reqs.m, &p};
    const void* f = reinterpret_cast<const void*>(direct_fn);
    const hipError_t e = launch.start || launch.stop
                             ? hipExtLaunchKernel(f, grid, threads, args, 0, launch.stream, launch.start, launch.stop, 0)
                             : hipLaunchKernel(f, grid, threads, args, 0, launch.stream);
    if (e != hipSuccess) return TOPKV_ERR_LAUNCH;
    *launched = true;
    return TOPKV_OK;
  } else {
    int cus = 0;
    const topkv_status_t st = cu_count(&cus);
    if (st != TOPKV_OK) return st;
    const int64_t tile = (int64_t)kThreads * kVpt;
    int64_t blocks = (bound + tile - 1) / tile;
    if (blocks > (int64_t)cus * kWgPerCu) blocks = (int64_t)cus * kWgPerCu;
    grid = dim3((unsigned)(blocks < 1 ? 1 : blocks));
    lds = sizeof(int32_t) * (kWaves + 3 * (size_t)num_reqs + 1);
    fn = kernel_for(vb, (gpt * vpg) % 64 == 0);
  }
  if (launch.start || launch.stop)
    hipExtLaunchKernelGGL(fn, grid, threads, lds, launch.stream, launch.start, launch.stop, 0, p, seq_lens);
  else
    hipLaunchKernelGGL(fn, grid, threads, lds, launch.stream, p, seq_lens);
  if (hipGetLastError() != hipSuccess) return TOPKV_ERR_LAUNCH;
  *launched = true;
  return TOPKV_OK;
}

topkv_status_t move_layer(const topkv_view_t* src, const topkv_view_t* dst, int32_t num_reqs,
                          const int32_t* seq_lens, int32_t head_count, int32_t window, hipStream_t stream) {
  topkv_launch_t launch = {stream, nullptr, nullptr};
  bool launched = false;
  return move_layer_impl(src, dst, num_reqs, seq_lens, head_count, window, launch, false, &launched);
}

// Layers [view.layer, view.layer + num_layers) of each pool side (a packed
// side's layer z at data + z * packed_layer_stride), in grids of
// topkv_engine_layers_per_grid layers (the bytes a layer moves: the packed
// side's regions, or for pool to pool the source tables' capacity); a move
// that neither a direct nor a live grid takes runs one launch per layer.
topkv_status_t move_layers(const topkv_view_t* src, const topkv_view_t* dst, int32_t num_layers,
                           int64_t packed_layer_stride, int32_t num_reqs, const int32_t* seq_lens,
                           int32_t head_count, int32_t window, hipStream_t stream) {
  if (!src || !dst || num_layers < 0 || packed_layer_stride < 0 || head_count <= 0) return TOPKV_ERR_INVALID_ARG;
  if (!valid_layout(src->layout) || !valid_layout(dst->layout)) return TOPKV_ERR_INVALID_ARG;
  const topkv_view_t* sides[2] = {src, dst};
  int64_t layer_bytes = 0;   // bytes one layer moves, at most (sizes the grids only)
  for (int i = 0; i < 2; ++i) {
    const topkv_view_t* v = sides[i];
    if (v->layout == TOPKV_LAYOUT_PACKED) {
      const int64_t regions = v->shards > 1 ? v->shards : 1;
      int64_t span;
      if (v->bytes < 0 || v->shards < 0 || __builtin_mul_overflow(regions, v->bytes, &span))
        return TOPKV_ERR_INVALID_ARG;
      if (num_layers > 1 && packed_layer_stride < span) return TOPKV_ERR_INVALID_ARG;   // layers would overlap
      layer_bytes = span;
      continue;
    }
    if (v->layer < 0 || num_layers > v->pool.num_layers - v->layer) return TOPKV_ERR_INVALID_ARG;
  }
  int64_t last;   // the last layer's offset on a packed side
  if (num_layers > 1 && __builtin_mul_overflow((int64_t)(num_layers - 1), packed_layer_stride, &last))
    return TOPKV_ERR_INVALID_ARG;
  if (num_layers == 0 || num_reqs == 0) return TOPKV_OK;
  if (layer_bytes == 0) {   // pool to pool: the source tables' capacity in tokens, every moved head
    const topkv_pool_t& g = src->pool;
    const int64_t factors[] = {src->bt_stride, g.page_size, g.planes, head_count, g.head_dim, g.elem_bytes};
    layer_bytes = num_reqs;
    for (const int64_t f : factors)
      if (f < 0 || __builtin_mul_overflow(layer_bytes, f, &layer_bytes)) {
        layer_bytes = INT64_MAX;   // only sizes the grids; the move itself validates the pool
        break;
      }
  }
  const int32_t per = topkv_engine_layers_per_grid(num_layers, layer_bytes, nullptr);
  if (per < 1) return TOPKV_ERR_INVALID_ARG;
  topkv_launch_t launch = {stream, nullptr, nullptr};
  for (int32_t j = 0; j < num_layers; j += per) {
    const int32_t n = num_layers - j < per ? num_layers - j : per;
    topkv_view_t s = *src, d = *dst;
    topkv_view_t* moved[2] = {&s, &d};
    for (topkv_view_t* v : moved) {
      if (v->layout == TOPKV_LAYOUT_PACKED)
        v->data = v->data ? static_cast<char*>(v->data) + (int64_t)j * packed_layer_stride : nullptr;
      else
        v->layer += j;
    }
    bool launched = false;
    topkv_status_t st = n > 1 ? move_layer_impl(&s, &d, num_reqs, seq_lens, head_count, window, launch, false,
                                                &launched, -1, n, packed_layer_stride)
                              : TOPKV_OK;
    if (st != TOPKV_OK) return st;
    if (launched) continue;
    // one launch per layer (one layer in this group, or a move that only the general grid takes)
    for (int32_t l = 0; l < n; ++l) {
      topkv_view_t s1 = s, d1 = d;
      topkv_view_t* one[2] = {&s1, &d1};
      for (topkv_view_t* v : one) {
        if (v->layout == TOPKV_LAYOUT_PACKED)
          v->data = v->data ? static_cast<char*>(v->data) + (int64_t)l * packed_layer_stride : nullptr;
        else
          v->layer += l;
      }
      st = move_layer_impl(&s1, &d1, num_reqs, seq_lens, head_count, window, launch, false, &launched);
      if (st != TOPKV_OK) return st;
    }
  }
  return TOPKV_OK;
}

topkv_view_t pool_view(int32_t layout, const topkv_pool_t* pool, int32_t layer, const int32_t* tables,
                       int32_t bt_stride, int32_t head_begin) {
  topkv_view_t v = {};
  v.layout = layout;
  v.layer = layer;
  v.head_begin = head_begin;
  v.bt_stride = bt_stride;
  v.block_tables = tables;
  v.pool = *pool;
  return v;
}

topkv_view_t packed_view(const void* data, int64_t bytes, int32_t shards = 1) {
  topkv_view_t v = {};
  v.layout = TOPKV_LAYOUT_PACKED;
  v.data = const_cast<void*>(data);
  v.bytes = bytes;
  v.shards = shards;
  return v;
}

}  // namespace topkv_reshard

using namespace topkv_reshard;

namespace topkv_internal {

topkv_status_t chunk_move(bool pack, const topkv_pool_t* pool, int32_t layer, int32_t layers, void* packed,
                          int64_t layer_cap, int64_t total_cap, int64_t layer_stride, int32_t num_reqs,
                          const int32_t* tables, int32_t bt_stride, const int32_t* seq_lens, int32_t seq_len,
                          int32_t window, const topkv_launch_t* launch, bool* launched) {
  *launched = false;
  const topkv_view_t pv = pool_view(TOPKV_LAYOUT_POOL, pool, layer, tables, bt_stride, 0);
  const topkv_view_t kv = packed_view(packed, layer_cap, 1);
  const topkv_status_t st =
      move_layer_impl(pack ? &pv : &kv, pack ? &kv : &pv, num_reqs, seq_lens, pool->num_heads, window, *launch, true,
                      launched, seq_lens ? -1 : seq_len, layers, layer_stride, total_cap, true);
  // anything this path does not take (limits, shapes) goes back to the caller's kernel
  if (st == TOPKV_ERR_INVALID_ARG || st == TOPKV_ERR_UNSUPPORTED || st == TOPKV_ERR_BOUNDS) {
    *launched = false;
    return TOPKV_OK;
  }
  return st;
}

}  // namespace topkv_internal

extern "C" {

topkv_status_t topkv_move_layer(const topkv_view_t* src, const topkv_view_t* dst, int32_t num_reqs,
                                const int32_t* seq_lens, int32_t head_count, int32_t window,
                                hipStream_t stream) {
  return move_layer(src, dst, num_reqs, seq_lens, head_count, window, stream);
}

topkv_status_t topkv_move_layers(const topkv_view_t* src, const topkv_view_t* dst, int32_t num_layers,
                                 int64_t packed_layer_stride, int32_t num_reqs, const int32_t* seq_lens,
                                 int32_t head_count, int32_t window, hipStream_t stream) {
  return move_layers(src, dst, num_layers, packed_layer_stride, num_reqs, seq_lens, head_count, window, stream);
}

topkv_status_t topkv_pack_layer_heads(const topkv_pool_t* src, int32_t layer, int32_t num_reqs,
                                      const int32_t* block_tables, int32_t bt_stride, const int32_t* seq_lens,
                                      int32_t head_begin, int32_t head_count, void* dst, int64_t dst_bytes,
                                      hipStream_t stream) {
  if (!src) return TOPKV_ERR_INVALID_ARG;
  const topkv_view_t s = pool_view(TOPKV_LAYOUT_POOL, src, layer, block_tables, bt_stride, head_begin);
  const topkv_view_t d = packed_view(dst, dst_bytes);
  return move_layer(&s, &d, num_reqs, seq_lens, head_count, 0, stream);
}

topkv_status_t topkv_unpack_layer_heads(const void* src, int64_t src_bytes, const topkv_pool_t* dst,
                                        int32_t layer, int32_t num_reqs, const int32_t* block_tables,
                                        int32_t bt_stride, const int32_t* seq_lens, int32_t head_begin,
                                        int32_t head_count, hipStream_t stream) {
  if (!dst) return TOPKV_ERR_INVALID_ARG;
  const topkv_view_t s = packed_view(src, src_bytes);
  const topkv_view_t d = pool_view(TOPKV_LAYOUT_POOL, dst, layer, block_tables, bt_stride, head_begin);
  return move_layer(&s, &d, num_reqs, seq_lens, head_count, 0, stream);
}

topkv_status_t topkv_pack_layer_shards(const topkv_pool_t* src, int32_t layer, int32_t num_reqs,
                                      const int32_t* block_tables, int32_t bt_stride, const int32_t* seq_lens,
                                      int32_t head_begin, int32_t head_count, int32_t shards, void* dst,
                                      int64_t shard_bytes, hipStream_t stream) {
  if (!src || shards < 1) return TOPKV_ERR_INVALID_ARG;
  const topkv_view_t s = pool_view(TOPKV_LAYOUT_POOL, src, layer, block_tables, bt_stride, head_begin);
  const topkv_view_t d = packed_view(dst, shard_bytes, shards);
  return move_layer(&s, &d, num_reqs, seq_lens, head_count, 0, stream);
}

topkv_status_t topkv_unpack_layer_shards(const void* src, int64_t shard_bytes, int32_t shards,
                                        const topkv_pool_t* dst, int32_t layer, int32_t num_reqs,
                                        const int32_t* block_tables, int32_t bt_stride, const int32_t* seq_lens,
                                        int32_t head_begin, int32_t head_count, hipStream_t stream) {
  if (!dst || shards < 1) return TOPKV_ERR_INVALID_ARG;
  const topkv_view_t s = packed_view(src, shard_bytes, shards);
  const topkv_view_t d = pool_view(TOPKV_LAYOUT_POOL, dst, layer, block_tables, bt_stride, head_begin);
  return move_layer(&s, &d, num_reqs, seq_lens, head_count, 0, stream);
}

topkv_status_t topkv_reblock_layer(const topkv_pool_t* src, int32_t src_layer, const int32_t* src_tables,
                                   int32_t src_stride, const topkv_pool_t* dst, int32_t dst_layer,
                                   const int32_t* dst_tables, int32_t dst_stride, int32_t num_reqs,
                                   const int32_t* seq_lens, hipStream_t stream) {
  if (!src || !dst) return TOPKV_ERR_INVALID_ARG;
  if (src->num_heads != dst->num_heads) return TOPKV_ERR_INVALID_ARG;
  const topkv_view_t s = pool_view(TOPKV_LAYOUT_POOL, src, src_layer, src_tables, src_stride, 0);
  const topkv_view_t d = pool_view(TOPKV_LAYOUT_POOL, dst, dst_layer, dst_tables, dst_stride, 0);
  return move_layer(&s, &d, num_reqs, seq_lens, src->num_heads, 0, stream);
}

}  // extern "C"
