// kc_internal.h -- shared definitions of the gfx950 kernels and the ABI layer.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstdio>
#include <vector>

#include "kc.h"

namespace kc {

constexpr uint32_t kPage = 4096;
constexpr uint32_t kWave = 64;
constexpr uint32_t kTilePages = 16;     // most pages, or units, of a tile
constexpr uint32_t kFences = 256;       // range-table entries in LDS: hashing pass, region diff
constexpr uint32_t kWideFences = 4096;  // the same: closure scan, pointer graph, list of out-of-range words
constexpr uint32_t kBuckets = 1024;     // entries of the LDS bucket index over the ranges

// 16-byte global accesses.  Data that streams through once (pages, packed
// snapshot, compared buffers) uses non-temporal loads and stores, which on
// gfx950 measured 7.2 TB/s for a read-only stream against 6.35 TB/s for
// plain loads.
//
// The addresses are typed as global memory (address space 1).  A plain
// pointer made from an integer compiles to a flat access, which counts on the
// LDS counter as well, so the first LDS wait after it (the hash reads its
// stage from LDS while the next chunk is in flight) would wait for the
// global loads too.
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
#define KC_GLOBAL __attribute__((address_space(1)))
__device__ __forceinline__ uint4 ld16(uint64_t addr) {
  const v4u v = *(const KC_GLOBAL v4u*)addr;
  return make_uint4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void st16(uint64_t addr, uint4 v) {
  const v4u x = {v.x, v.y, v.z, v.w};
  *(KC_GLOBAL v4u*)addr = x;
}
__device__ __forceinline__ uint4 ld16nt(uint64_t addr) {
  const v4u v = __builtin_nontemporal_load((const KC_GLOBAL v4u*)addr);
  return make_uint4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void st16nt(uint64_t addr, uint4 v) {
  const v4u x = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(x, (KC_GLOBAL v4u*)addr);
}
// An 8-byte global load through a plain pointer, kept a global access.
__device__ __forceinline__ uint64_t ld8g(const uint64_t* p) { return *(const KC_GLOBAL uint64_t*)p; }

// Hash units: a range is cut into units of 2^ushift bytes (4 KiB pages by
// default, up to 2 MiB for whole-allocation capture of large tensors); the
// hash table, bitmaps and packed slots count units.  The closure scan and the
// pointer graph always walk 4 KiB page tiles.
constexpr uint32_t kMinUnitShift = 12, kMaxUnitShift = 21;

// A tile: up to 16 consecutive units of one range.  Only a range's last unit
// can be partial (a range size that is not a multiple of the unit); last_len
// is the byte count of the tile's last unit.
struct Tile {
  uint64_t va;              // VA of the first unit
  uint32_t g;               // global index of the first unit
  uint32_t npages : 8;      // 1..16 units
  uint32_t last_len : 24;   // 1..unit bytes
};
static_assert(sizeof(Tile) == 16, "tile layout");

// Bytes of unit j of a tile of units of `unit` bytes.
__device__ __forceinline__ uint32_t unit_bytes(const Tile& t, uint32_t j, uint32_t unit) {
  return j + 1u == t.npages ? (uint32_t)t.last_len : unit;
}

// The 16 bytes at offset off of a page of len bytes, bytes at or past len
// cleared.
__device__ __forceinline__ uint4 clip16(uint4 v, uint32_t off, uint32_t len) {
  if (off + 16u <= len) return v;
  if (off >= len) return make_uint4(0, 0, 0, 0);
  const uint32_t keep = len - off;  // 1..15 bytes
  const auto cut = [&](uint32_t w, uint32_t i) -> uint32_t {
    const uint32_t lo = i * 4u;
    if (keep >= lo + 4u) return w;
    if (keep <= lo) return 0u;
    return w & ((1u << (8u * (keep - lo))) - 1u);
  };
  return make_uint4(cut(v.x, 0), cut(v.y, 1), cut(v.z, 2), cut(v.w, 3));
}

// The two 8-byte words of the 16 bytes at offset off of a page of len bytes,
// each cleared unless it lies wholly inside the page (a cleared word is never
// pointer-like: windows start at 1 or above).
__device__ __forceinline__ uint4 words_inside(uint4 v, uint32_t off, uint32_t len) {
  if (off + 16u <= len) return v;
  if (off + 8u <= len) return make_uint4(v.x, v.y, 0u, 0u);
  return make_uint4(0, 0, 0, 0);
}

// 16 bytes at tile segment s (1 KiB each, four per page) for this lane, with
// the words that are not wholly inside the range cleared.
__device__ __forceinline__ uint4 seg_words(const Tile& t, uint32_t s, uint32_t lane, uint4 v) {
  const uint32_t pg = s >> 2, off = (s & 3u) * 1024u + lane * 16u;
  return pg + 1u == t.npages ? words_inside(v, off, t.last_len) : v;
}

// Store only the first n (0..16) bytes of v at addr.
__device__ __forceinline__ void st_bytes(uint64_t addr, uint4 v, uint32_t n) {
  if (n >= 16u) {
    st16nt(addr, v);
    return;
  }
#pragma unroll
  for (uint32_t i = 0; i < 16u; ++i) {
    if (i < n) {
      const uint32_t w = i < 4u ? v.x : (i < 8u ? v.y : (i < 12u ? v.z : v.w));
      *(KC_GLOBAL uint8_t*)(addr + i) = (uint8_t)(w >> (8u * (i & 3u)));
    }
  }
}

// Sorted range table on the device (bases and one-past-end addresses), with
// a bucket index over [lo, lo + span) = [lowest base, highest end): bucket b
// covers addresses lo + [b << shift, (b + 1) << shift) and holds the last
// fence whose base is at or below the bucket's first address.
struct RangeTable {
  const uint64_t* base;
  const uint64_t* end;
  const uint16_t* bucket;  // kBuckets entries
  uint64_t lo, span;
  uint32_t n;
  uint32_t stride;   // LDS fence stride: fence i = range i * stride
  uint32_t n_fence;  // ceil(n / stride) <= kFences
  uint32_t shift;
  // The wide table (up to kWideFences fences, in dynamic LDS shared by the
  // waves of a workgroup): its stride, fence count and bucket index.
  const uint16_t* bucket_w;
  uint32_t stride_w, n_fence_w;
};

// The closure-scan totals are accumulated in kScanSlots slot pairs, each on
// its own 256-byte line: every wave adds its counts once at its end, and
// waves that finish together would otherwise queue on one address.
constexpr uint32_t kScanSlots = 64;
constexpr uint32_t kScanSlotStride = 32;  // u64 words between slots
constexpr uint32_t kScanCountWords = kScanSlots * kScanSlotStride;

struct ScanDev {
  uint64_t lo, span;                 // pointer-like iff (w - lo) < span
  RangeTable rt;
  uint32_t* tile_oob;                // per-tile out-of-range count
  unsigned long long* counts;        // slot s: [s * kScanSlotStride] n_ptr_like, [+1] n_in_range (accumulated)
};

struct HashParams {
  const Tile* tiles;
  uint32_t n_tiles;
  uint32_t tile0;          // index of tiles[0] in the rangeset's tile list
  uint32_t sub_shift;      // 1 << sub_shift parts per tile, each a wave's work
  const uint32_t* scan0;   // per tile: the scan tile of its first byte (null: 4 KiB units, the tile itself)
  uint64_t seed;
  const uint64_t* prior;   // nullable
  uint64_t* hash;
  uint64_t* zero_bm;       // output, or input when gathering
  uint64_t* changed_bm;
  const uint64_t* word_prefix;  // keep prefix per bitmap word (gathering; null: counted by each wave, with n_kept)
  uint64_t n_units;
  uint64_t* n_kept;
  uint8_t* packed;
  uint64_t* page_va;
  uint64_t cap_pages;
  uint32_t ushift;         // log2 of the hash unit (12: 4 KiB pages)
  ScanDev scan;
};

struct ProbeParams {
  const Tile* tiles;
  uint32_t n_tiles;
  const uint32_t* word_tile;  // tile of each bitmap word's first unit
  uint64_t n_units;
  uint64_t* zero_bm;
  uint64_t *clear_a, *clear_b;  // arrays to clear on the side
  uint64_t n_clear_a, n_clear_b;
  uint32_t ushift;
  uint32_t gshift;  // log2 of the units per group (6 or 4; set by the launcher, as n_groups)
  uint64_t n_groups;
};

// Up to this many bitmap words, the waves of a gathering hash pass count the kept units before theirs themselves.
// 64 MiB: the pass takes 1.3 us more, the launch that is saved took 4.2 and a gap; each wave loads all words at once.
constexpr uint64_t kInlineWords = 512;
// Up to this many tiles, the blocks that list out-of-range words count those before theirs themselves.
// 8 GiB: 9.8 us; with a prefix per tile 9.0, and three launches of 4.6 us to make it.  Every block with entries reads
// all the counts before its run, so beyond 12 GiB the three launches do it.
constexpr uint32_t kInlineTiles = 3u << 16;

// Exclusive-scan sources.
enum ScanSrcKind : uint32_t { kSrcKeepBits = 0, kSrcCounts = 1 };
struct ScanSrc {
  uint32_t kind;
  const uint64_t* zero_bm;     // keep bits: ~zero (& changed)
  const uint64_t* changed_bm;  // nullable
  uint64_t n_pages;
  const uint32_t* counts;      // per-item counts
  uint64_t n_items;            // words or counts
};

struct CmpPairDev {
  const uint8_t* cand;
  const uint8_t* gold;
  uint64_t n_elems;
  uint32_t dtype, tol;
  uint32_t n_tiles, esize;
  double atol, rtol;
};
static_assert(sizeof(CmpPairDev) == 56, "pair layout");

struct CmpTileDev {
  uint32_t pair, idx;
};

// Pairs carried in the kernel arguments of one compare launch (the variant
// that allocates nothing): pair records and the inclusive prefix of their
// tile counts, under the 4 KiB kernel-argument limit.
constexpr uint32_t kArgPairs = 48;
struct CmpArgPairs {
  CmpPairDev pair[kArgPairs];
  uint32_t tile_end[kArgPairs];
  uint32_t n;        // pairs in this launch
  uint32_t n_tiles;  // = tile_end[n - 1]
};
static_assert(sizeof(CmpArgPairs) <= 3072, "kernel arguments");

// Built-in grid of the compare, in workgroups per CU: twice what is resident
// (four), so that CUs whose workgroups met few differing elements take another
// one.  Each workgroup reads one run of consecutive tiles.  With less than 1 MiB of
// tiles per CU, half as many: the end of a run, and the adds of all workgroups at
// one pair's accumulators, weigh more (4 / 8 per CU, 11.3 % off: 1000 pairs of 128
// KiB 76 / 100 us, 5 pairs of 167 MiB in all 119 / 135; 417 pairs of 548 MiB 301 /
// 293).
constexpr uint32_t kCompareGridPerCu = 8;
constexpr uint64_t kCompareFewBytes = 1u << 20;
// Larger compares take runs of a fixed length instead, which the hardware hands out
// in order as workgroups end: a run whose elements all differ costs its workgroup
// many times an equal one (0.2, 0.4 and 0.8 ms per MiB of f32, bf16 and fp8), and
// with even runs of 4 to 15 MiB one wrong output among many right ones was the
// work of a few workgroups while the chip waited (10,000 uneven pairs, the last of
// 10 MiB all off, f32 / bf16 / fp8: 3.30 / 4.37 / 6.75 ms, so 2.51 / 2.53 / 2.57, all
// equal 2.49; 200 pairs of 150 MiB, the last all off as fp8: 17.1 ms, so 9.2, all
// equal 8.8).  Shorter runs cost nothing while pairs are many (those 10,000 of 8 GiB
// a side, runs of 4 / 1 / 0.5 / 0.25 MiB: equal 2.58 / 2.57 / 2.55 / 2.54 ms, 11.3 %
// off 2.79 / 2.66 / 2.63 / 2.61), but with one copy of the accumulators (kAccCopies)
// about 0.1 us each there when elements differ (one pair of 1 GiB, 1e-4 off, runs of
// 0.5 / 0.25 / 0.13 MiB: 350 / 413 / 781 us; 200 pairs of 150 MiB, runs of 1.8 / 0.9 /
// 0.5 MiB: 9.33 / 9.37 / 9.49 ms).
constexpr uint64_t kCompareRunBytes = 512u << 10;      // 1 MiB beyond kCompareLongBytes
constexpr uint64_t kCompareLongBytes = 16ull << 30;    // of a side
// Of lists of at least kTaperPairs pairs the end is cut finer: after the whole runs
// kTaperRuns of half a run, as many of a quarter, and so on to one tile, so that
// what differs at the very end is shared out as well.  With fewer pairs those runs
// would meet at one pair's accumulators.
constexpr uint32_t kTaperShift = 9, kTaperRuns = 1u << kTaperShift, kTaperPairs = 16;

// The tiles of each workgroup of a compare: the first `whole` take `run` tiles (a
// power of two) each, the others shrinking runs; run 0: all tiles shared out evenly.
struct CmpWalk {
  uint32_t grid, run, whole;
  uint32_t copies = 1;  // of each pair's accumulators (kAccCopies or one); workgroup b adds to copy b mod copies
};

// Tile of a small compare: when the pairs are no more than the CUs and none is
// larger than this, each gets a workgroup of 1024 threads, which reads it in one
// round (64 KiB a side) and writes its report itself.  16 pairs of 64 KiB: 8.0 us
// a call, 10.5 in four 16 KiB tiles each and a second kernel.  Where all elements
// of such pairs differ one CU has the work of four: as f32 17.7 us, as fp8 47.8,
// where a tile of 16 KiB per workgroup and a second kernel took 16.4 and 32.7.
constexpr uint32_t kCompareWideTile = 64u << 10;

// Large lists of few pairs keep kAccCopies copies of each pair's accumulators, one
// per XCD (workgroups go to the XCDs in turn), which the reports combine: adds from
// all XCDs to one copy cost about 0.1 us each and keep the loads of others waiting.
// bf16 with 1e-4 off, runs as above, one copy / eight: one pair of 8 GiB 2.91 / 2.64
// ms (runs of 4 MiB, one copy, 2.61), four of 4 GiB 5.72 / 5.13 (5.19), 40 of 4 GiB in
// all, one of them 2.5, 1.39 / 1.27 (1.36); the same when all is equal.  Not below the
// lengths where runs are short, where a run ends with a few thousand adds in all; nor
// with more pairs, which meet less and would have the reports read 4 KiB each.
constexpr uint32_t kAccCopies = 8;
constexpr uint32_t kAccCopyPairs = 512;
constexpr uint64_t kAccCopyBytes = 1ull << 30;  // of a side

constexpr uint32_t kAccWords = 64;  // per-pair accumulator words
// accumulator word map
enum : uint32_t {
  kAccMisElems = 0, kAccMisBytes, kAccNanBoth, kAccNanCand, kAccNanGold, kAccOverTol,
  kAccMaxAbs, kAccMaxRel, kAccFirstInv, kAccNotClose, kAccHist = 16  // 48 bins: words 16..63
};

// ---- launchers (in the files of their kernels) ---------------------------
hipError_t launch_fill_u64(uint64_t* p, uint64_t n, uint64_t v, hipStream_t s);
hipError_t launch_zero4(uint64_t* a, uint64_t na, uint64_t* b, uint64_t nb, uint64_t* c, uint64_t nc, uint64_t* d,
                        uint64_t nd, hipStream_t s);
// The hashing pass (kc_hash.hip); rows: most units per wave (16, 8 or 4); grid: waves (0: one per part of a tile).
hipError_t launch_page_hash(HashParams p, bool gather, bool prior, bool scan, uint32_t rows, uint32_t grid,
                            uint32_t n_cu, hipStream_t s);
hipError_t launch_probe_zero(ProbeParams p, uint64_t n_words, uint32_t n_cu, hipStream_t s);
hipError_t launch_scan(const ScanSrc& src, uint64_t* out, uint64_t* block_sums,
                       uint64_t* total_out, hipStream_t s);
// grid: waves (0: one per part of a tile)
hipError_t launch_gather(const Tile* tiles, uint32_t n_tiles, uint32_t per_tile, const uint64_t* zero_bm,
                         const uint64_t* changed_bm, const uint64_t* word_prefix,
                         uint8_t* packed, uint64_t* page_va, uint64_t cap_pages, uint32_t ushift,
                         uint32_t grid, hipStream_t s);
hipError_t launch_restore_zero(const Tile* tiles, uint32_t n_tiles, const uint64_t* zero_bm,
                               const uint64_t* changed_bm, unsigned long long* n_bad, uint32_t ushift,
                               uint32_t grid, hipStream_t s);
hipError_t launch_restore_scatter(const RangeTable& rt, const uint8_t* packed,
                                  const uint64_t* page_va, const uint64_t* n_kept,
                                  uint64_t cap_pages, unsigned long long* n_bad,
                                  bool delta, uint32_t ushift, hipStream_t s);
hipError_t launch_closure(const Tile* tiles, uint32_t n_tiles, uint32_t tile0,
                          const ScanDev& sd, uint32_t grid, uint32_t n_cu, hipStream_t s);
hipError_t launch_pointer_graph(const Tile* tiles, uint32_t n_tiles, uint64_t lo, uint64_t span,
                                const RangeTable& rt, uint64_t* edge_bm, uint32_t row_words, uint32_t grid,
                                uint32_t n_cu, hipStream_t s);
hipError_t launch_region_init(kc_region_diff_result* res, uint32_t n, uint64_t* bm_a, uint64_t* bm_b, uint64_t n_words,
                              hipStream_t s);
hipError_t launch_region_diff(const Tile* tiles, uint32_t n_tiles, const RangeTable& rt, const uint64_t* changed_bm,
                              const uint64_t* gold_zero_bm, const uint64_t* rank_prefix, const uint64_t* gold_page_va,
                              const uint64_t* gold_n_kept, uint64_t cap, const uint8_t* gold_packed,
                              kc_region_diff_result* res, uint32_t ushift, uint32_t grid, uint32_t n_cu,
                              hipStream_t s);
hipError_t launch_oob_emit(const Tile* tiles, uint32_t n_tiles, const ScanDev& sd,
                           const uint64_t* tile_prefix, kc_oob* oob, uint64_t cap, kc_scan_result* res,
                           uint64_t n_words, hipStream_t s);
// wide: workgroups of 1024 threads.  direct: every pair is one tile and the pass writes the reports (else the
// finalize does).
hipError_t launch_compare(const CmpPairDev* pairs, const CmpTileDev* tiles, uint32_t n_tiles, uint32_t tile_bytes,
                          unsigned long long* acc, kc_cmp_result* res, CmpWalk walk, bool wide, bool direct,
                          hipStream_t s);
hipError_t launch_compare_finalize(const CmpPairDev* pairs, uint32_t n_pairs, unsigned long long* acc, uint32_t copies,
                                   kc_cmp_result* res, hipStream_t s);
// The pass and the reports of the pairs in `a` (accumulators acc[pair * walk.copies * kAccWords ...], zero on entry
// and zeroed again; reports res[0 .. a.n)).
hipError_t launch_compare_args(const CmpArgPairs& a, uint32_t tile_bytes, unsigned long long* acc,
                               kc_cmp_result* res, CmpWalk walk, bool wide, hipStream_t s);

// ---- shared host helpers (kc_api.hip) ----------------------------------------
uint32_t grid_for(const kc_ctx* c, uint32_t op, uint32_t fallback_per_cu);  // persistent grid of an op
uint32_t elem_size(uint32_t dtype);                                         // bytes of one element
uint32_t compare_tile_bytes(const kc_ctx* c, const kc_pair* pairs, uint32_t n_pairs);
bool compare_wide(const kc_ctx* c, uint64_t n_pairs, uint64_t n_tiles, uint32_t tile_bytes);  // 1024-thread workgroups
CmpWalk compare_walk(const kc_ctx* c, uint64_t n_pairs, uint64_t n_tiles, uint32_t tile_bytes, uint32_t copies);
// Copies of each pair's accumulators, for a list of `bytes` a side in whole tiles.
inline uint32_t acc_copies(uint64_t n_pairs, uint64_t bytes) {
  return n_pairs <= kAccCopyPairs && bytes > kAccCopyBytes ? kAccCopies : 1u;
}

// ---- the compare that allocates nothing (kc_noalloc.hip) ---------------------
// Looks up, once per device, the device address of the static scratch array
// (the device must be current); KC_EHIP if the lookup fails.
int noalloc_bind(int device);

// ---- errors and device selection (kc_api.hip) ------------------------------
void set_error_text(const char* text);
void set_error(const char* what, hipError_t e);

#define KC_HIP(call)                          \
  do {                                        \
    hipError_t kc_e_ = (call);                \
    if (kc_e_ != hipSuccess) {                \
      ::kc::set_error(#call, kc_e_);          \
      return KC_EHIP;                         \
    }                                         \
  } while (0)

// Makes `dev` current for the scope of a call and restores the caller's device.
struct DeviceGuard {
  int prev = -1;
  bool ok = true;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) prev = -1;
    if (prev != dev) ok = hipSetDevice(dev) == hipSuccess;
    if (!ok) {
      (void)hipGetLastError();  // do not leave the failure for the caller's next HIP call
      char msg[64];
      std::snprintf(msg, sizeof(msg), "hipSetDevice(%d) failed", dev);
      set_error_text(msg);
    }
  }
  ~DeviceGuard() {
    int cur = -1;
    if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
  }
};

}  // namespace kc

// ---- library objects --------------------------------------------------------
struct kc_ctx {
  int device = 0;
  uint32_t n_cu = 256;
  kc_tuning tune[KC_OP_COUNT];
  uint8_t* cmp_dev = nullptr;  // pairs | tiles
  size_t cmp_dev_cap = 0;
  unsigned long long* cmp_acc = nullptr;  // accumulators: zero between calls (finalize resets them)
  size_t cmp_acc_cap = 0;
  bool cmp_acc_dirty = false;
  uint8_t* cmp_host = nullptr;  // pinned staging of pairs | tiles
  size_t cmp_host_cap = 0;
  hipEvent_t staged = nullptr;  // completion of the last staging copy
  bool staged_pending = false;
  bool timing = false;  // record events around the main kernel of each op
  hipEvent_t t_start[KC_OP_COUNT] = {};
  hipEvent_t t_stop[KC_OP_COUNT] = {};
  bool t_valid[KC_OP_COUNT] = {};
};

struct kc_rangeset {
  kc_ctx* ctx = nullptr;
  int device = 0;  // recorded at creation: destroy never touches the context
  uint32_t n_ranges = 0, n_tiles = 0;
  uint32_t ushift = 12;              // log2 of the hash unit; n_pages, n_words and the tiles count units
  uint64_t n_pages = 0, n_words = 0;
  uint64_t n_scan_words = 0;         // 8-byte words wholly inside the ranges
  std::vector<uint32_t> range_tile;  // first tile of each range (n + 1)
  uint64_t win_lo = 0, win_hi = 0;   // default pointer window
  std::vector<kc_range> host_ranges;
  // 4 KiB page tiles walked by the closure scan, its list emission and the
  // pointer graph (the same list as `tiles` when the unit is the page)
  uint32_t n_scan_tiles = 0;
  std::vector<uint32_t> scan_range_tile;
  kc::Tile* scan_tiles = nullptr;
  uint32_t per_tile = 16;            // most units of a tile in `tiles`
  uint32_t* word_tile = nullptr;     // tile of each bitmap word's first unit (device)
  uint32_t* hash_scan0 = nullptr;    // units above 4 KiB: the scan tile of each tile's first byte (device)
  void* dev = nullptr;
  kc::Tile* tiles = nullptr;
  uint64_t* bases = nullptr;
  uint64_t* ends = nullptr;
  uint32_t* tile_oob = nullptr;
  uint64_t* tile_prefix = nullptr;
  uint64_t* word_prefix = nullptr;
  uint64_t* block_sums = nullptr;
  unsigned long long* counts = nullptr;  // closure-scan slots (kScanCountWords)
  unsigned long long* n_bad = nullptr;   // rejected page VAs of a restore given no counter
  uint64_t* n_oob = nullptr;
  kc::RangeTable rt{};
};

struct kc_pairset {
  kc_ctx* ctx = nullptr;
  int device = 0;  // recorded at creation: destroy never touches the context
  uint32_t n_pairs = 0, tile_bytes = 0;
  uint64_t n_tiles = 0;
  std::vector<uint64_t> tile_off;
  void* dev = nullptr;
  kc::CmpPairDev* pairs = nullptr;
  kc::CmpTileDev* tiles = nullptr;
  unsigned long long* acc = nullptr;
  uint32_t copies = 1;             // of each pair's accumulators
  mutable bool acc_dirty = false;  // a failed compare left accumulators set
};

