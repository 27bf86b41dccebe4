// kc_snapshot.hip -- gfx950 kernels of the snapshot around the hashing pass
// (kc_hash.hip), of the restore and of the closure scan.
//
// Memory-bound streaming kernels over a tile list (up to 16 pages or units of one
// range per tile).  The standalone scan and the restore's zero fill are persistent
// grids of waves that stride over the tiles; the probe, the gather and the
// restore's scatter take one group, part or block per workgroup or wave, in address
// order.  The standalone scan puts several independent waves in a workgroup to
// share one range table, and the out-of-range emission uses one wave per page
// of a tile.  Global traffic is 16-byte loads / stores that cover whole 1-KiB
// runs.
#include <algorithm>

#include "kc_device.h"
#include "kc_internal.h"
#include "kc_xxh64.h"

namespace kc {
namespace {

// --------------------------------------------------------------- fill -----
__global__ void k_fill_u64(uint64_t* p, uint64_t n, uint64_t v) {
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

// Zero up to four arrays in one launch (index space = their concatenation).
__global__ void k_zero4(uint64_t* a, uint64_t na, uint64_t* b, uint64_t nb, uint64_t* c, uint64_t nc, uint64_t* d,
                        uint64_t nd) {
  const uint64_t n = na + nb + nc + nd;
  for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x) {
    if (i < na) a[i] = 0;
    else if (i < na + nb) b[i - na] = 0;
    else if (i < na + nb + nc) c[i - na - nb] = 0;
    else d[i - na - nb - nc] = 0;
  }
}

// ------------------------------------------------------------ zero probe --
// Exact zero bitmap of the units, written whole (nothing to clear first).  A
// workgroup takes a group of 64 or 16 consecutive units: its first wave reads
// the first 16 bytes of each, one lane per unit, and lists the units that begin
// with zeros; the listed units' 4 KiB blocks are then shared out to the waves,
// four blocks (16 KiB in flight) at a time, until a non-zero byte shows in the
// unit or it ends: the first block of every unit, then the second of every unit,
// and so on, so that units that only begin with zeros are left after their first
// (8 GiB in units of 64 KiB that hold a byte in every page: 4.17 ms a snapshot with
// a unit's blocks together, so 3.47).  A unit's tile is found from the tile of its bitmap word's
// first unit: each lane holds one of the 64 tiles from there on, and every lane
// searches them for its unit's.
//
// What bounds it: with most units non-zero, the one line of each unit that is
// read, and a chain of four dependent loads per group, so there are as many
// groups in flight as fit; with many zero units, their bytes.  Measured against
// persistent waves of four tiles each (8 per CU), all the units of a tile run
// through by one wave: 64 MiB with 30 % zero pages 23.5 -> 8.3 us, 1 MiB 5.9
// -> 4.5, 8 GiB in units of 64 KiB 59 -> 50; 30 GiB of pages with 2.7 % zero 400
// -> 373 us (7.8 million lines a page apart and 0.8 GiB of zeros).
//
// It also clears the two arrays that a closure scan accumulates into.
constexpr uint32_t kProbeWaves = 16;

template <bool PAGES>  // units of one block
__global__ __launch_bounds__(kProbeWaves * kWave) void k_probe_zero(ProbeParams p) {
  __shared__ uint64_t unit_va[kWave];
  __shared__ uint32_t unit_len[kWave], unit_at[kWave];  // of the listed units: bytes, place in the group
  __shared__ unsigned long long listed, nonzero;
  const uint32_t lane = threadIdx.x % kWave, wpb = blockDim.x / kWave;
  const uint32_t wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const uint32_t unit = 1u << p.ushift, bshift = p.ushift - 12u, group = 1u << p.gshift;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < p.n_clear_a + p.n_clear_b;
       i += (uint64_t)gridDim.x * blockDim.x) {
    if (i < p.n_clear_a) p.clear_a[i] = 0;
    else p.clear_b[i - p.n_clear_a] = 0;
  }
  for (uint64_t gr = blockIdx.x; gr < p.n_groups; gr += gridDim.x) {
    const uint64_t u0 = gr << p.gshift;
    if (wv == 0) {
      const uint32_t n = u0 < p.n_units ? (uint32_t)min(p.n_units - u0, (uint64_t)group) : 0u;
      const uint32_t t0 = const_load32(p.word_tile + (u0 >> 6)), t = t0 + lane;
      Tile tile{0, 0xFFFFFFFFu, 0, 0};
      if (t < p.n_tiles) tile = p.tiles[t];
      const uint32_t shape = (tile.npages << 24) | tile.last_len;  // npages 16 at most, last_len up to 2 MiB
      const uint32_t u = (uint32_t)u0 + lane;
      uint32_t at = 0;  // the last of the 64 tiles that starts at or before unit u
#pragma unroll
      for (uint32_t d = 32; d >= 1u; d >>= 1) at += (uint32_t)__shfl(tile.g, at + d, 64) <= u ? d : 0u;
      const uint32_t j = u - (uint32_t)__shfl(tile.g, at, 64), sh = __shfl(shape, at, 64);
      const uint64_t va = __shfl((unsigned long long)tile.va, at, 64) + ((uint64_t)j << p.ushift);
      const bool valid = lane < n;
      const uint32_t len = j + 1u == sh >> 24 ? sh & 0xFFFFFFu : unit;  // a partial unit is tested over its bytes only
      const bool zeros = valid && !nz16(clip16(valid ? ld16(va) : make_uint4(0, 0, 0, 0), 0u, len));
      const uint64_t m = __ballot(zeros);
      if (zeros) {
        const uint32_t i = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
        unit_va[i] = va;
        unit_len[i] = len;
        unit_at[i] = lane;
      }
      if (lane == 0) {
        listed = m;
        nonzero = 0;
      }
    }
    __syncthreads();
    const uint32_t n_listed = (uint32_t)__popcll(listed), n_blocks = n_listed << bshift;
    for (uint32_t b0 = wv * 4u; b0 < n_blocks; b0 += wpb * 4u) {
      const uint64_t seen = *(volatile unsigned long long*)&nonzero;  // blocks of units known not to be zero: skipped
      uint4 x[16];
      uint32_t place[4], bytes[4];
      uint32_t nth = PAGES ? 0u : b0 / n_listed, which = b0 - nth * n_listed;  // block b0 is the nth of this listed unit
#pragma unroll
      for (uint32_t i = 0; i < 4; ++i) {
        const uint32_t b = b0 + i, c = min(which, n_listed - 1u), off = nth * kPage;
        if (++which == n_listed && !PAGES) {
          which = 0u;
          ++nth;
        }
        place[i] = unit_at[c];
        const bool skip = b >= n_blocks || ((seen >> place[i]) & 1ull) != 0ull || off >= unit_len[c];
        bytes[i] = skip ? 0u : min(unit_len[c] - off, kPage);
        const __amdgpu_buffer_rsrc_t src = raw_rsrc(unit_va[c] + off, (bytes[i] + 15u) & ~15u);
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
          const v4u v = __builtin_amdgcn_raw_buffer_load_b128(src, j * 1024u + lane * 16u, 0, kNt);
          x[i * 4 + j] = make_uint4(v[0], v[1], v[2], v[3]);
        }
      }
      uint64_t found = 0;
#pragma unroll
      for (uint32_t i = 0; i < 4; ++i) {
        bool nz = false;
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) nz = nz || nz16(clip16(x[i * 4 + j], j * 1024u + lane * 16u, bytes[i]));
        if (__ballot(nz) != 0ull) found |= 1ull << place[i];
      }
      if (found != 0ull && lane == 0) atomicOr(&nonzero, (unsigned long long)found);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      const uint64_t zero = listed & ~nonzero;
      if (p.gshift == 6u) p.zero_bm[gr] = zero;
      else reinterpret_cast<uint16_t*>(p.zero_bm)[gr] = (uint16_t)zero;
    }
    __syncthreads();  // the list is rewritten for the next group
  }
}

// ------------------------------------------------ reduce-then-scan (u64) --
constexpr uint32_t kScanThreads = 256, kScanPerThread = 8;
constexpr uint32_t kScanBlock = kScanThreads * kScanPerThread;

__device__ __forceinline__ uint32_t scan_item(const ScanSrc& s, uint64_t i) {
  if (i >= s.n_items) return 0u;
  if (s.kind == kSrcCounts) return s.counts[i];
  uint64_t keep = ~s.zero_bm[i];
  if (s.changed_bm) keep &= s.changed_bm[i];
  if (i == s.n_items - 1 && (s.n_pages & 63u)) keep &= (1ull << (s.n_pages & 63u)) - 1ull;
  return (uint32_t)__popcll(keep);
}

// Exclusive scan of one value per thread across a 256-thread block.
__device__ __forceinline__ uint64_t block_exclusive(uint64_t x, uint64_t* lds4, uint64_t* total) {
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  uint64_t inc = x;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint64_t y = __shfl_up(inc, d, 64);
    if (lane >= (uint32_t)d) inc += y;
  }
  if (lane == 63) lds4[wave] = inc;
  __syncthreads();
  uint64_t pre = 0, tot = 0;
#pragma unroll
  for (uint32_t w = 0; w < kScanThreads / 64; ++w) {
    if (w < wave) pre += lds4[w];
    tot += lds4[w];
  }
  __syncthreads();
  if (total) *total = tot;
  return pre + inc - x;
}

__global__ __launch_bounds__(256) void k_scan_reduce(ScanSrc src, uint64_t* block_sums) {
  __shared__ uint64_t lds4[4];
  const uint64_t i0 = (uint64_t)blockIdx.x * kScanBlock + threadIdx.x * kScanPerThread;
  uint64_t s = 0;
#pragma unroll
  for (uint32_t i = 0; i < kScanPerThread; ++i) s += scan_item(src, i0 + i);
  uint64_t tot = 0;
  block_exclusive(s, lds4, &tot);
  if (threadIdx.x == 0) block_sums[blockIdx.x] = tot;
}

__global__ __launch_bounds__(1024) void k_scan_top(uint64_t* block_sums, uint32_t nb, uint64_t* total_out) {
  __shared__ uint64_t lds[16];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  uint64_t carry = 0;
  for (uint32_t base = 0; base < nb; base += 1024) {
    const uint32_t i = base + tid;
    const uint64_t x = i < nb ? block_sums[i] : 0ull;
    uint64_t inc = x;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint64_t y = __shfl_up(inc, d, 64);
      if (lane >= (uint32_t)d) inc += y;
    }
    if (lane == 63) lds[wave] = inc;
    __syncthreads();
    uint64_t pre = 0, tot = 0;
    for (uint32_t w = 0; w < 16; ++w) {
      if (w < wave) pre += lds[w];
      tot += lds[w];
    }
    if (i < nb) block_sums[i] = carry + pre + inc - x;
    carry += tot;
    __syncthreads();
  }
  if (tid == 0 && total_out) *total_out = carry;
}

__global__ __launch_bounds__(256) void k_scan_down(ScanSrc src, const uint64_t* block_sums, uint64_t* out) {
  __shared__ uint64_t lds4[4];
  const uint64_t i0 = (uint64_t)blockIdx.x * kScanBlock + threadIdx.x * kScanPerThread;
  uint32_t v[kScanPerThread];
  uint64_t s = 0;
#pragma unroll
  for (uint32_t i = 0; i < kScanPerThread; ++i) {
    v[i] = scan_item(src, i0 + i);
    s += v[i];
  }
  uint64_t run = block_exclusive(s, lds4, nullptr) + block_sums[blockIdx.x];
#pragma unroll
  for (uint32_t i = 0; i < kScanPerThread; ++i) {
    if (i0 + i < src.n_items) out[i0 + i] = run;
    run += v[i];
  }
}

// Whole scan in one block when the items fit in it (small inputs: one launch
// instead of three).
__global__ __launch_bounds__(256) void k_scan_small(ScanSrc src, uint64_t* out, uint64_t* total_out) {
  __shared__ uint64_t lds4[4];
  const uint64_t i0 = (uint64_t)threadIdx.x * kScanPerThread;
  uint32_t v[kScanPerThread];
  uint64_t s = 0;
#pragma unroll
  for (uint32_t i = 0; i < kScanPerThread; ++i) {
    v[i] = scan_item(src, i0 + i);
    s += v[i];
  }
  uint64_t tot = 0;
  uint64_t run = block_exclusive(s, lds4, &tot);
#pragma unroll
  for (uint32_t i = 0; i < kScanPerThread; ++i) {
    if (i0 + i < src.n_items) out[i0 + i] = run;
    run += v[i];
  }
  if (threadIdx.x == 0 && total_out) *total_out = tot;
}

// --------------------------------------------------------------- gather ---
// Kept units copied to their packed slots.  A wave takes a part of a tile, 64 KiB
// (a whole tile of pages) or, of many larger units, 256 KiB: one lane per 4 KiB block
// resolves whether its unit is kept and where its slot is, then the kept blocks
// are copied four at a time, 16 KiB in flight; a partial unit's slot is filled up
// with zeros.  The bytes moved bound it.  One such part per wave, in address
// order (2 GiB in 4096 ranges, 5 % of the pages kept, 43 us, eight persistent
// waves per CU 54; 8 GiB, all kept, 3.29 ms and 3.40; before, with whole tiles,
// 60 us and 3.38 ms, and 2 GiB in units of 2 MiB 1.68 ms, now 0.77).  Beyond
// kGatherLong of larger units, that is more workgroups than a call with little to
// copy is worth: 40 GiB in units of 64 KiB, nothing kept, 151 us, so 47; 1 % kept
// 234 and 170; all kept 15.5 and 15.8 ms.  Below, short parts spread few units better
// (2 GiB in units of 2 MiB, 1 % kept, 23 us, long ones 36).
constexpr uint64_t kGatherLong = 4ull << 30;

__global__ __launch_bounds__(64) void k_gather(const Tile* tiles, uint32_t n_tiles, uint32_t part, uint32_t part_shift,
                                               const uint64_t* zero_bm, const uint64_t* changed_bm,
                                               const uint64_t* word_prefix, uint8_t* packed, uint64_t* page_va,
                                               uint64_t cap, uint32_t ushift) {
  const uint32_t lane = threadIdx.x, unit = 1u << ushift;
  const uint64_t n_items = (uint64_t)n_tiles << part_shift;
  for (uint64_t it = blockIdx.x; it < n_items; it += gridDim.x) {
    const Tile tile = const_load(tiles + (it >> part_shift));
    // this lane's block, of the part's 16 or 64: its unit and place in it
    const uint32_t off = ((uint32_t)it & ((1u << part_shift) - 1u)) * part + lane * kPage;
    const uint32_t j = off >> ushift, inside = off & (unit - 1u);
    bool go = false;
    uint64_t dst = 0;
    if (lane * kPage < part && j < tile.npages) {
      const uint64_t g = (uint64_t)tile.g + j;
      uint64_t kw = ~zero_bm[g >> 6];
      if (changed_bm) kw &= changed_bm[g >> 6];
      const uint64_t slot = word_prefix[g >> 6] + (uint64_t)__popcll(kw & ((1ull << (g & 63u)) - 1ull));
      go = ((kw >> (g & 63u)) & 1ull) != 0ull && slot < cap;
      if (go && inside == 0u) page_va[slot] = tile.va + off;
      dst = (uint64_t)packed + (slot << ushift) + inside;
    }
    const uint32_t bytes = j < tile.npages ? unit_bytes(tile, j, unit) : 0u;
    const uint32_t len = bytes > inside ? min(bytes - inside, kPage) : 0u;  // of the block
    uint64_t mask = __ballot(go);
    while (mask) {
      uint64_t from[4], to[4];
      uint32_t cnt = 0, n[4];
#pragma unroll
      for (uint32_t i = 0; i < 4; ++i) {
        const uint32_t b = mask ? (uint32_t)__builtin_ctzll(mask) : 0u;
        from[i] = tile.va + __shfl(off, b, 64);
        to[i] = __shfl((unsigned long long)dst, b, 64);
        n[i] = __shfl(len, b, 64);
        if (mask) {
          mask &= mask - 1ull;
          ++cnt;
        }
      }
      uint4 x[16];
#pragma unroll
      for (uint32_t i = 0; i < 16; ++i) {
        const uint32_t o = (i & 3u) * 1024u + lane * 16u;
        if (i / 4u < cnt) x[i] = o < n[i / 4u] ? clip16(ld16nt(from[i / 4u] + o), o, n[i / 4u]) : make_uint4(0, 0, 0, 0);
      }
#pragma unroll
      for (uint32_t i = 0; i < 16; ++i)
        if (i / 4u < cnt) st16nt(to[i / 4u] + (i & 3u) * 1024u + lane * 16u, x[i]);
    }
  }
}

// -------------------------------------------------------------- restore ---
__global__ __launch_bounds__(64) void k_restore_zero(const Tile* tiles, uint32_t n_tiles,
                                                     const uint64_t* zero_bm, const uint64_t* changed_bm,
                                                     unsigned long long* n_bad, uint32_t ushift) {
  const uint32_t lane = threadIdx.x, unit = 1u << ushift;
  if (blockIdx.x == 0 && lane == 0) *n_bad = 0ull;  // the scatter that follows counts into it
  for (uint32_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
    const Tile tile = tiles[t];
    bool sel = false;
    if (lane < tile.npages) {
      const uint64_t g = (uint64_t)tile.g + lane;
      uint64_t w = zero_bm[g >> 6];
      if (changed_bm) w &= changed_bm[g >> 6];
      sel = ((w >> (g & 63u)) & 1ull) != 0ull;
    }
    uint32_t mask = (uint32_t)__ballot(sel);
    const uint4 z = make_uint4(0, 0, 0, 0);
    while (mask) {
      const uint32_t pg = (uint32_t)__builtin_ctz(mask);
      mask &= mask - 1u;
      const uint32_t len = unit_bytes(tile, pg, unit);  // never past the range's end
      const uint64_t uva = tile.va + ((uint64_t)pg << ushift);
      for (uint32_t o0 = 0; o0 < len; o0 += kPage) {
#pragma unroll
        for (uint32_t j = 0; j < 4; ++j) {
          const uint32_t o = o0 + j * 1024u + lane * 16u;
          if (o + 16u <= len) st16nt(uva + o, z);
          else if (o < len) st_bytes(uva + o, z, len - o);
        }
      }
    }
  }
}

// Packed units back to their VAs, one 4 KiB block per wave and WAVES waves
// (that many consecutive blocks) per workgroup, the grid covering every block
// of the capacity (no persistent stride).  Block b of the packed snapshot
// belongs to slot b >> (ushift - 12); the wave reads that slot's page-VA entry
// (one scalar load for the whole wave), validates it (4 KiB aligned, inside a
// range, the start of a unit of that range) with a scalar search of the range
// set's arrays, and copies the block with four 16-byte loads and stores per
// lane; of the last block of a range, only the bytes inside it (a second pass
// over the slots for these took 41 of 760 us on 2 GiB in 4096 ranges).
// Workgroups are dispatched in block order, so the waves in flight cover one
// compact, advancing window of both buffers: against a persistent grid
// striding four-block groups over the snapshot (with a range table loaded into
// LDS per workgroup) the one-wave form runs at the speed of a plain copy
// kernel between the same buffers.  Four-wave workgroups copy a full snapshot
// about 5 % slower (a workgroup's slot is freed only when its last wave ends)
// but dispatch a quarter of the workgroups, which is what a delta restore pays
// for when its kept count is far below the capacity the grid covers.
template <uint32_t WAVES>
__global__ __launch_bounds__(WAVES * kWave) void k_restore_scatter(RangeTable rt, const uint8_t* packed,
                                                                   const uint64_t* page_va, const uint64_t* n_kept,
                                                                   uint64_t cap, unsigned long long* n_bad,
                                                                   uint32_t ushift) {
  const uint32_t lane = threadIdx.x % kWave;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);  // so the block index is scalar
  const uint32_t bshift = ushift - 12u;  // 4 KiB blocks per unit: 1 << bshift
  const uint64_t unit = 1ull << ushift;
  const uint64_t nblk = min(*n_kept, cap) << bshift;
  for (uint64_t blk = (uint64_t)blockIdx.x * WAVES + wave; blk < nblk; blk += (uint64_t)gridDim.x * WAVES) {
    const uint64_t sub = blk & ((1ull << bshift) - 1ull);
    const uint64_t va = ((const KC_CONST uint64_t*)page_va)[blk >> bshift];  // one scalar load for the wave
    bool good = false, ok = false;
    if ((va & (kPage - 1)) == 0) {
      const RangeHit r = range_find_uniform(va, rt);
      if (r.a >= 0) {
        good = ((va - r.base) & (unit - 1ull)) == 0ull;
        const uint64_t at = va + (sub << 12);
        ok = good && at + kPage <= r.end;
        if (good && !ok && at < r.end) {  // the last bytes of a range, never past its end
          const uint32_t len = (uint32_t)(r.end - at);
#pragma unroll
          for (uint32_t j = 0; j < 4; ++j) {
            const uint32_t o = j * 1024u + lane * 16u;
            if (o < len) st_bytes(at + o, ld16nt((uint64_t)packed + blk * kPage + o), len - o);
          }
        }
      }
    }
    if (!good && sub == 0 && lane == 0) atomicAdd(n_bad, 1ull);  // counted once per slot
    if (!ok) continue;
    const uint64_t src = (uint64_t)packed + blk * kPage + lane * 16u, dst = va + (sub << 12) + lane * 16u;
    uint4 x[4];
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) x[j] = ld16nt(src + j * 1024u);
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) st16nt(dst + j * 1024u, x[j]);
  }
}

// --------------------------------------------------------- closure scan ---
// Standalone scan.  Workgroups of kWideWaves independent waves share the wide
// range table.
__global__ __launch_bounds__(kWideWaves * kWave) __attribute__((amdgpu_waves_per_eu(4))) void k_closure(
    const Tile* tiles, uint32_t n_tiles, uint32_t tile0, ScanDev sd) {
  __shared__ uint64_t queue[kWideWaves][kPtrQueue];
  const uint32_t lane = threadIdx.x % kWave, wv = threadIdx.x / kWave, wpb = blockDim.x / kWave;
  const uint32_t wave = blockIdx.x * wpb + wv, n_waves = gridDim.x * wpb;
  load_wide_fences(sd.rt, threadIdx.x, blockDim.x);
  __syncthreads();
  uint32_t n_ptr = 0, n_in = 0;  // n_ptr: of the wave; n_in: of this lane
  for (uint32_t t = wave; t < n_tiles; t += n_waves) {
    const Tile tile = tiles[t];
    uint32_t oob = 0;
    n_ptr += each_pointer(tile, sd.lo, sd.span, queue[wv], [&](uint64_t w, uint32_t) {
      if (wide_range_index(w, sd.rt) >= 0) ++n_in; else ++oob;
    });
    const uint32_t o = __ballot(oob != 0u) ? wave_sum_u32(oob) : 0u;
    if (lane == 0) sd.tile_oob[tile0 + t] = o;
  }
  const uint32_t b = wave_sum_u32(n_in);
  if (lane == 0) add_scan_counts(sd.counts, wave, n_ptr, b);
}

// Writes the out-of-range words of each tile at its prefix position, in
// ascending address order, up to the list capacity.  A block owns a run of
// up to 1024 consecutive tiles, one per thread: one parallel read of their counts
// lists the tiles with entries below the capacity, then each listed tile is read
// again with one wave per page (its four 1-KiB segments in
// one round trip, under way while the tile before it is searched), the waves'
// entries placed by a prefix over their counts.  Without a prefix per tile, a
// block with entries sums the counts before its run itself (up to kInlineTiles
// tiles: 768 KiB from the caches at most).  A chain of round trips bounds it,
// so what can be is loaded ahead, a block without entries ends after the first,
// and the range table is the wide one, all of it in LDS up to 4096 ranges.
// 2 GiB in 4096 ranges with 134 entries: 16.2 us, 21.4 before with three
// launches of 4.8 us for the prefix.
constexpr uint32_t kEmitThreads = kTilePages * kWave;  // one wave per page of a tile
// As many blocks while there are tiles (one per CU: few tiles each, listed tiles are revisited in parallel), or twice,
// three times as many, so that a block has no more tiles than threads.
constexpr uint32_t kEmitBlocks = 256;

__global__ __launch_bounds__(kEmitThreads) void k_oob_emit(const Tile* tiles, uint32_t n_tiles, uint32_t run,
                                                           ScanDev sd, const uint64_t* tile_prefix, kc_oob* oob,
                                                           uint64_t cap, kc_scan_result* res, uint64_t n_words) {
  __shared__ uint4 listed[kEmitThreads];        // the tiles
  __shared__ uint64_t listed_at[kEmitThreads];  // entries before the listed tile's
  __shared__ uint32_t n_listed;
  __shared__ uint32_t wave_cnt[2][kTilePages];
  __shared__ unsigned long long sums[2][kTilePages];
  const uint32_t tid = threadIdx.x, lane = tid % kWave, wv = tid / kWave;
  const uint64_t first = (uint64_t)blockIdx.x * run, end = min(first + run, (uint64_t)n_tiles);
  static_assert(kScanSlots == kWave, "one slot per lane");
  const unsigned long long* c = sd.counts + (size_t)lane * kScanSlotStride;
  const unsigned long long c0 = c[0], c1 = c[1];
  uint32_t count = 0;  // of this thread's tile in the slice
  uint4 tile = make_uint4(0, 0, 0, 0);
  if (first + tid < end) {
    count = sd.tile_oob[first + tid];
    tile = ld16((uint64_t)(tiles + first + tid));
  }
  uint32_t n = 0;  // entries before the run, of one thread: at most 8192 words a tile, kInlineTiles / 1024 tiles
  const uint4* counts = reinterpret_cast<const uint4*>(sd.tile_oob);
  if (!tile_prefix) {  // the first round of them with the others
    if (tid < first / 4u) {
      const uint4 x = counts[tid];
      n = x.x + x.y + x.z + x.w;
    }
    if (tid < (first & 3u)) n += sd.tile_oob[first - 1u - tid];
  }
  const unsigned long long n_ptr = wave_sum_u64(c0), n_in = wave_sum_u64(c1);
  const uint64_t total = n_ptr - n_in;  // pointer-like words are in a range or not
  if (blockIdx.x == 0 && tid == 0) {    // the result struct, from the slot totals
    res->n_words = n_words;
    res->n_ptr_like = n_ptr;
    res->n_in_range = n_in;
    res->n_oob = total;
    res->n_written = (uint32_t)(total < cap ? total : cap);
    res->truncated = total > cap ? 1u : 0u;
  }
  if (total == 0 || cap == 0) return;  // nothing to list: no tile to revisit
  if (!__syncthreads_or(count != 0u)) return;  // none in this run
  const uint64_t below = (1ull << lane) - 1ull;
  load_wide_fences(sd.rt, tid, kEmitThreads);  // the first barrier below makes it whole
  if (tid == 0) n_listed = 0u;
  uint64_t at = 0;  // entries before this thread's tile
  if (tile_prefix) {
    at = first + tid < end ? tile_prefix[first + tid] : 0ull;
    __syncthreads();
  } else {  // those before the run, and those before this tile in it
    for (uint64_t i = tid + kEmitThreads; i < first / 4u; i += kEmitThreads) {
      const uint4 x = counts[i];
      n += x.x + x.y + x.z + x.w;
    }
    const unsigned long long w = wave_sum_u64(n);
    uint32_t inc = count;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(inc, d, 64);
      if (lane >= (uint32_t)d) inc += y;
    }
    if (lane == kWave - 1u) {
      sums[0][wv] = inc;
      sums[1][wv] = w;
    }
    __syncthreads();
    at = inc - count;
#pragma unroll
    for (uint32_t i = 0; i < kTilePages; ++i) at += sums[1][i] + (i < wv ? sums[0][i] : 0ull);
  }
  if (count != 0u && at < cap) {
    const uint32_t i = atomicAdd(&n_listed, 1u);
    listed[i] = tile;
    listed_at[i] = at;
  }
  __syncthreads();
  const uint32_t n_list = n_listed;  // the same in every thread
  uint4 next[4];
  auto load = [&](uint32_t i) {
    const Tile it = i < n_list ? __builtin_bit_cast(Tile, listed[i]) : Tile{0, 0, 0, 0};
    const bool mine = wv < it.npages;
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j)
      next[j] = mine ? ld16(it.va + (uint64_t)(wv * 4u + j) * 1024u + lane * 16u) : make_uint4(0, 0, 0, 0);
  };
  load(0);
  for (uint32_t i = 0; i < n_list; ++i) {
    const Tile it = __builtin_bit_cast(Tile, listed[i]);
    uint4 x[4];
    uint64_t b0[4], b1[4];
    uint32_t cnt = 0;
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j)  // zero words (and pages past the tile) are never pointer-like
      x[j] = seg_words(it, wv * 4u + j, lane, next[j]);  // same words as the counting pass
    load(i + 1u);
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {
      const uint64_t w0 = ((uint64_t)x[j].y << 32) | x[j].x;
      const uint64_t w1 = ((uint64_t)x[j].w << 32) | x[j].z;
      b0[j] = __ballot((w0 - sd.lo) < sd.span && wide_range_index(w0, sd.rt) < 0);
      b1[j] = __ballot((w1 - sd.lo) < sd.span && wide_range_index(w1, sd.rt) < 0);
      cnt += (uint32_t)(__popcll(b0[j]) + __popcll(b1[j]));
    }
    if (lane == 0) wave_cnt[i & 1u][wv] = cnt;
    __syncthreads();  // the one barrier per tile: the counts of two tiles apart share a row
    uint64_t done = listed_at[i];
    for (uint32_t w = 0; w < wv; ++w) done += wave_cnt[i & 1u][w];
#pragma unroll
    for (uint32_t j = 0; j < 4; ++j) {  // segments in order, lanes in order, word 0 before word 1
      const uint64_t a = it.va + (uint64_t)(wv * 4u + j) * 1024u + lane * 16u;
      const bool o0 = ((b0[j] >> lane) & 1ull) != 0ull, o1 = ((b1[j] >> lane) & 1ull) != 0ull;
      const uint64_t r0 = done + (uint64_t)__popcll(b0[j] & below) + (uint64_t)__popcll(b1[j] & below);
      const uint64_t r1 = r0 + (o0 ? 1u : 0u);
      if (o0 && r0 < cap) {
        oob[r0].word_va = a;
        oob[r0].value = ((uint64_t)x[j].y << 32) | x[j].x;
      }
      if (o1 && r1 < cap) {
        oob[r1].word_va = a + 8u;
        oob[r1].value = ((uint64_t)x[j].w << 32) | x[j].z;
      }
      done += (uint64_t)__popcll(b0[j]) + (uint64_t)__popcll(b1[j]);
    }
  }
}

inline uint32_t blocks_for(uint64_t n, uint32_t per) { return (uint32_t)((n + per - 1) / per); }

}  // namespace

// ------------------------------------------------------------- launchers --
hipError_t launch_zero4(uint64_t* a, uint64_t na, uint64_t* b, uint64_t nb, uint64_t* c, uint64_t nc, uint64_t* d,
                        uint64_t nd, hipStream_t s) {
  const uint64_t n = na + nb + nc + nd;
  if (n == 0) return hipSuccess;
  const uint64_t nbk = blocks_for(n, 256);
  hipLaunchKernelGGL(k_zero4, dim3((uint32_t)(nbk < 4096 ? nbk : 4096)), dim3(256), 0, s, a, na, b, nb, c, nc, d, nd);
  return hipGetLastError();
}

hipError_t launch_fill_u64(uint64_t* p, uint64_t n, uint64_t v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const uint64_t nb = blocks_for(n, 256);
  const uint32_t grid = (uint32_t)(nb < 4096 ? nb : 4096);
  hipLaunchKernelGGL(k_fill_u64, dim3(grid), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

hipError_t launch_probe_zero(ProbeParams p, uint64_t n_words, uint32_t n_cu, hipStream_t s) {
  // Groups of 64 pages, or of 16 larger units (more groups: few units can be many bytes).
  p.gshift = p.ushift == kMinUnitShift ? 6u : 4u;
  p.n_groups = n_words << (6u - p.gshift);
  if (p.n_groups == 0 && p.n_clear_a + p.n_clear_b == 0) return hipSuccess;
  // Waves per group: so many that the chip has 16 per CU and that no wave has more than 256 KiB of zeros to read.
  const uint64_t fill = 16ull * n_cu / std::max<uint64_t>(1, p.n_groups), zeros = 1ull << (p.gshift + p.ushift);
  uint32_t wpb = 1;
  while (wpb < kProbeWaves && (wpb < fill || (uint64_t)wpb << 18 < zeros)) wpb *= 2u;
  const uint32_t grid = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(p.n_groups, 1u << 21));
  if (p.ushift == kMinUnitShift) hipLaunchKernelGGL(k_probe_zero<true>, dim3(grid), dim3(wpb * kWave), 0, s, p);
  else hipLaunchKernelGGL(k_probe_zero<false>, dim3(grid), dim3(wpb * kWave), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_scan(const ScanSrc& src, uint64_t* out, uint64_t* block_sums, uint64_t* total_out,
                       hipStream_t s) {
  const uint32_t nb = blocks_for(src.n_items, kScanBlock);
  if (nb <= 1) {
    hipLaunchKernelGGL(k_scan_small, dim3(1), dim3(kScanThreads), 0, s, src, out, total_out);
    return hipGetLastError();
  }
  if (nb > 0) {
    hipLaunchKernelGGL(k_scan_reduce, dim3(nb), dim3(kScanThreads), 0, s, src, block_sums);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(1024), 0, s, block_sums, nb, total_out);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || nb == 0) return e;
  hipLaunchKernelGGL(k_scan_down, dim3(nb), dim3(kScanThreads), 0, s, src, (const uint64_t*)block_sums, out);
  return hipGetLastError();
}

hipError_t launch_gather(const Tile* tiles, uint32_t n_tiles, uint32_t per_tile, const uint64_t* zero_bm,
                         const uint64_t* changed_bm, const uint64_t* word_prefix, uint8_t* packed,
                         uint64_t* page_va, uint64_t cap_pages, uint32_t ushift, uint32_t grid, hipStream_t s) {
  if (n_tiles == 0) return hipSuccess;
  const uint64_t tile = (uint64_t)per_tile << ushift;
  const uint32_t part = (ushift > kMinUnitShift && n_tiles * tile > kGatherLong ? kWave : 16u) * kPage;
  uint32_t part_shift = 0;  // 1 << part_shift parts per tile
  while (((uint64_t)part << part_shift) < tile) ++part_shift;
  const uint64_t n_items = (uint64_t)n_tiles << part_shift;
  const uint32_t blocks = (uint32_t)std::min<uint64_t>(grid == 0u ? n_items : std::min<uint64_t>(grid, n_items), 1u << 25);
  hipLaunchKernelGGL(k_gather, dim3(blocks), dim3(64), 0, s, tiles, n_tiles, part, part_shift, zero_bm, changed_bm,
                     word_prefix, packed, page_va, cap_pages, ushift);
  return hipGetLastError();
}

hipError_t launch_restore_zero(const Tile* tiles, uint32_t n_tiles, const uint64_t* zero_bm,
                               const uint64_t* changed_bm, unsigned long long* n_bad, uint32_t ushift, uint32_t grid,
                               hipStream_t s) {
  grid = std::max(1u, std::min(grid, std::max(1u, n_tiles)));
  hipLaunchKernelGGL(k_restore_zero, dim3(grid), dim3(64), 0, s, tiles, n_tiles, zero_bm, changed_bm, n_bad,
                     ushift);
  return hipGetLastError();
}

template <uint32_t WAVES>
void launch_scatter_waves(const RangeTable& rt, const uint8_t* packed, const uint64_t* page_va,
                          const uint64_t* n_kept, uint64_t cap_pages, unsigned long long* n_bad, uint32_t ushift,
                          hipStream_t s) {
  // WAVES blocks per workgroup over every 4 KiB block of the capacity (blocks past the kept count exit at once);
  // the kernel strides only if a capacity ever exceeded the grid limit
  const uint32_t bshift = ushift - 12u;
  const uint64_t kMaxGrid = 0x7FFFFFFFull;
  const uint64_t wgs = cap_pages > ((kMaxGrid * WAVES) >> bshift) ? kMaxGrid
                                                                   : ((cap_pages << bshift) + WAVES - 1) / WAVES;
  hipLaunchKernelGGL(k_restore_scatter<WAVES>, dim3((uint32_t)wgs), dim3(WAVES * kWave), 0, s, rt, packed, page_va,
                     n_kept, cap_pages, n_bad, ushift);
}

hipError_t launch_restore_scatter(const RangeTable& rt, const uint8_t* packed, const uint64_t* page_va,
                                  const uint64_t* n_kept, uint64_t cap_pages, unsigned long long* n_bad,
                                  bool delta, uint32_t ushift, hipStream_t s) {
  if (cap_pages == 0) return hipSuccess;
  if (delta)
    launch_scatter_waves<4>(rt, packed, page_va, n_kept, cap_pages, n_bad, ushift, s);
  else
    launch_scatter_waves<1>(rt, packed, page_va, n_kept, cap_pages, n_bad, ushift, s);
  return hipGetLastError();
}

hipError_t launch_closure(const Tile* tiles, uint32_t n_tiles, uint32_t tile0, const ScanDev& sd,
                          uint32_t grid, uint32_t n_cu, hipStream_t s) {
  if (n_tiles == 0) return hipSuccess;
  uint32_t blocks = 1, wpb = 1;
  wide_shape(std::min(grid, n_tiles), n_cu, &blocks, &wpb);  // grid counts waves
  hipLaunchKernelGGL(k_closure, dim3(blocks), dim3(wpb * kWave), wide_lds_bytes(sd.rt), s, tiles, n_tiles, tile0,
                     sd);
  return hipGetLastError();
}

hipError_t launch_oob_emit(const Tile* tiles, uint32_t n_tiles, const ScanDev& sd, const uint64_t* tile_prefix,
                           kc_oob* oob, uint64_t cap, kc_scan_result* res, uint64_t n_words, hipStream_t s) {
  static_assert(kInlineTiles <= kEmitBlocks * kEmitThreads, "a tile per thread");
  const uint32_t rounds = std::max(1u, blocks_for(n_tiles, kEmitBlocks * kEmitThreads));
  const uint32_t run = std::max(1u, blocks_for(n_tiles, kEmitBlocks * rounds));
  const uint32_t blocks = std::max(1u, blocks_for(n_tiles, run));
  hipLaunchKernelGGL(k_oob_emit, dim3(blocks), dim3(kEmitThreads), wide_lds_bytes(sd.rt), s, tiles, n_tiles, run, sd, tile_prefix, oob,
                     cap, res, n_words);
  return hipGetLastError();
}

}  // namespace kc
